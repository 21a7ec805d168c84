"""Weight gradients from row-major operands: group sizes around the 32-row
slices and the four slices in flight, experts whose rows lie in several groups
(one slice never spans two), tiles of 256 x 192 with partial rows and columns,
and infinities in a group's neighbours, which must not reach its gradients."""

from fractions import Fraction

import numpy as np
import pytest

import oracle
from gpu_util import device, rel_err
from test_gpu_backward import BwdRun

pytestmark = pytest.mark.gpu

TOL_BF16 = 2e-2
SIZES = (1, 0, 15, 16, 17, 31, 32, 33, 63, 64, 65, 95, 96, 97, 127, 128, 129, 160, 161, 193, 300)


@pytest.fixture(scope="module")
def dev():
    return device()


@pytest.mark.parametrize("loads,P,D,F", [
    (SIZES, 1, 64, 64),
    (SIZES, 3, 320, 192),
    ((900, 3, 0, 1, 40, 5, 17, 2), 8, 256, 448),  # the first expert on every device
    ((1, 1, 1, 1), 2, 512, 128),
    # the most experts and devices: more groups than experts, two per table thread
    (tuple(0 if e % 7 == 3 else 1 + e * e % 41 + 300 * (e % 97 == 5) for e in range(512)), 64, 64, 64),
], ids=["64x64", "320x192", "spill", "ones", "512 experts"])
def test_weight_gradients(dev, loads, P, D, F):
    import torch
    from paper_2601_17111_amd.synth import LayerConfig
    cfg = LayerConfig("wgrad", T=sum(loads), D=D, F=F, E=len(loads), K=1, P=P, alpha=Fraction(1),
                      dtype="bf16", routing=("loads", tuple(loads)))
    run = BwdRun(cfg, 1, dev)
    dx, dgates, *dw = run.backward(-1, save=True)
    W = run.host_weights(range(cfg.E))
    want_dx, _, want_dW = oracle.moe_backward(run.x.float().cpu().numpy(), run.inp.ids,
                                              run.inp.gates, lambda e: W[e],
                                              run.dy.float().cpu().numpy(), cfg.E)
    assert rel_err(dx, want_dx) <= TOL_BF16
    for e in range(cfg.E):
        if loads[e] == 0:
            assert not any(w[e].any() for w in dw)
            continue
        for got, want in zip((w[e] for w in dw), want_dW[e]):
            assert rel_err(got, want) <= TOL_BF16, (e, loads[e])
    # the same call again: the same bits
    for a, b in zip(dw, run.backward(-1, save=True)[2:]):
        assert np.array_equal(a, b)
    # rows of one expert become infinite: no other expert's gradient changes,
    # though their slices read across the ends of their groups
    bad = int(np.argmax(loads))
    run.x[torch.from_numpy((run.inp.ids[:, 0] == bad).copy()).to(dev)] = float("inf")
    run.dy[torch.from_numpy((run.inp.ids[:, 0] == bad).copy()).to(dev)] = float("inf")
    again = run.backward(-1, save=True)[2:]
    for e in range(cfg.E):
        if e != bad:
            for a, b in zip(dw, again):
                assert np.array_equal(a[e], b[e]), e


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_groups_without_rows(dev, dtype):
    """A group table that a program has written itself may hold groups of no
    rows: of an expert that has none, and beside an expert's other groups, on
    its native device and on others. The same gradients, bit for bit."""
    import torch
    from paper_2601_17111_amd import binding as B
    from paper_2601_17111_amd.synth import LayerConfig
    loads, P, D, F = (260, 0, 40, 17, 0, 90, 5, 0), 4, 128, 192
    cfg = LayerConfig("empty-groups", T=sum(loads), D=D, F=F, E=len(loads), K=1, P=P,
                      alpha=Fraction(1), dtype=dtype, routing=("loads", tuple(loads)))
    run = BwdRun(cfg, 1, dev)
    want = run.backward(-1, save=True)
    L = run.layer
    n = L.bufs.info_dict()["n_groups"]
    groups = L.bufs.groups[:n].cpu().tolist()
    have = {(d, e) for d, e, _, _ in groups}
    begin = L.bufs.device_rows.cpu().tolist()
    more = [g for g in ([d, e, sum(begin[:d]), 0] for d in range(P) for e in range(cfg.E))
            if (g[0], g[1]) not in have]
    more = more[::2] + more[1::2]  # some of every device first
    more = more[:2 * cfg.E + P - n]
    assert any(loads[e] > 0 for _, e, _, _ in more) and any(loads[e] == 0 for _, e, _, _ in more)
    table = sorted(groups + more, key=lambda g: g[:2])
    L.bufs.groups[:len(table)] = torch.tensor(table, dtype=torch.int32, device=dev)
    L.bufs.group_begin[:] = torch.tensor([sum(g[0] < d for g in table) for d in range(P + 1)],
                                         dtype=torch.int32, device=dev)
    for w in (L.dw_gate, L.dw_up, L.dw_down, L.dx_perm):
        w.fill_(float("nan"))
    L.ffn(run.gu, run.dn, -1, save_gate_up=True)
    L.combine(run.gates)
    got = L.backward(run.dy, run.gates, run.gu, run.gut, run.dnt, -1)
    torch.cuda.synchronize()
    assert not L.bufs.info_dict()["status"] & B.LLEP_STATUS_FFN_WAIT
    for a, b in zip(want, got):
        assert np.array_equal(a, b.float().cpu().numpy())
