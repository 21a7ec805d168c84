"""The weight-streaming forward (calls of few rows) against the oracle and,
bit for bit, against the tiled kernels: group sizes at the edges of its row
classes (16, 32, 64, 128 and 256 rows) and of its pieces (256 rows, 64 where
few), one k-stage per unit, column counts that leave a workgroup's last column
units empty, more units than workgroups, and the most experts and devices; and
the rule that chooses between the two."""

from fractions import Fraction

import numpy as np
import pytest

import oracle
from gpu_util import LayerRun, device, mark_workspace, ran_tiles, rel_err

pytestmark = pytest.mark.gpu

TOL_BF16 = 2e-2
EDGES = (1, 0, 15, 16, 17, 31, 32, 33, 63, 64, 65, 0, 127, 128, 129, 255, 256, 257, 300, 512, 529)


@pytest.fixture(scope="module")
def dev():
    return device()


def _cfg(loads, D, F, P=1):
    from paper_2601_17111_amd.synth import LayerConfig
    return LayerConfig(f"stream-D{D}-F{F}", T=sum(loads), D=D, F=F, E=len(loads), K=1, P=P,
                       alpha=Fraction(2), dtype="bf16", routing=("loads", tuple(loads)))


@pytest.mark.parametrize("loads,D,F", [
    (EDGES, 64, 64),       # one stage per unit, one column unit of four per piece
    (EDGES, 320, 192),     # 10 output units: the last workgroup unit half empty
    (EDGES, 1024, 576),
    # 34 output units: pieces of more than 64 rows (the units of smaller ones
    # would be (24 + 44) * 9 > the workgroups), the last unit half empty
    (EDGES, 1088, 576),
    # 180 and 90 units, pieces of more than 64 rows in both projections
    ((200, 70, 40, 20, 17, 5, 4, 3, 2, 2, 1, 1, 1, 1, 1, 1), 2880, 2880),
    ((3,), 128, 64),       # fewer units than workgroups
    ((1,) * 63 + (200,), 192, 640),
], ids=["64x64", "320x192", "1024x576", "1088x576", "2880x2880", "one-group", "one-hot"])
def test_stream_forward(dev, loads, D, F):
    import torch
    cfg = _cfg(loads, D, F)
    run = LayerRun(cfg, 1, dev)
    L = run.layer
    L.out_perm.fill_(float("nan"))
    mark_workspace(L)
    run.forward(-1)
    assert not ran_tiles(L)
    n = cfg.T
    out = L.out_perm[:n].clone()
    groups = L.bufs.groups[:L.bufs.info_dict()["n_groups"]].cpu().tolist()
    row_pair = L.row_pair[:n].cpu().numpy()
    W = run.host_weights(range(cfg.E))
    got = out.float().cpu().numpy()
    for (_, e, r0, rows) in groups:
        want = oracle.swiglu_ffn(run.inp.x[row_pair[r0:r0 + rows]].astype(np.float64),
                                 *(w.astype(np.float64) for w in W[e]))
        for i in range(rows):
            assert rel_err(got[r0 + i], want[i]) <= TOL_BF16, (e, rows, i)
    # the training forward, and the call again: the same bits; g and u are kept
    L.ffn(run.gu, run.dn, -1, save_gate_up=True)
    torch.cuda.synchronize()
    assert torch.equal(L.out_perm[:n], out)
    gu = L.gate_up[:n].clone()
    # the same rows in a call too large for the stream (an expert of 8200 rows
    # more): gemm.h's tiles give the same bits, g and u included
    big = LayerRun(_cfg(tuple(loads) + (8200,), D, F), 1, dev, weights=False)
    big.gu = torch.zeros((cfg.E + 1, 2 * F, D), dtype=torch.bfloat16, device=dev)
    big.dn = torch.zeros((cfg.E + 1, D, F), dtype=torch.bfloat16, device=dev)
    big.gu[:-1], big.dn[:-1] = run.gu, run.dn
    b = big.layer
    b.plan(big.ids)
    b.permute(big.ids, big.gates, big.x)
    b.x_perm[:n] = L.x_perm[:n]  # experts keep their rows' places
    mark_workspace(b)
    b.ffn(big.gu, big.dn, -1, save_gate_up=True)
    torch.cuda.synchronize()
    assert ran_tiles(b)
    assert torch.equal(b.out_perm[:n], out)
    assert torch.equal(b.gate_up[:n], gu)


@pytest.mark.parametrize("loads,P", [
    ((300, 2, 1, 40, 17, 0, 90, 5), 4),
    ((487,) + (1, 0, 2) * 5, 8),            # one expert on every device: pieces of many groups
    ((700, 3, 650, 1, 2, 0, 0, 40), 8),     # two of them, over several pieces
    ((16, 16, 16, 16), 2),
], ids=["spill", "hot", "two-hot", "even"])
def test_stream_one_device_and_plans(dev, loads, P):
    """One device's launch writes its rows alone, with the bits of the
    all-device launch; the LLEP and EP plans give the same bits per token."""
    import torch
    cfg = _cfg(loads, 256, 384, P=P).with_(alpha=Fraction(1))
    run = LayerRun(cfg, 2, dev)
    L = run.layer
    y = run.forward(-1).clone()
    out = L.out_perm.clone()
    rows = L.bufs.device_rows.cpu().tolist()
    at = 0
    for d in range(cfg.P):
        L.out_perm.fill_(float("nan"))
        L.ffn(run.gu, run.dn, d)
        torch.cuda.synchronize()
        assert torch.equal(L.out_perm[at:at + rows[d]], out[at:at + rows[d]])
        assert torch.isnan(L.out_perm[:at].float()).all()
        assert torch.isnan(L.out_perm[at + rows[d]:].float()).all()
        at += rows[d]
    L.set_mode("ep")
    assert torch.equal(run.forward(-1), y)


@pytest.mark.parametrize("loads", [
    # most experts with a few rows, some of every class, two spread over devices
    tuple(0 if e % 7 == 3 else 1 + e % 5 + 30 * (e % 61 == 8) + 1300 * (e == 77) + 330 * (e == 509)
          for e in range(512)),
    tuple(8 for _ in range(512)),
], ids=["spread", "even"])
def test_stream_most_experts_and_devices(dev, loads):
    """512 experts on 64 devices: the same bits as the tiles, which run when
    another 4200 pairs of the last expert follow."""
    import torch
    from paper_2601_17111_amd import binding as B
    from paper_2601_17111_amd.layer import LLEPLayer
    D, F, P, n = 192, 256, 64, sum(loads)
    cfg = _cfg(loads, D, F, P=P).with_(alpha=Fraction(1))
    assert n <= 4096
    run = LayerRun(cfg, 4, dev)
    L = run.layer
    mark_workspace(L)
    run.forward(-1)
    assert not ran_tiles(L)
    rows = L.pair_row.reshape(-1).long()
    out = L.out_perm[rows]
    T = n + 4200
    ids = torch.full((T, 1), 511, dtype=torch.int32, device=dev)
    ids[:n] = run.ids
    x = torch.zeros((T, D), dtype=torch.bfloat16, device=dev)
    x[:n] = run.x
    big = LLEPLayer(T, 1, cfg.E, P, D, F, T // P + 1, torch.bfloat16, dev)
    mark_workspace(big)
    big.forward(ids, torch.ones((T, 1), device=dev), x, run.gu, run.dn)
    torch.cuda.synchronize()
    assert ran_tiles(big)
    assert not big.bufs.info_dict()["status"] & B.LLEP_STATUS_FFN_WAIT
    assert torch.equal(big.out_perm[big.pair_row[:n].reshape(-1).long()], out)
    # one device at a time, and a sample against the oracle
    full = L.out_perm.clone()
    L.out_perm.fill_(float("nan"))
    for d in range(P):
        L.ffn(run.gu, run.dn, d)
    torch.cuda.synchronize()
    assert torch.equal(L.out_perm, full)
    sample = np.linspace(0, n - 1, 40).astype(int)
    W = run.host_weights(set(run.inp.ids[sample, 0].tolist()))
    got = out.float().cpu().numpy()
    for p in sample:
        w = (m.astype(np.float64) for m in W[int(run.inp.ids[p, 0])])
        want = oracle.swiglu_ffn(run.inp.x[p:p + 1].astype(np.float64), *w)[0]
        assert rel_err(got[p], want) <= TOL_BF16, p


@pytest.mark.parametrize("T,E,P,D,F,tiles", [
    (1024, 64, 8, 2560, 2048, (0, 0, 0)),  # 24 rows per expert: up to 1024 rows
    (1025, 64, 8, 2560, 2048, (1, 0, 0)),
    (1536, 64, 1, 2560, 2048, (1, 1, 1)),  # the only device: as all of them
    (2441, 64, 8, 2560, 768, (0, 0, 0)),   # more rows: D F R up to 5 10^9
    (2560, 64, 8, 2560, 768, (1, 1, 1)),
    (2029, 72, 8, 2560, 768, (0, 0, 0)),   # 4 10^9 with more than 64 experts
    (2048, 72, 8, 2560, 768, (1, 0, 0)),
    (4096, 172, 4, 2560, 1920, (1, 0, 1)),  # one device's rows: 2 10^10
], ids=lambda v: str(v) if isinstance(v, int) else "")
def test_dispatch(dev, T, E, P, D, F, tiles):
    """Both sides of every line of the rule that chooses between the stream and
    the tiles, for all devices at once, one device of an LLEP and one of a
    standard plan (tiles); whatever ran, the same bits."""
    import torch
    from paper_2601_17111_amd.synth import LayerConfig
    cfg = LayerConfig(f"route-T{T}-E{E}", T=T, D=D, F=F, E=E, K=1, P=P, alpha=Fraction(11, 10),
                      dtype="bf16", routing=("hot", 0.8, 1))
    run = LayerRun(cfg, 3, dev)
    L = run.layer
    out = {}
    for mode, device_tiles in (("llep", tiles[1]), ("ep", tiles[2])):
        L.set_mode(mode)
        mark_workspace(L)
        run.forward(-1)
        assert ran_tiles(L) == tiles[0], mode
        out[mode] = L.out_perm[L.pair_row.reshape(-1).long()].clone()
        full = L.out_perm.clone()
        d = L.bufs.info_dict()["max_device"]
        at = int(L.bufs.device_rows[:d].sum())
        n = int(L.bufs.device_rows[d])
        L.out_perm.fill_(float("nan"))
        mark_workspace(L)
        L.ffn(run.gu, run.dn, d)
        torch.cuda.synchronize()
        assert ran_tiles(L) == device_tiles, mode
        assert torch.equal(L.out_perm[at:at + n], full[at:at + n])
    assert torch.equal(out["llep"], out["ep"])
