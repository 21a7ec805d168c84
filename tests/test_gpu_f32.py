"""The float32 layer on the matrix cores, forward and backward, against the
float64 oracle to 1e-5: group sizes around its 64-row tiles and 32-row slices,
column counts with a half-filled last tile, an expert spread over several
devices, and experts without rows."""

from fractions import Fraction

import numpy as np
import pytest

import oracle
from gpu_util import device, rel_err
from test_gpu_backward import BwdRun

pytestmark = pytest.mark.gpu

TOL = 1e-5


@pytest.fixture(scope="module")
def dev():
    return device()


@pytest.mark.parametrize("loads,P,D,F", [
    ((1, 0, 31, 33), 1, 64, 64),
    ((63, 64, 65, 0, 1, 129, 32, 2), 2, 192, 128),
    ((400, 3, 1, 0, 5, 40, 17, 2), 4, 320, 192),   # the first expert on every device
    ((0, 0, 0, 7), 4, 512, 448),
], ids=["tiny", "edges", "spill", "one"])
def test_f32_layer(dev, loads, P, D, F):
    import torch
    from paper_2601_17111_amd.synth import LayerConfig
    cfg = LayerConfig("f32", T=sum(loads), D=D, F=F, E=len(loads), K=1, P=P, alpha=Fraction(1),
                      dtype="f32", routing=("loads", tuple(loads)))
    run = BwdRun(cfg, 3, dev)
    W = {e: tuple(w.astype(np.float64) for w in v)
         for e, v in run.host_weights(range(cfg.E)).items()}
    run.layer.forward(run.ids, run.gates, run.x, run.gu, run.dn, -1, save_gate_up=True)
    torch.cuda.synchronize()
    y = run.layer.y.cpu().numpy()
    assert rel_err(y, oracle.moe_output(run.inp.x, run.inp.ids, run.inp.gates, lambda e: W[e],
                                        list(range(cfg.T)))) <= TOL
    out = run.layer.out_perm.clone()
    run.layer.ffn(run.gu, run.dn, -1)
    assert torch.equal(run.layer.out_perm, out)  # the inference forward: the same bits
    dx, dgates, dwg, dwu, dwd = run.backward(-1)
    want_dx, want_dg, want_dW = oracle.moe_backward(run.x.cpu().numpy(), run.inp.ids,
                                                    run.inp.gates, lambda e: W[e],
                                                    run.dy.cpu().numpy(), cfg.E)
    assert rel_err(dx, want_dx) <= TOL
    assert rel_err(dgates, want_dg) <= TOL
    for e in range(cfg.E):
        if loads[e] == 0:
            assert not (dwg[e].any() or dwu[e].any() or dwd[e].any())
            continue
        for got, want in zip((dwg[e], dwu[e], dwd[e]), want_dW[e]):
            assert rel_err(got, want) <= TOL, e
