"""Plan and permutation of small calls (one launch each, up to 4096 pairs; the
permutation of rows of less than 4 KB up to 3072): at the edges of their slices
(256 pairs), tiles (1024) and ranges, for few and many experts, rows of less
than one 1 KB piece, of several, and of more than the 16 that are in flight at
once, one to four tokens per workgroup, and invalid ids; bit-exact against the
oracle."""

import math

import numpy as np
import pytest

import oracle
from gpu_util import assert_plan_equal, device, run_plan

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    return device()


@pytest.mark.parametrize("T,K,E,P,D,dtype", [
    (1, 1, 1, 1, 8, "bf16"), (1, 4, 32, 8, 2880, "bf16"), (1, 3, 4, 2, 72, "f32"),
    (5, 1, 16, 4, 520, "bf16"), (63, 4, 128, 8, 64, "bf16"), (64, 4, 128, 8, 64, "bf16"),
    (257, 1, 256, 8, 136, "bf16"), (51, 5, 255, 5, 4104, "bf16"), (341, 3, 12, 4, 72, "f32"),
    (128, 8, 512, 64, 72, "bf16"), (205, 5, 257, 1, 72, "bf16"), (819, 5, 64, 8, 264, "bf16"),
    (512, 8, 512, 8, 72, "bf16"), (4096, 1, 256, 64, 8, "f32"), (4097, 1, 256, 64, 8, "f32"),
    (60, 67, 32, 4, 72, "bf16"), (3072, 1, 32, 4, 72, "bf16"), (3073, 1, 32, 4, 72, "bf16"),
    (4096, 1, 16, 4, 2048, "bf16"), (4097, 1, 16, 4, 2048, "bf16"), (9, 1, 8, 4, 8192, "bf16"),
    (9, 2, 8, 4, 8200, "bf16"), (7, 3, 8, 4, 8200, "f32"), (33, 4, 8, 4, 7168, "bf16"),
])
@pytest.mark.parametrize("mode", ["llep", "ep"])
def test_small_plan_and_permutation(dev, T, K, E, P, D, dtype, mode):
    import torch
    from paper_2601_17111_amd import binding as B
    rng = np.random.default_rng(T * K + E)
    ids = np.where(rng.random((T, K)) < 0.5, 0, rng.integers(0, E, (T, K))).astype(np.int32)
    if T > 50:
        ids[T // 2, 0], ids[T - 1, K - 1] = E, -1
    cap = math.ceil(T * K / P)
    got, info, (params, bufs, ids_t) = run_plan(ids, E, P, cap, mode=mode, dev=dev)
    ref = oracle.plan(ids.reshape(-1).tolist(), E, P, cap, mode=mode)
    assert_plan_equal(got, info, ref)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    x = torch.randn((T, D), device=dev).to(tdt)
    gates = torch.rand((T, K), device=dev)
    R = T * K
    x_perm = torch.zeros((R, D), dtype=tdt, device=dev)
    gate_perm = torch.zeros(R, device=dev)
    row_pair = torch.full((R,), -7, dtype=torch.int32, device=dev)
    pair_row = torch.full((R,), -7, dtype=torch.int32, device=dev)
    B.llep_permute(params, bufs, ids_t, gates, x, x_perm, gate_perm, row_pair, pair_row)
    torch.cuda.synchronize()
    pr_ref, rp_ref = oracle.permute(ids.reshape(-1).tolist(), ref, E)
    n = info["total_rows"]
    assert np.array_equal(pair_row.cpu().numpy(), pr_ref)
    assert np.array_equal(row_pair[:n].cpu().numpy(), rp_ref)
    rp = torch.from_numpy(np.asarray(rp_ref).astype(np.int64))
    assert torch.equal(x_perm[:n].cpu(), x.cpu()[rp // K])
    assert not x_perm[n:].any()
    assert torch.equal(gate_perm[:n].cpu(), gates.reshape(-1).cpu()[rp])
