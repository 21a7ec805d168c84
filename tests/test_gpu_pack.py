"""The weight packing kernels move 8 KB units (64 columns x 64 bf16 or 32 f32
rows) of all three matrices in one launch: every element, at sizes of one unit
per matrix, of unequal sides, and of a unit count that leaves the last
workgroup partly filled; and, for the backward packing, sources that do not
start on 16-byte boundaries."""

import pytest

from gpu_util import device

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    return device()


def _blocks(p):
    """[E, n, k] in blocks of 16 n x 32 k."""
    E, n, k = p.shape
    return p.reshape(E, n // 16, 16, k // 32, 32).transpose(2, 3).reshape(E, -1)


@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("E,D,F", [(1, 64, 64), (3, 64, 192), (2, 320, 64), (5, 192, 448)])
def test_pack_every_element(dev, E, D, F, dtype, offset):
    import torch
    from paper_2601_17111_amd import binding as B
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    n = E * D * F

    def weights(*shape):
        # distinct bit patterns; `offset` elements off the allocation's alignment
        flat = torch.empty(n + offset, dtype=tdt, device=dev)
        flat[offset:] = torch.randn(n, device=dev).to(tdt)
        return flat[offset:].view(*shape)

    wg, wu, wd = weights(E, D, F), weights(E, D, F), weights(E, F, D)
    both = torch.stack([wg.reshape(E, D, -1, 32), wu.reshape(E, D, -1, 32)], 3).reshape(E, D, 2 * F)
    gut, dnt = B.llep_pack_weights_backward(wg, wu, wd)
    torch.cuda.synchronize()
    assert torch.equal(gut.reshape(E, -1), _blocks(both))
    assert torch.equal(dnt.reshape(E, -1), _blocks(wd))
    if offset:
        with pytest.raises(B.LLEPError):
            B.llep_pack_weights(wg, wu, wd)
        return
    gu, dn = B.llep_pack_weights(wg, wu, wd)
    torch.cuda.synchronize()
    assert torch.equal(gu.reshape(E, -1), _blocks(both.transpose(1, 2)))
    assert torch.equal(dn.reshape(E, -1), _blocks(wd.transpose(1, 2)))
