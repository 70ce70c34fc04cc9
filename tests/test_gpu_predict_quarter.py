"""The predictor at few token tiles and d no multiple of 128 runs by quarters of a tile: the mask bytes of the same tokens
inside a call of more tiles, which does not."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lx():
    import torch
    assert torch.cuda.is_available()
    from paper_2510_15964_amd import lx
    return lx


# token tiles, d, blocks
CASES = [
    (1, 64, 64),          # one step
    (1, 192, 128),        # a pair and a half
    (3, 1088, 320),       # 15 tiles: the ring of eight pairs and one step more
    (64, 448, 64),        # the most of the long ring
    (13, 576, 320),       # 65: the first of the short one
    (128, 320, 64),       # the most
]


def tiles_beyond(Tt, nblk):
    """Token tiles of a call that does not run by quarters."""
    return max(Tt, -(-129 * 64 // nblk))


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("Tt,d,nblk", CASES)
def test_mask_bytes_of_the_quarters(lx, Tt, d, nblk, dtype):
    import torch
    tdt = {"bf16": torch.bfloat16, "f16": torch.float16}[dtype]
    g = torch.Generator(device="cuda").manual_seed(d)
    X = torch.randn(64 * tiles_beyond(Tt, nblk), d, device="cuda", generator=g).to(tdt)
    W = torch.randn(nblk, d, device="cuda", generator=g).to(tdt)
    thr = 2.5 * d ** 0.5                             # a third of the blocks of a tile
    few = torch.full((Tt, nblk), 7, dtype=torch.uint8, device="cuda")
    lx.lx_mlp_predict_mask(X[:64 * Tt], W, thr, 64, mask=few)
    big = torch.cat([X, X])                          # more than 128 tiles of 64 x 64 in any case
    both = torch.full((big.shape[0] // 64, nblk), 7, dtype=torch.uint8, device="cuda")
    lx.lx_mlp_predict_mask(big, W, thr, 64, mask=both)
    torch.cuda.synchronize()
    assert torch.equal(few, both[:Tt]) and 0 < int(few.sum()) < few.numel()
    one = torch.full((1, nblk), 7, dtype=torch.uint8, device="cuda")
    lx.lx_mlp_predict_mask(X[:64 * Tt], W, thr, 64 * Tt, mask=one)
    torch.cuda.synchronize()
    assert torch.equal(one[0], few.amax(0))
