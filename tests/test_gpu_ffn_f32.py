"""The fp32 FFN kernels where their loops can go wrong: fewer steps than stages, contractions and lists that two halves
cut unevenly, more list rows than lanes, shared rows, capacities below the list; the order of the up-projection's sum."""
import numpy as np
import pytest

from paper_2510_15964_amd import inputs
from test_gpu_ffn import compare
from util import TOL, dev, host, rel_err_max

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lx():
    import torch
    assert torch.cuda.is_available()
    from paper_2510_15964_amd import lx
    return lx


@pytest.mark.parametrize("tile", [32, 64])
@pytest.mark.parametrize("d", [32, 96, 128, 160, 288])
def test_steps_around_the_ring(lx, oracle, tile, d):
    """1 to 9 steps of the first product; list rows of 0 to 9 entries, one of them empty, in the second."""
    c = inputs.ffn_bernoulli(12 * tile, d, 9 * tile, tile, tile, 0.5, 100 + d, dtype="f32", w_std=0.1)
    for i in range(12):
        c["mask"][i, :] = 0
        c["mask"][i, :i % 10] = 1
    compare(lx, oracle, c)


@pytest.mark.parametrize("rows", [65, 130])
def test_more_list_rows_than_lanes(lx, oracle, rows):
    c = inputs.ffn_bernoulli(32 * rows, 64, 224, 32, 32, 0.3, rows, dtype="f32", w_std=0.1)
    c["mask"][1:4, :] = 0
    c["mask"][rows - 1, :] = 0
    compare(lx, oracle, c)


@pytest.mark.parametrize("tile,rows,cap", [(32, 1, 7), (32, 2, 11), (64, 2, 5), (32, 8, 1), (32, 4, 0)])
def test_shared_rows_and_short_capacity(lx, oracle, tile, rows, cap):
    """Rows shared by several tiles, and fewer places than entries: the bits of the truncated mask."""
    import torch
    T, d, F = 8 * tile, 96, 12 * tile
    rng = np.random.default_rng(cap)
    m = (rng.random((rows, 12)) < 0.6).astype(np.uint8)
    kept = m.copy().reshape(-1)
    kept[np.flatnonzero(kept)[cap:]] = 0
    kept = kept.reshape(m.shape)
    c = inputs.ffn_bernoulli(T, d, F, tile, tile, 0.5, 7, dtype="f32", w_std=0.1)
    X, Wu, Wd = (dev(c[k], "f32") for k in ("X", "W_up", "W_down"))
    out = []
    for mask, n in ((m, cap), (kept, 12 * rows)):
        full = lx.lx_mask_compact(torch.from_numpy(mask).cuda())
        bl = lx.BlockList(rows, 12, full.row_ptr, full.col_idx, n)
        gt = 8 // rows
        H = torch.zeros(max(n, 1) * gt * tile * tile, device="cuda")
        Y, dX = torch.full_like(X, float("nan")), torch.full_like(X, float("nan"))
        ws = torch.empty(lx.lx_sparse_ffn_bwd_workspace_bytes(lx.LX_F32, T, d, F, tile, tile, n * gt, 0) + 256, dtype=torch.uint8, device="cuda")
        lx.lx_sparse_ffn_fwd(X, Wu, Wd, bl, tile, tile, Y, H)
        lx.lx_sparse_ffn_bwd_dx(X, H, Wu, Wd, bl, tile, tile, dX, ws)
        out.append((host(Y), host(dX)))
    for a, b in zip(*out):
        assert np.array_equal(a, b)
    Y = oracle.ffn_fwd(c["X"], c["W_up"], c["W_down"], np.repeat(kept, 8 // rows, axis=0), tile, tile)[1]
    assert rel_err_max(out[0][0], Y) <= TOL["f32"] if cap else not out[0][0].any()


@pytest.mark.parametrize("tile", [32, 64])
def test_up_projection_adds_in_ascending_order(lx, tile):
    """H, to the last bit, from one fused multiply-add per term: the product is exact in 64 bits, and rounding the sum
    to 53 bits first moves no result of these seeds."""
    import torch
    T, d, F = 2 * tile, 416, 2 * tile
    rng = np.random.default_rng(5)
    X = rng.standard_normal((T, d)).astype(np.float32)
    W = (rng.standard_normal((F, d)) * 0.1).astype(np.float32)
    X[:, ::7] *= np.float32(1e-20)
    W[:, ::7] *= np.float32(1e-19)          # subnormal products
    want = np.zeros((T, F), np.float32)
    for k in range(d):
        want = (want.astype(np.float64) + X[:, k:k + 1].astype(np.float64) * W[:, k].astype(np.float64)).astype(np.float32)
    want = np.maximum(want, 0)
    bl = lx.lx_mask_compact(torch.ones((2, 2), dtype=torch.uint8, device="cuda"))
    H = torch.zeros(4 * tile * tile, device="cuda")
    Xd = dev(X, "f32")
    lx.lx_sparse_ffn_fwd(Xd, dev(W, "f32"), dev(np.zeros((d, F), np.float32), "f32"), bl, tile, tile, torch.empty_like(Xd), H)
    got = host(H).reshape(2, 2, tile, tile).transpose(0, 2, 1, 3).reshape(T, F)
    assert np.array_equal(got, want)


def test_row_strides_beyond_32_bit_offsets(lx):
    """d and F of 2^27: eight rows no longer lie within 4 GiB (64-bit addresses per lane).  Values at a few places."""
    import torch
    if torch.cuda.mem_get_info()[0] < 100 << 30:
        pytest.skip("needs 90 GB of device memory")
    n = 1 << 27
    at = torch.tensor([0, 31, n // 2 + 5, n - 1], device="cuda")
    g = torch.Generator(device="cuda").manual_seed(1)
    sets = (torch.randn((32, 4), device="cuda", generator=g) for _ in range(2))
    X, W = (torch.zeros((32, n), device="cuda").index_copy_(1, at, v) for v in sets)
    bl = lx.lx_mask_compact(torch.ones((1, 1), dtype=torch.uint8, device="cuda"))
    H, Y = torch.empty(1024, device="cuda"), torch.empty((32, n), device="cuda")
    lx.lx_sparse_ffn_fwd(X, W, torch.zeros((n, 32), device="cuda"), bl, 32, 32, Y, H)
    small = (X[:, at].double() @ W[:, at].double().t()).clamp(min=0)
    assert rel_err_max(host(H).reshape(32, 32), host(small)) <= TOL["f32"] and not Y.any()
    del W, Y
    # a list of one block, the last one, of n neurons
    bl = lx.BlockList(1, n // 32, torch.tensor([0, 1], dtype=torch.int32, device="cuda"),
                      torch.tensor([n // 32 - 1], dtype=torch.int32, device="cuda"), 1)
    Wd = torch.zeros((32, n), device="cuda")
    Wd[:, n - 32:] = torch.randn((32, 32), device="cuda", generator=g)
    Wu = torch.zeros((n, 32), device="cuda")
    Wu[n - 32:] = torch.randn((32, 32), device="cuda", generator=g)
    x, y = torch.randn((32, 32), device="cuda", generator=g), torch.empty((32, 32), device="cuda")
    lx.lx_sparse_ffn_fwd(x, Wu, Wd, bl, 32, 32, y, H)
    want = (x.double() @ Wu[n - 32:].double().t()).clamp(min=0) @ Wd[:, n - 32:].double().t()
    assert rel_err_max(host(y), host(want)) <= TOL["f32"]
