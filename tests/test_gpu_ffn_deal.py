"""Launches with lists per group of token tiles: every way of dealing the work, tiles with one stage, lists whose two
halves differ, rows up to 64 and beyond.  Rows are independent, so sampled token tiles equal, bit for bit, a call that
holds that tile alone."""
import numpy as np
import pytest

from paper_2510_15964_amd import inputs
from util import FRO, dev, host, rel_err_fro

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lx():
    import torch
    assert torch.cuda.is_available()
    from paper_2510_15964_amd import lx
    return lx


# element type, token tiles, tiles per list row, d, neuron blocks, capacity, products with one stage (bits), order of the
# second product, density
CASES = [
    ("bf16", 66, 1, 1024, 48, 2851, 1, 1, 0.8),
    ("f16", 80, 1, 320, 48, 3443, 1, 2, 0.8),
    ("bf16", 129, 1, 1600, 24, 2788, 1, 0, 0.8),       # more groups than are ranked
    ("bf16", 80, 1, 2048, 12, 275, 2, 0, 0.2),
    ("f16", 96, 1, 2048, 32, 2767, 3, 0, 0.8),
    ("bf16", 49, 1, 1152, 40, 500, 0, 0, 0.2),        # chunks cut by an XCD's eighth
    ("bf16", 100, 2, 1600, 24, 330, 0, 0, 0.25),
    ("bf16", 128, 1, 512, 40, 1000, 0, 1, 0.15),
    ("f16", 3, 1, 832, 40, 70, 0, 2, 0.5),
    ("bf16", 64, 1, 64, 1100, 70400, 0, 2, 0.01),     # 64 rows, a capacity beyond 16 bits
]


@pytest.mark.parametrize("lora", [False, True])
@pytest.mark.parametrize("dtype,Tt,gt,d,Fb,cap,lean,order,density", CASES)
def test_deals(lx, dtype, Tt, gt, d, Fb, cap, lean, order, density, lora):
    import torch
    T, F, rows = 64 * Tt, 64 * Fb, Tt // gt
    rng = np.random.default_rng(Tt + d)
    m = (rng.random((rows, Fb)) < density * rng.uniform(0.3, 1.2, (rows, 1))).astype(np.uint8)
    m[rows // 2] = 0
    m[0] = 0
    m[0, Fb // 3] = 1
    assert m.sum() <= cap
    g = torch.Generator(device="cuda").manual_seed(d)
    tdt = dev(np.zeros(1, np.float32), dtype).dtype

    def normal(*shape, std=1.0):
        return (torch.randn(shape, device="cuda", generator=g) * std).to(tdt)

    X, dY, Wu, Wd = normal(T, d), normal(T, d), normal(F, d, std=0.05), normal(d, F, std=0.05)
    Wut, Wdt = lx.lx_ffn_pack_weights(Wu, Wd)
    mats = inputs.lora_matrices(d, F, 16, 3)
    A, B = (dev(mats[k], dtype) for k in ("A_pad", "B_pad"))

    def run(X, dY, mask, cap, tiles):
        n, t = tiles * cap, X.shape[0]
        full = lx.lx_mask_compact(torch.from_numpy(np.ascontiguousarray(mask)).cuda())
        bl = lx.BlockList(mask.shape[0], Fb, full.row_ptr, full.col_idx, cap)
        H = torch.full((max(n, 1) * 4096,), float("nan"), dtype=tdt, device="cuda")
        Y, dX = torch.full_like(X, float("nan")), torch.full_like(X, float("nan"))
        if lora:
            U = torch.empty((t, 64), dtype=tdt, device="cuda")
            wf, wb = (torch.empty(b, dtype=torch.uint8, device="cuda") for b in (
                lx.lx_sparse_ffn_lora_fwd_workspace_bytes(t, d), lx.lx_sparse_ffn_lora_bwd_workspace_bytes(t, d, F, n)))
            dA, dB = torch.empty((64, d), device="cuda"), torch.empty((F, 64), device="cuda")
            lx.lx_sparse_ffn_lora_fwd(X, Wu, A, B, Wd, bl, Y, H, U, wf)
            lx.lx_sparse_ffn_lora_bwd(X, dY, H, U, Wut, Wdt, A, B, bl, dX, dA, dB, wb)
        else:
            wb = torch.empty(lx.lx_sparse_ffn_bwd_workspace_bytes(lx.LX_F16 if dtype == "f16" else lx.LX_BF16, t, d, F, 64, 64, n, 1),
                             dtype=torch.uint8, device="cuda")
            lx.lx_sparse_ffn_fwd(X, Wu, Wd, bl, 64, 64, Y, H)
            lx.lx_sparse_ffn_bwd_dx(dY, H, Wu, Wd, bl, 64, 64, dX, wb, W_up_t=Wut, W_down_t=Wdt)
        return Y, dX, H, full.row_ptr.cpu().numpy().astype(np.int64)

    Y, dX, H, ptr = run(X, dY, m, cap, gt)
    assert torch.isfinite(Y.float()).all() and torch.isfinite(dX.float()).all()
    lens = m.sum(axis=1).astype(np.int64)
    sample = {0, Tt - 1, int(lens.argmax()) * gt, int(rows // 2) * gt} | set(rng.integers(0, Tt, 4).tolist())
    for i in sorted(sample):
        r, s = i // gt, slice(64 * i, 64 * i + 64)
        y, dx, h, _ = run(X[s].contiguous(), dY[s].contiguous(), m[r:r + 1], max(int(lens[r]), 1), 1)
        if lora:      # X A^T and dZ B are cut by the number of tiles and then rounded: two roundings, as the gate has them
            for a, b in ((y, Y[s]), (dx, dX[s])):
                a, b = host(a), host(b)
                assert np.abs(a - b).max() == 0 if not b.any() else rel_err_fro(a, b) <= FRO[dtype], i
        else:
            assert torch.equal(y, Y[s]) and torch.equal(dx, dX[s]), i
            blocks = (ptr[r] + np.arange(lens[r])) * gt + i % gt
            assert torch.equal(h.view(-1, 4096)[:lens[r]], H.view(-1, 4096)[torch.from_numpy(blocks).cuda()]), i


# like CASES: lists of few entries, whose tiles' whole lists go to one XCD in the first product
THIN = [
    ("bf16", 129, 1, 1600, 24, 700, 0, 0, 0.15),      # rows beyond one scan
    ("f16", 150, 3, 832, 40, 330, 0, 0, 0.12),
    ("bf16", 64, 1, 512, 128, 800, 0, 2, 0.06),
    ("bf16", 100, 1, 704, 30, 400, 0, 1, 0.1),        # two rows per lane
]


@pytest.mark.parametrize("lora", [False, True])
@pytest.mark.parametrize("dtype,Tt,gt,d,Fb,cap,lean,order,density", THIN)
def test_deals_of_thin_lists(lx, dtype, Tt, gt, d, Fb, cap, lean, order, density, lora):
    test_deals(lx, dtype, Tt, gt, d, Fb, cap, lean, order, density, lora)
