"""FFN launches of few tiles, which run by quarters of them: the bits of the call with one token tile per workgroup
asked for, which runs by whole tiles."""
import numpy as np
import pytest

from paper_2510_15964_amd import inputs
from util import dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lx():
    import torch
    assert torch.cuda.is_available()
    from paper_2510_15964_amd import lx
    return lx


# element type, token tiles, tiles per list row, d, neuron blocks, listed blocks per row (None: a row each of 0, 1, 2, ...),
# slack of the capacity.  Steps of the first product: d / 64, of the second: the listed blocks; by pairs through rings of
# eight pairs (up to 64 tiles) or four (up to 128)
CASES = [
    ("bf16", 1, 1, 64, 8, 1, 0),          # one step each
    ("f16", 1, 1, 128, 8, 3, 0),          # one pair; a pair and a half
    ("bf16", 1, 1, 192, 24, 15, 0),
    ("bf16", 1, 1, 896, 24, 16, 3),       # seven pairs, eight: the ring
    ("f16", 1, 1, 960, 40, 17, 0),
    ("bf16", 1, 1, 1088, 40, 18, 0),
    ("bf16", 2, 2, 1152, 80, 64, 0),      # 64 entries: the last before a second fetch; 128 tiles
    ("f16", 1, 1, 2048, 128, 67, 0),      # a second fetch
    ("bf16", 4, 1, 448, 12, None, 5),     # a list per tile, the first one empty
    ("f16", 6, 2, 576, 10, None, 0),      # tiles share lists
    ("bf16", 3, 3, 512, 24, 21, 0),       # one list, 63 tiles and 24
    ("bf16", 3, 3, 512, 24, 22, 0),       # 66: the shorter ring
    ("bf16", 16, 1, 512, 16, 8, 0),       # 128 of both: the most
]


@pytest.mark.parametrize("kind", ["plain", "bias", "lora"])
@pytest.mark.parametrize("dtype,Tt,gt,d,Fb,n,slack", CASES)
def test_bits_of_the_quarters(lx, dtype, Tt, gt, d, Fb, n, slack, kind):
    import torch
    T, F, rows = 64 * Tt, 64 * Fb, Tt // gt
    rng = np.random.default_rng(Tt + d)
    m = np.zeros((rows, Fb), np.uint8)
    for i in range(rows):
        m[i, rng.permutation(Fb)[:n if n is not None else 2 * i]] = 1
    nnz = int(m.sum())
    cap = nnz + slack
    assert cap * gt <= 128 and Tt * d // 64 <= 128
    bl = lx.lx_mask_compact(torch.from_numpy(m).cuda(), nnz_cap=cap)
    g = torch.Generator(device="cuda").manual_seed(d)
    tdt = dev(np.zeros(1, np.float32), dtype).dtype

    def normal(*shape, std=1.0):
        return (torch.randn(shape, device="cuda", generator=g) * std).to(tdt)

    X, dY, Wu, Wd = normal(T, d), normal(T, d), normal(F, d, std=0.05), normal(d, F, std=0.05)
    Wut, Wdt = lx.lx_ffn_pack_weights(Wu, Wd)
    mats = inputs.lora_matrices(d, F, 16, 3)
    A, B = (dev(mats[k], dtype) for k in ("A_pad", "B_pad"))
    bias = dict(b_up=normal(F), b_down=normal(d)) if kind == "bias" else {}
    lxt = {"bf16": lx.LX_BF16, "f16": lx.LX_F16}[dtype]

    def run(tiles):
        lx.lx_ffn_set_token_tiles_per_workgroup(tiles)
        try:
            H = torch.full((cap * gt * 4096,), float("nan"), dtype=tdt, device="cuda")
            Y, dX = torch.full_like(X, float("nan")), torch.full_like(X, float("nan"))
            more = []
            if kind == "lora":
                U = torch.empty(T, 64, dtype=tdt, device="cuda")
                more = [torch.empty(64, d, device="cuda"), torch.empty(F, 64, device="cuda")]
                wf = torch.empty(lx.lx_sparse_ffn_lora_fwd_workspace_bytes(T, d), dtype=torch.uint8, device="cuda")
                wb = torch.empty(lx.lx_sparse_ffn_lora_bwd_workspace_bytes(T, d, F, cap * gt), dtype=torch.uint8, device="cuda")
                lx.lx_sparse_ffn_lora_fwd(X, Wu, A, B, Wd, bl, Y, H, U, wf)
                lx.lx_sparse_ffn_lora_bwd(X, dY, H, U, Wut, Wdt, A, B, bl, dX, *more, wb)
            else:
                wb = torch.empty(lx.lx_sparse_ffn_bwd_workspace_bytes(lxt, T, d, F, 64, 64, cap * gt, 1), dtype=torch.uint8,
                                 device="cuda")
                lx.lx_sparse_ffn_fwd(X, Wu, Wd, bl, 64, 64, Y, H, **bias)
                lx.lx_sparse_ffn_bwd_dx(dY, H, Wu, Wd, bl, 64, 64, dX, wb, W_up_t=Wut, W_down_t=Wdt)
            torch.cuda.synchronize()
        finally:
            lx.lx_ffn_set_token_tiles_per_workgroup(0)
        return [H[:nnz * gt * 4096], H[nnz * gt * 4096:], Y, dX] + more

    quarters, whole = run(0), run(1)
    assert torch.isnan(quarters[1]).all()             # nothing beyond the lists
    for a, b in zip(quarters[:1] + quarters[2:], whole[:1] + whole[2:]):
        assert torch.isfinite(a).all() and torch.equal(a, b)
