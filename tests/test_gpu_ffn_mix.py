"""Launches with one list row, wide tiles and a rest by narrower ones: every tile gives the same bits, so the results
are those of a workgroup per token tile."""
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


# element type, token tiles, d, neuron blocks, capacity, listed blocks, tile of the rest (test_ffn_mix.py: "4x4": none is
# left; None: the list runs by the plan's own tile, or by the tile for its length)
CASES = [
    ("bf16", 61, 1024, 90, 67, 67, "2x2 deep"),       # one token tile in the last group, a ragged group of entries
    ("f16", 61, 512, 110, 96, 93, "2x4"),
    ("bf16", 127, 512, 64, 41, 41, "2x4"),
    ("f16", 126, 768, 80, 65, 65, "2x2 deep"),        # two in the last
    ("bf16", 97, 1024, 64, 48, 41, "2x2 deep"),
    ("bf16", 128, 512, 48, 42, 32, "4x4"),            # the list leaves nothing
    ("f16", 128, 512, 90, 65, 58, None),              # more than half a round is left
    ("bf16", 130, 768, 64, 40, 12, None),             # far shorter than its capacity
]
# the second product: element type, token tiles, d, listed blocks, tile of the rest
DOWN = [
    ("bf16", 130, 2048, 9, "2x2 deep"),               # two token tiles in the last group
    ("f16", 165, 2048, 9, "2x4"),
    ("bf16", 117, 2112, 20, "2x2 deep"),              # 33 column chunks: one in the last group, one token tile too
    ("f16", 163, 2112, 70, "2x4"),                    # three tiles; more entries than are fetched at once
]


@pytest.mark.parametrize("lora", [False, True])
@pytest.mark.parametrize("dtype,Tt,d,n,tail", DOWN)
def test_bits_of_the_second_products_mix(lx, dtype, Tt, d, n, tail, lora):
    compare(lx, dtype, Tt, d, n + 3, n, n, lora)


@pytest.mark.parametrize("lora", [False, True])
@pytest.mark.parametrize("dtype,Tt,d,Fb,cap,n,tail", CASES)
def test_bits_of_the_mix(lx, dtype, Tt, d, Fb, cap, n, tail, lora):
    compare(lx, dtype, Tt, d, Fb, cap, n, lora)


@pytest.mark.parametrize("dtype,Tt,d,Fb,cap,n", [c[:6] for c in CASES[:2]] + [c[:3] + (c[3] + 3, c[3], c[3]) for c in DOWN[:3]])
def test_bits_of_the_mix_with_a_bias(lx, dtype, Tt, d, Fb, cap, n):
    compare(lx, dtype, Tt, d, Fb, cap, n, False, True)


def compare(lx, dtype, Tt, d, Fb, cap, n, lora, bias=False):
    import torch
    T, F = 64 * Tt, 64 * Fb
    rng = np.random.default_rng(Tt + d)
    m = np.zeros((1, Fb), np.uint8)
    m[0, rng.permutation(Fb)[:n]] = 1
    bl = lx.lx_mask_compact(torch.from_numpy(m).cuda(), nnz_cap=cap)
    g = torch.Generator(device="cuda").manual_seed(d)
    tdt = dev(np.zeros(1, np.float32), dtype).dtype

    def normal(*shape, std=1.0):
        return (torch.randn(shape, device="cuda", generator=g) * std).to(tdt)

    X, dY, Wu, Wd = normal(T, d), normal(T, d), normal(F, d, std=0.05), normal(d, F, std=0.05)
    Wut, Wdt = lx.lx_ffn_pack_weights(Wu, Wd)
    mats = inputs.lora_matrices(d, F, 16, 3)
    A, B = (dev(mats[k], dtype) for k in ("A_pad", "B_pad"))
    biases = dict(b_up=normal(F), b_down=normal(d)) if bias else {}
    lxt = {"bf16": lx.LX_BF16, "f16": lx.LX_F16}[dtype]

    def run(tiles):
        lx.lx_ffn_set_token_tiles_per_workgroup(tiles)
        try:
            H = torch.full((cap * Tt * 4096,), float("nan"), dtype=tdt, device="cuda")
            Y, dX = torch.full_like(X, float("nan")), torch.full_like(X, float("nan"))
            if lora:
                U = torch.empty(T, 64, dtype=tdt, device="cuda")
                dA, dB = torch.empty(64, d, device="cuda"), torch.empty(F, 64, device="cuda")
                wf = torch.empty(lx.lx_sparse_ffn_lora_fwd_workspace_bytes(T, d), dtype=torch.uint8, device="cuda")
                wb = torch.empty(lx.lx_sparse_ffn_lora_bwd_workspace_bytes(T, d, F, cap * Tt), dtype=torch.uint8, device="cuda")
                lx.lx_sparse_ffn_lora_fwd(X, Wu, A, B, Wd, bl, Y, H, U, wf)
                lx.lx_sparse_ffn_lora_bwd(X, dY, H, U, Wut, Wdt, A, B, bl, dX, dA, dB, wb)
                more = [dA, dB]
            else:
                wb = torch.empty(lx.lx_sparse_ffn_bwd_workspace_bytes(lxt, T, d, F, 64, 64, cap * Tt, 1), dtype=torch.uint8,
                                 device="cuda")
                lx.lx_sparse_ffn_fwd(X, Wu, Wd, bl, 64, 64, Y, H, **biases)
                lx.lx_sparse_ffn_bwd_dx(dY, H, Wu, Wd, bl, 64, 64, dX, wb, W_up_t=Wut, W_down_t=Wdt)
                more = []
            torch.cuda.synchronize()
        finally:
            lx.lx_ffn_set_token_tiles_per_workgroup(0)
        return [H[:n * Tt * 4096], H[n * Tt * 4096:], Y, dX] + more

    mixed, single = run(0), run(1)
    assert torch.isnan(mixed[1]).all()                # nothing beyond the list
    for a, b in zip(mixed[:1] + mixed[2:], single[:1] + single[2:]):
        assert torch.isfinite(a).all() and torch.equal(a, b)
