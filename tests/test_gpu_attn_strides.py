"""16-bit attention at token strides on both sides of the one up to which a tile's transfers have one 32-bit offset per lane:
the bits of the same call on contiguous tensors."""
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


@pytest.mark.parametrize("D,dtype,ss,apart", [
    (64, "bf16", (1 << 25) - 8, False),          # the last row's offset is 2^32 - 2^26 - 1008 bytes
    (128, "f16", (1 << 25) - 8, True),           # query side and key side in launches of their own
    (64, "f16", 1 << 25, True),                  # the first stride of 64-bit addresses
    (128, "bf16", 1 << 25, False),
])
def test_token_strides_around_the_32_bit_limit(lx, D, dtype, ss, apart):
    import torch
    Hh, S = 2, 128
    c = inputs.attn_blocks(1, Hh, S, D, 0.7, 78, dtype=dtype, force_diagonal=True)
    torch.cuda.empty_cache()
    buf = torch.empty((S - 1) * ss + 8 * Hh * D, dtype=dev(c["Q"], dtype).dtype, device="cuda")
    at = lambda i: buf.as_strided((1, Hh, S, D), (Hh * D, D, ss, 1), i * Hh * D)
    rows, cols = lx.lx_mask_compact_pair(torch.from_numpy(c["mask"]).cuda())
    lxt = {"bf16": lx.LX_BF16, "f16": lx.LX_F16}[dtype]
    ws = torch.empty(lx.lx_sparse_attn_bwd_workspace_bytes(lxt, 1, Hh, S, D), dtype=torch.uint8, device="cuda")

    def call(new):
        Q, K, V, dO, O, dQ, dK, dV = (new(i) for i in range(8))
        for t, k in ((Q, "Q"), (K, "K"), (V, "V"), (dO, "dO")):
            t.copy_(dev(c[k], dtype))
        for t in (O, dQ, dK, dV):
            t.fill_(float("nan"))
        LSE = torch.full((1, Hh, S), float("nan"), device="cuda")
        lx.lx_sparse_attn_fwd(Q, K, V, rows, c["scale"], c["causal"], O, LSE)
        lx.lx_sparse_attn_bwd_dx(Q, K, V, O, LSE, dO, rows, cols, c["scale"], c["causal"], dQ, K if apart else dK, dV, ws)
        torch.cuda.synchronize()
        return [t.contiguous() for t in (O, LSE, dQ, K if apart else dK, dV)]

    wide = call(at)
    plain = call(lambda i: torch.empty((1, Hh, S, D), dtype=buf.dtype, device="cuda"))
    for a, b in zip(wide, plain):
        assert torch.isfinite(a).all() and torch.equal(a, b)
    del buf, wide
    torch.cuda.empty_cache()
