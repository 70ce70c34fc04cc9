"""Attention backward of small calls: the query side and the key side in one launch.  An output over an input keeps the two
launches apart, so the two ways are compared bit for bit; the oracle holds the small ones (test_gpu_attn.py)."""
import numpy as np
import pytest

from util import dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lx():
    import torch
    assert torch.cuda.is_available()
    from paper_2510_15964_amd import lx
    return lx


CASES = [
    ("bf16", 1, 1, 64, 64, 1.0, True, 1, "bhsd"),        # one block
    ("f16", 1, 1, 64, 128, 1.0, False, 1, "bhsd"),
    ("bf16", 1, 12, 320, 64, 0.4, True, 1, "bhsd"),
    ("bf16", 3, 5, 256, 128, 0.3, True, 3, "bshd"),
    ("f16", 2, 7, 448, 64, 0.5, False, 2, "bshd"),
    ("bf16", 3, 32, 512, 64, 0.2, True, 1, "bshd"),      # 768 rows: two per workgroup
    ("bf16", 1, 8, 4096, 64, 0.3, True, 1, "bhsd"),      # 64 rows per head
    ("bf16", 1, 3, 4160, 64, 0.2, True, 1, "bhsd"),      # more: dealt by their number
    ("f16", 8, 36, 384, 64, 0.6, True, 1, "bhsd"),       # 1728 short rows
    ("bf16", 4, 8, 512, 128, 1.0, True, 1, "bhsd"),      # 256 rows at head size 128
    ("bf16", 1, 8, 1024, 128, 0.3, False, 1, "bshd"),    # 128 without causality
    ("f16", 1, 6, 4096, 64, 0.3, False, 1, "bhsd"),      # 384
]
# An output, or the rescaled LSE, so many bytes behind the start of what it overlaps: calls that two launches in order allow
PLACES = [("dQ", "O", 0), ("dK", "K", 0), ("dV", "V", 0), ("dK", "O", 0), ("dV", "O", 1040), ("dK", "O", -48), ("dV", "O", (1 << 17) - 16),
          ("dV", "LSE", -1024), ("dK", "LSE", 0), ("dK", "row_ptr", 0), ("dV", "col_idx", -4096), ("dQ", "dV", 0), ("dQ", "dK", 272),
          ("NegLse2", "LSE", 0)]


@pytest.mark.parametrize("dtype,B,Hh,S,D,density,causal,mask_batch,layout", CASES)
def test_one_launch_equals_two(lx, dtype, B, Hh, S, D, density, causal, mask_batch, layout):
    import torch
    nb = S // 64
    rng = np.random.default_rng(S + D)
    m = rng.random((mask_batch, Hh, nb, nb)) < density
    if causal:
        m &= np.tril(np.ones((nb, nb), bool))
    m[:, 0, 0, :] = False                 # a query block without keys, a key block without queries
    m[:, -1, :, nb // 2] = False
    m[:, -1, nb - 1, 0] = True
    mask = torch.from_numpy(m.astype(np.uint8)).cuda()
    active = torch.ones(Hh, dtype=torch.uint8, device="cuda")
    if Hh > 2:
        active[1] = 0
    g = torch.Generator(device="cuda").manual_seed(S)
    tdt = dev(np.zeros(1, np.float32), dtype).dtype

    def new(fill):
        return fill((B, Hh, S, D)) if layout == "bhsd" else fill((B, S, Hh, D)).transpose(1, 2)

    def like(x):
        return torch.full_like(x, float("nan"))      # (keeps the strides)

    Q, K, V, dO = (new(lambda sh: torch.randn(sh, device="cuda", generator=g).to(tdt)) for _ in range(4))
    rows, cols = lx.lx_mask_compact_pair(mask)
    O, LSE = like(Q), torch.empty((B, Hh, S), device="cuda")
    scale = D ** -0.5
    lx.lx_sparse_attn_fwd(Q, K, V, rows, scale, causal, O, LSE, mask_batch=mask_batch, head_active=active)
    ws = torch.empty(lx.lx_sparse_attn_bwd_workspace_bytes(lx.LX_F16 if dtype == "f16" else lx.LX_BF16, B, Hh, S, D), dtype=torch.uint8,
                     device="cuda")

    def bwd(O, dQ, r, launches):
        dK, dV = like(K), like(V)
        lx.lx_attn_set_rows_per_workgroup(r)
        lx.lx_profile_begin(lx.LX_K_ATTN_BWD_DQ, 4)
        try:
            lx.lx_sparse_attn_bwd_dx(Q, K, V, O, LSE, dO, rows, cols, scale, causal, dQ, dK, dV, ws, mask_batch=mask_batch,
                                     head_active=active)
        finally:
            lx.lx_attn_set_rows_per_workgroup(0)
            assert lx.lx_profile_end()[1] == launches      # of the query side alone
        return dQ, dK, dV

    for r in (0, 1, 3):
        one = bwd(O, like(Q), r, 0)
        shared = torch.empty_like(O)
        shared.copy_(O)
        assert shared.stride() == O.stride()
        two = bwd(shared, shared, r, 1)
        for a, b in zip(one, two):
            assert torch.isfinite(a.float()).all() and torch.equal(a, b), r


@pytest.mark.parametrize("place", PLACES)
def test_outputs_over_inputs(lx, place):
    """What the order of two launches allows to overlap gives the bits of buffers apart."""
    import torch
    B, Hh, S, D, nb = 2, 4, 128, 64, 2
    stats, part, apart = B * Hh * S * 4, B * Hh * S * D * 2, 1 << 20
    mask = torch.tril(torch.ones(1, Hh, nb, nb, dtype=torch.uint8, device="cuda"))
    mask[0, 1, 1, 0] = 0
    g = torch.Generator(device="cuda").manual_seed(5)
    Q, K, V, dO = (torch.randn(B, Hh, S, D, device="cuda", generator=g).to(torch.bfloat16) for _ in range(4))
    rows, cols = lx.lx_mask_compact_pair(mask)
    O, LSE = torch.empty_like(Q), torch.empty((B, Hh, S), device="cuda")
    lx.lx_sparse_attn_fwd(Q, K, V, rows, D ** -0.5, True, O, LSE)
    names = ["Q", "K", "V", "O", "dO", "dQ", "dK", "dV", "LSE", "row_ptr", "col_idx", "ws"]

    def run(place, launches):
        arena = torch.zeros((len(names) + 1) * apart, dtype=torch.uint8, device="cuda")
        at = {k: (i + 1) * apart for i, k in enumerate(names)}
        if place and place[0] == "NegLse2":
            at["ws"] = at[place[1]] + place[2] - stats           # (the second half of the workspace)
        elif place:
            at[place[0]] = at[place[1]] + place[2]

        def new(k, like):
            n = like.numel() * like.element_size()
            return arena[at[k]:at[k] + n].view(like.dtype).view(like.shape)

        out = {k: new(k, Q) for k in ("dQ", "dK", "dV")}
        for t in out.values():
            t.fill_(float("nan"))
        ins = {}
        for k, t in dict(Q=Q, K=K, V=V, O=O, dO=dO, LSE=LSE, row_ptr=rows.row_ptr, col_idx=rows.col_idx).items():
            ins[k] = new(k, t)
            ins[k].copy_(t)
        ws = arena[at["ws"]:at["ws"] + 2 * stats]
        lists = lx.BlockList(rows.rows, rows.cols, ins["row_ptr"], ins["col_idx"], rows.nnz_cap)
        lx.lx_profile_begin(lx.LX_K_ATTN_BWD_DQ, 1)
        try:
            lx.lx_sparse_attn_bwd_dx(ins["Q"], ins["K"], ins["V"], ins["O"], ins["LSE"], ins["dO"], lists, cols, D ** -0.5, True,
                                     out["dQ"], out["dK"], out["dV"], ws)
        finally:
            assert lx.lx_profile_end()[1] == launches
        return out

    one, two = run(None, 0), run(place, 1)
    for k in one:
        if k == "dQ" and place[0] == "dQ" and place[1] in one:
            continue                                             # (overwritten by the output that is wanted)
        assert torch.isfinite(one[k].float()).all() and torch.equal(one[k], two[k]), k


@pytest.mark.parametrize("dtype,D,B,Hh,launches", [("bf16", 64, 2, 6, 0), ("f16", 128, 1, 6, 0), ("bf16", 64, 8, 24, 1), ("f16", 128, 4, 10, 1)])
def test_rows_emptied_by_their_list_s_capacity(lx, dtype, D, B, Hh, launches):
    """Query rows that the capacity of the row list leaves without a block, but that the column list still names, have
    LSE = -inf, and no part in dK and dV: as if the mask did not list them."""
    import torch
    S = 640
    nb = S // 64
    g = torch.Generator(device="cuda").manual_seed(D + B)
    mask = (torch.rand(1, Hh, nb, nb, device="cuda", generator=g) < 0.6).to(torch.uint8)
    short = mask.clone()
    short[0, Hh - 2, 7:] = 0                                 # the last rows in list order
    short[0, Hh - 1] = 0
    tdt = dev(np.zeros(1, np.float32), dtype).dtype
    Q, K, V, dO = (torch.randn(B, Hh, S, D, device="cuda", generator=g).to(tdt) for _ in range(4))
    ws = torch.empty(lx.lx_sparse_attn_bwd_workspace_bytes(lx.LX_BF16, B, Hh, S, D), dtype=torch.uint8, device="cuda")

    def run(rows, cols):
        O, dQ, dK, dV = (torch.full_like(Q, float("nan")) for _ in range(4))
        LSE = torch.full((B, Hh, S), float("nan"), device="cuda")
        lx.lx_sparse_attn_fwd(Q, K, V, rows, D ** -0.5, False, O, LSE)
        lx.lx_profile_begin(lx.LX_K_ATTN_BWD_DQ, 1)
        try:
            lx.lx_sparse_attn_bwd_dx(Q, K, V, O, LSE, dO, rows, cols, D ** -0.5, False, dQ, dK, dV, ws)
        finally:
            assert lx.lx_profile_end()[1] == launches
        return O, LSE, dQ, dK, dV

    cols = lx.lx_mask_compact(mask, transpose=True)
    cut = run(lx.lx_mask_compact(mask, nnz_cap=int(short.sum())), cols)
    ref = run(*lx.lx_mask_compact_pair(short))
    assert torch.isneginf(cut[1][:, Hh - 1]).all()
    for a, b in zip(cut, ref):
        assert torch.equal(a, b)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("ss,launches", [((1 << 25) - 8, 0), (1 << 25, 1)])
def test_long_token_strides_run_in_two(lx, D, ss, launches):
    """From the strides on that have 64-bit addresses; bits as of contiguous tensors: test_gpu_attn_strides.py."""
    import torch
    Hh, S = 2, 64
    torch.cuda.empty_cache()
    buf = torch.empty((S - 1) * ss + 8 * Hh * D, dtype=torch.bfloat16, device="cuda")
    Q, K, V, dO, O, dQ, dK, dV = (buf.as_strided((1, Hh, S, D), (Hh * D, D, ss, 1), i * Hh * D) for i in range(8))
    for t in (Q, K, V, dO):
        t.normal_()
    rows, cols = lx.lx_mask_compact_pair(torch.ones(1, Hh, 1, 1, dtype=torch.uint8, device="cuda"))
    LSE = torch.empty((1, Hh, S), device="cuda")
    ws = torch.empty(lx.lx_sparse_attn_bwd_workspace_bytes(lx.LX_BF16, 1, Hh, S, D), dtype=torch.uint8, device="cuda")
    lx.lx_sparse_attn_fwd(Q, K, V, rows, D ** -0.5, True, O, LSE)
    lx.lx_profile_begin(lx.LX_K_ATTN_BWD_DQ, 1)
    try:
        lx.lx_sparse_attn_bwd_dx(Q, K, V, O, LSE, dO, rows, cols, D ** -0.5, True, dQ, dK, dV, ws)
        torch.cuda.synchronize()
    finally:
        assert lx.lx_profile_end()[1] == launches
    assert all(torch.isfinite(t.float()).all() for t in (dQ, dK, dV))
    del buf, Q, K, V, dO, O, dQ, dK, dV
    torch.cuda.empty_cache()
