"""GPU parity: block-sparse attention forward / backward against the CPU
oracle, called through the C ABI (ctypes binding)."""
import numpy as np
import pytest

from paper_2510_15964_amd import inputs
import emulate16
from util import (FRO, TOL, assert_within_emulated, dev, host, rel_err, rel_err_fro,
                  rel_err_max, lx_dtype)

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lx():
    import torch
    assert torch.cuda.is_available()
    from paper_2510_15964_amd import lx
    return lx


def run_gpu(lx, c, layout="bhsd"):
    import torch
    B, Hh, S, D = c["B"], c["Hh"], c["S"], c["D"]

    def place(a):
        t = dev(a, c.get("dtype", "bf16"))
        if layout == "bshd":                      # [B,S,Hh,D] storage viewed as [B,Hh,S,D]
            t = t.permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3)
        return t

    Q, K, V, dO = (place(c[k]) for k in ("Q", "K", "V", "dO"))
    mask = torch.from_numpy(c["mask"]).cuda()
    bl_r = lx.lx_mask_compact(mask)
    bl_c = lx.lx_mask_compact(mask, transpose=True)
    ha = torch.from_numpy(c["head_active"]).cuda()
    O = torch.full_like(Q, float("nan"))
    LSE = torch.full((B, Hh, S), float("nan"), dtype=torch.float32, device="cuda")
    lx.lx_sparse_attn_fwd(Q, K, V, bl_r, c["scale"], c["causal"], O, LSE,
                          mask_batch=c["mask_batch"], head_active=ha)
    dQ, dK, dV = (torch.full_like(Q, float("nan")) for _ in range(3))
    ws = torch.empty(lx.lx_sparse_attn_bwd_workspace_bytes(lx_dtype(lx, c.get("dtype", "bf16")), B, Hh, S, D),
                     dtype=torch.uint8, device="cuda")
    lx.lx_sparse_attn_bwd_dx(Q, K, V, O, LSE, dO, bl_r, bl_c, c["scale"], c["causal"], dQ, dK, dV,
                             ws, mask_batch=c["mask_batch"], head_active=ha)
    torch.cuda.synchronize()
    return dict(O=host(O), LSE=host(LSE), dQ=host(dQ), dK=host(dK), dV=host(dV))


def run_oracle(oracle, c):
    O, L = oracle.attn_fwd(c["Q"], c["K"], c["V"], c["mask"], c["scale"], c["causal"],
                           c["head_active"], c["blk"])
    dQ, dK, dV = oracle.attn_bwd(c["Q"], c["K"], c["V"], c["dO"], c["mask"], c["scale"],
                                 c["causal"], c["head_active"], c["blk"])
    # the ideal 16-bit pipeline on the same input: what the element-wise gate is derived from
    return dict(O=O, LSE=L, dQ=dQ, dK=dK, dV=dV, emul=emulate16.attn_realisations(c))


def check(got, ref, label="", fro_from_emul=False, dtype="bf16"):
    """Gates per tensor: max-rel <= TOL, Frobenius <= FRO, and the rms-floored element-wise error
    at most EMUL_FACTOR times that of the ideal 16-bit pipeline on the same input (ref["emul"]: the
    realisations of emulate16.attn_realisations, whose largest figure counts).
    fro_from_emul: the Frobenius gate of the gradients is a quarter above the ideal pipeline's
    Frobenius error instead (inputs whose ideal pipeline already exceeds FRO)."""
    tol = TOL[dtype]
    emul = ref["emul"]
    fro_gate = {k: FRO[dtype] for k in ("O", "dQ", "dK", "dV")}
    if fro_from_emul:
        fro_gate.update({k: max(FRO[dtype], 1.25 * max(rel_err_fro(e[k], ref[k]) for e in emul))
                         for k in ("dQ", "dK", "dV")})
    ninf = np.isneginf(ref["LSE"])
    assert np.array_equal(np.isneginf(got["LSE"]), ninf), "rows without keys must give LSE = -inf"
    errs = {k: rel_err_max(got[k], ref[k]) for k in ("O", "dQ", "dK", "dV")}
    fro = {k: rel_err_fro(got[k], ref[k]) for k in ("O", "dQ", "dK", "dV")}
    floor = {k: rel_err(got[k], ref[k]) for k in ("O", "dQ", "dK", "dV")}
    ideal = {k: max(rel_err(e[k], ref[k]) for e in emul) for k in ("O", "dQ", "dK", "dV")}
    fin = ~ninf
    errs["LSE"] = float(np.max(np.abs(got["LSE"][fin] - ref["LSE"][fin]))) if fin.any() else 0.0
    print(f"[attn {label}] max-rel {errs} fro {fro} rms-floored {floor} (ideal pipeline {ideal})", flush=True)
    for k in ("O", "dQ", "dK", "dV"):
        assert np.isfinite(got[k]).all(), k
        assert errs[k] <= tol, (k, errs[k])
        assert fro[k] <= fro_gate[k], (k, fro[k])
        if dtype == "f32":               # fp32 meets the element-wise gate as it stands
            assert floor[k] <= tol, (k, floor[k])
        else:                            # 16-bit: against the ideal 16-bit pipeline on this input
            assert_within_emulated(got[k], ref[k], [e[k] for e in emul], k)
    assert errs["LSE"] <= tol        # absolute, natural-log units
    # rows with no allowed key: exact zeros
    assert not got["O"][ninf].any() and not got["dQ"][ninf].any()


@pytest.mark.parametrize("kw,seed", [
    (dict(B=2, Hh=3, S=256, D=64, density=0.4), 1),
    (dict(B=1, Hh=2, S=320, D=128, density=0.5), 2),
    (dict(B=2, Hh=2, S=192, D=64, density=1.0), 3),
    (dict(B=1, Hh=4, S=256, D=64, density=0.3, causal=False), 4),
    (dict(B=2, Hh=4, S=128, D=128, density=0.5, head_keep=0.5), 5),
    (dict(B=3, Hh=2, S=192, D=64, density=0.4, mask_batch=3), 6),
    (dict(B=1, Hh=2, S=256, D=64, density=0.4, force_diagonal=True), 7),
    (dict(B=1, Hh=1, S=64, D=64, density=1.0), 8),
    (dict(B=1, Hh=2, S=128, D=64, density=0.0), 9),
])
def test_small_shapes(lx, oracle, kw, seed):
    c = inputs.attn_blocks(seed=seed, dtype="bf16", **kw)
    check(run_gpu(lx, c), run_oracle(oracle, c), str(kw))


@pytest.mark.parametrize("kw,seed", [
    (dict(B=2, Hh=3, S=448, D=64, density=0.4), 31),            # 7 blocks: ragged last group
    (dict(B=1, Hh=2, S=320, D=128, density=0.5), 32),
    (dict(B=1, Hh=2, S=576, D=64, density=0.25, causal=False), 33),
    (dict(B=2, Hh=2, S=256, D=64, density=0.3, head_keep=0.5), 34),
])
def test_rows_per_workgroup(lx, oracle, kw, seed):
    """A workgroup that walks several rows of the mask as one stream of blocks gives the
    same bits as one workgroup per row, and both match the oracle."""
    c = inputs.attn_blocks(seed=seed, dtype="bf16", **kw)
    ref = run_oracle(oracle, c)
    try:
        outs = {}
        for r in (1, 2, 3, 4, 8):
            lx.lx_attn_set_rows_per_workgroup(r)
            outs[r] = run_gpu(lx, c)
            check(outs[r], ref, f"{kw} rows/wg={r}")
        for r in (2, 3, 4, 8):
            for k in outs[1]:
                assert np.array_equal(outs[r][k], outs[1][k], equal_nan=True), (r, k)
    finally:
        lx.lx_attn_set_rows_per_workgroup(0)
    with pytest.raises(Exception):
        lx.lx_attn_set_rows_per_workgroup(9)


def test_large_score_range(lx, oracle):
    """Scores spread over tens of log2 units: the running reference point of the online softmax
    has to move repeatedly and the accumulators are rescaled (the forward kernel rescales only
    when the maximum has moved by more than a slack, which N(0,1) scores rarely do)."""
    c = inputs.attn_blocks(2, 2, 512, 64, 0.5, seed=41, dtype="bf16")
    c["Q"] = c["Q"] * np.float32(8.0)          # exact in bf16
    # With near-one-hot probabilities dS = P (dP - Delta) cancels strongly, so the one bf16
    # rounding of dS weighs more in the gradients' Frobenius error than the two-roundoff gate
    # derived for ordinary scores allows, already in the ideal pipeline (5.1e-3 for dQ:
    # test_emulated_gate.py); the gradients are gated at a quarter above the ideal pipeline's
    # Frobenius error on this input (a sum over all elements, stable between realisations),
    # the forward output keeps the ordinary gate.
    check(run_gpu(lx, c), run_oracle(oracle, c), "large score range", fro_from_emul=True)


def test_strided_layout(lx, oracle):
    """[B,S,Hh,D] storage (heads interleaved) through the stride arguments."""
    c = inputs.attn_blocks(2, 3, 192, 64, 0.5, seed=21, dtype="bf16")
    a = run_gpu(lx, c, layout="bshd")
    b = run_gpu(lx, c, layout="bhsd")
    for k in a:
        assert np.array_equal(a[k], b[k], equal_nan=True), k
    check(a, run_oracle(oracle, c), "bshd")


def test_unused_key_blocks_are_never_read(lx, oracle):
    c = inputs.attn_blocks(1, 2, 256, 64, 0.5, seed=22, dtype="bf16")
    c["mask"][0, :, :, 1] = 0
    ref = run_gpu(lx, c)
    K, V = c["K"].copy(), c["V"].copy()
    K[:, :, 64:128] = np.nan
    V[:, :, 64:128] = np.nan
    got = run_gpu(lx, dict(c, K=K, V=V))
    for k in ("O", "LSE", "dQ"):
        assert np.array_equal(got[k], ref[k]), k
    keep = np.ones(256, dtype=bool)
    keep[64:128] = False
    for k in ("dK", "dV"):
        assert np.array_equal(got[k][:, :, keep], ref[k][:, :, keep]), k
        assert not got[k][:, :, ~keep].any()          # unused keys receive zero gradient


def test_config3_full_size_sampled_heads(lx, oracle):
    """The OPT-1.3B attention at full size in the benchmark's launch configuration; the
    oracle checks sampled (batch, head) pairs, which are independent."""
    c = inputs.config3_attn()
    got = run_gpu(lx, c)
    on = np.nonzero(c["head_active"])[0]
    off = np.nonzero(c["head_active"] == 0)[0]
    for (b, h) in [(0, int(on[0])), (5, int(on[len(on) // 2])), (7, int(on[-1]))]:
        sub = dict(c, B=1, Hh=1, mask=c["mask"][:, h:h + 1], head_active=np.ones(1, np.uint8),
                   **{k: c[k][b:b + 1, h:h + 1] for k in ("Q", "K", "V", "dO")})
        ref = run_oracle(oracle, sub)
        check({k: v[b:b + 1, h:h + 1] for k, v in got.items()}, ref, f"config3 b={b} h={h}")
    for h in off:                                       # inactive heads: zeros, LSE = -inf
        assert not got["O"][:, h].any() and np.all(np.isneginf(got["LSE"][:, h]))
        assert not got["dQ"][:, h].any() and not got["dK"][:, h].any() and not got["dV"][:, h].any()


def test_config4_shape_sampled_heads(lx, oracle):
    """OPT-6.7B attention half (head size 128, 2048 tokens), reduced batch."""
    c = inputs.attn_blocks(1, 4, 2048, 128, 0.25, seed=4000, dtype="bf16")
    got = run_gpu(lx, c)
    for h in (0, 3):
        sub = dict(c, Hh=1, mask=c["mask"][:, h:h + 1], head_active=np.ones(1, np.uint8),
                   **{k: c[k][:, h:h + 1] for k in ("Q", "K", "V", "dO")})
        check({k: v[:, h:h + 1] for k, v in got.items()}, run_oracle(oracle, sub), f"config4 h={h}")


def test_list_longer_than_its_capacity_is_truncated(lx):
    """Row list with a capacity bound that was too small: the forward pass ignores the entries
    after the first nnz_cap and gives the bits of the truncated mask."""
    import torch
    c = inputs.attn_blocks(1, 2, 384, 64, 0.6, seed=51, dtype="bf16")
    mask = c["mask"]                                   # [1, Hh, nb, nb]
    nnz = int(mask.sum())
    cap = nnz - 4
    trunc = mask.copy()
    idx = np.argwhere(mask.reshape(-1, mask.shape[-1]))   # (row, col) in list order
    for r, col in idx[cap:]:
        trunc.reshape(-1, mask.shape[-1])[r, col] = 0
    Q, K, V = (dev(c[k], "bf16") for k in ("Q", "K", "V"))

    def run(m):
        bl = lx.lx_mask_compact(torch.from_numpy(np.ascontiguousarray(m)).cuda(), nnz_cap=cap)
        O = torch.full_like(Q, float("nan"))
        LSE = torch.full((c["B"], c["Hh"], c["S"]), float("nan"), dtype=torch.float32, device="cuda")
        lx.lx_sparse_attn_fwd(Q, K, V, bl, c["scale"], c["causal"], O, LSE, mask_batch=1)
        torch.cuda.synchronize()
        return host(O), host(LSE)

    a, b = run(mask), run(trunc)
    assert np.isfinite(a[0]).all()
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])


@pytest.mark.parametrize("r", [0, 1, 8])
def test_rows_of_one_and_two_blocks(lx, oracle, r):
    """Every row of the mask lists one block (the diagonal) or two (diagonal and the block
    before): the shortest rows there are, where a row hands over to the next one in the very step
    in which the next row's own tiles were requested."""
    for width in (1, 2):
        c = inputs.attn_blocks(2, 3, 512, 64, 1.0, seed=40 + width, dtype="bf16")
        nb = 512 // 64
        q, k = np.arange(nb)[:, None], np.arange(nb)[None, :]
        c["mask"] = np.broadcast_to(((q - k >= 0) & (q - k < width)).astype(np.uint8),
                                    c["mask"].shape).copy()
        lx.lx_attn_set_rows_per_workgroup(r)
        try:
            got = run_gpu(lx, c)
        finally:
            lx.lx_attn_set_rows_per_workgroup(0)
        check(got, run_oracle(oracle, c), f"band of {width}, rows per workgroup {r}")


@pytest.mark.parametrize("D", [64, 128])
def test_blocks_above_the_diagonal_of_a_causal_mask(lx, oracle, D):
    """A list that holds blocks above the diagonal although the call is causal (a predictor or a
    pattern pool may produce one): their keys all lie after the queries, so they contribute
    nothing, as in the oracle, whose key test is k <= q wherever the block lies.  Row 0 of head 1
    lists ONLY such blocks: no allowed key, O = 0, LSE = -inf."""
    c = inputs.attn_blocks(2, 2, 320, D, 0.5, seed=61, dtype="bf16")
    rng = np.random.default_rng(5)
    nb = 320 // 64
    up = np.triu(np.ones((nb, nb), np.uint8), 1)
    c["mask"] = c["mask"] | (up[None, None] & (rng.random(c["mask"].shape) < 0.5)).astype(np.uint8)
    c["mask"][0, 1, 0] = [0, 1, 0, 1, 1]
    ref = run_oracle(oracle, c)
    assert np.isneginf(ref["LSE"][:, 1, :64]).all()
    check(run_gpu(lx, c), ref, f"blocks above the diagonal, D={D}")


@pytest.mark.parametrize("kw,seed", [
    (dict(B=2, Hh=3, S=256, D=64, density=0.4), 81),
    (dict(B=1, Hh=2, S=320, D=128, density=0.5), 82),
    (dict(B=1, Hh=4, S=256, D=64, density=0.3, causal=False), 83),
    (dict(B=2, Hh=4, S=128, D=128, density=0.5, head_keep=0.5), 84),
    (dict(B=3, Hh=2, S=192, D=64, density=0.4, mask_batch=3), 85),
    (dict(B=1, Hh=2, S=128, D=64, density=0.0), 86),
    (dict(B=1, Hh=2, S=1024, D=64, density=0.3), 87),          # the benchmark's sequence length
])
def test_fp32_attention(lx, oracle, kw, seed):
    """LX_F32 attention (the correctness configuration): forward and backward within the fp32 gates
    of the oracle -- 1e-5 on the largest error, on the element-wise error with an rms floor and on
    LSE, 2e-6 on the Frobenius error."""
    c = inputs.attn_blocks(seed=seed, dtype="f32", **kw)
    check(run_gpu(lx, c), run_oracle(oracle, c), f"f32 {kw}", dtype="f32")


@pytest.mark.parametrize("B,Hh,S,D,density,causal,dtype,rows", [
    (1, 2, 4160, 64, 0.04, True, "bf16", 0),        # 65 row blocks per head
    (1, 1, 4224, 128, 0.05, False, "f16", 3),
    (1, 1, 4160, 64, 0.05, True, "f32", 0),
])
def test_more_than_64_row_blocks_per_head(lx, oracle, B, Hh, S, D, density, causal, dtype, rows):
    """Sequences of more than 4096 tokens: a head has more rows than the 64 lanes that rank the
    rows of a head group by list length, so the rows are dealt to the workgroups in the fixed
    order instead."""
    c = inputs.attn_blocks(B, Hh, S, D, density, seed=95, dtype=dtype, causal=causal)
    lx.lx_attn_set_rows_per_workgroup(rows)
    try:
        check(run_gpu(lx, c), run_oracle(oracle, c), f"long {dtype} S={S} D={D}", dtype=dtype)
    finally:
        lx.lx_attn_set_rows_per_workgroup(0)


def test_more_entries_than_one_fill_of_the_block_table(lx, oracle):
    """A workgroup's sequence of ring entries (a row's own tiles, then its listed blocks) is written
    into an LDS table of 512 entries at a time: eight dense rows of 65 blocks are 528 entries, so
    the walk refills the table in the middle of a row."""
    c = inputs.attn_blocks(1, 1, 4160, 64, 1.0, seed=97, dtype="bf16", causal=False)
    lx.lx_attn_set_rows_per_workgroup(8)
    try:
        check(run_gpu(lx, c), run_oracle(oracle, c), "two table fills")
    finally:
        lx.lx_attn_set_rows_per_workgroup(0)


def test_fp32_attention_strided_and_above_diagonal(lx, oracle):
    c = inputs.attn_blocks(2, 2, 320, 64, 0.5, seed=88, dtype="f32")
    nb = 320 // 64
    up = np.triu(np.ones((nb, nb), np.uint8), 1)
    c["mask"] = c["mask"] | (up[None, None] & (np.random.default_rng(6).random(c["mask"].shape) < 0.5)).astype(np.uint8)
    c["mask"][0, 1, 0] = [0, 1, 0, 1, 1]        # row 0 of head 1: only blocks above the diagonal
    ref = run_oracle(oracle, c)
    a = run_gpu(lx, c, layout="bshd")
    b = run_gpu(lx, c, layout="bhsd")
    for k in a:
        assert np.array_equal(a[k], b[k], equal_nan=True), k
    check(a, ref, "f32 bshd, blocks above the diagonal", dtype="f32")


@pytest.mark.parametrize("D,dtype", [(64, "bf16"), (128, "f16")])
def test_token_strides_beyond_32_bit_offsets(lx, D, dtype):
    """A token stride of 2^28 elements (all tensors interleaved in one buffer of 127 strides, of which only the
    128 token rows are touched): the bits of the same call on contiguous tensors."""
    import torch
    Hh, S, ss = 2, 128, 1 << 28
    c = inputs.attn_blocks(1, Hh, S, D, 0.7, 77, dtype=dtype, force_diagonal=True)
    torch.cuda.empty_cache()
    buf = torch.empty((S - 1) * ss + 8 * Hh * D, dtype=dev(c["Q"], dtype).dtype, device="cuda")
    at = lambda i: buf.as_strided((1, Hh, S, D), (Hh * D, D, ss, 1), i * Hh * D)
    mask = torch.from_numpy(c["mask"]).cuda()
    rows, cols = lx.lx_mask_compact_pair(mask)
    ws = torch.empty(lx.lx_sparse_attn_bwd_workspace_bytes(lx_dtype(lx, dtype), 1, Hh, S, D), dtype=torch.uint8,
                     device="cuda")

    def call(new):
        Q, K, V, dO, O, dQ, dK, dV = (new(i) for i in range(8))
        for t, k in ((Q, "Q"), (K, "K"), (V, "V"), (dO, "dO")):
            t.copy_(dev(c[k], dtype))
        for t in (O, dQ, dK, dV):
            t.fill_(float("nan"))
        LSE = torch.full((1, Hh, S), float("nan"), device="cuda")
        lx.lx_sparse_attn_fwd(Q, K, V, rows, c["scale"], c["causal"], O, LSE)
        lx.lx_sparse_attn_bwd_dx(Q, K, V, O, LSE, dO, rows, cols, c["scale"], c["causal"], dQ, dK, dV, ws)
        torch.cuda.synchronize()
        return [t.contiguous() for t in (O, LSE, dQ, dK, dV)]

    wide = call(at)
    plain = call(lambda i: torch.empty((1, Hh, S, D), dtype=buf.dtype, device="cuda"))
    for a, b in zip(wide, plain):
        assert torch.isfinite(a).all() and torch.equal(a, b)
    del buf, wide
    torch.cuda.empty_cache()


@pytest.mark.parametrize("B,Hh,S,D,kw", [
    (4, 8, 512, 64, dict(density=0.4)),                   # one pair per XCD, 32 workgroups each
    (4, 12, 512, 128, dict(density=1.0)),                 # and a rest of four pairs
    (3, 10, 320, 64, dict(density=0.5, causal=False)),    # 15 pairs: a rest of seven, runs that cross pairs
    (2, 5, 4096, 64, dict(density=0.05)),                 # a head per pair
])
def test_order_of_the_workgroups(lx, B, Hh, S, D, kw):
    """Few rows per workgroup (an XCD's workgroups ordered by their length) against eight (pair after pair): same bits."""
    c = inputs.attn_blocks(B, Hh, S, D, seed=B * S + Hh, dtype="bf16", **kw)
    out = []
    for rows in (8, 1, 2, 3):
        print(B, Hh, S, D, "rows per workgroup", rows, flush=True)
        lx.lx_attn_set_rows_per_workgroup(rows)
        try:
            out.append(run_gpu(lx, c))
        finally:
            lx.lx_attn_set_rows_per_workgroup(0)
        for k in ("O", "dQ", "dK", "dV"):
            assert np.isfinite(out[-1][k]).all()
            assert np.array_equal(out[-1][k], out[0][k]), (rows, k)
        assert np.array_equal(out[-1]["LSE"], out[0]["LSE"])
