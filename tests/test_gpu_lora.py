"""GPU parity: sparse FFN with a LoRA branch on the up-projection (Sec. II-C / II-D) -- forward,
input gradient and the gradients of the trainable A and B -- against the CPU oracle."""
import numpy as np
import pytest

from paper_2510_15964_amd import inputs
from test_gpu_ffn_tiles import CAPACITIES
from util import FRO, TOL, compact_blocks, dev, host, rel_err_fro, rel_err_max, round_to

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lx():
    import torch
    assert torch.cuda.is_available()
    from paper_2510_15964_amd import lx
    return lx


def make_case(T, d, F, r, density, seed, rows=None, dtype="bf16"):
    c = inputs.ffn_bernoulli(T, d, F, 64, 64, density, seed, dtype=dtype, w_std=0.05)
    rng = np.random.default_rng(seed + 17)
    A = np.zeros((64, d), np.float32)
    B = np.zeros((F, 64), np.float32)
    A[:r] = round_to(rng.standard_normal((r, d)) / np.sqrt(d), dtype)
    B[:, :r] = round_to(rng.standard_normal((F, r)) * 0.05, dtype)
    c.update(A_pad=A, B_pad=B, r=r)
    if rows is not None:                      # list rows shared by groups of token tiles
        m = c["mask"][:rows]
        c["list_mask"] = np.ascontiguousarray(m)
        c["mask"] = np.repeat(m, (T // 64) // rows, axis=0)
    return c


def grouped_compact(a, mask_rows, gt):
    """[T,F] -> compact blocks in the layout of shared list rows: [entry][tile of the group]."""
    out = []
    for r in range(mask_rows.shape[0]):
        for j in np.nonzero(mask_rows[r])[0]:
            for g in range(gt):
                i = r * gt + g
                out.append(a[i * 64:(i + 1) * 64, j * 64:(j + 1) * 64])
    return np.stack(out) if out else np.zeros((0, 64, 64), a.dtype)


def run_both(lx, oracle, c):
    import torch
    T, d, F, r, dt = c["T"], c["d"], c["F"], c["r"], c["dtype"]
    lm = c.get("list_mask", c["mask"])
    gt = (T // 64) // lm.shape[0]
    X, Wu, Wd, dY, Ap, Bp = (dev(c[k], dt) for k in ("X", "W_up", "W_down", "dY", "A_pad", "B_pad"))
    bl = lx.lx_mask_compact(torch.from_numpy(lm).cuda())
    nblk = max(bl.nnz_cap * gt, 1)
    H_act = torch.full((nblk * 4096 + 4096,), float("nan"), dtype=X.dtype, device="cuda")
    Y = torch.full_like(X, float("nan"))
    U = torch.full((T, 64), float("nan"), dtype=X.dtype, device="cuda")
    lx.lx_sparse_ffn_lora_fwd(X, Wu, Ap, Bp, Wd, bl, Y, H_act, U)
    Uo, Ho, Yo = oracle.ffn_lora_fwd(c["X"], c["W_up"], c["A_pad"][:r], c["B_pad"][:, :r], c["W_down"],
                                     c["mask"], 64, 64)
    nnz = int(lm.sum())
    got = dict(U=host(U), Y=host(Y), H=host(H_act[:nnz * gt * 4096]).reshape(-1, 64, 64))
    assert torch.isnan(H_act[nblk * 4096:]).all()
    ref = dict(U=np.pad(Uo, ((0, 0), (0, 64 - r))), Y=Yo, H=grouped_compact(Ho, lm, gt))
    # backward: both sides take the oracle's stored activations and U, rounded to the run dtype
    Hq, Uq = round_to(Ho, dt), round_to(ref["U"], dt)
    H_in = torch.zeros_like(H_act)
    H_in[:nnz * gt * 4096] = dev(grouped_compact(Hq, lm, gt).reshape(-1), dt)
    Wut, Wdt = lx.lx_ffn_pack_weights(Wu, Wd)
    ws = torch.empty(lx.lx_sparse_ffn_lora_bwd_workspace_bytes(T, d, F, bl.nnz_cap * gt), dtype=torch.uint8,
                     device="cuda")
    dX = torch.full_like(X, float("nan"))
    dA = torch.full((64, d), float("nan"), dtype=torch.float32, device="cuda")
    dB = torch.full((F, 64), float("nan"), dtype=torch.float32, device="cuda")
    lx.lx_sparse_ffn_lora_bwd(X, dY, H_in, dev(Uq, dt), Wut, Wdt, Ap, Bp, bl, dX, dA, dB, ws)
    torch.cuda.synchronize()
    g = oracle.ffn_lora_bwd(c["X"], c["dY"], c["W_up"], c["A_pad"][:r], c["B_pad"][:, :r], c["W_down"],
                            c["mask"], Hq > 0, Uq[:, :r], 64, 64)
    got.update(dX=host(dX), dA=host(dA), dB=host(dB))
    ref.update(dX=g["dX"], dA=np.pad(g["dA"], ((0, 64 - r), (0, 0))), dB=np.pad(g["dB"], ((0, 0), (0, 64 - r))))
    return got, ref


def check(got, ref, label, dtype="bf16"):
    errs, fro = {}, {}
    for k in ("U", "H", "Y", "dX", "dA", "dB"):
        assert np.isfinite(got[k]).all(), k
        if not ref[k].any():
            assert not got[k].any(), k
            continue
        errs[k], fro[k] = rel_err_max(got[k], ref[k]), rel_err_fro(got[k], ref[k])
    print(f"[lora {label}] max-rel {errs} fro {fro}", flush=True)
    for k in errs:
        assert errs[k] <= TOL[dtype], (k, errs[k])
        assert fro[k] <= FRO[dtype], (k, fro[k])


@pytest.mark.parametrize("T,d,F,r,density,seed", [
    (256, 128, 512, 16, 0.4, 1),
    (512, 256, 1024, 64, 0.2, 2),
    (128, 64, 384, 8, 1.0, 3),
    (320, 192, 640, 1, 0.5, 4),
])
def test_lora_matches_oracle(lx, oracle, T, d, F, r, density, seed):
    c = make_case(T, d, F, r, density, seed)
    got, ref = run_both(lx, oracle, c)
    check(got, ref, f"T={T} d={d} F={F} r={r}")
    assert not got["dA"][r:].any() and not got["dB"][:, r:].any() and not got["U"][:, r:].any()


def test_lora_shared_list_rows(lx, oracle):
    c = make_case(512, 128, 768, 16, 0.4, 5, rows=2)
    got, ref = run_both(lx, oracle, c)
    check(got, ref, "two list rows for eight tiles")


def test_lora_empty_mask_and_unlisted_blocks(lx, oracle):
    c = make_case(256, 128, 512, 16, 0.0, 6)
    got, ref = run_both(lx, oracle, c)
    assert not got["Y"].any() and not got["dX"].any() and not got["dA"].any() and not got["dB"].any()
    c = make_case(256, 128, 512, 16, 0.5, 7)
    c["mask"][:, 3] = 0                                    # a neuron block no tile lists
    got, ref = run_both(lx, oracle, c)
    check(got, ref, "block 3 unlisted")
    assert not got["dB"][3 * 64:4 * 64].any()


def test_zero_branch_equals_the_plain_ffn_bit_for_bit(lx, oracle):
    """B = 0: the extra step adds exact zeros, so Y and H equal the plain kernels' output."""
    import torch
    c = make_case(256, 128, 512, 16, 0.4, 8)
    c["B_pad"][:] = 0
    got, _ = run_both(lx, oracle, c)
    X, Wu, Wd = (dev(c[k], "bf16") for k in ("X", "W_up", "W_down"))
    bl = lx.lx_mask_compact(torch.from_numpy(c["mask"]).cuda())
    H = torch.zeros(bl.nnz_cap * 4096, dtype=X.dtype, device="cuda")
    Y = torch.empty_like(X)
    lx.lx_sparse_ffn_fwd(X, Wu, Wd, bl, 64, 64, Y, H)
    assert np.array_equal(host(Y), got["Y"])
    assert np.array_equal(host(H[:got["H"].size]).reshape(got["H"].shape), got["H"])


def test_lora_bench_widths_reduced_tokens(lx, oracle):
    """OPT-1.3B FFN widths with 512 tokens (the oracle's fp64 loops set the size), rank 16."""
    c = make_case(512, 2048, 8192, 16, 0.11, 9)
    got, ref = run_both(lx, oracle, c)
    check(got, ref, "d=2048 F=8192")


def test_lora_bench_shape_full_size_sampled(lx, oracle):
    """The benchmark's LoRA FFN call (4096 tokens, OPT-1.3B widths, its planted-support mask and
    seeded LoRA matrices) in the launch configuration the benchmark times.  The oracle checks
    what it can compute piece by piece: U for all tokens; H, Y and dX of sampled token tiles
    (tiles are independent); the rows of dB of sampled neuron blocks, from the problem sliced to
    that block (dB of a block needs only that block's weights); and dA and dB in full from a
    second backward call whose dY is zero outside the sampled tiles (the sums then run over
    those tiles only).  The backward calls take the oracle's rounded U and, wherever an output
    is compared, the oracle's rounded activations, so both sides use the same ReLU gate."""
    import torch
    T, d, F, r = 4096, 2048, 8192, 16
    f = inputs.ffn_planted_support(8192, d, F, 64, 64, 0.5, 4.0, seed=2000)
    lo = inputs.lora_matrices(d, F, r, seed=2200)
    X, dYh, mask = f["X"][:T], f["dY"][:T], np.ascontiguousarray(f["mask"][:T // 64])
    A, B = lo["A_pad"][:r], np.ascontiguousarray(lo["B_pad"][:, :r])
    tiles = (0, 29, 63)
    blocks = [int(np.argmax(mask.sum(0))), int(np.argsort(mask.sum(0))[len(mask[0]) // 2]),
              int(np.argmin(mask.sum(0)))]
    rp = np.concatenate([[0], np.cumsum(mask.sum(1, dtype=np.int64))])
    pos = lambda i, j: int(rp[i] + mask[i, :j].sum())          # compact block of (tile i, block j)

    Xd, Wu, Wd, Ap, Bp = (dev(a, "bf16") for a in (X, f["W_up"], f["W_down"], lo["A_pad"], lo["B_pad"]))
    bl = lx.lx_mask_compact(torch.from_numpy(mask).cuda())
    nnz = int(mask.sum())
    assert bl.nnz_cap >= nnz
    H_act = torch.zeros((bl.nnz_cap * 4096,), dtype=Xd.dtype, device="cuda")
    Y = torch.empty_like(Xd)
    U = torch.empty((T, 64), dtype=Xd.dtype, device="cuda")
    lx.lx_sparse_ffn_lora_fwd(Xd, Wu, Ap, Bp, Wd, bl, Y, H_act, U)
    torch.cuda.synchronize()
    Yg, Ug, Hg = host(Y), host(U), host(H_act).reshape(-1, 64, 64)

    def gate(name, g, ref):
        e, fr = rel_err_max(g, ref), rel_err_fro(g, ref)
        print(f"[lora full size] {name}: max-rel {e:.2e} fro {fr:.2e}", flush=True)
        assert e <= TOL["bf16"] and fr <= FRO["bf16"], (name, e, fr)

    # forward, per sampled tile; the oracle's U of every token comes from the block-sliced calls
    H_in = Hg.copy()
    tile_ref = {}
    for i in tiles:
        sl = slice(i * 64, (i + 1) * 64)
        Uo, Ho, Yo = oracle.ffn_lora_fwd(X[sl], f["W_up"], A, B, f["W_down"], mask[i:i + 1], 64, 64)
        gate(f"U tile {i}", Ug[sl, :r], Uo)
        gate(f"Y tile {i}", Yg[sl], Yo)
        js = np.nonzero(mask[i])[0]
        Hc = np.stack([Ho[:, j * 64:(j + 1) * 64] for j in js])
        gate(f"H tile {i}", Hg[rp[i]:rp[i + 1]], Hc)
        Hq = round_to(Ho, "bf16")
        for j in js:
            H_in[pos(i, j)] = Hq[:, j * 64:(j + 1) * 64]
        tile_ref[i] = (Hq, round_to(Uo, "bf16"))
    assert not Ug[:, r:].any()
    blk_ref = {}
    U_all = None
    for j in blocks:
        jb = slice(j * 64, (j + 1) * 64)
        Wu_j, B_j = f["W_up"][jb], B[jb]
        Wd_j = np.ascontiguousarray(f["W_down"][:, jb])
        m_j = np.ascontiguousarray(mask[:, j:j + 1])
        Uo, Ho, _ = oracle.ffn_lora_fwd(X, Wu_j, A, B_j, Wd_j, m_j, 64, 64)
        U_all = Uo
        Hq = round_to(Ho, "bf16")
        for i in np.nonzero(mask[:, j])[0]:
            H_in[pos(i, j)] = Hq[i * 64:(i + 1) * 64]
        blk_ref[j] = (Wu_j, B_j, Wd_j, m_j, Hq)
    gate("U all tokens", Ug[:, :r], U_all)
    Uq = round_to(U_all, "bf16")
    U_in = dev(np.pad(Uq, ((0, 0), (0, 64 - r))), "bf16")
    H_in_d = dev(H_in.reshape(-1), "bf16")

    Wut, Wdt = lx.lx_ffn_pack_weights(Wu, Wd)
    ws = torch.empty(lx.lx_sparse_ffn_lora_bwd_workspace_bytes(T, d, F, bl.nnz_cap), dtype=torch.uint8,
                     device="cuda")

    def backward(dY_host):
        dX = torch.full_like(Xd, float("nan"))
        dA = torch.full((64, d), float("nan"), dtype=torch.float32, device="cuda")
        dB = torch.full((F, 64), float("nan"), dtype=torch.float32, device="cuda")
        lx.lx_sparse_ffn_lora_bwd(Xd, dev(dY_host, "bf16"), H_in_d, U_in, Wut, Wdt, Ap, Bp, bl, dX, dA, dB, ws)
        torch.cuda.synchronize()
        out = host(dX), host(dA), host(dB)
        assert all(np.isfinite(o).all() for o in out)
        return out

    # first call: the benchmark's dY
    dXg, dAg, dBg = backward(dYh)
    assert not dAg[r:].any() and not dBg[:, r:].any()
    sum_dA, sum_dB = np.zeros((r, d)), np.zeros((F, r))
    for i in tiles:
        sl = slice(i * 64, (i + 1) * 64)
        Hq, Uq_i = tile_ref[i]
        g = oracle.ffn_lora_bwd(X[sl], dYh[sl], f["W_up"], A, B, f["W_down"], mask[i:i + 1], Hq > 0, Uq_i,
                                64, 64)
        gate(f"dX tile {i}", dXg[sl], g["dX"])
        sum_dA += g["dA"]
        sum_dB += g["dB"]
    for j in blocks:
        Wu_j, B_j, Wd_j, m_j, Hq = blk_ref[j]
        g = oracle.ffn_lora_bwd(X, dYh, Wu_j, A, B_j, Wd_j, m_j, Hq > 0, Uq, 64, 64)
        rows = dBg[j * 64:(j + 1) * 64, :r]
        if m_j.any():
            gate(f"dB block {j} ({int(m_j.sum())} tiles)", rows, g["dB"])
        else:
            assert not rows.any()
    # second call: dY zero outside the sampled tiles
    dY2 = np.zeros_like(dYh)
    for i in tiles:
        dY2[i * 64:(i + 1) * 64] = dYh[i * 64:(i + 1) * 64]
    dX2, dA2, dB2 = backward(dY2)
    gate("dA (sampled tiles)", dA2[:r], sum_dA)
    gate("dB (sampled tiles)", dB2[:, :r], sum_dB)
    untouched = np.ones(T // 64, bool)
    untouched[list(tiles)] = False
    assert not dX2.reshape(T // 64, 64, d)[untouched].any()
    listed = mask[list(tiles)].any(0)
    assert not dB2.reshape(F // 64, 64, 64)[~listed].any()


@pytest.mark.parametrize("Tt,d,F,rows,dtype", [
    (9, 128, 192, 9, "bf16"),       # one tile into the second group of eight
    (64, 64, 192, 64, "f16"),       # the last count that runs by quadrants; one K step
    (65, 192, 128, 65, "bf16"),     # the first that runs by tiles
    (66, 128, 192, 2, "f16"),       # list rows shared by 33 tiles
    (130, 64, 128, 1, "bf16"),
])
def test_lora_token_tile_counts(lx, oracle, Tt, d, F, rows, dtype):
    """U and G on both sides of the count from which a workgroup takes a whole token tile."""
    c = make_case(64 * Tt, d, F, 16, 0.5, 40 + Tt, rows=None if rows == Tt else rows, dtype=dtype)
    got, ref = run_both(lx, oracle, c)
    check(got, ref, f"{Tt} tiles d={d} F={F} rows={rows} {dtype}", dtype=dtype)


# token tiles, d, listed blocks, list rows; the tiles of the two products that carry the low-rank step (checked in
# test_ffn_plan.py)
LORA_TILES = [
    (129, 64, 6, 1, "1x2", "1x1 many"),
    (51, 64, 40, 1, "1x4", "quarters"),
    (103, 64, 9, 1, "2x2", "quarters"),
    (57, 768, 9, 1, "2x2 deep", "1x1 many"),
    (103, 512, 9, 1, "2x4", "2x2 deep"),
    (115, 64, 17, 1, "4x4", "quarters"),
    (42, 1024, 17, 2, "1x4 deep", "1x1 many"),
    (103, 576, 1, 1, "quarters", "2x2"),
    (85, 1536, 1, 1, "quarters", "1x4"),
    (103, 576, 8, 1, "2x2 deep", "2x4"),
    (129, 1024, 1, 1, "1x1", "4x4"),
    (98, 512, 12, 2, "1x1 many", "1x4 deep"),
    (97, 512, 1, 1, "quarters", "1x2"),
    (6, 192, 3, 6, "quarters", "quarters"),
    (21, 512, 17, 1, "1x2", "1x1"),
    (24, 640, 9, 3, "1x1", "1x1"),
]


@pytest.mark.parametrize("Tt,d,Fb,rows,up,dx", LORA_TILES)
def test_lora_every_tile(lx, Tt, d, Fb, rows, up, dx):
    """The low-rank step in every tile, odd token tile counts and short last groups of entries among them, against the
    definitions in float64 (all blocks listed; both sides take the same stored activations and U)."""
    import torch
    T, F, r, dt = 64 * Tt, 64 * Fb, 16, "bf16"
    rng = np.random.default_rng(Tt + d)
    q = lambda *s, std: round_to(rng.standard_normal(s) * std, dt).astype(np.float64)
    X, dY, Wu, Wd = q(T, d, std=1), q(T, d, std=1), q(F, d, std=0.05), q(d, F, std=0.05)
    A, B = np.zeros((64, d)), np.zeros((F, 64))
    A[:r], B[:, :r] = q(r, d, std=1 / np.sqrt(d)), q(F, r, std=0.05)
    d32 = lambda a: dev(a.astype(np.float32), dt)
    Xd, Wud, Wdd, Ad, Bd = (d32(a) for a in (X, Wu, Wd, A, B))
    bl = lx.lx_mask_compact(torch.ones((rows, Fb), dtype=torch.uint8, device="cuda"))
    gt, nb = Tt // rows, Tt * Fb
    blocks = lambda a: np.ascontiguousarray(a.reshape(rows, gt, 64, Fb, 64).transpose(0, 3, 1, 2, 4)).reshape(nb, 64, 64)
    H_act = torch.full(((nb + 1) * 4096,), float("nan"), dtype=Xd.dtype, device="cuda")
    Y, dX = (torch.full_like(Xd, float("nan")) for _ in range(2))
    U = torch.full((T, 64), float("nan"), dtype=Xd.dtype, device="cuda")
    lx.lx_sparse_ffn_lora_fwd(Xd, Wud, Ad, Bd, Wdd, bl, Y, H_act, U)
    torch.cuda.synchronize()
    assert torch.isnan(H_act[nb * 4096:]).all()
    Uo = X @ A.T
    Ho = np.maximum(X @ Wu.T + Uo @ B.T, 0)
    got = dict(U=host(U), H=host(H_act[:nb * 4096]).reshape(nb, 64, 64), Y=host(Y))
    ref = dict(U=Uo, H=blocks(Ho), Y=Ho @ Wd.T)
    Hq, Uq = round_to(Ho.astype(np.float32), dt), round_to(Uo.astype(np.float32), dt)
    H_act[:nb * 4096] = dev(blocks(Hq).reshape(-1), dt)
    Wut, Wdt = lx.lx_ffn_pack_weights(Wud, Wdd)
    ws = torch.empty(lx.lx_sparse_ffn_lora_bwd_workspace_bytes(T, d, F, nb), dtype=torch.uint8, device="cuda")
    dA = torch.full((64, d), float("nan"), dtype=torch.float32, device="cuda")
    dB = torch.full((F, 64), float("nan"), dtype=torch.float32, device="cuda")
    lx.lx_sparse_ffn_lora_bwd(Xd, d32(dY), H_act, dev(Uq, dt), Wut, Wdt, Ad, Bd, bl, dX, dA, dB, ws)
    torch.cuda.synchronize()
    dZ = (dY @ Wd) * (Hq > 0)
    got.update(dX=host(dX), dA=host(dA), dB=host(dB))
    ref.update(dX=dZ @ Wu + (dZ @ B) @ A, dA=(dZ @ B).T @ X, dB=dZ.T @ Uq.astype(np.float64))
    check(got, ref, f"{up} / {dx}")


@pytest.mark.parametrize("dtype,Tt,d,Fb,nnz,rows,by_cap,by_list", CAPACITIES)
def test_lora_capacity_does_not_change_results(lx, dtype, Tt, d, Fb, nnz, rows, by_cap, by_list):
    """The cases of the plain FFN's capacity test with a LoRA branch: same bits in every output."""
    import torch
    T, F, gt = Tt * 64, Fb * 64, Tt // rows
    rng = np.random.default_rng(2000 + Tt)
    mask = np.zeros((rows, Fb), np.uint8)
    for r in mask:
        r[rng.choice(Fb, nnz, replace=False)] = 1
    dt = dev(np.zeros(1, np.float32), dtype).dtype
    g = torch.Generator(device="cuda").manual_seed(Tt)
    mk = lambda *s: (torch.randn(s, device="cuda", generator=g) * 0.1).to(dt)
    X, dY, Wu, Wd, A, B = mk(T, d), mk(T, d), mk(F, d), mk(d, F), mk(64, d), mk(F, 64)
    Wut, Wdt = lx.lx_ffn_pack_weights(Wu, Wd)
    out = []
    for cap in (max(rows * nnz, 1), rows * Fb):
        print(dtype, Tt, d, Fb, nnz, rows, "capacity", cap, flush=True)
        bl = lx.lx_mask_compact(torch.from_numpy(mask).cuda(), nnz_cap=cap)
        H = torch.full(((cap * gt + 1) * 4096,), float("nan"), dtype=dt, device="cuda")
        Y, dX, U = (torch.full((T, n), float("nan"), dtype=dt, device="cuda") for n in (d, d, 64))
        dA, dB = (torch.full(s, float("nan"), device="cuda") for s in ((64, d), (F, 64)))
        ws = torch.empty(lx.lx_sparse_ffn_lora_bwd_workspace_bytes(T, d, F, cap * gt), dtype=torch.uint8, device="cuda")
        lx.lx_sparse_ffn_lora_fwd(X, Wu, A, B, Wd, bl, Y, H, U)
        lx.lx_sparse_ffn_lora_bwd(X, dY, H, U, Wut, Wdt, A, B, bl, dX, dA, dB, ws)
        torch.cuda.synchronize()
        n = rows * nnz * gt * 4096
        assert torch.isnan(H[n:]).all()
        out.append((H[:n], Y, U, dX, dA, dB))
        assert not any(torch.isnan(t).any() for t in out[-1])
    for a, b in zip(*out):
        assert torch.equal(a, b)
