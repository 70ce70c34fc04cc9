"""GPU: the FFN products at the edges of their tiles with ONE list row for all token tiles: odd numbers
of token tiles (the last group of two or four is short), column counts that are no multiple of a
workgroup's columns, lists around 64 entries (they are fetched 64 at a time) and cut lists."""
import numpy as np
import pytest

from paper_2510_15964_amd import inputs
from util import FRO, TOL, dev, host, lx_dtype, rel_err_fro, rel_err_max, round_to

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lx():
    import torch
    assert torch.cuda.is_available()
    from paper_2510_15964_amd import lx
    return lx


EDGES = [
    ("bf16", 1, 64, 3, 1, False),        # one tile, one column chunk, one block
    ("bf16", 3, 320, 8, 5, True),        # short groups of two and four, columns short of 128 and 256
    ("f16", 7, 192, 70, 63, False),      # one entry short of a fetch
    ("bf16", 5, 448, 70, 64, False),
    ("bf16", 9, 128, 70, 65, True),      # one entry into the second fetch
    ("f16", 2, 576, 140, 129, False),
    ("bf16", 61, 128, 16, 9, False),     # many workgroups, ragged groups of entries
    ("bf16", 103, 512, 12, 9, True),     # 2 x 4 tiles in the first product, short last groups on both sides
    ("bf16", 103, 576, 12, 8, False),    # 2 x 4 tiles in the second, columns short of a workgroup's
    ("f16", 86, 1536, 3, 1, False),      # 2 x 2 tiles, eight wavefronts
    ("bf16", 21, 512, 40, 37, False),
]


@pytest.mark.parametrize("dtype,Tt,d,Fb,nnz,bias", EDGES)
def test_tile_edges(lx, oracle, dtype, Tt, d, Fb, nnz, bias):
    """Every number of token tiles per workgroup gives the same bits; sampled tiles match the oracle."""
    import torch
    T, F = Tt * 64, Fb * 64
    c = inputs.ffn_bernoulli(T, d, F, 64, 64, 0.5, 700 + nnz, dtype=dtype, w_std=0.05)
    rng = np.random.default_rng(nnz)
    row = np.zeros((1, Fb), np.uint8)
    row[0, rng.choice(Fb, nnz, replace=False)] = 1
    b_up = round_to(rng.standard_normal(F) * 0.1, dtype) if bias else None
    b_down = round_to(rng.standard_normal(d), dtype) if bias else None
    X, Wu, Wd, dY = (dev(c[k], dtype) for k in ("X", "W_up", "W_down", "dY"))
    bu, bd = (dev(b, dtype) if bias else None for b in (b_up, b_down))
    bl = lx.lx_mask_compact(torch.from_numpy(row).cuda(), nnz_cap=nnz)
    Wut, Wdt = lx.lx_ffn_pack_weights(Wu, Wd)
    ws = torch.empty(lx.lx_sparse_ffn_bwd_workspace_bytes(lx_dtype(lx, dtype), T, d, F, 64, 64, nnz * Tt, 1) + 256,
                     dtype=torch.uint8, device="cuda")

    def run(tiles):
        print(dtype, Tt, d, Fb, nnz, "tiles per workgroup", tiles, flush=True)
        lx.lx_ffn_set_token_tiles_per_workgroup(tiles)
        try:
            H = torch.full(((nnz * Tt + 1) * 4096,), float("nan"), dtype=X.dtype, device="cuda")
            Y, dX = (torch.full((T + 64, d), float("nan"), dtype=X.dtype, device="cuda") for _ in range(2))
            lx.lx_sparse_ffn_fwd(X, Wu, Wd, bl, 64, 64, Y[:T], H, b_up=bu, b_down=bd)
            lx.lx_sparse_ffn_bwd_dx(dY, H, Wu, Wd, bl, 64, 64, dX[:T], ws, W_up_t=Wut, W_down_t=Wdt)
            torch.cuda.synchronize()
        finally:
            lx.lx_ffn_set_token_tiles_per_workgroup(0)
        for t, end in ((H, nnz * Tt * 4096), (Y, T), (dX, T)):
            assert torch.isnan(t[end:]).all() and not torch.isnan(t[:end]).any()
        return H[:nnz * Tt * 4096], Y[:T], dX[:T]

    ref = run(1)
    for tiles in (2, 4, 0):
        for a, b in zip(run(tiles), ref):
            assert torch.equal(a, b), tiles
    act = host(ref[0]).reshape(nnz, Tt, 64, 64)
    for i in sorted({0, Tt // 2, Tt - 1}):
        sl = slice(i * 64, (i + 1) * 64)
        _, Yo = oracle.ffn_fwd(c["X"][sl], c["W_up"], c["W_down"], row, 64, 64, b_up, b_down)
        gate = np.zeros((64, F), bool)
        gate.reshape(64, Fb, 64)[:, np.flatnonzero(row[0])] = (act[:, i] > 0).transpose(1, 0, 2)
        _, dXo = oracle.ffn_bwd_dx(c["dY"][sl], c["W_up"], c["W_down"], row, gate, 64, 64)
        for g, r in ((host(ref[1][sl]), Yo), (host(ref[2][sl]), dXo)):
            assert rel_err_max(g, r) <= TOL[dtype] and rel_err_fro(g, r) <= FRO[dtype]


CUT = [(65, 1024, 33), (65, 4352, 33)]


@pytest.mark.parametrize("Tt,d,nnz", CUT)
def test_cut_lists(lx, Tt, d, nnz):
    """With room for partial sums the lists of the last round may be cut (with four tiles per workgroup, or two and four, here):
    equal to the uncut call to rounding."""
    import torch
    T, F = Tt * 64, 64 * 64
    g = torch.Generator(device="cuda").manual_seed(nnz)
    mk = lambda *s: (torch.randn(s, device="cuda", generator=g) * 0.05).to(torch.bfloat16)
    X, Wu, Wd = mk(T, d), mk(F, d), mk(d, F)
    row = torch.zeros((1, 64), dtype=torch.uint8, device="cuda")
    row[0, torch.randperm(64, device="cuda", generator=g)[:nnz]] = 1
    bl = lx.lx_mask_compact(row, nnz_cap=nnz)
    H = torch.zeros((nnz * Tt * 4096,), dtype=X.dtype, device="cuda")
    out = []
    for tiles in (0, 2, 4):
        lx.lx_ffn_set_token_tiles_per_workgroup(tiles)
        try:
            for nbytes in (0, lx.lx_sparse_ffn_split_workspace_bytes(lx.LX_BF16, T, d, 64, bl)):
                print(Tt, d, nnz, "tiles", tiles, "partial sums", nbytes, flush=True)
                ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda") if nbytes else None
                Y = torch.full_like(X, float("nan"))
                lx.lx_sparse_ffn_fwd(X, Wu, Wd, bl, 64, 64, Y, H, workspace=ws)
                torch.cuda.synchronize()
                out.append(Y.float())
        finally:
            lx.lx_ffn_set_token_tiles_per_workgroup(0)
    for Y in out[1:]:
        assert torch.isfinite(Y).all()
        assert (Y - out[0]).norm() <= 1e-3 * out[0].norm()
        assert (Y - out[0]).abs().max() <= 2 ** -7 * out[0].abs().max()


# dtype, token tiles, d, neuron blocks, listed blocks per list row, list rows; the first product's tile by the
# capacity of every block and by the list (checked in test_ffn_plan.py)
CAPACITIES = [
    ("bf16", 24, 64, 96, 1, 1, "4x4", "1x1"),
    ("f16", 61, 64, 48, 5, 1, "4x4", "1x2"),
    ("bf16", 24, 64, 96, 24, 1, "4x4", "2x2 deep"),
    ("bf16", 25, 64, 96, 48, 1, "4x4", "2x4"),
    ("bf16", 48, 1024, 96, 48, 1, "2x4", "4x4"),
    ("bf16", 24, 64, 96, 0, 1, "4x4", "1x1"),          # nothing listed
    ("bf16", 18, 512, 48, 24, 1, "2x2 deep", "1x2"),
    ("f16", 13, 64, 96, 45, 1, "2x2", "1x2"),
    ("bf16", 18, 64, 96, 48, 2, "1x4", "1x2"),
    ("bf16", 18, 1024, 48, 24, 2, "1x4 deep", "1x2"),
    ("f16", 60, 64, 48, 12, 3, "4x4", "2x2 deep"),
    ("bf16", 8, 1024, 96, 1, 8, "1x4 deep", "1x1"),
    ("bf16", 60, 64, 24, 5, 60, "1x4", "1x1"),
    ("bf16", 60, 512, 48, 24, 60, "1x2", "1x4"),
    ("f16", 42, 1024, 17, 17, 2, "1x4 deep", "1x4 deep"),   # every block listed
    ("bf16", 50, 1024, 12, 12, 2, "1x1 many", "1x1 many"),
    # with the exact capacity a kernel of one tile runs, with every block as capacity one that chooses: the same tile
    ("bf16", 40, 64, 24, 23, 2, "1x2", "1x2"),
    ("f16", 40, 512, 24, 23, 2, "2x2 deep", "2x2 deep"),
    ("bf16", 36, 64, 48, 33, 3, "2x2", "2x2"),
    ("bf16", 108, 512, 12, 11, 3, "2x4", "2x4"),
    ("f16", 72, 64, 48, 33, 3, "4x4", "4x4"),
    ("bf16", 72, 64, 24, 17, 24, "1x4", "1x4"),
    ("bf16", 66, 1024, 12, 11, 66, "1x4 deep", "1x4 deep"),
    ("bf16", 26, 1024, 8, 5, 1, "1x1", "1x1"),
]


@pytest.mark.parametrize("dtype,Tt,d,Fb,nnz,rows,by_cap,by_list", CAPACITIES)
def test_capacity_does_not_change_results(lx, dtype, Tt, d, Fb, nnz, rows, by_cap, by_list):
    """A list handed over with room for every block may run by another tile, or another kernel of the same tile, than
    with its exact capacity: same bits."""
    import torch
    T, F, gt = Tt * 64, Fb * 64, Tt // rows
    rng = np.random.default_rng(1000 + Tt)
    mask = np.zeros((rows, Fb), np.uint8)
    for r in mask:
        r[rng.choice(Fb, nnz, replace=False)] = 1
    dt = dev(np.zeros(1, np.float32), dtype).dtype
    g = torch.Generator(device="cuda").manual_seed(Tt)
    mk = lambda *s: (torch.randn(s, device="cuda", generator=g) * 0.1).to(dt)
    X, dY, Wu, Wd = mk(T, d), mk(T, d), mk(F, d), mk(d, F)
    Wut, Wdt = lx.lx_ffn_pack_weights(Wu, Wd)
    out = []
    for cap in (max(rows * nnz, 1), rows * Fb):
        print(dtype, Tt, d, Fb, nnz, rows, "capacity", cap, flush=True)
        bl = lx.lx_mask_compact(torch.from_numpy(mask).cuda(), nnz_cap=cap)
        H = torch.full(((cap * gt + 1) * 4096,), float("nan"), dtype=dt, device="cuda")
        Y, dX = (torch.full((T + 64, d), float("nan"), dtype=dt, device="cuda") for _ in range(2))
        ws = torch.empty(lx.lx_sparse_ffn_bwd_workspace_bytes(lx_dtype(lx, dtype), T, d, F, 64, 64, cap * gt, 1),
                         dtype=torch.uint8, device="cuda")
        lx.lx_sparse_ffn_fwd(X, Wu, Wd, bl, 64, 64, Y[:T], H)
        lx.lx_sparse_ffn_bwd_dx(dY, H, Wu, Wd, bl, 64, 64, dX[:T], ws, W_up_t=Wut, W_down_t=Wdt)
        torch.cuda.synchronize()
        n = rows * nnz * gt * 4096
        assert torch.isnan(H[n:]).all() and torch.isnan(Y[T:]).all() and torch.isnan(dX[T:]).all()
        assert not any(torch.isnan(t).any() for t in (H[:n], Y[:T], dX[:T]))
        out.append((H[:n], Y[:T], dX[:T]))
    for a, b in zip(*out):
        assert torch.equal(a, b)


# token tiles, d, listed blocks; the second product's tile and the pieces its last lists are cut into
CUT_BY_TILE = [(65, 256, 129, "2x2", 3), (130, 192, 129, "2x4", 3), (16, 4352, 128, "4x4", 3)]


@pytest.mark.parametrize("Tt,d,nnz,tile,pieces", CUT_BY_TILE)
def test_cut_lists_by_tile(lx, Tt, d, nnz, tile, pieces):
    """The reduction of every tile that cuts lists: equal to the uncut call to the rounding of fp32 sums."""
    import torch
    T, F = Tt * 64, nnz * 64
    g = torch.Generator(device="cuda").manual_seed(nnz)
    mk = lambda *s: (torch.randn(s, device="cuda", generator=g) * 0.05).to(torch.bfloat16)
    X, Wu, Wd = mk(T, d), mk(F, d), mk(d, F)
    bl = lx.lx_mask_compact(torch.ones((1, nnz), dtype=torch.uint8, device="cuda"))
    H = torch.zeros((nnz * Tt * 4096,), dtype=X.dtype, device="cuda")
    nbytes = lx.lx_sparse_ffn_split_workspace_bytes(lx.LX_BF16, T, d, 64, bl)
    assert nbytes > 0
    out = []
    for n in (0, nbytes):
        ws = torch.empty(n, dtype=torch.uint8, device="cuda") if n else None
        Y = torch.full_like(X, float("nan"))
        lx.lx_sparse_ffn_fwd(X, Wu, Wd, bl, 64, 64, Y, H, workspace=ws)
        torch.cuda.synchronize()
        out.append(Y.float())
    assert torch.isfinite(out[1]).all()
    assert (out[1] - out[0]).norm() <= 1e-3 * out[0].norm()              # few elements round the other way
    assert (out[1] - out[0]).abs().max() <= 2 ** -7 * out[0].abs().max()  # and by one unit of bf16 at most
