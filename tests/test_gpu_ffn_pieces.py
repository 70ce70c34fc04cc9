"""First product by pieces of lists: every length of a piece and of the longest ones, one round and two, one and two tiles per lane of the
scan, empty, short and full lists, a capacity of every block and one that cuts lists.  Rows are independent, so sampled token tiles
equal, bit for bit, a call that holds that tile alone."""
import random

import numpy as np
import pytest

import ffn_plan
from test_gpu_ffn_deal import lx, test_deals as check_deals  # noqa: F401
from util import dev

# element type, token tiles, d, neuron blocks, capacity, density (the lists' mean is three quarters of that); most entries of a piece
CASES = [
    ("bf16", 50, 3200, 60, 1600, 0.6, 3),     # 2.6 entries per workgroup of a round
    ("f16", 97, 640, 70, 3550, 0.66, 7),
    ("bf16", 64, 320, 110, 3400, 0.6, 6),     # one tile per lane
    ("bf16", 65, 2048, 64, 2400, 0.74, 5),
    ("bf16", 128, 3200, 64, 6700, 0.99, 7),   # two rounds
    ("f16", 127, 704, 48, 2700, 0.5, 5),
    ("bf16", 100, 3264, 48, 4800, 0.2, 2),    # every block as capacity: workgroups that find nothing
    ("f16", 96, 3200, 40, 1650, 0.44, 3),
    ("bf16", 60, 640, 150, 5200, 0.55, 8),
    ("f16", 128, 3200, 80, 8100, 0.99, 8),    # two rounds of the longest pieces
    ("f16", 65, 1024, 64, 2300, 0.56, 4),
    ("bf16", 64, 704, 72, 2300, 0.26, 2),
]


def lengths(Tt, d, Fb, density):
    """Of the lists that the deals' test draws."""
    rng = np.random.default_rng(Tt + d)
    m = (rng.random((Tt, Fb)) < density * rng.uniform(0.3, 1.2, (Tt, 1))).astype(np.uint8)
    m[Tt // 2] = 0
    m[0] = 0
    m[0, Fb // 3] = 1
    return m.sum(axis=1)


@pytest.fixture(scope="module")
def L():
    return ffn_plan.load()


def check_items(L, lens, cap):
    """Every entry within the capacity in one piece, none beyond it; the most entries of a piece, and the lengths that occur."""
    items, per = ffn_plan.even_items(L, lens, cap)
    seen, left = set(), cap
    for tile, first, n in items:
        assert 1 <= n <= per
        new = {(tile, e) for e in range(first, first + n)}
        assert not new & seen
        seen |= new
    for tile, n in enumerate(lens):
        n, left = min(int(n), left), left - min(int(n), left)
        assert {e for t, e in seen if t == tile} == set(range(n)), tile
    assert len(seen) == min(int(sum(lens)), cap)
    return per, {n for _, _, n in items}


def test_cases_have_every_length(L):
    pers, found = [], set()
    for _, Tt, d, Fb, cap, density, per in CASES:
        got, ns = check_items(L, lengths(Tt, d, Fb, density), cap)
        pers.append((got, per))
        found |= ns
    assert all(a == b for a, b in pers), pers
    assert {p for p, _ in pers} == set(range(2, 9)) and found == set(range(1, 9))


def test_every_entry_in_one_piece(L):
    rng = random.Random(5)
    pers = set()
    for _ in range(120):
        Tt, most = rng.randint(1, 128), rng.choice((1, 3, 12, 40, 90, 500))
        lens = [0 if rng.random() < 0.1 else rng.randint(0, most) for _ in range(Tt)]
        total = sum(lens)
        for cap in {total, total + 700, max(1, total // 2), max(1, total - 3)}:
            if cap < 1 << 16:
                pers.add(check_items(L, lens, cap)[0])
    assert pers == set(range(2, 9))
    assert check_items(L, [65535], 65535)[0] == 8       # products beyond 2^22 in the pieces' bounds


@pytest.mark.gpu
@pytest.mark.parametrize("lora", [False, True])
@pytest.mark.parametrize("dtype,Tt,d,Fb,cap,density,per", CASES)
def test_pieces(lx, dtype, Tt, d, Fb, cap, density, per, lora):  # noqa: F811
    check_deals(lx, dtype, Tt, 1, d, Fb, cap, None, None, density, lora)


def test_cases_take_that_route(L):
    for _, Tt, d, Fb, cap, *_ in CASES + [CUT]:
        assert ffn_plan.sdd_by(L, Tt, 1, d, cap, Tt * Fb, 0, cap)[0] == "pieces", (Tt, d, Fb)
        assert ffn_plan.sdd_by(L, Tt, 1, d, cap, Tt * Fb, 1, cap)[0] != "pieces"


# token tiles, d, share of the blocks, room for a tenth more: by pieces or not, for what the rule says of them
RULES = [
    (128, 4096, 0.077, True),
    (74, 3712, 0.077, True),        # pieces of three fill one round: 0.91 - 0.95 of the time
    (63, 3904, 0.111, False),       # of four: 1.05 - 1.10 with lists that have much in common, 0.96 with others
    (58, 3776, 0.111, False),
    (89, 3712, 0.077, False),
    (64, 4096, 0.13, True),
    (116, 4160, 0.111, False),      # the longest pieces in one round: 1.19
    (112, 4992, 0.13, True),        # two rounds
]


@pytest.mark.parametrize("Tt,d,share,by", RULES)
def test_rule(L, Tt, d, share, by):
    Fb = d // 16
    cap = int(1.1 * share * Tt * Fb) + 64
    assert (ffn_plan.sdd_by(L, Tt, 1, d, cap, Tt * Fb, 0, cap)[0] == "pieces") == by


CUT = (None, 100, 640, 60, 2600, 0.8)      # the lists have some 3500 entries


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_lists_beyond_their_capacity(lx, dtype):  # noqa: F811
    """A list cut in the middle and tiles wholly beyond the capacity, with a bias: the bits of the lists without what is cut, and
    nothing written past the capacity."""
    import torch
    _, Tt, d, Fb, cap, density = CUT
    T, F = 64 * Tt, 64 * Fb
    rng = np.random.default_rng(9)
    m = (rng.random((Tt, Fb)) < density * rng.uniform(0.3, 1.2, (Tt, 1))).astype(np.uint8)
    cut = m.copy()
    rr, cc = np.nonzero(m)
    assert cap < len(rr) and 0 < cut[rr[cap]].sum() and rr[cap - 1] == rr[cap] and rr[cap] < Tt - 5
    cut[rr[cap:], cc[cap:]] = 0
    g = torch.Generator(device="cuda").manual_seed(3)
    tdt = dev(np.zeros(1, np.float32), dtype).dtype
    X, dY, Wu, Wd, bu = ((torch.randn(s, device="cuda", generator=g) * a).to(tdt)
                         for s, a in (((T, d), 1.0), ((T, d), 1.0), ((F, d), 0.05), ((d, F), 0.05), ((F,), 0.5)))
    Wut, Wdt = lx.lx_ffn_pack_weights(Wu, Wd)
    lxt = {"bf16": lx.LX_BF16, "f16": lx.LX_F16}[dtype]

    def run(mask):
        bl = lx.lx_mask_compact(torch.from_numpy(mask).cuda(), nnz_cap=cap)
        H = torch.full(((cap + 8) * 4096,), float("nan"), dtype=tdt, device="cuda")
        Y, dX = torch.full_like(X, float("nan")), torch.full_like(X, float("nan"))
        ws = torch.empty(lx.lx_sparse_ffn_bwd_workspace_bytes(lxt, T, d, F, 64, 64, cap, 1), dtype=torch.uint8, device="cuda")
        lx.lx_sparse_ffn_fwd(X, Wu, Wd, bl, 64, 64, Y, H, b_up=bu)
        assert torch.isnan(H[cap * 4096:]).all()
        lx.lx_sparse_ffn_bwd_dx(dY, H, Wu, Wd, bl, 64, 64, dX, ws, W_up_t=Wut, W_down_t=Wdt)
        torch.cuda.synchronize()
        return Y, dX, H[:cap * 4096]

    for a, b in zip(run(m), run(cut)):
        assert torch.isfinite(a.float()).all() and torch.equal(a, b)
    # the bias, on tiles that another kernel runs alone
    lens = m.sum(axis=1)
    Y, _, H = run(m)
    for i in (0, 17, int(lens[:50].argmax())):
        bl = lx.lx_mask_compact(torch.from_numpy(m[i:i + 1]).cuda(), nnz_cap=int(lens[i]))
        h = torch.empty(int(lens[i]) * 4096, dtype=tdt, device="cuda")
        y = torch.empty_like(X[:64])
        lx.lx_sparse_ffn_fwd(X[64 * i:64 * i + 64].contiguous(), Wu, Wd, bl, 64, 64, y, h, b_up=bu)
        at = int(lens[:i].sum()) * 4096
        assert torch.equal(h, H[at:at + h.numel()]) and torch.equal(y, Y[64 * i:64 * i + 64]), i
