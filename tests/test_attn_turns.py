"""Attention by turns: on the host, which launches run so, that every row of the mask falls to one workgroup and slot and that the
ranks even out; on the GPU, the bits of calls that run so against the same calls with one row per workgroup."""
import random

import numpy as np
import pytest

import attn_plan
from paper_2510_15964_amd import inputs
from test_gpu_attn import lx, run_gpu  # noqa: F401
from util import dev, lx_dtype

# batch, heads, tokens, head size, causal, mask per batch entry, density, element type, layout; rows per workgroup by turns of the
# forward, dQ and dK/dV launches (0: not by turns).  Cohorts of one and of several pairs, the last one partly filled, XCDs with
# one pair more than others, pairs that a batch entry's heads do not divide, a single row per pair, 64 of them
CASES = [
    (2, 40, 2048, 128, True, False, 0.2, "bf16", "bhsd", (5, 5, 5)),
    (7, 30, 576, 64, True, True, 0.3, "bf16", "bhsd", (2, 2, 0)),       # 7 x 9 rows a cohort
    (5, 39, 448, 128, True, False, 0.4, "bf16", "bhsd", (3, 3, 3)),     # 25 pairs on one XCD and 24 on the others
    (7, 25, 768, 128, False, True, 0.1, "bf16", "bhsd", (5, 5, 5)),
    (4, 24, 1984, 64, True, False, 0.15, "bf16", "bhsd", (3, 3, 0)),
    (1, 40, 4096, 128, True, False, 0.05, "bf16", "bhsd", (5, 5, 5)),   # 64 rows a pair
    (7, 37, 448, 64, True, True, 0.4, "f16", "bshd", (2, 2, 3)),
    (2, 39, 1216, 64, False, False, 0.3, "bf16", "bshd", (0, 0, 2)),
    (7, 39, 704, 64, True, False, 0.3, "f16", "bhsd", (0, 0, 5)),
    (4, 40, 1600, 64, True, False, 0.1, "bf16", "bshd", (4, 4, 0)),
    (7, 39, 1024, 64, True, False, 0.2, "bf16", "bhsd", (5, 5, 0)),
    (7, 37, 192, 128, False, False, 1.0, "f16", "bshd", (2, 2, 2)),
    (8, 37, 320, 128, True, False, 0.6, "bf16", "bshd", (4, 4, 4)),
    (24, 26, 64, 128, True, True, 0.5, "f16", "bhsd", (2, 2, 2)),       # lists of one block and none
]


@pytest.fixture(scope="module")
def L():
    return attn_plan.load()


def test_ranks_are_permutations_of_even_sums(L):
    for n in range(1, 65):
        for turns in range(2, 9):
            ranks = [[L.rank_in_turn(r, k, n, turns) for r in range(n)] for k in range(turns)]
            assert all(sorted(x) == list(range(n)) for x in ranks)
            sums = [sum(x) for x in zip(*ranks)]
            assert max(sums) - min(sums) <= 1


def test_every_row_once(L):
    """The kernels' arithmetic (RowSet::init_turns), for a cohort's rows in any order of lengths."""
    rng = random.Random(2)
    seen = 0
    for B, Hh, nblk, slots in [(c[0], c[1], c[2] // 64, n) for c in CASES for n in set(attn_plan.SLOTS[c[3]].values())] + \
            [(rng.randint(1, 10), rng.randint(1, 40), rng.randint(1, 64), 256 * rng.choice((2, 3, 4))) for _ in range(2000)]:
        pairs, rows = B * Hh, attn_plan.shape(L, B, Hh, nblk, slots, may_turn=False)[0]
        t = attn_plan.turns(L, pairs, nblk, slots, rows)
        assert (t[0] if t else 0) == attn_plan.shape(L, B, Hh, nblk, slots)[5]
        if t:
            turns, places, cohorts, V, grid = t
            G, taken = V * nblk, set()
            assert turns <= 5 and G <= 64 and grid == 8 * places * G <= slots
            # no cohorts take fewer turns, and no larger ones as few
            least = {v: -(-(-(-(-(-pairs // 8)) // v)) // (slots // 8 // (v * nblk))) for v in range(1, 64 // nblk + 1)}
            assert turns == min(least.values()) and V == max(v for v in least if least[v] == turns)
            for x in range(8):
                order = {}
                for s in range(grid // 8):
                    place, r = s // G, s % G
                    for k in range(turns):
                        number = k * places + place
                        if number >= cohorts:
                            continue
                        c = number + cohorts * x // 8
                        c -= cohorts if c >= cohorts else 0
                        if c not in order:
                            rows = [(x + 8 * (c * V + lane // nblk), lane % nblk) for lane in range(G)]
                            order[c] = rng.sample(rows, G)
                            order[c].sort(key=lambda p: p[0] >= pairs)         # those that there are first
                        row = order[c][L.rank_in_turn(r, k, G, turns)]
                        if row[0] < pairs:
                            assert row not in taken
                            taken.add(row)
            assert len(taken) == pairs * nblk
            seen += 1
    assert seen >= 30


def test_cases_take_that_route(L):
    for c in CASES:
        assert attn_plan.launches(L, *c[:5]) == c[9], c
    for D, k, turns in [(64, 0, {2, 3, 4, 5}), (64, 1, {2, 3, 4, 5}), (64, 2, {2, 3, 5})] + [(128, k, {2, 3, 4, 5}) for k in range(3)]:
        assert {c[9][k] for c in CASES if c[3] == D} >= turns, (D, k)
    for B, Hh, S, D in WIDE:
        assert all(attn_plan.shape(L, B, Hh, S // 64, n)[5] == 2 for n in attn_plan.SLOTS[D].values()), (B, Hh, S, D)


# batch, heads, tokens, head size that run so or not, for what the rule says of them
RULES = [
    (8, 33, 256, 128, (3, 3, 3)),       # 264 workgroups of four rows the other way: CUs with two of them next to CUs with one
    (8, 18, 640, 128, (0, 0, 0)),       # 4, 3 and 3 rows to a workgroup are 3.3 of them: 1.03 - 1.10 of the time by turns
    (5, 38, 1024, 64, (0, 0, 0)),       # three workgroups to every CU: 1.07 - 1.09
    (7, 39, 640, 128, (0, 0, 0)),       # six rows, several rounds otherwise: 1.06 - 1.08
    (8, 40, 128, 128, (0, 0, 0)),       # two rows either way
    (3, 29, 1600, 64, (0, 0, 0)),       # three rows either way: 1.17
    (2, 40, 2048, 64, (0, 0, 0)),
]


@pytest.mark.parametrize("B,Hh,S,D,turns", RULES)
def test_rule(L, B, Hh, S, D, turns):
    assert attn_plan.launches(L, B, Hh, S, D, True) == turns


def test_choice_takes_little_of_the_host(L):
    """Short sequences of many heads, whose calls wait for the host: the choice is no search over the cohorts (200 - 400 ns a
    launch, six times the count of rows per workgroup)."""
    for pairs, nblk, slots, rows in [(320, 2, 512, 2), (700, 1, 512, 1), (320, 3, 512, 2), (330, 4, 1024, 2)]:
        turns, count = (min(f(pairs, nblk, slots, rows) for _ in range(50)) for f in (L.turns_ns, L.rows_ns))
        assert turns <= 2 * count + 10, (pairs, nblk, slots, turns, count)


def same(a, b):
    for k in b:
        assert np.array_equal(a[k], b[k], equal_nan=True), k


def both_ways(lx, call):  # noqa: F811
    got = call()
    try:
        lx.lx_attn_set_rows_per_workgroup(1)
        same(got, call())
    finally:
        lx.lx_attn_set_rows_per_workgroup(0)
    return got


@pytest.mark.gpu
@pytest.mark.parametrize("B,Hh,S,D,causal,per_batch,density,dtype,layout,turns", CASES)
def test_same_bits(lx, B, Hh, S, D, causal, per_batch, density, dtype, layout, turns):  # noqa: F811
    c = inputs.attn_blocks(B, Hh, S, D, density, seed=11, dtype=dtype, causal=causal, head_keep=0.9, mask_batch=B if per_batch else 1)
    got = both_ways(lx, lambda: run_gpu(lx, c, layout))
    assert all(np.isfinite(got[k]).all() for k in ("O", "dQ", "dK", "dV"))


def run_lists(lx, c, rows, cols, new):  # noqa: F811
    """Both calls on the given lists; new(): an uninitialised tensor of the call's shape."""
    import torch
    Q, K, V, dO, O, dQ, dK, dV = (new(i) for i in range(8))
    for t, k in ((Q, "Q"), (K, "K"), (V, "V"), (dO, "dO")):
        t.copy_(dev(c[k], c["dtype"]))
    for t in (O, dQ, dK, dV):
        t.fill_(float("nan"))
    B, Hh, S, D = Q.shape
    LSE = torch.full((B, Hh, S), float("nan"), device="cuda")
    ws = torch.empty(lx.lx_sparse_attn_bwd_workspace_bytes(lx_dtype(lx, c["dtype"]), B, Hh, S, D), dtype=torch.uint8, device="cuda")
    lx.lx_sparse_attn_fwd(Q, K, V, rows, c["scale"], c["causal"], O, LSE)
    lx.lx_sparse_attn_bwd_dx(Q, K, V, O, LSE, dO, rows, cols, c["scale"], c["causal"], dQ, dK, dV, ws)
    torch.cuda.synchronize()
    return {k: t.float().cpu().numpy() for k, t in (("O", O), ("LSE", LSE), ("dQ", dQ), ("dK", dK), ("dV", dV))}


@pytest.mark.gpu
@pytest.mark.parametrize("cut", [False, True])
def test_pattern_lists_and_cut_ones(lx, cut):  # noqa: F811
    """Lists combined from a pool, a head without a pattern among them; lists longer than their capacity, where some rows lose a
    part and others all of their entries."""
    import torch
    B, Hh, S, D = 5, 39, 448, 128
    c = inputs.attn_blocks(B, Hh, S, D, 0.5, seed=12, dtype="f16")
    if cut:
        lists = [lx.lx_mask_compact(torch.from_numpy(c["mask"]).cuda(), transpose=t, nnz_cap=int(0.6 * c["mask"].sum())) for t in (False, True)]
        assert any(lengths(x, x.nnz_cap) != lengths(x, 1 << 30) for x in lists)
    else:
        pool = lx.lx_mask_compact_pair(torch.from_numpy(np.ascontiguousarray(inputs.pattern_pool(S // 64, seed=3, causal=True))).cuda())
        hp = torch.from_numpy(np.random.default_rng(4).integers(-1, 8, Hh).astype(np.int32)).cuda()
        lists = lx.lx_attn_combine_patterns(pool[0], pool[1], S // 64, hp)
    both_ways(lx, lambda: run_lists(lx, c, *lists, lambda i: torch.empty((B, Hh, S, D), dtype=torch.float16, device="cuda")))


def lengths(bl, cap):
    p = np.minimum(bl.row_ptr.cpu().numpy(), cap)
    return (p[1:] - p[:-1]).tolist()


WIDE = [(24, 26, 64, 128), (36, 30, 64, 64)]      # batch, heads, tokens, head size


@pytest.mark.gpu
@pytest.mark.parametrize("B,Hh,S,D", WIDE)
def test_long_token_strides(lx, B, Hh, S, D):  # noqa: F811
    """The kernels with 64-bit addresses by turns: the bits of the same call on contiguous tensors."""
    import torch
    c = inputs.attn_blocks(B, Hh, S, D, 0.6, seed=13, dtype="bf16")
    rows, cols = lx.lx_mask_compact_pair(torch.from_numpy(c["mask"]).cuda())
    n, ss = B * Hh * D, 1 << 25
    torch.cuda.empty_cache()
    buf = torch.empty((S - 1) * ss + 8 * n, dtype=torch.bfloat16, device="cuda")
    wide = both_ways(lx, lambda: run_lists(lx, c, rows, cols, lambda i: buf.as_strided((B, Hh, S, D), (Hh * D, D, ss, 1), i * n)))
    same(wide, run_lists(lx, c, rows, cols, lambda i: torch.empty((B, Hh, S, D), dtype=torch.bfloat16, device="cuda")))
    del buf
    torch.cuda.empty_cache()
