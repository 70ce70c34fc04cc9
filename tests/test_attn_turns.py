"""Attention by turns: on the host, that every row of the mask falls to one workgroup and slot and that the ranks even out; on the
GPU, the bits of calls that run so against the same calls with one row per workgroup."""
import random

import numpy as np
import pytest

import attn_plan
from paper_2510_15964_amd import inputs
from test_gpu_attn import lx, run_gpu  # noqa: F401

# batch, heads, tokens, head size, causal, mask per batch entry, density: of an odd and an even number of turns, with cohorts of one and
# of several pairs, the last one partly filled, XCDs with one pair more than others, and pairs that a batch entry's heads do not divide
CASES = [
    (2, 40, 2048, 128, True, False, 0.2),      # five turns
    (7, 30, 576, 64, True, True, 0.3),         # two, 7 x 9 rows a cohort
    (5, 39, 448, 128, True, False, 0.4),       # three, 25 pairs on one XCD and 24 on the others
    (7, 25, 768, 128, False, True, 0.1),
    (4, 24, 1984, 64, True, False, 0.15),
    (1, 40, 4096, 128, True, False, 0.05),     # 64 rows a pair
]
ROOM = {64: (4, 3), 128: (2, 2)}               # workgroups per CU: forward and dQ; dK and dV


@pytest.fixture(scope="module")
def L():
    return attn_plan.load()


def plans(L, B, Hh, S, D):
    return [t for t in (attn_plan.turns(L, B * Hh, S // 64, 256 * n, r) for n in ROOM[D] for r in range(1, 9)) if t]


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
    for pairs, nblk, slots in [(B * Hh, S // 64, 256 * n) for B, Hh, S, D, *_ in CASES for n in ROOM[D]] + \
            [(rng.randint(8, 400), rng.randint(1, 64), 256 * rng.choice((2, 3, 4))) for _ in range(60)]:
        for t in {attn_plan.turns(L, pairs, nblk, slots, r) for r in (1, 2, 4, 8)} - {None}:
            turns, places, cohorts, V, grid = t
            G, taken = V * nblk, set()
            assert turns <= 8 and G <= 64 and grid == 8 * places * G <= slots
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
    for B, Hh, S, D, *_ in CASES:
        assert plans(L, B, Hh, S, D), (B, Hh, S, D)


def test_choice_takes_little_of_the_host(L):
    """Short sequences of many heads, whose calls wait for the host: the choice is no search over the cohorts (200 - 400 ns a
    launch, six times the count of rows per workgroup)."""
    for pairs, nblk, slots, rows in [(320, 2, 512, 2), (700, 1, 512, 1), (320, 3, 512, 2), (330, 4, 1024, 2)]:
        turns, count = (min(f(pairs, nblk, slots, rows) for _ in range(50)) for f in (L.turns_ns, L.rows_ns))
        assert turns <= 2 * count + 10, (pairs, nblk, slots, turns, count)


@pytest.mark.gpu
@pytest.mark.parametrize("B,Hh,S,D,causal,per_batch,density", CASES)
def test_same_bits(lx, B, Hh, S, D, causal, per_batch, density):  # noqa: F811
    c = inputs.attn_blocks(B, Hh, S, D, density, seed=11, dtype="bf16", causal=causal, head_keep=0.9, mask_batch=B if per_batch else 1)
    got = run_gpu(lx, c)
    try:
        lx.lx_attn_set_rows_per_workgroup(1)
        want = run_gpu(lx, c)
    finally:
        lx.lx_attn_set_rows_per_workgroup(0)
    for k in want:
        assert np.array_equal(got[k], want[k], equal_nan=True), k
