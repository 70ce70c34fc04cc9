"""Attention backward: when the query side and the key side may share a launch, on the host."""
import itertools
import random

import pytest

import attn_plan
from test_gpu_attn_one_launch import CASES, PLACES


@pytest.fixture(scope="module")
def L():
    return attn_plan.load()


def bytes_of(n, stride, row):
    return {sum(i * s for i, s in zip(ix, stride)) + b for ix in itertools.product(*map(range, n)) for b in range(row)}


def test_tensors_meet_against_every_byte(L):
    """Exact for nested dimensions in any order, interleaved tensors among them; otherwise never "apart" by mistake."""
    rng = random.Random(3)
    seen = {True: 0, False: 0}
    for _ in range(400):
        n, row = [rng.randint(1, 4) for _ in range(3)], 8
        stride, span = [0] * 3, row
        for i in rng.sample(range(3), 3):
            stride[i] = span + 8 * rng.choice([0, 0, 1, 2, 5])       # room for other tensors in between
            span = stride[i] * (n[i] - 1) + span
        mine = bytes_of(n, stride, row)
        for delta in {rng.randint(-span - 9, span + 9) for _ in range(6)} | {8 * rng.randint(-span // 8, span // 8) for _ in range(6)}:
            want = not mine.isdisjoint({b + delta for b in mine})
            assert attn_plan.meet(L, n, stride, row, delta) == want, (n, stride, delta)
            seen[want] += 1
    assert min(seen.values()) > 500
    for _ in range(2000):
        n, row = [rng.randint(1, 4) for _ in range(3)], 8
        stride = [8 * rng.randint(0, 12) for _ in range(3)]
        mine = bytes_of(n, stride, row)
        delta = rng.randint(-300, 300)
        if not mine.isdisjoint({b + delta for b in mine}):
            assert attn_plan.meet(L, n, stride, row, delta), (n, stride, delta)


def test_outputs_of_a_packed_buffer_are_apart(L):
    """dQ, dK and dV as the three parts of one [B, S, 3, Hh, D] buffer."""
    B, Hh, S, D = 3, 12, 320, 64
    n, stride, row = (B, Hh, S), (2 * S * 3 * Hh * D, 2 * D, 2 * 3 * Hh * D), 2 * D
    part = 2 * Hh * D
    for k in (1, 2):
        assert not attn_plan.meet(L, n, stride, row, k * part) and not attn_plan.meet(L, n, stride, row, -k * part)
    assert attn_plan.meet(L, n, stride, row, part - 16) and attn_plan.meet(L, n, stride, row, 3 * part)


@pytest.mark.parametrize("place", PLACES)
def test_overlapping_buffers_keep_the_launches_apart(L, place):
    """Every place of test_gpu_attn_one_launch.py: laid out as there, in one arena."""
    B, Hh, S, D = 2, 4, 128, 64
    stats, part = B * Hh * S * 4, B * Hh * S * D * 2
    n, stride, row = (B, Hh, S), (2 * Hh * S * D, 2 * S * D, 2 * D), 2 * D
    names = ["Q", "K", "V", "O", "dO", "dQ", "dK", "dV", "LSE", "row_ptr", "col_idx", "Delta", "NegLse2"]
    base = {k: (1 << 30) + i * (part + (1 << 20)) for i, k in enumerate(names)}
    ask = lambda at: attn_plan.sides_apart(L, n, stride, row, [at[k] for k in names], stats, 4 * (Hh * 2 + 1), 4 * Hh * 4)
    assert ask(base)
    assert not ask(dict(base, **{place[0]: base[place[1]] + place[2]})), place


def test_neighbours_are_not_overlaps(L):
    """Buffers that follow each other without a gap share the launch."""
    B, Hh, S, D = 2, 4, 128, 64
    stats, part = B * Hh * S * 4, B * Hh * S * D * 2
    n, stride, row = (B, Hh, S), (2 * Hh * S * D, 2 * S * D, 2 * D), 2 * D
    at = [(1 << 30) + i * part for i in range(8)]
    at += [at[-1] + part, at[-1] + part + stats]
    at += [at[-1] + 36, at[-1] + 100, at[-1] + 100 + stats]
    assert attn_plan.sides_apart(L, n, stride, row, at, stats, 36, 64)


def test_the_cases_run_as_they_claim(L):
    """test_gpu_attn_one_launch.py compares one launch with two: all its calls are small enough for one."""
    for _, B, Hh, S, D, _, causal, *_ in CASES:
        nb = S // 64
        assert L.pays(D, B * Hh * nb, nb, causal, nb), (B, Hh, S, D)
    assert L.pays(64, 768, 64, 1, 64) and not L.pays(64, 769, 64, 1, 64) and L.pays(64, 1728, 11, 1, 11) and not L.pays(64, 1729, 1, 1, 1)
    assert L.pays(128, 256, 64, 1, 64) and not L.pays(128, 257, 1, 1, 1)


@pytest.mark.parametrize("D,rows,nblk,mean,one", [
    (64, 768, 64, 64, True), (64, 1728, 4, 4, True), (128, 128, 64, 64, True), (128, 192, 4, 4, False), (128, 256, 64, 64, False),
    (128, 256, 64, 6, True), (128, 256, 16, 16, False), (128, 256, 2, 2, True),
])
def test_without_causality_long_lists_run_in_two(L, D, rows, nblk, mean, one):
    """Head size 128, where one launch took up to 1.5 times as long as two."""
    assert bool(L.pays(D, rows, nblk, 0, mean)) == one
