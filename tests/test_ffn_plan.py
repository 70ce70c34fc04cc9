"""The tile rules of the 16-bit FFN products, on the host: the choice by the list's length against the choice by its
capacity, and that the GPU tests reach every kernel and every tile, by the route that the launchers take."""
import random

import pytest

import ffn_plan
from ffn_plan import TILES
from test_gpu_ffn_tiles import CAPACITIES, CUT, CUT_BY_TILE, EDGES
from test_gpu_ffn_quarter import CASES as QUARTERS
from test_gpu_lora import LORA_TILES
from test_gpu_lora_grads import CASES as GRADS
from test_gpu_predict_quarter import CASES as PREDICT, tiles_beyond


@pytest.fixture(scope="module")
def L():
    return ffn_plan.load()


# token tiles, d, neuron blocks, listed blocks (one list for all tiles): a tenth of the neurons of OPT layers
SHARED = [(64, 2048, 128, 14), (128, 2048, 128, 14), (32, 2560, 160, 20), (16, 4096, 256, 26), (128, 4096, 256, 28),
          (61, 5120, 320, 32)]


@pytest.mark.parametrize("Tt,d,Fb,n", SHARED)
def test_first_product_survives_a_loose_capacity(L, Tt, d, Fb, n):
    """Twice, four times and every block as capacity: by the model at most 15 % slower than with the exact one.  (By
    the capacity's tile it was up to 2.5 times.)"""
    us = lambda tile: L.sdd_us(tile, Tt, Tt, d, n)
    exact = us(L.sdd_tile(Tt, Tt, d, n, Fb, 0, n))
    worst = 0.0
    for cap in (2 * n, 4 * n, Fb):
        assert us(L.sdd_tile(Tt, Tt, d, cap, Fb, 0, n)) <= 1.15 * exact, cap
        worst = max(worst, us(L.sdd_tile_of_capacity(Tt, Tt, d, cap, 0)) / exact)
    print(Tt, d, n, "capacity's tile", worst)


def test_items_always_fit_the_launch(L):
    """Whatever the sizes, capacity, length and knob: the tile that a kernel picks needs no more workgroups than were
    launched, and an exact capacity's own tile is kept."""
    rng = random.Random(5)
    for _ in range(20000):
        rows = rng.choice([1, rng.randint(1, 40)])
        gt = rng.choice([1, rng.randint(1, 40)])
        Tt, d, Fb, want = rows * gt, 64 * rng.randint(1, 80), rng.randint(1, 320), rng.choice([0, 0, 1, 2, 4])
        blocks = rows * Fb
        cap = rng.choice([blocks, rng.randint(1, blocks)])
        n = rng.randint(0, cap)
        tile = L.sdd_tile(Tt, gt, d, cap, blocks, want, n)
        assert L.sdd_needed(tile, Tt, gt, n) <= L.sdd_launched(Tt, gt, d, cap, blocks, want), (Tt, gt, d, Fb, cap, n)
        assert L.sdd_tile(Tt, gt, d, cap, blocks, want, cap) == L.sdd_tile_of_capacity(Tt, gt, d, cap, want)


def test_labels_of_the_gpu_cases(L):
    for _, Tt, d, Fb, nnz, rows, by_cap, by_list in CAPACITIES:
        gt, blocks = Tt // rows, rows * Fb
        got = (TILES[L.sdd_tile_of_capacity(Tt, gt, d, blocks, 0)], TILES[L.sdd_tile(Tt, gt, d, blocks, blocks, 0, rows * nnz)])
        assert got == (by_cap, by_list), (Tt, d, Fb, nnz, rows, got)
    for Tt, d, nnz, tile, pieces in CUT_BY_TILE:
        assert ffn_plan.dsd_by(L, Tt, Tt, d, 64 * nnz, nnz, 1 << 40) == ("tile", tile, pieces), (Tt, d, nnz)
        assert ffn_plan.dsd_by(L, Tt, Tt, d, 64 * nnz, nnz)[2] == 1
    # (no partial sums: the uncut call) four tiles per workgroup cut either, two the wider one
    cut = [[ffn_plan.dsd_by(L, Tt, Tt, d, 64 * 64, nnz, 1 << 40, want)[2] > 1 for want in (2, 4)] for Tt, d, nnz in CUT]
    assert cut == [[False, True], [True, True]]
    for Tt, d, Fb, rows, up, dx in LORA_TILES:
        gt, cap = Tt // rows, rows * Fb
        first, second = ffn_plan.sdd_by(L, Tt, gt, d, cap, cap, 0, cap), ffn_plan.dsd_by(L, Tt, gt, d, 64 * Fb, cap)
        assert (first[1] or first[0], second[1] or second[0]) == (up, dx), (Tt, d, Fb, rows)


def test_gpu_cases_reach_every_tile(L):
    """First product, with and without the low-rank step: the cases of the two capacity tests, by a kernel of every tile
    alone and by the kernels that choose among a set.  Second product: test_tile_edges (the library's choice and every
    knob value) and the capacity test; with the low-rank step test_lora_every_tile, which holds both products against
    the definitions; the reductions: test_cut_lists_by_tile.  (Quarters, mixed launches and tiles of one stage have tests of
    their own.)"""
    alone, chosen, down = set(), set(), set()
    for _, Tt, d, Fb, nnz, rows, _, _ in CAPACITIES:
        for cap in (max(rows * nnz, 1), rows * Fb):
            gt = Tt // rows
            route, tile = ffn_plan.sdd_by(L, Tt, gt, d, cap, rows * Fb, 0, rows * nnz)
            if route == "tile":
                alone.add(tile)
            elif route == "set":
                own = L.sdd_tile_of_capacity(Tt, gt, d, cap, 0)
                chosen.add(("narrow" if TILES[own] in ("2x2", "1x4", "1x2", "1x1") else "wide", tile))
            route, tile, _ = ffn_plan.dsd_by(L, Tt, gt, d, 64 * Fb, cap)
            if route == "tile":
                down.add(tile)
    for _, Tt, d, Fb, nnz, _ in EDGES:
        for want in (0, 1, 2, 4):
            route, tile, _ = ffn_plan.dsd_by(L, Tt, Tt, d, 64 * Fb, nnz, 0, want)
            if route == "tile":
                down.add(tile)
    every = set(TILES)
    assert alone == every, every - alone
    sets = ({("wide", t) for t in ("4x4", "2x4", "2x2 deep", "1x4 deep", "1x2", "1x1")} |
            {("narrow", t) for t in ("2x2", "1x4", "1x2", "1x1")})
    assert chosen == sets, sets - chosen
    assert down == every, every - down
    assert {c[4] for c in LORA_TILES} == every | {"quarters"} and {c[5] for c in LORA_TILES} == every | {"quarters"}
    assert {c[3] for c in CUT_BY_TILE} == {"4x4", "2x4", "2x2"}


def test_lora_gradients_by_quadrants(L):
    """The GPU cases but the first run so; not a single tile, nor where quadrants were the slower ones at any density."""
    assert [L.grads_by_quads(Tt, d, F) for Tt, d, F, *_ in GRADS] == [0] + [1] * (len(GRADS) - 1)
    for Tt, d in ((2, 5120), (8, 1024), (32, 768), (64, 2048), (16, 5120), (32, 3200)):
        assert L.grads_by_quads(Tt, d, 4 * d), (Tt, d)
    for Tt, d in ((1, 768), (1, 5120), (24, 5120), (48, 3200), (65, 768)):
        assert not L.grads_by_quads(Tt, d, 4 * d), (Tt, d)


def test_cases_of_the_quarters(L):
    """test_gpu_ffn_quarter.py compares quarters with one token tile per workgroup asked for, and test_gpu_predict_quarter.py
    with a call of more tiles."""
    for _, Tt, gt, d, Fb, n, slack in QUARTERS:
        rows = Tt // gt
        nnz = rows * n if n is not None else sum(2 * i for i in range(rows))
        by = lambda want: (ffn_plan.sdd_by(L, Tt, gt, d, nnz + slack, rows * Fb, want, nnz)[0],
                           ffn_plan.dsd_by(L, Tt, gt, d, 64 * Fb, nnz + slack, 0, want)[0])
        assert by(0) == ("quarters", "quarters") and "quarters" not in by(1), (Tt, d, Fb)
    for Tt, d, nblk in PREDICT:
        assert d % 128 and L.predict_quarters(Tt * nblk // 64, d) and not L.predict_quarters(2 * tiles_beyond(Tt, nblk) * nblk // 64, d)
