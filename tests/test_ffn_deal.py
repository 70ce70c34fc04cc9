"""How launches with lists per group of token tiles deal their work to workgroups, on the host."""
import ctypes as C
import os
import subprocess

import pytest

from test_gpu_ffn_deal import CASES, THIN

HERE = os.path.dirname(os.path.abspath(__file__))
BY_CHUNK, BY_RANK, UNRANKED = range(3)


@pytest.fixture(scope="module")
def L(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp("deal") / "deal.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Wno-unknown-pragmas", "-shared", "-fPIC",
                    os.path.join(HERE, "ffn_deal_shim.cpp"), "-o", lib], check=True)
    return C.CDLL(lib)


@pytest.mark.parametrize("order", [BY_CHUNK, BY_RANK, UNRANKED])
def test_every_unit_has_one_workgroup(L, order):
    for GM in [1, 2, 3, 7, 8, 31, 32, 33, 49, 64, 100, 127, 128, 129, 200]:
        for GN in [1, 2, 3, 4, 5, 7, 8, 9, 13, 16, 17, 20, 80]:
            units = [L.unit_of(order, GM, GN, w) for w in range((GM * GN + 7) // 8 * 8)]
            got = sorted(u for u in units if u >= 0)
            assert got == list(range(GM * GN)), (GM, GN)


def test_parts_of_a_chunk_get_long_and_short_lists(L):
    """Lengths that fall linearly with the rank: no XCD has more than 1.1 times the mean (from 32 units on)."""
    for GM in (32, 49, 64, 100, 128):
        for GN in (1, 3, 5, 9, 13, 20):
            if GM * GN < 256:
                continue
            load = [0.0] * 8
            for w in range((GM * GN + 7) // 8 * 8):
                u = L.unit_of(BY_CHUNK, GM, GN, w)
                if u >= 0:
                    load[w % 8] += 1.5 - u % GM / GM
            assert max(load) <= 1.1 * sum(load) / 8, (GM, GN, load)


def test_quotients(L):
    for b in [1, 2, 3, 5, 7, 63, 64, 65, 127, 128, 1000, 4095, 99991]:
        for a in list(range(0, 3000)) + [b * k + e for k in (1, 2, 63, 1000) for e in (-1, 0, 1)] + [(1 << 22) - 1, 1 << 22, (1 << 30) + 7]:
            assert L.quick(a, b) == a // b, (a, b)


def test_labels_of_the_gpu_cases(L):
    for _, Tt, gt, d, Fb, cap, lean, order, _ in CASES + THIN:
        assert (L.lean_of(Tt, gt, d, Fb, cap), L.order_of(Tt, gt, d, Fb, cap)) == (lean, order), (Tt, gt, d, Fb)
    assert {c[6] for c in CASES} == {0, 1, 2, 3} and {c[7] for c in CASES} == {BY_CHUNK, BY_RANK, UNRANKED}


# token tiles, d, share of the blocks: bit 1 of lean_of, order (F = 4 d, capacity: a tenth more than the mean)
RULES = [
    (128, 4096, 0.08, 2, BY_CHUNK), (128, 4096, 0.2, 0, BY_RANK), (96, 4096, 0.2, 0, BY_RANK), (81, 4096, 0.4, 0, BY_RANK),
    (81, 4096, 0.05, 2, BY_CHUNK), (128, 2048, 0.11, 2, BY_CHUNK), (96, 2048, 1.0, 2, BY_CHUNK), (128, 2048, 0.9, 0, BY_RANK),
    (96, 768, 0.2, 0, BY_RANK), (64, 1280, 0.1, 0, BY_RANK), (128, 3200, 0.2, 0, BY_CHUNK), (64, 5120, 0.2, 0, BY_CHUNK),
]


@pytest.mark.parametrize("Tt,d,share,lean,order", RULES)
def test_deals_where_the_other_one_was_slower(L, Tt, d, share, lean, order):
    Fb = 4 * d // 64
    cap = min(Tt * Fb, int(1.1 * share * Tt * Fb) + 64)
    assert (L.lean_of(Tt, 1, d, Fb, cap) & 2, L.order_of(Tt, 1, d, Fb, cap)) == (lean, order)


def test_first_products_of_thin_lists_take_whole_ones(L):
    """Lists of 6 - 10 entries in the mean, where halves were up to 1.13 times as slow; not the longer ones."""
    for Tt, mean in ((64, 6), (96, 7), (64, 10), (128, 10)):
        assert not L.halves_of(Tt, 1, 2048, 128, int(1.1 * mean * Tt) + 64), (Tt, mean)
    for Tt, mean in ((64, 13), (96, 13), (128, 14), (64, 50)):
        assert L.halves_of(Tt, 1, 2048, 128, int(1.1 * mean * Tt) + 64), (Tt, mean)
    assert {L.halves_of(*c[1:6]) for c in CASES} == {0, 1}
    assert not any(L.halves_of(*c[1:6]) for c in THIN)
