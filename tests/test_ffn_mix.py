"""Launches with one list row, wide tiles and a rest by narrower ones: who computes what, on the host."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

from ffn_plan import TILES
from test_gpu_ffn_mix import CASES, DOWN

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def L(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp("mix") / "mix.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Wno-unknown-pragmas", "-shared", "-fPIC",
                    os.path.join(HERE, "ffn_mix_shim.cpp"), "-o", lib], check=True)
    return C.CDLL(lib)


@pytest.mark.parametrize("Tt", [4, 5, 33, 61, 62, 63, 64, 97, 116, 128, 250])
def test_every_block_has_one_workgroup(L, Tt):
    seen, out = set(), (C.c_int * 4)()
    for n in list(range(1, 200, 3)) + [512, 1000, 1279]:
        tail = L.mix_tail(Tt, n)
        if tail == -2:
            continue
        seen.add(tail)
        grid, got = L.mix_grid(Tt, n), np.zeros((Tt + 4, n + 4), int)
        for w in range(grid + 64):
            if L.mix_item(Tt, n, w, out):
                assert w < grid and out[0] < Tt and out[2] < n
                got[out[0]:out[0] + out[1], out[2]:out[2] + out[3]] += 1
        assert (got[:Tt, :n] == 1).all(), (Tt, n)
    assert Tt < 33 or len(seen) > 1


def test_the_grid_holds_shorter_lists(L):
    out = (C.c_int * 4)()
    for Tt, cap in [(61, 96), (128, 74), (117, 300), (250, 64)]:
        grid = L.mix_grid(Tt, cap)
        for n in range(1, cap + 1):
            if L.keeps_own(cap, n) and L.mix_tail(Tt, n) != -2:
                assert not any(L.mix_item(Tt, n, w, out) for w in range(grid, grid + 300)), (Tt, cap, n)


@pytest.mark.parametrize("dtype,Tt,d,Fb,cap,n,tail", CASES)
def test_the_cases_run_as_they_claim(L, dtype, Tt, d, Fb, cap, n, tail):
    assert L.may_mix(Tt, d, cap, Fb, 0) and not L.may_mix(Tt, d, cap, Fb, 1)
    got = L.mix_tail(Tt, n) if L.keeps_own(cap, n) else -2
    assert tail == (None if got == -2 else "4x4" if got == -1 else TILES[got])


@pytest.mark.parametrize("dtype,Tt,d,n,tail", DOWN)
def test_the_second_products_run_as_they_claim(L, dtype, Tt, d, n, tail):
    assert TILES[L.down_tail(Tt, d, n, 0)] == tail and L.down_tail(Tt, d, n, 1) == -2
