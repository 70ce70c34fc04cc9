"""The library's rules for the launches of the attention calls (csrc/attn_plan.h) for the tests."""
import ctypes as C
import os
import subprocess
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))


def load():
    lib = os.path.join(tempfile.mkdtemp(), "attn_plan.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-shared", "-fPIC", os.path.join(HERE, "attn_plan_shim.cpp"), "-o", lib],
                   check=True)
    L = C.CDLL(lib)
    L.pays.argtypes = [C.c_int, C.c_longlong, C.c_int, C.c_int, C.c_double]
    return L


def arr(v):
    return (C.c_longlong * len(v))(*v)


def meet(L, n, stride, row, delta):
    return bool(L.meet(arr(n), arr(stride), C.c_longlong(row), C.c_longlong(delta)))


def sides_apart(L, n, stride, row, at, stats, ptrs, entries):
    return bool(L.sides_apart(arr(n), arr(stride), C.c_longlong(row), arr(at), *map(C.c_longlong, (stats, ptrs, entries))))


def turns(L, pairs, nblk, slots, rows_per_wg):
    """turns, places, cohorts, pairs of a cohort, grid; None: not by turns."""
    out = (C.c_int * 5)()
    L.turns(pairs, nblk, slots, rows_per_wg, out)
    return tuple(out) if out[0] else None
