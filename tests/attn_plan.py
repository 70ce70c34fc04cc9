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
    L.turns_ns.restype = L.rows_ns.restype = C.c_double
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


SLOTS = {64: {"fwd": 1024, "dq": 1024, "dkv": 768}, 128: {"fwd": 512, "dq": 512, "dkv": 512}}      # workgroups that the chip holds


def shape(L, B, Hh, nblk, slots, may_turn=True, forced=0):
    """rows per workgroup, heads of a group, workgroups of a group, spread, grid, turns (0: not by turns) of a launch."""
    out = (C.c_int * 6)()
    L.shape(B, Hh, nblk, slots, int(may_turn), forced, out)
    return tuple(out)


def launches(L, B, Hh, S, D, causal):
    """Rows per workgroup by turns, 0 where a launch does not run so, of the forward, dQ and dK/dV launches (head size D, lists
    with room for every block, ordinary strides)."""
    nblk = S // 64
    one = bool(L.pays(D, B * Hh * nblk, nblk, int(causal), float(nblk)))
    return tuple(0 if one and k != "fwd" else shape(L, B, Hh, nblk, SLOTS[D][k])[5] for k in ("fwd", "dq", "dkv"))
