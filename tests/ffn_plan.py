"""The library's tile rules (csrc/ffn_plan.h) for the tests: which tile a call of given sizes runs with."""
import ctypes as C
import os
import subprocess
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
TILES = ("4x4", "2x4", "2x2", "2x2 deep", "1x4", "1x4 deep", "1x2", "1x1", "1x1 many")   # order of TileId


def load():
    d = tempfile.mkdtemp()
    lib = os.path.join(d, "ffn_plan.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Wno-unknown-pragmas", "-shared", "-fPIC",
                    os.path.join(HERE, "ffn_plan_shim.cpp"), "-o", lib], check=True)
    L = C.CDLL(lib)
    L.sdd_us.restype = C.c_float
    L.dsd_tile.argtypes = [C.c_int] * 4 + [C.c_longlong, C.c_int, C.POINTER(C.c_int)]
    L.dsd_by.argtypes = [C.c_int] * 5 + [C.c_longlong, C.c_int, C.POINTER(C.c_int), C.POINTER(C.c_int)]
    return L


ROUTES = ("nothing", "quarters", "set", "mix", "lean", "tile", "pieces")      # order of Route


def sdd_by(L, Tt, gt, d, cap, blocks, want, n):
    """(route, tile) of the first product of a list of n entries."""
    t = C.c_int(0)
    r = ROUTES[L.sdd_by(Tt, gt, d, cap, blocks, want, n, C.byref(t))]
    return r, None if t.value < 0 else TILES[t.value]


def dsd_by(L, Tt, gt, d, F, cap, part_bytes=0, want=0):
    """(route, tile, pieces) of the second product."""
    t, p = C.c_int(0), C.c_int(0)
    r = ROUTES[L.dsd_by(Tt, gt, d, F, cap, part_bytes, want, C.byref(t), C.byref(p))]
    return r, None if t.value < 0 else TILES[t.value], p.value


def dsd(L, Tt, gt, d, cap, part_bytes=0, want=0):
    """(tile, pieces) of the second product."""
    p = C.c_int(0)
    return TILES[L.dsd_tile(Tt, gt, d, cap, part_bytes, want, C.byref(p))], p.value


def even_items(L, lens, cap):
    """The pieces of lists of these lengths, capacity cap, as their workgroups find them: ([(tile, first, entries)], most entries)."""
    ptr = [0]
    for n in lens:
        ptr.append(ptr[-1] + int(n))
    room = cap // 8 + len(lens) + 512
    out, per = (C.c_int * (3 * room))(), C.c_int(0)
    grid = L.even_items((C.c_int * len(ptr))(*ptr), len(lens), cap, room, out, C.byref(per))
    assert grid <= room
    return [tuple(out[3 * w:3 * w + 3]) for w in range(grid) if out[3 * w] >= 0], per.value
