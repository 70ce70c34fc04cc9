"""How mask compaction jobs are divided among workgroups (csrc/compact_plan.h), on the host: which way takes which layout, and
that every part stays within what the kernel's integers and its stage hold."""
import ctypes as C
import os
import random
import subprocess
import tempfile

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
FLAT, TURNED, BY_ROW = range(3)
STAGE = 32768


@pytest.fixture(scope="module")
def parts():
    lib = os.path.join(tempfile.mkdtemp(), "compact_plan.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", os.path.join(HERE, "compact_plan_shim.cpp"),
                    "-o", lib], check=True)
    L = C.CDLL(lib)
    L.parts.argtypes = [C.c_int] * 3 + [C.c_longlong] * 3 + [C.POINTER(C.c_int)]

    def call(*job):
        out = (C.c_int * 4)()
        L.parts(*job, out)
        return tuple(out)
    return call


def size(rng, most):
    return min(most, round(2 ** rng.uniform(0, most.bit_length())))


def test_parts_cover_the_rows_within_their_limits(parts):
    rng = random.Random(5)
    seen = set()
    for _ in range(20000):
        b, r, c = size(rng, 100000), size(rng, 1 << 20), size(rng, (1 << 31) - 1)
        if b * r >= 1 << 31 or b * r * c > 288 << 30:
            continue
        layout = rng.randrange(3)
        strides = ((r * c, c, 1), (r * c, 1, r), (2 * r * c, 2 * c, 2))[layout]
        n, rows, chunk, by = parts(b, r, c, *strides)
        seen.add((layout, by))
        assert 1 <= n <= 65535 and (n - 1) * rows < b * r <= n * rows           # no part is empty
        assert by == FLAT if layout == 0 and c < 1 << 30 else by in (TURNED, BY_ROW) or min(r, c) == 1
        if by == FLAT:
            assert rows * c < 1 << 30
        elif by == TURNED:
            assert rows % r == 0 and 0 < chunk * c <= STAGE
        elif c <= STAGE:
            assert 0 < chunk * c <= STAGE and chunk <= 4096
    assert {(0, FLAT), (1, TURNED), (1, BY_ROW), (2, BY_ROW)} <= seen


@pytest.mark.parametrize("b,r,c", [(1, (1 << 18) - 1, 4096), (1, 1 << 18, 4096), (300000, 64, 64), (1, 1 << 20, 1100), (1, 1, (1 << 30) - 1),
                                   (300, 1, (1 << 30) - 1), (1, 1 << 22, 1 << 14)])
def test_rows_one_after_the_other_are_flat_at_any_number_of_them(parts, b, r, c):
    assert parts(b, r, c, r * c, c, 1)[3] == FLAT
