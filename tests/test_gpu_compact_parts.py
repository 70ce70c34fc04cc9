"""Mask compaction where a workgroup's part of the rows takes several passes (the bytes of the first are loaded ahead),
rows and columns in either orientation."""
import numpy as np
import pytest

from test_gpu_compact import _check, lx  # noqa: F401  (a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,offset", [
    ((3000, 1000), 0),        # 64 parts of 47 KB, two passes of 32 KB at most each
    ((3000, 1000), 7),
    ((1500, 32, 64), 0),      # whole masks of 2 KB
    ((1500, 32, 64), 9),
    ((80, 4096, 7), 0),       # one mask a pass, rows at the end of what it holds
])
@pytest.mark.parametrize("transpose", [False, True])
def test_parts_of_several_passes(lx, oracle, shape, offset, transpose):  # noqa: F811
    rng = np.random.default_rng(shape[0] + offset)
    mask = (rng.random(shape) < 0.1).astype(np.uint8)
    mask[mask > 0] = rng.integers(1, 256, size=int(mask.sum()), dtype=np.uint8)
    _check(lx, oracle, mask, transpose, offset)


@pytest.mark.parametrize("shape,offset", [
    ((1, 1), 3),              # a byte that no word of four is
    ((2047, 1), 1),           # every byte a row; a step of 2048 bytes short of one, with the bytes before it
    ((1, 2049), 2),           # a byte into the second step
    ((5, 3), 1),              # rows shorter than a lane's four bytes
    ((700, 3), 3),            # parts that start at any alignment
    ((1, 2, 40000), 5),       # rows longer than a part and than the stage
    ((9, 181, 181), 0),       # a mask just within the stage
    ((4, 182, 181), 1),       # ... and just beyond it
    ((4097, 2, 4), 0),        # many small masks
])
@pytest.mark.parametrize("transpose", [False, True])
def test_contiguous_bytes_four_a_lane(lx, oracle, shape, offset, transpose):  # noqa: F811
    rng = np.random.default_rng(shape[0] + 31 * offset)
    mask = (rng.random(shape) < 0.6).astype(np.uint8)
    mask[mask > 0] = rng.integers(1, 256, size=int(mask.sum()), dtype=np.uint8)
    _check(lx, oracle, mask, transpose, offset)
