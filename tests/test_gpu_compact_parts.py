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
