"""Mask compaction where a workgroup's part of the rows takes several steps of 2048 bytes or several stages, from any address, rows and
columns in either orientation."""
import numpy as np
import pytest

from test_gpu_compact import _check, lx  # noqa: F401  (a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,offset", [
    ((3000, 1000), 0),        # 64 parts of 47 KB: 23 steps by rows; 16 parts of 63 columns, ten to a stage
    ((3000, 1000), 7),
    ((1500, 32, 64), 0),      # whole masks of 2 KB
    ((1500, 32, 64), 9),
    ((80, 4096, 7), 0),       # by columns one mask to a stage
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


def test_the_longest_row_of_a_part(lx):  # noqa: F811
    """2^30 - 1 bytes from an odd address, a few of them active: the first ones, the last ones, and where a byte's number in the
    part passes 2^22 (rows by division) and the last step begins."""
    import torch
    n = 2 ** 30 - 1
    buf = torch.zeros(n + 1, dtype=torch.uint8, device="cuda")
    at = sorted({0, 1, 2, 3, 2 ** 22 - 1, 2 ** 22, n - 2049, n - 2048} | set(range(n - 5, n)))
    buf[1:][torch.tensor(at, device="cuda")] = 7
    bl = lx.lx_mask_compact(buf[1:].view(1, n), nnz_cap=64)
    assert bl.row_ptr.tolist() == [0, len(at)]
    assert bl.col_idx[:len(at)].tolist() == at


@pytest.mark.parametrize("shape", [((1 << 18) + 3, 4097), (70000, 127, 127)])
def test_masks_beyond_2_to_30_bytes(lx, shape):  # noqa: F811
    import torch
    rng = np.random.default_rng(shape[0])
    n = int(np.prod(shape))
    flat = np.unique(np.concatenate([rng.integers(0, n, 5000), [0, n - 1]]))
    mask = torch.zeros(n, dtype=torch.uint8, device="cuda")
    mask[torch.from_numpy(flat).cuda()] = 1
    bl = lx.lx_mask_compact(mask.view(shape), nnz_cap=6000)
    rows = n // shape[-1]
    rp = np.searchsorted(flat, np.arange(rows + 1, dtype=np.int64) * shape[-1])
    assert np.array_equal(bl.row_ptr.cpu().numpy(), rp)
    assert np.array_equal(bl.col_idx[:len(flat)].cpu().numpy(), flat % shape[-1])


@pytest.mark.parametrize("shape", [
    (2, 70000),               # 16 parts of 4375 rows, more than a scan holds
    (40000, 3),               # rows longer than the stage
    (3, 5, 4100),             # parts that start inside a mask
    (7, 190, 200),
])
def test_columns_of_masks_that_no_stage_holds(lx, oracle, shape):  # noqa: F811
    """Masks that are contiguous in the other orientation and go row by row."""
    rng = np.random.default_rng(shape[0])
    mask = (rng.random(shape) < 0.3).astype(np.uint8)
    mask[mask > 0] = rng.integers(1, 256, size=int(mask.sum()), dtype=np.uint8)
    _check(lx, oracle, mask, transpose=True, offset=3)


@pytest.mark.parametrize("shape,strides", [
    ((1, 9, 11), (0, 16, 1)),                 # rows with a gap
    ((5, 61, 67), (61 * 67 + 13, 67, 1)),     # masks with a gap, several parts
    ((5, 61, 67), (61 * 67 * 3, 67 * 3, 3)),  # every third byte
    ((2, 5000, 3), (3, 6, 1)),                # masks interleaved row by row, several parts
    ((1, 2, 33000), (0, 1, 2)),               # rows longer than the stage, interleaved
    ((3, 40, 50), (0, 50, 1)),                # one mask thrice
])
def test_masks_of_any_strides(lx, oracle, shape, strides):  # noqa: F811
    """Through the C interface: the Python one takes contiguous masks."""
    import torch
    rng = np.random.default_rng(shape[1])
    buf = (rng.random(sum((n - 1) * s for n, s in zip(shape, strides)) + 1) < 0.4).astype(np.uint8) * 5
    mask = np.lib.stride_tricks.as_strided(buf, shape, strides)
    dev = torch.from_numpy(buf).cuda()
    rows = shape[0] * shape[1]
    row_ptr = torch.empty(rows + 1, dtype=torch.int32, device="cuda")
    col_idx = torch.empty(mask.size, dtype=torch.int32, device="cuda")
    lx._check(lx._lib.lx_mask_compact(dev.data_ptr(), *shape, *strides, row_ptr.data_ptr(), col_idx.data_ptr(), mask.size,
                                      lx._stream()), "lx_mask_compact")
    rp, ci = oracle.mask_compact(np.ascontiguousarray(mask.reshape(rows, shape[2])))
    assert np.array_equal(row_ptr.cpu().numpy(), rp)
    assert np.array_equal(col_idx.cpu().numpy()[:rp[-1]], ci)
