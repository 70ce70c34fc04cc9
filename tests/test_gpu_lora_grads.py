"""Gradients of the two LoRA matrices for few token tiles: a workgroup per quadrant of a product, whose wavefronts share
out the tiles.  The sums are those of the other way but for the order of fp32 additions, so the bounds of test_gpu_lora.py hold."""
import pytest

from test_gpu_lora import check, lx, make_case, run_both  # noqa: F401  (a fixture)

pytestmark = pytest.mark.gpu


CASES = [
    (1, 64, 64, 1, 1.0, "bf16"),       # one tile: by parts, of which there is one
    (2, 64, 64, 1, 1.0, "bf16"),       # one product of each kind, two wavefronts with work
    (3, 192, 320, 3, 0.3, "f16"),      # fewer tiles than wavefronts; blocks that no tile lists
    (8, 576, 64, 8, 0.7, "bf16"),      # nine chunks of dA: a second group of eight products
    (17, 128, 640, 1, 0.5, "bf16"),    # one list: dB first; ranges of three tiles, the last one short
    (20, 64, 192, 5, 0.4, "f16"),      # lists per group of four tiles
    (64, 128, 128, 64, 0.05, "bf16"),  # the most tiles, a few of them per block
]


@pytest.mark.parametrize("Tt,d,F,rows,density,dtype", CASES)
def test_gradients_by_quadrants(lx, oracle, Tt, d, F, rows, density, dtype):  # noqa: F811
    c = make_case(64 * Tt, d, F, 16, density, 70 + Tt, rows=None if rows == Tt else rows, dtype=dtype)
    got, ref = run_both(lx, oracle, c)
    check(got, ref, f"{Tt} tiles d={d} F={F} rows={rows} {dtype}", dtype=dtype)
