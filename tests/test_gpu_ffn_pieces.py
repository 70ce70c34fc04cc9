"""First product by pieces of lists: every length of a piece, one round and two, one and two tiles per lane of the scan,
empty, short and full lists, a capacity of every block.  Rows are independent, so sampled token tiles equal, bit for bit, a call
that holds that tile alone."""
import pytest

from test_gpu_ffn_deal import lx, test_deals as check_deals  # noqa: F401

# element type, token tiles, d, neuron blocks, capacity, density (the lists' mean is three quarters of that)
CASES = [
    ("bf16", 50, 3200, 60, 1600, 0.6),        # 2.6 entries per workgroup of a round
    ("f16", 97, 640, 70, 3550, 0.66),
    ("bf16", 64, 320, 110, 3400, 0.6),        # one tile per lane
    ("bf16", 65, 2048, 64, 2400, 0.74),
    ("bf16", 128, 3200, 64, 6700, 0.99),      # two rounds
    ("f16", 127, 704, 48, 2700, 0.5),
    ("bf16", 100, 3264, 48, 4800, 0.2),       # every block as capacity: workgroups that find nothing
]


@pytest.mark.gpu
@pytest.mark.parametrize("lora", [False, True])
@pytest.mark.parametrize("dtype,Tt,d,Fb,cap,density", CASES)
def test_pieces(lx, dtype, Tt, d, Fb, cap, density, lora):  # noqa: F811
    check_deals(lx, dtype, Tt, 1, d, Fb, cap, None, None, density, lora)


def test_cases_take_that_route(tmp_path):
    import ffn_plan
    L = ffn_plan.load()
    for _, Tt, d, Fb, cap, density in CASES:
        assert ffn_plan.sdd_by(L, Tt, 1, d, cap, Tt * Fb, 0, cap)[0] == "pieces", (Tt, d, Fb)
        assert ffn_plan.sdd_by(L, Tt, 1, d, cap, Tt * Fb, 1, cap)[0] != "pieces"
