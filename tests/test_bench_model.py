"""bench.py's accounting of the attention backward call in one launch and in two."""
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)


def test_backward_in_one_launch_is_counted_once():
    import bench
    from paper_2510_15964_amd import build
    build.ensure()
    from paper_2510_15964_amd import lx
    dq, dkv, fwd = lx.LX_K_ATTN_BWD_DQ, lx.LX_K_ATTN_BWD_DKV, lx.LX_K_ATTN_FWD
    model = {fwd: (1, 2.0, 4.0), dq: (1, 3.0, 62.0), dkv: (1, 4.0, 62.0)}
    assert bench.one_launch_backward(lx, model, {fwd: 3, dq: 3, dkv: 3}, 10.0) == model
    one = bench.one_launch_backward(lx, model, {fwd: 3, dq: 0, dkv: 3}, 10.0)
    assert one == {fwd: (1, 2.0, 4.0), dkv: (1, 7.0, 84.0)}
    assert sum(n * fl for n, fl, _ in one.values()) == sum(n * fl for n, fl, _ in model.values())
