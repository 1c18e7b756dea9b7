"""The dense-step statistics of a call.

Block widths 16 and 32 launch every dense step block by block: prop_launches counts
them all, and prop_bytes / prop_launches is the traffic of one block's step.  At 64 a
launch takes a group of blocks.
"""
import pytest

import graphgen as gg
from test_gpu_group_steps import sc  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("block", [16, 32])
@pytest.mark.parametrize("precision", [0, 1])
def test_launches_and_bytes_of_narrow_blocks(sc, block, precision):  # noqa: F811
    n, u, v = gg.tree_plus_gnp(1100, 8.0, 3)
    g = sc.sc_build_graph(n, u, v)
    o = sc.sc_default_options(method=sc.SC_TGT, precision=precision, block=block,
                              flags=sc.SC_TIME_KERNELS)
    _, st = sc.sc_all_edges_ex(g, 0.5, 5, o)
    blocks = -(-n // block)
    assert st["prop_launches"] == 3 * blocks            # l = 3, 4, 5
    t = 8 if precision else 4
    least = 2.0 * n * block * t + 4.0 * 2 * g.m + t * n   # state read and written, ids, degrees
    per = st["prop_bytes"] / st["prop_launches"]
    assert least < per < 1.2 * least
    # every 15th counted launch is timed, by events around that launch alone: a launch
    # that cannot move its bytes faster than 20 TB/s through the caches
    assert st["prop_timed"] == -(-st["prop_launches"] // 15)
    assert st["prop_ms"] > 0
    assert per / (st["prop_ms"] / st["prop_timed"] * 1e-3) < 20e12
    g.free()
