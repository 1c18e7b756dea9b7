"""The allocation-free entry point on graphs that share n and the edge count.

Two such graphs get the same slot count but waves of different half-edge totals.
The second call reuses the first one's zeroed columns, so the columns must sit at
the same place in the static array whatever the totals are: calls alternating
between the graphs give what the allocating per-source run gives.
"""
import numpy as np
import pytest

import graphgen as gg

pytestmark = pytest.mark.gpu


def test_static_calls_alternating_between_equal_sized_graphs():
    import torch
    from paper_2305_16086_amd import sc
    graphs = [gg.barabasi_albert(3000, 5, s) for s in (31, 32, 33)]
    assert len({len(u) for _, u, _ in graphs}) == 1
    # the first wave of 1,024 sources holds a different number of half-edges in each
    tops = {int(np.sort(gg.degrees(n, u, v)[:1024]).sum()) for n, u, v in graphs}
    assert len(tops) == 3
    hs, refs = [], []
    for n, u, v in graphs:
        g = sc.sc_build_graph(n, u, v)
        sc.sc_lambda_star(g)
        o = sc.sc_default_options(method=sc.SC_TGT_PLUS, flags=sc.SC_PER_SOURCE)
        refs.append(sc.sc_all_edges_ex(g, 0.02, 0, o)[0])
        hs.append(g)
    for turn in range(2):
        for g, ref in zip(hs, refs):
            out = torch.empty(g.m, dtype=torch.float64, device="cuda")
            sc.sc_all_edges_static(g, 0.02, 0, sc.sc_default_options(method=sc.SC_TGT_PLUS), out)
            np.testing.assert_allclose(out.cpu().numpy(), ref, atol=1e-12, rtol=0)
    for g in hs:
        g.free()
