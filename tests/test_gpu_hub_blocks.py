"""TGT+ of a group with a block of hubs.

64 hubs joined to 40,000 nodes: the first block has 2.56 M half-edges, so one wave per
half-edge for every slice of the group's eight blocks would pass the 2^32 threads of a
launch (the waves take the half-edges in turn instead).  Leaves of degree 1 hang on
hub 0, one in each of the next blocks: the truncation of the other edges is 1, so these
eight blocks are one group and only their edges to the leaves need walks.  Against
block width 32: the same walk counts, and estimates to FP64 rounding.
"""
import numpy as np
import pytest

import graphgen as gg
from test_gpu_group_steps import sc  # noqa: F401

pytestmark = pytest.mark.gpu


def test_walk_counts_of_a_hub_block(sc):  # noqa: F811
    n, hubs = 40000, 64
    leaves = 64 * np.arange(1, 8)                      # one in each of blocks 1 .. 7
    rest = np.setdiff1d(np.arange(hubs, n), leaves)
    u = np.concatenate([np.repeat(np.arange(hubs), len(rest)), np.zeros(len(leaves), np.int64),
                        np.zeros(hubs - 1, np.int64)])
    v = np.concatenate([np.tile(rest, hubs), leaves, np.arange(1, hubs)])
    u, v = gg.canonical_edges(n, u, v)
    g = sc.sc_build_graph(n, u, v)
    runs = []
    for block in (64, 32):
        print(f"[gpu] hub block n={n} m={g.m} block={block}", flush=True)
        o = sc.sc_default_options(method=sc.SC_TGT_PLUS, precision=1, block=block, tilde_tau=2,
                                  lambda_star=0.5)
        nr = np.empty(2 * g.m, np.int64)
        tau = np.empty(g.m, np.int32)
        out, st = sc.sc_all_edges_ex(g, 0.1, 0, o, nr_out=nr, tau_out=tau)
        runs.append((out, nr, tau, st["walks"]))
    out, nr, tau, walks = runs[0]
    hung = np.isin(v, leaves)
    assert (tau[hung] > 2).all() and (tau[~hung] <= 2).all() and hung.sum() == 7
    assert walks == nr.sum() > 0
    np.testing.assert_array_equal(nr, runs[1][1])
    np.testing.assert_allclose(out, runs[1][0], atol=1e-12, rtol=0)
    g.free()
