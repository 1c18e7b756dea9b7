"""The variants of a group's steps (block width 64) give the same bits.

The steps of large graphs (beyond 140,000 nodes: whole rows in the two-hop step and the
step after it, one slice after the other in the others) and those of states beyond a
buffer descriptor's reach (64-bit addresses, no skipping) are taken at small sizes
through the library's limits, and compared with the usual ones.  Every variant adds a row's
neighbours in slot order, so sums, recordings and walk counts are equal.  Sizes: those
of the group and slice bookkeeping, rows around the chunk, light and heavy lengths, a
row cut into chunks (above 4,096 neighbours), hubs first (blocks with more half-edges
than the graph has nodes), complete graphs of light and of heavy rows only.
"""
import os

import numpy as np
import pytest

import graphgen as gg
from test_gpu_group_steps import exact_degree_graph, sc  # noqa: F401

pytestmark = pytest.mark.gpu


def hub_graph(n, hubs, seed):
    """`hubs` nodes joined to everything, beside a sparse graph."""
    n, u, v = gg.tree_plus_gnp(n, 4.0, seed)
    a = np.repeat(np.arange(hubs), n)
    b = np.tile(np.arange(n), hubs)
    u = np.concatenate([u, a[a != b]])
    v = np.concatenate([v, b[a != b]])
    return (n, *gg.canonical_edges(n, u, v))


GRAPHS = {
    "one block": lambda: exact_degree_graph(50, 1),
    "six blocks": lambda: exact_degree_graph(380, 2),
    "33 blocks": lambda: exact_degree_graph(2049, 3),
    "giant row": lambda: hub_graph(4700, 1, 4),
    "hubs first": lambda: hub_graph(700, 70, 5),
    "complete": lambda: gg.complete_graph(129),
    "heavy rows only": lambda: gg.complete_graph(261),
}


@pytest.mark.parametrize("name", list(GRAPHS))
@pytest.mark.parametrize("precision", [0, 1])
def test_variants_agree(sc, name, precision, monkeypatch):  # noqa: F811
    n, u, v = GRAPHS[name]()
    print(f"[gpu] step variants, {name} n={n} m={len(u)} precision={precision}", flush=True)
    net = sc.sc_mlp_load(os.path.join(os.path.dirname(sc.__file__), "weights", "closure_ba_gnp.bin"))
    calls = [(0.5, L, dict(method=sc.SC_TGT, max_L=11)) for L in (3, 5, 7)]
    calls += [(0.05, 0, dict(method=sc.SC_TGT, max_L=11))]          # last steps differ by block
    calls += [(0.4, 0, dict(method=sc.SC_TGT_PLUS, tilde_tau=t, max_L=7)) for t in (2, 3, 4)]
    calls += [(0.3, 0, dict(method=sc.SC_TGT_PLUS, max_L=9)),        # the planned switch step
              (0.05, 0, dict(method=sc.SC_LEARNED, mlp=net.handle, max_L=11)),
              (0.05, 0, dict(method=sc.SC_LEARNED, mlp=net.handle, max_L=11, force_fallback=1))]

    def run(limits):
        for k in ("SC_STEP_BITMAP_NODES", "SC_STEP_BUFFER_BYTES"):
            monkeypatch.delenv(k, raising=False)
        for k, x in limits.items():
            monkeypatch.setenv(k, x)
        g = sc.sc_build_graph(n, u, v)
        res = []
        for eps, L, kw in calls:
            nr = np.zeros(2 * g.m, np.int64)
            tr = {} if kw["method"] == sc.SC_LEARNED else dict(nr_out=nr)
            res.append((sc.sc_all_edges_ex(g, eps, L, sc.sc_default_options(precision=precision, **kw),
                                           **tr)[0].copy(), nr))
        g.free()
        return res

    ref = run({})
    for limits in ({"SC_STEP_BITMAP_NODES": "0"}, {"SC_STEP_BUFFER_BYTES": "0"},
                   {"SC_STEP_BITMAP_NODES": "0", "SC_STEP_BUFFER_BYTES": "0"}):
        for (out, nr), (out0, nr0), call in zip(run(limits), ref, calls):
            np.testing.assert_array_equal(nr, nr0, err_msg=f"{limits} {call}")
            np.testing.assert_array_equal(out, out0, err_msg=f"{limits} {call}")
    net.free()


def test_beyond_the_bitmap_limit(sc):  # noqa: F811
    # 140,001 nodes take the large graphs' steps as they are; FP64 against width 32
    n, u, v = gg.barabasi_albert(140001, 2, 6)
    g = sc.sc_build_graph(n, u, v)
    outs = [sc.sc_all_edges_ex(g, 0.5, 5, sc.sc_default_options(method=sc.SC_TGT, precision=1,
                                                                block=b))[0] for b in (64, 32)]
    np.testing.assert_allclose(outs[0], outs[1], atol=1e-12, rtol=0)
    g.free()
