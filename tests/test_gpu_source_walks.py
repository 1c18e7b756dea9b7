"""Per-source TGT+: the variants of its kernels agree.

* walks with the column in LDS (waves with many chunks per source) against the
  general walk kernel, for a graph that fits the LDS, one with a prefix of its
  nodes there, and one whose ids need 32 bits: the same walk counts, and sums
  that differ by the rounding of their grouping only (1e-12);
* the head's workgroup sizes (chosen by the number of sources) and places of the
  columns (by the number of nodes): the same switch steps and walk counts per source;
* selections with ties and long candidate lists against the oracle.
"""
import numpy as np
import pytest

import graphgen as gg
from test_gpu_per_source import TOL, check_against_oracle, run_ps, sc  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [300, 13600, 13601, 70000])
def test_walks_with_column_in_lds(sc, n, monkeypatch):  # noqa: F811
    graph = gg.tree_plus_gnp(n, 8.0, 11)
    src = np.arange(0, n, n // 8, dtype=np.int32)[:8]
    kw = dict(sources=src, tilde_tau=1, L=9)
    monkeypatch.setenv("SC_SOURCE_LDS_CHUNKS", str(10 ** 12))
    ref, _, _, _, nr2 = run_ps(sc, graph, 0.02, **kw)
    monkeypatch.setenv("SC_SOURCE_LDS_CHUNKS", "1")
    out, _, _, _, nr = run_ps(sc, graph, 0.02, **kw)
    assert np.ceil(nr[nr > 0] / 64).sum() > 128              # more than one unit
    np.testing.assert_array_equal(out, ref)
    monkeypatch.setenv("SC_SOURCE_PART_CAPACITY", "200")     # in batches
    out, _, _, _, _ = run_ps(sc, graph, 0.02, **kw)
    np.testing.assert_array_equal(nr, nr2)
    np.testing.assert_allclose(out, ref, atol=TOL, rtol=0)


@pytest.mark.parametrize("n", [1200, 4096, 4097])            # both columns in LDS up to 4,096 nodes
def test_head_workgroup_sizes(sc, n):  # noqa: F811
    graph = gg.barabasi_albert(n, 6, 4)
    n, u, v = graph
    _, _, _, tt, nr = run_ps(sc, graph, 0.02)                # more than 1,024: 256 threads
    for count in (512, 513, 1024):                           # 1,024, 512 and 512 threads
        src = np.random.default_rng(count).permutation(n)[:count].astype(np.int32)
        _, _, _, tt2, nr2 = run_ps(sc, graph, 0.02, sources=src)
        np.testing.assert_array_equal(tt2[src], tt[src])
        listed = np.zeros(n, bool)
        listed[src] = True
        hl = np.concatenate([listed[u], listed[v]])
        np.testing.assert_array_equal(nr2[hl], nr[hl])


@pytest.mark.parametrize("n", [4096, 4097])
def test_columns_against_oracle(sc, n):  # noqa: F811
    graph = gg.barabasi_albert(n, 5, 8)
    src = np.array([0, 1, 17, n // 2, n - 1], np.int32)
    out, st, tau, tt, nr = run_ps(sc, graph, 0.03, sources=src)
    check_against_oracle(graph, 0.03, out, st, tau, tt, nr, sources=src)


@pytest.mark.parametrize("gamma", [64, 65, 100, 200])
def test_selection_with_ties(sc, gamma):  # noqa: F811
    graph = gg.king_grid(200)
    out, _, tau, tt, nr = run_ps(sc, graph, 0.05, gamma=gamma, max_L=31)
    check_against_oracle(graph, 0.05, out, None, tau, tt, nr, gamma=gamma)


@pytest.mark.parametrize("gamma,rule", [(10, 0), (0, 0), (100, 1)])
def test_heavy_sources_step_together(sc, gamma, rule, monkeypatch):  # noqa: F811
    # every source left to the heavy kernels at its first push, and none
    n, u, v = gg.barabasi_albert(6000, 5, 9)
    hub = np.arange(1, 2501)                                  # node 0: a list of the whole workgroup
    u, v = gg.canonical_edges(n, np.concatenate([u, np.zeros(len(hub), u.dtype)]),
                              np.concatenate([v, hub]))
    src = np.r_[0, 1, 2, np.random.default_rng(1).permutation(np.arange(3, n))[:60]].astype(np.int32)
    kw = dict(sources=src, gamma=gamma, switch_rule=rule)
    monkeypatch.setenv("SC_SOURCE_HEAVY_VOLUME", str(10 ** 12))
    ref, st, _, tt, nr = run_ps(sc, (n, u, v), 0.02, **kw)
    monkeypatch.setenv("SC_SOURCE_HEAVY_VOLUME", "1")
    out, st2, _, tt2, nr2 = run_ps(sc, (n, u, v), 0.02, **kw)
    np.testing.assert_array_equal(tt2, tt)
    np.testing.assert_array_equal(nr2, nr)
    np.testing.assert_array_equal(out, ref)
    assert st2["push_edges"] == st["push_edges"] and st2["walk_steps"] == st["walk_steps"]
