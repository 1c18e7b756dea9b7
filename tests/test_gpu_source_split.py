"""Heavy sources in launches of any size.

Sources whose pushes outgrow a workgroup leave their head and are stepped together,
whatever the number of sources of the launch: at the head's workgroup sizes (1,024, 512
and 256 threads up to 512, 1,024 and more sources), over several waves of few slots, and
with every source leaving or none, the switch steps, walk counts and estimates are
the same bit for bit (all sums are of whole numbers).
"""
import numpy as np
import pytest

import graphgen as gg
from test_gpu_per_source import run_ps, sc  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def graph():
    # node 0: a list that a whole workgroup pushes
    n, u, v = gg.barabasi_albert(6000, 5, 9)
    hub = np.arange(1, 2501)
    return (n, *gg.canonical_edges(n, np.concatenate([u, np.zeros(len(hub), u.dtype)]),
                                   np.concatenate([v, hub])))


@pytest.mark.parametrize("count,slots", [(512, 0), (513, 0), (1025, 0), (6000, 0), (1500, 600)])
def test_all_sources_leave_or_none(sc, graph, count, slots, monkeypatch):  # noqa: F811
    n = graph[0]
    src = None
    if count < n:
        src = np.r_[0, 1 + np.random.default_rng(count).permutation(n - 1)[:count - 1]].astype(np.int32)
    if slots:
        monkeypatch.setenv("SC_SOURCE_SLOT_BYTES", str(slots * 24 * n))
    runs = []
    for volume in (10 ** 12, 1, 60000):
        monkeypatch.setenv("SC_SOURCE_HEAVY_VOLUME", str(volume))
        runs.append(run_ps(sc, graph, 0.05, sources=src))
    ref, st, _, tt, nr = runs[0]
    for out2, st2, _, tt2, nr2 in runs[1:]:
        np.testing.assert_array_equal(tt2, tt)
        np.testing.assert_array_equal(nr2, nr)
        np.testing.assert_array_equal(out2, ref)
        assert st2["push_edges"] == st["push_edges"] and st2["walk_steps"] == st["walk_steps"]
