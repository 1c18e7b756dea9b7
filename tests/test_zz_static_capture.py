"""The allocation-free entry point recorded into a graph.

The replays come between eager calls of other layouts (another graph's columns lie where
the recorded call's were) and of the same layout, and between replays of another
recording: every result equals the allocating per-source run (1e-12, the tolerance of
the static calls).  The calls before the recordings leave the columns of the recorded
layout zeroed, so the recording itself may not rely on that.
"""
import ctypes as C

import numpy as np
import pytest

import graphgen as gg
from test_gpu_per_source import sc  # noqa: F401

pytestmark = pytest.mark.gpu


def test_recorded_calls_between_eager_ones(sc):  # noqa: F811
    import torch
    cases = [(gg.barabasi_albert(3000, 5, 31), 0.02), (gg.tree_plus_gnp(800, 8.0, 22), 0.03),
             (gg.barabasi_albert(3000, 5, 32), 0.02)]
    hs, refs, outs = [], [], []
    for (n, u, v), eps in cases:
        g = sc.sc_build_graph(n, u, v)
        sc.sc_lambda_star(g)
        o = sc.sc_default_options(method=sc.SC_TGT_PLUS, flags=sc.SC_PER_SOURCE)
        refs.append(sc.sc_all_edges_ex(g, eps, 0, o)[0])
        outs.append(torch.empty(g.m, dtype=torch.float64, device="cuda"))
        hs.append(g)

    def call(k):
        o = sc.sc_default_options(method=sc.SC_TGT_PLUS, flags=sc.SC_DEVICE_PTRS | sc.SC_PER_SOURCE)
        o.stream = torch.cuda.current_stream().cuda_stream
        rc = sc.lib().sc_all_edges_static(hs[k].handle, cases[k][1], 0, C.byref(o),
                                          outs[k].data_ptr(), None)
        assert rc == 0, sc.sc_last_error()

    def check(k, what):
        torch.cuda.synchronize()
        np.testing.assert_allclose(outs[k].cpu().numpy(), refs[k], atol=1e-12, rtol=0, err_msg=what)
        outs[k].fill_(-1.0)

    for k in (1, 0, 0):
        call(k)
        check(k, f"eager call {k} before the recordings")
    recorded = {}
    for k in (0, 1):
        recorded[k] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(recorded[k]):
            call(k)
    # eager 0 right after the recordings, then replays and eager calls in turn
    for turn, (kind, k) in enumerate([("eager", 1), ("replay", 0), ("eager", 0), ("replay", 1),
                                      ("eager", 2), ("replay", 0), ("replay", 1), ("replay", 1),
                                      ("replay", 0), ("eager", 2), ("eager", 1), ("replay", 0)]):
        print(f"[gpu] static, {kind} {k}", flush=True)
        if kind == "eager":
            call(k)
        else:
            recorded[k].replay()
        check(k, f"turn {turn}: {kind} {k}")
    for g in hs:
        g.free()
