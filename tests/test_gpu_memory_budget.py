"""Calls where device memory is short take smaller work buffers instead of failing.

The budget is the library's own (SC_DEVICE_BYTES_LIMIT, on the bytes it holds), set to
what a call has with one basis, or with the 24 block states and the one candidate
summary that a call held before blocks were grouped.  The results do not depend on the
group or on whether the Lanczos runs are made side by side: they are equal bit for bit.
"""
import gc

import numpy as np
import pytest

import graphgen as gg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sc():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2305_16086_amd import sc as scmod
    return scmod


def live_bytes(sc, monkeypatch):
    """Bytes the library holds, to 64 KB: the smallest budget under which a tiny graph fits."""
    gc.collect()
    lo, hi = 0, 1 << 40
    while hi - lo > 65536:
        mid = (lo + hi) // 2
        monkeypatch.setenv("SC_DEVICE_BYTES_LIMIT", str(mid))
        try:
            sc.sc_build_graph(*gg.complete_graph(3)).free()
            hi = mid
        except sc.ScError:
            lo = mid
    monkeypatch.delenv("SC_DEVICE_BYTES_LIMIT")
    return hi


def test_lambda_star_with_room_for_one_basis(sc, monkeypatch):
    n, u, v = gg.barabasi_albert(20011, 6, 1)
    g = sc.sc_build_graph(n, u, v)
    ref = sc.sc_lambda_star(g)
    g.free()
    g = sc.sc_build_graph(n, u, v)
    base = live_bytes(sc, monkeypatch)
    basis = 602 * n * 8
    print(f"[gpu] lambda* within {1.3 * basis / 1e6:.0f} MB", flush=True)
    monkeypatch.setenv("SC_DEVICE_BYTES_LIMIT", str(base + 1.3 * basis))
    assert sc.sc_lambda_star(g) == ref
    g.free()


@pytest.mark.parametrize("method,precision,block", [(0, 0, 64), (1, 0, 64), (1, 1, 64), (1, 0, 32),
                                                    (0, 1, 16)])
def test_dense_call_with_room_for_few_blocks(sc, method, precision, block, monkeypatch):
    n, u, v = gg.barabasi_albert(20000, 6, 2)
    o = sc.sc_default_options(method=method, precision=precision, block=block,
                              tilde_tau=2 if method else -1)
    g = sc.sc_build_graph(n, u, v)
    ref = sc.sc_all_edges_ex(g, 0.1, 5, o)[0]
    g.free()
    g = sc.sc_build_graph(n, u, v)
    base = live_bytes(sc, monkeypatch)
    state = n * block * (8 if precision else 4)
    room = 24 * state + (28 << 20) + 40 * 2 * g.m   # states, summary, sums and walk buffers
    monkeypatch.setenv("SC_DEVICE_BYTES_LIMIT", str(base + room))
    print(f"[gpu] method {method} precision {precision} block {block} within {room / 1e6:.0f} MB",
          flush=True)
    out = sc.sc_all_edges_ex(g, 0.1, 5, o)[0]
    np.testing.assert_array_equal(out, ref)
    monkeypatch.delenv("SC_DEVICE_BYTES_LIMIT")
    np.testing.assert_array_equal(sc.sc_all_edges_ex(g, 0.1, 5, o)[0], ref)
    g.free()


def test_learned_call_with_room_for_few_blocks(sc, monkeypatch):
    import os
    n, u, v = gg.barabasi_albert(10000, 6, 2)
    net = sc.sc_mlp_load(os.path.join(os.path.dirname(sc.__file__), "weights", "closure_ba_gnp.bin"))
    o = sc.sc_default_options(method=sc.SC_LEARNED, mlp=net.handle)
    g = sc.sc_build_graph(n, u, v)
    lam = sc.sc_lambda_star(g)
    ref = sc.sc_all_edges_ex(g, 1e-2, 0, o)[0]
    g.free()
    g = sc.sc_build_graph(n, u, v)
    o.lambda_star = lam
    base = live_bytes(sc, monkeypatch)
    # recordings, features and sums as ever, beside them 24 states
    room = 24 * n * 64 * 4 + 2 * g.m * (2 * 9 * 4 + 40) + g.m * (16 * 4 + 64)
    monkeypatch.setenv("SC_DEVICE_BYTES_LIMIT", str(base + room))
    out = sc.sc_all_edges_ex(g, 1e-2, 0, o)[0]
    np.testing.assert_array_equal(out, ref)
    g.free()
    net.free()


def test_neighbour_lists_after_a_failed_build(sc, monkeypatch):
    # budgets that end at every buffer of the first call in turn, then none
    n, u, v = gg.tree_plus_gnp(700, 8.0, 5)
    g = sc.sc_build_graph(n, u, v)
    o = sc.sc_default_options(method=sc.SC_TGT, precision=1)
    ref = sc.sc_all_edges_ex(g, 0.5, 5, o)[0]
    g.free()
    g = sc.sc_build_graph(n, u, v)
    base = live_bytes(sc, monkeypatch)
    refused = 0
    for room in np.geomspace(1e4, 4e7, 60):
        monkeypatch.setenv("SC_DEVICE_BYTES_LIMIT", str(base + room))
        try:
            out = sc.sc_all_edges_ex(g, 0.5, 5, o)[0]
        except sc.ScError as e:
            assert e.code == sc.SC_ENOMEM
            refused += 1
            continue
        np.testing.assert_array_equal(out, ref)
    assert 0 < refused < 60
    g.free()
