"""Calls where device memory is short take smaller work buffers instead of failing.

The budget is the library's own (SC_DEVICE_BYTES_LIMIT, on the bytes it holds).  lambda*
with room for one basis: the results do not depend on whether the Lanczos runs are made
side by side, they are equal bit for bit.
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
