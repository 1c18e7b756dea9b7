"""Steps that run a group of source blocks per launch (block width 64).

Sizes where the group and slice bookkeeping can go wrong: one block to two groups of
blocks (up to 32 blocks each, 2 or 4 slices per block, so every remainder of the
slices modulo the 8 XCDs), light-row counts that are no multiple of the 8-row groups
or of the 4 groups of a workgroup, rows of exactly 8, 9, 16, 17, 64, 65, 255, 256 and
257 neighbours (one chunk, chunk remainders, the last light and the first heavy
length), and blocks whose last steps differ within a group.

Tolerances: those of the other traversal tests.  FP64: sums of at most 257 products
of values <= 1 over at most 12 steps, 1e-12.  FP32: relative rounding (d + L) 6e-8 of
probabilities that sum to at most L + 1, 2e-5.  TGT+ takes the recorded walks, so it
adds FP64 means of the same samples.
"""
import numpy as np
import pytest

import graphgen as gg
from oracle import tgt as otgt

pytestmark = pytest.mark.gpu

DEGREES = (8, 9, 16, 17, 64, 65, 255, 256, 257)


@pytest.fixture(scope="module")
def sc():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2305_16086_amd import sc as scmod
    return scmod


def exact_degree_graph(n, seed):
    """Sparse random graph whose nodes 0, 7, 14, ... have the listed degrees (those below n)."""
    rng = np.random.default_rng(seed)
    n, u, v = gg.tree_plus_gnp(n, 6.0, seed)
    rows = {x: set() for x in range(n)}
    for a, b in zip(u.tolist(), v.tolist()):
        rows[a].add(b)
        rows[b].add(a)
    fixed = []
    for i, d in enumerate(DEGREES):
        x = 7 * i
        if x >= n or d >= n - 10:
            break
        while len(rows[x]) < d:
            y = int(rng.integers(0, n))
            if y != x and y not in fixed and y not in rows[x]:
                rows[x].add(y)
                rows[y].add(x)
        for y in [y for y in rows[x] if y not in fixed and len(rows[y]) > 4]:
            if len(rows[x]) <= d:
                break
            rows[x].discard(y)
            rows[y].discard(x)
        fixed.append(x)
    e = [(x, y) for x in rows for y in rows[x] if x < y]
    return n, np.array([a for a, _ in e], np.int64), np.array([b for _, b in e], np.int64)


# 64-source blocks: 1, 2, 3, 5, 6, 7, 13, 32, 33 and 36 of them
SIZES = [50, 66, 190, 300, 380, 447, 821, 2048, 2049, 2250]


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("precision", [1, 0])
def test_tgt_groups(sc, n, precision):
    n, u, v = exact_degree_graph(n, n)
    if n > 300:
        deg = gg.degrees(n, u, v)
        assert {8, 16, 17, 255, 256, 257} <= set(deg[[7 * i for i in range(9)]].tolist())
    print(f"[gpu] group steps n={n} m={len(u)} precision={precision}", flush=True)
    g = sc.sc_build_graph(n, u, v)
    G = otgt.Graph(n, u, v)
    tol = 1e-12 if precision else 2e-5
    for L, eps in ((3, 0.5), (6, 0.5), (0, 0.05)):   # L = 0: last steps differ by block
        o = sc.sc_default_options(method=sc.SC_TGT, precision=precision, max_L=11)
        tau = np.empty(g.m, np.int32)
        out, _ = sc.sc_all_edges_ex(g, eps, L, o, tau_out=tau)
        np.testing.assert_allclose(out, otgt.truncated_sc(G, tau), atol=tol, rtol=0)
    g.free()


@pytest.mark.parametrize("n,tilde", [(190, 2), (447, 3), (2250, 2), (2250, 4)])
def test_tgt_plus_groups(sc, n, tilde):
    n, u, v = exact_degree_graph(n, n + 1)
    print(f"[gpu] group tails n={n} m={len(u)} tilde={tilde}", flush=True)
    g = sc.sc_build_graph(n, u, v)
    m = g.m
    o = sc.sc_default_options(method=sc.SC_TGT_PLUS, precision=1, tilde_tau=tilde, max_L=7)
    tau = np.empty(m, np.int32)
    tt = np.empty(n, np.int32)
    nr = np.empty(2 * m, np.int64)
    out, st = sc.sc_all_edges_ex(g, 0.4, 0, o, tau_out=tau, tilde_tau_out=tt, nr_out=nr)
    G = otgt.Graph(n, u, v)
    rng = np.random.default_rng(1)
    pick = np.unique(np.concatenate([rng.choice(m, 40, replace=False), [0, m - 1]]))
    srcs = np.unique(np.concatenate([u[pick], v[pick]]))
    ref = otgt.tgt_plus_replay(G, tau, tt, nr[:m], nr[m:], seed=o.seed, sources=srcs)[-1]
    both = np.isin(u, srcs) & np.isin(v, srcs)
    assert both.sum() >= len(pick)
    np.testing.assert_allclose(out[both], ref[both], atol=1e-12, rtol=0)
    g.free()


def test_mask_state_survives_changing_precision_and_width(sc):
    # one handle, runs of different slice counts, widths and group layouts in turn
    n, u, v = exact_degree_graph(821, 3)
    G = otgt.Graph(n, u, v)
    g = sc.sc_build_graph(n, u, v)
    ref = otgt.truncated_sc(G, np.full(g.m, 5))
    for precision, block in ((0, 64), (1, 64), (0, 16), (1, 32), (0, 64), (1, 64), (0, 32)):
        o = sc.sc_default_options(method=sc.SC_TGT, precision=precision, block=block)
        out, _ = sc.sc_all_edges_ex(g, 0.5, 5, o)
        np.testing.assert_allclose(out, ref, atol=1e-12 if precision else 2e-5, rtol=0)
    g.free()
