"""lambda* where a Lanczos run ends otherwise than by converging, and at the row lengths
where the matrix product changes hands.

* a run that reaches its step limit (600) is not converged: lambda_converged is 0 and
  the value still carries the residual norm where that leaves it below 1.  King-move
  torus of 301 x 301 nodes: the eigenvalues are ((1 + 2 cos a)(1 + 2 cos b) - 1) / 8
  over a, b = 2 pi k / 301, the largest non-trivial one is 1.6e-4 from its neighbour,
  so 600 steps leave a residual near 1e-6.  On the cycle with chords of length 2 the
  residual exceeds the distance to 1;
* a Krylov space that closes within the first steps (complete graphs: one step);
* rows of 31, 32, 33 and 64 neighbours: the longest that 8 lanes sum, the first that a
  wave sums, and a whole wave.

An upper estimate may exceed the eigenvalue by the residual (1e-9 where converged).
"""
import numpy as np
import pytest

import graphgen as gg
from test_gpu_lanczos import nmat, sc  # noqa: F401

pytestmark = pytest.mark.gpu


def torus(k):
    x = np.arange(k * k).reshape(k, k)
    pairs = [(x, np.roll(x, s, axis=(0, 1))) for s in ((0, 1), (1, 0), (1, 1), (1, -1))]
    u = np.concatenate([a.ravel() for a, _ in pairs])
    v = np.concatenate([b.ravel() for _, b in pairs])
    u, v = gg.canonical_edges(k * k, u, v)
    return k * k, u, v


def converged(sc, g):  # noqa: F811
    o = sc.sc_default_options(method=sc.SC_TGT, max_L=3)
    _, st = sc.sc_all_edges_ex(g, 0.5, 0, o)
    return st["lambda_converged"]


def test_step_limit_is_not_convergence(sc):  # noqa: F811
    k = 301
    n, u, v = torus(k)
    assert len(u) == 4 * n
    t = 2 * np.pi / k
    ref = (3 * (1 + 2 * np.cos(t)) - 1) / 8
    g = sc.sc_build_graph(n, u, v)
    lam = sc.sc_lambda_star(g)
    print(f"[gpu] lambda* of a torus {lam} {ref}", flush=True)
    assert converged(sc, g) == 0
    assert ref <= lam < 1.0
    g.free()


def test_step_limit_with_a_residual_beyond_one(sc):  # noqa: F811
    n = 20001
    x = np.arange(n)
    u, v = gg.canonical_edges(n, np.r_[x, x], np.r_[(x + 1) % n, (x + 2) % n])
    g = sc.sc_build_graph(n, u, v)
    lam = sc.sc_lambda_star(g)
    print(f"[gpu] lambda* of a cycle with chords {lam}", flush=True)
    assert converged(sc, g) == 0
    assert 0.999 < lam < 1.0
    g.free()


@pytest.mark.parametrize("n", [3, 4, 6, 129])
def test_krylov_space_closes_at_once(sc, n):  # noqa: F811
    n, u, v = gg.complete_graph(n)
    g = sc.sc_build_graph(n, u, v)
    lam = sc.sc_lambda_star(g)
    assert abs(lam - 1.0 / (n - 1)) <= 1e-12
    assert converged(sc, g) == 1
    g.free()


def test_rows_at_the_limits_of_the_product(sc):  # noqa: F811
    # a ring of 2,000 nodes with chords, and nodes 0..3 with exactly these neighbour counts
    n, degrees = 2000, (31, 32, 33, 64)
    x = np.arange(n)
    u = np.r_[x, x]
    v = np.r_[(x + 1) % n, (x + 7) % n]
    keep = (u >= 4) & (v >= 4)
    u, v = u[keep], v[keep]
    rng = np.random.default_rng(3)
    for node, d in enumerate(degrees):
        u = np.r_[u, np.full(d, node)]
        v = np.r_[v, rng.choice(np.arange(4, n), d, replace=False)]
    u, v = gg.canonical_edges(n, u, v)
    assert gg.degrees(n, u, v)[:4].tolist() == list(degrees)
    g = sc.sc_build_graph(n, u, v)
    lam = sc.sc_lambda_star(g)
    w = np.linalg.eigvalsh(nmat(n, u, v))
    ref = np.abs(w[:-1]).max()
    assert ref - 1e-11 <= lam <= ref + 1e-8
    g.free()
