"""The Lanczos runs behind lambda* and the spectrum, at the sizes where their chunking
can go wrong: fewer rows than one chunk, chunk remainders, more than one chunk per 64
rows, rows summed by 8 lanes (128 neighbours and fewer), by a wave (129 and more) and
by a workgroup (above 4,096), and a basis of more than one update segment (1,024
columns).  Against numpy's dense eigensolver.

lambda* is an upper estimate: the largest Ritz value plus a residual below 1e-9.  The
spectrum's eigenvalues converge with the square of the residual (tolerance 1e-8), its
vectors' residuals are within it plus FP64 rounding over the basis.
"""
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


def nmat(n, u, v):
    d = gg.degrees(n, u, v)
    N = np.zeros((n, n))
    N[u, v] = N[v, u] = 1.0 / np.sqrt(d[u] * d[v])
    return N


def with_hubs(n, degrees, seed):
    n, u, v = gg.tree_plus_gnp(n, 8.0, seed)
    rng = np.random.default_rng(seed)
    for x, d in enumerate(degrees):
        t = rng.choice(np.arange(len(degrees), n), size=d, replace=False)
        u = np.concatenate([u, np.full(d, x)])
        v = np.concatenate([v, t])
    u, v = gg.canonical_edges(n, u, v)
    return n, u, v


@pytest.mark.parametrize("n,hubs", [(3, ()), (40, ()), (64, ()), (65, ()), (1000, (120, 130)),
                                    (3001, (127, 128, 129, 2500))])
def test_lambda_star(sc, n, hubs):
    graph = gg.complete_graph(3) if n == 3 else with_hubs(n, hubs, n) if hubs else \
        gg.tree_plus_gnp(n, 8.0, n)
    n, u, v = graph
    g = sc.sc_build_graph(n, u, v)
    lam = sc.sc_lambda_star(g)
    w = np.linalg.eigvalsh(nmat(n, u, v))
    ref = np.abs(w[:-1]).max()
    print(f"[gpu] lambda* n={n} {lam} {ref}", flush=True)
    assert ref - 1e-11 <= lam <= ref + 1e-8
    g.free()


def test_lambda_star_giant_row(sc):
    # a row above 4,096 neighbours; the reference by power iteration on the deflated matrix
    import scipy.sparse as sp
    import scipy.sparse.linalg as spl
    n, u, v = with_hubs(9000, (5000, 300), 5)
    d = gg.degrees(n, u, v).astype(float)
    A = sp.coo_matrix((1 / np.sqrt(d[u] * d[v]), (u, v)), shape=(n, n))
    N = (A + A.T).tocsr()
    top = np.sqrt(d / d.sum())
    op = spl.LinearOperator((n, n), matvec=lambda x: N @ x - top * (top @ x), dtype=float)
    ref = np.abs(spl.eigsh(op, k=2, which="LM", return_eigenvectors=False, tol=1e-12)).max()
    g = sc.sc_build_graph(n, u, v)
    lam = sc.sc_lambda_star(g)
    assert ref - 1e-10 <= lam <= ref + 1e-8
    g.free()


@pytest.mark.parametrize("n,omega", [(65, 20), (700, 40), (1501, 128)])
def test_spectrum_vectors(sc, n, omega):
    n, u, v = gg.tree_plus_gnp(n, 7.0, n)
    g = sc.sc_build_graph(n, u, v)
    kept, _ = sc.sc_compute_spectrum(g, omega)
    lam, phi = sc.sc_get_spectrum(g)
    assert kept == omega
    N = nmat(n, u, v)
    w = np.linalg.eigvalsh(N)
    w = w[np.argsort(-np.abs(w))]
    np.testing.assert_allclose(np.abs(lam), np.abs(w[:omega]), atol=1e-12)
    assert np.abs(N @ phi - phi * lam).max() <= 2e-8
    assert np.abs(phi.T @ phi - np.eye(omega)).max() <= 1e-8
    g.free()


def test_spectrum_basis_of_several_segments(sc):
    # all eigenpairs of a 1,300-node graph: the basis passes 1,024 columns
    n, u, v = gg.tree_plus_gnp(1300, 9.0, 4)
    g = sc.sc_build_graph(n, u, v)
    kept, _ = sc.sc_compute_spectrum(g, 256, max_iter=1299, tol=1e-30)
    lam, phi = sc.sc_get_spectrum(g)
    w = np.linalg.eigvalsh(nmat(n, u, v))
    w = w[np.argsort(-np.abs(w))]
    assert kept == 256
    np.testing.assert_allclose(np.abs(lam), np.abs(w[:256]), atol=1e-10)
    g.free()
