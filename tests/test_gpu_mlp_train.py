"""The closure network's training kernels against the float64 reference at the sizes
where their tiling can go wrong: less than one 16-sample tile, tile remainders, one
tile per workgroup, and more tiles than workgroups (several tiles each).

Tolerance: a gradient component is a sum over samples of products that pass through
at most ~150 FP32 operations, and the sum itself takes at most ~100 additions in a
row, each with relative rounding 2^-24 of the running sum of magnitudes: 250 * 6e-8
= 1.5e-5 of the sum of the terms' magnitudes (2e-5 with the fast exponential).
"""
import numpy as np
import pytest

from oracle import mlp as omlp

pytestmark = pytest.mark.gpu


def _abs_grad(theta, X, z, w):
    """Gradient and, per component, the sum of its terms' magnitudes (weights 0/1)."""
    p = omlp.unpack(theta)
    y, (X, a1, h1, a2, h2) = omlp.forward(theta, X)
    dy = (2.0 / len(z)) * (w * (y - z))[:, None]
    da2 = (dy @ p["W3"]) * omlp.silu_grad(a2)
    da1 = (da2 @ p["W2"]) * omlp.silu_grad(a1)
    ab1 = (np.abs(da2) @ np.abs(p["W2"])) * np.abs(omlp.silu_grad(a1))
    g = {"W1": da1.T @ X, "b1": da1.sum(0), "W2": da2.T @ h1, "b2": da2.sum(0),
         "W3": dy.T @ h2, "b3": dy.sum(0)}
    a = {"W1": ab1.T @ np.abs(X), "b1": ab1.sum(0), "W2": np.abs(da2).T @ np.abs(h1),
         "b2": np.abs(da2).sum(0), "W3": np.abs(dy).T @ np.abs(h2), "b3": np.abs(dy).sum(0)}
    return omlp.pack(g), omlp.pack(a), float(np.mean(w * (y - z) ** 2))


@pytest.mark.parametrize("N,weighted", [(1, False), (15, True), (16, False), (17, True),
                                        (8192, True), (8193, True), (20011, False)])
def test_gradient_and_first_adam_step(N, weighted):
    import torch
    from paper_2305_16086_amd import sc
    rng = np.random.default_rng(N)
    Xh = rng.normal(size=(N, 16)).astype(np.float32)
    zh = rng.normal(size=N).astype(np.float32)
    wh = (rng.random(N) > 0.2).astype(np.float32) if weighted else np.ones(N, np.float32)
    net = sc.sc_mlp_create(5)
    ident = np.concatenate([np.zeros(16), np.ones(16)]).astype(np.float32)
    sc.sc_mlp_set(net, norm=ident, range_=np.concatenate([-9 * np.ones(16), 9 * np.ones(16)]))
    th = sc.sc_mlp_get(net)[0].astype(np.float64)
    X, z = torch.from_numpy(Xh).cuda().reshape(-1), torch.from_numpy(zh).cuda()
    w = torch.from_numpy(wh).cuda() if weighted else None
    g, loss = sc.sc_mlp_grad(net, X, z, w)
    ref, mag, ref_loss = _abs_grad(th, Xh.astype(np.float64), zh.astype(np.float64),
                                   wh.astype(np.float64))
    tol = 2e-5 * mag + 1e-12
    assert abs(loss - ref_loss) <= 2e-5 * (ref_loss + 1.0)
    assert np.all(np.abs(g - ref) <= tol)
    # one Adam step on the whole set: theta - lr g / (|g| + 1e-8)
    lr = 2e-3
    losses = sc.sc_mlp_train(net, X, z, w, sc.sc_default_train_options(epochs=1, batch=N, lr=lr))
    new = sc.sc_mlp_get(net)[0]
    step = lr * ref / (np.abs(ref) + 1e-8)
    err = np.abs(new - (th - step))
    assert np.all(err <= lr * np.minimum(2.0, tol / (np.abs(ref) + 1e-8)) + 1e-6)
    assert abs(losses[0] - ref_loss) <= 2e-5 * (ref_loss + 1.0)


def test_training_is_deterministic():
    import torch
    from paper_2305_16086_amd import sc
    rng = np.random.default_rng(8)
    N = 5003
    X = torch.from_numpy(rng.normal(size=(N, 16)).astype(np.float32)).cuda()
    z = torch.from_numpy(rng.normal(size=N).astype(np.float32)).cuda()
    out = []
    for _ in range(2):
        net = sc.sc_mlp_create(3)
        sc.sc_mlp_train(net, X, z, None, sc.sc_default_train_options(epochs=2, batch=1000))
        out.append(sc.sc_mlp_get(net)[0])
    np.testing.assert_array_equal(out[0], out[1])
