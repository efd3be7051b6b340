"""The training kernels (forward and backward in one pass, weight gradients over parts of
the batch, their sum with Adam) at batch sizes around their edges: the smallest batch
(one part), parts that end short or stay empty, and more rows than one part holds."""

import numpy as np
import pytest

from oracle import mlp as M

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [128, 640, 1152, 4224])
def test_gradients_and_step_at_batch_edges(B):
    """Every gradient element within 2^-6 of the sum of its absolute terms: each product's
    two bfloat16 factors may sit one rounding flip (2^-7 relative) away on the GPU, and
    the FP32 sums over at most 4224 rows err by less than 4224 * 2^-24 = 2.5e-4 of it.
    Nothing in a step depends on scheduling, so two calls agree bit for bit."""
    from paper_1707_05163_amd import Surrogate
    s = Surrogate(3)
    rng = np.random.default_rng(B)
    layers = [(W, (rng.standard_normal(b.shape) * 0.05).astype(np.float32))
              for W, b in s.get_params()]
    s.set_params(layers)
    for (W, b), (W2, b2) in zip(layers, s.get_params()):
        assert np.array_equal(W, W2) and np.array_equal(b, b2)
    X = np.zeros((B, 64), np.float32)
    X[:, :60] = rng.standard_normal((B, 60)) * 0.5
    T = (rng.standard_normal((B, 2)) * 0.3).astype(np.float32)
    g, loss = s.gradients(X, T)
    g2, loss2 = s.gradients(X, T)
    assert loss == loss2
    W = [w.astype(np.float64) for w, _ in layers]
    b = [v.astype(np.float64) for _, v in layers]
    yo, cache = M.forward(W, b, X.astype(np.float64), mirror=True)
    dW, db = M.backward(W, b, cache, yo, T.astype(np.float64), mirror=True)
    hs, zs = cache
    dz = (yo - T.astype(np.float64)) / B
    for l in range(4, -1, -1):
        dzq = M._q(dz, True)
        assert np.array_equal(g[l][0], g2[l][0]) and np.array_equal(g[l][1], g2[l][1]), l
        assert (np.abs(g[l][0] - dW[l]) <= 2.0 ** -6 * (np.abs(hs[l]).T @ np.abs(dzq))
                + 1e-30).all(), l
        assert (np.abs(g[l][1] - db[l]) <= 2.0 ** -6 * np.abs(dz).sum(axis=0) + 1e-30).all(), l
        if l > 0:
            dz = (dzq @ M._q(W[l], True).T) * M.gelu_grad(zs[l - 1])
    # the first Adam step from these gradients: lr g / (|g| + eps), in FP32 (2 ulp of the
    # weight, and of the step itself a few 2^-22)
    assert s.train_step(X, T, lr=1e-3) == loss
    for l, (W2, b2) in enumerate(s.get_params()):
        for new, old, q in ((W2, layers[l][0], g[l][0]), (b2, layers[l][1], g[l][1])):
            step = 1e-3 * q.astype(np.float64) / (np.abs(q.astype(np.float64)) + 1e-8)
            tol = 2.0 ** -22 * np.abs(old) + 1e-3 * 2.0 ** -10
            assert (np.abs(new - (old - step)) <= tol).all(), l
