"""The two-launch training step (widths 128 and 256, 2-4 hidden layers) and the layer kernels beside
it: gradients against the FP64 reference with the bounds of test_gpu_surrogate (cosine > 0.999,
relative L2 < 2e-2 per block), the Adam update against its formula in FP64, and the BF16 weights
that an update leaves against those of a network given the same parameters."""
import numpy as np
import pytest

from oracle import mlp

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sur():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0807_0602_amd import surrogate
    return surrogate


def _theta(rng, d_in, width, depth):
    return np.concatenate([np.concatenate([rng.normal(0, 1 / np.sqrt(i), o * i), rng.normal(0, 0.3, o)])
                           for o, i in mlp.layer_shapes(d_in, width, depth)]).astype(np.float32)


def _problem(rng, n, d_in):
    return (rng.normal(size=(n, d_in)).astype(np.float32), rng.normal(0, 0.5, (n, 2)).astype(np.float32),
            rng.uniform(0.5, 2.0, n).astype(np.float32))


# row counts around the 64-row padding, the 128-row chunks and the 256-row groups of the sums
@pytest.mark.parametrize("d_in,width,depth", [(1, 128, 2), (32, 256, 2), (5, 256, 3), (4, 128, 4), (5, 192, 3), (5, 256, 5)])
@pytest.mark.parametrize("n", [1, 65, 128, 257, 330, 1090])
def test_gradients(sur, d_in, width, depth, n):
    print(f"case: train gradients d_in={d_in} width={width} depth={depth} rows={n}", flush=True)
    rng = np.random.default_rng(n + width + depth)
    theta = _theta(rng, d_in, width, depth)
    net = sur.Network(d_in, width, depth, max_batch=1152, max_data=64, seed=3)
    net.set_params(theta)
    X, T, w = _problem(rng, n, d_in)
    loss, g = net.grad(X, T, w)
    lo, go = mlp.loss_and_grad(theta.astype(np.float64), *(a.astype(np.float64) for a in (X, T, w)), d_in, width, depth)
    assert abs(loss - lo) <= 2e-2 * lo
    p = 0
    for o, i in mlp.layer_shapes(d_in, width, depth):
        for size in (o * i, o):
            a, b = g[p:p + size].astype(np.float64), go[p:p + size]
            p += size
            assert a @ b > 0.999 * np.linalg.norm(a) * np.linalg.norm(b)
            assert np.linalg.norm(a - b) < 2e-2 * np.linalg.norm(b)
    assert np.array_equal(net.grad(X, T, w)[1], g) and np.array_equal(net.params(), theta)


# 16 rows per block up to 4096 rows (256 units) or 8192 (128 units), 32 beyond
@pytest.mark.parametrize("d_in,width,depth,n", [(5, 256, 4, 4096), (5, 256, 3, 4097), (4, 128, 2, 8192), (5, 128, 3, 8200)])
def test_gradients_of_large_batches(sur, d_in, width, depth, n):
    print(f"case: train gradients d_in={d_in} width={width} depth={depth} rows={n}", flush=True)
    rng = np.random.default_rng(n + width + depth)
    theta = _theta(rng, d_in, width, depth)
    net = sur.Network(d_in, width, depth, max_batch=8256, max_data=64, seed=3)
    net.set_params(theta)
    X, T, w = _problem(rng, n, d_in)
    loss, g = net.grad(X, T, w)
    lo, go = mlp.loss_and_grad(theta.astype(np.float64), *(a.astype(np.float64) for a in (X, T, w)), d_in, width, depth)
    assert abs(loss - lo) <= 2e-2 * lo
    p = 0
    for o, i in mlp.layer_shapes(d_in, width, depth):
        for size in (o * i, o):
            a, b = g[p:p + size].astype(np.float64), go[p:p + size]
            p += size
            assert a @ b > 0.999 * np.linalg.norm(a) * np.linalg.norm(b)
            assert np.linalg.norm(a - b) < 2e-2 * np.linalg.norm(b)


@pytest.mark.parametrize("d_in,width,depth,n", [(5, 256, 4, 192), (4, 128, 2, 64), (5, 320, 2, 64)])
def test_update_follows_adam(sur, d_in, width, depth, n):
    rng = np.random.default_rng(n)
    theta = _theta(rng, d_in, width, depth)
    lr, b1, b2, eps = 1e-3, 0.9, 0.999, 1e-8
    net = sur.Network(d_in, width, depth, max_batch=256, max_data=64, lr=lr, seed=3)
    net.set_params(theta)
    m = np.zeros(theta.size)
    v = np.zeros(theta.size)
    for t in (1, 2, 3):
        X, T, w = _problem(rng, n, d_in)
        before = net.params().astype(np.float64)
        g = net.grad(X, T, w)[1].astype(np.float64)
        net.step(X, T, w)
        m = b1 * m + (1 - b1) * g
        v = b2 * v + (1 - b2) * g * g
        want = before - lr * (m / (1 - b1 ** t)) / (np.sqrt(v / (1 - b2 ** t)) + eps)
        # FP32 rounding of theta and of the update (|update| <= a few lr, eight roundings of 2^-24,
        # 1 - b2^t formed from the rounded b2: 2^-24 / 1e-3 relative)
        tol = 2.0 ** -23 * np.abs(before).max() + 4 * lr * (8 * 2.0 ** -24 + 2.0 ** -24 / 1e-3)
        assert np.abs(net.params() - want).max() <= tol
    fresh = sur.Network(d_in, width, depth, max_batch=256, max_data=64, seed=9)
    fresh.set_params(net.params())
    X, T, w = _problem(rng, n, d_in)
    assert np.array_equal(fresh.predict(X)[0], net.predict(X)[0])
    assert np.array_equal(fresh.grad(X, T, w)[1], net.grad(X, T, w)[1])
