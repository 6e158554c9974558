"""Predictions by the whole-network kernel (widths up to 256) and by the layer kernels (wider), at
the edges of their row tiles, against the FP64 reference: BF16 hidden layers keep the bound of
test_gpu_surrogate (relative L2 < 3e-2).  The device-pointer form gives the same bits."""
import ctypes as C

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


def _network(S, d_in, width, depth, seed, max_batch=64):
    rng = np.random.default_rng(seed)
    theta = np.concatenate([np.concatenate([rng.normal(0, 1 / np.sqrt(i), o * i), rng.normal(0, 0.3, o)])
                            for o, i in mlp.layer_shapes(d_in, width, depth)]).astype(np.float32)
    net = S.Network(d_in, width, depth, max_batch=max_batch, max_data=64, seed=seed)
    net.set_params(theta)
    net.set_norm(np.full(d_in, 0.1), np.full(d_in, 1.5), np.full(d_in, -1.0), np.full(d_in, 1.0))
    return net, theta.astype(np.float64)


@pytest.mark.parametrize("d_in,width,depth", [(1, 64, 1), (5, 64, 3), (4, 128, 2), (32, 192, 2), (32, 256, 4), (5, 256, 4),
                                              (5, 256, 1), (5, 320, 2)])
@pytest.mark.parametrize("rows", [1, 16, 17, 4096, 4097, 4129])
def test_predict_matches_reference(sur, d_in, width, depth, rows):
    import torch
    from paper_0807_0602_amd import _lib as L
    print(f"case: predict d_in={d_in} width={width} depth={depth} rows={rows}", flush=True)
    net, theta = _network(sur, d_in, width, depth, seed=rows + width)
    X = np.random.default_rng(rows).normal(size=(rows, d_in)).astype(np.float32)
    Y, inside = net.predict(X)
    x64 = (X.astype(np.float64) - np.float32(0.1)) / 1.5
    ref, _, _ = mlp.forward(theta, x64, d_in, width, depth)
    assert np.isfinite(Y).all()
    assert np.linalg.norm(Y - ref) < 3e-2 * np.linalg.norm(ref)
    assert np.array_equal(inside, (np.abs(X) <= 1.0).all(axis=1))
    if width > 256:
        return
    Xd = torch.from_numpy(X).to("cuda:0")
    Yd = torch.full((rows, 2), float("nan"), device="cuda:0")
    Hd = torch.full((rows,), 7, dtype=torch.uint8, device="cuda:0")
    L.check(L.scf_sur_predict_noalloc(net._h, C.c_void_p(Xd.data_ptr()), rows, C.c_void_p(Yd.data_ptr()),
                                      C.c_void_p(Hd.data_ptr())))
    torch.cuda.synchronize()
    assert np.array_equal(Yd.cpu().numpy(), Y) and np.array_equal(Hd.cpu().numpy().astype(bool), inside)


def test_no_hull_before_data_and_nan_inputs(sur):
    """Without data or norm every row is outside the hull; NaN inputs are outside and give NaN."""
    net = sur.Network(3, 128, 2, max_batch=64, max_data=64, seed=1)
    X = np.zeros((40, 3), np.float32)
    assert not net.predict(X)[1].any()
    net.set_norm(np.zeros(3), np.ones(3), np.full(3, -1.0), np.full(3, 1.0))
    X[7, 1] = np.nan
    Y, inside = net.predict(X)
    assert np.isnan(Y[7]).all() and not inside[7] and inside.sum() == 39 and np.isfinite(np.delete(Y, 7, 0)).all()
