"""Device predictions whose outputs lie over their inputs (scf_sur_predict_noalloc): Y from the start
of X or from inside it, the hull flags over X, before any norm is set too.  Each gives the bits of
scf_sur_predict, at widths whose separate outputs come from the whole-network kernel (so that this also
holds it to the layer kernels) and at wider ones."""
import ctypes as C

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

ROWS = 300


@pytest.fixture(scope="module")
def sur():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0807_0602_amd import surrogate
    return surrogate


@pytest.mark.parametrize("d_in,width,depth", [(1, 64, 1), (2, 128, 2), (5, 256, 4), (5, 320, 2)])
# floats from X to Y and bytes from X to the flags, None: a buffer of its own
@pytest.mark.parametrize("y_at,in_at", [(0, None), (7, None), (None, 0), (None, 4 * ROWS - 10), (0, 8 * ROWS)])
@pytest.mark.parametrize("norm", [True, False])
def test_outputs_over_inputs(sur, d_in, width, depth, y_at, in_at, norm):
    import torch
    from paper_0807_0602_amd import _lib as L
    print(f"case: outputs over inputs {d_in} {width}x{depth} Y {y_at} flags {in_at} norm={norm}", flush=True)
    net = sur.Network(d_in, width, depth, max_batch=512, max_data=64, seed=3)
    if norm:
        net.set_norm(np.full(d_in, 0.1), np.full(d_in, 1.5), np.full(d_in, -1.0), np.full(d_in, 1.0))
    X = np.random.default_rng(width + d_in).uniform(-1.1, 1.1, (ROWS, d_in)).astype(np.float32)
    want, inside = net.predict(X)
    assert not norm or 0 < inside.sum() < ROWS
    pool = torch.zeros((max(4 * d_in, 12) + 16) * ROWS, dtype=torch.uint8, device="cuda:0")
    pool[: 4 * ROWS * d_in] = torch.from_numpy(X.reshape(-1).view(np.uint8)).to("cuda:0")
    own = torch.empty(ROWS * 9, dtype=torch.uint8, device="cuda:0")
    y = (own, 0) if y_at is None else (pool, 4 * y_at)
    f = (own, 8 * ROWS) if in_at is None else (pool, in_at)
    L.check(L.scf_sur_predict_noalloc(net._h, C.c_void_p(pool.data_ptr()), ROWS, C.c_void_p(y[0].data_ptr() + y[1]),
                                      C.c_void_p(f[0].data_ptr() + f[1])))
    torch.cuda.synchronize()
    got = y[0][y[1]: y[1] + 8 * ROWS].cpu().numpy().view(np.float32).reshape(ROWS, 2)
    flags = f[0][f[1]: f[1] + ROWS].cpu().numpy()
    assert np.array_equal(got, want) and np.array_equal(flags.astype(bool), inside) and flags.max() <= 1
    net.close()
