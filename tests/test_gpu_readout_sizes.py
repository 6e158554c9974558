"""Density read-outs on either side of the sizes where the way to the host changes (page-locked memory, FP32
widened in the caller's arrays, FP64), into arrays that start off their alignment: the FP32 sums of the
populations of the same state, as the read-out's definition has them, bit for bit."""
import ctypes as C

import numpy as np
import pytest

from paper_0807_0602_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def scf():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0807_0602_amd import scf as S
    return S


def _sums(f):
    """Running FP32 sums over the directions, in order."""
    s = np.zeros(f.shape[1:], np.float32)
    for q in f:
        s += q.astype(np.float32)
    return s


def _read(call, handle, n):
    """Both fields into arrays 8 bytes off a 16-byte boundary, with guards around them."""
    from paper_0807_0602_amd import _lib as L
    mem = [np.full(n + 9, -7.0) for _ in range(2)]
    fields = [m[(1 if m.ctypes.data % 16 == 0 else 2):][:n] for m in mem]
    L.check(call(handle, *(f.ctypes.data_as(C.POINTER(C.c_double)) for f in fields)))
    for m in mem:
        assert (m == -7.0).sum() == 9
    return fields


# 65536 nodes through page-locked memory, 5242880 in FP32
@pytest.mark.parametrize("nx,ny", [(1021, 64), (1024, 64), (1025, 64), (331, 211), (2048, 2560), (2053, 2557)])
def test_channel(scf, nx, ny):
    from paper_0807_0602_amd import _lib as L
    print(f"case: density read-out {nx} x {ny}", flush=True)
    left = np.arange(nx) < nx // 3
    rng = np.random.default_rng(nx)
    f = [np.where(left, a, b) + rng.uniform(-1e-3, 1e-3, (ny, nx)) for a, b in ((2.0, 0.06), (0.06, 2.0))]
    ch = scf.Channel(inputs.Geometry(nx, ny, nx // 4, nx // 2), inputs.Params(gw=(-0.2, 0.2)), *f)
    ch.step(3)
    got = _read(L.scf_get_density, ch._h, nx * ny)
    for n, pops in zip(got, ch.populations()):
        assert np.array_equal(n.reshape(ny, nx), _sums(pops))


@pytest.mark.parametrize("nx,ny,nz", [(64, 32, 32), (65, 32, 32), (101, 61, 53)])
def test_channel_3d(scf, nx, ny, nz):
    from paper_0807_0602_amd import _lib as L
    print(f"case: density read-out {nx} x {ny} x {nz}", flush=True)
    left = np.arange(nx) < nx // 3
    rng = np.random.default_rng(nx)
    f = [np.where(left, a, b) + rng.uniform(-1e-3, 1e-3, (nz, ny, nx)) for a, b in ((2.0, 0.06), (0.06, 2.0))]
    ch = scf.Channel3(nx, ny, nz, nx // 4, nx // 2, inputs.Params(gw=(-0.2, 0.2)), *f, walls_y=True, walls_z=True)
    ch.step(3)
    got = _read(L.scf3_get_density, ch._h, nx * ny * nz)
    for n, pops in zip(got, ch.populations()):
        assert np.array_equal(n.reshape(nz, ny, nx), _sums(pops))
