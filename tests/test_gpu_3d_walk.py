"""The three tile shapes of the 3-D walk (256 x 4, 128 x 4, 64 x 8 nodes of x and z), the schedule a
new context picks and the two-kernel step with 64-bit addresses, bit for bit against the two-kernel
step at boxes with ragged tiles, boxes narrower than a tile and walls on every side."""
import numpy as np
import pytest

from paper_0807_0602_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def S():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0807_0602_amd import scf
    return scf


def _fields(nx, ny, nz, seed):
    rng = np.random.default_rng(seed)
    liq = np.arange(nx) < max(1, nx // 3)
    return [np.where(liq, a, b) + rng.uniform(-1e-3, 1e-3, (nz, ny, nx)) for a, b in ((2.0, 0.06), (0.06, 2.0))]


# x sizes at which each shape leaves the fewest columns idle, and z sizes around 4 and 8
@pytest.mark.parametrize("nx,ny,nz,x0,x1,wy,wz", [
    (3, 3, 3, 1, 2, True, True), (40, 7, 9, 0, 12, True, False), (64, 9, 8, 16, 64, True, True),
    (65, 5, 17, 10, 50, False, True), (128, 6, 4, 0, 128, True, True), (130, 11, 5, 30, 100, True, False),
    (256, 8, 4, 64, 192, True, True), (300, 5, 13, 0, 0, False, False), (513, 4, 6, 100, 513, True, True)])
@pytest.mark.parametrize("cy", [1, 3, 64])
def test_walk_equals_two_kernels(S, nx, ny, nz, x0, x1, wy, wz, cy):
    print(f"case: 3-D walk {nx}x{ny}x{nz} walls {wy} {wz} cy={cy}", flush=True)
    a, b = _fields(nx, ny, nz, nx + nz)
    prm = inputs.Params(G=0.9, gw=(-0.2, 0.15), tau=(1.25, 0.8))
    out = []
    for fused in (True, False, None):
        ch = S.Channel3(nx, ny, nz, x0, x1, prm, a, b, walls_y=wy, walls_z=wz)
        if fused is None:
            assert ch.schedule() == {"fused": True, "cy": 16}
        else:
            ch.set_schedule(fused, cy)
        out.append(ch.step(5).populations())
    assert np.array_equal(out[0], out[1]) and np.array_equal(out[2], out[1])


@pytest.mark.parametrize("nx,ny,nz", [(300, 121, 90), (512, 96, 96), (130, 200, 150)])
def test_default_schedule_large(S, nx, ny, nz):
    """Boxes large enough for the walk by default, past the last-level cache."""
    print(f"case: 3-D default schedule {nx}x{ny}x{nz}", flush=True)
    a, b = _fields(nx, ny, nz, 5)
    prm = inputs.Params(G=0.9, gw=(-0.2, 0.2))
    out = []
    for two in (False, True):
        ch = S.Channel3(nx, ny, nz, nx // 4, nx - nx // 4, prm, a, b, walls_y=True, walls_z=True)
        if two:
            ch.set_schedule(False)
        out.append(ch.step(4).density())
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])


def test_wide_two_kernel_step(S):
    """A box whose components pass 4 GiB (64-bit addresses): a z-independent slit equals the same
    slit four nodes deep in every z slice."""
    nx, ny, nz = 512, 340, 340
    print(f"case: 3-D wide {nx}x{ny}x{nz}", flush=True)
    a, b = _fields(nx, ny, 1, 3)
    prm = inputs.Params(G=0.9, gw=(-0.2, 0.2))
    dens = []
    for depth in (4, nz):
        ch = S.Channel3(nx, ny, depth, 128, 384, prm, *(np.ascontiguousarray(np.broadcast_to(f, (depth, ny, nx)))
                                                        for f in (a, b)), walls_y=True)
        assert ch.schedule()["fused"] == (depth == 4)
        dens.append(ch.step(4).density())
        ch.close()
    for k in range(2):
        assert (dens[1][k] == dens[0][k][:1]).all()
