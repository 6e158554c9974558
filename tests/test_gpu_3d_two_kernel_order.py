"""The two-kernel 3-D step on either side of the size from which its rows are no longer dealt to the XCDs
in eighths, and past it with ragged blocks, bit for bit against the walk."""
import numpy as np
import pytest

from paper_0807_0602_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,nz", [(200, 200, 99), (200, 200, 100), (130, 181, 171), (1021, 61, 67)])
def test_rows_side_by_side_equal_the_walk(nx, ny, nz):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0807_0602_amd import scf
    print(f"case: 3-D two kernels {nx}x{ny}x{nz}", flush=True)
    rng = np.random.default_rng(nx)
    left = np.arange(nx) < nx // 3
    f = [np.where(left, a, b) + rng.uniform(-1e-3, 1e-3, (nz, ny, nx)) for a, b in ((2.0, 0.06), (0.06, 2.0))]
    out = []
    for fused in (False, True):
        ch = scf.Channel3(nx, ny, nz, nx // 4, nx - nx // 4, inputs.Params(gw=(-0.2, 0.15), tau=(1.25, 0.8)), *f,
                          walls_y=True, walls_z=True)
        ch.set_schedule(fused, 9)
        ch.step(4)
        out.append((ch.density(), ch.observe()["mass"]))
        ch.close()
    assert all(np.array_equal(x, y) for x, y in zip(*(o[0] for o in out))) and out[0][1] == out[1][1]
