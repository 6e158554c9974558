"""Walks of so few tiles that a CU gets one at most take the tile shape of half the threads; explicit
schedules of such boxes, bit for bit against the two-kernel step."""
import numpy as np
import pytest

from paper_0807_0602_amd import inputs

pytestmark = pytest.mark.gpu


# 128 x 4 tiles: 256, the most that one per CU takes, 260, and few
@pytest.mark.parametrize("nx,ny,nz,cy", [(256, 32, 64, 4), (256, 33, 65, 8), (260, 25, 40, 5), (40, 100, 30, 4), (300, 40, 21, 64)])
def test_few_tiles_equal_two_kernels(nx, ny, nz, cy):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0807_0602_amd import scf
    print(f"case: 3-D walk of few tiles {nx}x{ny}x{nz} cy={cy}", flush=True)
    rng = np.random.default_rng(nx)
    left = np.arange(nx) < nx // 3
    f = [np.where(left, a, b) + rng.uniform(-1e-3, 1e-3, (nz, ny, nx)) for a, b in ((2.0, 0.06), (0.06, 2.0))]
    out = []
    for fused in (False, True):
        ch = scf.Channel3(nx, ny, nz, nx // 4, nx - nx // 4, inputs.Params(gw=(-0.2, 0.15), tau=(1.25, 0.8)), *f,
                          walls_y=True, walls_z=True)
        ch.set_schedule(fused, cy)
        out.append(ch.step(5).populations())
        ch.close()
    assert np.array_equal(*out)


def test_few_tiles_take_smaller_blocks():
    """300 x 120 x 90 in 60 rows: 575 us per step with 92 tiles of 256 x 4, 444 with 138 of 128 x 4; two
    kernels, which the bound refers to, take 385."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0807_0602_amd import scf
    print("case: 3-D walk of few tiles, time", flush=True)
    left = np.arange(300) < 75
    f = [np.where(left, a, b) + np.zeros((90, 120, 300)) for a, b in ((2.0, 0.06), (0.06, 2.0))]
    ch = scf.Channel3(300, 120, 90, 75, 225, inputs.Params(gw=(-0.2, 0.2)), *f, walls_y=True, walls_z=True)
    ms = []
    for fused in (False, True):
        ch.set_schedule(fused, 60)
        ch.step(10)
        best = np.inf
        for _ in range(5):
            e0, e1 = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            e0.record()
            ch.step(20)
            e1.record()
            e1.synchronize()
            best = min(best, e0.elapsed_time(e1) / 20)
        ms.append(best)
    print(f"  two kernels {ms[0]:.4f} ms per step, walk of 60 rows {ms[1]:.4f}", flush=True)
    assert ms[1] < 1.3 * ms[0]
