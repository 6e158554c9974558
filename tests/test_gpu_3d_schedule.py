"""Setting the schedule that a 3-D context reports keeps the step it runs: the default schedule is the
form chosen for the box's size, whether it was ever set or not."""
import numpy as np
import pytest

from paper_0807_0602_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,nz,steps", [(96, 24, 24, 400), (300, 121, 90, 30)])
def test_set_back_what_was_read(nx, ny, nz, steps):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0807_0602_amd import scf
    print(f"case: 3-D schedule read and set back, {nx}x{ny}x{nz}", flush=True)
    left = np.arange(nx) < nx // 4
    f = [np.where(left, a, b) + np.zeros((nz, ny, nx)) for a, b in ((2.0, 0.06), (0.06, 2.0))]
    ch = scf.Channel3(nx, ny, nz, nx // 4, 3 * nx // 4, inputs.Params(gw=(-0.2, 0.2)), *f, walls_y=True, walls_z=True)

    def ms():
        best = np.inf
        for _ in range(6):
            e0, e1 = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            e0.record()
            ch.step(steps)
            e1.record()
            e1.synchronize()
            best = min(best, e0.elapsed_time(e1))
        return best

    ms()
    default = ms()
    read = ch.schedule()
    ch.set_schedule(**read)
    assert ch.schedule() == read
    same = ms()
    ch.set_schedule(fused=not read["fused"], cy=3)
    ch.set_schedule(**read)
    again = ms()
    print(f"  {default / steps:.4f} ms per step, set back {same / steps:.4f}, after another {again / steps:.4f}", flush=True)
    assert max(same, again) < 1.5 * default    # 16 rows taken literally: 10 times at 96 x 24 x 24
