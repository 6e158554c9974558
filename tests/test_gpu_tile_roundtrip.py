"""Tiles kept as given by an explicit number of blocks per CU: what scf_get_tile reports, set back, runs
the same step, and a number above the occupancy counts as one."""
import numpy as np
import pytest

from paper_0807_0602_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _us(torch, ch, steps=96):
    ch.step(steps)
    best = np.inf
    for _ in range(6):
        e0, e1 = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        e0.record()
        ch.step(steps)
        e1.record()
        e1.synchronize()
        best = min(best, e0.elapsed_time(e1))
    return best * 1e3 / steps


# 1000 x 1000: the pipelined step takes 17 us; whole-width walks of 48 rows per tile, and persistent
# ones of more blocks than fit, take longer
@pytest.mark.parametrize("tile", [dict(bx=256, cy=48, order=3, fuse=2, blocks_per_cu=1),
                                  dict(bx=256, cy=16, order=6, fuse=2, blocks_per_cu=32)])
def test_explicit_blocks_per_cu(torch, tile):
    from paper_0807_0602_amd import scf
    print(f"case: {tile} read and set back", flush=True)
    case = inputs.Case(inputs.Geometry(1000, 1000, 250, 750), inputs.Params(gw=(-0.2, 0.2)), seed=2, liquid_x1=250)
    ch = scf.Channel.from_case(case)
    default = _us(torch, ch)
    ch.set_tile(graph_steps=24, **tile)
    given = _us(torch, ch)
    read = ch.tile()
    assert read == dict(graph_steps=24, **tile)
    ch.set_tile(**read)
    back = _us(torch, ch)
    print(f"  us per step: default {default:.2f}, as given {given:.2f}, set back {back:.2f}", flush=True)
    assert given > 1.2 * default          # the walk
    assert back > 0.9 * given
