"""Narrow tiles of boxes that leave most of the pipelined step's 256 lanes idle run the two-step walk, bit
for bit as the two-kernel step and faster than the default schedule; wider boxes keep the pipelined step
whatever the tile."""
import numpy as np
import pytest

from paper_0807_0602_amd import inputs

pytestmark = pytest.mark.gpu

TWO_KERNEL = 1


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


def _make(nx, ny, n):
    from paper_0807_0602_amd import scf
    case = inputs.Case(inputs.Geometry(nx, ny, nx // 4, nx - nx // 4), inputs.Params(gw=(-0.25, 0.2), tau=(1.25, 0.8)),
                       seed=2, liquid_x1=nx // 4)
    if n == 1:
        return scf.Channel.from_case(case)
    return scf.Batch([case] * n, sample_every=1 << 20, max_samples=2, fields=[case.fields()] * n)


# `share`: the most of the default schedule's time that the tile may take (measured 0.45, 0.73, 0.53, 0.56)
@pytest.mark.parametrize("nx,ny,n,bx,order,share", [
    (16, 60000, 1, 64, 6, 0.7), (40, 30000, 1, 128, 6, 0.9), (48, 48, 400, 64, 1, 0.75), (64, 20, 1000, 64, 6, 0.75)])
def test_narrow_tile_runs_the_walk(torch, nx, ny, n, bx, order, share):
    print(f"case: {n} of {nx}x{ny} with bx={bx}", flush=True)
    ch, ref = _make(nx, ny, n), _make(nx, ny, n)
    if n == 1:
        ref.set_variant(TWO_KERNEL)
    else:
        ref.set_tile(256, 8, 0, 1, 1)
    default = _us(torch, ch)
    ch.set_tile(bx, 16, 24, order, 2)
    tile = _us(torch, ch)
    print(f"  us per step: default {default:.2f}, bx={bx} {tile:.2f}", flush=True)
    assert tile < share * default
    ch, d = _make(nx, ny, n), () if n == 1 else (n - 1,)
    ch.set_tile(bx, 16, 4, order, 2)
    for a, b in zip(ch.step(11).density(*d), ref.step(11).density(*d)):
        assert np.array_equal(a, b)


def test_wider_boxes_keep_the_pipelined_step(torch):
    print("case: 1000x1000 with bx=64", flush=True)
    ch = _make(1000, 1000, 1)
    default = _us(torch, ch)
    ch.set_tile(64, 16, 24, 6, 2)
    assert _us(torch, ch) < 1.15 * default      # the walk takes 1.7 times as long
