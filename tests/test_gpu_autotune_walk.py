"""The autotuner weighs the two-step walk against the node-parallel and the pipelined step: it finds the
narrow walk where that is faster, and what it reports and records runs the same step again."""
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


def _batch(n):
    from paper_0807_0602_amd import scf
    case = inputs.Case(inputs.Geometry(n, n, 0, 0), inputs.Params(), seed=4, liquid_x1=n // 3)
    return scf.Batch([case] * 900, sample_every=1 << 20, max_samples=2, fields=[case.fields()] * 900)


def test_finds_the_narrow_walk(torch, tmp_path):
    """900 boxes of 40 x 40: the pipelined step leaves five of six lanes idle."""
    print("case: autotuned batch of 900 boxes of 40 x 40", flush=True)
    path = str(tmp_path / "tune.txt")
    a, b, c = _batch(40), _batch(40), _batch(40)
    default = _us(torch, a)
    chosen = a.autotune(3, cache=path)
    tuned = _us(torch, a)
    print(f"  us per step: default {default:.2f}, {chosen} {tuned:.2f}", flush=True)
    assert chosen["fuse"] == 2 and chosen["bx"] <= 128
    assert tuned < 0.75 * default
    assert b.autotune(3, cache=path) == chosen
    assert _us(torch, b) < 1.2 * tuned
    c.set_tile(**chosen)
    assert c.tile() == chosen and _us(torch, c) < 1.2 * tuned
