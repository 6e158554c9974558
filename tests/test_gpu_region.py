"""The node-parallel step of small boxes (1-4 steps per launch, see k_step_region), bit for bit
against the two-kernel step: every number of steps per launch, remainders, tiles ragged at the box
edge, boxes smaller than a region, masks and batches; and boxes just past it.
The row-walking kernels, which small boxes reach only with an explicit number of blocks per CU,
keep their own cases here."""
import numpy as np
import pytest

from paper_0807_0602_amd import inputs

pytestmark = pytest.mark.gpu

TWO_KERNEL = 1


@pytest.fixture(scope="module")
def scf():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0807_0602_amd import scf as S
    return S


def _case(nx, ny, x0, x1, seed=3, mask=False):
    solid = inputs.rough_mask(nx, ny, x0, x1, seed=seed, bumps=max(2, nx // 30)) if mask else None
    return inputs.Case(inputs.Geometry(nx, ny, x0, x1, solid=solid), inputs.Params(gw=(-0.25, 0.2), tau=(1.25, 0.8)),
                       seed=seed, liquid_x1=max(x0, nx // 3))


def _reference(S, case, steps):
    ch = S.Channel.from_case(case)
    ch.set_variant(TWO_KERNEL)
    return ch.step(steps).populations()


# (box, mask, steps): small regions with four steps per launch (3 x 3 up to their 256 tiles), large
# regions with four, three and two steps, and boxes past the two-step limit of 4 x 256 tiles; steps
# leave every remainder
@pytest.mark.parametrize("nx,ny,x0,x1,mask", [
    (3, 3, 1, 2, False), (8, 9, 2, 6, False), (9, 10, 0, 9, False), (131, 17, 20, 111, True), (200, 24, 50, 150, False),
    (64, 288, 16, 48, True), (72, 289, 10, 60, False), (400, 97, 0, 400, True), (4096, 22, 1024, 3072, False),
    (2049, 130, 500, 1500, False), (4097, 203, 512, 3584, True), (8191, 131, 2000, 6000, False)])
@pytest.mark.parametrize("steps", [1, 6, 11])
def test_region_equals_two_kernel(scf, nx, ny, x0, x1, mask, steps):
    case = _case(nx, ny, x0, x1, mask=mask)
    print(f"case: region {nx}x{ny} mask={mask} steps={steps}", flush=True)
    ref = _reference(scf, case, steps)
    for gs in (0, 5):
        ch = scf.Channel.from_case(case)
        ch.set_tile(256, 16, graph_steps=gs, order=6, fuse=2)
        assert np.array_equal(ch.step(steps).populations(), ref), gs


def test_region_batch_equals_solo(scf):
    cases = [_case(96, 96, 0, 0), _case(131, 17, 20, 111, mask=True), _case(3, 3, 1, 2), _case(320, 42, 0, 320, seed=5)]
    print("case: region batch of four, 23 steps", flush=True)
    b = scf.Batch(cases, sample_every=7, max_samples=8)
    b.step(23)
    for i, c in enumerate(cases):
        a, d = scf.Channel.from_case(c).step(23).density(), b.density(i)
        ch = scf.Channel.from_case(c)
        ch.set_variant(TWO_KERNEL)
        e = ch.step(23).density()
        for k in range(2):
            assert np.array_equal(a[k], d[k]) and np.array_equal(e[k], d[k]), i


@pytest.mark.parametrize("bx,cy,order", [(64, 1, 0), (64, 3, 3), (128, 8, 1), (256, 5, 2), (256, 16, 6), (512, 1 << 30, 0)])
@pytest.mark.parametrize("nx,ny,x0,x1,mask", [(3, 3, 1, 2, False), (131, 17, 20, 111, True), (64, 10, 32, 64, False)])
def test_walk_with_explicit_blocks(scf, bx, cy, order, nx, ny, x0, x1, mask):
    """blocks_per_cu = 1 keeps the row-walking kernels in small boxes."""
    case = _case(nx, ny, x0, x1, mask=mask)
    print(f"case: walk {nx}x{ny} bx={bx} cy={cy} order={order}", flush=True)
    ref = _reference(scf, case, 11)
    ch = scf.Channel.from_case(case)
    ch.set_tile(bx, cy, graph_steps=4, order=order, fuse=2, blocks_per_cu=1)
    assert np.array_equal(ch.step(11).populations(), ref)
