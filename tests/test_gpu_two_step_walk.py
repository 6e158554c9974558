"""The two-step walk (k_step_fused2) bit for bit against the two-kernel step where it runs: under the
default schedule in boxes past the node-parallel step's size that are too low for the pipelined one, and
with an explicit number of blocks per CU at every block width, over several strips, with general rest
fractions and masses, walls to the edge and batches that mix masks."""
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


def _case(nx, ny, x0, x1, seed=3, mask=False, **params):
    solid = inputs.rough_mask(nx, ny, x0, x1, seed=seed, bumps=max(2, nx // 30)) if mask else None
    prm = dict(gw=(-0.25, 0.2), tau=(1.25, 0.8))
    return inputs.Case(inputs.Geometry(nx, ny, x0, x1, solid=solid), inputs.Params(**{**prm, **params}), seed=seed,
                       liquid_x1=max(x0, nx // 3))


def _equal(a, b):
    return all(np.array_equal(x, y) for x, y in zip(a, b))


@pytest.mark.parametrize("nx,ny,mask", [(120001, 9, False), (250000, 5, True), (300007, 3, False)])
def test_default_schedule_of_low_boxes(scf, nx, ny, mask):
    print(f"case: two-step walk by default, {nx}x{ny} mask={mask}", flush=True)
    case = _case(nx, ny, nx // 4, nx // 2, mask=mask)
    ch, ref = scf.Channel.from_case(case), scf.Channel.from_case(case)
    ref.set_variant(TWO_KERNEL)
    for steps in (1, 2, 67):
        assert _equal(ch.step(steps).density(), ref.step(steps).density()), steps


# strips of 58, 122, 224 and 480 columns: two to four of them, the last ragged; 512-lane blocks fill a CU
# alone, so that one of them per CU is their occupancy and a persistent list asks for more
@pytest.mark.parametrize("bx,cy,order,bpc", [(64, 5, 0, 1), (128, 16, 6, 1), (256, 7, 3, 1), (256, 16, 4, 2),
                                             (512, 16, 1, 1), (512, 16, 6, 4)])
@pytest.mark.parametrize("case", [
    _case(1201, 37, 300, 900), _case(1201, 37, 300, 900, mask=True), _case(500, 12, 250, 500, tau=(2.0, 0.8)),
    _case(481, 33, 0, 0), _case(230, 24, 60, 170, alpha=(4 / 9, 0.6), mass=(1.0, 1.5), tau=(1.2, 0.9))],
    ids=["strips", "rough", "wall_to_edge", "open", "alpha_mass"])
def test_explicit_blocks(scf, case, bx, cy, order, bpc):
    print(f"case: two-step walk bx={bx} cy={cy} order={order} blocks={bpc} {case.geom.nx}x{case.geom.ny}", flush=True)
    ch, ref = scf.Channel.from_case(case), scf.Channel.from_case(case)
    ref.set_variant(TWO_KERNEL)
    ch.set_tile(bx, cy, graph_steps=6, order=order, fuse=2, blocks_per_cu=bpc)
    for steps in (2, 13):
        assert _equal(ch.step(steps).density(), ref.step(steps).density()), steps
    assert np.array_equal(ch.populations(), ref.populations())


@pytest.mark.parametrize("bx,order,bpc", [(64, 1, 1), (256, 6, 1), (512, 3, 1)])
def test_batch_of_masked_and_row_walled(scf, bx, order, bpc):
    print(f"case: two-step walk of a mixed batch, bx={bx} order={order}", flush=True)
    cases = [_case(1201, 37, 300, 900, mask=True), _case(3, 9, 1, 2), _case(700, 42, 100, 600, seed=5), _case(96, 130, 0, 96)]
    b = scf.Batch(cases, sample_every=7, max_samples=8)
    b.set_tile(bx, 9, graph_steps=14, order=order, fuse=2, blocks_per_cu=bpc)
    b.step(23)
    recs, n = b.observe()
    assert n == 4
    for i, c in enumerate(cases):
        ref = scf.Channel.from_case(c)
        ref.set_variant(TWO_KERNEL)
        for s in range(n):
            o = ref.observe()
            assert recs[i][s]["mass"] == o["mass"] and recs[i][s]["flags"] == o["flags"], (i, s)
            ref.step(7 if s < n - 1 else 2)
        assert _equal(b.density(i), ref.density()), i
