"""Read-outs of one context from several threads, beyond the sizes that go through page-locked memory:
densities and populations are both prepared in the idle population buffer, large predictions in the
activations.  Every thread gets what a lone one gets."""
import threading

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


def _all_alike(calls, repeats):
    """Run the calls in threads of their own; each must give its first, lone result every time."""
    want = [c() for c in calls]
    wrong = []

    def turn(k):
        for _ in range(repeats):
            got = calls[k]()
            if not all(np.array_equal(x, y) for x, y in zip(got, want[k])):
                wrong.append(k)

    threads = [threading.Thread(target=turn, args=(k,)) for k in range(len(calls))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong


def test_channel(scf):
    print("case: 400 x 300 channel from four threads", flush=True)
    case = inputs.Case(inputs.Geometry(400, 300, 100, 300), inputs.Params(gw=(-0.2, 0.2)), seed=2, liquid_x1=120)
    ch = scf.Channel.from_case(case)
    ch.step(9)
    _all_alike([ch.density, ch.populations, ch.density, lambda: [ch.observe()["mass"]]], 12)


def test_channel_3d(scf):
    print("case: 65 x 40 x 44 duct from three threads", flush=True)
    left = np.arange(65) < 20
    f = [np.where(left, a, b) + np.zeros((44, 40, 65)) for a, b in ((2.0, 0.06), (0.06, 2.0))]
    ch = scf.Channel3(65, 40, 44, 16, 48, inputs.Params(gw=(-0.2, 0.2)), *f, walls_y=True, walls_z=True)
    ch.step(5)
    _all_alike([ch.density, ch.populations, lambda: [ch.observe()["mass"]]], 8)


@pytest.mark.parametrize("width", [128, 320])
def test_predictions(scf, width):
    print(f"case: 117000 rows of width {width} from three threads", flush=True)
    from paper_0807_0602_amd.surrogate import Network
    net = Network(5, width, 2, max_batch=8192, max_data=64)
    rows = [np.random.default_rng(k).uniform(-1, 1, (117000, 5)).astype(np.float32) for k in range(3)]
    _all_alike([lambda X=X: net.predict(X) for X in rows], 4)
    net.close()
