"""The page-locked buffers of small read-outs belong to the process: destroying a context waits for its
own stream only, more calls at once than there are buffers fall back to copies, and contexts created
after the last one was destroyed read out as before."""
import threading

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


def _make(kind, stream):
    from paper_0807_0602_amd import scf, surrogate
    case = inputs.capillary_small(seed=1)
    if kind == "channel":
        return scf.Channel.from_case(case, stream=stream)
    if kind == "batch":
        return scf.Batch([case], sample_every=5, max_samples=4, stream=stream)
    if kind == "duct":
        f = [np.full((6, 6, 12), v) for v in (2.0, 0.06)]
        return scf.Channel3(12, 6, 6, 3, 9, inputs.Params(), *f, stream=stream)
    return surrogate.Network(3, 64, 2, max_batch=64, max_data=64, stream=stream)


@pytest.mark.parametrize("kind", ["channel", "batch", "duct", "network"])
def test_destroying_a_context_waits_for_its_own_stream_only(torch, kind):
    print(f"case: {kind} destroyed while another stream works", flush=True)
    own, other = torch.cuda.Stream(), torch.cuda.Stream()
    ctx = _make(kind, own)
    if kind == "network":
        ctx.predict(np.zeros((4, 3), np.float32))
    else:
        ctx.step(5)
        ctx.observe()
    a = torch.ones((8192, 8192), device="cuda:0")
    (a @ a).sum().item()
    end = torch.cuda.Event()
    with torch.cuda.stream(other):
        for _ in range(30):       # some 200 ms of work
            a @ a
        end.record()
    ctx.close()
    assert not end.query()
    other.synchronize()


def test_more_calls_at_once_than_buffers(torch):
    """Twelve contexts read out in threads of their own, then their last one goes and others come."""
    print("case: twelve contexts in twelve threads, twice", flush=True)
    from paper_0807_0602_amd import scf
    for turn in range(2):
        cases = [inputs.Case(inputs.Geometry(150 + 5 * k, 60 + k, 30, 90), inputs.Params(gw=(-0.2, 0.2)), seed=k + turn,
                             liquid_x1=40) for k in range(12)]
        chans = [scf.Channel.from_case(c, stream=torch.cuda.Stream()) for c in cases]
        want = [ch.step(4).density() for ch in chans]
        mass = [ch.observe()["mass"] for ch in chans]
        wrong = []

        def read(k):
            for _ in range(20):
                if not all(np.array_equal(x, y) for x, y in zip(chans[k].density(), want[k])) \
                        or chans[k].observe()["mass"] != mass[k]:
                    wrong.append(k)

        threads = [threading.Thread(target=read, args=(k,)) for k in range(12)]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        assert not wrong
        for ch in chans:
            ch.close()
