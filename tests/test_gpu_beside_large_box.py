"""Small float64 work beside a large box on another stream, and the same work on
its several routes: a workgroup of the split kernels finds a place wherever one of
the large box's ends, and their results are the unsplit kernels', bit for bit."""
import time

import numpy as np
import pytest

from gpu_util import note
from paper_1301_3423_amd import inputs, rlb

pytestmark = pytest.mark.gpu


def _box(stream):
    s = rlb.Solver(32, 32, 32, precision="fp64", eta_s=0.5, stream=stream)
    s.init_fields(*inputs.random_box(32, 32, 32, 0.3, seed=1))
    return s, 200


def _tubes(stream):
    lens = [int(n) for n in np.random.default_rng(1).integers(200, 4001, 24)]
    b = rlb.Batch([dict(n=n, eta_s=0.2) for n in lens], precision="fp64", stream=stream)
    for j, n in enumerate(lens):
        b.init_tube(j, *inputs.shock_tube(n, 1.0, 0.8))
    return b, 300


def _stream_beside(a, big):
    """A stream that does not share the hardware queue of stream a."""
    import torch
    for _ in range(8):
        b = torch.cuda.Stream()
        big.step(20)
        done = torch.cuda.Event()
        done.record(a)
        with torch.cuda.stream(b):
            torch.zeros(64, device="cuda").add_(1.0)
        b.synchronize()
        apart = not done.query()
        a.synchronize()
        if apart:
            return b
    pytest.skip("every stream shares the hardware queue of the large box")


@pytest.mark.parametrize("work", [_box, _tubes])
def test_small_work_does_not_wait_for_the_large_box(work):
    """Were every launch of the small work held back until a step of the large
    box drains, each of its steps would take some part of that step; a tenth of
    it is allowed, five times what they take."""
    import torch
    a = torch.cuda.Stream()
    big = rlb.Solver(256, 256, 256, precision="mixed", eta_s=0.5, stream=a)
    fields, _ = inputs.random_box_device(256, 256, 256, 0.4, 3)
    torch.cuda.synchronize()
    big.init_fields(*fields)
    b = _stream_beside(a, big)
    small, steps = work(b)
    for s, n, st in ((small, steps, b), (big, 20, a)):          # first use
        s.step(n)
        st.synchronize()
    t0 = time.perf_counter()
    big.step(20)
    a.synchronize()
    per = (time.perf_counter() - t0) / 20
    big.step(300)
    done = torch.cuda.Event()
    done.record(a)
    t0 = time.perf_counter()
    small.step(steps)
    b.synchronize()
    took = time.perf_counter() - t0
    beside = not done.query()
    a.synchronize()
    note("%d small steps beside a box of %.2f ms per step: %.1f ms" % (steps, per * 1e3, took * 1e3))
    assert beside and took < steps * per / 10


@pytest.mark.parametrize("order", [3, 2])
@pytest.mark.parametrize("n", [1, 6, 31, 32, 33, 300, 2100])
def test_a_tube_gives_one_result_on_every_route(n, order):
    """As a batch, a 1 x 1 x n box and a served request (by one workgroup, or from
    2048 cells on as a box)."""
    r = np.random.default_rng(n)
    T = 1.0 + 0.2 * r.random(n)
    f = [T ** 3, 3 * T ** 4, 0.1 * r.random(n), -0.2 * r.random(n), 0.3 * r.random(n)]
    b = rlb.Batch([dict(n=n, eta_s=0.3)], order=order)
    b.init_tube(0, *f)
    b.step(23)
    s = rlb.Solver(1, 1, n, eta_s=0.3, order=order)
    s.init_fields(*f)
    s.step(23)
    sv = rlb.Server(256 << 20, chunk_steps=10, max_tubes=2)
    sv.submit("tube", (1, 1, n), "fp64", 23, f, eta_s=0.3, order=order)
    served = sv.drain(timeout_s=60)[0]
    sv.close()
    box = s.read_fields()
    assert served["rc"] == 0 and served["flags"] == 0 and b.status(0) == (0, 23)
    for k, v in b.read_tube(0).items():
        assert np.array_equal(v, box[k]) and np.array_equal(v, served["fields"][k]), k


@pytest.mark.parametrize("order", [3, 2])
@pytest.mark.parametrize("shape", [(6, 5, 4), (20, 19, 21), (32, 32, 32), (33, 32, 32)])
def test_a_box_gives_one_result_served_or_not(shape, order):
    f = inputs.random_box(*shape, 0.4, seed=4)
    s = rlb.Solver(*shape, eta_s=0.3, order=order)
    s.init_fields(*f)
    s.step(7)
    sv = rlb.Server(1 << 30, chunk_steps=2, max_tubes=2)
    sv.submit("box", shape, "fp64", 7, f, eta_s=0.3, order=order)
    served = sv.drain(timeout_s=60)[0]
    sv.close()
    assert served["rc"] == 0 and served["flags"] == 0
    for k, v in s.read_fields().items():
        assert np.array_equal(v, served["fields"][k]), k
