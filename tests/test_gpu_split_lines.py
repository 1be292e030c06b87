"""The sizes on either side of every line between the split and the two-lane
float64 kernel: both patterns give the bits of the served box, which always takes
the two-lane kernel."""
import numpy as np
import pytest

from gpu_util import note
from paper_1301_3423_amd import inputs, rlb

pytestmark = pytest.mark.gpu

SHAPES = {3: [(32, 16, 12), (5, 1229, 1), (32, 32, 9), (13, 709, 1), (64, 16, 16), (5, 29, 113), (32, 32, 32),
              (33, 993, 1)],          # 6144, 6145, 9216, 9217, 16384, 16385, 32768 and 32769 cells
          2: [(32, 16, 16), (3, 2731, 1)]}                                                # 8192 and 8193


@pytest.mark.parametrize("order,shape", [(o, s) for o in SHAPES for s in SHAPES[o]])
def test_bits_on_either_side_of_a_line(order, shape):
    note("line %s order %d" % (shape, order))
    f = inputs.random_box(*shape, 0.4, seed=2)
    sv = rlb.Server(1 << 30, chunk_steps=2, max_tubes=2)
    sv.submit("box", shape, "fp64", 5, f, eta_s=0.3, order=order)
    served = sv.drain(timeout_s=60)[0]
    sv.close()
    assert served["rc"] == 0 and served["flags"] == 0
    for pattern in ("ab", "aa"):
        s = rlb.Solver(*shape, eta_s=0.3, order=order, pattern=pattern)
        s.init_fields(*f)
        s.step(5)
        assert s.status() == (0, 5)
        for k, v in s.read_fields().items():
            assert np.array_equal(v, served["fields"][k]), (pattern, k)
