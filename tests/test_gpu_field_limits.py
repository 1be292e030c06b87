"""Cells within an ulp of |v| = 1: host fields of a large box, checked on the device,
are refused and accepted as those of a small one, checked on the host, whose sum
of squares is not fused."""
import numpy as np
import pytest

from gpu_util import note
from paper_1301_3423_amd import rlb

pytestmark = pytest.mark.gpu

# the sum of squares reaches 1 only unfused, or only fused
EDGE = [(-0.2225556625973378, 0.6859706126789553, 0.6927577466811313),
        (0.20528090832368218, -0.3804270010807354, 0.9017400099399616)]


def _outcome(s, cells, v, at):
    f = [np.full(cells, x) for x in (1.0, 3.0, 0.0, 0.0, 0.0)]
    for k in range(3):
        f[2 + k][at] = v[k]
    try:
        s.init_fields(*f)
    except rlb.RLBError as e:
        return e.code, str(e)
    return rlb.OK, s.status()[0]


@pytest.mark.parametrize("v", EDGE)
def test_large_and_small_boxes_accept_the_same_cells(v):
    accepted = v[0] * v[0] + v[1] * v[1] + v[2] * v[2] < 1.0
    small, large = (rlb.Solver(64, ny, 32, precision="fp64", tau=0.9) for ny in (1, 33))   # 2048 and 67,584 cells
    for at in (0, 1000):
        a, b = _outcome(small, 2048, v, at), _outcome(large, 67584, v, at)
        note("v = %r in cell %d: small box %r, large box %r" % (v, at, a, b))
        assert a == b and (a[0] == rlb.OK) == accepted
        assert accepted or "cell %d has" % at in a[1]
