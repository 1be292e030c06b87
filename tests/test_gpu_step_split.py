"""float64 boxes small enough for the kernel that splits a cell over four
wavefronts (k_step_split): axes below the displacements, ragged last blocks,
the last size of its range and the first beyond it, against the oracle; both
streaming patterns give the same bits on either side of the line."""
import numpy as np
import pytest

from gpu_util import field_errors, note
from oracle import rlb as orlb
from paper_1301_3423_amd import inputs, rlb

pytestmark = pytest.mark.gpu

# third order: up to 36,864 cells; second order: up to 16,384
SHAPES = [(1, 1, 1), (1, 1, 63), (65, 1, 1), (6, 5, 4), (7, 13, 11), (64, 8, 6), (32, 32, 16), (25, 26, 26), (36, 32, 32),
          (37, 32, 32)]


@pytest.mark.parametrize("order", [3, 2])
@pytest.mark.parametrize("shape", SHAPES)
def test_matches_oracle_in_both_patterns(lat, lat2, shape, order):
    note("split step %s order %d" % (shape, order))
    fields = inputs.random_box(*shape, 0.4, seed=sum(shape))
    o = orlb.Solver(*shape, lat=lat if order == 3 else lat2, order=order, eta_s=0.3)
    o.init_fields(*fields)
    o.step(3)
    ref, got = o.read_fields(), []
    for pattern in ("ab", "aa"):
        s = rlb.Solver(*shape, precision="fp64", eta_s=0.3, order=order, pattern=pattern)
        s.init_fields(*fields)
        s.step(3)
        got.append(s.read_fields())
        assert s.status() == (0, 3)
        err = field_errors(got[-1], ref)
        assert max(err.values()) <= 1e-12, (pattern, err)
    for k in got[0]:
        assert np.array_equal(got[0][k], got[1][k]), k


def test_walls(lat):
    shape = (19, 20, 21)
    fields = inputs.random_box(*shape, 0.4, seed=9)
    solid = np.zeros(shape[::-1], bool)
    solid[:, :6] = True
    solid[3, 12, 5] = True
    s = rlb.Solver(*shape, precision="fp64", eta_s=0.3)
    s.set_walls(solid)
    s.init_fields(*fields)
    s.step(4)
    o = orlb.Solver(*shape, lat=lat, eta_s=0.3, solid=solid)
    o.init_fields(*fields)
    o.step(4)
    err = field_errors(s.read_fields(), o.read_fields())
    assert s.status() == (0, 4)
    assert max(err.values()) <= 1e-12, err
