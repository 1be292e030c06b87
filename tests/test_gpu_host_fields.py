"""Host fields at the boundary: large boxes are checked on the device after the
copy, tubes pass through pinned slots that the kernels read and write."""
import numpy as np
import pytest

from gpu_util import note
from paper_1301_3423_amd import inputs, rlb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pattern", ["ab", "aa"])
@pytest.mark.parametrize("shape", [(41, 40, 40), (64, 33, 32)])      # 65,600 and 67,584 cells: on the device
@pytest.mark.parametrize("field,value,words", [(0, 0.0, "cell"), (0, np.inf, "non-finite"), (1, -1.0, "cell"),
                                               (2, np.nan, "non-finite"), (4, 1.0, "cell")])
def test_bad_cell_of_a_large_box_is_refused(shape, pattern, field, value, words):
    fields = inputs.random_box(*shape, 0.3, seed=3)
    s = rlb.Solver(*shape, precision="mixed", tau=0.9, pattern=pattern)
    s.init_fields(*fields)
    s.step(1)
    before = s.read_fields()
    for at in (0, fields[0].size - 1):
        bad = [f.copy() for f in fields]
        if field == 4:
            bad[2].ravel()[at] = bad[3].ravel()[at] = 0.0
        bad[field].ravel()[at] = value
        note("bad value %r in field %d, cell %d of %s" % (value, field, at, shape))
        with pytest.raises(rlb.RLBError) as e:
            s.init_fields(*bad)
        assert e.value.code == rlb.ENONPHYS and words in str(e.value)
    after = s.read_fields()
    assert s.status() == (0, 1)
    for k in before:
        assert np.array_equal(before[k], after[k])


def test_tubes_of_many_lengths_share_the_slots():
    """More tubes than slots, and one longer than a slot holds (16,384 cells):
    reading at once returns each tube's own fields, after a bad one too."""
    lens = [5, 700, 16384, 20000, 1, 64, 300, 2, 9, 16383, 31, 450]
    b = rlb.Batch([dict(n=n, tau=0.9) for n in lens], precision="fp64")
    fields = []
    for j, n in enumerate(lens):
        r = np.random.default_rng(j)
        T = 1.0 + 0.3 * r.random(n)
        fields.append([T ** 3, 3 * T ** 4, 0.2 * r.random(n), 0.1 * r.random(n), -0.3 * r.random(n)])
        if j % 3 == 1:
            bad = [a.copy() for a in fields[j]]
            bad[3][-1] = np.nan
            with pytest.raises(rlb.RLBError) as e:
                b.init_tube(j, *bad)
            assert e.value.code == rlb.ENONPHYS and "non-finite" in str(e.value)
        b.init_tube(j, *fields[j])
    for j in list(range(len(lens))) + [3, 0, 2]:
        got = b.read_tube(j)
        g = 1.0 / np.sqrt(1.0 - sum(v * v for v in fields[j][2:]))
        assert np.max(np.abs(got["n"] / fields[j][0] - 1.0)) < 1e-12
        assert np.max(np.abs(got["eps"] / fields[j][1] - 1.0)) < 1e-12
        assert np.max(np.abs(got["U"][0] - g)) < 1e-12 * np.max(g)
        for k in range(3):
            assert np.max(np.abs(got["U"][1 + k] - g * fields[j][2 + k])) < 1e-12 * np.max(g)
