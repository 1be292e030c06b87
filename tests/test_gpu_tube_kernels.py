"""The two tube kernels over what each is used for: one workgroup per tube in the
server (float64 and second-order tubes up to the longest it takes, more steps in one
launch than its step counters hold) and, with its waits bounded through the
environment, mixed batches of many chunks; tiles at the edges of every number of
steps per launch.  One is compared with the other bit for bit, and with the oracle."""
import numpy as np
import pytest

from gpu_util import field_errors, note
from oracle import rlb as orlb
from paper_1301_3423_amd import inputs, rlb

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-12, "mixed": 1e-5}


def _batch(lens, precision, order):
    b = rlb.Batch([dict(n=n, eta_s=0.3) for n in lens], precision=precision, order=order)
    fields = [inputs.shock_tube(n, 1.0, 0.7 + 0.05 * (j % 5)) for j, n in enumerate(lens)]
    for j, f in enumerate(fields):
        b.init_tube(j, *f)
    return b, fields


@pytest.mark.parametrize("precision,order", [("fp64", 3), ("fp64", 2), ("mixed", 3), ("mixed", 2)])
def test_served_tubes_equal_the_batch(precision, order):
    lens, steps = [2047, 2017, 65, 200, 7], [45, 45, 600, 300, 1000]   # short ones: one launch
    b, fields = _batch(lens, precision, order)
    b.step(steps)
    sv = rlb.Server(512 << 20, chunk_steps=50, max_tubes=8)
    ids = [sv.submit("tube", (1, 1, n), precision, s, f, eta_s=0.3, order=order)
           for n, s, f in zip(lens, steps, fields)]
    done = {c["id"]: c for c in sv.drain(timeout_s=100)}
    sv.close()
    for j, i in enumerate(ids):
        note("served tube %s order %d: %d cells, %d steps" % (precision, order, lens[j], steps[j]))
        assert done[i]["rc"] == 0 and done[i]["flags"] == 0 and b.status(j) == (0, steps[j])
        for k, v in b.read_tube(j).items():
            assert np.array_equal(v, done[i]["fields"][k]), k


@pytest.mark.parametrize("precision,order", [("fp64", 3), ("fp64", 2), ("mixed", 2)])
def test_served_tube_of_many_steps_matches_oracle(lat, lat2, precision, order):
    n, steps = 65, 300
    f = inputs.shock_tube(n, 1.0, 0.8)
    sv = rlb.Server(256 << 20, chunk_steps=50, max_tubes=2)
    sv.submit("tube", (1, 1, n), precision, steps, f, eta_s=0.3, order=order)
    done = sv.drain(timeout_s=60)[0]
    sv.close()
    o = orlb.Solver(1, 1, n, lat=lat if order == 3 else lat2, order=order, eta_s=0.3)
    o.init_fields(*f)
    o.step(steps)
    err = field_errors(done["fields"], o.read_fields())
    assert done["rc"] == 0 and done["flags"] == 0
    assert max(err.values()) <= TOL[precision], err


def test_many_chunks_by_one_workgroup_equal_tiles(monkeypatch):
    lens, steps = [4000, 1999, 65, 200], [60, 45, 300, 600]
    out = []
    for limit in (None, "4194304"):
        if limit:
            monkeypatch.setenv("RLB_TUBE_SPIN_LIMIT", limit)
        b, _ = _batch(lens, "mixed", 3)
        b.step(steps)
        assert [b.status(j) for j in range(len(lens))] == [(0, s) for s in steps]
        out.append([b.read_tube(j) for j in range(len(lens))])
    for x, y in zip(*out):
        for k in x:
            assert np.array_equal(x[k], y[k]), k


@pytest.mark.parametrize("k", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("precision,order", [("fp64", 3), ("fp64", 2), ("mixed", 3), ("mixed", 2)])
def test_tile_edges_of_every_launch_length(lat, lat2, precision, order, k):
    """A call of k steps on few tubes is one launch (float64 above three: of three
    and the rest); lengths around one, two and three tiles of it, and below."""
    most = 3 if precision == "fp64" else 5
    cells = (32 if precision == "fp64" else 64) - 12 * (min(k, most) - 1)
    lens = sorted({n for c in (cells, 2 * cells, 3 * cells) for n in (c - 1, c, c + 1)} | {2, 7, 13})
    b, fields = _batch(lens, precision, order)
    for _ in range(2):
        b.step(k)
    for j, n in enumerate(lens):
        o = orlb.Solver(1, 1, n, lat=lat if order == 3 else lat2, order=order, eta_s=0.3)
        o.init_fields(*fields[j])
        o.step(2 * k)
        err = field_errors(b.read_tube(j), o.read_fields())
        assert b.status(j) == (0, 2 * k)
        assert max(err.values()) <= TOL[precision], (n, err)


def test_a_tube_among_thousands_finds_its_tiles():
    """float64 tubes of 1 to 40 cells in one batch against each tube in a batch of
    its own."""
    rng = np.random.default_rng(7)
    lens = [int(n) for n in rng.integers(2, 41, 3000)]
    steps = [int(s) for s in rng.integers(0, 6, len(lens))]
    b, fields = _batch(lens, "fp64", 3)
    b.step(steps)
    for j in [0, 1, 2, len(lens) - 1] + [int(i) for i in rng.integers(0, len(lens), 40)]:
        one = rlb.Batch([dict(n=lens[j], eta_s=0.3)], precision="fp64")
        one.init_tube(0, *fields[j])
        one.step(steps[j])
        assert b.status(j) == (0, steps[j])
        for k, v in one.read_tube(0).items():
            assert np.array_equal(v, b.read_tube(j)[k]), (j, lens[j], steps[j], k)
