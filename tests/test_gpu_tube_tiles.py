"""Few tubes are stepped by launches of several steps over 64-lane tiles
(k_tubes_tile): edges of its tiles (64 - 12 (k - 1) cells for k steps per
launch), tubes shorter than a tile or than the displacements, step counts
that end inside a launch, and the search for a block's tube among many."""
import numpy as np
import pytest

from gpu_util import field_errors, note
from oracle import rlb as orlb
from paper_1301_3423_amd import inputs, rlb

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-12, "mixed": 1e-5}

# below the displacement range, tile sizes for k = 5, 4, 3, 2, 1 and their neighbours
LENGTHS = [1, 2, 6, 7, 15, 16, 17, 28, 29, 40, 41, 51, 52, 53, 63, 64, 65, 105, 129]
STEPS = [1, 2, 3, 4, 5, 6, 7, 9, 10, 11, 0, 13, 5, 4, 3, 2, 1, 8, 12]


def _fields(n, r):
    if n < 2:
        return [np.array([1.0]), np.array([3.0]), np.zeros(1), np.zeros(1), np.array([0.2])]
    return inputs.shock_tube(n, 1.0, 1.0 / r)


@pytest.mark.parametrize("order", [3, 2])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_tile_edges_match_oracle(lat, lat2, precision, order):
    tubes = [dict(n=n, eta_s=0.1) if n % 2 else dict(n=n, tau=0.9) for n in LENGTHS]
    fields = [_fields(n, 1.2 + 0.03 * j) for j, n in enumerate(LENGTHS)]
    b = rlb.Batch(tubes, precision=precision, order=order)
    for j, f in enumerate(fields):
        b.init_tube(j, *f)
    note("tiles %s order %d: lengths %s, steps %s" % (precision, order, LENGTHS, STEPS))
    b.step(STEPS)
    b.step(STEPS)
    for j, t in enumerate(tubes):
        o = orlb.Solver(1, 1, t["n"], lat=lat if order == 3 else lat2, order=order,
                        **{k: t[k] for k in ("tau", "eta_s") if k in t})
        o.init_fields(*fields[j])
        o.step(2 * STEPS[j])
        err = field_errors(b.read_tube(j), o.read_fields())
        assert b.status(j) == (0, 2 * STEPS[j])
        assert max(err.values()) <= TOL[precision], (t, err)


@pytest.mark.parametrize("ntubes", [65, 4100])
def test_many_short_tubes_find_their_tiles(monkeypatch, ntubes):
    """In mixed precision the tiles give the bits of the persistent kernel;
    64 tubes are searched in one round, 64^2 in two, more in three."""
    rng = np.random.default_rng(ntubes)
    lens = [int(n) for n in rng.integers(1, 9, ntubes)]
    lens[ntubes // 2] = 300
    steps = [int(s) for s in rng.integers(0, 8, ntubes)]
    out = []
    for limit in (None, "4194304"):       # with a spin limit set, the persistent kernel runs
        if limit:
            monkeypatch.setenv("RLB_TUBE_SPIN_LIMIT", limit)
        b = rlb.Batch([dict(n=n, tau=0.8 + 0.01 * (j % 7)) for j, n in enumerate(lens)], precision="mixed")
        for j, n in enumerate(lens):
            b.init_tube(j, *_fields(n, 1.1 + 0.1 * (j % 5)))
        b.step(steps)
        out.append([b.read_tube(j) for j in range(ntubes)])
        assert all(b.status(j) == (0, steps[j]) for j in range(0, ntubes, 37))
    for j in range(ntubes):
        for k in ("n", "eps", "U", "P"):
            assert np.array_equal(out[0][j][k], out[1][j][k]), (j, lens[j], steps[j], k)


def test_flags_come_from_stored_cells_only():
    """A shock the scheme does not survive flags its own tube and no other."""
    b = rlb.Batch([dict(n=400, eta_s=0.1), dict(n=400, eta_s=0.01), dict(n=64, eta_s=0.1)], precision="fp64")
    for j, r in enumerate((1.3, 2.0, 1.3)):
        b.init_tube(j, *inputs.shock_tube(b.tubes[j]["n"], 1.0, 1.0 / r))
    b.step(60)
    assert b.status(0)[0] == 0 and b.status(2)[0] == 0
    assert b.status(1)[0] & rlb.FLAG_NONPHYSICAL
