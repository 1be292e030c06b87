"""Batches take the tile kernel whatever the number of tubes."""
import pytest

from gpu_util import note
from paper_1301_3423_amd import inputs, rlb

pytestmark = pytest.mark.gpu


def test_many_short_tubes_take_tiles(monkeypatch):
    """2000 tubes of 64 cells: one workgroup per tube takes eight turns at the 256
    CUs, the tiles one.  The batch must not take the former's time (it is asked for
    by setting a spin limit); three quarters of it leave room for noise, the tiles
    need little more than half."""
    import torch
    b = rlb.Batch([dict(n=64, eta_s=0.2)] * 2000, precision="mixed")
    f = inputs.shock_tube(64, 1.0, 0.8)
    for j in range(len(b)):
        b.init_tube(j, *f)
    took = {}
    for limit in (None, "4194304"):
        if limit:
            monkeypatch.setenv("RLB_TUBE_SPIN_LIMIT", limit)
        times = []
        for _ in range(4):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            b.step(100)
            e1.record()
            torch.cuda.synchronize()
            times.append(e0.elapsed_time(e1))
        took[limit] = min(times)
    note("2000 tubes of 64 cells, 100 steps: %.2f ms, one workgroup each %.2f ms" % tuple(took.values()))
    assert took[None] < 0.75 * took["4194304"]
