"""The times of a step (opts.timing) that was queued ahead of a plan it did not fit and started over: the
binning, the pair tests and the sweeps are those of the run that counted."""
import numpy as np
import pytest

import workloads
import paper_2501_05340_amd as pc
from tests.gpu_helpers import gpu_step

pytestmark = pytest.mark.gpu


def test_times_of_a_step_that_started_over():
    """A plain grid, then one of fewer than three cells, where every sphere searches the whole box: some
    ms, against the microseconds of pair tests that left at once and of the sweeps."""
    plain = workloads.make_box(20_000, seed=3, phi=0.2, radius=1.0, e=0.9)
    fast = plain.copy()
    fast.vx[7] = 14.0 / fast.dt  # reach 2 r + 2 v dt = 30 of the side of 75
    opts = dict(timing=1, split_quantile=0.0)
    ctx = pc.Context(plain.n, pc.pcol_default_opts(**opts))
    for _ in range(2):
        assert min(gpu_step(plain, ctx=ctx)[3]["nc"]) >= 3
    got = gpu_step(fast, ctx=ctx)[3]
    want = min((gpu_step(fast, **opts)[3] for _ in range(3)), key=lambda st: st["ms_detect"])
    assert got["nc"] == want["nc"] and min(got["nc"]) < 3
    search = want["ms_detect"]
    assert search > 0.2  # the whole box for every sphere
    assert got["ms_detect"] > 0.5 * search
    assert got["ms_sweeps"] < want["ms_sweeps"] + 0.5 * search
    assert got["ms_bin"] > 0.0 and got["ms_advance"] > 0.0
