"""The pair filter's edges: home cells of one sphere to several batches of 64, candidate lists of one
to many chunks of 64 and more survivors than a queue holds, in the middle of a box and across its
periodic corner.  Every pair that passes is decided by the rule, so the step equals the oracle's
bitwise (pairs and contact times) whatever the filter lets through."""
import numpy as np
import pytest

import oracle
import workloads
from tests.gpu_helpers import compare_step, gpu_step

pytestmark = pytest.mark.gpu


def _clump(m, at, seed):
    """m spheres within one cell's width of the point `at` of a periodic box, and a few alone."""
    rng = np.random.default_rng(seed)
    L = 30.0
    x = np.concatenate([(at + rng.uniform(0.0, 6.0, (m, 3))) % L, rng.uniform(0.0, L, (20, 3))])
    n = len(x)
    v = rng.normal(size=(n, 3)) * 0.6
    r = rng.uniform(0.15, 0.45, n)
    return workloads.Box(*x.T.copy(), *v.T.copy(), r, r ** 3, (L,) * 3, 1.0, 0.9)


@pytest.mark.parametrize("at", [11.0, 27.0])
@pytest.mark.parametrize("m", [1, 2, 3, 63, 64, 65, 66, 128, 129, 193, 400])
def test_clump_matches_oracle(m, at):
    box = _clump(m, at, m)
    for kw in ({"home_cells": 1}, {"home_cells": 4}, {"home_cells": 4, "contact_slots": 2}):
        compare_step(box, gpu_step(box, **kw), oracle.step(box))
