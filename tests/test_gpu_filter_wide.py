"""The pair filters where their bounds are tightest: the binary32 filter over home cells of one sphere to
several batches of 64 and more survivors than its queue holds, and both filters in boxes of 1e4 to 1e6
radii, whose coordinates round by up to 1e-10 radii, with pairs that graze each other or touch at the
very end of the step, near the far corner and across the periodic one.  The step equals the oracle's
bitwise (every pair against every other) whatever a filter lets through."""
import numpy as np
import pytest

import oracle
import workloads
from tests.gpu_helpers import compare_step, gpu_step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("at", [11.0, 27.0])
@pytest.mark.parametrize("m", [1, 63, 64, 65, 129, 193, 400, 700])
def test_binary32_clump_matches_oracle(m, at):
    """m spheres within one cell's width of the point `at`, and a few alone."""
    rng = np.random.default_rng(m)
    L = 30.0
    x = np.concatenate([(at + rng.uniform(0.0, 6.0, (m, 3))) % L, rng.uniform(0.0, L, (20, 3))])
    v = rng.normal(size=x.shape) * 0.6
    r = rng.uniform(0.15, 0.45, len(x))
    box = workloads.Box(*x.T.copy(), *v.T.copy(), r, r ** 3, (L,) * 3, 1.0, 0.9)
    ref = oracle.step(box)
    for kw in ({"home_cells": 1}, {"home_cells": 4}, {"home_cells": 4, "contact_slots": 2}):
        compare_step(box, gpu_step(box, filter=1, **kw), ref)


def _grazing(L, at, seed):
    """Pairs on a lattice of spacing 9 around the point `at`: each meets with an impact parameter of the
    contact distance times 1 + d, or head-on at the time dt (1 + d), d from 0 to 1e-3 either way."""
    rng = np.random.default_rng(seed)
    site = at + 9.0 * (np.stack(np.meshgrid(*[np.arange(-3, 3)] * 3, indexing="ij")).reshape(3, -1).T)
    k = len(site)
    d = np.concatenate([[0.0], 10.0 ** np.arange(-15, -2), -(10.0 ** np.arange(-15, -2))])[np.arange(k) % 27]
    r = rng.uniform(0.5, 1.0, (k, 2))
    s, dt = r.sum(1), 1.0
    n = rng.normal(size=(k, 3))
    n /= np.linalg.norm(n, axis=1)[:, None]
    t = np.cross(n, rng.normal(size=(k, 3)))
    t /= np.linalg.norm(t, axis=1)[:, None]
    graze = rng.random(k) < 0.5
    speed = rng.uniform(0.5, 1.5, k)
    along = np.where(graze, 0.4 * speed * dt, s + speed * dt * (1.0 + d))  # closest approach at 0.4 dt
    across = np.where(graze, s * (1.0 + d), 0.0)
    b = site + along[:, None] * n + across[:, None] * t
    va = rng.normal(size=(k, 3)) * 0.2
    vb = va - speed[:, None] * n
    x, v = np.concatenate([site, b]) % L, np.concatenate([va, vb])
    x[x >= L] = 0.0
    rr = np.concatenate([r[:, 0], r[:, 1]])
    order = rng.permutation(2 * k)
    return workloads.Box(*x[order].T.copy(), *v[order].T.copy(), rr[order], rr[order] ** 3, (L,) * 3, dt, 0.9)


@pytest.mark.parametrize("flt", [0, 1])
@pytest.mark.parametrize("corner", ["far", "across"])
@pytest.mark.parametrize("L", [1e4, 1e5, 1e6])
def test_grazing_pairs_in_wide_boxes(L, corner, flt):
    box = _grazing(L, L - 40.0 if corner == "far" else 0.0, int(np.log10(L)))
    ref = oracle.step(box, grid=False)
    assert 50 < ref.n_pairs < 216  # some of each kind
    reach = 2.0 * box.r.max() + 2.0 * np.sqrt(box.vx ** 2 + box.vy ** 2 + box.vz ** 2).max() * box.dt
    for cells in (5, 40):
        g = gpu_step(box, filter=flt, cell_mult=L / (reach * cells))
        assert compare_step(box, g, ref) == 0 and g[3]["n_pairs"] == ref.n_pairs
