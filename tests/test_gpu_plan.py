"""Steps queued ahead of their plan, and the one-pass scan.  A context meets, in one shape (sphere
count, box, step), states whose grids differ: another cell size, more cells than it has room for, a
split grid after a plain one, fewer than three cells, data it refuses.  Every step equals the one of a
fresh context bitwise (state, pairs, times and the counts of the statistics), and a refused call
changes nothing."""
import numpy as np
import pytest
import torch

import oracle
import workloads
import paper_2501_05340_amd as pc
from tests.gpu_helpers import FIELDS, gpu_step, to_host

pytestmark = pytest.mark.gpu

L = 80.0
COUNTS = ("n_pairs", "n_sweeps", "pair_tests", "contacts", "n_overflow", "nc", "home_cells", "max_cell",
          "reach", "n_wide", "rho_c")


def _state(n, r, fast, seed):
    """n spheres of radius about r; a few of them `fast` times as fast as the others."""
    rng = np.random.default_rng(seed)
    x, v = rng.uniform(0.0, L, (3, n)), rng.normal(size=(3, n))
    v[:, :5] *= fast
    rr = r * rng.uniform(0.9, 1.1, n)
    return workloads.Box(*x, *v, rr, rr ** 3, (L,) * 3, 0.4, 0.9)


@pytest.mark.parametrize("n,opts", [(5000, {}), (5000, {"filter": 1}), (5000, {"split_quantile": 0.0}),
                                    (300_000, {})])
def test_grids_that_change_under_one_shape(n, opts):
    states = [_state(n, 0.8, 1, 1), _state(n, 0.8, 1, 2), _state(n, 0.8, 1, 2), _state(n, 0.8, 1, 2),
              _state(n, 0.8, 6, 3), _state(n, 0.2, 1, 4), _state(n, 0.05, 1, 5), _state(n, 3.0, 8, 6),
              _state(n, 0.8, 1, 2), _state(n, 0.05, 8, 7)]
    ctx = pc.Context(n, pc.pcol_default_opts(**opts))
    for k, box in enumerate(states):
        g, want = gpu_step(box, ctx=ctx), gpu_step(box, **opts)
        for f in FIELDS:
            assert np.array_equal(g[0][f], want[0][f]), (k, f)
        assert np.array_equal(g[1], want[1]) and np.array_equal(g[2], want[2], equal_nan=True), k
        assert {c: g[3][c] for c in COUNTS} == {c: want[3][c] for c in COUNTS}, k
        if k in (1, 7):  # data it refuses, between steps of the shape
            for f, val, code in (("vx", np.inf, pc.PCOL_E_INVALID), ("y", L, pc.PCOL_E_INVALID),
                                 ("vz", 60.0, pc.PCOL_E_BOX)):
                p = pc.Particles.from_box(box)
                getattr(p, f)[n // 2] = val
                before = to_host(p)
                with pytest.raises(pc.PcolError) as ei:
                    pc.pcol_step(ctx, p, box.L, box.dt, box.e)
                assert ei.value.code == code
                torch.cuda.synchronize()
                after = to_host(p)
                assert all(np.array_equal(before[q], after[q]) for q in FIELDS)


@pytest.mark.parametrize("nc", [(1, 1, 1), (15, 13, 21), (16, 16, 16), (17, 241, 1), (64, 64, 65), (129, 127, 131)])
def test_scan_over_tiles(nc):
    """Element counts below, at and above a scan tile of 4096 and over hundreds of tiles: one sphere
    in each of up to 5000 elements, deposited bitwise as by the oracle (no node sums two spheres
    of more than rounding: 8 terms)."""
    rng = np.random.default_rng(nc[0])
    ne = nc[0] * nc[1] * nc[2]
    e = rng.permutation(ne)[:5000]
    c = np.stack([e % nc[0], e // nc[0] % nc[1], e // (nc[0] * nc[1])])
    box = tuple(float(v) for v in nc)
    x = c + rng.uniform(0.0, 0.999, c.shape)
    a = rng.normal(size=(2, len(e)))
    dev = lambda v: torch.as_tensor(np.ascontiguousarray(v)).cuda()
    ctx = pc.Context(1)
    out = pc.pcol_deposit(ctx, *dev(x), dev(a), nc, box)
    got = out.cpu().numpy().transpose(3, 0, 1, 2)
    ref, mag = oracle.deposit(*x, a, nc, box), oracle.deposit(*x, np.abs(a), nc, box)
    k = 8 if min(nc) > 1 else 64
    assert np.all(np.abs(got - ref) <= 2.0 * (k - 1) * 2.0 ** -53 * mag)
