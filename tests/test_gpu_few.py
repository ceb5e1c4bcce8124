"""Steps of fewer than 4096 spheres, which one workgroup bins and sweeps from a context's second
call of a shape on.  Every form of step, at the edges of its sizes, against a fresh context's first
call (the path of many kernels) on the same states, bitwise: state, pairs, times, spins and the
counts of the statistics; and what that path cannot take (slots that overflow, more cells than LDS
holds, fewer than three of them, refused data, a sweep cap) between such steps."""
import numpy as np
import pytest
import torch

import workloads
import paper_2501_05340_amd as pc
from tests.gpu_helpers import FIELDS, to_host

pytestmark = pytest.mark.gpu

COUNTS = ("n_pairs", "n_sweeps", "pair_tests", "contacts", "n_overflow", "n_recheck", "nc", "home_cells",
          "max_cell", "reach", "band", "n_wide", "rho_c")


def _step(ctx, box, form, seed=0):
    p = pc.Particles.from_box(box)
    n = box.n
    partner = torch.full((n,), -7, dtype=torch.int32, device="cuda")
    tcoll = torch.full((n,), -7.0, dtype=torch.float64, device="cuda")
    w = torch.as_tensor(np.random.default_rng(seed).normal(size=(3, n))).cuda()
    args = (box.dt, box.e)
    if form == "walls":
        st = pc.pcol_step_walls(ctx, p, box.L, (1, 0, 1), *args, partner, tcoll)
    elif form == "spin":
        st = pc.pcol_step_spin(ctx, p, w, box.L, *args, 0.3, partner, tcoll)
    elif form == "spin walls":
        st = pc.pcol_step_spin_walls(ctx, p, w, box.L, (0, 1, 0), *args, 0.3, partner, tcoll)
    else:
        st = pc.pcol_step(ctx, p, box.L, *args, partner, tcoll)
    torch.cuda.synchronize()
    out = to_host(p)
    out.update(partner=partner.cpu().numpy(), tcoll=tcoll.cpu().numpy(), w=w.cpu().numpy())
    return out, {c: st[c] for c in COUNTS}


def _same(a, b, what):
    for k in a[0]:
        assert np.array_equal(a[0][k], b[0][k], equal_nan=True), (what, k)
    assert a[1] == b[1], what


@pytest.mark.parametrize("form,opts", [("plain", {}), ("plain", {"filter": 1}), ("plain", {"order": 1}),
                                       ("plain", {"contact_slots": 2}), ("plain", {"cell_mult": 1.4}),
                                       ("walls", {}), ("spin", {}), ("spin walls", {})])
@pytest.mark.parametrize("n", [300, 1023, 1024, 1025, 2500, 4095, 4096])
def test_repeated_steps_equal_first_ones(n, form, opts):
    boxes = [workloads.make_box(n, seed=n + k, phi=phi, e=0.9, L=(n * 4.19 / 0.25) ** (1 / 3),
                                **({"radius": 1.0} if k % 2 else {"lognormal": (0.8, 0.2, 0.5, 1.2)}))
             for k, phi in enumerate((0.25, 0.25, 0.25, 0.25))]
    for b in boxes:
        b.dt = 0.3
    ctx = pc.Context(n, pc.pcol_default_opts(**opts))
    for k, box in enumerate(boxes + boxes[:2]):
        want = _step(pc.Context(n, pc.pcol_default_opts(**opts)), box, form, k)
        _same(_step(ctx, box, form, k), want, (n, form, k))


def test_what_goes_to_the_other_kernels():
    """One shape: a usual state; a dilute one of more than 8192 cells; one of fewer than three cells
    on an axis; a clump whose contacts overflow; refused data after each; then a sweep cap."""
    n, L = 900, 40.0
    rng = np.random.default_rng(1)

    def state(r, v, span):
        x = rng.uniform(0.0, span, (3, n))
        return workloads.Box(*x, *(rng.normal(size=(3, n)) * v), np.full(n, r), np.ones(n), (L,) * 3, 0.4, 0.9)

    usual, dilute, coarse, clump = state(0.6, 1, L), state(0.05, 0.2, L), state(4.0, 2.5, L), state(0.3, 2, 12.0)
    ctx = pc.Context(n)
    for k, box in enumerate([usual, usual, dilute, dilute, usual, usual, coarse, usual, usual, clump, clump, usual]):
        _same(_step(ctx, box, "plain"), _step(pc.Context(n), box, "plain"), k)
        p = pc.Particles.from_box(box)
        p.z[n - 1] = -1.0
        before = to_host(p)
        with pytest.raises(pc.PcolError) as ei:
            pc.pcol_step(ctx, p, box.L, box.dt, box.e)
        assert ei.value.code == pc.PCOL_E_INVALID
        torch.cuda.synchronize()
        after = to_host(p)
        assert all(np.array_equal(before[f], after[f]) for f in FIELDS)
    dense = workloads.make_box(n, seed=5, phi=0.3, radius=1.0, e=0.9)
    need = _step(pc.Context(n), dense, "plain")[1]["n_sweeps"]
    assert need > 2
    for cap in (1, need - 1, need):
        ctx = pc.Context(n, pc.pcol_default_opts(max_sweeps=cap))
        for _ in range(3):
            p = pc.Particles.from_box(dense)
            if cap < need:
                with pytest.raises(pc.PcolError) as ei:
                    pc.pcol_step(ctx, p, dense.L, dense.dt, dense.e)
                assert ei.value.code == pc.PCOL_E_SWEEPS
                torch.cuda.synchronize()
                got = to_host(p)
                assert all(np.array_equal(got[f], getattr(dense, f)) for f in FIELDS)
            else:
                _same(_step(ctx, dense, "plain"), _step(pc.Context(n), dense, "plain"), cap)


def test_detect_after_a_step_of_few():
    """The sorted state that a step leaves in the context serves pcol_detect and pcol_resolve."""
    box = workloads.make_box(1500, seed=3, phi=0.2, radius=1.0, e=0.9)
    ctx = pc.Context(box.n)
    for _ in range(2):
        _step(ctx, box, "plain")
    p = pc.Particles.from_box(box)
    key, t = pc.pcol_detect(ctx, p, box.L, box.dt)
    other = pc.Context(box.n)
    pc.pcol_bin(other, p, box.L, box.dt)
    key2, t2 = pc.pcol_detect(other, p, box.L, box.dt)
    assert torch.equal(key, key2) and torch.equal(t, t2)
