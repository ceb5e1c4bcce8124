"""The queued sweeps at the edges of their lists: sphere counts around a workgroup and around the
shards of the list, slots that overflow (the sweeps are queued again with the exact search) and a
context that meets a step with overflow after one without.  All equal the oracle's step bitwise."""
import numpy as np
import pytest
import torch

import oracle
import workloads
import paper_2501_05340_amd as pc
from tests.gpu_helpers import compare_step, gpu_step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [255, 256, 257, 2047, 2049, 4097, 17_000])
@pytest.mark.parametrize("slots", [12, 1])
def test_list_sizes_match_oracle(n, slots):
    a = workloads.make_box(n, seed=n, phi=0.3, radius=1.0, e=0.9)
    ctx = pc.Context(n, pc.pcol_default_opts(contact_slots=slots))
    ref = oracle.step(a)
    for _ in range(2):
        g = gpu_step(a, ctx=ctx)
        compare_step(a, g, ref)
        assert g[3]["n_sweeps"] == ref.n_sweeps and g[3]["n_pairs"] == ref.n_pairs


def test_batched_overflow_then_none():
    """Slots of one contact overflow on dense boxes; the same context then steps boxes without."""
    ctx = pc.Context(4700, pc.pcol_default_opts(contact_slots=1, autotune=0))
    for phi in (0.3, 0.02, 0.3):
        boxes = [workloads.make_box(n, seed=n, phi=phi, radius=1.0, e=0.9) for n in (900, 2500, 1300)]
        off = np.cumsum([0] + [b.n for b in boxes])
        cat = [np.concatenate([getattr(b, f) for b in boxes])
               for f in ("x", "y", "z", "vx", "vy", "vz", "r", "m")]
        p = pc.Particles(*[torch.as_tensor(c).cuda() for c in cat])
        partner = torch.empty(p.n, dtype=torch.int32, device="cuda")
        tcoll = torch.empty(p.n, dtype=torch.float64, device="cuda")
        st = pc.pcol_step_batched(ctx, p, off, [b.L for b in boxes], 0.4, 0.9, partner, tcoll)
        torch.cuda.synchronize()
        ref = [oracle.step(b) for b in boxes]
        want = np.concatenate([np.where(r.partner >= 0, r.partner + o, -1)
                               for r, o in zip(ref, off)])
        assert np.array_equal(partner.cpu().numpy(), want)
        assert np.array_equal(tcoll.cpu().numpy(), np.concatenate([r.tcoll for r in ref]), equal_nan=True)
        assert np.array_equal(p.x.cpu().numpy(), np.concatenate([r.x for r in ref]))
        assert st["n_sweeps"] == max(r.n_sweeps for r in ref)
        assert st["n_overflow"] > 0 or phi < 0.1
