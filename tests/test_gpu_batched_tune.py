"""The autotuner times whole steps.  Contacts that overflow their slots stop sweeps that cannot search, so
on such boxes the candidates have to be captured with the search (k_sweep's second template flag): of
the sweeps traced in the first call, all but the ones that found the overflow out can search."""
import numpy as np
import pytest
import torch
from torch.profiler import ProfilerActivity, profile

import oracle
import workloads
import paper_2501_05340_amd as pc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("slots", [1, 12])
def test_candidates_run_their_sweeps(slots, tmp_path, monkeypatch):
    monkeypatch.setenv("PCOL_TUNE_CACHE", str(tmp_path / "tune.txt"))
    boxes = [workloads.make_box(n, seed=n, phi=0.3, radius=1.0, e=0.9) for n in (900, 2500, 1300)]
    off = np.cumsum([0] + [b.n for b in boxes])
    cat = [np.concatenate([getattr(b, f) for b in boxes]) for f in ("x", "y", "z", "vx", "vy", "vz", "r", "m")]
    p = pc.Particles(*[torch.as_tensor(c).cuda() for c in cat])
    partner = torch.empty(p.n, dtype=torch.int32, device="cuda")
    ctx = pc.Context(p.n, pc.pcol_default_opts(contact_slots=slots))
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        st = pc.pcol_step_batched(ctx, p, off, [b.L for b in boxes], 0.4, 0.9, partner)
        torch.cuda.synchronize()
    assert st["tuned"] == 1
    ran = {flag: sum(e.count for e in prof.key_averages() if f"k_sweep<false, {flag}>" in e.key)
           for flag in ("false", "true")}
    assert sum(ran.values()) > 0, "no sweeps in the trace"
    per = 11  # later sweeps in a captured step (12 less the first)
    if st["n_overflow"]:
        assert ran["false"] <= 3 * per and ran["true"] >= 9 * per, ran
    else:
        assert ran["true"] == 0, ran
    ref = [oracle.step(b) for b in boxes]
    want = np.concatenate([np.where(r.partner >= 0, r.partner + o, -1) for r, o in zip(ref, off)])
    assert np.array_equal(partner.cpu().numpy(), want)
    assert st["n_sweeps"] == max(r.n_sweeps for r in ref)
    assert (st["n_overflow"] > 0) == (slots == 1)
