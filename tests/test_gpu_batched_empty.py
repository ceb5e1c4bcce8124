"""A batch of no spheres: every count is its own (no pair, one sweep that resolves none), whatever the
context has stepped before it, and the next step is not touched by it."""
import numpy as np
import pytest
import torch

import oracle
import workloads
import paper_2501_05340_amd as pc
from tests.gpu_helpers import compare_step, gpu_step

pytestmark = pytest.mark.gpu

NONE = {"n_pairs": 0, "n_sweeps": 1, "contacts": 0, "n_overflow": 0, "finished_on_host": 0}


@pytest.mark.parametrize("slots", [12, 1])
def test_empty_batch_after_a_step(slots):
    box = workloads.make_box(3000, seed=5, phi=0.3, radius=1.0, e=0.9)
    ctx = pc.Context(box.n, pc.pcol_default_opts(contact_slots=slots, autotune=0))
    none = pc.Particles(*[torch.empty(0, dtype=torch.float64, device="cuda") for _ in range(8)])
    ref = oracle.step(box)
    for step in range(2):
        if step:
            compare_step(box, gpu_step(box, ctx=ctx), ref)
        st = pc.pcol_step_batched(ctx, none, [0, 0, 0], [30.0, (9.0, 12.0, 15.0)], box.dt, box.e)
        assert {k: st[k] for k in NONE} == NONE, step
    got = gpu_step(box, ctx=ctx)
    compare_step(box, got, ref)
    assert got[3]["n_pairs"] == ref.n_pairs and got[3]["n_sweeps"] == ref.n_sweeps
