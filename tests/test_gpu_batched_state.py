"""A batched step takes the place of the last binning: pcol_detect and pcol_resolve are refused after it
until pcol_bin runs again (also when the batch itself was refused by its data), and then find what
they found before."""
import numpy as np
import pytest
import torch

import workloads
import paper_2501_05340_amd as pc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bad", [False, True])
@pytest.mark.parametrize("first", ["bin", "step"])
def test_detect_and_resolve_need_a_binning_after_a_batch(first, bad):
    box = workloads.make_box(3000, seed=8, phi=0.25, radius=1.0, e=0.9)
    ctx = pc.Context(box.n, pc.pcol_default_opts(autotune=0))
    p = pc.Particles.from_box(box)
    active = torch.ones(box.n, dtype=torch.uint8, device="cuda")
    pc.pcol_bin(ctx, p, box.L, box.dt)
    key, tmin = pc.pcol_detect(ctx, p, box.L, box.dt)
    if first == "step":
        pc.pcol_step(ctx, p.clone(), box.L, box.dt, box.e)
    # the same spheres, box and dt as a batch of one box
    q = p.clone()
    if bad:
        q.vx[box.n // 2] = np.inf
        with pytest.raises(pc.PcolError) as ei:
            pc.pcol_step_batched(ctx, q, [0, box.n], [box.L], box.dt, box.e)
        assert ei.value.code == pc.PCOL_E_INVALID
    else:
        pc.pcol_step_batched(ctx, q, [0, box.n], [box.L], box.dt, box.e)
    for call in (lambda: pc.pcol_detect(ctx, p, box.L, box.dt),
                 lambda: pc.pcol_resolve(ctx, p, box.L, box.dt, box.e, key, active)):
        with pytest.raises(pc.PcolError) as ei:
            call()
        assert ei.value.code == pc.PCOL_E_STATE
    pc.pcol_bin(ctx, p, box.L, box.dt)
    key2, tmin2 = pc.pcol_detect(ctx, p, box.L, box.dt)
    assert torch.equal(key, key2) and torch.equal(tmin, tmin2)
