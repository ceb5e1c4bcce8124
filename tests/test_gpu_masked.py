"""pcol_detect with an active mask: either of its two ways (the pair tests of all spheres, the exact
search of the active ones), on both sides of the share of active spheres that chooses between them,
with slots that overflow, a split grid, and a box of fewer than three cells; keys and times equal the
oracle's earliest partners over the active set."""
import numpy as np
import pytest
import torch

import oracle
import workloads
import paper_2501_05340_amd as pc

pytestmark = pytest.mark.gpu

BOXES = {
    "plain": dict(n=4000, phi=0.25, radius=1.0),
    "split": dict(n=12_000, phi=0.3, lognormal=(1.0, 0.25, 0.5, 2.0)),
    "small": dict(n=130, phi=0.1, radius=1.0),
}


@pytest.mark.parametrize("which", list(BOXES))
@pytest.mark.parametrize("slots,flt", [(12, 0), (1, 0), (12, 1)])
def test_masked_detect_matches_oracle(which, slots, flt):
    box = workloads.make_box(seed=7, e=0.9, **BOXES[which])
    ctx = pc.Context(box.n, pc.pcol_default_opts(contact_slots=slots, filter=flt))
    p = pc.Particles.from_box(box)
    pc.pcol_bin(ctx, p, box.L, box.dt)
    order = np.random.default_rng(1).permutation(box.n)
    for m in (0, 1, box.n // 20, box.n // 16, box.n // 16 + 1, box.n // 2, box.n - 1, box.n):
        act = np.zeros(box.n, dtype=np.uint8)
        act[order[:m]] = 1
        key, tmin = pc.pcol_detect(ctx, p, box.L, box.dt, active=torch.from_numpy(act).cuda())
        torch.cuda.synchronize()
        partner, t, _ = oracle.earliest(box, active=act)
        has = partner >= 0
        k = key.cpu().numpy().view(np.uint64)
        assert np.array_equal(k == np.uint64(2 ** 64 - 1), ~has), m
        assert np.array_equal((k[has] & np.uint64(0xFFFFFFFF)).astype(np.int64), partner[has]), m
        assert np.array_equal(tmin.cpu().numpy(), t), m
