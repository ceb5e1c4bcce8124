"""pcol_detect with an active mask at the edges of its ways: sphere counts around the one below which it only
searches, active counts around the share that chooses the pair tests, active spheres spread over the
box, together in one corner (neighbours in the sorted order) and in runs of the caller's order, calls in
a row with masks on both sides of the share, and a step in between.  Keys and times equal the oracle's
earliest partners over the active set."""
import numpy as np
import pytest
import torch

import oracle
import workloads
import paper_2501_05340_amd as pc

pytestmark = pytest.mark.gpu


def _masks(box, m, seed):
    order = np.random.default_rng(seed).permutation(box.n)
    corner = np.argsort(np.maximum(np.maximum(box.x, box.y), box.z))
    for ids in (order[:m], corner[:m], (np.arange(m) + box.n // 3) % box.n):
        act = np.zeros(box.n, dtype=np.uint8)
        act[ids] = 1
        yield act


@pytest.mark.parametrize("n,slots", [(1, 12), (2, 12), (63, 12), (4095, 12), (4096, 12), (4097, 1), (20_011, 12),
                                     (40_003, 1)])
def test_masked_detect_at_the_edges(n, slots):
    box = workloads.make_box(n, seed=n, phi=0.25 if n > 63 else 0.05, radius=1.0, e=0.9,
                             **({"L": 17.0} if n <= 63 else {}))
    ctx = pc.Context(box.n, pc.pcol_default_opts(contact_slots=slots))
    p = pc.Particles.from_box(box)
    pc.pcol_bin(ctx, p, box.L, box.dt)
    k = 0
    for m in (0, 1, n // 24, n // 24 + 1, n // 300, n):
        for act in _masks(box, min(m, n), m):
            key, tmin = pc.pcol_detect(ctx, p, box.L, box.dt, active=torch.from_numpy(act).cuda())
            torch.cuda.synchronize()
            partner, t, _ = oracle.earliest(box, active=act)
            has = partner >= 0
            q = key.cpu().numpy().view(np.uint64)
            assert np.array_equal(q == np.uint64(2 ** 64 - 1), ~has), m
            assert np.array_equal((q[has] & np.uint64(0xFFFFFFFF)).astype(np.int64), partner[has]), m
            assert np.array_equal(tmin.cpu().numpy(), t), m
            k += 1
            if k % 5 == 0:  # its records serve the next detects
                pc.pcol_step(ctx, p.clone(), box.L, box.dt, box.e)
