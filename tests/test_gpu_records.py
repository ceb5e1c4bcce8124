"""Records stored a wave at a time: every record size (1 to 8 source components) at counts around a
wave and a workgroup, deposited within the oracle's summation bound; and steps of such counts (the
sorted and the output records) bitwise as the oracle's."""
import numpy as np
import pytest
import torch

import oracle
import workloads
import paper_2501_05340_amd as pc
from tests.gpu_helpers import compare_step, gpu_step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("comp", range(1, 9))
@pytest.mark.parametrize("n", [1, 63, 64, 65, 257, 5000])
def test_deposit_every_record_size(n, comp):
    nc, L = (5, 7, 6), (1.0, 2.0, 1.5)
    x, y, z, a = workloads.deposit_case(n, seed=n + comp, L=L, comp=comp)
    dev = lambda v: torch.as_tensor(np.ascontiguousarray(v)).cuda()
    out = pc.pcol_deposit(pc.Context(1), dev(x), dev(y), dev(z), dev(a), nc, L)
    got = out.cpu().numpy().transpose(3, 0, 1, 2)
    ref, mag = oracle.deposit(x, y, z, a, nc, L), oracle.deposit(x, y, z, np.abs(a), nc, L)
    assert np.all(np.abs(got - ref) <= 2.0 * max(n - 1, 0) * 2.0 ** -53 * mag * (1 + 1e-6))


@pytest.mark.parametrize("n", [64, 65, 255, 257, 4097, 5001])
def test_step_record_counts(n):
    box = workloads.make_box(max(n, 300), seed=n, phi=0.2, radius=1.0, e=0.9)
    box = workloads.Box(*[v[:n].copy() for v in box.arrays()], box.L, box.dt, box.e)
    compare_step(box, gpu_step(box), oracle.step(box))
