"""The deposition onto nearly 2^31 elements, where the scan's last tile reaches past the largest int less
a tile: spheres with no node in common, the last element among them, whose nodes wrap to the first ones.
Every node then holds one term, w a, exact by the rule; all other nodes are zero."""
import numpy as np
import pytest
import torch

import paper_2501_05340_amd as pc

pytestmark = pytest.mark.gpu

NC = (1310, 1261, 1300)  # 2^31 - 648 elements


def test_deposit_onto_almost_two_to_the_31_elements():
    assert 2 ** 31 - 4096 < NC[0] * NC[1] * NC[2] < 2 ** 31
    if torch.cuda.mem_get_info()[0] < 60 << 30:
        pytest.skip("needs 60 GB of device memory")
    cells = np.array([[5, 6, 7], [700, 600, 500], [1309, 1260, 1299], [3, 1260, 650], [1308, 2, 1297]])
    f = np.array([[0.5, 0.25, 0.125], [0.0, 0.75, 0.5], [0.5, 0.5, 0.75], [0.125, 0.625, 0.25], [0.25, 0.5, 0.5]])
    a = np.array([[3.0, -2.0, 7.0, 0.5, -11.0]])
    want = {}
    for c, g, s in zip(cells, f, a[0]):
        for b in range(8):
            bits = (b & 1, b >> 1 & 1, b >> 2)
            w = np.prod([g[d] if bits[d] else 1.0 - g[d] for d in range(3)])  # dyadic: exact
            i, j, k = ((c[d] + bits[d]) % NC[d] for d in range(3))
            node = (int(k) * NC[1] + int(j)) * NC[0] + int(i)
            assert node not in want
            if w:
                want[node] = w * s
    dev = lambda v: torch.as_tensor(np.ascontiguousarray(v)).cuda()
    ctx = pc.Context(1)
    try:
        out = torch.full((NC[2], NC[1], NC[0], 1), 9.0, dtype=torch.float64, device="cuda")
        pc.pcol_deposit(ctx, *[dev(v) for v in (cells + f).T], dev(a), NC, tuple(float(v) for v in NC), out)
        flat = out.view(-1)
        at = torch.tensor(sorted(want), device="cuda")
        assert flat[at].cpu().tolist() == [want[k] for k in sorted(want)]
        flat[at] = 0.0
        for part in flat.split(1 << 28):
            assert not bool(part.any())
    finally:
        ctx.close()
        out = flat = part = None
        torch.cuda.empty_cache()
