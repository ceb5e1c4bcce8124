"""What pcol_deposit waits for: the check of the positions, not the node sums, which may still run when it
returns; and its scratch, which a deposition on another stream must not touch before they are done."""
import numpy as np
import pytest
import torch

import oracle
import paper_2501_05340_amd as pc

pytestmark = pytest.mark.gpu

U = 2.0 ** -53


def _case(n, seed, comp=3):
    rng = np.random.default_rng(seed)
    x, a = rng.uniform(0.0, 0.999, (3, n)), rng.normal(size=(comp, n))
    return x, a, [torch.as_tensor(v).cuda() for v in x], torch.as_tensor(a).cuda()


def _check(out, x, a, nc):
    ref, mag = oracle.deposit(*x, a, nc, (1.0,) * 3), oracle.deposit(*x, np.abs(a), nc, (1.0,) * 3)
    got = out.cpu().numpy().transpose(3, 0, 1, 2)
    assert np.all(np.abs(got - ref) <= 2.0 * (8 * len(x[0]) - 1) * U * mag)


def test_returns_before_the_node_sums():
    """20,000 spheres in one element are one thread's serial sum, some ms."""
    x, a, xd, ad = _case(20_000, 1)
    ctx = pc.Context(1)
    out = pc.pcol_deposit(ctx, *xd, ad, (1, 1, 1), (1.0,) * 3)  # scratch made
    for _ in range(2):
        torch.cuda.synchronize()
        pc.pcol_deposit(ctx, *xd, ad, (1, 1, 1), (1.0,) * 3, out)
        assert not torch.cuda.current_stream().query()
        _check(out, x, a, (1, 1, 1))


def test_next_call_on_another_stream():
    """Depositions alternating between two streams on one context, a bad position among them."""
    big, small = _case(20_000, 2), _case(300, 3)
    ctx = pc.Context(1)
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    outs = []
    for k in range(6):
        x, a, xd, ad = big if k % 2 == 0 else small
        nc = (1, 1, 1) if k % 2 == 0 else (3, 2, 5)
        with torch.cuda.stream(streams[k % 2]):
            outs.append((pc.pcol_deposit(ctx, *xd, ad, nc, (1.0,) * 3), x, a, nc))
            if k == 3:
                with pytest.raises(pc.PcolError) as ei:
                    pc.pcol_deposit(ctx, xd[0] + 1.0, xd[1], xd[2], ad, nc, (1.0,) * 3)
                assert ei.value.code == pc.PCOL_E_INVALID
    torch.cuda.synchronize()
    for o in outs:
        _check(*o)
