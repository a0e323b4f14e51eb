"""Whole step-1 transforms of more short lines than one grid of any of their
passes takes."""
import pytest
import torch

from helpers import TOL, host, real_input, rel_l2
from paper_2202_12756_amd import Plan

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("x", [1, 2])
def test_planes_past_one_grid_of_y(x):
    """2^24 + 3 planes of N = 16 in place (19 GB): the y pass takes a tile of
    256 lanes per plane, so it needs more than one grid, as the z pass does.  The
    entries at both ends and around the launches' ends equal those of a small
    plan, bit for bit, and the field comes back."""
    n, planes = 16, (1 << 24) + 3 * x
    p = Plan(n, torch.float32, slab_x=x, batch=planes // x, inplace=True)
    q = Plan(n, torch.float32, slab_x=x, batch=2, inplace=True)
    buf, small = p.empty_inplace(), q.empty_inplace()
    buf.zero_()
    last = p.batch - 2
    at = [0, (1 << 23) // x - 1, (1 << 23) // x + 1, (1 << 24) // x - 1, last]
    want, ref = [], []
    for i, b in enumerate(at):
        xin, xref = real_input(q.real_shape, 35000 + 10 * x + i, torch.float32)
        p.real_view(buf)[b:b + 2].copy_(xin)
        q.real_view(small).copy_(xin)
        ref.append(xref)
        want.append(q.r2c_(small).clone())
    p.r2c_(buf)
    torch.cuda.synchronize()
    for b, f in zip(at, want):
        assert torch.equal(buf[b:b + 2], f), b
    out = p.c2r_(buf, scale=1.0 / n ** 2)
    torch.cuda.synchronize()
    for b, xref in zip(at, ref):
        assert rel_l2(host(out[b:b + 2]), xref) <= TOL[torch.float32], b
