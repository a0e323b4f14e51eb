"""Many short lines: sets narrower than a tile, whose columns are numbered
through, and step-1 transforms of more lines than one grid of any of their passes
takes."""
import pytest
import torch

import oracle
from helpers import TOL, cplx_input, host, real_input, rel_l2
from paper_2202_12756_amd import PencilPlan, Plan

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


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("order", ["natural", "send", "paper"])
@pytest.mark.parametrize("n,x,batch", [(16, 1, 2), (16, 4, 33), (32, 2, 9), (64, 4, 3)])
def test_lines_of_narrow_sets(n, x, batch, order, dtype):
    """y and x lines of 9, 17 and 33 columns, the last tile ragged."""
    p = Plan(n, dtype, slab_x=x, batch=batch, fuse_pack=order in ("send", "paper"),
             paper_order=order == "paper")
    a, ref = cplx_input((batch, x, n, n // 2 + 1), 38000 + n, dtype)
    if order != "natural":
        a = p.pack(a)
    for sign in (-1, +1):
        want = oracle.c2c_axis(ref, -2, sign)
        if order != "natural":
            want = oracle.pack_slab(want, n // x, paper_order=order == "paper")
        assert rel_l2(host(p.y_c2c(a.clone(), sign)), want) <= TOL[dtype]
    g, gref = cplx_input(p.pencil_shape, 38500 + n, dtype)
    if order == "paper":  # [p][Y][X][K]: x = i X + x_l
        gref = gref.transpose(0, 1, 3, 2, 4)
    gref = gref.reshape(batch, n, x, n // 2 + 1)
    for sign in (-1, +1):
        got = host(p.x_c2c(g.clone(), sign))
        if order == "paper":
            got = got.transpose(0, 1, 3, 2, 4)
        want = oracle.c2c_axis(gref, 1, sign)
        assert rel_l2(got.reshape(want.shape), want) <= TOL[dtype]


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("n,pr,pc", [(16, 2, 2), (16, 4, 8), (32, 2, 4), (32, 8, 16)])
def test_short_pencil_lines(n, pr, pc, dtype):
    """y and x lines of short pencils, the last column's odd width included."""
    for col in (0, pc - 1):
        p = PencilPlan(n, dtype, (pr, pc), col, batch=5)
        a, ref = cplx_input(p.ypencil_shape, 39000 + n + col, dtype)
        ref = ref.transpose(0, 1, 3, 2, 4).reshape(5, n, p.x, p.w)  # y = c' Y + y_l
        for sign in (-1, +1):
            got = host(p.y_c2c(a.clone(), sign)).transpose(0, 1, 3, 2, 4).reshape(5, n, p.x, p.w)
            assert rel_l2(got, oracle.c2c_axis(ref, 1, sign)) <= TOL[dtype]
        g, gref = cplx_input(p.xpencil_shape, 39500 + n + col, dtype)

        def lines(v):  # x = r X + x_l
            if p.h > 1:
                return v.reshape(5, n, n // pr, p.w)
            return v.transpose(0, 1, 3, 2, 4, 5).reshape(5, n, p.g * p.y, p.w)

        for sign in (-1, +1):
            assert rel_l2(lines(host(p.x_c2c(g.clone(), sign))),
                          oracle.c2c_axis(lines(gref), 1, sign)) <= TOL[dtype]


@pytest.mark.parametrize("n,pr,pc", [(16, 1, 8), (32, 1, 16), (64, 1, 32), (128, 1, 64), (128, 4, 64)])
def test_rows_into_chunks_of_one_bin(n, pr, pc):
    """FP32 z rows written one bin to a chunk, 64 rows of a grid and more (a row or
    two to a thread) and fewer."""
    p = PencilPlan(n, torch.float32, (pr, pc), 0, batch=3)
    f, ref = real_input(p.real_shape, 39800 + n, torch.float32)
    want = oracle.r2c_last(ref)
    got = p.z_r2c(f)
    for c in range(pc):
        k0, k1 = p.kz_range(c)
        assert rel_l2(host(p.chunk(got, c)), want[..., k0:k1]) <= TOL[torch.float32]
