"""GPU parity of the kernels that take several axes of the transform in one
memory pass, against the FP64 oracle at the sizes where their tiles change.
Tolerances: the rel-L2 bounds of the separate passes (FP64 1e-13, FP32 5e-6).
"""
import pytest
import torch

import oracle
from helpers import TOL, cplx_input, host, real_input, rel_l2
from paper_2202_12756_amd import Plan

pytestmark = pytest.mark.gpu

F64, F32 = torch.float64, torch.float32
DTYPES = pytest.mark.parametrize("dtype", [F64, F32], ids=["f64", "f32"])


@DTYPES
@pytest.mark.parametrize("order", ["natural", "send", "paper", "inplace"])
@pytest.mark.parametrize("n,x,batch", [(64, 1, 3), (64, 16, 1), (128, 2, 3), (128, 8, 1),
                                       (256, 1, 1), (256, 4, 3)])
def test_plane_step1(n, x, batch, order, dtype):
    """Step 1 and its inverse plane by plane, in every row layout, on
    non-Hermitian input (the real columns' imaginary parts included)."""
    p = Plan(n, dtype, slab_x=x, batch=batch, fuse_pack=order in ("send", "paper"),
             paper_order=order == "paper", inplace=order == "inplace")
    xin, xref = real_input(p.real_shape, 21000 + n + x, dtype)
    want = oracle.r2c2d_planes(xref)
    g, gref = cplx_input((batch, x, n, n // 2 + 1), 21500 + n + x, dtype)
    back = 0.5 * oracle.c2r2d_planes(gref, n)
    if order == "inplace":
        buf = p.empty_inplace()
        p.real_view(buf).copy_(xin)
        S = host(p.r2c_(buf))
        out = p.c2r_(g.clone(), scale=0.5)
    else:
        S = host(p.r2c(xin))
        if order != "natural":
            want = oracle.pack_slab(want, n // x, paper_order=order == "paper")
            g = p.pack(g)
        out = p.c2r(g, scale=0.5)
    torch.cuda.synchronize()
    assert rel_l2(S, want) <= TOL[dtype]
    assert rel_l2(host(out), back) <= TOL[dtype]
