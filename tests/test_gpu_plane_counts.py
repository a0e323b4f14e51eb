"""Step 1 of N = 128 and FP32 256 on both sides of the number of planes from which
one workgroup takes a plane, against the separate z and y passes."""
import pytest
import torch

from helpers import TOL
from paper_2202_12756_amd import Plan

pytestmark = pytest.mark.gpu

F64, F32 = torch.float64, torch.float32


@pytest.mark.parametrize("order", ["natural", "send", "paper", "inplace"])
@pytest.mark.parametrize("n,x,batch,dtype", [
    (128, 4, 23, F64), (128, 4, 24, F64), (128, 4, 39, F64), (128, 4, 40, F64), (128, 4, 23, F32),
    (128, 4, 24, F32), (256, 4, 31, F32), (256, 4, 32, F32), (256, 4, 47, F32), (256, 4, 48, F32)])
def test_counts_around_the_rule(n, x, batch, order, dtype):
    p = Plan(n, dtype, slab_x=x, batch=batch, fuse_pack=order in ("send", "paper"),
             paper_order=order == "paper", inplace=order == "inplace")
    s = Plan(n, dtype, slab_x=x, batch=batch)
    torch.manual_seed(40000 + n + batch)
    f = torch.randn(s.real_shape, dtype=dtype, device="cuda")
    g = torch.view_as_complex(torch.randn(s.spectrum_shape + (2,), dtype=dtype, device="cuda"))
    want = s.y_c2c(s.z_r2c(f), -1)
    back = s.z_c2r(s.y_c2c(g.clone(), +1), scale=0.25, weighted=True)
    if order == "inplace":
        buf = p.empty_inplace()
        p.real_view(buf).copy_(f)
        F = p.r2c_(buf)
        out = p.r2c_adjoint_(g.clone(), scale=0.25)
    else:
        if order != "natural":
            want, g = p.pack(want), p.pack(g)
        F = p.r2c(f)
        out = p.inverse_keep(g, scale=0.25, adjoint=True)
        assert torch.equal(out, p.r2c_adjoint(g.clone(), scale=0.25))

    def off(a, b):
        return (torch.linalg.vector_norm(a - b) / torch.linalg.vector_norm(b)).item()

    assert off(F, want) <= TOL[dtype] and off(out, back) <= TOL[dtype]
