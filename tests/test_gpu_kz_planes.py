"""The kz planes of a forward transform by themselves: no plane takes on
rounding errors of another one's size.  A rel-L2 over the whole spectrum cannot
see that.

A field that is constant along z has X[M] = Re Z[0] - Im Z[0] = 0 exactly in
every row (the packed row's real and imaginary parts go through the same
additions), and zeros stay zero through y and x: the plane kz = N/2 holds exact
zeros.  With alternating signs along z the same holds for kz = 0.
"""
import pytest
import torch

import synth
from paper_2202_12756_amd import Plan

pytestmark = pytest.mark.gpu

F64, F32 = torch.float64, torch.float32
DTYPES = pytest.mark.parametrize("dtype", [F64, F32], ids=["f64", "f32"])

# (n, x, batch): step 1 of slabs (x < n) and whole grids
PLANE_TILES = [(32, 4, 2), (32, 32, 2), (64, 8, 2), (64, 64, 1), (128, 8, 1), (128, 128, 1),
               (256, 2, 1), (256, 256, 1), (512, 2, 1), (512, 512, 1), (1024, 2, 1)]


def _spectrum(p, inplace, f):
    if not inplace:
        return p.r2c(f)
    buf = p.empty_inplace()
    p.real_view(buf).copy_(f)
    return p.r2c_(buf)


@DTYPES
@pytest.mark.parametrize("inplace", [False, True], ids=["out_of_place", "inplace"])
@pytest.mark.parametrize("n,x,batch", PLANE_TILES)
def test_empty_planes_stay_empty(n, x, batch, inplace, dtype):
    p = Plan(n, dtype, slab_x=x, batch=batch, inplace=inplace)
    g = synth.uniform((batch, x, n, 1), 31000 + n + x, dtype, "cpu").cuda().expand(p.real_shape)
    sign = torch.ones(n, dtype=dtype, device="cuda")
    sign[1::2] = -1
    F = _spectrum(p, inplace, g.contiguous())
    assert torch.count_nonzero(F[..., n // 2]) == 0
    assert torch.count_nonzero(F[..., 0]) > 0
    F = _spectrum(p, inplace, g * sign)
    assert torch.count_nonzero(F[..., 0]) == 0
    assert torch.count_nonzero(F[..., n // 2]) > 0
