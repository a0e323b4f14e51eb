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

import oracle
import synth
from helpers import TOL, host, rel_l2
from paper_2202_12756_amd import Plan

pytestmark = pytest.mark.gpu

F64, F32 = torch.float64, torch.float32
DTYPES = pytest.mark.parametrize("dtype", [F64, F32], ids=["f64", "f32"])

# (n, x, batch): step 1 of slabs (x < n) and whole grids
PLANE_TILES = [(32, 4, 2), (32, 32, 2), (64, 8, 2), (64, 64, 1), (128, 8, 1), (128, 8, 24),
               (128, 128, 1), (256, 8, 24),
               (256, 2, 1), (256, 256, 1), (512, 2, 1), (512, 512, 1), (1024, 2, 1)]
ROW_TILES = [(2048, 1, 2), (4096, 1, 1)]
BOXES = [(16, 16, 3), (32, 32, 97)]


def _spectrum(p, inplace, f):
    if not inplace:
        return p.r2c(f)
    buf = p.empty_inplace()
    p.real_view(buf).copy_(f)
    return p.r2c_(buf)


@DTYPES
@pytest.mark.parametrize("inplace", [False, True], ids=["out_of_place", "inplace"])
@pytest.mark.parametrize("n,x,batch", BOXES + PLANE_TILES + ROW_TILES)
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


@DTYPES
@pytest.mark.parametrize("n,x,batch", BOXES + [(32, 4, 2), (64, 64, 1), (128, 8, 24), (128, 128, 1), (256, 2, 1),
                                               (512, 2, 1), (1024, 1, 1), (2048, 1, 1)])
def test_odd_planes_beside_a_strong_kz_0(n, x, batch, dtype):
    """g(x, y) + 1e-4 noise: the odd kz see only the differences f[n] -
    f[n + N/2] of z's first butterflies, which are exact (1 <= g < 2), so each
    odd plane is as accurate as on the noise alone.  Its reference is the
    transform of f - g (exact too), as g has no odd kz."""
    p = Plan(n, dtype, slab_x=x, batch=batch)
    g = 1.5 + 0.5 * synth.uniform((batch, x, n, 1), 32000 + n, dtype, "cpu")
    f = g + 1e-4 * synth.uniform(p.real_shape, 32500 + n, dtype, "cpu")
    rest = (f.double() - g.double()).numpy()
    want = oracle.r2c3d(rest) if x == n else oracle.r2c2d_planes(rest)
    got = host(p.r2c(f.cuda()))
    for k in (1, 3, n // 4 + 1, n // 2 - 1):
        assert rel_l2(got[..., k], want[..., k]) <= TOL[dtype], k


@DTYPES
@pytest.mark.parametrize("n", [16, 1024, 2048, 4096])
def test_z_pass_near_the_largest_value(n, dtype):
    """Rows whose kz = 0 bin is 0.9 of the type's largest value keep it, and
    the other bins are 0 (a constant row)."""
    p = Plan(n, dtype, slab_x=1)
    top = 0.9 * torch.finfo(dtype).max
    F = p.z_r2c(torch.full(p.real_shape, top / n, dtype=dtype, device="cuda"))
    assert torch.isfinite(torch.view_as_real(F)).all()
    # log2 N rounded additions, one unit each
    assert ((F[..., 0].real / top - 1).abs() <= (n.bit_length() + 2) * torch.finfo(dtype).eps).all()
    assert torch.count_nonzero(F[..., 0].imag) == 0 and torch.count_nonzero(F[..., n // 2]) == 0


INVERSES = BOXES + [(32, 32, 2), (32, 4, 2), (64, 64, 1), (64, 2, 1), (128, 128, 1), (128, 2, 1),
                    (128, 8, 24), (256, 8, 24), (256, 256, 1), (256, 2, 1), (512, 512, 1),
                    (512, 16, 1), (1024, 16, 1), (2048, 8, 1), (4096, 4, 1)]


@DTYPES
@pytest.mark.parametrize("n,x,batch,order", [(*c, o) for c in INVERSES for o in
                                             ("natural", "inplace", "send")
                                             if o != "send" or c[1] < c[0]])
def test_imaginary_parts_that_do_not_count(n, x, batch, order, dtype):
    """A bin that is its own Hermitian partner counts by its real part alone
    (w Re(G) in the inverse's definition): infinities and NaN there leave the
    result as zeros do, bit for bit, and the rest of the spectrum is the same."""
    p = Plan(n, dtype, slab_x=x, batch=batch, inplace=order == "inplace", fuse_pack=order == "send")
    own = [0, n // 2]
    torch.manual_seed(33000 + n)
    g = torch.randn((batch, x, n, n // 2 + 1, 2), dtype=dtype, device="cuda")

    def inverse(value):
        v = g.clone()
        for ky in own:
            for kz in own:
                v[:, own if x == n else slice(None), ky, kz, 1] = value
        c = torch.view_as_complex(v)
        if order == "inplace":
            return p.c2r_(c, scale=0.5).clone()
        return p.c2r(p.pack(c) if order == "send" else c, scale=0.5)

    want = inverse(0.0)
    assert torch.isfinite(want).all()
    for value in (float("inf"), float("nan")):
        assert torch.equal(inverse(value), want)


@DTYPES
@pytest.mark.parametrize("n", [16, 64, 1024, 2048, 4096])
def test_z_pass_discards_edge_imaginary_parts(n, dtype):
    """gfft_exec_z_c2r: the imaginary parts of kz = 0 and kz = N/2 are
    discarded, whatever they hold."""
    p = Plan(n, dtype, slab_x=1)
    torch.manual_seed(34000 + n)
    g = torch.randn(p.spectrum_shape + (2,), dtype=dtype, device="cuda")
    out = []
    for value in (0.0, float("inf"), float("nan")):
        v = g.clone()
        v[..., 0, 1] = value
        v[..., n // 2, 1] = value
        out.append(p.z_c2r(torch.view_as_complex(v)))
    assert torch.isfinite(out[0]).all()
    assert torch.equal(out[1], out[0]) and torch.equal(out[2], out[0])


@DTYPES
@pytest.mark.parametrize("n,batch", [(16, 2), (32, 97), (32, 2), (64, 1)])
def test_scales_at_the_ends_of_the_range(n, batch, dtype):
    """The scale is applied between the sums: before z in the inverse, after z
    in the adjoint.  A spectrum of g in every bin is N^3 g at the origin, N^2 g
    after x and y and g / N once scaled by N^-3; a constant field N g likewise.
    So both come out as g and N g to rounding (sums of equal values and powers
    of two are exact; 32 eps is ample) from g / N just above the smallest normal
    value to N^2 g at a quarter of the largest."""
    p = Plan(n, dtype, batch=batch)
    fi = torch.finfo(dtype)
    for g in (0.25 * fi.max / n ** 2, 1.1 * fi.tiny * n):
        G = torch.zeros(p.spectrum_shape, dtype=p.cdtype, device="cuda")
        torch.view_as_real(G)[..., 0] = g
        f = p.c2r(G, scale=1.0 / n ** 3)
        assert torch.isfinite(f).all()
        at = f[:, 0, 0, 0] / g
        assert ((at - 1).abs() <= 32 * fi.eps).all()
        h = torch.full(p.real_shape, g * n, dtype=dtype, device="cuda")
        A = p.c2r_adjoint(h, scale=1.0 / n ** 3)
        assert torch.isfinite(torch.view_as_real(A)).all()
        assert ((A[:, 0, 0, 0].real / (g * n) - 1).abs() <= 32 * fi.eps).all()
