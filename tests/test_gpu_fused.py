"""GPU parity of the kernels that take several axes of the transform in one
memory pass, against the FP64 oracle at the sizes where their tiles change.
Tolerances: the rel-L2 bounds of the separate passes (FP64 1e-13, FP32 5e-6).
"""
import pytest
import torch

import oracle
from helpers import TOL, cplx_input, host, real_input, rel_l2
from paper_2202_12756_amd import PencilPlan, Plan, _lib

pytestmark = pytest.mark.gpu

F64, F32 = torch.float64, torch.float32
DTYPES = pytest.mark.parametrize("dtype", [F64, F32], ids=["f64", "f32"])


@DTYPES
@pytest.mark.parametrize("order", ["natural", "send", "paper", "inplace"])
@pytest.mark.parametrize("n,x,batch", [(32, 1, 3), (32, 8, 2), (64, 1, 3), (64, 16, 1), (128, 2, 3), (128, 8, 1),
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


def _offset(shape, dtype, nbytes=16):
    """An empty buffer that starts 16 bytes past a line boundary."""
    skip = nbytes // torch.empty((), dtype=dtype).element_size()
    size = 1
    for v in shape:
        size *= v
    return torch.empty(size + skip, dtype=dtype, device="cuda")[skip:].view(shape)


@pytest.mark.parametrize("aligned", [True, False], ids=["line", "off_line"])
@pytest.mark.parametrize("n,batch,dtype", [(128, 3, F64), (128, 2, F32), (256, 1, F64),
                                           (256, 2, F32), (512, 1, F64), (512, 1, F32)])
def test_split_y_full_grid(n, batch, dtype, aligned):
    """Full grids through the two-pass kernels against the separate z, y and
    x passes, with the adjoints' weights, on buffers on and off the 128-byte
    line grid; up to 256^3 also against the oracle."""
    p = Plan(n, dtype, batch=batch)
    xin, xref = real_input(p.real_shape, 22000 + n, dtype)
    out = p.empty_spectrum() if aligned else _offset(p.spectrum_shape, p.cdtype)
    F = p.r2c(xin, out)
    W = p.c2r_adjoint(xin, scale=3.0)
    sep, sepw = p.z_r2c(xin), p.z_r2c(xin, scale=3.0, weighted=True)
    for s in (sep, sepw):
        p.y_c2c(s, -1)
        p.x_c2c(s, -1)
    tol = TOL[dtype]

    def off(a, b):
        return (torch.linalg.vector_norm(a - b) / torch.linalg.vector_norm(b)).item()

    assert off(F, sep) <= tol and off(W, sepw) <= tol
    if n <= 256 and aligned:
        assert rel_l2(host(F), oracle.r2c3d(xref)) <= tol
    del sep, sepw, W, F, out, xref
    # inverse on a non-Hermitian half spectrum
    g, gref = cplx_input(p.spectrum_shape, 22500 + n, dtype)
    gs = g.clone()
    p.x_c2c(gs, +1)
    p.y_c2c(gs, +1)
    want, wantw = p.z_c2r(gs, scale=0.5), p.z_c2r(gs, scale=0.25, weighted=True)
    work = torch.empty_like(g) if aligned else _offset(p.spectrum_shape, p.cdtype)
    got = p.c2r(work.copy_(g), scale=0.5)
    gotw = p.r2c_adjoint(work.copy_(g), scale=0.25)
    assert off(got, want) <= tol and off(gotw, wantw) <= tol
    if n == 128 and aligned:
        assert rel_l2(host(got), 0.5 * oracle.c2r3d(gref, n)) <= tol


@DTYPES
@pytest.mark.parametrize("n,ranks,batch", [(64, 1, 3), (64, 8, 2), (64, 64, 2), (128, 16, 2),
                                           (256, 1, 1), (256, 8, 1), (1024, 64, 1)])
def test_x_pass_orders(n, ranks, batch, dtype):
    """x passes on both sides of the tile order's bounds (elements under
    4 KB apart, up to and beyond 512 KB), on buffers on and off the 128-byte
    line grid, both signs."""
    p = Plan(n, dtype, slab_x=n // ranks, batch=batch)
    pen, ref = cplx_input(p.pencil_shape, 23000 + n + ranks, dtype)
    for sign in (-1, +1):
        want = oracle.c2c_axis(ref, 1, sign)
        for buf in (torch.empty_like(pen), _offset(p.pencil_shape, p.cdtype)):
            got = p.x_c2c(buf.copy_(pen), sign)
            torch.cuda.synchronize()
            assert rel_l2(host(got), want) <= TOL[dtype]


@pytest.mark.parametrize("n,x,batch", [(2048, 1, 3), (2048, 8, 1), (4096, 1, 1), (4096, 4, 1)])
def test_lines_of_64_elements_per_thread(n, x, batch):
    """FP32 x and y lines of 2048 and 4096, both signs, on buffers on and off
    the 128-byte line grid."""
    p = Plan(n, F32, slab_x=x, batch=batch)
    for shape, axis, run in ((p.pencil_shape, 1, p.x_c2c), (p.spectrum_shape, 2, p.y_c2c)):
        data, ref = cplx_input(shape, 27000 + n + x, F32)
        for sign in (-1, +1):
            want = oracle.c2c_axis(ref, axis, sign)
            for buf in (torch.empty_like(data), _offset(shape, p.cdtype)):
                got = run(buf.copy_(data), sign)
                torch.cuda.synchronize()
                assert rel_l2(host(got), want) <= TOL[F32]


@DTYPES
@pytest.mark.parametrize("inplace", [False, True], ids=["out_of_place", "inplace"])
@pytest.mark.parametrize("n,batch", [(16, 1), (16, 7), (32, 1), (32, 63), (32, 65)])
def test_small_grids(n, batch, inplace, dtype):
    """Whole grids of N = 16 and 32, with the adjoints, the inverse on
    non-Hermitian input."""
    p = Plan(n, dtype, batch=batch, inplace=inplace)
    tol = TOL[dtype]
    xin, xref = real_input(p.real_shape, 24000 + n + batch, dtype)
    g, gref = cplx_input((batch, n, n, n // 2 + 1), 24500 + n + batch, dtype)

    def fwd(call, call_, scale):
        if not inplace:
            return call(xin, **scale)
        buf = p.empty_inplace()
        p.real_view(buf).copy_(xin)
        return call_(buf, **scale)

    F = fwd(p.r2c, p.r2c_, {})
    A = fwd(p.c2r_adjoint, p.c2r_adjoint_, {"scale": 3.0})
    f = (p.c2r_ if inplace else p.c2r)(g.clone(), scale=0.5)
    a = (p.r2c_adjoint_ if inplace else p.r2c_adjoint)(g.clone(), scale=0.25)
    torch.cuda.synchronize()
    assert rel_l2(host(F), oracle.r2c3d(xref)) <= tol
    assert rel_l2(host(A), 3.0 * oracle.c2r3d_adjoint(xref)) <= tol
    assert rel_l2(host(f), 0.5 * oracle.c2r3d(gref, n)) <= tol
    assert rel_l2(host(a), 0.25 * oracle.r2c3d_adjoint(gref, n)) <= tol


@DTYPES
@pytest.mark.parametrize("n,x,batch,order", [
    (512, 2, 3, "natural"), (512, 16, 1, "send"), (512, 8, 1, "send"), (512, 2, 1, "inplace"),
    (1024, 1, 2, "natural"), (1024, 16, 1, "send"), (1024, 8, 1, "send"), (1024, 4, 1, "send"),
    (1024, 2, 1, "paper"), (2048, 1, 2, "natural"), (2048, 8, 1, "send"), (2048, 2, 1, "send"), (2048, 1, 1, "send"), (2048, 2, 1, "paper"),
    (2048, 1, 1, "inplace"), (4096, 1, 1, "natural"), (4096, 4, 1, "send"), (4096, 2, 1, "send")])
def test_long_rows_step1(n, x, batch, order, dtype):
    """Step 1 of long rows with y split between the z and y passes, and the
    layouts that keep the whole y pass (fewer rows of a plane per chunk than
    the step, the paper's order, in place), against the separate passes
    (and one plane of them against the oracle), weighted and not."""
    p = Plan(n, dtype, slab_x=x, batch=batch, fuse_pack=order in ("send", "paper"),
             paper_order=order == "paper", inplace=order == "inplace")
    s = Plan(n, dtype, slab_x=x, batch=batch)
    tol = TOL[dtype]

    def off(a, b):
        return (torch.linalg.vector_norm(a - b) / torch.linalg.vector_norm(b)).item()

    xin, xref = real_input(s.real_shape, 26000 + n, dtype)
    sep, sepw = s.z_r2c(xin), s.z_r2c(xin, scale=3.0, weighted=True)
    for a in (sep, sepw):
        s.y_c2c(a, -1)
    assert rel_l2(host(sep[:1, :1]), oracle.r2c2d_planes(xref[:1, :1])) <= tol
    g, _ = cplx_input(s.spectrum_shape, 26500 + n, dtype)
    gy = s.y_c2c(g.clone(), +1)
    want, wantw = s.z_c2r(gy, scale=0.5), s.z_c2r(gy, scale=0.25, weighted=True)
    if order == "inplace":
        def padded():
            buf = p.empty_inplace()
            p.real_view(buf).copy_(xin)
            return buf
        F, W = p.r2c_(padded()), p.c2r_adjoint_(padded(), scale=3.0)
        f, w = p.c2r_(g.clone(), scale=0.5), p.r2c_adjoint_(g.clone(), scale=0.25)
    else:
        if order != "natural":
            sep, sepw, g = p.pack(sep), p.pack(sepw), p.pack(g)
        F, W = p.r2c(xin), p.c2r_adjoint(xin, scale=3.0)
        f, w = p.c2r(g.clone(), scale=0.5), p.r2c_adjoint(g.clone(), scale=0.25)
        assert torch.equal(p.inverse_keep(g, scale=0.5), f)
    assert off(F, sep) <= tol and off(W, sepw) <= tol
    assert off(f, want) <= tol and off(w, wantw) <= tol


@pytest.mark.parametrize("n,x,batch,dtype", [
    (16, 1, 3, F32), (16, 2, 3, F32), (64, 4, 5, F32), (64, 4, 5, F64), (512, 1, 1, F32),
    (512, 1, 1, F64), (256, 4, 1, F64), (1024, 2, 1, F32)])
def test_pack_run_lengths(n, x, batch, dtype):
    """The slab pack is the oracle's permutation, bit for bit, for runs of
    one to many rounds of a workgroup, whole, paired and odd."""
    p = Plan(n, dtype, slab_x=x, batch=batch)
    s, ref = cplx_input((batch, x, n, n // 2 + 1), 27000 + n + x, dtype)
    send = p.pack(s)
    back = p.unpack(send)
    torch.cuda.synchronize()
    assert (host(send) == oracle.pack_slab(ref, n // x)).all()
    assert torch.equal(back, s)


@pytest.mark.parametrize("dtype,n,pr,pc", [(F32, 1024, 4, 2), (F64, 512, 2, 1), (F32, 64, 8, 2)])
def test_pencil_pack_runs(dtype, n, pr, pc):
    """The second exchange's pack with runs of a power of two: long (spread
    over the run), and short, and the Nyquist column's odd ones."""
    for col in {0, pc - 1}:
        p = PencilPlan(n, dtype, (pr, pc), col)
        a, _ = cplx_input(p.ypencil_shape, 28000 + n + col, dtype)
        b = p.pack2(a)
        want = a.view(p.batch, p.pc, p.x, p.h, n // pr, p.w).permute(0, 1, 3, 2, 4, 5)
        torch.cuda.synchronize()
        assert torch.equal(b, want.reshape(p.send2_shape))
        assert torch.equal(p.unpack2(b), a)


@DTYPES
@pytest.mark.parametrize("n,pr,pc", [(64, 2, 8), (128, 4, 32), (512, 64, 64), (1024, 128, 128),
                                     (2048, 512, 512)])
def test_narrow_pencils(n, pr, pc, dtype):
    """y lines of kz chunks narrower than a tile, several planes to a tile,
    the last column's odd width and a ragged last tile included."""
    for col in (0, pc - 1):
        p = PencilPlan(n, dtype, (pr, pc), col, batch=3)
        a, ref = cplx_input(p.ypencil_shape, 29000 + n + col, dtype)
        # y = c' Y + y_l runs over (block, y_l)
        ref = ref.transpose(0, 1, 3, 2, 4).reshape(3, n, p.x, p.w)
        for sign in (-1, +1):
            got = host(p.y_c2c(a.clone(), sign)).transpose(0, 1, 3, 2, 4).reshape(3, n, p.x, p.w)
            assert rel_l2(got, oracle.c2c_axis(ref, 1, sign)) <= TOL[dtype]


@pytest.mark.parametrize("n", [16, 32])
def test_rows_past_one_grid(n):
    """More rows than one launch of the z passes (n = 16) or plane passes
    (n = 32) takes, in place: the entries at both ends and around the end of
    the first slice equal those of a small plan, bit for bit."""
    slice_ = (1 << 28) // n
    p = Plan(n, F32, slab_x=1, batch=slice_ + 3, inplace=True)
    q = Plan(n, F32, slab_x=1, batch=2, inplace=True)
    buf, small = p.empty_inplace(), q.empty_inplace()
    buf.zero_()

    def fwd(plan, b):
        if n == 32:
            return plan.r2c_(b)
        a = plan._inplace_ptr(b)
        plan._exec(_lib.gfft_exec_z_r2c, a, a, 1.0, 0)
        return b

    def inv(plan, b, scale):
        if n == 32:
            return plan.c2r_(b, scale=scale)
        a = plan._inplace_ptr(b)
        plan._exec(_lib.gfft_exec_z_c2r, a, a, scale, 0)
        return plan.real_view(b)

    at = [0, slice_ - 1, slice_ + 1]
    want, ref = [], []
    for i, b in enumerate(at):
        xin, xref = real_input(q.real_shape, 29000 + n + i, F32)
        p.real_view(buf)[b:b + 2].copy_(xin)
        q.real_view(small).copy_(xin)
        ref.append(xref)
        want.append(fwd(q, small).clone())
    fwd(p, buf)
    torch.cuda.synchronize()
    for b, f in zip(at, want):
        assert torch.equal(buf[b:b + 2], f)
    out = inv(p, buf, 1.0 / (n if n == 16 else n * n))
    torch.cuda.synchronize()
    for b, xref in zip(at, ref):
        assert rel_l2(host(out[b:b + 2]), xref) <= TOL[F32]
