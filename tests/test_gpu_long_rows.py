"""The z passes of rows of 2048 and 4096 in the layouts and counts of rows that
select their kernels: pencil chunks, in place, and fewer rows than a workgroup
takes."""
import pytest
import torch

import oracle
from helpers import TOL, cplx_input, host, real_input, rel_l2
from paper_2202_12756_amd import PencilPlan, Plan, _lib

pytestmark = pytest.mark.gpu

DTYPES = pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])


@DTYPES
@pytest.mark.parametrize("n,pr,pc,batch", [(2048, 512, 4, 2), (2048, 2048, 1024, 3), (2048, 1024, 1024, 1),
                                           (4096, 1024, 8, 1), (4096, 4096, 2048, 3),
                                           (4096, 4096, 2048, 1)])
def test_pencil_rows(n, pr, pc, batch, dtype):
    """Forward into the chunks of the first exchange and back, weighted and not; the
    last grids have 2 to 6 rows, fewer than a workgroup (2 to 8) or no multiple of
    it."""
    p = PencilPlan(n, dtype, (pr, pc), 0, batch=batch)
    f, ref = real_input(p.real_shape, 43000 + n + pr, dtype)
    want = oracle.r2c_last(ref)
    for weighted in (False, True):
        got = p.z_r2c(f, scale=0.5, weighted=weighted)
        full = torch.cat([p.chunk(got, c) for c in range(pc)], dim=-1)
        w = 0.5 * want.copy()
        if weighted:
            w[..., 1:-1] *= 2.0
        assert rel_l2(host(full), w) <= TOL[dtype]
    # back, from bins with imaginary parts at kz = 0 and N/2 (discarded)
    g, gref = cplx_input((batch, p.x, p.y, n // 2 + 1), 43500 + n + pr, dtype)
    send = torch.empty(p.send_shape, dtype=p.cdtype, device="cuda")
    for c in range(pc):
        k0, k1 = p.kz_range(c)
        p.chunk(send, c).copy_(g[..., k0:k1])
    for weighted in (False, True):
        h = gref.copy()
        if weighted:
            h[..., 1:-1] *= 0.5
        got = p.z_c2r(send, scale=0.25, weighted=weighted)
        assert rel_l2(host(got), 0.25 * oracle.c2r_last(h, n)) <= TOL[dtype]


@DTYPES
@pytest.mark.parametrize("n", [2048, 4096])
def test_rows_in_place(n, dtype):
    p = Plan(n, dtype, slab_x=1, inplace=True)
    buf = p.empty_inplace()
    f, ref = real_input((1, 1, n, n), 44000 + n, dtype)
    p.real_view(buf).copy_(f)
    a = p._inplace_ptr(buf)
    p._exec(_lib.gfft_exec_z_r2c, a, a, 1.0, 0)
    assert rel_l2(host(buf), oracle.r2c_last(ref)) <= TOL[dtype]
    g, gref = cplx_input(buf.shape, 44500 + n, dtype)
    buf.copy_(g)
    p._exec(_lib.gfft_exec_z_c2r, a, a, 0.25, 0)
    assert rel_l2(host(p.real_view(buf)), 0.25 * oracle.c2r_last(gref, n)) <= TOL[dtype]
    p.real_view(buf).copy_(f)
    assert rel_l2(host(p.r2c_(buf)), oracle.r2c2d_planes(ref)) <= TOL[dtype]
    assert rel_l2(host(p.c2r_(buf, scale=1.0 / n ** 2)), ref) <= TOL[dtype]
    torch.cuda.synchronize()


@DTYPES
def test_c2r_rows_of_2048_on_both_sides_of_the_l2_size(dtype):
    """One plane (its FP64 spectrum fits the L2s) and three."""
    for x, batch in ((1, 1), (1, 3)):
        p = Plan(2048, dtype, slab_x=x, batch=batch)
        g, gref = cplx_input(p.spectrum_shape, 45000 + batch, dtype)
        assert rel_l2(host(p.z_c2r(g, scale=0.5)), 0.5 * oracle.c2r_last(gref, 2048)) <= TOL[dtype]
