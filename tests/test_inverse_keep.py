"""The inverse that leaves its input as it is (gfft_exec_inverse_keep, used by
the autograd functions): bit for bit what c2r / r2c_adjoint give on a copy, on
every route an inverse can take."""
import pytest
import torch

from helpers import cplx_input, real_input
from paper_2202_12756_amd import Plan, _lib, irfft3, rfft3

F64, F32 = torch.float64, torch.float32


def test_null_plan_is_refused_on_the_host():
    assert _lib.gfft_exec_inverse_keep(None, None, None, None, 1.0, 0, None) == _lib.GFFT_E_INVALID_ARG
    assert _lib.gfft_inverse_work_bytes(None) == 0


@pytest.mark.gpu
@pytest.mark.parametrize("n,x,batch,dtype,terms", [
    (16, 16, 3, F64, 0), (32, 32, 2, F32, 0), (32, 32, 65, F32, 0), (64, 64, 1, F64, 0),
    (128, 128, 2, F32, 0), (256, 256, 1, F64, 0), (512, 512, 1, F64, 0), (64, 64, 2, F32, 2),
    (16, 8, 3, F32, 0), (64, 8, 1, F64, 0), (256, 2, 3, F64, 0), (512, 4, 1, F32, 3)])
def test_same_bits_and_input_kept(n, x, batch, dtype, terms):
    p = Plan(n, dtype, slab_x=x, batch=batch, mfma_terms=terms)
    g, _ = cplx_input(p.spectrum_shape, 25000 + n, dtype)
    g0 = g.clone()
    for adjoint, call in ((False, p.c2r), (True, p.r2c_adjoint)):
        got = p.inverse_keep(g, scale=0.5, adjoint=adjoint)
        want = call(g.clone(), scale=0.5)
        assert torch.equal(got, want)
        assert torch.equal(g, g0)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [F64, F32], ids=["f64", "f32"])
def test_views_of_spectra(dtype):
    """Lazy conjugates, strided, expanded and 8-byte-aligned spectra, as the
    input of irfft3 and as the gradient that reaches rfft3."""
    n = 32
    p = Plan(n, dtype, batch=2)
    g, _ = cplx_input(p.spectrum_shape, 25500, dtype)
    views = {
        "conj": g.conj(),
        "transposed": g.transpose(1, 2),
        "expanded": g[:1].expand(p.spectrum_shape),
        "odd_start": torch.cat([g.new_zeros(1), g.reshape(-1)])[1:].view(p.spectrum_shape),
    }
    u, _ = real_input(p.real_shape, 25600, dtype)
    for name, v in views.items():
        plain = v.resolve_conj().clone(memory_format=torch.contiguous_format)
        assert torch.equal(irfft3(v, p, 0.25), p.c2r(plain.clone(), scale=0.25)), name
        uu = u.clone().requires_grad_(True)
        (gu,) = torch.autograd.grad(rfft3(uu, p), uu, v)
        assert torch.equal(gu, p.r2c_adjoint(plain.clone())), name


@pytest.mark.gpu
def test_bad_buffers_are_refused():
    p = Plan(64, F64)
    g, out = p.empty_spectrum(), p.empty_real()
    work = torch.empty_like(g)
    s = torch.cuda.current_stream().cuda_stream
    keep = lambda a, w, o: _lib.gfft_exec_inverse_keep(p._h, a, w, o, 1.0, 0, s)  # noqa: E731
    assert _lib.gfft_inverse_work_bytes(p._h) == g.numel() * 16
    assert keep(g.data_ptr(), None, out.data_ptr()) == _lib.GFFT_E_INVALID_ARG
    assert keep(g.data_ptr(), g.data_ptr(), out.data_ptr()) == _lib.GFFT_E_INVALID_ARG
    assert keep(g.data_ptr(), out.data_ptr(), out.data_ptr()) == _lib.GFFT_E_INVALID_ARG
    assert keep(g.data_ptr(), work.data_ptr() + 8, out.data_ptr()) == _lib.GFFT_E_ALIGN
    q = Plan(64, F64, inplace=True)
    assert _lib.gfft_exec_inverse_keep(q._h, g.data_ptr(), work.data_ptr(), g.data_ptr(), 1.0, 0,
                                       s) == _lib.GFFT_E_INVALID_ARG
