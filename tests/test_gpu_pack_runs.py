"""Packs on both sides of the rules that choose between whole runs to a
workgroup and runs in parts: bit for bit the permutation, and back."""
import pytest
import torch

from helpers import cplx_input
from paper_2202_12756_amd import PencilPlan, Plan

pytestmark = pytest.mark.gpu

F64, F32 = torch.float64, torch.float32


@pytest.mark.parametrize("n,x,batch,dtype", [
    (128, 1, 7, F32), (1024, 1, 1, F32), (2048, 1, 1, F32), (1024, 1, 1, F64), (1024, 1, 8, F64),
    (64, 8, 3, F64), (128, 16, 3, F64)])
def test_slab_runs(n, x, batch, dtype):
    """Odd FP32 runs of 65, 513 and 1025; FP64 513 in arrays up to and beyond
    64 MB; 264 and 1040 (two and five rounds, the last nearly empty)."""
    p = Plan(n, dtype, slab_x=x, batch=batch)
    s, _ = cplx_input((batch, x, n, p.k), 36000 + n, dtype)
    want = s.view(batch, x, n // x, x, p.k).transpose(1, 2)
    send = p.pack(s)
    assert torch.equal(send, want)
    assert torch.equal(p.unpack(send), s)


@pytest.mark.parametrize("n,pr,pc,dtype", [(128, 8, 2, F64), (256, 16, 4, F32), (1024, 8, 2, F64),
                                           (2048, 128, 2, F64)])
def test_pencil_runs(n, pr, pc, dtype):
    """Power-of-two runs of 512 and 256 elements, of 512 KB in planes 2 MB apart,
    and of 128 KB in planes 8 MB apart (eight elements a thread)."""
    p = PencilPlan(n, dtype, (pr, pc), 0)
    torch.manual_seed(37000 + n)
    a = torch.view_as_complex(torch.randn(p.ypencil_shape + (2,), dtype=dtype, device="cuda"))
    want = a.view(1, pc, p.x, p.h, n // pr, p.w).transpose(2, 3)
    send = p.pack2(a)
    assert torch.equal(send, want.reshape(p.send2_shape))
    assert torch.equal(p.unpack2(send), a)
