"""The access-pattern yardstick follows its pass onto the numbered-through tiles."""
import pytest
import torch

from paper_2202_12756_amd import PencilPlan, Plan, _lib

pytestmark = pytest.mark.gpu

F64, F32 = torch.float64, torch.float32


def _us(run):
    run()
    best = float("inf")
    for _ in range(5):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        run()
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3)
    return best


@pytest.mark.parametrize("n,pr,pc,axis,dtype", [(64, 1, 32, 0, F32), (1024, 64, 512, 0, F64),
                                                (32, 4, 16, 1, F32)])
def test_narrow_chunks(n, pr, pc, axis, dtype):
    """On one bin to a chunk a tile per line set leaves all but one or two of its
    lanes idle and takes 5 to 30 times as long as the pass; the copy takes the
    pass's own tiles (twice its time allowed)."""
    rows = (n // pr) * (n // pc)
    p = PencilPlan(n, dtype, (pr, pc), 0, batch=max(1, (1 << 24) // (rows * n)))
    shape = p.ypencil_shape if axis == 0 else p.xpencil_shape
    torch.manual_seed(41000 + n)
    a = torch.view_as_complex(torch.randn(shape + (2,), dtype=dtype, device="cuda"))
    b = a.clone()

    def copy():
        p._exec(_lib.gfft_exec_pass_copy, axis, b.data_ptr())

    copy()
    assert torch.equal(b, a.conj().resolve_conj())
    line = p.y_c2c if axis == 0 else p.x_c2c
    assert _us(copy) <= 2.0 * _us(lambda: line(a, -1))


@pytest.mark.parametrize("dtype", [F64, F32], ids=["f64", "f32"])
@pytest.mark.parametrize("n,x", [(16, 2), (32, 4), (64, 8)])
def test_short_lines(n, x, dtype):
    """Slabs of N = 16, 32 and (paper's order) 64: every element's conjugate."""
    p = Plan(n, dtype, slab_x=x, batch=5, paper_order=True)
    torch.manual_seed(42000 + n)
    for axis, shape in ((0, p.spectrum_shape), (1, p.pencil_shape)):
        a = torch.view_as_complex(torch.randn(shape + (2,), dtype=dtype, device="cuda"))
        assert torch.equal(p.pass_copy(a.clone(), axis), a.conj().resolve_conj())
