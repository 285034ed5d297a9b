"""mfq_op_geometry shows what the operator holds."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p,n,amp", [(1, 33, 0.1), (2, 5, 0.1), (4, 6, 0.1), (4, 6, 0.0), (8, 4, 0.1)])
@pytest.mark.parametrize("prec", [0, 1, 2])
def test_geometry_reads_the_operators_data(p, n, amp, prec):
    """Cleared data give a zero tensor, and the tensor of the data as bound is the FP64 operator's to one
    rounding of c_q (or of each entry)."""
    import torch
    import paper_1910_13247_amd as mfq
    space = mfq.Space(mfq.Mesh(n, amp), p)
    op = mfq.Operator(space, 0.5, prec)
    g, ref = op.geometry(), mfq.Operator(space, 0.5).geometry()
    assert (g - ref).abs().max().item() <= (2.0 ** -52 if prec == 0 else 2.0 ** -23) * ref.abs().max().item()
    assert (ref[..., 0] > 0).all()
    op.buffer.zero_()
    torch.cuda.synchronize()
    assert (op.geometry() == 0).all()
