"""FP32 operators against the FP64 ones on the same input: the geometry of a curved mesh must cost no
more accuracy than a stored tensor does."""
import pytest

pytestmark = pytest.mark.gpu


def _error(p, n, amp, seed):
    import torch
    import paper_1910_13247_amd as mfq
    space = mfq.Space(mfq.Mesh(n, amp), p)
    x = space.random(seed, mfq.MFQ_FP32)
    y = mfq.Operator(space, 0.5, mfq.MFQ_FP32).vmult(x).double()
    ref = mfq.Operator(space, 0.5, mfq.MFQ_FP64).vmult(x.double())
    return ((y - ref).norm() / ref.norm()).item()


@pytest.mark.parametrize("p", range(1, 9))
def test_fp32_curved_geometry(p):
    """Relative error on the curved mesh over the error on the undeformed one, same coefficient.  There
    the point step rounds c_q and one product per component.  With the tensor held to one rounding per
    entry the ratio is 1.06 on average over p (1.03 to 1.07), with c_q rounded and the rest in FP64 1.05;
    with g, D and the tensor formed in FP32 1.09 to 1.16.  Both forms of the cell loop (one launch, and
    by colours), mean over both and over seeds."""
    sizes = ({1: 40, 2: 20, 3: 13, 4: 10, 5: 8, 6: 7, 7: 6, 8: 5}[p], {1: 100, 2: 64, 3: 43, 4: 33, 5: 26, 6: 22, 7: 19, 8: 17}[p])
    r = [_error(p, n, 0.1, seed) / _error(p, n, 0.0, seed) for n in sizes for seed in (1, 2, 3, 4)]
    print(f"p={p} ratio {sum(r) / len(r):.3f}", flush=True)
    assert sum(r) / len(r) <= 1.085
