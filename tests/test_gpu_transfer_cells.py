"""The restriction of the highest degrees in FP64 where it goes cell by cell: a single coarse cell and meshes of
17 cells per direction and more."""
import numpy as np
import pytest

from oracle import gmg
from synthetic import uniform_vector

pytestmark = pytest.mark.gpu


def _apply(M, x):
    """M (x) M (x) M on a cube of values"""
    for ax in range(3):
        x = np.moveaxis(np.tensordot(M, x, (1, ax)), 0, ax)
    return x


@pytest.mark.parametrize("p", [7, 8])
@pytest.mark.parametrize("nc", [1, 16, 17, 18])
@pytest.mark.parametrize("bc", [0, 1])
def test_restriction(p, nc, bc):
    """k u |P^T| |x| for the three passes' sums, k = 3 (2 S + 2) + 4, and 64 u on the entries of the 1D tables
    (the matrix of one cell, repeated)."""
    import torch
    import paper_1910_13247_amd as mfq
    print(f"p={p} nc={nc} bc={bc}", flush=True)
    tr = mfq.Transfer(mfq.Space(mfq.Mesh(nc), p, bc), mfq.Space(mfq.Mesh(2 * nc), p, bc))
    S = 2 * p
    one = gmg.prolongation_1d(p, 1, p, 2)
    P = np.zeros((S * nc + 1, p * nc + 1))
    near = np.zeros(P.shape, bool)
    for k in range(nc):
        P[S * k:S * k + S + 1, p * k:p * k + p + 1] = one
        near[S * k:S * k + S + 1, p * k:p * k + p + 1] = True
    if bc:
        P[[0, -1], :] = 0
        P[:, [0, -1]] = 0
    x = uniform_vector(tr.fine.n_dofs, 8)
    got = torch.full((tr.coarse.n_dofs,), 9.0, dtype=torch.float64, device="cuda")
    tr.restrict(torch.from_numpy(x).cuda(), got)
    x = x.reshape((S * nc + 1,) * 3)
    u = 2.0 ** -53
    big, sure = _apply((np.abs(P) + 64 * u * near).T, np.abs(x)), _apply(np.abs(P).T, np.abs(x))
    err = np.abs(got.cpu().numpy().reshape(big.shape) - _apply(P.T, x))
    assert (err <= (3 * (2 * S + 2) + 4) * u * big + (big - sure)).all()


@pytest.mark.parametrize("p,n", [(7, 34), (8, 34), (7, 2)])
def test_residual_in_the_restriction(p, n):
    """b - A x formed by the restriction or stored before it: the same V-cycle bitwise."""
    import torch
    import paper_1910_13247_amd as mfq
    print(f"p={p} n={n}", flush=True)
    out = []
    for fused in (True, False):
        op = mfq.Operator(mfq.Space(mfq.Mesh(n, 0.1), p), 0.5)
        op.set_fused_updates(fused)
        sv = mfq.Solver(op, mfq.MFQ_SOLVER_GMG_FP64, coarse_mode=1, coarse_dofs=100)
        out.append(sv.precondition(op.space.random(31)))
        del sv, op
    torch.cuda.synchronize()
    assert torch.isfinite(out[0]).all() and torch.equal(out[0], out[1])
