"""Operators at the limits of what the entry points accept."""
import numpy as np
import pytest

from oracle import ebe

pytestmark = pytest.mark.gpu


def test_largest_q1_mesh():
    """Q1 on 1024^3 cells, the largest mesh (1,076,890,625 DoFs, 2^32 cell pencils): the operator binds, and
    rows agree with the oracle's (2 k u32 of the summed magnitudes, k = 8 (p + 1) + 16)."""
    import torch
    import paper_1910_13247_amd as mfq
    p, n = 1, 1024
    print("Q1 1024^3 FP32", flush=True)
    op = mfq.Operator(mfq.Space(mfq.Mesh(n), p), 0.5, mfq.MFQ_FP32)
    x = op.space.random(3, mfq.MFQ_FP32)
    y = op.vmult(x)
    torch.cuda.synchronize()
    N1 = n + 1
    rows = np.concatenate([np.random.default_rng(4).integers(0, op.n_dofs, 24),
                           [1 + N1 + N1 * N1, op.n_dofs - 2 - N1 - N1 * N1, op.n_dofs - 1, 32 + 2 * N1 + N1 * N1]])
    xn = x.cpu().numpy()
    yo = ebe.ebe_rows(p, n, 0.0, 0.5, xn, 1, rows)
    mag = ebe.ebe_rows(p, n, 0.0, 0.5, xn, 1, rows, magnitude=True)
    yg = y[torch.from_numpy(rows).cuda()].double().cpu().numpy()
    assert np.all(np.abs(yg - yo) <= 2 * (8 * (p + 1) + 16) * 2.0 ** -24 * mag + 1e-30)
