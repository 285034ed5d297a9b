"""The operator's coloured form, on meshes above the sizes at which the one-launch form takes over
(FP64: 67, 45, 31, 22, 19, 13, 11, 11 cells per direction for p = 1..8; FP32: 79, 49, 40, 23, 21, 15, 14,
11), with a ragged last brick along x, in every geometry form, both precisions, overwriting and accumulating."""
import itertools

import numpy as np
import pytest

from oracle import ebe
from synthetic import uniform_vector

pytestmark = pytest.mark.gpu

U32 = 2.0 ** -24
BRICK = {1: (32, 2), 2: (14, 2), 3: (16, 1), 4: (5, 2), 5: (7, 1), 6: (4, 1), 7: (4, 1), 8: (3, 1)}  # cells x, y
SIZES = {1: 79, 2: 49, 3: 40, 4: 27, 5: 22, 6: 15, 7: 14, 8: 11}
FORMS = [(0.0, 0.0, 1), (0.0, 0.5, 1), (0.1, 0.5, 1), (0.1, 0.5, 0)]


def _rows(p, n):
    """Nodes around a corner of the first brick, of the second (odd coordinates before, even after), and
    of the last cells, and nodes of the boundary faces and the ragged brick's end."""
    bx, by = BRICK[p]
    N1, E = p * n + 1, p * n
    rows = set()
    for c in ((bx, by, 1), (2 * bx, 2 * by, 2), (n - 1, n - 1, n - 1)):
        for o in itertools.product((-1, 0, 1), repeat=3):
            I, J, K = (p * ci + oi for ci, oi in zip(c, o))
            rows.add(I + N1 * (J + N1 * K))
    a = E - p
    for I, J, K in ((E, a, a), (a, E, a), (a, a, E), (E, E, E), (E, E, a), (0, 0, 0), (0, p, 1), (p, 0, 1), (1, p, 0)):
        rows.add(I + N1 * (J + N1 * K))
    return np.array(sorted(rows))


@pytest.mark.parametrize("p", range(1, 9))
@pytest.mark.parametrize("amp,alpha,bc", FORMS)
def test_coloured_rows(p, amp, alpha, bc):
    """Against the oracle's rows.  FP64: 1e-12 of the largest; FP32: 2 k u32 of the summed magnitudes, k = 8 (p
    + 1) + 16; accumulating adds 8 roundings (one per colour) of the sum's magnitude."""
    import torch
    import paper_1910_13247_amd as mfq
    n = SIZES[p]
    print(f"coloured p={p} n={n} amp={amp} alpha={alpha} bc={bc}", flush=True)
    space = mfq.Space(mfq.Mesh(n, amp), p, bc)
    x = uniform_vector(space.n_dofs, seed=200 + p).astype(np.float32).astype(np.float64)
    y0 = uniform_vector(space.n_dofs, seed=210 + p).astype(np.float32).astype(np.float64)
    rows = _rows(p, n)
    yo = ebe.ebe_rows(p, n, amp, alpha, x, bc, rows)
    mag = ebe.ebe_rows(p, n, amp, alpha, x, bc, rows, magnitude=True)
    at = torch.from_numpy(rows).cuda()
    k = 8 * (p + 1) + 16
    for prec, u in ((mfq.MFQ_FP64, 2.0 ** -53), (mfq.MFQ_FP32, U32)):
        op = mfq.Operator(space, alpha, prec)
        xt = torch.from_numpy(x).to(op.dtype).cuda()
        y = op.vmult(xt, torch.full_like(xt, float("nan")))
        ya = op.vmult_add(xt, torch.from_numpy(y0).to(op.dtype).cuda())
        assert torch.isfinite(y).all() and torch.isfinite(ya).all()
        y, ya = (v[at].double().cpu().numpy() for v in (y, ya))
        tol = 1e-12 * np.abs(yo).max() if prec == mfq.MFQ_FP64 else 2 * k * u * mag + 1e-30
        assert np.all(np.abs(y - yo) <= tol)
        assert np.all(np.abs(ya - (yo + y0[rows])) <= tol + 8 * u * (mag + np.abs(y0[rows])))


@pytest.mark.parametrize("p", range(1, 9))
@pytest.mark.parametrize("amp,alpha,bc", FORMS)
def test_coloured_equals_fused(p, amp, alpha, bc):
    """Every node: a smoother step through the coloured operator is bitwise the fused step, whose kernel
    gathers and sums node by node (p > 1: the plain one goes plane by plane)."""
    import torch
    import paper_1910_13247_amd as mfq
    n = SIZES[p]
    print(f"coloured and fused p={p} n={n} amp={amp} alpha={alpha} bc={bc}", flush=True)
    for prec in (mfq.MFQ_FP64, mfq.MFQ_FP32):
        op = mfq.Operator(mfq.Space(mfq.Mesh(n, amp), p, bc), alpha, prec)
        b, x0, dinv = (op.space.random(s, prec) for s in (1, 2, 3))
        out = []
        for fused in (True, False):
            op.set_fused_updates(fused)
            x = x0.clone()
            op.chebyshev(dinv, b, x, False, 2, 0.2, 2.0)
            out.append(x)
        assert torch.isfinite(out[0]).all()
        assert torch.equal(out[0], out[1]), (out[0] - out[1]).abs().max().item()


# (degree, cells, amplitude, coefficients): each solve alone runs its operators in one launch, together
# they are more workgroups than that form takes, so the batch goes by colours
BATCHES = [(4, 16, 0.0, (0.2, 0.4, 0.6, 0.8)), (4, 16, 0.1, (0.0, 0.3, 0.5, 0.7)), (2, 40, 0.0, (0.3, 0.6)),
           (6, 12, 0.0, (0.0, 0.0)), (5, 16, 0.0, (0.2, 0.5, 0.8)), (8, 9, 0.0, (0.4, 0.6))]


@pytest.mark.parametrize("p,n,amp,alphas", BATCHES)
def test_batched_colours_equal_single_launch(p, n, amp, alphas):
    import torch
    import paper_1910_13247_amd as mfq
    print(f"batched colours p={p} n={n} amp={amp}", flush=True)
    st = torch.cuda.Stream()
    sols, bs, alone = [], [], []
    for i, a in enumerate(alphas):
        op = mfq.Operator(mfq.Space(mfq.Mesh(n, amp), p), a)
        sols.append(mfq.Solver(op, mfq.MFQ_SOLVER_GMG_MIXED, coarse_mode=1))
        bs.append(op.space.random(600 + i))
    torch.cuda.synchronize()
    for sv, b in zip(sols, bs):
        x = sv.op.new_vector()
        sv.begin(b, x, rtol=1e-10, max_iter=300, stream=st)
        while not mfq.batch_step([sv], iters=2)[0]:
            pass
        assert sv.end()[0] == mfq.MFQ_OK
        alone.append(x)
    batch = mfq.Batch(8, stream=st)
    xs = []
    for sv, b in zip(sols, bs):
        xs.append(sv.op.new_vector())
        sv.begin(b, xs[-1], rtol=1e-10, max_iter=300, stream=st)
    pending, steps = list(range(len(sols))), 0
    while pending:
        flags = batch.run([sols[i] for i in pending], iters=2, stream=st)
        pending = [i for i, f in zip(pending, flags) if not f]
        steps += 1
        assert steps < 300
    torch.cuda.synchronize()
    for sv, x, ref in zip(sols, xs, alone):
        assert sv.end()[0] == mfq.MFQ_OK
        assert torch.equal(x, ref)
