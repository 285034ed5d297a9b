"""Device bytes that an operator reports (CPU: no device is touched)."""
import pytest

BRICK = {1: (32, 2, 1), 2: (14, 2, 1), 3: (16, 1, 1), 4: (5, 2, 1), 5: (7, 1, 1), 6: (4, 1, 1), 7: (4, 1, 1), 8: (3, 1, 1)}


def _bytes(p, n, amp, prec):
    import paper_1910_13247_amd as mfq
    lib = mfq._lib
    m = lib.mfq_mesh_create(n, amp)
    s = lib.mfq_space_create(m, p, 1)
    op = lib.mfq_op_create(s, 0.5, prec)
    b = lib.mfq_op_device_bytes(op)
    lib.mfq_op_destroy(op)
    lib.mfq_space_destroy(s)
    lib.mfq_mesh_destroy(m)
    return b


@pytest.mark.parametrize("p", range(1, 9))
@pytest.mark.parametrize("amp", [0.0, 0.1])
def test_matrix_core_operator_holds_six_values_per_point(p, amp):
    """The index lattice and six FP32 values per quadrature point of every brick, nothing more."""
    import paper_1910_13247_amd as mfq
    up = lambda b: -(-b // 256) * 256
    for n in (1, 7, 40):
        bx, by, bz = BRICK[p]
        bricks = -(-n // bx) * -(-n // by) * -(-n // bz)
        idx = up(bricks * (bx * p + 1) * (by * p + 1) * (bz * p + 1) * 4)
        assert _bytes(p, n, amp, mfq.MFQ_FP32_MFMA) == idx + up(bricks * bx * by * bz * (p + 1) ** 3 * 6 * 4)
