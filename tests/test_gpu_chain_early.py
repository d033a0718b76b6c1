"""The one-pass chain whose first gathers of a block leave before the block ahead of it is multiplied (chain_early)."""
import numpy as np
import pytest

import tf_inputs as ti

pytestmark = pytest.mark.gpu


def _near_diagonal(n, lengths, rng):
    """Row j: lengths[j % len] entries of the columns around j."""
    length = np.minimum(np.resize(np.asarray(lengths), n), n)
    rowptr = np.concatenate([[0], np.cumsum(length)]).astype(np.int32)
    first = np.clip(np.arange(n) - length // 2, 0, n - length)
    cols = np.repeat(first, length) + np.arange(rowptr[-1]) - np.repeat(rowptr[:-1], length)
    return ti.Csr(n, n, rowptr, cols.astype(np.int32), rng.standard_normal(rowptr[-1]))


@pytest.mark.parametrize("transposed", [False, True])
@pytest.mark.parametrize("n,bcol,ccol,lengths", [
    (49152, 64, 20, [5]), (49151, 64, 20, [5]), (65537, 49, 23, [4]), (65553, 57, 2, [1]), (64001, 50, 16, [5, 4, 3]),
    (80001, 63, 33, [0] * 16 + [5] * 16), (80003, 64, 48, [0, 1, 2, 3, 4, 5, 6, 7, 8, 9]), (90007, 64, 64, [7]), (74000, 64, 130, [7, 6]),
    (60000, 55, 100, [3] * 15 + [33]), (52000, 63, 70, [2] * 2000 + [900]), (50000, 64, 161, [4])])
def test_first_gathers_ahead_of_the_multiplications(n, bcol, ccol, lengths, transposed):
    """fp64 at 49 to 64 columns of B from 24 MiB (36 MiB over five entries a row): one to ten entries a row, rows of none in
    blocks of their own, cut rows, one to several groups of column blocks, blocks that the last rows do not fill."""
    import paper_2407_00243_amd as tf
    from gpu_util import Case, assert_parity
    rng = np.random.default_rng(n + bcol)
    A = _near_diagonal(n, lengths, rng)
    B, C = rng.standard_normal((n, bcol)), rng.standard_normal((bcol, ccol))
    prob = ti.Problem("early", "gemm_spmm", np.dtype(np.float64), A, B, C)
    given = ti.Problem("early", "gemm_spmm", np.dtype(np.float64), A, B, np.ascontiguousarray(C.T)) if transposed else prob
    c = Case(given, **(dict(flags=tf.TF_FLAG_C_TRANSPOSED) if transposed else {}))
    try:
        assert c.plan.schedule()["execution"] == tf.TF_EXECUTE_ONE_PASS
        for _ in range(2):
            assert_parity(prob, c.run())
    finally:
        c.close()
