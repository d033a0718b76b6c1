"""The chain in one pass over A, D = (A B) C, which the library takes by itself (no tile parameter given)
for a dense B where it is the faster order: small-integer entries, so that the result must equal the
oracle bit for bit whatever the order of the sums."""
import numpy as np
import pytest

import oracle
import tf_inputs as ti

pytestmark = pytest.mark.gpu


def _check(A, bcol, ccol, dtype, seed=5, transposed=False):
    import paper_2407_00243_amd as tf
    from gpu_util import Case
    B = ti.dense_small_int(A.n_rows, bcol, dtype, seed)
    C = ti.dense_small_int(*((ccol, bcol) if transposed else (bcol, ccol)), dtype, seed + 1)
    D_ref, _ = (oracle.chain_ct if transposed else oracle.chain)(A, B, C)
    prob = ti.Problem("chain", "gemm_spmm", np.dtype(dtype), A, B, C)
    c = Case(prob, **(dict(flags=tf.TF_FLAG_C_TRANSPOSED) if transposed else {}))
    try:
        for _ in range(2):
            assert np.array_equal(c.run().astype(np.float64), D_ref)
    finally:
        c.close()


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("bcol", [2, 4, 5, 15, 16, 17, 31, 33, 48, 49, 64, 65, 96, 97, 127, 128])
def test_every_depth_and_ragged_rows_of_b(dtype, bcol):
    """One size below, at and above every depth the kernel is instantiated for; rows of B whose last
    16-byte piece is moved back; n not a multiple of sixteen."""
    A = ti.random_local_csr(1203, 9, 6, 0.0, dtype, 21, int_values=True, empty_row_prob=0.0)
    _check(A, bcol, 2 * bcol + 3, dtype)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("ccol", [4, 7, 16, 23, 40, 48, 64, 65, 80, 96, 130])
def test_every_column_grouping_and_ragged_rows_of_d(dtype, ccol):
    A = ti.random_local_csr(700, 5, 5, 0.0, dtype, 22, int_values=True, empty_row_prob=0.0)
    _check(A, 20, ccol, dtype, transposed=ccol % 2 == 0)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("per_row", [1, 3, 12, 40, 200])
def test_rows_cut_into_parts_and_several_passes(dtype, per_row):
    """Few rows with many entries are cut into up to sixteen parts; a block takes several passes."""
    A = ti.random_local_csr(150, 149, per_row, 0.0, dtype, 23, int_values=True, empty_row_prob=0.0)
    _check(A, 24, 24, dtype)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("bcol,ccol,n", [(128, 128, 32768), (128, 128, 32785), (128, 128, 40000), (128, 128, 65600),
                                         (128, 16, 33000), (80, 64, 50033)])
def test_rounds_that_do_not_take_all_waves(dtype, bcol, ccol, n):
    """Blocks that are left after whole rounds are dealt over the workgroups (256 compute units, 2048 to 3072 waves:
    none, one, a fifth of the waves and a few, after one round and after two)."""
    A = ti.random_local_csr(n, 9, 4, 0.0, dtype, 24, int_values=True, empty_row_prob=0.0)
    _check(A, bcol, ccol, dtype)


@pytest.mark.parametrize("empty", [0.3, 0.97])
def test_rows_of_many_lengths_and_empty_rows(empty):
    """Rows sorted by length inside windows; empty rows are zeros even where B holds no finite number."""
    import torch
    import paper_2407_00243_amd as tf
    from gpu_util import dev
    n, w = 5000, 32
    rng = np.random.default_rng(3)
    lens = np.where(rng.random(n) < empty, 0, rng.integers(1, 40, n))
    rowptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    row = np.repeat(np.arange(n), lens)
    colidx = np.clip(row + rng.integers(-20, 21, row.size), 1, n - 1).astype(np.int32)
    A = ti.Csr(n, n, rowptr, colidx, rng.integers(-2, 3, row.size).astype(np.float32))
    _check(A, w, 2 * w, np.float32)
    B = torch.zeros((n, w), device="cuda")
    B[0] = float("inf")                                    # row 0 of B is read by no row of A
    D = torch.full((n, w), float("nan"), device="cuda")
    with tf.Plan(A, w, w, False) as plan:
        plan.run(B, dev(np.eye(w, dtype=np.float32)), D, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert not D.cpu().numpy().any()
        C = torch.full((w, w), float("inf"), device="cuda")
        plan.run(B, C, D, torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
    assert not D.cpu().numpy()[lens == 0].any()
