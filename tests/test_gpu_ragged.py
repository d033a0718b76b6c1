"""Widths that are no whole number of 16-byte pieces in the kernels of the two wavefronts: rows gathered
and stored in pieces of which the last is moved back, rows of B of the dense product the same way.
Small-integer entries: the result must equal the oracle bit for bit."""
import numpy as np
import pytest

import oracle
import tf_inputs as ti

pytestmark = pytest.mark.gpu


def _far(n, dtype, seed):
    """Rows of 0 to 11 entries, all of them half of the matrix away (no tile fuses one), a few rows with the
    diagonal entry only, and one row long enough to be split."""
    rng = np.random.default_rng(seed)
    lens = rng.integers(0, 12, n)
    lens[5] = 300
    diag = rng.random(n) < 0.1
    lens[diag] = 1
    rows = np.repeat(np.arange(n), lens)
    cols = (rows + n // 2 + rng.integers(-n // 8, n // 8, rows.size)) % n
    cols[np.isin(rows, np.flatnonzero(diag))] = rows[np.isin(rows, np.flatnonzero(diag))]
    order = np.lexsort((cols, rows))
    rowptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    return ti.Csr(n, n, rowptr, cols[order].astype(np.int32), rng.integers(-2, 3, rows.size).astype(dtype))


def _check(A, B, C, kind, streams=None, **params):
    from gpu_util import Case
    D_ref, _ = oracle.chain(A, B, C)
    c = Case(ti.Problem("ragged", kind, C.dtype, A, B, C), **params)
    try:
        if streams is not None:
            assert c.plan.schedule()["first_wavefront_streams"] == streams
        for fused in (True, False):
            assert np.array_equal(c.run(fused).astype(np.float64), D_ref)
    finally:
        c.close()


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("ccol", [1, 2, 3, 4, 5, 7, 9, 30, 31, 41, 63, 65, 67, 127, 130, 257, 258, 259, 385, 515])
@pytest.mark.parametrize("far", [0, 1])
def test_gathered_rows_of_every_width(dtype, ccol, far):
    """Tiles in LDS (rows near the diagonal) and the streaming first wavefront (far rows); widths around
    one piece, one wave of pieces and the column slices of the tiles."""
    n = 611
    A = _far(n, dtype, 7) if far else ti.random_local_csr(n, 9, 6, 0.0, dtype, 21, int_values=True, empty_row_prob=0.1)
    B = ti.random_local_csr(n, n - 1, 9, 0.0, dtype, 22, int_values=True, empty_row_prob=0.1)
    C = ti.dense_small_int(n, ccol, dtype, 5)
    _check(A, B, C, "spmm_spmm", ct_size=64, **(dict(streams=1) if far else {}))
    _check(A, B, C, "spmm_spmm")               # (the library's choice: the plain pair of operations)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("ccol,col_slice", [(30, 16), (33, 16), (35, 5), (70, 64), (66, 16), (9, 2)])
def test_ragged_column_slices_of_tiles(dtype, ccol, col_slice):
    if (col_slice * np.dtype(dtype).itemsize) % 16 and (ccol * np.dtype(dtype).itemsize) % 16 == 0:
        pytest.skip("slices of an aligned width are whole pieces")
    n = 611
    A = ti.random_local_csr(n, 9, 6, 0.0, dtype, 21, int_values=True, empty_row_prob=0.1)
    _check(A, A, ti.dense_small_int(n, ccol, dtype, 5), "spmm_spmm", col_slice=col_slice, ct_size=64)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("bcol", [1, 2, 3, 4, 5, 15, 17, 31, 33, 48, 63, 65, 96, 127, 129, 250, 257, 260])
def test_streaming_product_with_every_depth(dtype, bcol):
    """One size below and above every depth the product is instantiated for, aligned or not, into D1 rows
    and rows of D of any alignment."""
    n = 611
    A = _far(n, dtype, 8)
    ccol = (41, 64, 23, 130)[bcol % 4]
    B, C = ti.dense_small_int(n, bcol, dtype, 5), ti.dense_small_int(bcol, ccol, dtype, 6)
    _check(A, B, C, "gemm_spmm", streams=1, ct_size=64)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("bcol,ccol", [(32, 92), (36, 128), (5, 128), (1, 120), (64, 130), (17, 127)])
@pytest.mark.parametrize("transposed", [0, 1])
def test_graph_with_narrow_rows_of_b_multiplies_a_by_b_first(dtype, bcol, ccol, transposed):
    """Far rows and bCol well below cCol: Y = A B, which the workspace then holds, D = Y C; rows split over
    lane groups, and empty rows, which are zeros even where C holds no finite number."""
    import ctypes
    import torch
    import paper_2407_00243_amd as tf
    from gpu_util import dev, dev_csr
    n = 40000
    rng = np.random.default_rng(4)
    lens = rng.integers(0, 9, n)
    lens[rng.integers(0, n, 20)] = rng.integers(100, 2000, 20)
    lens[:50] = 0
    rowptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    colidx = rng.integers(0, n, rowptr[-1]).astype(np.int32)
    A = ti.Csr(n, n, rowptr, colidx, rng.integers(-2, 3, colidx.size).astype(dtype))
    B = ti.dense_small_int(n, bcol, dtype, 5)
    C = ti.dense_small_int(*((ccol, bcol) if transposed else (bcol, ccol)), dtype, 6)
    D_ref, _ = (oracle.chain_ct if transposed else oracle.chain)(A, B, C)
    Y_ref = oracle.chain(A, B, np.eye(bcol, dtype=dtype))[0]
    D = torch.full((n, ccol), float("nan"), dtype=dev(B).dtype, device="cuda")
    stream = torch.cuda.current_stream().cuda_stream
    with tf.Plan(dev_csr(A), bcol, ccol, False, flags=tf.TF_FLAG_C_TRANSPOSED if transposed else 0) as plan:
        Bd, Cd = dev(B), dev(C)
        plan.run(Bd, Cd, D, stream)
        torch.cuda.synchronize()
        assert np.array_equal(D.cpu().numpy().astype(np.float64), D_ref)
        Y = np.empty((n, bcol), dtype=dtype)
        hip = ctypes.CDLL("libamdhip64.so")
        hip.hipMemcpy.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_size_t, ctypes.c_int]
        assert hip.hipMemcpy(Y.ctypes.data, plan.workspace(), Y.nbytes, 2) == 0
        assert np.array_equal(Y.astype(np.float64), Y_ref)
        Cd.fill_(float("inf"))
        plan.run(Bd, Cd, D, stream)
        torch.cuda.synchronize()
        assert not D[:50].cpu().numpy().any()


def test_small_plan_without_baseline_still_runs_the_plain_pair():
    """The pack of all rows exists for the fused calls, the baseline calls stay refused."""
    import paper_2407_00243_amd as tf
    from gpu_util import Case
    n = 3000
    A = ti.random_local_csr(n, 9, 6, 0.0, np.float32, 21, int_values=True, empty_row_prob=0.1)
    C = ti.dense_small_int(n, 20, np.float32, 5)
    c = Case(ti.Problem("pair", "spmm_spmm", C.dtype, A, A, C), flags=tf.TF_FLAG_NO_BASELINE)
    try:
        assert np.array_equal(c.run().astype(np.float64), oracle.chain(A, A, C)[0])
        with pytest.raises(Exception):
            c.run(False)
    finally:
        c.close()
