"""The ways in which the fused calls run the chain where the library chooses (tf_schedule_view.execution)."""
import numpy as np
import pytest

import oracle
import tf_inputs as ti

pytestmark = pytest.mark.gpu


def far_csr(n, dtype, seed):
    """Rows of 0 to 8 entries anywhere in the matrix, a few long enough to be split over lane groups."""
    rng = np.random.default_rng(seed)
    lens = rng.integers(0, 9, n)
    lens[rng.integers(0, n, 20)] = rng.integers(100, 2000, 20)
    rowptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    colidx = rng.integers(0, n, rowptr[-1]).astype(np.int32)
    return ti.Csr(n, n, rowptr, colidx, rng.integers(-2, 3, colidx.size).astype(dtype))


def _problem(execution, dtype):
    import paper_2407_00243_amd as tf
    local = lambda n: ti.random_local_csr(n, 9, 6, 0.0, dtype, 21, int_values=True, empty_row_prob=0.1)
    if execution == tf.TF_EXECUTE_PLAIN_PAIR:
        A = local(3000)
        return ti.Problem("pair", "spmm_spmm", np.dtype(dtype), A, A, ti.dense_small_int(3000, 20, dtype, 6))
    A, bcol, ccol = (local(3000), 24, 40) if execution == tf.TF_EXECUTE_ONE_PASS else (far_csr(40000, dtype, 4), 32, 92)
    return ti.Problem("chain", "gemm_spmm", np.dtype(dtype), A, ti.dense_small_int(A.n_rows, bcol, dtype, 5),
                      ti.dense_small_int(bcol, ccol, dtype, 6))


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("execution", [1, 2, 3])
def test_workspace_holds_the_d1_rows_for_whoever_asked_for_it(execution, dtype):
    """After tf_plan_workspace a fused execution leaves D1 row i in slot spill_slot[i], whatever way the
    library had chosen for the plan; small-integer entries, so D and D1 must be exact."""
    from gpu_util import Case, read_workspace
    prob = _problem(execution, dtype)
    D_ref, _ = oracle.chain(prob.A, prob.B, prob.C)
    eye = ti.Csr(prob.n, prob.n, np.arange(prob.n + 1, dtype=np.int32), np.arange(prob.n, dtype=np.int32),
                 np.ones(prob.n, dtype))
    D1_ref, _ = oracle.chain(eye, prob.B, prob.C)
    c = Case(prob)
    try:
        s = c.plan.schedule()
        assert s["execution"] == execution
        assert np.array_equal(c.run().astype(np.float64), D_ref)
        c.plan.workspace()
        assert np.array_equal(c.run().astype(np.float64), D_ref)
        ws = read_workspace(c.plan, s, c.ccol, dtype).astype(np.float64)
        rows = np.flatnonzero(s["spill_slot"] >= 0)
        assert rows.size and np.array_equal(ws[s["spill_slot"][rows]], D1_ref[rows])
    finally:
        c.close()


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("bcol", [4, 30, 64, 127])
@pytest.mark.parametrize("n,even", [(150, True), (5000, True), (20000, False)])
def test_padding_of_the_one_pass_chain_adds_nothing(dtype, bcol, n, even):
    """Rows cut into parts of unequal length (few rows) and blocks of unequal rows are padded: where B holds
    infinities, a row of D is infinite if its row of A reads one of them, and its finite sum if not."""
    import paper_2407_00243_amd as tf
    from gpu_util import Case
    rng = np.random.default_rng(8)
    lens = np.full(n, 7) if even else rng.integers(1, 14, n)
    rowptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    rows = np.repeat(np.arange(n), lens)
    colidx = np.minimum(np.maximum(rows - 6, 0) + (np.arange(rows.size) - rowptr[rows]), n - 1).astype(np.int32)
    A = ti.Csr(n, n, rowptr, colidx, rng.integers(1, 4, rows.size).astype(dtype))
    B, C = rng.integers(1, 4, (n, bcol)).astype(dtype), rng.integers(1, 4, (bcol, 20)).astype(dtype)
    hit = rng.random(n) < 0.05
    D_ref, _ = oracle.chain(A, np.where(hit[:, None], dtype(0), B), C)
    D_ref[np.unique(rows[hit[colidx]])] = np.inf
    B[hit] = np.inf
    c = Case(ti.Problem("chain", "gemm_spmm", np.dtype(dtype), A, B, C))
    try:
        assert c.plan.schedule()["execution"] == tf.TF_EXECUTE_ONE_PASS
        assert np.isinf(D_ref).any() and np.isfinite(D_ref).any()
        assert np.array_equal(c.run().astype(np.float64), D_ref)
    finally:
        c.close()


def _rows_of(lens, dtype, rng):
    """Rows of the given lengths whose columns lie around the diagonal, in no order, some twice."""
    n = lens.size
    rowptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    rows = np.repeat(np.arange(n), lens)
    reach = np.repeat(np.maximum(lens, 8), lens)
    colidx = np.clip(rows + rng.integers(-reach, reach + 1), 0, n - 1).astype(np.int32)
    return ti.Csr(n, n, rowptr, colidx, rng.integers(-2, 3, rows.size).astype(dtype))


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("bcol,ccol", [(8, 8), (50, 23), (64, 64), (128, 128)])
@pytest.mark.parametrize("kind", ["few", "many"])
def test_long_rows_among_short_ones_are_cut(dtype, bcol, ccol, kind):
    """Blocks of the one-pass chain that hold a row far longer than the others: rows of just below and above
    every number of parts, next to each other, first and last, up to the longest row that a block takes."""
    import paper_2407_00243_amd as tf
    from gpu_util import Case
    rng = np.random.default_rng(9)
    if kind == "few":
        lens = np.full(60011, 5)
        lens[[0, 17, 18, 40, 41, 42, 43, 5000, 5016, 9999, 60009, 60010]] = [
            33, 200, 1024, 16, 17, 31, 32, 0, 513, 80, 129, 640]
    else:
        lens = np.minimum(np.exp(rng.normal(1.3, 1.2, 50000)).astype(np.int64), 1024)
    A = _rows_of(lens, dtype, rng)
    B, C = ti.dense_small_int(A.n_rows, bcol, dtype, 5), ti.dense_small_int(bcol, ccol, dtype, 6)
    c = Case(ti.Problem("chain", "gemm_spmm", np.dtype(dtype), A, B, C))
    try:
        assert c.plan.schedule()["execution"] == tf.TF_EXECUTE_ONE_PASS
        assert np.array_equal(c.run().astype(np.float64), oracle.chain(A, B, C)[0])
    finally:
        c.close()


@pytest.mark.parametrize("dtype,bcol,ccol,n", [
    (np.float64, 128, 128, 8000),      # 4 column groups, one per workgroup, as many waves as the machine holds
    (np.float64, 128, 128, 16000),     # two per workgroup
    (np.float64, 127, 95, 16000),      # 3 groups: two and one
    (np.float64, 128, 128, 33000),     # all in one
    (np.float32, 100, 120, 16000), (np.float32, 16, 300, 12000), (np.float32, 16, 300, 4000), (np.float64, 96, 70, 9000)])
def test_column_groups_of_the_one_pass_chain_over_workgroups(dtype, bcol, ccol, n):
    import paper_2407_00243_amd as tf
    from gpu_util import Case
    A = ti.random_local_csr(n, 5, 5, 0.0, dtype, 31, int_values=True, empty_row_prob=0.0)
    B, C = ti.dense_small_int(n, bcol, dtype, 5), ti.dense_small_int(bcol, ccol, dtype, 6)
    c = Case(ti.Problem("chain", "gemm_spmm", np.dtype(dtype), A, B, C))
    try:
        assert c.plan.schedule()["execution"] == tf.TF_EXECUTE_ONE_PASS
        assert np.array_equal(c.run().astype(np.float64), oracle.chain(A, B, C)[0])
    finally:
        c.close()


def _hubs(n, dtype, rng, values):
    """Far rows, among them some around every length at which a row is cut into parts of a block, takes a block, the
    four blocks of a workgroup, or several times that (32 entries for each part, 1 to 64 parts a block)."""
    lens = rng.integers(0, 9, n)            # (thousands of rows of one to four entries: several to a lane group)
    hubs = [32 * g + d for g in (1, 2, 4, 8, 16, 32, 64, 128, 256) for d in (-1, 0, 1, 3)] + [6001, 12345, 20000]
    lens[rng.permutation(n)[:len(hubs)]] = hubs
    rowptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    colidx = rng.integers(0, n, rowptr[-1]).astype(np.int32)
    return ti.Csr(n, n, rowptr, colidx, values(colidx.size).astype(dtype))


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("kind,bcol,ccol,slices", [
    ("spmm", 0, 64, 1), ("spmm", 0, 64, 2), ("spmm", 0, 30, 0), ("spmm", 0, 300, 0), ("spmm", 0, 1, 0), ("spmm", 0, 3, 0),
    ("spmm", 0, 4, 0), ("spmm", 0, 8, 0), ("spmm", 0, 13, 0), ("gemm", 128, 41, 0), ("gemm", 128, 128, 4), ("gemm", 32, 92, 0)])
def test_rows_cut_over_lane_groups_waves_and_workgroups(dtype, kind, bcol, ccol, slices):
    """In the second wavefront, in Y = A B and in the unfused second operation, for every number of lanes per row.
    The counts of the pieces are back at zero after every run."""
    from gpu_util import Case
    n = 30011
    rng = np.random.default_rng(12)
    A = _hubs(n, dtype, rng, lambda k: rng.integers(-2, 3, k))
    sparse = kind == "spmm"
    B = ti.random_local_csr(n, 50, 4, 0.0, dtype, 22, int_values=True) if sparse else ti.dense_small_int(n, bcol, dtype, 5)
    C = ti.dense_small_int(n if sparse else bcol, ccol, dtype, 6)
    D_ref, _ = oracle.chain(A, B, C)
    c = Case(ti.Problem("hubs", kind + "_spmm", np.dtype(dtype), A, B, C), gather_slices=slices)
    try:
        s = c.plan.schedule()
        assert np.array_equal(np.unique(s["wf1_unit_ptr"]), s["wf1_unit_ptr"])      # a cut row is in one unit
        for fused in (True, True, False, True, False):
            assert np.array_equal(c.run(fused).astype(np.float64), D_ref)
    finally:
        c.close()


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("ccol,slices", [(128, 4), (130, 0)])
def test_padding_of_gathered_rows_adds_nothing(dtype, ccol, slices):
    """Blocks of rows of unequal length, and of rows cut into unequal parts, are padded: where D1 holds infinities, a
    row of D is infinite if its row of A reads one of them, and its finite sum if not."""
    from gpu_util import Case
    n, bcol = 30011, 32
    rng = np.random.default_rng(13)
    A = _hubs(n, dtype, rng, lambda k: rng.integers(1, 3, k))
    B, C = rng.integers(1, 4, (n, bcol)).astype(dtype), rng.integers(1, 4, (bcol, ccol)).astype(dtype)
    hit = rng.random(n) < 0.002
    D_ref, _ = oracle.chain(A, np.where(hit[:, None], dtype(0), B), C)
    D_ref[np.unique(np.repeat(np.arange(n), np.diff(A.rowptr))[hit[A.colidx]])] = np.inf
    B[hit] = np.inf
    c = Case(ti.Problem("padding", "gemm_spmm", np.dtype(dtype), A, B, C), gather_slices=slices)
    try:
        assert c.plan.schedule()["first_wavefront_streams"] and np.isinf(D_ref).any() and np.isfinite(D_ref).any()
        for fused in (True, False):
            assert np.array_equal(c.run(fused).astype(np.float64), D_ref)
    finally:
        c.close()


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("kind,bcol,ccol", [("gemm", 64, 41), ("gemm", 128, 33), ("gemm", 36, 96), ("gemm", 128, 70), ("gemm", 20, 23),
                                            ("gemm", 64, 260), ("gemm", 64, 128), ("spmm", 0, 41), ("spmm", 0, 23), ("spmm", 0, 70),
                                            ("spmm", 0, 300)])
def test_slices_of_one_cache_line_and_padded_rows(dtype, kind, bcol, ccol):
    """A workspace whose slices and rows the library chooses: whole lines, the last one partly used, three and more
    slices (shared unevenly by the eight XCDs), rows padded to a line; and Y = A B over slices of rows of B."""
    import paper_2407_00243_amd as tf
    from gpu_util import Case, read_workspace
    n = max(60013, 14000000 // (ccol * np.dtype(dtype).itemsize))         # (rows that reach beyond an L2)
    rng = np.random.default_rng(14)
    A = _hubs(n, dtype, rng, lambda k: rng.integers(-2, 3, k))
    sparse = kind == "spmm"
    B = _rows_of(rng.integers(0, 6, n), dtype, rng) if sparse else ti.dense_small_int(n, bcol, dtype, 5)
    C = ti.dense_small_int(n if sparse else bcol, ccol, dtype, 6)
    D_ref, _ = oracle.chain(A, B, C)
    c = Case(ti.Problem("lines", kind + "_spmm", np.dtype(dtype), A, B, C))
    try:
        s = c.plan.schedule()
        es, line = np.dtype(dtype).itemsize, s["d1_slice_cols"] * np.dtype(dtype).itemsize
        assert s["far_rows"] and (s["d1_slices"] - 1) * s["d1_slice_cols"] < ccol <= s["d1_slices"] * s["d1_slice_cols"]
        if ccol * es > 128 and (ccol - 1) % (128 // es) + 1 >= 16 // es and ccol * es <= 1024:
            assert line == 128
        for fused in (True, False, True):
            assert np.array_equal(c.run(fused).astype(np.float64), D_ref)
        c.plan.workspace()
        assert np.array_equal(c.run().astype(np.float64), D_ref)
        ws = read_workspace(c.plan, s, ccol, dtype)
        rows = np.flatnonzero(s["spill_slot"] >= 0)
        eye = ti.Csr(n, n, np.arange(n + 1, dtype=np.int32), np.arange(n, dtype=np.int32), np.ones(n, dtype))
        assert np.array_equal(ws[s["spill_slot"][rows]].astype(np.float64), oracle.chain(eye, B, C)[0][rows])
    finally:
        c.close()


@pytest.mark.parametrize("dtype,n,h,ccol", [(np.float64, 40001, 10, 41), (np.float32, 60000, 6, 70),
                                            (np.float64, 20001, 2, 79), (np.float32, 30001, 1, 33)])
def test_both_operations_over_all_rows_of_a_large_band(dtype, n, h, ccol):
    """CSR B, D1 beyond 12 MB: rows with many entries run as the plain pair, the pair and the tiles give the
    exact D for small-integer entries."""
    from gpu_util import Case
    import paper_2407_00243_amd as tf
    rng = np.random.default_rng(n)
    cols = np.arange(n)[:, None] + np.arange(-h, h + 1)
    keep = (cols >= 0) & (cols < n)
    rowptr = np.concatenate([[0], np.cumsum(keep.sum(1))]).astype(np.int32)
    A = ti.Csr(n, n, rowptr, cols[keep].astype(np.int32), rng.integers(-2, 3, int(rowptr[-1])).astype(dtype))
    prob = ti.Problem("band", "spmm_spmm", np.dtype(dtype), A, A, ti.dense_small_int(n, ccol, dtype, 6))
    D_ref, _ = oracle.chain(prob.A, prob.B, prob.C)
    for given, expected in ((dict(), tf.TF_EXECUTE_WAVEFRONTS if h == 2 else tf.TF_EXECUTE_PLAIN_PAIR),
                            (dict(gather_slices=1), tf.TF_EXECUTE_WAVEFRONTS)):
        c = Case(prob, **given)
        try:
            assert c.plan.schedule()["execution"] == expected
            assert np.array_equal(c.run().astype(np.float64), D_ref)
        finally:
            c.close()


@pytest.mark.parametrize("bcol,ccol,expected", [(64, 32, "WAVEFRONTS"), (32, 128, "GATHER_FIRST")])
def test_static_calls_beside_calls_of_the_same_plan(bcol, ccol, expected):
    """Rows cut over several workgroups: a call with the library's own workspace shares no sums and no counts with the
    plan's other calls, on streams of their own and one after the other."""
    import torch
    import paper_2407_00243_amd as tf
    from gpu_util import Case
    n = 30011
    rng = np.random.default_rng(15)
    A = _hubs(n, np.float32, rng, lambda k: rng.integers(-2, 3, k))
    B, C = ti.dense_small_int(n, bcol, np.float32, 5), ti.dense_small_int(bcol, ccol, np.float32, 6)
    D_ref, _ = oracle.chain(A, B, C)
    c = Case(ti.Problem("beside", "gemm_spmm", np.dtype(np.float32), A, B, C))
    try:
        assert c.plan.schedule()["execution"] == getattr(tf, "TF_EXECUTE_" + expected)
        c.plan.prepare_unfused()
        calls = [c.plan.run, lambda *a: tf.tf_gemm_spmm_static(c.plan.handle, *a), c.plan.run_unfused]
        streams = [torch.cuda.Stream() for _ in calls]
        Ds = [[torch.full((n, ccol), float("nan"), device="cuda") for _ in range(8)] for _ in calls]
        torch.cuda.synchronize()
        for k in range(8):
            # (the unfused call of a gather-first plan may run over the row list of the others)
            for call, stream, D in zip(calls, streams, Ds):
                call(c.B, c.C, D[k], stream.cuda_stream)
        torch.cuda.synchronize()
        for D in Ds:
            for d in D:
                assert np.array_equal(d.cpu().numpy().astype(np.float64), D_ref)
    finally:
        c.close()


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_unfused_calls_beside_the_plain_pair(dtype):
    """Both run over the packed copy of all rows, with sums and counts of their own for rows that are cut."""
    import torch
    import paper_2407_00243_amd as tf
    from gpu_util import Case
    n, ccol = 20011, 32
    rng = np.random.default_rng(16)
    lens = np.full(n, 5)
    lens[rng.permutation(n)[:40]] = rng.integers(1, 16000, 40)
    rowptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    near = np.clip(np.repeat(np.arange(n), lens) + np.concatenate([np.arange(k) - k // 2 for k in lens]), 0, n - 1)
    A = ti.Csr(n, n, rowptr, near.astype(np.int32), rng.integers(-2, 3, near.size).astype(dtype))
    C = ti.dense_small_int(n, ccol, dtype, 6)
    D_ref, _ = oracle.chain(A, A, C)
    c = Case(ti.Problem("beside", "spmm_spmm", np.dtype(dtype), A, A, C))
    try:
        assert c.plan.schedule()["execution"] == tf.TF_EXECUTE_PLAIN_PAIR
        c.plan.prepare_unfused()
        streams = [torch.cuda.Stream() for _ in range(2)]
        Ds = [[torch.full((n, ccol), float("nan"), device="cuda", dtype=c.tdtype) for _ in range(6)] for _ in streams]
        torch.cuda.synchronize()
        for k in range(6):
            c.plan.run(c.B, c.C, Ds[0][k], streams[0].cuda_stream)
            c.plan.run_unfused(c.B, c.C, Ds[1][k], streams[1].cuda_stream)
        torch.cuda.synchronize()
        for D in Ds:
            for d in D:
                assert np.array_equal(d.cpu().numpy().astype(np.float64), D_ref)
    finally:
        c.close()


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("ccol,most", [(1, 6), (3, 13), (4, 6), (4, 13), (8, 6), (41, 9), (64, 9), (96, 9), (300, 9)])
def test_lanes_past_a_row_of_b_add_nothing(dtype, ccol, most):
    """CSR B, rows of no entry to thousands beside each other, C in one slice and in several: lanes without an entry
    gather row 0 of C, which is NaN here and named by nobody; where C holds infinities, a row of D is infinite if it
    reads one of them through B, and its finite sum if not."""
    from gpu_util import Case
    n = 30011
    rng = np.random.default_rng(17)
    A = _hubs(n, dtype, rng, lambda k: rng.integers(1, 3, k))
    lens = rng.integers(0, most, n)
    lens[rng.permutation(n)[:16]] = [7, 8, 9, 15, 16, 17, 63, 64, 65, 127, 300, 511, 512, 513, 1500, 3000]
    lens[[0, n - 1]] = 257, 258
    rowptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    colidx = rng.integers(1, n, rowptr[-1]).astype(np.int32)
    B = ti.Csr(n, n, rowptr, colidx, rng.integers(1, 3, colidx.size).astype(dtype))
    C = rng.integers(1, 4, (n, ccol)).astype(dtype)
    hit = rng.random(n) < 0.002
    D_ref, _ = oracle.chain(A, B, np.where(hit[:, None], dtype(0), C))
    rows_of = lambda M, named: np.unique(np.repeat(np.arange(n), np.diff(M.rowptr))[named[M.colidx]])
    hit_d1 = np.zeros(n, bool)
    hit_d1[rows_of(B, hit)] = True
    D_ref[rows_of(A, hit_d1)] = np.inf
    C[hit] = np.inf
    C[0] = np.nan
    c = Case(ti.Problem("past", "spmm_spmm", np.dtype(dtype), A, B, C))
    try:
        assert np.isinf(D_ref).any() and np.isfinite(D_ref).any()
        for fused in (True, False):
            assert np.array_equal(c.run(fused).astype(np.float64), D_ref)
    finally:
        c.close()


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_static_calls_with_cut_rows_slices_and_padding(dtype):
    """The library's own workspace behind plans with rows cut over workgroups: three and more slices, rows padded to
    a line, and Y = A B over slices of B; one after the other, so that each finds what another plan left there."""
    import torch
    import paper_2407_00243_amd as tf
    from gpu_util import Case
    es = np.dtype(dtype).itemsize
    rng = np.random.default_rng(18)
    cases = []
    try:
        for bcol, ccol, execution in ((128, 288 // es, tf.TF_EXECUTE_WAVEFRONTS), (128, 164 // es, tf.TF_EXECUTE_WAVEFRONTS),
                                      (128, 92 // es, tf.TF_EXECUTE_WAVEFRONTS), (256 // es, 512 // es, tf.TF_EXECUTE_GATHER_FIRST)):
            n = max(60013, 14000000 // (ccol * es))         # (rows that reach beyond an L2)
            A = _hubs(n, dtype, rng, lambda k: rng.integers(-2, 3, k))
            B, C = ti.dense_small_int(n, bcol, dtype, 5), ti.dense_small_int(bcol, ccol, dtype, 6)
            c = Case(ti.Problem("static", "gemm_spmm", np.dtype(dtype), A, B, C))
            cases.append((c, oracle.chain(A, B, C)[0]))
            s = c.plan.schedule()
            assert s["far_rows"] and s["execution"] == execution
            if execution == tf.TF_EXECUTE_WAVEFRONTS:
                assert s["d1_slices"] * s["d1_slice_cols"] > ccol
        stream = torch.cuda.current_stream().cuda_stream
        for _ in range(2):
            for c, D_ref in cases:
                D = torch.full(D_ref.shape, float("nan"), dtype=c.tdtype, device="cuda")
                tf.tf_gemm_spmm_static(c.plan.handle, c.B, c.C, D, stream)
                torch.cuda.synchronize()
                assert np.array_equal(D.cpu().numpy().astype(np.float64), D_ref)
    finally:
        for c, _ in cases:
            c.close()
