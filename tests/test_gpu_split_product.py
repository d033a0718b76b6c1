"""fp32 products on the bf16 matrix cores (k_gemm_split, k_gather_gemm): operands split in three."""
import numpy as np
import pytest

import tf_inputs as ti

pytestmark = pytest.mark.gpu


def _products(B, C, how):
    """B C through the unfused product (A = 1), through the one-pass chain (A = 1; C as it is or transposed), or through a
    first wavefront that streams: rows of D that take one row of D1 as it is, from the registers (the first half) or
    from the workspace (the others, which lie in another tile)."""
    import paper_2407_00243_amd as tf
    from gpu_util import Case
    n = B.shape[0]
    cols = np.arange(n)
    if how == "streaming":
        cols[n // 2:] = np.roll(cols[n // 2:], n // 4)
    A = ti.Csr(n, n, np.arange(n + 1, dtype=np.int32), cols.astype(np.int32), np.ones(n, np.float32))
    params = dict(streaming=dict(ct_size=16, p=1), transposed=dict(flags=tf.TF_FLAG_C_TRANSPOSED)).get(how, {})
    c = Case(ti.Problem("product", "gemm_spmm", np.dtype(np.float32), A, B, C.T.copy() if how == "transposed" else C), **params)
    try:
        s = c.plan.schedule()
        if how == "streaming":
            assert s["first_wavefront_streams"]
        if how in ("one_pass", "transposed"):
            assert s["execution"] == tf.TF_EXECUTE_ONE_PASS
        return c.run(fused=how != "unfused"), cols
    finally:
        c.close()


@pytest.mark.parametrize("n,how", [(33, "unfused"), (32768, "unfused"), (32785, "unfused"), (70001, "unfused"),
                                   (32767, "streaming"), (32799, "streaming"), (70001, "streaming"), (17, "one_pass"),
                                   (4097, "one_pass"), (70001, "one_pass"), (4097, "transposed")])
@pytest.mark.parametrize("bcol,ccol", [(4, 1), (15, 32), (16, 32), (17, 33), (31, 41), (32, 31), (33, 48), (64, 96), (65, 33), (96, 50), (100, 100),
                                       (127, 128), (128, 64), (128, 130), (52, 16), (90, 7), (128, 17)])
def test_products_are_closer_than_sums_rounded_at_every_product(bcol, ccol, n, how):
    """Against 64 bits.  The six products of the parts are exact and what is left out is below 2^-26 of a product; with a
    rounding of 2^-24 at each of bcol products the norm of the error stays within 2^-24 sqrt(bcol) of the norm of the
    terms, and so within that of the result (the terms are independent); no element errs by more than bcol of them."""
    if how in ("one_pass", "transposed") and ccol < 4:
        ccol = 4                                  # (narrower rows of D take two wavefronts)
    rng = np.random.default_rng(bcol + n)
    B, C = rng.standard_normal((n, bcol), dtype=np.float32), rng.standard_normal((bcol, ccol), dtype=np.float32)
    got, cols = _products(B, C, how)
    want = (B.astype(np.float64) @ C.astype(np.float64))[cols]
    W = (np.abs(B).astype(np.float64) @ np.abs(C).astype(np.float64))[cols]
    assert np.all(np.abs(got - want) <= bcol * 2.0 ** -24 * W)
    if n > 1000:
        assert np.linalg.norm(got - want) <= 2.0 ** -24 * np.sqrt(bcol) * np.linalg.norm(want)


@pytest.mark.parametrize("n,bcol,ccol", [(699100, 32, 32), (381401, 64, 48), (300001, 96, 64), (214001, 128, 90)])
@pytest.mark.parametrize("how", ["unfused", "streaming"])
def test_rows_that_pass_through_the_cache(n, bcol, ccol, how):
    """Products whose operands and results are more than 256 MiB read rows of B of whole lines past the caches; the bound of
    above.  (On the host 1 in 16 rows.)"""
    rng = np.random.default_rng(n)
    B, C = rng.standard_normal((n, bcol), dtype=np.float32), rng.standard_normal((bcol, ccol), dtype=np.float32)
    got, cols = _products(B, C, how)
    got, B = got[5::16], B[cols[5::16]]
    W = np.abs(B).astype(np.float64) @ np.abs(C).astype(np.float64)
    assert np.all(np.abs(got - B.astype(np.float64) @ C.astype(np.float64)) <= bcol * 2.0 ** -24 * W)


@pytest.mark.parametrize("how", ["unfused", "streaming", "one_pass", "transposed"])
@pytest.mark.parametrize("bcol,ccol", [(20, 32), (32, 40), (50, 33), (128, 96)])
@pytest.mark.parametrize("where", ["B", "C"])
def test_numbers_that_the_parts_do_not_hold(bcol, ccol, where, how):
    """Rows of B, or columns of C, of infinities, NaN, numbers near the ends of the type's range and below it, and of these
    among ordinary ones: results as 64 bits give them, infinities and NaN where they belong, to the precision of
    above, and of the smallest normal number for each product."""
    n = 40100 if how in ("unfused", "streaming") else 4100
    rng = np.random.default_rng(bcol)
    B, C = rng.standard_normal((n, bcol), dtype=np.float32), rng.standard_normal((bcol, ccol), dtype=np.float32)
    part = B[100:1100:7] if where == "B" else C.T
    scales = [np.float32(x) for x in (1e-38, 1e-30, 1e-28, 1e-26, 1e-20, 1e-12, 1e17, 1e19, 1e30, 1e36)]
    for k in range(0, len(part), 2):
        if k % 3 == 0:
            part[k] *= scales[k // 2 % len(scales)]
        else:
            part[k, k % bcol] = (np.inf, -np.inf, np.nan, 1e36, 1e-36, 1e-42, 0.0)[k // 2 % 7]
    part[1] = 0
    got, cols = _products(B, C, how)
    with np.errstate(invalid="ignore"):
        want = (B.astype(np.float64) @ C.astype(np.float64))[cols]
        W = (np.abs(B).astype(np.float64) @ np.abs(C).astype(np.float64))[cols]
    assert np.array_equal(np.isnan(got), np.isnan(want))
    inf = np.isinf(want)
    assert np.array_equal(got[inf], want[inf])
    ok = np.isfinite(want)
    assert ok.any() and np.all(np.abs(got[ok] - want[ok]) <= bcol * (2.0 ** -24 * W[ok] + 2.0 ** -126))


@pytest.mark.parametrize("how", ["unfused", "one_pass"])
@pytest.mark.parametrize("row_exp,col_exp", [(-90, 0), (-89, -4), (-47, -47), (-48, -47), (-4, -90), (0, -91), (-91, 0), (59, 59), (60, 0),
                                             (0, 60), (36, 36), (35, 36), (59, 11), (59, 12), (59, 13), (11, 59), (13, 59), (-126, 59), (59, -126)])
def test_operands_at_the_bounds_of_the_split(row_exp, col_exp, how):
    """Every row of B and column of C of one magnitude, at and on either side of where the parts cease to hold them."""
    n, bcol, ccol = (40000, 64, 48) if how == "unfused" else (4100, 64, 48)
    rng = np.random.default_rng(7)
    B = (np.ldexp(rng.uniform(0.5, 1.99, (n, bcol)), row_exp) * rng.choice([-1, 1], (n, bcol))).astype(np.float32)
    C = (np.ldexp(rng.uniform(0.5, 1.99, (bcol, ccol)), col_exp) * rng.choice([-1, 1], (bcol, ccol))).astype(np.float32)
    got, _ = _products(B, C, how)
    want = B.astype(np.float64) @ C.astype(np.float64)
    W = np.abs(B).astype(np.float64) @ np.abs(C).astype(np.float64)
    assert np.all(np.abs(got - want) <= bcol * (2.0 ** -24 * W + 2.0 ** -126))
    if row_exp + col_exp > -100:
        assert np.linalg.norm(got - want) <= 2.0 ** -24 * np.sqrt(bcol) * np.linalg.norm(want)


@pytest.mark.parametrize("bcol,ccol", [(128, 144), (128, 160), (128, 200), (96, 250), (64, 400), (52, 447)])
@pytest.mark.parametrize("n", [500, 30000])
def test_wide_products_in_several_workgroups(bcol, ccol, n):
    """The one-pass chain where C in three parts is more than the LDS of a workgroup holds, or nearly so."""
    rng = np.random.default_rng(ccol)
    B, C = rng.standard_normal((n, bcol), dtype=np.float32), rng.standard_normal((bcol, ccol), dtype=np.float32)
    got, _ = _products(B, C, "one_pass")
    W = np.abs(B).astype(np.float64) @ np.abs(C).astype(np.float64)
    assert np.all(np.abs(got - B.astype(np.float64) @ C.astype(np.float64)) <= bcol * 2.0 ** -24 * W)


@pytest.mark.parametrize("how", ["unfused", "streaming", "one_pass", "transposed"])
@pytest.mark.parametrize("bcol,ccol", [(32, 40), (64, 33), (128, 96)])
@pytest.mark.parametrize("b_exp,c_exp", [(-112, 58), (-120, 50), (-60, -60), (-126, 35), (-140, 34), (-20, -105), (34, -140), (-47, -78), (-126, 100)])
def test_small_elements_whose_row_and_column_have_large_ones_elsewhere(bcol, ccol, b_exp, c_exp, how):
    """The largest element of a row of B meets a zero of C and the largest of a column of C a zero of B, so that a result is
    one product of small elements: within 2^-24 for its rounding, 2^-24 for what the six products of parts leave out and
    2^-28 for sums of small parts, to the spacing of the type's smallest numbers."""
    n = 40100 if how in ("unfused", "streaming") else 4100
    rng = np.random.default_rng(bcol)
    B, C = np.zeros((n, bcol), np.float32), np.zeros((bcol, ccol), np.float32)
    B[:, 1], C[3, :] = 1.0, 1.0
    at = bcol - 1 - np.arange(n) % (bcol // 2)
    small = np.ldexp(rng.uniform(1, 2, n), b_exp) * rng.choice([-1, 1], n)
    B[np.arange(n), at] = small
    C[bcol // 2:] = np.ldexp(rng.uniform(1, 2, (bcol - bcol // 2, ccol)), c_exp)
    got, cols = _products(B, C, how)
    want = (B[np.arange(n), at].astype(np.float64)[:, None] * C[at].astype(np.float64))[cols]
    assert np.all(np.abs(got - want) <= (2 + 2.0 ** -4) * 2.0 ** -24 * np.abs(want) + 2.0 ** -149)


def _products_rounded_at_every_one(B, C):
    """B C by the fp32 instructions, which products of few rows take (the oracle of how close sums rounded at every product are)."""
    return np.concatenate([_products(B[i:i + 16000], C, "unfused")[0] for i in range(0, len(B), 16000)])


@pytest.mark.parametrize("how", ["unfused", "one_pass"])
@pytest.mark.parametrize("bcol,ccol", [(64, 48), (128, 64)])
@pytest.mark.parametrize("positive", [False, True])
@pytest.mark.parametrize("terms", [1, 2, 3, 4, 8, 16, 32, 64])
def test_no_further_off_than_sums_rounded_at_every_product(bcol, ccol, terms, positive, how):
    """Rows of B of few to 64 numbers that are not zeros, against 64 bits: the error of the split product in the
    2-norm is at most that of the fp32 instructions on the same operands (to 1 %: over 2 million results the norms' own
    deviation is 0.1 %)."""
    n = 40000
    rng = np.random.default_rng(bcol + terms)
    B = np.zeros((n, bcol), np.float32)
    at = np.argsort(rng.random((n, bcol)), axis=1)[:, :terms]
    np.put_along_axis(B, at, rng.standard_normal((n, terms), dtype=np.float32), axis=1)
    C = rng.standard_normal((bcol, ccol), dtype=np.float32)
    if positive:
        B, C = np.abs(B), np.abs(C)
    got = _products(B, C, how)[0]
    want = B.astype(np.float64) @ C.astype(np.float64)
    err, other = np.linalg.norm(got - want), np.linalg.norm(_products_rounded_at_every_one(B, C) - want)
    assert err <= 1.01 * other, f"{err / np.linalg.norm(want):.3e}, by the fp32 instructions {other / np.linalg.norm(want):.3e}"


@pytest.mark.parametrize("how", ["unfused", "one_pass"])
@pytest.mark.parametrize("bcol,ccol", [(64, 48), (128, 64)])
def test_single_products_are_rounded_once(bcol, ccol, how):
    """One product a result, among them 0x1.00ff8p0 squared, of which m l and l m make up 2^-24: within 2^-24 of it for its
    rounding, and 2^-24 of that for sums of small parts that are cut off (112 of them at 2^-32 and less)."""
    n = 40000
    rng = np.random.default_rng(bcol)
    B, C = np.zeros((n, bcol), np.float32), rng.uniform(1, 2, (bcol, ccol)).astype(np.float32)
    at = np.arange(n) % bcol
    B[np.arange(n), at] = rng.uniform(1, 2, n)
    B[: n // 2, :][np.arange(n // 2), at[: n // 2]] = float.fromhex("0x1.00ff8p0")
    C[:, ::2] = float.fromhex("0x1.00ff8p0")
    got = _products(B, C, how)[0]
    want = B[np.arange(n), at].astype(np.float64)[:, None] * C[at].astype(np.float64)
    assert np.all(np.abs(got - want) <= 2.0 ** -24 * want * (1 + 112 * 2.0 ** -8))
