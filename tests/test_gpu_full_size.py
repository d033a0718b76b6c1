"""Parity at the full benchmark sizes, in the launch configuration bench.py times: every row of D
of every configuration, fused and unfused, against the oracle's chain over all rows."""
import numpy as np
import pytest

import oracle
import tf_inputs as ti
from util import check_schedule, check_schedule_general

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cfg", [1, 2, 3, 4, 5])
def test_full_size_config(cfg):
    import bench
    import paper_2407_00243_amd as tf
    from gpu_util import Case, TOL
    print(f"config {cfg}: generating", flush=True)
    prob = ti.config(cfg)
    params = bench.tile_params(cfg)
    c = Case(prob, **params)
    try:
        s = c.plan.schedule()
        if params.get("flags", 0) & tf.TF_FLAG_REORDER or not params.get("ct_size"):
            check_schedule_general(prob.A, s)
        else:
            check_schedule(prob.A, s, params["ct_size"], params["p"])
        print(f"config {cfg}: oracle over all {prob.n} rows", flush=True)
        D_ref, W = oracle.chain(prob.A, prob.B, prob.C, parallel=True)
        lens = np.diff(prob.A.rowptr)
        tol = TOL[np.dtype(prob.dtype)]
        for fused in (True, False):
            print(f"config {cfg}: running fused={fused}", flush=True)
            D = c.run(fused=fused)
            assert np.all(np.isfinite(D)), "a row of D was not written"
            assert np.all(D[lens == 0] == 0)
            err = oracle.rowwise_rel_err(D, D_ref, W)
            print(f"config {cfg}: fused={fused} row-wise rel err {err:.2e} over all rows", flush=True)
            assert err <= tol, f"cfg{cfg} fused={fused}: {err:.3e} > {tol:.0e}"
    finally:
        c.close()


@pytest.mark.parametrize("cfg", [1, 2])
def test_full_size_config_in_two_wavefronts(cfg):
    """The configurations that the library runs in one pass, in the two wavefronts of its own tiling: every
    row of D, and the D1 rows that the first one leaves for the second."""
    import bench
    import paper_2407_00243_amd as tf
    from gpu_util import Case, TOL, read_workspace
    prob = ti.config(cfg)
    c = Case(prob, **bench.tile_params(cfg))
    try:
        s = c.plan.schedule()
        assert s["automatic"] == 1 and s["execution"] == tf.TF_EXECUTE_ONE_PASS and not s["first_wavefront_streams"]
        c.plan.workspace()
        D_ref, W = oracle.chain(prob.A, prob.B, prob.C, parallel=True)
        D = c.run()
        assert np.all(np.isfinite(D)), "a row of D was not written"
        tol = TOL[np.dtype(prob.dtype)]
        err = oracle.rowwise_rel_err(D, D_ref, W)
        assert err <= tol, f"cfg{cfg}: {err:.3e} > {tol:.0e}"
        eye = ti.Csr(prob.n, prob.n, np.arange(prob.n + 1, dtype=np.int32), np.arange(prob.n, dtype=np.int32),
                     np.ones(prob.n, prob.dtype))
        D1_ref, W1 = oracle.chain(eye, prob.B, prob.C, parallel=True)
        rows = np.flatnonzero(s["spill_slot"] >= 0)
        ws = read_workspace(c.plan, s, c.ccol, prob.dtype)
        err = oracle.rowwise_rel_err(ws[s["spill_slot"][rows]], D1_ref[rows], W1[rows])
        assert rows.size and err <= tol, f"cfg{cfg} D1: {err:.3e} > {tol:.0e}"
    finally:
        c.close()
