"""Iterations launched against iterations needed. A solve without a history launches its iterations in
batches, a read of the stop flag after each; a residual that falls little at first (smooth and local
right-hand sides) must not make it launch many times what is needed."""
import numpy as np
import pytest

import qh_inputs as qi

from .gpu_setup import gpu_context

pytestmark = pytest.mark.gpu


def _rhs(kind, M):
    if kind == "constant":
        return np.ones(M.shape[0])
    if kind == "point":
        u = np.zeros(M.shape[0])
        u[u.size // 2] = 1.0
        return u
    return M @ np.random.default_rng(1).standard_normal(M.shape[0])


# a batch is at most 8 or twice the iterations before it, so at most three times the need and 8 are
# launched; the node system of 20^3 with a constant right-hand side needs 60, edges at 40 times the
# explicit limit 650
@pytest.mark.parametrize("kind", ["constant", "point", "noise"])
@pytest.mark.parametrize("system,n,mult", [("node", 20, 10.0), ("node", 33, 10.0), ("edge", 14, 40.0)])
def test_fp64_solve_launches_what_it_needs(system, n, mult, kind):
    import paper_2103_06737_amd as qh
    ctx = gpu_context(qi.BoxMesh(n), mult * 7.68e-10 / n)
    node = system == "node"
    M = ctx.matrix(5 if node else 0)
    rhs = _rhs(kind, M)
    for tol in (1e-8, 1e-12):
        ctx.timing(True)
        x, st = ctx.field_solve(qh.SYS_NODE if node else qh.SYS_EDGE, rhs, tol=tol, max_it=20000)
        launched = ctx.timing_read()["cg_spmv"][1]
        ctx.timing(False)
        assert st["res"] <= tol and st["iters"] <= launched <= 3 * st["iters"] + 8, (launched, st)
    ctx.close()


# the same in mixed precision: a segment between reliable updates reduces the residual by 3e-5 at most
# (FP32 vectors hold no more), so a slow start followed by a fast end takes about the FP64 solve's
# iterations; twice as many would be a recurrence that has lost its directions
@pytest.mark.parametrize("kind", ["constant", "point", "noise"])
@pytest.mark.parametrize("system,n,mult", [("node", 20, 10.0), ("node", 33, 10.0), ("edge", 14, 40.0)])
def test_mixed_solve_keeps_its_segments(system, n, mult, kind):
    import paper_2103_06737_amd as qh
    ctx = gpu_context(qi.BoxMesh(n), mult * 7.68e-10 / n)
    node = system == "node"
    M = ctx.matrix(5 if node else 0)
    rhs, which = _rhs(kind, M), qh.SYS_NODE if node else qh.SYS_EDGE
    for tol in (1e-8, 1e-12):
        _, ref = ctx.field_solve(which, rhs, tol=tol, max_it=20000)
        ctx.timing(True)
        x, st = ctx.field_solve(which, rhs, tol=tol, max_it=20000, solver=qh.SOLVER_MIXED)
        launched = ctx.timing_read()["cg_spmv"][1]
        ctx.timing(False)
        assert st["res"] <= tol and st["fallback"] == 0 and st["iters"] <= 2 * ref["iters"], (st, ref)
        assert launched <= 3 * st["iters"] + 8, (launched, st)
    ctx.close()


def test_step_with_no_iterations_allowed():
    """A cap of zero or below: no iteration, whichever solver and size, and none is counted."""
    import paper_2103_06737_amd as qh
    for n in (4, 12):
        ctx = gpu_context(qi.BoxMesh(n), 10 * 7.68e-10 / n)
        mi = ctx.mesh_info()
        ctx.fields_init_synthetic(qi.white(mi.n_edges, 0, 3), qi.white(mi.n_edges, 0, 5), 1e2, 0.1, 0.0)
        for sv in (qh.SOLVER_FP64, qh.SOLVER_MIXED):
            for cap in (0, -5):
                p = ctx.step_params(field_mode=qh.FIELDS_SOLVE, solver=sv, gauss=0, max_it_edge=cap)
                st = ctx.pic_step(p, 1, allow=(qh.QH_ENOTCONV,))[0]
                assert st["edge_iters"] == 0, (n, sv, cap, st["edge_iters"])
        ctx.close()
