"""Right-hand sides and fields that are not finite, or whose norms overflow: every solve reports that it did
not converge, whatever the solver, the preconditioner and the system's size (4^3: one launch, 12^3: many)."""
import numpy as np
import pytest

import qh_inputs as qi

from .gpu_setup import gpu_context

pytestmark = pytest.mark.gpu


def _context(n, learned=False):
    ctx = gpu_context(qi.BoxMesh(n), 10 * 7.68e-10 / n)
    if learned:
        ctx.precond_train(steps=5, lr=3e-3, seed=1, validate_every=0)
    return ctx


def _configs():
    import paper_2103_06737_amd as qh
    return [(pc, sv) for pc in (qh.PC_JACOBI, qh.PC_LEARNED) for sv in (qh.SOLVER_FP64, qh.SOLVER_MIXED)]


@pytest.mark.parametrize("n", [4, 12])
@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan, 1e160])
def test_solve_of_nonfinite_rhs_is_refused(n, bad):
    import paper_2103_06737_amd as qh
    ctx = _context(n, True)
    rhs = np.random.default_rng(n).standard_normal(ctx.mesh_info().n_int_edges)
    good = rhs.copy()
    rhs[rhs.size // 2] = bad
    for pc, sv in _configs():
        with pytest.raises(qh.QhError) as e:
            ctx.field_solve(qh.SYS_EDGE, rhs, precond=pc, solver=sv)
        assert e.value.code == qh.QH_ENOTCONV
        x, st = ctx.field_solve(qh.SYS_EDGE, good, precond=pc, solver=sv)  # and leaves nothing behind
        assert st["res"] <= 1e-8 and np.isfinite(x).all()
    ctx.close()


@pytest.mark.parametrize("n", [4, 12])
def test_step_on_overflowing_fields_is_reported(n):
    """e of 1e170 V (right-hand sides of 1e158: eps0 is in the matrices): the squares of the residual and
    of its target overflow both."""
    import paper_2103_06737_amd as qh
    ctx = _context(n, True)
    mi = ctx.mesh_info()
    e = 1e170 * np.random.default_rng(n).standard_normal(mi.n_edges)
    for pc, sv in _configs():
        ctx.fields_upload(e, np.zeros(mi.n_faces, np.int64))
        with pytest.raises(qh.QhError) as ex:
            ctx.pic_step(ctx.step_params(field_mode=qh.FIELDS_SOLVE, precond=pc, solver=sv, gauss=0), 1)
        assert ex.value.code == qh.QH_ENOTCONV
    ctx.close()


@pytest.mark.parametrize("n", [4, 12])
def test_gauss_correction_of_overflowing_divergence_is_reported(n):
    """e = grad phi of 1e170 V: curl-free, so the edge solve starts at its solution to rounding (r0 of 1e142
    V, finite), but the squares of the divergence and of its target overflow: the correction cannot be
    solved, and the step says so. e stays what the edge solve gave."""
    import paper_2103_06737_amd as qh
    ctx = _context(n, True)
    mi = ctx.mesh_info()
    top = ctx.topology()
    phi = 1e170 * np.random.default_rng(n).standard_normal(mi.n_nodes)
    phi[top["wall_node"].astype(bool)] = 0.0
    e = phi[top["edges"][:, 1]] - phi[top["edges"][:, 0]]
    for pc, sv in _configs():
        ctx.fields_upload(e, np.zeros(mi.n_faces, np.int64))
        with pytest.raises(qh.QhError) as ex:
            ctx.pic_step(ctx.step_params(field_mode=qh.FIELDS_SOLVE, precond=pc, solver=sv), 1)
        assert ex.value.code == qh.QH_ENOTCONV
        assert np.array_equal(ctx.fields_download()[0], e)
    ctx.close()
