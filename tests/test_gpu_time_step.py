"""A context whose time step changes gives what a context created with that time step gives: the solves,
the field update, the preconditioner's factor, its training loss and gradient, bit for bit."""
import numpy as np
import pytest

import qh_inputs as qi

from .gpu_setup import gpu_context

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [4, 12])
@pytest.mark.parametrize("learned_before", [False, True])
def test_change_of_time_step(n, learned_before):
    import paper_2103_06737_amd as qh
    mesh = qi.BoxMesh(n, 1.0, jitter=0.1)
    dts = [7.68e-10 / n, 10 * 7.68e-10 / n, 3 * 7.68e-10 / n]
    changed = gpu_context(mesh, dts[0])
    mi = changed.mesh_info()
    rng = np.random.default_rng(n)
    rhs = rng.standard_normal(mi.n_int_edges) * 1e-12
    V = np.sign(rng.standard_normal((mi.n_int_edges, 16))).astype(np.float32)
    we, wa = qi.white(mi.n_edges, 0, 3), qi.white(mi.n_edges, 0, 5)
    w = (0.05 * rng.standard_normal(qh.MLP_NPARAM)).astype(np.float32)

    def outputs(ctx):
        out = [ctx.field_solve(qh.SYS_EDGE, rhs, precond=pc, solver=sv)[0]
               for pc in (qh.PC_JACOBI, qh.PC_LEARNED) for sv in (qh.SOLVER_FP64, qh.SOLVER_MIXED)]
        loss, grad = ctx.precond_loss_grad(V)
        ctx.fields_init_synthetic(we, wa, 1e2, 0.1, 1e-3)
        ctx.pic_step(ctx.step_params(field_mode=qh.FIELDS_SOLVE), 1)
        e, b = ctx.fields_download()
        return out + [ctx.precond_factor()[2], np.array([loss]), grad, e, b]

    if learned_before:
        changed.precond_set_weights(w)
        outputs(changed)
    for dt in dts[1:]:
        changed.set_physics(qi.EPS0, qi.MU0, dt, qi.QE * 2.0 ** -40, 2.0 ** -56)
        changed.precond_set_weights(w)
        fresh = gpu_context(mesh, dt)
        fresh.precond_set_weights(w)
        for k, (a, f) in enumerate(zip(outputs(changed), outputs(fresh))):
            assert np.array_equal(a, f), (dt, k)
        fresh.close()
    changed.close()
