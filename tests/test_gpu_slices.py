"""The sliced products at their edges: fewer rows than one slice of 64, one row past a slice,
several slices with a remainder, one slice per wave and more; systems with PEC and natural walls,
compact and wide columns (the 24^3 box numbered at random in test_gpu_parity.py)."""
import numpy as np
import pytest

import qh_inputs as qi
from oracle.complex_ import Complex
from oracle.whitney import Operators

pytestmark = pytest.mark.gpu


def systems(mesh, dt, natural):
    cx = Complex(mesh.xyz, mesh.tets)
    op = Operators(cx, qi.EPS0, qi.MU0)
    ie = np.arange(cx.Ne) if natural else cx.int_edges
    A = (op.Meps + dt * dt / 4 * op.S)[ie][:, ie].tocsr()
    return A


# interior edges 26, 117, 316, 1981, 9519 with PEC walls; every edge (98, 1115) with natural ones; and
# 2293 slices (146,692 edges), past the 2048 with one width for all: rounds of several lengths
@pytest.mark.parametrize("n,natural", [(2, False), (3, False), (4, False), (7, False), (12, False), (2, True), (5, True),
                                       (28, False)])
def test_edge_solves_and_application(n, natural):
    import paper_2103_06737_amd as qh
    mesh = qi.BoxMesh(n)
    dt = 10 * 7.68e-10 / n
    ctx = qh.Context(0)
    if natural:
        ctx.set_boundary(qh.BC_NEUMANN)
    ctx.mesh_upload(mesh.xyz, mesh.tets)
    ctx.set_physics(qi.EPS0, qi.MU0, dt, qi.QE * 2.0 ** -40, 2.0 ** -56)
    A = systems(mesh, dt, natural)
    assert A.shape[0] == ctx.info.n_int_edges
    rhs = A @ np.random.default_rng(n).standard_normal(A.shape[0])
    ctx.precond_train(steps=20, lr=3e-3, seed=1, validate_every=0)
    for pc in (qh.PC_JACOBI, qh.PC_LEARNED):
        for solver in (qh.SOLVER_FP64, qh.SOLVER_MIXED):
            x, st = ctx.field_solve(qh.SYS_EDGE, rhs, tol=1e-10, precond=pc, solver=solver)
            # the solver's own FP64 matrix agrees with the oracle's to rounding: 1e-13 of the terms
            assert np.linalg.norm(A @ x - rhs) <= 1e-10 * np.linalg.norm(rhs) + 1e-13 * np.linalg.norm(abs(A) @ abs(x))
    # z = G^T (G r) against the factor as returned, rounded to BF16 as the application holds it:
    # FP64 sums of at most 64 terms per row in each pass
    import scipy.sparse as sp
    gr, gc, gv = ctx.precond_factor()
    u = gv.view(np.uint32).astype(np.uint64)
    h = ((u + 0x7fff + ((u >> 16) & 1)) & 0xffff0000).astype(np.uint32).view(np.float32)
    G = sp.csr_matrix((h.astype(np.float64), (gr, gc)), shape=A.shape)
    r = np.random.default_rng(n + 1).standard_normal(A.shape[0])
    z = ctx.precond_apply(r)
    assert (abs(z - G.T @ (G @ r)) <= 128 * 2.0 ** -53 * (abs(G).T @ (abs(G) @ abs(r)))).all()
    ctx.close()


@pytest.mark.parametrize("n", [2, 3, 5, 6, 9])  # interior nodes 1, 8, 64, 125, 512
def test_node_solve(n):
    import paper_2103_06737_amd as qh
    mesh = qi.BoxMesh(n)
    ctx = qh.Context(0)
    ctx.mesh_upload(mesh.xyz, mesh.tets)
    ctx.set_physics(qi.EPS0, qi.MU0, 1e-10, qi.QE * 2.0 ** -40, 2.0 ** -56)
    cx = Complex(mesh.xyz, mesh.tets)
    op = Operators(cx, qi.EPS0, qi.MU0)
    K = (cx.G.T @ op.Meps @ cx.G).tocsr()[cx.int_nodes][:, cx.int_nodes]
    rhs = K @ np.random.default_rng(n).standard_normal(K.shape[0])
    for solver in (qh.SOLVER_FP64, qh.SOLVER_MIXED):
        x, st = ctx.field_solve(qh.SYS_NODE, rhs, tol=1e-10, solver=solver)
        assert np.linalg.norm(K @ x - rhs) <= 1e-10 * np.linalg.norm(rhs) + 1e-13 * np.linalg.norm(abs(K) @ abs(x))
    ctx.close()


@pytest.mark.parametrize("n", [4, 7, 12])  # one launch with entries in registers, one launch, many launches
@pytest.mark.parametrize("learned", [False, True])
def test_iteration_cap_and_start_at_the_solution(n, learned):
    """A solve stops at its iteration cap with the iterate of that many steps (the residual it
    reports is that iterate's), takes none from a start that meets the target, and continues from
    a start to the same solution."""
    import paper_2103_06737_amd as qh
    mesh = qi.BoxMesh(n)
    dt = 10 * 7.68e-10 / n
    ctx = qh.Context(0)
    ctx.mesh_upload(mesh.xyz, mesh.tets)
    ctx.set_physics(qi.EPS0, qi.MU0, dt, qi.QE * 2.0 ** -40, 2.0 ** -56)
    A = systems(mesh, dt, False)
    rhs = A @ np.random.default_rng(n).standard_normal(A.shape[0])
    pc = qh.PC_LEARNED if learned else qh.PC_JACOBI
    if learned:
        ctx.precond_train(steps=20, lr=3e-3, seed=1, validate_every=0)
    for solver in (qh.SOLVER_FP64, qh.SOLVER_MIXED):
        if solver == qh.SOLVER_FP64 and not learned:  # (the others restart as FP64 Jacobi at their cap)
            x3, st = ctx.field_solve(qh.SYS_EDGE, rhs, tol=1e-10, max_it=3, precond=pc, solver=solver,
                                     allow=(qh.QH_ENOTCONV,))
            res = np.linalg.norm(A @ x3 - rhs) / np.linalg.norm(rhs)
            # the reported norm is of the same residual with the library's matrix: 1e-12 of rounding
            assert st["iters"] == 3 and abs(res - st["res"]) <= 1e-12 and st["res"] > 1e-10
        x, st = ctx.field_solve(qh.SYS_EDGE, rhs, tol=1e-10, precond=pc, solver=solver)
        assert st["iters"] > 3 and st["res"] <= 1e-10 and st["fallback"] == 0
        y, st0 = ctx.field_solve(qh.SYS_EDGE, rhs, x0=x, tol=2e-10, precond=pc, solver=solver)
        assert st0["iters"] == 0 and np.array_equal(x, y)
        # half way: fewer iterations from there, to the same target
        h, st1 = ctx.field_solve(qh.SYS_EDGE, rhs, tol=1e-5, precond=pc, solver=solver)
        z, st2 = ctx.field_solve(qh.SYS_EDGE, rhs, x0=h, tol=1e-10, precond=pc, solver=solver)
        assert 0 < st2["iters"] < st["iters"] and st2["res"] <= 1e-10
    ctx.close()
