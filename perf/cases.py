"""Performance cases: what a program does with this framework, through its public entry points.

Five kinds of work. `cycle` is one step of the full particle-in-cell cycle (push, deposit, implicit
field update) on a box; `beam` the same on the cylindrical cavity with absorbing walls, its
injection included; `push` one step in frozen fields (gather, push, walk, deposit); `solve` one
solve of the edge or the node system for a right-hand side on the host; `train` a few optimiser
steps of the learned preconditioner. Sizes, densities, time steps and tolerances are those of the
repository's workloads (qh_inputs.CONFIGS, BEAM_CYL), of its tests and its benchmark, or lie
between them.

A step returns the state it updates. In frozen fields the deposits come as the integers they are.
In a cycle the fields and the next step's deposits follow an iterative solve that stops at its
tolerance (1e-8, the benchmark's), so they come in SI units in single precision (6e-8), which
holds the digits the tolerance does; b, g and Q are integer multiples of the units u_b and u_q.
Stand-alone solves go to 1e-12 and return the solution in double precision.
"""
import math

import numpy as np
import torch  # before the library, which then shares its HIP runtime

import paper_2103_06737_amd as qh
import qh_inputs as qi

U_B = 2.0 ** -56
DT_CFL = 7.68e-10  # explicit limit x n of the uniform n^3 box (the lattice is self-similar)


def listed():
    return [
        # smallest step a program takes: the jittered 4^3 cube of the tests, latency alone
        dict(name="cycle_box4_1k", kind="cycle", n=4, jitter=0.1, electrons=1000, ions=False, mode="solve",
             solver="fp64", precond="jacobi", natural=False, dt_mult=0.05, density=1e3, tol=1e-8),
        # the beam of the paper's table: 90,000 tets, 60,000 particles in flight, 10 injected per step
        dict(name="beam_cylinder_60k", kind="beam", nr=10, nz=50, in_flight=60000, tol=1e-6),
        # the 32^3 beam workload: 1M electrons in frozen random fields
        dict(name="push_beam32_1m", kind="push", n=32, electrons=1_000_000, load="beam", dt=1e-11),
        # thermal plasma in a frozen field at the benchmark's time step, density per box and sort
        # interval: many face crossings, particles drifting away from the last sort
        dict(name="push_plasma40_4m", kind="push", n=40, electrons=3_906_250, load="uniform", dt=1.92e-10),
        # two species on a graded box of odd size, mixed-precision Jacobi solve
        dict(name="cycle_graded25_2x400k", kind="cycle", n=25, z_ratio=1.05, electrons=400_000, ions=True,
             mode="solve", solver="mixed", precond="jacobi", natural=False, dt_mult=8.0, density=1e14, tol=1e-8),
        # natural walls with a plane-wave pulse, wave-equation update, FP64 Jacobi solve
        dict(name="cycle_wave21_plane_150k", kind="cycle", n=21, electrons=150_000, ions=False, mode="wave",
             solver="fp64", precond="jacobi", natural=True, dt_mult=10.0, density=1e13, tol=1e-8),
        # middle of the range with the learned preconditioner and the FP64 solve
        dict(name="cycle_plasma16_250k", kind="cycle", n=16, electrons=250_000, ions=False, mode="solve",
             solver="fp64", precond="learned", natural=False, dt_mult=10.0, density=1e14, tol=1e-8),
        # the benchmark's cycle (learned preconditioner, mixed-precision solve, its density per
        # box) at 48^3: the largest step here
        dict(name="cycle_plasma48_6.75m", kind="cycle", n=48, electrons=6_750_000, ions=False, mode="solve",
             solver="mixed", precond="learned", natural=False, dt_mult=10.0, density=1e16, tol=1e-8),
        # the benchmark's edge system (64^3: 1.8M unknowns, 29M nonzeros), its default solver
        dict(name="edge64_learned_mixed", kind="solve", n=64, system="edge", solver="mixed", precond="learned"),
        # a smaller one of odd size with the plain solver
        dict(name="edge33_jacobi_fp64", kind="solve", n=33, system="edge", solver="fp64", precond="jacobi"),
        # the Gauss-law (node) system of the same 64^3 mesh
        dict(name="node64_jacobi_fp64", kind="solve", n=64, system="node", solver="fp64", precond="jacobi"),
        # training of the preconditioner: forward, backward and Adam on the GPU
        dict(name="train_box24_4steps", kind="train", n=24, steps=4),
    ]


def draw(rng):
    """One more case of the same ranges."""
    def between(lo, hi):
        return math.exp(rng.uniform(math.log(lo), math.log(hi)))

    kind = rng.choice(["cycle", "cycle", "cycle", "push", "push", "beam", "solve", "solve", "train"])
    if kind == "beam":
        return dict(kind=kind, nr=rng.randint(4, 10), nz=rng.randint(20, 50), in_flight=int(between(3e3, 6e4)), tol=1e-6)
    if kind == "push":
        return dict(kind=kind, n=round(between(6, 40)), electrons=int(between(2e3, 3.9e6)),
                    load=rng.choice(["beam", "uniform"]), dt=between(1e-11, 5e-11))
    if kind == "train":
        return dict(kind=kind, n=round(between(6, 24)), steps=rng.randint(1, 4))
    if kind == "solve":
        system = rng.choice(["edge", "edge", "node"])
        learned = system == "edge" and rng.random() < 0.5
        return dict(kind=kind, n=round(between(4, 44)), system=system, solver=rng.choice(["fp64", "mixed"]),
                    precond="learned" if learned else "jacobi")
    n = round(between(4, 40))
    natural = rng.random() < 0.25
    learned = rng.random() < 0.5
    return dict(kind=kind, n=n, electrons=int(between(1000, 26 * n ** 3 + 2000)), ions=rng.random() < 0.3,
                mode=rng.choice(["solve", "solve", "wave"]), solver=rng.choice(["fp64", "mixed"]),
                precond="learned" if learned else "jacobi", natural=natural,
                z_ratio=rng.choice([1.0, 1.0, 1.03]), dt_mult=10.0 if learned else rng.uniform(1.0, 10.0),
                density=between(1e12, 1e14), tol=1e-8)


# ------------------------------------------------------------------------------- contexts

_kept = {}  # meshes and the network a program keeps, by what defines them


def _keep(key, make, most=6):
    if key not in _kept:
        while len(_kept) >= most:
            _kept.pop(next(iter(_kept)))
        _kept[key] = make()
    return _kept[key]


def _box(n, jitter=0.0, z_ratio=1.0):
    return _keep(("box", n, jitter, z_ratio), lambda: qi.BoxMesh(n, 1.0, jitter=jitter, z_ratio=z_ratio))


def _network():
    """A network trained once on a 16^3 box at ten times the explicit limit, as a blob."""
    def make():
        ctx = qh.Context(0)
        mesh = qi.BoxMesh(16)
        ctx.mesh_upload(mesh.xyz, mesh.tets)
        ctx.set_physics(qi.EPS0, qi.MU0, 10.0 * DT_CFL / 16, qi.QE * 2.0 ** -40, U_B)
        ctx.precond_train(steps=150, lr=3e-3, seed=1, validate_every=0)
        return ctx.precond_save()
    return _keep(("network",), make)


def _context(mesh, dt, weight, natural=False, absorb=False):
    ctx = qh.Context(0)
    if natural:
        ctx.set_boundary(qh.BC_NEUMANN)
    if absorb:
        ctx.set_walls(qh.WALLS_ABSORB)
    ctx.mesh_upload(mesh.xyz, mesh.tets)
    ctx.set_physics(qi.EPS0, qi.MU0, dt, qi.QE * weight * 2.0 ** -40, U_B)
    return ctx


class _State:
    """A context and the buffers its outputs go to."""

    def __init__(self, ctx, prm, weight, case):
        mi = ctx.mesh_info()
        self.ctx, self.prm, self.case = ctx, prm, case
        self.u_q = qi.QE * weight * 2.0 ** -40
        self.e = torch.empty(mi.n_edges, dtype=torch.float64, device="cuda")
        self.b = torch.empty(mi.n_faces, dtype=torch.int64, device="cuda")
        self.g = torch.empty(mi.n_edges, dtype=torch.int64, device="cuda")
        self.q = torch.empty(mi.n_nodes, dtype=torch.int64, device="cuda")
        self.inject, self.at = [], 0

    def deposits(self):
        self.ctx.deposits_download_dev(self.g.data_ptr(), self.q.data_ptr())
        return self.g, self.q

    def fields(self):
        self.ctx.fields_download_dev(self.e.data_ptr(), self.b.data_ptr())
        return self.e, self.b


def _solver(case):
    return (qh.SOLVER_MIXED if case["solver"] == "mixed" else qh.SOLVER_FP64,
            qh.PC_LEARNED if case["precond"] == "learned" else qh.PC_JACOBI)


def _prepare_cycle(case, seed):
    n, ne = case["n"], case["electrons"]
    mesh = _box(n, case.get("jitter", 0.0), case.get("z_ratio", 1.0))
    weight = case["density"] / ne
    dt = case["dt_mult"] * DT_CFL / n
    solver, precond = _solver(case)
    ctx = _context(mesh, dt, weight, natural=case["natural"])
    mi = ctx.mesh_info()
    # thermal start: a weak random E beside the uniform B_z (none inside natural walls, where it
    # is no equilibrium and the pulse drives the fields)
    ctx.fields_init_synthetic(qi.white(mi.n_edges, seed, 3), qi.white(mi.n_edges, seed, 5), 1e2,
                              0.0 if case["natural"] else 0.1, 0.0)
    cfg = dict(n_e=ne, n_i=ne if case["ions"] else 0, v_th_e=1e6, v_th_i=2e4)
    for name, (x, v, tet) in qi.make_particles(mesh, cfg, seed=seed).items():
        qm, z = (-qi.QE / qi.ME, -1) if name == "e" else (qi.QE / qi.MI, 1)
        ctx.particles_upload(ctx.species_add(qm, z), x, v, tet)
    ctx.charge_background(1)
    if case["natural"]:
        ctx.set_plane_wave(1e3 / (2 * math.pi * 300e6), 300e6, 150e6, 4.0 / (2 * math.pi * 150e6))
    if precond == qh.PC_LEARNED:
        ctx.precond_load(_network())
    prm = qh.Context.step_params(field_mode=qh.FIELDS_WAVE if case["mode"] == "wave" else qh.FIELDS_SOLVE,
                                 sort_every=20, precond=precond, tol_edge=case["tol"], tol_node=1e-8,
                                 check_every=16, solver=solver)
    return _State(ctx, prm, weight, case)


def _prepare_beam(case, seed):
    c = qi.BEAM_CYL
    mesh = _keep(("cylinder", case["nr"], case["nz"]), lambda: qi.CylinderMesh(c["R"], c["L"], case["nr"], case["nz"]))
    ctx = _context(mesh, c["dt"], c["weight"], absorb=True)
    mi = ctx.mesh_info()
    ctx.fields_upload(np.zeros(mi.n_edges), np.zeros(mi.n_faces, np.int64))
    sid = ctx.species_add(-qi.QE / qi.ME, -1)
    # the beam in flight: uniform along the tube, inside the beam radius
    gen = qi.rng(seed, 40)
    k = case["in_flight"]
    r, phi = c["r_b"] * np.sqrt(gen.random(k)), 2.0 * np.pi * gen.random(k)
    x = np.stack([r * np.cos(phi), r * np.sin(phi), c["L"] * (0.001 + 0.998 * gen.random(k))], axis=1)
    v = np.zeros((k, 3), np.float32)
    v[:, 2] = c["v_p"]
    ctx.particles_upload(sid, x.astype(np.float32), v)
    prm = qh.Context.step_params(field_mode=qh.FIELDS_SOLVE, tol_edge=case["tol"], tol_node=1e-8, check_every=8)
    s = _State(ctx, prm, c["weight"], case)
    s.sid = sid
    s.inject = [qi.beam_injection(mesh, c["per_step"], c["r_b"], c["v_p"], seed=seed, step=j) for j in range(48)]
    return s


def _prepare_push(case, seed):
    mesh = _box(case["n"])
    ctx = _context(mesh, case["dt"], 1.0)
    mi = ctx.mesh_info()
    beam = case["load"] == "beam"
    ctx.fields_init_synthetic(qi.white(mi.n_edges, seed, 3), qi.white(mi.n_edges, seed, 5), 1e4 if beam else 0.0, 0.1,
                              1e-3 if beam else 0.0)
    cfg = dict(n_e=case["electrons"], n_i=0, v_th_e=1e5 if beam else 1e6, load=case["load"], beam_sigma=0.1,
               drift_z=1e7)
    x, v, tet = qi.make_particles(mesh, cfg, seed=seed)["e"]
    ctx.particles_upload(ctx.species_add(-qi.QE / qi.ME, -1), x, v, tet)
    prm = qh.Context.step_params(field_mode=qh.FIELDS_FROZEN, sort_every=20)
    return _State(ctx, prm, 1.0, case)


def _handle(n, learned):
    """The assembled systems of an n^3 box, kept by a program that solves for many right-hand sides."""
    def make():
        mesh = qi.BoxMesh(n)
        return _context(mesh, 10.0 * DT_CFL / n, 1.0)
    ctx = _keep(("handle", n), make)
    if learned and not getattr(ctx, "network_loaded", False):
        ctx.precond_load(_network())
        ctx.network_loaded = True
    return ctx


def _solution(case, seed):
    n, edge = case["n"], case["system"] == "edge"
    count = 7 * n ** 3 - 9 * n ** 2 + 3 * n if edge else (n - 1) ** 3  # interior edges or nodes of the box
    return np.random.Generator(np.random.PCG64([seed, 77])).standard_normal(count)


def _prepare_solve(case, seed):
    edge = case["system"] == "edge"
    solver, precond = _solver(case)
    ctx = _handle(case["n"], precond == qh.PC_LEARNED)
    M = _keep(("matrix", case["n"], edge), lambda: ctx.matrix(0 if edge else 5))
    return dict(ctx=ctx, rhs=M @ _solution(case, seed), system=qh.SYS_EDGE if edge else qh.SYS_NODE, solver=solver,
                precond=precond)


def _prepare_train(case, seed):
    ctx = _context(_box(case["n"]), 10.0 * DT_CFL / case["n"], 1.0)
    ctx.precond_train(steps=0)  # sets the preconditioner up
    gen = qi.rng(seed, 50)
    w = np.concatenate([gen.standard_normal(64 * 16) * (2 / 16) ** 0.5, np.zeros(64),
                        gen.standard_normal(64 * 64) * (2 / 64) ** 0.5, np.zeros(64),
                        gen.standard_normal(64) * 0.02, np.zeros(1)]).astype(np.float32)
    return dict(ctx=ctx, w=w, seed=seed % 100003, steps=case["steps"])


def prepare(case, seed):
    return {"cycle": _prepare_cycle, "beam": _prepare_beam, "push": _prepare_push, "solve": _prepare_solve,
            "train": _prepare_train}[case["kind"]](case, int(seed))


# ------------------------------------------------------------------------------- one pass

def run(s):
    if isinstance(s, dict):
        ctx = s["ctx"]
        if "rhs" in s:
            x, _ = ctx.field_solve(s["system"], s["rhs"], tol=1e-12, max_it=20000, precond=s["precond"],
                                   solver=s["solver"])
            return {"x": x}
        ctx.precond_set_weights(s["w"])
        ctx.precond_train(steps=s["steps"], lr=3e-3, seed=s["seed"], validate_every=0)
        return {"weights": ctx.precond_get_weights()}
    if s.inject:
        s.ctx.particles_inject(s.sid, *s.inject[s.at % len(s.inject)])
        s.at += 1
    s.ctx.pic_step(s.prm, 1)
    g, q = s.deposits()
    if s.case["kind"] == "push":
        return {"g": g, "Q": q}
    e, b = s.fields()
    return {"e": e.float(), "b": b * U_B, "g": g * s.u_q, "Q": q * s.u_q}


# ------------------------------------------------------------------------------- what it takes

def _sizes(case):
    """(nodes, edges, faces, tets) of the case's mesh."""
    if case["kind"] == "beam":
        nr, nz = case["nr"], case["nz"]
        n2, tri = 1 + 3 * nr * (nr + 1), 6 * nr * nr
        e2 = n2 + tri - 1
        nn = n2 * (nz + 1)
        ne = e2 * (nz + 1) + n2 * nz + e2 * nz
        nt = 3 * tri * nz
        return nn, ne, nt + ne - nn + 1, nt
    n = case["n"]
    return (n + 1) ** 3, 7 * n ** 3 + 9 * n * n + 3 * n, 12 * n ** 3 + 6 * n * n, 6 * n ** 3


def work(case):
    """Each input read once and each output written once: particle state (28 B each way), mesh
    records (136 B per tet), deposits and fields, the systems' matrices (16 entries per edge, 15
    per node, a value and a 2-byte column) and vectors; one application of each matrix."""
    nn, ne, nf, nt = _sizes(case)
    kind = case["kind"]
    if kind == "solve":
        rows, per = (ne, 16) if case["system"] == "edge" else (nn, 15)
        v = 4 if case["solver"] == "mixed" else 8
        return dict(bytes=(v + 2) * per * rows + 16 * rows, flops=2 * per * rows)
    if kind == "train":
        entries = 8.5 * ne
        return dict(bytes=32 * entries, flops=case["steps"] * entries * 3.9e4)
    particles = case["in_flight"] if kind == "beam" else case["electrons"] * (2 if case.get("ions") else 1)
    byt = 56 * particles + 136 * nt + 8 * (ne + nn)
    flops = 150 * particles
    if kind != "push":
        byt += 10 * (16 * ne + 15 * nn + 14 * ne) + 16 * (ne + nf)
        flops += 2 * (16 * ne + 15 * nn + 14 * ne)
    return dict(bytes=byt, flops=flops)


def exact(case, seed):
    """A solve's right-hand side is made from its solution. A step (a push in single precision, a
    walk with exact integer deposits, an iterative field update) and training have no short
    64-bit form."""
    if case["kind"] != "solve":
        return None
    return {"x": _solution(case, int(seed))}
