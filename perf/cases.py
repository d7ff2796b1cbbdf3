"""Work that programs using this framework have it do, for timing and for checking results.

Every case goes through the public calls (``pipeline.NewtonStep``, ``NewtonSolver``, ``DirkStepper`` and the methods of
``hdg.Context``) at sizes of the repository's own workloads (``synth.config``, ``bench.py``, the tests) and between
them.  ``kind`` says which path a case takes:

* ``step``      one whole Newton step (element systems, condensation, assembly, Schwarz set-up, GMRES, recovery);
* ``dirk``      one three-stage DIRK time step with lagged artificial viscosity and the reduced-basis guess: the
                Newton driver's own loop, with its residual norms and host decisions;
* ``condense``  element systems, condensation and assembly as separate calls, with resident or streamed systems;
* ``residual``  element systems and the nonlinear residual norm (the convergence check of each Newton iteration);
* ``matvec``    the trace operator applied to one vector;
* ``schwarz``   set-up of the Schwarz preconditioner and one application;
* ``gmres``     one GMRES cycle on a given trace system.

``p`` is a degree, or several separated by commas (drawn per element with a fixed seed).
"""
import dataclasses
import functools
import math

import numpy as np
import torch

from paper_2608_27863_amd import hdg, pipeline, synth

PREC = {"fp64": hdg.HDG_FP64, "mixed": hdg.HDG_MIXED}
AV = dict(c_av=2e-3, eps=1e-10, s_max=math.inf, rho_min=1e-8, p_min=1e-8, smooth_iters=2)
F64 = torch.float64


def _case(name, kind, n, p, **more):
    c = dict(kind=kind, nx=n[0], ny=n[1], nz=n[2], p=str(p), walls=False, prec="fp64", schwarz="fp64", m=30, chunk=0)
    c.update(more)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the large partition at p = 4 (FP64 condensation in chunks of 256, FP32 Schwarz inverses, GMRES(50))
        _case("step-p4", "step", (8, 8, 8), 4, schwarz="mixed", m=50, chunk=256),
        # the mixed-precision step on the 8^3 p = 3 mesh
        _case("step-p3-mixed", "step", (8, 8, 8), 3, prec="mixed", schwarz="mixed"),
        # the small FP64 parity mesh: a step of a few milliseconds, launches count
        _case("step-p2", "step", (4, 4, 4), 2),
        # the smallest step: latency only
        _case("step-p1", "step", (2, 2, 2), 1, m=10),
        # one implicit time step of a small run: about ten Newton iterations and the driver around them
        _case("dirk-p2", "dirk", (3, 3, 3), 2, m=40),
        # uneven degrees on a walled box, elements numbered by degree
        _case("condense-degrees", "condense", (8, 5, 5), "2,3,4", walls=True),
        # streamed element systems at p = 4, mixed precision, a ragged last chunk
        _case("condense-p4-streamed", "condense", (5, 5, 4), 4, prec="mixed", chunk=48, stream=True),
        # many low-order elements
        _case("condense-p1", "condense", (12, 12, 12), 1),
        # the residual evaluation of a Newton iteration
        _case("residual-p3", "residual", (9, 7, 8), 3),
        # the operator application inside GMRES, at the large partition's size
        _case("matvec-p4", "matvec", (12, 12, 12), 4),
        # preconditioner set-up and application in FP64
        _case("schwarz-p3", "schwarz", (8, 8, 8), 3),
        # a GMRES cycle on a mid-sized system with FP32 preconditioner blocks
        _case("gmres-p2", "gmres", (10, 10, 10), 2, schwarz="mixed"),
    ]


def draw(rng):
    kind = rng.choice(["step", "condense", "condense", "residual", "matvec", "schwarz", "gmres", "dirk"])
    p = rng.choice(["1", "2", "3", "4", "2,3,4", "1,3"])
    if kind == "dirk":
        p = rng.choice(["1", "2"])
    top = max(int(v) for v in p.split(","))
    # elements: spread over the logarithm, up to what the largest listed case of that kind costs
    most = {"step": {1: 2000, 2: 1200, 3: 512, 4: 200}, "condense": {1: 3000, 2: 1000, 3: 400, 4: 120},
            "residual": {1: 3000, 2: 1500, 3: 500, 4: 120}, "matvec": {1: 4000, 2: 3000, 3: 2000, 4: 1500},
            "schwarz": {1: 2000, 2: 1000, 3: 512, 4: 200}, "gmres": {1: 2000, 2: 1200, 3: 500, 4: 250},
            "dirk": {1: 64, 2: 36, 3: 8, 4: 8}}[kind][top]
    target = math.exp(rng.uniform(math.log(8), math.log(most)))
    n = [max(2, round(target ** (1 / 3) * math.exp(rng.uniform(-0.4, 0.4)))) for _ in range(2)]
    n.append(min(max(2, round(target / (n[0] * n[1]))), max(2, most // (n[0] * n[1]))))
    ne = n[0] * n[1] * n[2]
    prec = rng.choice(["fp64", "mixed"]) if kind in ("step", "condense") else "fp64"
    more = dict(prec=prec, schwarz=rng.choice(["fp64", "mixed"]), m=rng.randint(8, 40), walls=rng.random() < 0.4,
                chunk=rng.choice([0, 0, rng.randint(5, max(6, ne))]))
    if kind == "dirk":
        more.update(prec="fp64", walls=False, m=40, chunk=0)
    if kind == "condense" and prec == "mixed" and rng.random() < 0.5:
        more["stream"] = True
    return _case(None, kind, n, p, **more)


# ------------------------------------------------------------------ inputs
@functools.lru_cache(maxsize=4)
def _base(n, p, walls, viscous):
    """Mesh and noise-free state of a case (the same for every seed)."""
    ps = [int(v) for v in p.split(",")]
    ne = n[0] * n[1] * n[2]
    ep = ps[0] if len(ps) == 1 else np.random.default_rng(7).choice(ps, size=ne)
    ly = 2 * math.pi
    yc = None
    if walls:  # wall-normal stretching, as the boundary-layer workload
        yc = np.concatenate([[0.0], np.cumsum((2 * math.pi / n[0]) / 10 * 1.15 ** np.arange(n[1]))])
        ly = float(yc[-1])
    mesh = synth.box_mesh(n, lengths=(2 * math.pi, ly, 2 * math.pi), periodic=(True, not walls, True), y_coords=yc,
                          perturb=0.02, p=ep, seed=3)
    if len(ps) > 1:
        mesh = synth.group_by_degree(mesh)
    if walls:
        mach, field = 0.5, lambda x: synth.bl_state(x, 0.5, ly)
    else:
        mach, field = 1.25, lambda x: synth.tgv_state(x, 1.25)
    if viscous:
        field = _compressive
    return synth.make_state(mesh, field, mach=mach, nu_amp=5e-4, seed=1, gmres_m=30,
                            reynolds=400.0 if viscous else 1600.0, boundary_field=field)


def _compressive(x):
    """Taylor-Green vortex with a compression wave, which the viscosity sensor responds to."""
    u = synth.tgv_state(x, 1.25)
    rho = u[..., 0]
    v = [u[..., 1] / rho + 0.4 * np.sin(x[..., 0]), u[..., 2] / rho, u[..., 3] / rho]
    pr = 0.4 * (u[..., 4] - 0.5 * (u[..., 1] ** 2 + u[..., 2] ** 2 + u[..., 3] ** 2) / rho)
    return np.stack([rho, rho * v[0], rho * v[1], rho * v[2],
                     pr / 0.4 + 0.5 * rho * (v[0] ** 2 + v[1] ** 2 + v[2] ** 2)], axis=-1)


def _workload(case, seed):
    """The case's state with the seed's noise on U and Uhat and the seed's viscosity level."""
    b = _base((case["nx"], case["ny"], case["nz"]), case["p"], case["walls"], case["kind"] == "dirk")
    r = np.random.default_rng(seed)
    noise = 1e-3
    return dataclasses.replace(b, U=b.U + r.uniform(-noise, noise, b.U.shape),
                               Uhat=b.Uhat + r.uniform(-noise, noise, b.Uhat.shape),
                               nu=b.nu * r.uniform(0.5, 1.5), gmres_m=case["m"], seed=seed)


def _mesh(case):
    return _base((case["nx"], case["ny"], case["nz"]), case["p"], case["walls"], case["kind"] == "dirk").mesh


class _Trace:
    """Sizes and block pattern of a mesh's trace operator: one block row per face, columns = the faces that share an
    element with it (ascending), block starts rounded up to 16 entries, Schwarz blocks to 32."""

    def __init__(self, mesh):
        ef = mesh.elem_face.astype(np.int64)
        nf = mesh.n_face
        self.b = 5 * (mesh.face_p().astype(np.int64) + 1) ** 2
        self.off = np.concatenate([[0], np.cumsum(self.b)])
        pairs = np.unique((ef[:, :, None] * nf + ef[:, None, :]).ravel())
        self.row, self.col = pairs // nf, pairs % nf
        size = self.b[self.row] * self.b[self.col]
        self.val = np.concatenate([[0], np.cumsum((size + 15) // 16 * 16)])
        self.f = self.b[ef].sum(axis=1)
        self.inv = np.concatenate([[0], np.cumsum((self.f ** 2 + 31) // 32 * 32)])
        self.index = lambda F, G: np.searchsorted(pairs, F * nf + G)
        self.ef, self.N, self.nnzb = ef, int(self.off[-1]), len(pairs)


def _system(case, seed):
    """A trace operator with the decay of a condensed one (a dominant diagonal, couplings of order one per row) and a
    right-hand side, from the seed alone."""
    t = _Trace(_mesh(case))
    g = torch.Generator(device="cuda").manual_seed(seed)
    S = torch.randn(int(t.val[-1]), generator=g, dtype=F64, device="cuda")
    S.mul_(0.5 / math.sqrt(11.0 * float(t.b.mean())))
    size = t.b[t.row] * t.b[t.col]
    for k in np.unique(t.val[1:] - t.val[:-1] - size):  # padding entries are zero
        if k:
            at = (t.val[:-1] + size)[t.val[1:] - t.val[:-1] - size == k]
            S[torch.as_tensor(at[:, None] + np.arange(k), device="cuda")] = 0.0
    d = np.flatnonzero(t.row == t.col)
    for b in np.unique(t.b):
        at = t.val[d[t.b == b]]
        S[torch.as_tensor(at[:, None] + np.arange(b) * (b + 1), device="cuda")] += 2.0
    x = torch.randn(t.N, generator=g, dtype=F64, device="cuda")
    return t, S, x / x.norm()


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("matvec", "schwarz", "gmres"):
        t, S, x = _system(case, seed)
        b = _base((case["nx"], case["ny"], case["nz"]), case["p"], case["walls"], False)
        ctx = hdg.Context(b.mesh, b)
        prec = PREC[case["schwarz"]]
        s = dict(case=case, ctx=ctx, S=S, x=x, y=torch.empty_like(x), prec=prec)
        if kind != "matvec":
            s["Sinv"] = torch.empty(int(t.inv[-1]), dtype=F64 if prec == hdg.HDG_FP64 else torch.float32, device="cuda")
            s["info"] = torch.zeros(b.mesh.n_elem, dtype=torch.int32, device="cuda")
            s["set_up"] = torch.empty(ctx.workspace_size(2, prec), dtype=torch.uint8, device="cuda")
        if kind == "schwarz":
            s["work"] = torch.empty(ctx.workspace_size(3, prec), dtype=torch.uint8, device="cuda")
        if kind == "gmres":
            s["work"] = torch.empty(ctx.workspace_size(4, prec, 0, case["m"]), dtype=torch.uint8, device="cuda")
            s["hist"] = torch.empty(case["m"] + 1, dtype=F64, device="cuda")
            ctx.hdg_asm_setup(prec, S, s["Sinv"], s["info"], s["set_up"])
        return s
    wl = _workload(case, seed)
    st = pipeline.NewtonStep(wl, prec=PREC[case["prec"]], asm_prec=PREC[case["schwarz"]], m=case["m"],
                             chunk=case["chunk"] or None, stream_E=bool(case.get("stream")))
    s = dict(case=case, st=st)
    if kind == "dirk":
        s["start"] = [v.clone() for v in (st.Q, st.U, st.Uhat)]
        s["solver"] = pipeline.NewtonSolver(st, rb_max=4)
        s["stepper"] = pipeline.DirkStepper(s["solver"], av=dict(AV, h_m=2 * math.pi / case["nx"]))
    if kind == "residual":
        s["work"] = torch.empty(st.ctx.workspace_size(6), dtype=torch.uint8, device="cuda")
        s["norms"] = torch.zeros(3, dtype=F64, device="cuda")
    return s


# --------------------------------------------------------------------- run
def run(state):
    kind = state["case"]["kind"]
    if kind == "matvec":
        state["ctx"].hdg_face_matvec(state["S"], state["x"], state["y"])
        return {"y": state["y"]}
    if kind == "schwarz":
        state["ctx"].hdg_asm_setup(state["prec"], state["S"], state["Sinv"], state["info"], state["set_up"])
        state["ctx"].hdg_asm_block_apply(state["prec"], state["Sinv"], state["x"], state["y"], state["work"])
        return {"Sinv": state["Sinv"], "info": state["info"], "z": state["y"]}
    if kind == "gmres":
        state["ctx"].hdg_gmres(state["prec"], state["S"], state["Sinv"], state["x"], state["case"]["m"], state["y"],
                               state["hist"], state["work"])
        return {"x": state["y"], "hist": state["hist"]}
    st = state["st"]
    if kind == "step":
        st.run()
        return {"S": st.S, "g": st.g, "dUhat": st.dUhat, "dQU": st.dQU, "info": st.info, "asm_info": st.asm_info}
    if kind == "condense":
        st.residual_jacobian()
        st.condense()
        st.assemble()
        return {"SK": st.SK, "S": st.S, "g": st.g, "info": st.info}
    if kind == "residual":
        for e0, n in st.chunks:
            st._rj(e0, n)
            st.ctx.hdg_residual_gather(e0, n, st.E_chunk(e0, n), state["work"])
        st.ctx.hdg_residual_norm(state["work"], state["norms"])
        return {"E": st.E, "norms": state["norms"]}
    # dirk: from the same state each time
    solver = state["solver"]
    for dst, src in zip((st.Q, st.U, st.Uhat), state["start"]):
        dst.copy_(src)
    solver.count = solver.head = 0
    state["stepper"].step()
    return {"Q": st.Q, "U": st.U, "Uhat": st.Uhat}


# -------------------------------------------------------------------- work
def _elements(case):
    """(Np, trace size per component, f) of every element."""
    m = _mesh(case)
    t = _Trace(m)
    return [((int(p) + 1) ** 3, int(f) // 5, int(f)) for p, f in zip(m.elem_p, t.f)], t


def _condense_flops(elements):
    """Elimination of the gradient by its mass matrix (54 of the 75 couplings of conserved to gradient fields are
    nonzero; a trace row meets the nodes of its face), then of the conserved fields by a dense LU."""
    total = 0.0
    for Np, w, f in elements:
        p1 = round(Np ** (1 / 3))
        u = 5 * Np
        total += 6.0 * Np * Np * (Np + w) + 108.0 * (Np + w) * (Np * Np + w * p1 * p1)
        total += 2.0 * u ** 3 / 3 + 2.0 * u * u * (f + 1) + 2.0 * f * u * (f + 1)
    return total


def work(case):
    el, t = _elements(case)
    kind, m = case["kind"], case["m"]
    ld = [(20 * Np + f + 8) // 8 * 8 for Np, _, f in el]
    state = 8.0 * (41 * sum(Np for Np, _, _ in el) + 3 * t.N)
    E = 8.0 * sum((20 * Np + f) * l for (Np, _, f), l in zip(el, ld))
    SK = 8.0 * sum(f * (f + 1) for _, _, f in el)
    S = 8.0 * float((t.b[t.row] * t.b[t.col]).sum())
    es = 8.0 if case["schwarz"] == "fp64" else 4.0
    inv = es * sum(f * f for _, _, f in el)
    inv_flops = 2.0 * sum(f ** 3 for _, _, f in el)
    cond_bytes, cond_flops = state + E + SK + S, _condense_flops(el)
    krylov_bytes = m * (S + inv) + 8.0 * t.N * sum(4 * (j + 1) + 8 for j in range(m))
    krylov_flops = m * (S / 4 + 2 * inv / es) + 2.0 * t.N * sum(4 * (j + 1) for j in range(m))
    if kind == "matvec":
        return {"bytes": S + 16.0 * t.N, "flops": S / 4}
    if kind == "schwarz":
        return {"bytes": S + inv + 16.0 * t.N, "flops": inv_flops + 2 * inv / es}
    if kind == "gmres":
        return {"bytes": krylov_bytes, "flops": krylov_flops}
    if kind == "residual":
        return {"bytes": state + E, "flops": 0.0}
    if kind == "condense":
        return {"bytes": cond_bytes, "flops": cond_flops}
    step = {"bytes": cond_bytes + inv + krylov_bytes, "flops": cond_flops + inv_flops + krylov_flops}
    if kind == "dirk":
        return {k: 8 * v for k, v in step.items()}  # three stages of two to three iterations
    return step


# ------------------------------------------------------------------- exact
def _lagrange(nodes, x):
    """Values and derivatives of the Lagrange polynomials of `nodes` at `x`: [x, node]."""
    n = len(nodes)
    L, D = np.ones((len(x), n)), np.zeros((len(x), n))
    for a in range(n):
        others = [k for k in range(n) if k != a]
        den = np.prod([nodes[a] - nodes[k] for k in others])
        L[:, a] = np.prod([x - nodes[k] for k in others], axis=0) / den
        for j in others:
            rest = [x - nodes[k] for k in others if k != j]
            D[:, a] += (np.prod(rest, axis=0) if rest else 1.0) / den
    return L, D


def _flux(u, q, nu, wl):
    """Total flux F^c - F^v - nu q at one point: u [5], q [15] (3c+j) -> [5, 3]."""
    rho, mom, rE = u[0], u[1:4], u[4]
    q = q.reshape(5, 3)
    v, E = mom / rho, rE / rho
    e = E - 0.5 * (v * v).sum()
    pr = (wl.gamma - 1) * (rE - 0.5 * rho * (v * v).sum())
    T = wl.gamma * (wl.gamma - 1) * wl.mach ** 2 * e
    mu = (1.4042 * T ** 1.5 / (T + 0.40417) if wl.visc_law == 1 else torch.ones_like(T)) / wl.reynolds
    dv = (q[1:4] - v[:, None] * q[0]) / rho  # [i, j]
    de = (q[4] - E * q[0]) / rho - v @ dv
    eye = torch.eye(3, dtype=u.dtype, device=u.device)
    tau = mu * (dv + dv.T - 2.0 / 3.0 * eye * torch.trace(dv))
    F = torch.cat([mom[None], mom[:, None] * v + pr * eye - tau,
                   ((rE + pr) * v - v @ tau - wl.gamma * mu / wl.prandtl * de)[None]])
    return F - nu * q


def _element_systems(wl, es, dev):
    """[[A B R_qu],[C D R_uh]] of elements `es`, which share their degree and their faces' degrees: [b, n+f, n+f+1]."""
    mesh = wl.mesh
    T = lambda a: torch.as_tensor(np.ascontiguousarray(a), dtype=F64, device=dev)  # noqa: E731
    p, fp = int(mesh.elem_p[es[0]]), mesh.face_p()
    p1, nq, nb = p + 1, p + 2, len(es)
    Np = p1 ** 3
    no, fo = mesh.node_offsets(), mesh.face_offsets()
    get = lambda a, k: T(np.stack([a[k * no[e]:k * (no[e] + Np)].reshape(k, Np) for e in es]))  # noqa: E731
    U, Un, Q, nu = get(wl.U, 5), get(wl.Un, 5), get(wl.Q, 15), get(wl.nu, 1)[:, 0]
    X8 = T(mesh.vert_xyz[mesh.elem_vert[es]])
    nodes = synth.gll_points(p)
    corner = np.array([-1.0, 1.0])

    def basis(kind, pts):
        """Values and reference derivatives of the tensor basis at pts [g, 3]: [g, node], [3, g, node] (x fastest)."""
        one = [_lagrange(kind, pts[:, d]) for d in range(3)]
        prod = lambda a, b, c: np.einsum("gi,gj,gk->gkji", a, b, c).reshape(len(pts), -1)  # noqa: E731
        val = prod(one[0][0], one[1][0], one[2][0])
        der = [prod(*[one[d][1 if d == k else 0] for d in range(3)]) for k in range(3)]
        return T(val), T(np.stack(der))

    def geometry(pts):
        _, D = basis(corner, pts)
        J = torch.einsum("dgv,bvj->bgjd", D, X8)  # dx_j / dxi_d
        return torch.linalg.inv(J), torch.linalg.det(J)

    jac = lambda fn, arg: torch.func.vmap(torch.func.vmap(torch.func.jacfwd(fn, argnums=arg)))  # noqa: E731
    twice = lambda fn: torch.func.vmap(torch.func.vmap(fn))  # noqa: E731
    flux = lambda u, q, n_: _flux(u, q, n_, wl)  # noqa: E731
    sizes = [5 * (int(fp[F]) + 1) ** 2 for F in mesh.elem_face[es[0]]]
    n, f = 20 * Np, sum(sizes)
    M = torch.zeros((nb, n + f, n + f + 1), dtype=F64, device=dev)
    q_rows = lambda c, j: slice((3 * c + j) * Np, (3 * c + j + 1) * Np)  # noqa: E731
    u_rows = lambda c: slice((15 + c) * Np, (16 + c) * Np)  # noqa: E731
    col = lambda s: slice(s * Np, (s + 1) * Np)  # noqa: E731
    # volume
    x1, w1 = np.polynomial.legendre.leggauss(nq)
    g2, g1, g0 = np.meshgrid(x1, x1, x1, indexing="ij")
    W1 = np.einsum("i,j,k->ijk", w1, w1, w1).ravel()
    pts = np.stack([g0.ravel(), g1.ravel(), g2.ravel()], axis=-1)
    phi, dref = basis(nodes, pts)
    G, det = geometry(pts)
    W = det * T(W1)
    dphi = torch.einsum("bgdj,dgi->bgji", G, dref)
    u, un, q, ng = (torch.einsum("gi,bci->bgc", phi, v) for v in (U, Un, Q, nu[:, None]))
    ng = ng[..., 0]
    F = twice(flux)(u, q, ng)
    dF = torch.cat([jac(flux, 1)(u, q, ng), jac(flux, 0)(u, q, ng)], dim=-1)  # [b, g, c, j, 20]
    mass = torch.einsum("bg,gi,gk->bik", W, phi, phi)
    for c in range(5):
        for j in range(3):
            M[:, q_rows(c, j), col(3 * c + j)] = mass
            M[:, q_rows(c, j), col(15 + c)] = torch.einsum("bg,bgi,gk->bik", W, dphi[:, :, j], phi)
            M[:, q_rows(c, j), -1] = (torch.einsum("bg,bg,gi->bi", W, q[..., 3 * c + j], phi)
                                      + torch.einsum("bg,bg,bgi->bi", W, u[..., c], dphi[:, :, j]))
        M[:, u_rows(c), -1] = (wl.alpha * torch.einsum("bg,bg,gi->bi", W, u[..., c] - un[..., c], phi)
                               - wl.dt * torch.einsum("bg,bgj,bgji->bi", W, F[:, :, c], dphi))
        for s in range(20):
            test = torch.einsum("bg,bgj,bgji->bgi", W, dF[:, :, c, :, s], dphi)
            M[:, u_rows(c), col(s)] = -wl.dt * torch.einsum("bgi,gk->bik", test, phi)
        M[:, u_rows(c), col(15 + c)] += wl.alpha * mass
    # faces
    at = 0
    for lf in range(6):
        faces = mesh.elem_face[es, lf]
        pf = int(fp[faces[0]])
        Nf, d = (pf + 1) ** 2, lf // 2
        t0, t1 = [a for a in range(3) if a != d]
        xf, wf = np.polynomial.legendre.leggauss(pf + 2)
        s1, s0 = np.meshgrid(xf, xf, indexing="ij")
        pts = np.zeros((s0.size, 3))
        pts[:, d], pts[:, t0], pts[:, t1] = 2.0 * (lf & 1) - 1.0, s0.ravel(), s1.ravel()
        phi, _ = basis(nodes, pts)
        L, _ = _lagrange(synth.gll_points(pf), xf)
        mu = T(np.einsum("ta,sb->tsab", L, L).reshape(s0.size, Nf))
        G, det = geometry(pts)
        N = (2.0 * (lf & 1) - 1.0) * det[..., None] * G[:, :, d] * T(np.outer(wf, wf).ravel())[:, None]
        A = N.norm(dim=-1)
        trace = lambda a: T(np.stack([a[fo[k]:fo[k + 1]].reshape(5, Nf) for k in faces]))  # noqa: E731
        u, q, ng = (torch.einsum("gi,bci->bgc", phi, v) for v in (U, Q, nu[:, None]))
        ng = ng[..., 0]
        uh, ub = (torch.einsum("ga,bca->bgc", mu, trace(a)) for a in (wl.Uhat, wl.Ub))

        def normal_flux(uh_, q_, u_, n_, N_, A_):
            return _flux(uh_, q_, n_, wl) @ N_ + wl.tau * A_ * (u_ - uh_)

        args = (uh, q, u, ng, N, A)
        fh = twice(normal_flux)(*args)
        d_uh, d_q, d_u = (jac(normal_flux, k)(*args) for k in range(3))
        d_qu = torch.cat([d_q, d_u], dim=-1)
        bc = torch.as_tensor(np.asarray(mesh.face_bc)[faces] == 1, device=dev)[:, None, None]
        eye = torch.eye(5, dtype=F64, device=dev) * A[..., None, None]
        r_h = torch.where(bc, A[..., None] * (uh - ub), fh)  # boundary faces: the prescribed state
        h_qu = torch.where(bc[..., None], torch.zeros_like(d_qu), d_qu)
        h_uh = torch.where(bc[..., None], eye, d_uh)
        for c in range(5):
            tc = slice(n + at + c * Nf, n + at + (c + 1) * Nf)
            for j in range(3):
                M[:, q_rows(c, j), tc] = -torch.einsum("bg,gi,ga->bia", N[..., j], phi, mu)
                M[:, q_rows(c, j), -1] -= torch.einsum("bg,bg,gi->bi", N[..., j], uh[..., c], phi)
            M[:, u_rows(c), -1] += wl.dt * torch.einsum("bg,gi->bi", fh[..., c], phi)
            M[:, tc, -1] = torch.einsum("bg,ga->ba", r_h[..., c], mu)
            for s in range(20):
                M[:, u_rows(c), col(s)] += wl.dt * torch.einsum("bg,gi,gk->bik", d_qu[:, :, c, s], phi, phi)
                M[:, tc, col(s)] = torch.einsum("bg,ga,gk->bak", h_qu[:, :, c, s], mu, phi)
            for s in range(5):
                ts = slice(n + at + s * Nf, n + at + (s + 1) * Nf)
                M[:, u_rows(c), ts] = wl.dt * torch.einsum("bg,gi,ga->bia", d_uh[:, :, c, s], phi, mu)
                M[:, tc, ts] = torch.einsum("bg,ga,gk->bak", h_uh[:, :, c, s], mu, mu)
        at += sizes[lf]
    return M


def _groups(mesh, most):
    """Elements of equal size (their own degree and their faces'), at most `most` together."""
    fp = mesh.face_p()
    key = {}
    for e in range(mesh.n_elem):
        key.setdefault((int(mesh.elem_p[e]), *(int(v) for v in fp[mesh.elem_face[e]])), []).append(e)
    for k, es in sorted(key.items()):
        for i in range(0, len(es), most):
            yield k, es[i:i + most]


def _exact_condense(case, seed, solve_trace):
    wl = _workload(case, seed)
    mesh, dev = wl.mesh, "cuda"
    t = _Trace(mesh)
    SKo = np.concatenate([[0], np.cumsum(t.f * (t.f + 1))])
    SK = torch.empty(int(SKo[-1]), dtype=F64, device=dev)
    keep = {}
    for k, es in _groups(mesh, 16 if "4" in case["p"] else 32):
        M = _element_systems(wl, np.array(es), dev)
        n = 20 * (k[0] + 1) ** 3
        X = torch.linalg.solve(M[:, :n, :n], M[:, :n, n:])
        R = M[:, n:, n:] - M[:, n:, :n] @ X
        R[:, :, -1] *= -1.0
        for i, e in enumerate(es):
            SK[int(SKo[e]):int(SKo[e + 1])] = R[i].T.reshape(-1)
            if solve_trace:
                keep[e] = X[i]
        del M, X, R
    S = torch.zeros(int(t.val[-1]), dtype=F64, device=dev)
    g = torch.zeros(t.N, dtype=F64, device=dev)
    for e in range(mesh.n_elem):
        f = int(t.f[e])
        K = SK[int(SKo[e]):int(SKo[e + 1])].reshape(f + 1, f).T
        o = np.concatenate([[0], np.cumsum(t.b[t.ef[e]])])
        for a in range(6):
            Fa = t.ef[e, a]
            g[int(t.off[Fa]):int(t.off[Fa + 1])] += K[o[a]:o[a + 1], f]
            for b in range(6):
                at = int(t.val[t.index(Fa, t.ef[e, b])])
                block = K[o[a]:o[a + 1], o[b]:o[b + 1]]
                S[at:at + block.numel()] += block.T.reshape(-1)
    if not solve_trace:
        return SK, S, g, None, None
    D = torch.zeros((t.N, t.N), dtype=F64, device=dev)
    for k in range(t.nnzb):
        F, G = int(t.row[k]), int(t.col[k])
        bF, bG, at = int(t.b[F]), int(t.b[G]), int(t.val[k])
        D[int(t.off[F]):int(t.off[F + 1]), int(t.off[G]):int(t.off[G + 1])] = S[at:at + bF * bG].reshape(bG, bF).T
    x = torch.linalg.solve(D, g)
    parts = []
    for e in range(mesh.n_elem):
        xe = torch.cat([x[int(t.off[F]):int(t.off[F + 1])] for F in t.ef[e]])
        parts.append(-(keep[e][:, -1] + keep[e][:, :-1] @ xe))
    return SK, S, g, x, torch.cat(parts)


def exact(case, seed):
    kind = case["kind"]
    mesh = _mesh(case)
    top = max(int(v) for v in case["p"].split(","))
    if kind == "residual":
        if mesh.n_elem > 600 or "," in case["p"] and mesh.n_elem > 250:
            return None
        wl = _workload(case, seed)
        t = _Trace(mesh)
        n = 20 * (mesh.elem_p.astype(np.int64) + 1) ** 3
        ld = (n + t.f + 8) // 8 * 8
        Eo = np.concatenate([[0], np.cumsum((n + t.f) * ld)])
        E = torch.zeros(int(Eo[-1]), dtype=F64, device="cuda")
        sq, R = torch.zeros(2, dtype=F64, device="cuda"), torch.zeros(t.N, dtype=F64, device="cuda")
        for k, es in _groups(mesh, 16):
            M = _element_systems(wl, np.array(es), "cuda")
            for i, e in enumerate(es):
                rows = int(n[e] + t.f[e])
                E[int(Eo[e]):int(Eo[e + 1])].view(rows, int(ld[e]))[:, :rows + 1] = M[i]
                r = M[i, :, -1]
                cut = 15 * (k[0] + 1) ** 3
                sq += torch.stack([r[:cut].square().sum(), r[cut:int(n[e])].square().sum()])
                o = int(n[e]) + np.concatenate([[0], np.cumsum(t.b[t.ef[e]])])
                for a in range(6):
                    F = t.ef[e, a]
                    R[int(t.off[F]):int(t.off[F + 1])] += r[o[a]:o[a + 1]]
        eo = E if not case["chunk"] or not case.get("stream") else None
        return {"E": eo, "norms": torch.cat([sq.sqrt(), R.norm()[None]])}
    if kind in ("condense", "step"):
        if mesh.n_elem > {1: 2000, 2: 1000, 3: 600, 4: 220}[top] or "," in case["p"] and mesh.n_elem > 250:
            return None
        small = kind == "step" and _Trace(mesh).N <= 10000
        SK, S, g, x, d = _exact_condense(case, seed, small)
        if kind == "condense":
            return {"SK": SK, "S": S, "g": g, "info": None}
        if small and case["m"] < 30:  # the cycle may stop short of the solution
            x = d = None
        return {"S": S, "g": g, "dUhat": x, "dQU": d, "info": None, "asm_info": None}
    if kind == "dirk":
        return None
    t, S, x = _system(case, seed)
    if kind == "matvec":
        y = torch.zeros(t.N, dtype=F64, device="cuda")
        for bF in np.unique(t.b):
            for bG in np.unique(t.b):
                ks = np.flatnonzero((t.b[t.row] == bF) & (t.b[t.col] == bG))
                for i in range(0, len(ks), 4096):
                    k = ks[i:i + 4096]
                    at = torch.as_tensor(t.val[k][:, None] + np.arange(bF * bG), device="cuda")
                    blk = S[at].view(len(k), int(bG), int(bF))
                    xs = x[torch.as_tensor(t.off[t.col[k]][:, None] + np.arange(bG), device="cuda")]
                    to = torch.as_tensor(t.off[t.row[k]][:, None] + np.arange(bF), device="cuda")
                    y.index_add_(0, to.reshape(-1), (blk * xs[:, :, None]).sum(1).reshape(-1))
        return {"y": y}
    if kind == "gmres":
        if t.N > 10000 or case["m"] < 30:  # a shorter cycle may stop short of the solution
            return None
        return {"x": torch.linalg.solve(_dense(t, S), x), "hist": None}
    inv = torch.zeros(int(t.inv[-1]), dtype=F64, device="cuda")
    z = torch.zeros(t.N, dtype=F64, device="cuda")
    for e in range(mesh.n_elem):
        b = t.b[t.ef[e]]
        o = np.concatenate([[0], np.cumsum(b)])
        f = int(t.f[e])
        P = torch.empty((f, f), dtype=F64, device="cuda")
        for a in range(6):
            for c in range(6):
                at = int(t.val[t.index(t.ef[e, a], t.ef[e, c])])
                P[o[a]:o[a + 1], o[c]:o[c + 1]] = S[at:at + int(b[a] * b[c])].view(int(b[c]), int(b[a])).T
        P = torch.linalg.inv(P)
        inv[int(t.inv[e]):int(t.inv[e]) + f * f] = P.T.reshape(-1)
        at = torch.as_tensor(np.concatenate([np.arange(t.off[F], t.off[F + 1]) for F in t.ef[e]]), device="cuda")
        z.index_add_(0, at, P @ x[at])
    return {"Sinv": inv, "info": None, "z": z}


def _dense(t, S):
    D = torch.zeros((t.N, t.N), dtype=F64, device="cuda")
    for k in range(t.nnzb):
        F, G = int(t.row[k]), int(t.col[k])
        bF, bG, at = int(t.b[F]), int(t.b[G]), int(t.val[k])
        D[int(t.off[F]):int(t.off[F + 1]), int(t.off[G]):int(t.off[G + 1])] = S[at:at + bF * bG].view(bG, bF).T
    return D
