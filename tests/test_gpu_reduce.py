"""The two routes of the FP64 condensation: elimination of the gradient through its
mass matrix where the element system has the HDG structure, the dense LU of all
columns where any entry says otherwise.  Both against each other on the same
systems, and the choice against systems altered in every place the structure
check has to see."""
import numpy as np
import pytest

from gpu_common import RTOL_FP64, e_view, rel_err, sk_view

pytestmark = pytest.mark.gpu

U64 = 2.0 ** -53


def _workload(p, walls):
    from paper_2608_27863_amd import synth
    n = (3, 2, 2)
    ep = p if isinstance(p, int) else np.random.default_rng(2).choice(p, size=12)
    mesh = synth.box_mesh(n, periodic=(True, not walls, True), p=ep, perturb=0.1, seed=4)
    if walls:
        mesh = synth.set_boundary_types(mesh, {(1, 0): 4, (1, 1): 3})
    f = lambda x: synth.tgv_state(x, 1.25)  # noqa: E731
    return synth.make_state(mesh, f, mach=1.25, noise=1e-3, nu_amp=5e-4, seed=5, boundary_field=f)


def _condensed(st, E):
    import torch
    st.E.copy_(E)
    st.condense()
    torch.cuda.synchronize()
    assert not st.info.any().item()
    return st.SK.cpu().numpy().copy(), st.E.cpu().numpy().copy()


def _reduced(ctx, Ehost, e):
    """Whether element e's factored system has the scaled gradient rows [I | Y | r]."""
    Ev, _ = e_view(ctx, Ehost, e)
    return Ev[0, 0] == 1.0 and not Ev[0, 1:int(ctx.layout["elem_n"][e]) * 3 // 4].any()


@pytest.mark.parametrize("p,walls,chunk", [(1, False, None), (2, True, 5), (3, False, 12), (4, True, 7),
                                           ((1, 2, 3, 4), True, 5)])
def test_both_routes_agree(p, walls, chunk):
    import torch
    from paper_2608_27863_amd import pipeline
    wl = _workload(p, walls)
    print(f"[reduce] p={p} walls={walls} chunk={chunk}", flush=True)
    st = pipeline.NewtonStep(wl, chunk=chunk)
    ctx = st.ctx
    st.residual_jacobian()
    E0 = st.E.clone()
    E1 = E0.clone()
    for e in range(ctx.n_elem):  # one entry of no consequence outside the structure: the dense route
        n = int(ctx.layout["elem_n"][e])
        E1[int(ctx.layout["E_off"][e]) + n // 20] = 1e-290
    d = torch.as_tensor(wl.x, dtype=torch.float64, device="cuda")
    SK, dQU, fact = [], [], []
    for E in (E0, E1):
        sk, _ = _condensed(st, E)
        st.ctx.hdg_recover_interior(0, 0, ctx.n_elem, st.E, d, st.dQU)
        torch.cuda.synchronize()
        SK.append(sk)
        fact.append(st.E.cpu().numpy().copy())
        dQU.append(st.dQU.cpu().numpy().copy())
    assert all(_reduced(ctx, fact[0], e) for e in range(ctx.n_elem))
    assert not any(_reduced(ctx, fact[1], e) for e in range(ctx.n_elem))
    host, no, fo = E0.cpu().numpy(), ctx.layout["node_off"], ctx.layout["face_off"]
    for e in range(ctx.n_elem):
        for a, b in zip(sk_view(ctx, SK[0], e), sk_view(ctx, SK[1], e)):
            assert rel_err(a, b) <= 2 * RTOL_FP64  # each is within RTOL_FP64 of the oracle
    for e in (0, ctx.n_elem - 1):
        # recovered increments: two backward-stable solves with A differ by at most
        # the a-priori forward bound of each, 4 cond(A) u (|x_r| + |X_B| |dUh|)
        Ev, _ = e_view(ctx, host, e)
        n = int(ctx.layout["elem_n"][e])
        A = Ev[:n, :n]
        X = np.linalg.solve(A, Ev[:n, n:])
        dl = np.concatenate([wl.x[fo[F]:fo[F + 1]] for F in wl.mesh.elem_face[e]])
        size = np.linalg.norm(np.abs(X[:, -1]) + np.abs(X[:, :-1]) @ np.abs(dl))
        got = [v[20 * int(no[e]):20 * int(no[e + 1])] for v in dQU]
        assert np.linalg.norm(got[0] - got[1]) <= 8 * np.linalg.cond(A, 1) * U64 * size


@pytest.mark.parametrize("p", [1, 2])
def test_altered_systems_take_the_dense_route(p):
    """One alteration per element, in each place that the elimination relies on; the
    result is the condensation of the altered system, and the unaltered elements keep
    theirs bit for bit."""
    from paper_2608_27863_amd import pipeline
    wl = _workload(p, False)
    print(f"[reduce] altered systems, p={p}", flush=True)
    st = pipeline.NewtonStep(wl)
    ctx = st.ctx
    st.residual_jacobian()
    E0 = st.E.clone()
    ref, _ = _condensed(st, E0)
    p1 = p + 1
    Np = p1 ** 3
    n, f = 20 * Np, int(ctx.layout["elem_f"][0])
    nfp = p1 * p1
    inner = next(i for i in range(Np) if i % p1 == p1 - 1)  # a node off the face -x
    at = {  # element: (row, column)
        0: (4 * Np, 4 * Np),                       # the mass matrix of one field
        1: (0, 14 * Np + Np - 1),                  # a gradient row's zero block
        2: (14 * Np + Np - 1, 19 * Np + Np - 1),   # G of component 4
        3: (3 * Np, n + nfp),                      # H of component 1
        4: (2, n + nfp),                           # component 0's rows in component 1's trace columns
        5: (15 * Np, 14 * Np),                     # the mass row and the energy's gradient
        6: (16 * Np + 1, 12 * Np),                 # a momentum row and the energy's gradient
        7: (n, inner),                             # a trace row and a node off its face
        8: (n + f - 1, 0),                         # the last trace row (face +z) and a node at -z
    }
    E1 = E0.clone()
    scale = {}
    for e, (r, c) in at.items():
        o = int(ctx.layout["E_off"][e])
        ld = (int(ctx.layout["E_off"][e + 1]) - o) // (n + f)
        scale[e] = float(E1[o])
        E1[o + r * ld + c] += 0.25 * scale[e]
    got, fact = _condensed(st, E1)
    host = E1.cpu().numpy()
    for e in range(ctx.n_elem):
        assert _reduced(ctx, fact, e) == (e not in at), e
        S, g = sk_view(ctx, got, e)
        if e in at:
            Ev, _ = e_view(ctx, host, e)
            R = Ev[n:, n:] - Ev[n:, :n] @ np.linalg.solve(Ev[:n, :n], Ev[:n, n:])
            assert rel_err(S, R[:, :-1]) <= RTOL_FP64, e
        else:
            Sr, gr = sk_view(ctx, ref, e)
            assert np.array_equal(S, Sr) and np.array_equal(g, gr)


def test_workspace_is_bounded_and_pieces_agree():
    """A call over a whole mesh needs no more workspace than the bound, and equals the
    calls chunk by chunk (tests/test_gpu_c0.py holds chunkings to the same bits)."""
    from paper_2608_27863_amd import hdg, synth
    mesh = synth.box_mesh((10, 10, 10), p=4)
    ctx = hdg.Context(mesh, synth.make_state(synth.box_mesh((2, 2, 2), p=1), lambda x: synth.tgv_state(x, 1.25),
                                             mach=1.25))
    whole, part = ctx.workspace_size(1), ctx.workspace_size(1, e0=100, ne=100)
    assert part < whole <= (9 << 29) + 4096
    assert ctx.workspace_size(1, e0=0, ne=300) == whole


@pytest.mark.parametrize("p,walls,chunk", [(1, False, 5), (2, True, None), (3, True, 7), (4, False, 12),
                                           ((1, 2, 3, 4), True, 5)])
def test_mixed_routes_agree(p, walls, chunk):
    """HDG_MIXED: S^K and g^K of both routes within its 1e-10 of an FP64 solve, and the
    X stored for the recovery within what the route through all columns leaves, or 1e-11."""
    import torch
    from paper_2608_27863_amd import hdg, pipeline
    wl = _workload(p, walls)
    print(f"[reduce] mixed, p={p} walls={walls} chunk={chunk}", flush=True)
    st = pipeline.NewtonStep(wl, prec=hdg.HDG_MIXED, chunk=chunk)
    ctx = st.ctx
    st.residual_jacobian()
    E0 = st.E.clone()
    E1 = E0.clone()
    for e in range(ctx.n_elem):
        E1[int(ctx.layout["E_off"][e]) + int(ctx.layout["elem_n"][e]) // 20] = 1e-290
    out = [_condensed(st, E) for E in (E0, E1)]
    host = E0.cpu().numpy()
    for e in range(ctx.n_elem):
        if e not in (0, 5, ctx.n_elem - 1):
            continue
        n = int(ctx.layout["elem_n"][e])
        Ev, _ = e_view(ctx, host, e)
        X = np.linalg.solve(Ev[:n, :n], Ev[:n, n:])
        R = Ev[n:, n:] - Ev[n:, :n] @ X
        err = []
        for SK, fact in out:
            S, g = sk_view(ctx, SK, e)
            assert rel_err(S, R[:, :-1]) <= 1e-10 and rel_err(g, -R[:, -1]) <= 1e-10
            err.append(rel_err(e_view(ctx, fact, e)[0][:n, n:], X))
        print(f"  element {e}: X {err[0]:.2e} (all columns: {err[1]:.2e})")
        assert err[0] <= max(err[1], 1e-11)
    torch.cuda.synchronize()


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("p", [1, 2, 3])
def test_pivot_search_with_ties(p, precision):
    """Systems of whole numbers in [-2, 2]: in the first pivot columns nearly every largest
    value is tied, also between the rows that different waves hold.  n = 160, 540 and
    1280 pivot columns pass every size at which the panels change their split.  S = D - B
    A^{-1} C against the same in 64 bits.  Tolerance: a backward-stable solve is within
    4 cond(A) u of |B| |A^{-1} C|, here two of them (u of the factorisation's type)."""
    import torch
    from paper_2608_27863_amd import hdg, pipeline
    wl = _workload(p, False)
    print(f"[reduce] ties, p={p} {precision}", flush=True)
    st = pipeline.NewtonStep(wl, prec=hdg.HDG_FP64 if precision == "fp64" else hdg.HDG_MIXED_FAST)
    ctx = st.ctx
    rng = np.random.default_rng(11)
    host = rng.integers(-2, 3, size=st.E.numel()).astype(np.float64)
    st.E.copy_(torch.as_tensor(host))
    st.condense()
    torch.cuda.synchronize()
    assert not st.info.any().item()
    SK = st.SK.cpu().numpy()
    for e in (0, ctx.n_elem - 1):
        Ev, _ = e_view(ctx, host, e)
        n = int(ctx.layout["elem_n"][e])
        X = np.linalg.solve(Ev[:n, :n], Ev[:n, n:])
        R = Ev[n:, n:] - Ev[n:, :n] @ X
        S, g = sk_view(ctx, SK, e)
        size = np.linalg.norm(np.abs(Ev[n:, :n]) @ np.abs(X))
        tol = 8 * np.linalg.cond(Ev[:n, :n], 1) * (U64 if precision == "fp64" else 2.0 ** -24) * size
        assert np.linalg.norm(S - R[:, :-1]) <= tol and np.linalg.norm(g + R[:, -1]) <= tol, e
