"""Failures on the route through the reduced systems: pivots planted so that the gradient
rows keep their structure, the one-call step on states that are not finite, and a
mass matrix without an inverse.  The planted values are ordinary data: every kernel runs
to its normal end."""
import math

import numpy as np
import pytest

from gpu_common import e_view, sk_view

pytestmark = pytest.mark.gpu

U64 = 2.0 ** -53


@pytest.fixture(scope="module")
def systems():
    import torch
    from paper_2608_27863_amd import pipeline, synth
    wl = synth.config(0)  # 4^3 periodic, p = 2: 405 gradient and 135 conserved unknowns per element
    print("[reduced failure] element systems of the 4^3 p=2 mesh", flush=True)
    st = pipeline.NewtonStep(wl)
    st.residual_jacobian()
    torch.cuda.synchronize()
    return wl, st, st.E.clone()


def _sys(ctx, E, e):
    n, f = int(ctx.layout["elem_n"][e]), int(ctx.layout["elem_f"][e])
    o0, o1 = int(ctx.layout["E_off"][e]), int(ctx.layout["E_off"][e + 1])
    return E[o0:o1].view(n + f, (o1 - o0) // (n + f))


def _keeps_structure(Ev, Np):
    """The same mass matrix in all gradient rows and the same G_j for every component."""
    A = Ev[:15 * Np].cpu().numpy()
    M = A[:Np, :Np]
    return all(np.array_equal(A[r * Np:(r + 1) * Np, r * Np:(r + 1) * Np], M) and
               np.array_equal(A[r * Np:(r + 1) * Np, (15 + r // 3) * Np:(16 + r // 3) * Np],
                              A[r % 3 * Np:(r % 3 + 1) * Np, 15 * Np:16 * Np]) for r in range(15))


@pytest.mark.parametrize("prec", ["FP64", "MIXED"])
def test_planted_pivots_of_reduced_systems(systems, prec):
    """info counts the gradient's 15 N_p pivots, taken with the mass matrix, before those of
    the conserved rows; all other elements keep their bits."""
    import torch
    from paper_2608_27863_amd import hdg, pipeline
    wl, st0, E0 = systems
    ctx = st0.ctx
    st = pipeline.NewtonStep(wl, prec=getattr(hdg, "HDG_" + prec), ctx=ctx, share=st0)
    print(f"[reduced failure] {prec}, clean and planted", flush=True)
    st.E.copy_(E0)
    st.condense()
    torch.cuda.synchronize()
    assert not st.info.any().item()
    ref = st.SK.clone()
    Np, n, k = 27, 540, 70
    E = E0.clone()
    _sys(ctx, E, 3)[15 * Np + 5, :] = 0.0  # an empty conserved row: no pivot is left for the last column
    s = _sys(ctx, E, 10)                   # an empty column k of u in every row, G_j of each component alike
    for c in range(5):
        for j in range(3):
            s[(3 * c + j) * Np:(3 * c + j + 1) * Np, (15 + c) * Np + k % Np] = 0.0
    s[15 * Np:, 15 * Np + k] = 0.0
    _sys(ctx, E, 21)[15 * Np + 2, 15 * Np] = math.inf
    _sys(ctx, E, 40)[16 * Np, 15 * Np] = math.nan
    expect = {3: n, 10: 15 * Np + k + 1, 21: 15 * Np + 1, 40: 15 * Np + 1}
    assert all(_keeps_structure(_sys(ctx, E, e), Np) for e in expect)
    st.E.copy_(E)
    st.condense()
    torch.cuda.synchronize()
    info = st.info.cpu().numpy()
    got = {int(e): int(info[e]) for e in np.nonzero(info)[0]}
    print(f"  info: {got}")
    assert got == expect
    o = ctx.layout["SK_off"]
    for e in range(ctx.n_elem):
        if e not in expect:
            assert torch.equal(st.SK[int(o[e]):int(o[e + 1])], ref[int(o[e]):int(o[e + 1])]), e


@pytest.mark.parametrize("prec", ["FP64", "MIXED"])
@pytest.mark.parametrize("value", [math.nan, math.inf, 0.0])
def test_one_call_step_reports_a_state_that_is_not_finite(systems, prec, value):
    """The one-call step runs without the structure check: a density of NaN, infinity or zero at
    one element's nodes is reported for that element at its first conserved pivot, and for
    no other; the failing iteration is seen by the driver."""
    import torch
    from paper_2608_27863_amd import hdg, pipeline
    wl, st0, E0 = systems
    ctx = st0.ctx
    st = pipeline.NewtonStep(wl, prec=getattr(hdg, "HDG_" + prec), ctx=ctx)
    e, Np = 17, 27
    st.run()
    torch.cuda.synchronize()
    assert not st.info.any().item()
    no = int(ctx.layout["node_off"][e])
    st.U[5 * no:5 * no + Np] = value
    print(f"[reduced failure] one-call step, {prec}, density {value} in element {e}", flush=True)
    st.run()
    torch.cuda.synchronize()
    info = st.info.cpu().numpy()
    assert {int(i): int(info[i]) for i in np.nonzero(info)[0]} == {e: 15 * Np + 1}
    assert f"element {e} " in pipeline.NewtonSolver(st).pivot_failure()


def _random_structured(shape, Np, f, zero_row, r):
    """A system with the structure of the gradient rows, well conditioned although row zero_row of
    the mass matrix is zero: random couplings of ordinary size in every place that a formed
    system fills."""
    n, p1, w = 20 * Np, round(Np ** (1 / 3)), f // 5
    E = np.zeros(shape)
    M = np.eye(Np) + 0.1 * r.standard_normal((Np, Np))
    M[zero_row] = 0.0
    G, H = r.standard_normal((3, Np, Np)), r.standard_normal((3, Np, w))
    nfp = w // 6
    idx = np.stack(np.unravel_index(np.arange(Np), (p1, p1, p1)))[::-1]  # x fastest
    for c in range(5):
        cols = np.concatenate([n + 5 * nfp * lf + nfp * c + np.arange(nfp) for lf in range(6)])
        for j in range(3):
            rows = (3 * c + j) * Np + np.arange(Np)
            E[rows[:, None], rows] = M
            E[rows[:, None], (15 + c) * Np + np.arange(Np)] = G[j]
            E[rows[:, None], cols] = H[j]
        read = 3 * Np * (1, 4, 4, 4, 5)[c]  # columns of the gradients that row c's fluxes read
        rows = (15 + c) * Np + np.arange(Np)
        E[rows, :read] = r.standard_normal((Np, read))
        for lf in range(6):
            on = np.nonzero(np.tile(idx[lf // 2] == (p1 - 1 if lf % 2 else 0), 15))[0]
            t = n + 5 * nfp * lf + nfp * c + np.arange(nfp)
            E[t[:, None], on[on < read]] = r.standard_normal((nfp, int((on < read).sum())))
    E[15 * Np:, 15 * Np:n + f + 1] = r.standard_normal((5 * Np + f, 5 * Np + f + 1))
    E[:15 * Np, n + f] = r.standard_normal(15 * Np)
    return E


def test_mass_matrix_without_an_inverse(systems):
    """Gradient rows with the structure but a singular M, in systems that have a solution all
    the same: the LU of all columns takes them.  Tolerance: a backward-stable solve is within
    4 cond(A) u of |C| |A^{-1} B|, here two of them."""
    import torch
    wl, st0, E0 = systems
    ctx, Np, n = st0.ctx, 27, 540
    E, r = E0.clone(), np.random.default_rng(8)
    for e, row in ((5, 0), (60, 13)):
        s = _sys(ctx, E, e)
        s.copy_(torch.as_tensor(_random_structured(tuple(s.shape), Np, int(ctx.layout["elem_f"][e]), row, r)))
    print("[reduced failure] singular mass matrices in elements 5 and 60", flush=True)
    assert all(_keeps_structure(_sys(ctx, E, e), Np) for e in (5, 60))
    host = E.cpu().numpy()
    st0.E.copy_(E)
    st0.condense()
    torch.cuda.synchronize()
    assert not st0.info.any().item()
    SK = st0.SK.cpu().numpy()
    for e in (5, 60):
        Ev, _ = e_view(ctx, host, e)
        X = np.linalg.solve(Ev[:n, :n], Ev[:n, n:])
        R = Ev[n:, n:] - Ev[n:, :n] @ X
        S, g = sk_view(ctx, SK, e)
        tol = 8 * np.linalg.cond(Ev[:n, :n], 1) * U64 * np.linalg.norm(np.abs(Ev[n:, :n]) @ np.abs(X))
        print(f"  element {e}: |S| {np.linalg.norm(R[:, :-1]):.2e}, tolerance {tol:.2e}")
        assert tol <= 1e-3 * np.linalg.norm(R[:, :-1])
        assert np.linalg.norm(S - R[:, :-1]) <= tol and np.linalg.norm(g + R[:, -1]) <= tol, e


@pytest.mark.parametrize("kind,eps", [("row", 1e-2), ("row", 1e-4), ("row", 1e-8), ("row", 1e-12), ("column", 1e-8),
                                      ("near", 1e-3), ("near", 1e-6), ("near", 1e-9), ("near", 1e-12)])
def test_ill_conditioned_mass_matrix(systems, kind, eps):
    """Gradient rows with the structure, A well conditioned and M less and less so (a row or a
    column scaled by eps, or a row that differs from another by eps): S^K and g^K within
    what a solve with pivoting over all of A allows, 8 cond(A) u |C| |A^{-1} B|."""
    import torch
    wl, st0, E0 = systems
    ctx, Np, n = st0.ctx, 27, 540
    r = np.random.default_rng(9)
    M = np.eye(Np) + 0.1 * r.standard_normal((Np, Np))
    if kind == "row":
        M[4] *= eps
    elif kind == "column":
        M[:, 4] *= eps
    else:
        M[4] = M[9] + eps * r.standard_normal(Np)
    E = E0.clone()
    print(f"[reduced failure] mass matrix, {kind} {eps}: cond {np.linalg.cond(M):.1e}", flush=True)
    for e in (5, 60):
        s = _sys(ctx, E, e)
        new = _random_structured(tuple(s.shape), Np, int(ctx.layout["elem_f"][e]), 4, r)
        for k in range(15):
            new[k * Np:(k + 1) * Np, k * Np:(k + 1) * Np] = M
        s.copy_(torch.as_tensor(new))
        assert _keeps_structure(s, Np)
    host = E.cpu().numpy()
    st0.E.copy_(E)
    st0.condense()
    torch.cuda.synchronize()
    assert not st0.info.any().item()
    SK = st0.SK.cpu().numpy()
    for e in (5, 60):
        Ev, _ = e_view(ctx, host, e)
        X = np.linalg.solve(Ev[:n, :n], Ev[:n, n:])
        R = Ev[n:, n:] - Ev[n:, :n] @ X
        S, g = sk_view(ctx, SK, e)
        tol = 8 * np.linalg.cond(Ev[:n, :n], 1) * U64 * np.linalg.norm(np.abs(Ev[n:, :n]) @ np.abs(X))
        err = np.linalg.norm(S - R[:, :-1])
        print(f"  element {e}: |S| {np.linalg.norm(R[:, :-1]):.2e}, error {err:.2e}, tolerance {tol:.2e}")
        assert tol <= 1e-3 * np.linalg.norm(R[:, :-1])
        assert err <= tol and np.linalg.norm(g + R[:, -1]) <= tol, e
