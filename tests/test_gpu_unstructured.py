"""Systems without the structure of the HDG gradient equations, in HDG_MIXED: the
refinement has to see every entry of A, also in the field blocks that are zero in
systems the library forms itself."""
import numpy as np
import pytest

from gpu_common import e_view, rel_err, sk_view

pytestmark = pytest.mark.gpu

RTOL_MIXED = 1e-10  # HDG_MIXED's bound on S^K and g^K against an FP64 solve (one refinement step)
RTOL_X = 1e-7       # X itself: an FP32 solve is within about 1e-5, a step squares that (times a margin)


def _step(p):
    from paper_2608_27863_amd import hdg, pipeline, synth
    mesh = synth.box_mesh((3, 2, 2), p=p, perturb=0.1, seed=4)
    wl = synth.make_state(mesh, lambda x: synth.tgv_state(x, 1.25), mach=1.25, noise=1e-3, nu_amp=5e-4, seed=5)
    return pipeline.NewtonStep(wl, prec=hdg.HDG_MIXED)


def _check(st, E, elems):
    import torch
    ctx, host = st.ctx, E.cpu().numpy()
    st.E.copy_(E)
    st.condense()
    torch.cuda.synchronize()
    assert not st.info.any().item()
    SK, fact = st.SK.cpu().numpy(), st.E.cpu().numpy()
    for e in elems:
        n = int(ctx.layout["elem_n"][e])
        Ev, _ = e_view(ctx, host, e)
        X = np.linalg.solve(Ev[:n, :n], Ev[:n, n:])
        R = Ev[n:, n:] - Ev[n:, :n] @ X
        S, g = sk_view(ctx, SK, e)
        err = rel_err(S, R[:, :-1]), rel_err(g, -R[:, -1]), rel_err(e_view(ctx, fact, e)[0][:n, n:], X)
        print(f"  element {e}: S {err[0]:.2e} g {err[1]:.2e} X {err[2]:.2e}", flush=True)
        assert max(err[:2]) <= RTOL_MIXED and err[2] <= RTOL_X, e


@pytest.mark.parametrize("p", [1, 2, 3])
def test_entries_in_blocks_that_formed_systems_leave_zero(p):
    """One entry per element, in a field block of A that the fluxes make zero."""
    st = _step(p)
    ctx = st.ctx
    st.residual_jacobian()
    E = st.E.clone()
    Np = (p + 1) ** 3
    at = {0: (0, 14 * Np + Np - 1),             # a gradient row and another gradient field
          1: (1, 19 * Np),                      # a gradient row and another component
          2: (15 * Np, 14 * Np),                # the mass row and the energy's gradient
          3: (16 * Np + 1, 12 * Np),            # a momentum row and the energy's gradient
          4: (14 * Np + Np - 1, 15 * Np + 1)}   # the last gradient row and the density
    print(f"[unstructured] one entry, p={p}", flush=True)
    for e, (r, c) in at.items():
        o, n, f = int(ctx.layout["E_off"][e]), 20 * Np, int(ctx.layout["elem_f"][e])
        ld = (int(ctx.layout["E_off"][e + 1]) - o) // (n + f)
        E[o + r * ld + c] += 0.25 * float(E[o])
    _check(st, E, at)


@pytest.mark.parametrize("p", [1, 2])
def test_full_systems(p):
    """Random systems, no zero anywhere, the diagonal of A dominant."""
    import torch
    st = _step(p)
    ctx = st.ctx
    print(f"[unstructured] full systems, p={p}", flush=True)
    r = np.random.default_rng(3)
    host = r.standard_normal(st.E.numel())
    for e in range(ctx.n_elem):
        n = int(ctx.layout["elem_n"][e])
        Ev, _ = e_view(ctx, host, e)
        Ev[np.arange(n), np.arange(n)] += 4.0 * np.sqrt(n)
    _check(st, torch.as_tensor(host, device="cuda"), (0, ctx.n_elem - 1))
