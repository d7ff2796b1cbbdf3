"""Infinities and NaN stay where the arithmetic puts them: an entry that takes no part
in a result does not reach it through a product with a zero."""
import numpy as np
import pytest

from gpu_common import e_view, sk_view

pytestmark = pytest.mark.gpu


def _mesh(n, p, walls=False):
    from paper_2608_27863_amd import synth
    ne = n[0] * n[1] * n[2]
    ep = p if isinstance(p, int) else np.random.default_rng(3).choice(p, size=ne)
    return synth.box_mesh(n, periodic=(True, not walls, True), p=ep, perturb=0.1, seed=4)


def _workload(n, p):
    from paper_2608_27863_amd import synth
    return synth.make_state(_mesh(n, p), lambda x: synth.tgv_state(x, 1.25), mach=1.25, noise=1e-3, nu_amp=5e-4,
                            seed=5)


@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("p", [1, 2, 3, 4, (1, 2, 4)])
def test_trace_of_one_face_reaches_that_face_only(p, value):
    """A non-finite trace state on one face: the rows of the nodes off that face, and of the
    other faces, are bit for bit those of a finite one."""
    import torch
    from paper_2608_27863_amd import pipeline
    wl = _workload((3, 2, 2), p)
    print(f"[nonfinite] trace of a face, p={p} {value}", flush=True)
    st = pipeline.NewtonStep(wl)
    ctx = st.ctx
    st.residual_jacobian()
    torch.cuda.synchronize()
    clean = st.E.cpu().numpy().copy()
    F = 7
    fo = ctx.layout["face_off"]
    st.Uhat[int(fo[F]):int(fo[F + 1])] = value
    st.residual_jacobian()
    torch.cuda.synchronize()
    got = st.E.cpu().numpy()
    hit = 0
    for e in range(ctx.n_elem):
        a, b = e_view(ctx, clean, e)[0], e_view(ctx, got, e)[0]
        n = int(ctx.layout["elem_n"][e])
        p1 = round((n // 20) ** (1 / 3))
        sizes = [int(fo[G + 1] - fo[G]) for G in wl.mesh.elem_face[e]]
        rows = np.ones(b.shape[0], dtype=bool)
        for lf, G in enumerate(wl.mesh.elem_face[e]):
            if G != F:
                continue
            hit += 1
            idx = np.stack(np.unravel_index(np.arange(n // 20), (p1, p1, p1)))[::-1]  # x fastest
            on = idx[lf // 2] == (p1 - 1 if lf % 2 else 0)
            rows[:n] &= ~np.tile(on, 20)
            rows[n + sum(sizes[:lf]):n + sum(sizes[:lf + 1])] = False
        assert np.array_equal(a[rows], b[rows]), e
        assert rows.all() or not np.isfinite(b[~rows]).all()
    assert hit == 2


@pytest.mark.parametrize("n,p", [((2, 2, 2), 1), ((2, 2, 2), 4), ((4, 3, 3), (1, 2, 4)), ((6, 6, 6), 4)])
def test_matvec_with_an_infinite_entry(n, p):
    """S with one infinite entry in the last column of a face row: the product's entry is
    that infinity, every other one is that of the finite operator."""
    import torch
    from paper_2608_27863_amd import hdg, synth
    wl = synth.make_state(synth.box_mesh((2, 2, 2), p=1), lambda x: synth.tgv_state(x, 1.25), mach=1.25)
    ctx = hdg.Context(_mesh(n, p), wl)
    print(f"[nonfinite] matvec, {n} p={p}: {ctx.n_face} faces", flush=True)
    rp, vo, fo = (ctx.layout[k] for k in ("bsr_row_ptr", "bsr_val_off", "face_off"))
    g = torch.Generator("cuda").manual_seed(1)
    S = torch.randn(int(vo[-1]), dtype=torch.float64, device="cuda", generator=g)
    x = torch.rand(ctx.N_uh, dtype=torch.float64, device="cuda", generator=g) + 0.5
    y, z = torch.empty_like(x), torch.empty_like(x)
    ctx.hdg_face_matvec(S, x, y)
    at = {}
    col = ctx.layout["bsr_col"]
    for F, i, sign in ((0, 0, 1.0), (ctx.n_face // 2, 3, -1.0), (ctx.n_face - 1, -1, 1.0)):
        k = int(rp[F + 1]) - 1  # the row's last block, column-major
        bF, bG = int(fo[F + 1] - fo[F]), int(fo[col[k] + 1] - fo[col[k]])
        S[int(vo[k]) + (bG - 1) * bF + i % bF] = sign * float("inf")
        at[int(fo[F]) + i % bF] = sign * float("inf")
    ctx.hdg_face_matvec(S, x, z)
    y, z = y.cpu().numpy(), z.cpu().numpy()
    for i, v in at.items():
        assert z[i] == v, (i, z[i])
        z[i] = y[i]
    assert np.array_equal(y, z)


@pytest.mark.parametrize("prec", ["FP64", "MIXED_FAST"])
@pytest.mark.parametrize("p", [1, 2, 4])
def test_trace_block_entry_stays_in_place(p, prec):
    """A NaN in D (trace row r, trace column c) is a NaN in S^K at (r, c) and nowhere else,
    also in the columns next to a last panel of fewer than 64 (reduced systems of 40, 136
    and 628 columns, whole ones of 160, 540 and 2500)."""
    import torch
    from paper_2608_27863_amd import hdg, pipeline
    wl = _workload((2, 2, 2), p)
    print(f"[nonfinite] an entry of D, p={p} {prec}", flush=True)
    st = pipeline.NewtonStep(wl, prec=getattr(hdg, "HDG_" + prec))
    ctx = st.ctx
    st.residual_jacobian()
    E = st.E.clone()
    st.condense()
    torch.cuda.synchronize()
    ref = st.SK.cpu().numpy().copy()
    at = {e: (11 * e + 2, e) for e in range(ctx.n_elem)}
    for e, (r, c) in at.items():
        o, n, f = (int(ctx.layout[k][e]) for k in ("E_off", "elem_n", "elem_f"))
        ld = (int(ctx.layout["E_off"][e + 1]) - o) // (n + f)
        E[o + (n + r) * ld + n + c] = float("nan")
    st.E.copy_(E)
    st.condense()
    torch.cuda.synchronize()
    assert not st.info.any().item()
    got = st.SK.cpu().numpy()
    for e, (r, c) in at.items():
        S, g = sk_view(ctx, got, e)
        Sr, gr = sk_view(ctx, ref, e)
        assert np.isnan(S[r, c])
        S = S.copy()
        S[r, c] = Sr[r, c]
        assert np.array_equal(S, Sr) and np.array_equal(g, gr), e
