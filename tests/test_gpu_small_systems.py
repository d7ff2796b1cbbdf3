"""Matvec, Schwarz apply and the GMRES vector kernels on both sides of the sizes at
which another kernel takes over (faces, elements, block sides), against plain
FP64 sums of the same data."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

U64 = 2.0 ** -53


def _context(n, p, walls=False):
    from paper_2608_27863_amd import hdg, synth
    ne = n[0] * n[1] * n[2]
    ep = p if isinstance(p, int) else np.random.default_rng(3).choice(p, size=ne)
    mesh = synth.box_mesh(n, periodic=(True, not walls, True), p=ep)
    wl = synth.make_state(synth.box_mesh((2, 2, 2), p=1), lambda x: synth.tgv_state(x, 1.25), mach=1.25)
    return hdg.Context(mesh, wl), mesh


def _system(ctx, seed):
    """Random blocks with a dominant diagonal, zero padding, and a vector (host arrays)."""
    r = np.random.default_rng(seed)
    rp, col, vo, fo = (ctx.layout[k] for k in ("bsr_row_ptr", "bsr_col", "bsr_val_off", "face_off"))
    S = np.zeros(int(vo[-1]))
    blocks = {}
    for F in range(ctx.n_face):
        bF = int(fo[F + 1] - fo[F])
        for k in range(int(rp[F]), int(rp[F + 1])):
            G = int(col[k])
            bG = int(fo[G + 1] - fo[G])
            B = r.standard_normal((bF, bG)) * (0.5 / np.sqrt(11.0 * bG))
            if F == G:
                B += 2.0 * np.eye(bF)
            blocks[F, G] = B
            S[int(vo[k]):int(vo[k]) + bF * bG] = B.T.ravel()
    return S, blocks, r.standard_normal(ctx.N_uh)


@pytest.mark.parametrize("n,p,walls", [((2, 2, 2), 1, False), ((5, 5, 5), 4, False), ((6, 6, 5), 4, False),
                                       ((8, 8, 3), 3, True), ((6, 6, 5), (1, 2, 4), True), ((6, 5, 6), (2, 3), False),
                                       ((9, 9, 4), 2, False), ((9, 9, 9), 1, True)])
def test_matvec_on_both_sides_of_the_switch(n, p, walls):
    import torch
    ctx, _ = _context(n, p, walls)
    print(f"[small] matvec, {n} p={p}: {ctx.n_face} faces", flush=True)
    S, blocks, x = _system(ctx, 1)
    y = torch.empty(ctx.N_uh, dtype=torch.float64, device="cuda")
    ctx.hdg_face_matvec(torch.as_tensor(S, device="cuda"), torch.as_tensor(x, device="cuda"), y)
    got = y.cpu().numpy()
    fo = ctx.layout["face_off"]
    ref, size, terms = np.zeros(ctx.N_uh), np.zeros(ctx.N_uh), np.zeros(ctx.N_uh)
    for (F, G), B in blocks.items():
        a, b = slice(int(fo[F]), int(fo[F + 1])), slice(int(fo[G]), int(fo[G + 1]))
        ref[a] += B @ x[b]
        size[a] += np.abs(B) @ np.abs(x[b])
        terms[a] += B.shape[1]
    # each side sums `terms` products: |error| <= terms u sum |product|
    assert np.all(np.abs(got - ref) <= 2 * (terms + 2) * U64 * size)


@pytest.mark.parametrize("prec", ["FP64", "MIXED"])
@pytest.mark.parametrize("n,p", [((2, 2, 2), 1), ((6, 6, 7), 2), ((6, 6, 8), 2), ((5, 5, 5), 3), ((8, 4, 4), 3),
                                 ((8, 6, 6), 3), ((8, 10, 5), 3), ((3, 3, 3), 4), ((6, 7, 6), (1, 3))])
def test_schwarz_apply_on_both_sides_of_the_switch(n, p, prec):
    import torch
    from paper_2608_27863_amd import hdg
    ctx, mesh = _context(n, p)
    pc = getattr(hdg, "HDG_" + prec)
    print(f"[small] Schwarz apply {prec}, {n} p={p}: {ctx.n_elem} elements", flush=True)
    r = np.random.default_rng(2)
    dt = np.float64 if prec == "FP64" else np.float32
    ao, fo, f = ctx.layout["asm_off"], ctx.layout["face_off"], ctx.layout["elem_f"]
    M = np.zeros(int(ao[-1]), dtype=dt)
    for e in range(ctx.n_elem):
        M[int(ao[e]):int(ao[e]) + int(f[e]) ** 2] = r.standard_normal(int(f[e]) ** 2)
    x = r.standard_normal(ctx.N_uh)
    z = torch.empty(ctx.N_uh, dtype=torch.float64, device="cuda")
    work = torch.empty(ctx.workspace_size(3, pc), dtype=torch.uint8, device="cuda")
    ctx.hdg_asm_block_apply(pc, torch.as_tensor(M, device="cuda"), torch.as_tensor(x, device="cuda"), z, work)
    got = z.cpu().numpy()
    ref, size = np.zeros(ctx.N_uh), np.zeros(ctx.N_uh)
    for e in range(ctx.n_elem):
        at = np.concatenate([np.arange(fo[F], fo[F + 1]) for F in mesh.elem_face[e]])
        A = M[int(ao[e]):int(ao[e]) + int(f[e]) ** 2].reshape(int(f[e]), int(f[e])).T.astype(np.float64)
        np.add.at(ref, at, A @ x[at])
        np.add.at(size, at, np.abs(A) @ np.abs(x[at]))
    assert np.all(np.abs(got - ref) <= 2 * (int(f.max()) + 4) * U64 * size)


@pytest.mark.parametrize("n,p,m", [((2, 2, 2), 1, 1), ((2, 2, 2), 1, 40), ((3, 2, 2), (1, 2, 4), 30), ((4, 4, 4), 2, 33),
                                   ((7, 7, 7), 1, 200), ((6, 6, 6), 3, 25)])
def test_gmres_vector_kernels(n, p, m):
    """A converging cycle against the solution, its residual estimates against the true
    preconditioned residuals of a reference cycle; slices of the vectors from 64 entries
    (one workgroup's tile) up, remainders among them, up to the longest cycle."""
    import torch
    from paper_2608_27863_amd import hdg
    ctx, mesh = _context(n, p)
    print(f"[small] GMRES({m}), {n} p={p}: {ctx.N_uh} unknowns", flush=True)
    S, blocks, b = _system(ctx, 5)
    fo = ctx.layout["face_off"]
    dev = dict(dtype=torch.float64, device="cuda")
    Sd, bd = torch.as_tensor(S, device="cuda"), torch.as_tensor(b, device="cuda")
    Sinv = torch.empty(int(ctx.layout["asm_off"][-1]), **dev)
    info = torch.zeros(ctx.n_elem, dtype=torch.int32, device="cuda")
    ctx.hdg_asm_setup(0, Sd, Sinv, info, torch.empty(ctx.workspace_size(2), dtype=torch.uint8, device="cuda"))
    x, hist = torch.empty(ctx.N_uh, **dev), torch.empty(m + 1, **dev)
    ctx.hdg_gmres(hdg.HDG_FP64, Sd, Sinv, bd, m, x, hist,
                  torch.empty(ctx.workspace_size(4, 0, 0, m), dtype=torch.uint8, device="cuda"))
    assert not info.any().item()
    h = hist.cpu().numpy()
    assert np.all(np.isfinite(h)) and np.all(np.diff(h) <= 1e-14 * h[0])
    got = x.cpu().numpy()

    def mul(v):
        out = np.zeros_like(v)
        for (F, G), B in blocks.items():
            out[fo[F]:fo[F + 1]] += B @ v[fo[G]:fo[G + 1]]
        return out

    # the estimate of the last step is the norm of M^{-1} (b - S x)
    res, z = torch.as_tensor(b - mul(got), device="cuda"), torch.empty(ctx.N_uh, **dev)
    ctx.hdg_asm_block_apply(0, Sinv, res, z, torch.empty(ctx.workspace_size(3), dtype=torch.uint8, device="cuda"))
    true = float(z.norm())
    # rounding of the residual itself: about 1e-15 of h[0] here (S is a few times the identity)
    assert abs(true - h[-1]) <= 1e-10 * true + 1e-13 * h[0]
    if m >= 25:
        assert np.linalg.norm(b - mul(got)) <= 1e-12 * np.linalg.norm(b)


@pytest.mark.parametrize("n,p", [((11, 10, 10), 1), ((8, 8, 5), 2)])
def test_gradient_rows_by_several_nodes(n, p):
    """A call over many small elements gives a workgroup 8 (p = 1) or 3 nodes (p = 2): the
    same bits as calls over few elements, one node a workgroup."""
    import torch
    from paper_2608_27863_amd import pipeline, synth
    mesh = synth.box_mesh(n, periodic=(True, True, True), p=p, perturb=0.1, seed=3)
    wl = synth.make_state(mesh, lambda x: synth.tgv_state(x, 1.25), mach=1.25, noise=1e-3, nu_amp=5e-4, seed=5)
    print(f"[small] gradient rows, {mesh.n_elem} elements at p={p}", flush=True)
    got = []
    for chunk in (mesh.n_elem, 100):
        st = pipeline.NewtonStep(wl, chunk=chunk)
        st.E.fill_(float("nan"))
        st.residual_jacobian()
        torch.cuda.synchronize()
        got.append(st.E.clone())
        del st
    assert torch.equal(got[0], got[1])


@pytest.mark.parametrize("prec", ["FP64", "MIXED"])
def test_schwarz_apply_off_16_bytes(prec):
    """480-row inverses (columns of whole lines) that start one entry off a 16-byte boundary,
    from as many elements on as take the kernel of 16-byte loads: the same product."""
    import torch
    from paper_2608_27863_amd import hdg
    ctx, mesh = _context((8, 8, 7), 3)
    pc = getattr(hdg, "HDG_" + prec)
    print(f"[small] Schwarz apply {prec}, inverses off 16 bytes, {ctx.n_elem} elements", flush=True)
    dt = torch.float64 if prec == "FP64" else torch.float32
    g = torch.Generator("cuda").manual_seed(3)
    n = int(ctx.layout["asm_off"][-1])
    buf = torch.randn(n + 1, dtype=dt, device="cuda", generator=g)
    x = torch.randn(ctx.N_uh, dtype=torch.float64, device="cuda", generator=g)
    work = torch.empty(ctx.workspace_size(3, pc), dtype=torch.uint8, device="cuda")
    out = []
    for M in (buf[1:], buf[1:].clone()):
        z = torch.empty_like(x)
        ctx.hdg_asm_block_apply(pc, M, x, z, work)
        out.append(z)
    # both sum the columns in increasing order, row by row
    assert buf[1:].data_ptr() % 16 != 0 and torch.equal(out[0], out[1])
