"""Pivot searches full of ties in well-conditioned systems, where a wrong exchange would show
in FP32 too."""
import numpy as np
import pytest

from gpu_common import e_view, rel_err, sk_view

pytestmark = pytest.mark.gpu


def _hadamard(n):
    H = np.ones((1, 1))
    while H.shape[0] < n:
        H = np.block([[H, H], [H, -H]])
    return H


def _tied(n, r):
    """Blocks of +-1 with orthogonal rows (32 x 32, then 4 x 4), the rows of all blocks
    shuffled: every column's largest value is shared by the rows of its block that are left,
    wherever they lie, and the elimination stays in small whole numbers and halves."""
    A = np.zeros((n, n))
    i = 0
    while i < n:
        b = 32 if n - i >= 32 else 4
        A[i:i + b, i:i + b] = _hadamard(b)
        i += b
    return A[r.permutation(n)]


@pytest.mark.parametrize("prec", ["FP64", "MIXED", "MIXED_FAST"])
@pytest.mark.parametrize("p", [1, 2, 3])
def test_ties(p, prec):
    """n = 160, 540 and 1280 columns: every size at which the panels change their split.  The
    tolerances: 8 cond(A) u (u of the factorisation's type) of |C| |A^{-1} B|, and a hundredth
    of the result at most; HDG_MIXED to its 1e-10."""
    import torch
    from paper_2608_27863_amd import hdg, pipeline, synth
    mesh = synth.box_mesh((3, 2, 2), p=p)
    wl = synth.make_state(mesh, lambda x: synth.tgv_state(x, 1.25), mach=1.25)
    st = pipeline.NewtonStep(wl, prec=getattr(hdg, "HDG_" + prec))
    ctx = st.ctx
    print(f"[ties] p={p} {prec}", flush=True)
    r = np.random.default_rng(12)
    host = r.integers(-2, 3, size=st.E.numel()).astype(np.float64)
    for e in range(ctx.n_elem):
        n = int(ctx.layout["elem_n"][e])
        Ev, _ = e_view(ctx, host, e)
        Ev[:n, :n] = _tied(n, r)
    st.E.copy_(torch.as_tensor(host))
    st.condense()
    torch.cuda.synchronize()
    assert not st.info.any().item()
    SK = st.SK.cpu().numpy()
    u = 2.0 ** (-24 if prec == "MIXED_FAST" else -53)
    for e in range(ctx.n_elem):
        Ev, _ = e_view(ctx, host, e)
        n = int(ctx.layout["elem_n"][e])
        A = Ev[:n, :n]
        X = np.linalg.solve(A, Ev[:n, n:])
        R = Ev[n:, n:] - Ev[n:, :n] @ X
        S, g = sk_view(ctx, SK, e)
        if prec == "MIXED":
            assert rel_err(S, R[:, :-1]) <= 1e-10 and rel_err(g, -R[:, -1]) <= 1e-10, e
            continue
        size = np.abs(Ev[n:, :n]) @ np.abs(X)
        for got, want, s in ((S, R[:, :-1], size[:, :-1]), (g, -R[:, -1], size[:, -1])):
            tol = 8 * np.linalg.cond(A, 1) * u * np.linalg.norm(s)
            assert tol <= 1e-2 * np.linalg.norm(want)
            assert np.linalg.norm(got - want) <= tol, e
