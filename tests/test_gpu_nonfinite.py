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
