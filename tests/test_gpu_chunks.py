"""Single-stage ray kernels: whole chunks of 16 samples run without a test per sample, the rest of a ray with
one. Sample counts on both sides of a chunk, half and group edge, odd candidate counts, paired and not, against
the FP64 oracle (the repository's gates); and a repeated call gives the same bits."""
import numpy as np
import pytest

import oracle
from gpu_helpers import TOL, TOL_GRAD, cands, geom_pair, make_slice, report

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _dev(a):
    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.float32), device="cuda")


@pytest.mark.parametrize("n,na,nb,nt,C", [(16, 6, 16, 15, 3), (16, 6, 16, 16, 10), (20, 5, 24, 17, 9), (24, 8, 24, 24, 11),
                                          (31, 6, 33, 31, 12), (32, 7, 32, 32, 2), (40, 66, 40, 41, 17), (61, 8, 61, 68, 9),
                                          (64, 16, 64, 64, 12)])
def test_sample_chunks(n, na, nb, nt, C):
    from oracle.adjoint import objective_and_grad
    from paper_2109_11920_amd.api import Context
    g, og = geom_pair(n, na, nb, nt)
    rng = np.random.default_rng(nt)
    S, _ = make_slice(og, seed=nt)
    S = S.astype(np.float32).astype(np.float64)
    th = cands(nt, C)
    mu = np.stack([oracle.rasterize_mu(og, t, 0.8) for t in th]).astype(np.float32)
    F = rng.uniform(0.0, 2.0, (C, n, n)).astype(np.float32)
    ctx = Context(0)
    runs = []
    for _ in range(2):
        y = ctx.project(g, _dev(mu), _dev(F))
        J, grad, _ = ctx.objective_grad_ex(g, _dev(S), _dev(th), 0.8, 4, 2)
        J2, img, _ = ctx.objective(g, _dev(S), _dev(th), 0.8, 4, want_image=True)
        runs.append([x.cpu().numpy().copy() for x in (y, J, grad, J2, img)])
    ctx.close()
    for a, b in zip(*runs):
        np.testing.assert_array_equal(a, b)
    y, J, grad, J2, img = runs[0]
    for c in sorted({0, C // 2, C - 1}):
        att = oracle.attenuation(og, mu[c].astype(np.float64))
        report(f"project cand {c}", y[c], oracle.project(og, att, F[c].astype(np.float64)), TOL)
        Jr, gr = objective_and_grad(og, S, th[c], float(np.float32(0.8)), 4, True)
        report(f"J cand {c}", [J[c], J2[c]], [Jr, Jr], TOL)
        report(f"gradient cand {c}", grad[c], gr, TOL_GRAD)
