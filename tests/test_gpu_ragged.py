"""Sample counts that are no multiple of 4 in the column-group gather: the blocks at the rays' end stage the
layout's padding rows as zeros. Each remainder, with and without opposed-ray pairing (even and odd angle
counts), every candidates-per-workgroup variant the counts select, and the angle split of few candidates,
against the FP64 oracle (relative L2 and largest error within the repository's gates)."""
import numpy as np
import pytest

import oracle
from gpu_helpers import TOL, TOL_GRAD, cands, geom_pair, make_slice, report

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2109_11920_amd.api import Context
    c = Context(0)
    yield c
    c.close()


def _dev(a):
    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.float32), device="cuda")


@pytest.mark.parametrize("n,na,nb,nt,C", [(32, 6, 32, 33, 1), (33, 7, 33, 33, 12), (34, 8, 32, 34, 10), (35, 5, 36, 35, 3),
                                          (47, 16, 47, 47, 33), (64, 10, 64, 66, 40), (109, 6, 109, 109, 17)])
def test_ragged_samples(ctx, n, na, nb, nt, C):
    from oracle.adjoint import objective_and_grad
    g, og = geom_pair(n, na, nb, nt)
    rng = np.random.default_rng(n + nt)
    S, _ = make_slice(og, seed=n)
    S = S.astype(np.float32).astype(np.float64)
    th = cands(nt, C)
    mu = np.stack([oracle.rasterize_mu(og, t, 0.8) for t in th]).astype(np.float32)
    z = rng.uniform(0.2, 2.0, (C, na, nb)).astype(np.float32)
    x = ctx.backproject(g, _dev(mu), _dev(z)).cpu().numpy()
    pick = sorted({0, C // 2, C - 1})
    for c in pick:
        att = oracle.attenuation(og, mu[c].astype(np.float64))
        report(f"backproject n={n} nt={nt} cand {c}", x[c], oracle.backproject(og, att, z[c].astype(np.float64)), TOL)
    K = 4
    J, grad, _ = ctx.objective_grad_ex(g, _dev(S), _dev(th), 0.8, K, 2)
    J2, img, _ = ctx.objective(g, _dev(S), _dev(th), 0.8, K, want_image=True)
    for c in pick:
        Jr, gr = objective_and_grad(og, S, th[c], float(np.float32(0.8)), K, True)
        Fr = oracle.evaluate(og, S, th[c], float(np.float32(0.8)), K)[1]
        report(f"J cand {c}", [J[c].item(), J2[c].item()], [Jr, Jr], TOL)
        report(f"image cand {c}", img[c].cpu().numpy(), Fr, TOL)
        report(f"gradient cand {c}", grad[c].cpu().numpy(), gr, TOL_GRAD)
