"""The column-group gather off its first sizes. Sample counts that are no multiple of 4: the blocks at the
rays' end stage the layout's padding rows as zeros. Detectors finer than the pixels: bin windows of two and
three. Each remainder, with and without opposed-ray pairing (even and odd angle
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
                                          (47, 16, 47, 47, 33), (64, 10, 64, 66, 40), (109, 6, 109, 109, 17),
                                          # wider bin windows: the smallest and largest detector of each, one
                                          # to 4 candidates per workgroup, paired and not
                                          (46, 8, 49, 46, 17), (45, 9, 48, 44, 40), (49, 6, 86, 50, 33), (33, 7, 58, 33, 2),
                                          (48, 8, 85, 48, 40), (40, 10, 80, 40, 33), (36, 5, 72, 35, 3), (16, 6, 32, 32, 5)])
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


@pytest.mark.parametrize("n,na,nb,nt,C", [(32, 2, 32, 32, 1), (33, 14, 34, 33, 8), (40, 131, 40, 41, 2), (64, 258, 64, 64, 5),
                                          (121, 18, 128, 124, 1), (40, 70, 48, 40, 3), (33, 9, 58, 37, 8),
                                          (36, 20, 64, 36, 1), (50, 131, 100, 49, 2)])
def test_few_candidate_gather_equals_tile_gather(ctx, monkeypatch, n, na, nb, nt, C):
    # 8 x 8 tiles with a wave per 8 angles against 16 x 16 tiles: one to 17 blocks (more than the waves of a
    # workgroup), a last block of one angle, ragged image edges; same arithmetic, so the same bits
    g, og = geom_pair(n, na, nb, nt)
    rng = np.random.default_rng(na)
    S = _dev(rng.poisson(20.0, (na, nb)))
    th = _dev(cands(na, C))
    z = _dev(rng.uniform(0.2, 2.0, (C, na, nb)))
    out = {}
    for flag in ("1", "0"):
        monkeypatch.setenv("BOAC_GATHER_SPLIT", flag)
        mu = ctx.rasterize_mu(g, th, 0.8)
        out[flag] = [ctx.backproject(g, mu, z), *ctx.objective_grad_ex(g, S, th, 0.8, 3, 2)]
        out[flag] = [x.cpu().numpy().copy() for x in out[flag]]
    for a, b in zip(out["1"], out["0"]):
        np.testing.assert_array_equal(a, b)
