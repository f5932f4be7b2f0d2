"""Sizes that hold the attenuation of every angle: sample counts that are no multiple of 4 and detectors finer
than the pixels. No attenuation there is derived from the opposed ray's, so paths of any optical depth are exact
at both angle halves, and turning opposed-ray pairing off changes no bit; few and many candidates (each gather
variant), against the FP64 oracle."""
import numpy as np
import pytest

import oracle
from gpu_helpers import TOL, cands, geom_pair, report

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# remainders 1 to 3 of the sample count, bin windows of 2 and 3; slot staging (34 x 12), column groups of 1 to 4
SHAPES = [(33, 6, 33, 33, 2), (34, 8, 34, 34, 12), (35, 6, 35, 35, 45), (64, 10, 64, 66, 40), (48, 8, 60, 48, 2),
          (49, 6, 70, 50, 33), (40, 10, 80, 40, 70), (36, 8, 64, 37, 3)]


def _dev(a):
    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.float32), device="cuda")


@pytest.mark.parametrize("n,na,nb,nt,C", SHAPES)
def test_deep_paths_at_both_angle_halves(n, na, nb, nt, C):
    # attenuation of 4 to 8 per cm over 25.6 cm: depths of 100 and more, where exp(-T) of a whole ray is 0 in FP32.
    # A depth L is good to L 2^-23, and samples deeper than 20 add nothing: 3e-6 of a ray, within TOL
    from paper_2109_11920_amd.api import Context
    g, og = geom_pair(n, na, nb, nt)
    rng = np.random.default_rng(n)
    mu = rng.uniform(4.0, 8.0, (C, n, n)).astype(np.float32)
    F = rng.uniform(0.5, 2.0, (C, n, n)).astype(np.float32)
    z = rng.uniform(0.2, 2.0, (C, na, nb)).astype(np.float32)
    far = z.copy()
    far[:, :na // 2] = 0.0  # the second half of the angles alone
    with Context(0) as ctx:
        y = ctx.project(g, _dev(mu), _dev(F)).cpu().numpy()
        x, xf = (ctx.backproject(g, _dev(mu), _dev(w)).cpu().numpy() for w in (z, far))
    for c in sorted({0, C // 2, C - 1}):
        att = oracle.attenuation(og, mu[c].astype(np.float64))
        ref = oracle.project(og, att, F[c].astype(np.float64))
        report(f"project cand {c}, first half", y[c][:na // 2], ref[:na // 2], TOL)
        report(f"project cand {c}, second half", y[c][na // 2:], ref[na // 2:], TOL)
        report(f"backproject cand {c}", x[c], oracle.backproject(og, att, z[c].astype(np.float64)), TOL)
        report(f"backproject cand {c}, second half", xf[c], oracle.backproject(og, att, far[c].astype(np.float64)), TOL)


@pytest.mark.parametrize("n,na,nb,nt,C", SHAPES)
def test_pairing_switch_changes_nothing(monkeypatch, n, na, nb, nt, C):
    from paper_2109_11920_amd.api import Context
    g, _ = geom_pair(n, na, nb, nt)
    rng = np.random.default_rng(n)
    S = _dev(rng.poisson(20.0, (na, nb)))
    th = _dev(cands(n, C))
    z = _dev(rng.uniform(0.2, 2.0, (C, na, nb)))
    out = []
    for flag in ("1", "0"):
        monkeypatch.setenv("BOAC_OPPOSED_RAYS", flag)
        with Context(0) as ctx:
            mu = ctx.rasterize_mu(g, th, 0.8)
            res = [ctx.backproject(g, mu, z), *ctx.objective_grad_ex(g, S, th, 0.8, 3, 2),
                   *ctx.objective(g, S, th, 0.8, 3, want_image=True)]
            out.append([r.cpu().numpy().copy() for r in res])
    for a, b in zip(*out):
        np.testing.assert_array_equal(a, b)
