"""Images staged in row bands: the attenuation build, the projection, the reverse sweep and the tail take each
ray's samples band by band. Smallest and uneven band splits, rays and samples that are multiples of nothing,
paired and not, against the FP64 oracle (the repository's gates); and every launch shape a saved plan may
hold gives the same values to summation order (a ray's own arithmetic does not depend on it)."""
import json

import numpy as np
import pytest

import oracle
from gpu_helpers import TOL, TOL_GRAD, cands, geom_pair, make_slice, report

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _dev(a):
    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.float32), device="cuda")


# 140/141: the last single-stage and first two-band size of the pair image; 199/200: of one image; 201 x 18: an
# odd number of half angles; short rays that end inside the image, long ones that start far outside
@pytest.mark.parametrize("n,na,nb,nt,C", [(141, 6, 141, 141, 2), (199, 4, 199, 199, 1), (200, 8, 200, 200, 2),
                                          (201, 18, 70, 230, 1), (203, 5, 203, 203, 2), (230, 6, 64, 101, 3),
                                          (256, 8, 256, 256, 1)])
def test_bands_match_oracle(n, na, nb, nt, C):
    from oracle.adjoint import objective_and_grad
    from paper_2109_11920_amd.api import Context
    g, og = geom_pair(n, na, nb, nt)
    rng = np.random.default_rng(n)
    S, _ = make_slice(og, seed=n)
    S = S.astype(np.float32).astype(np.float64)
    th = cands(n, C)
    mu = np.stack([oracle.rasterize_mu(og, t, 0.8) for t in th]).astype(np.float32)
    F = rng.uniform(0.0, 2.0, (C, n, n)).astype(np.float32)
    ctx = Context(0)
    y = ctx.project(g, _dev(mu), _dev(F)).cpu().numpy()
    J, grad, _ = ctx.objective_grad_ex(g, _dev(S), _dev(th), 0.8, 3, 2)
    for c in sorted({0, C - 1}):
        att = oracle.attenuation(og, mu[c].astype(np.float64))
        report(f"project n={n} cand {c}", y[c], oracle.project(og, att, F[c].astype(np.float64)), TOL)
        Jr, gr = objective_and_grad(og, S, th[c], float(np.float32(0.8)), 3, True)
        report(f"J cand {c}", [J[c].item()], [Jr], TOL)
        report(f"gradient cand {c}", grad[c].cpu().numpy(), gr, TOL_GRAD)
    ctx.close()


@pytest.mark.parametrize("n,na,nb", [(202, 6, 75), (210, 5, 64)])
def test_bands_launch_shapes(n, na, nb, tmp_path):
    from paper_2109_11920_amd.api import Context
    C = 2
    g, og = geom_pair(n, na, nb, n)
    rng = np.random.default_rng(nb)
    S = _dev(rng.poisson(20.0, (na, nb)))
    th = _dev(cands(n, C))
    F = _dev(rng.uniform(0.0, 2.0, (C, n, n)))
    ref = None
    for block, rpt in [(None, 0), (64, 1), (64, 4), (192, 3), (256, 2), (1024, 1), (1024, 4)]:
        f = tmp_path / f"plan_{block}_{rpt}.json"
        if block:
            f.write_text(json.dumps({f"ray:{n}x{na}x{nb}x{n}:{C}:{x}": [block, rpt] for x in (1, 2)}))
        ctx = Context(0, tune_cache=str(f))
        y = ctx.project(g, ctx.rasterize_mu(g, th, 0.8), F)
        J, grad, _ = ctx.objective_grad_ex(g, S, th, 0.8, 2, 2)
        out = [x.cpu().numpy().copy() for x in (y, J, grad)]
        ctx.close()
        if ref is None:
            ref = out
            continue
        np.testing.assert_array_equal(out[0], ref[0])  # per ray: the same bits
        np.testing.assert_array_equal(out[2], ref[2])
        np.testing.assert_allclose(out[1], ref[1], rtol=1e-6)
