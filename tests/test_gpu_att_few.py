"""The attenuation build of few candidates, a ray over 8 lanes, gives one thread per ray's values bit for bit: rays of
one group of 4 samples to more than a round of 8 groups, each remainder, one to many rays per lane group, paired and
not; and any candidate count the same values (its launch shape, its own and the projection's, is chosen by the count)."""
import numpy as np
import pytest

from gpu_helpers import TOL, cands, geom_pair, oracle, report

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _dev(a):
    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.float32), device="cuda")


@pytest.mark.parametrize("n,na,nb,nt,C", [(6, 2, 5, 2, 1), (8, 3, 8, 4, 2), (16, 5, 16, 29, 3), (20, 6, 24, 32, 1), (20, 7, 21, 33, 9),
                                          (32, 6, 32, 35, 2), (32, 48, 32, 32, 8), (64, 64, 64, 64, 8), (64, 9, 70, 66, 30),
                                          (96, 10, 96, 127, 4), (128, 8, 128, 128, 1), (192, 4, 64, 300, 2)])
def test_scan_over_lanes_equals_thread_per_ray(monkeypatch, n, na, nb, nt, C):
    from paper_2109_11920_amd.api import Context
    g, og = geom_pair(n, na, nb, nt)
    rng = np.random.default_rng(nt)
    mu = rng.uniform(0.0, 0.3, (C, n, n)).astype(np.float32)
    F = rng.uniform(0.0, 2.0, (C, n, n)).astype(np.float32)
    out = []
    for flag in ("1", "0"):
        monkeypatch.setenv("BOAC_ATT_SCAN", flag)
        with Context(0) as ctx:
            out.append(ctx.project(g, _dev(mu), _dev(F)).cpu().numpy())
    np.testing.assert_array_equal(out[0], out[1])
    att = oracle.attenuation(og, mu[-1].astype(np.float64))
    report(f"project n={n} nt={nt}", out[0][-1], oracle.project(og, att, F[-1].astype(np.float64)), TOL)


@pytest.mark.parametrize("n,na,nb,nt", [(96, 96, 96, 96), (61, 36, 61, 61), (128, 20, 100, 128), (150, 9, 150, 150), (192, 12, 96, 192)])
def test_any_candidate_count_gives_the_same_values(n, na, nb, nt):
    from paper_2109_11920_amd.api import Context
    g, _ = geom_pair(n, na, nb, nt)
    th = cands(n, 70)
    rng = np.random.default_rng(n)
    F = rng.uniform(0.0, 2.0, (70, n, n)).astype(np.float32)
    with Context(0) as ctx:
        mu = ctx.rasterize_mu(g, _dev(th), 0.8)
        ref = ctx.project(g, mu, _dev(F)).cpu().numpy()
        for C in (1, 2, 5, 9, 16, 23, 40):
            np.testing.assert_array_equal(ctx.project(g, mu[:C].contiguous(), _dev(F[:C])).cpu().numpy(), ref[:C])
