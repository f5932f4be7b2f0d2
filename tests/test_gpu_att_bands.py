"""The attenuation build by row bands deals the rays to workgroups by their direction along the bands: angle counts
with few or no rays of one direction, angles exactly along the rows, odd splits, half the angles and all, against the
FP64 oracle; and any candidate count (so any launch shape) the same values."""
import numpy as np
import pytest

from gpu_helpers import TOL, geom_pair, oracle, report

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _dev(a):
    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.float32), device="cuda")


@pytest.mark.parametrize("pair", ["1", "0"])
@pytest.mark.parametrize("n,na,nb,nt,C", [(200, 2, 200, 200, 1), (200, 3, 64, 200, 2), (204, 4, 70, 204, 1), (210, 5, 64, 150, 3),
                                          (200, 6, 60, 301, 1), (283, 7, 64, 284, 1), (200, 8, 65, 200, 2), (199, 22, 64, 232, 1)])
def test_directions(monkeypatch, n, na, nb, nt, C, pair):
    from paper_2109_11920_amd.api import Context
    monkeypatch.setenv("BOAC_OPPOSED_RAYS", pair)
    g, og = geom_pair(n, na, nb, nt)
    rng = np.random.default_rng(na)
    mu = rng.uniform(0.0, 0.3, (C, n, n)).astype(np.float32)
    F = rng.uniform(0.0, 2.0, (C, n, n)).astype(np.float32)
    with Context(0) as ctx:
        y = ctx.project(g, _dev(mu), _dev(F)).cpu().numpy()
    att = oracle.attenuation(og, mu[-1].astype(np.float64))
    report(f"project n={n} na={na}", y[-1], oracle.project(og, att, F[-1].astype(np.float64)), TOL)


@pytest.mark.parametrize("n,na,nb,nt", [(200, 18, 64, 200), (256, 9, 100, 256), (210, 40, 210, 210)])
def test_any_candidate_count_gives_the_same_values(n, na, nb, nt):
    from paper_2109_11920_amd.api import Context
    g, _ = geom_pair(n, na, nb, nt)
    rng = np.random.default_rng(n)
    mu = _dev(rng.uniform(0.0, 0.2, (60, n, n)))
    F = _dev(rng.uniform(0.0, 2.0, (60, n, n)))
    with Context(0) as ctx:
        ref = ctx.project(g, mu, F).cpu().numpy()
        for C in (1, 3, 8, 16, 24, 41):
            np.testing.assert_array_equal(ctx.project(g, mu[:C].contiguous(), F[:C].contiguous()).cpu().numpy(), ref[:C])
