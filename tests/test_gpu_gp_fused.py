"""The fused acquisition kernel and the search's selections at the edges of their ranges: one observation, the
64-row blocks, the largest fit that fits in LDS and the first that does not; pools up to the largest size."""
import numpy as np
import pytest

import oracle.bo as obo

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2109_11920_amd.api import Context
    c = Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("n,M,d", [(1, 1, 8), (16, 17, 2), (63, 15, 8), (64, 16, 8), (256, 4097, 8), (1023, 33, 8),
                                   (1024, 50, 64), (1025, 33, 8)])
def test_ei_at_fit_sizes(ctx, n, M, d):
    from paper_2109_11920_amd.api import gp_fit
    rng = np.random.default_rng(n)
    U = rng.uniform(size=(n, d))
    y = 1e5 + 300 * np.sum((U - 0.4) ** 2, axis=1)
    grid = [0.5 * np.sqrt(d / 8)]
    # FP64 throughout; a nugget of 1e-4 bounds the covariance's condition number by n / 1e-4 ~ 1e7, so the
    # variance is good to ~1e-9 and its root to ~1e-7 (times a margin) where it is largest off
    m = gp_fit(U, y, grid, noise=1e-4)
    ref = obo.GP(U, y, grid[0], 1.0, 1e-4)
    Q = rng.uniform(size=(M, d))
    ei, mu, sd = ctx.gp_ei(m, torch.as_tensor(Q, device="cuda"), float(y.min()), 0.0, want_mu_sigma=True)
    mu_r, sd_r = ref.predict(Q)
    ei_r = obo.expected_improvement(mu_r, sd_r, float(y.min()), 0.0)
    for got, want in ((mu, mu_r), (sd, sd_r), (ei, ei_r)):
        assert np.abs(got.cpu().numpy() - want).max() / ref.s < 1e-6


@pytest.mark.parametrize("P,n_global,n_local,per_step,n_taken", [(1024, 4, 0, 1023, 3), (1025, 4, 0, 1025, 0),
                                                                 (4096, 4, 1, 1000, 70), (8192, 4, 4, 2500, 1),
                                                                 (8192, 4, 0, 8192, 130)])
def test_search_at_pool_sizes(ctx, P, n_global, n_local, per_step, n_taken):
    # pools of 4092 to 32768 entries: every entries-per-thread variant of the greedy choice, rounds kept whole
    # or cut, against the host search
    from paper_2109_11920_amd.api import gp_fit
    from paper_2109_11920_amd.bo import chaotic_acquire
    rng = np.random.default_rng(P + per_step)
    U = rng.uniform(size=(70, 8))
    y = 1e5 + 300 * np.sum((U - 0.4) ** 2, axis=1)
    m = gp_fit(U, y, obo.LENGTH_GRID, noise=obo.NOISE)
    best = float(y.min())
    z = rng.uniform(0.01, 0.99, size=(P, 8))
    taken = rng.uniform(size=(n_taken, 8)) if n_taken else None
    kw = dict(n_global=n_global, n_local=n_local, centres=5, radius0=0.1, shrink=0.85, exclusion=0.2, per_step=per_step)
    dev = lambda a: torch.tensor(a, dtype=torch.float64, device="cuda")
    props, vmax, nq = ctx.gp_chaos_search(m, best, 0.0, dev(z), dev(taken) if n_taken else None, 12, **kw)
    host, hmax, hq = chaotic_acquire(lambda Q: ctx.gp_ei(m, dev(np.ascontiguousarray(Q)), best, 0.0).cpu().numpy(), z, 12,
                                     taken, **kw)
    np.testing.assert_array_equal(props.cpu().numpy(), host)
    assert vmax == hmax and nq == hq
