"""The greedy choice's exclusion at any size: radii whose square is below the single-precision range keep points out
as larger ones do, against the host search."""
import numpy as np
import pytest

import oracle.bo as obo

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [8, 3])
@pytest.mark.parametrize("size", [1e-3, 1e-18, 1e-21, 1e-23, 1e-25, 1e-34, 1e-40])
def test_search_at_exclusion_radii(size, d):
    from paper_2109_11920_amd.api import Context, gp_fit
    from paper_2109_11920_amd.bo import chaotic_acquire
    rng = np.random.default_rng(7)
    U = rng.uniform(size=(40, d))
    y = 1e5 + 300 * np.sum((U - 0.4) ** 2, axis=1)
    m = gp_fit(U, y, obo.LENGTH_GRID, noise=obo.NOISE)
    best = float(y.min())
    # chains within a few radii of the box's corner
    z = size * rng.uniform(0.1, 4.0, size=(64, d))
    kw = dict(n_global=1, n_local=0, centres=4, radius0=0.1, shrink=0.85, exclusion=2.0 * size, per_step=64)
    dev = lambda a: torch.tensor(a, dtype=torch.float64, device="cuda")
    with Context(0) as ctx:
        props, vmax, nq = ctx.gp_chaos_search(m, best, 0.0, dev(z), None, 64, **kw)
        host, hmax, hq = chaotic_acquire(lambda Q: ctx.gp_ei(m, dev(np.ascontiguousarray(Q)), best, 0.0).cpu().numpy(), z, 64,
                                         None, **kw)
    assert 1 < len(host) < 64  # some points exclude others
    np.testing.assert_array_equal(props.cpu().numpy(), host)
    assert vmax == hmax and nq == hq
