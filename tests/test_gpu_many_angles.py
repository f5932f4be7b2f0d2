"""Few candidates at many angles: the 8 x 8-tile gather holds the sums of at most 4096 angles in LDS and takes more
in rounds, so any admitted angle count runs (held sums of every angle asked for more LDS than there is above 4456
to 4776 angles). The last single round and the first second one, odd counts and pairing off up to the limit of 8192
angles, bin windows of one to three, against 16 x 16 tiles (same arithmetic: the same bits) and the FP64 oracle."""
import numpy as np
import pytest

import oracle
from gpu_helpers import TOL, geom_pair, report

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,na,nb,nt,C,pair", [(32, 513, 32, 32, 1, "1"), (32, 1025, 32, 32, 8, "1"), (32, 4095, 32, 32, 1, "1"),
                                               (33, 4097, 33, 35, 2, "1"), (32, 4801, 32, 32, 1, "1"),
                                               (32, 8192, 32, 32, 2, "0"), (32, 8192, 32, 32, 1, "1"),
                                               (33, 4461, 58, 32, 1, "1"), (32, 4803, 64, 33, 1, "1")])
def test_any_angle_count(monkeypatch, n, na, nb, nt, C, pair):
    from paper_2109_11920_amd.api import Context
    monkeypatch.setenv("BOAC_OPPOSED_RAYS", pair)
    g, og = geom_pair(n, na, nb, nt)
    rng = np.random.default_rng(na)
    mu = rng.uniform(0.0, 0.1, (C, n, n)).astype(np.float32)
    z = rng.uniform(0.2, 2.0, (C, na, nb)).astype(np.float32)
    out = []
    for flag in ("1", "0"):
        monkeypatch.setenv("BOAC_GATHER_SPLIT", flag)
        with Context(0) as ctx:
            out.append(ctx.backproject(g, torch.as_tensor(mu, device="cuda"), torch.as_tensor(z, device="cuda")).cpu().numpy())
    np.testing.assert_array_equal(out[0], out[1])
    att = oracle.attenuation(og, mu[-1].astype(np.float64))
    report(f"backproject {na} angles", out[0][-1], oracle.backproject(og, att, z[-1].astype(np.float64)), TOL)
