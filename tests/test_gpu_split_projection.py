"""The projection of few candidates, a ray over 8 lanes, in both its variants (the loads ahead of the image stage in
small launches) against one thread per ray, bit for bit, through a whole evaluation: below, at and above the line
between the variants (64 workgroups of 256 rays on 256 CUs), one chunk of samples to two per lane, paired and not."""
import numpy as np
import pytest

from gpu_helpers import TOL, cands, geom_pair, make_slice, oracle, report

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,na,nb,nt,C", [(8, 4, 8, 7, 1), (32, 63, 32, 32, 8), (32, 65, 32, 32, 8), (64, 127, 64, 64, 2),
                                          (64, 128, 64, 65, 4), (64, 256, 64, 64, 2), (64, 160, 64, 64, 8),
                                          (96, 43, 96, 129, 4), (40, 110, 40, 256, 4)])
def test_split_equals_thread_per_ray(monkeypatch, n, na, nb, nt, C):
    from paper_2109_11920_amd.api import Context
    g, og = geom_pair(n, na, nb, nt)
    S, _ = make_slice(og, seed=n)
    S = S.astype(np.float32)
    th = cands(na, C)
    out = []
    for flag in ("1", "0"):
        monkeypatch.setenv("BOAC_FWD_SPLIT", flag)
        with Context(0) as ctx:
            J, F, _ = ctx.objective(g, torch.as_tensor(S, device="cuda"), torch.as_tensor(th, dtype=torch.float32, device="cuda"),
                                    0.8, 4, want_image=True)
            out.append([J.cpu().numpy(), F.cpu().numpy()])
    np.testing.assert_array_equal(out[0][1], out[1][1])
    np.testing.assert_allclose(out[0][0], out[1][0], rtol=1e-6)  # the same terms in another order
    Jr, Fr = oracle.evaluate(og, S.astype(np.float64), th[-1], float(np.float32(0.8)), 4)[:2]
    report(f"J n={n} na={na}", out[0][0][-1:], [Jr], TOL)
    report(f"image n={n} na={na}", out[0][1][-1], Fr, TOL)
