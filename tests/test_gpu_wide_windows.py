"""Detectors finer than the pixels (bin windows of two and three) in the column-group gather are no less accurate
than in the general kernel: the reconstruction after many iterations, where both operators' roundings add up,
against the FP64 oracle. Both runs hold every angle. The two differ in the order of their sums, so their errors
do by a few percent; a window summed in one run was 15 to 32% further off."""
import json

import numpy as np
import pytest

import oracle
from gpu_helpers import cands, f32, geom_pair, make_slice, rel_l2

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,na,nb,nt,C", [(48, 20, 62, 48, 2), (40, 16, 76, 40, 2), (40, 16, 76, 40, 12)])
def test_no_further_off_than_the_general_kernel(monkeypatch, tmp_path, n, na, nb, nt, C):
    from paper_2109_11920_amd.api import Context
    monkeypatch.setenv("BOAC_OPPOSED_RAYS", "0")
    g, og = geom_pair(n, na, nb, nt)
    plan = tmp_path / "general.json"
    plan.write_text(json.dumps({f"back:{n}x{na}x{nb}x{nt}:{C}:0": [16, 16, 1, 1, 0]}))
    off = {"column groups": [], "general": []}
    for seed in (31, 32, 33):
        S = f32(make_slice(og, seed=seed, counts=5e7)[0])
        th = cands(seed, C)
        ref = [oracle.evaluate(og, S, th[c], 0.8, 200)[1] for c in range(2)]
        for name, cache in (("column groups", tmp_path / "none.json"), ("general", plan)):
            with Context(0, tune_cache=str(cache)) as ctx:
                F = ctx.objective(g, torch.as_tensor(S, dtype=torch.float32, device="cuda"),
                                  torch.as_tensor(th, dtype=torch.float32, device="cuda"), 0.8, 200, want_image=True)[1]
            off[name] += [rel_l2(F[c].cpu().numpy(), ref[c]) for c in range(2)]
    mean = {k: float(np.mean(v)) for k, v in off.items()}
    print(f"[parity] image after 200 iterations: {mean}", flush=True)
    assert mean["column groups"] <= 1.1 * mean["general"]
