"""A context keeps its latest launch plans. Its results do not depend on what it planned before: many shapes and
candidate counts in one context (more than it keeps), plan switches turned between calls, the no-allocation call
and both batch schedules in between, each against a context of its own."""
import numpy as np
import pytest

from gpu_helpers import cands, geom_pair

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SWITCHES = ("BOAC_OPPOSED_RAYS", "BOAC_FWD_SPLIT", "BOAC_ATT_SCAN", "BOAC_GATHER_SPLIT")


def _call(ctx, k):
    from paper_2109_11920_amd.api import SliceBatch
    n, na = 32 + 4 * (k % 3), 6 + 2 * (k % 5)
    C = 1 + k % 11
    g, _ = geom_pair(n, na, n, n)
    S = torch.as_tensor(np.random.default_rng(k).poisson(20.0, (na, n)), dtype=torch.float32, device="cuda")
    th = torch.as_tensor(cands(k, C), dtype=torch.float32, device="cuda")
    J, img, _ = ctx.objective(g, S, th, 0.8, 3, want_image=True)
    _, grad, _ = ctx.objective_grad_ex(g, S, th, 0.8, 2, 1)
    Jn, imgn, _ = ctx.objective_noalloc(g, S, th, 0.8, 3, torch.empty(C, device="cuda"),
                                        torch.empty(C, dtype=torch.int32, device="cuda"),
                                        torch.empty(C, n, n, device="cuda"))
    out = [J, img, grad, Jn, imgn]
    stream = torch.cuda.Stream()
    for mode in ("lanes", "persistent"):
        ctx.set_batch_mode(mode)
        sb = SliceBatch.make(g, S, th, False)
        stream.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(stream):
            ctx.evaluate_batch([sb], 0.8, 2, 2)
        stream.synchronize()
        out.append(sb.obj)
    ctx.set_batch_mode("lanes")
    return [x.cpu().numpy().copy() for x in out]


def test_plans_of_earlier_calls_change_nothing(monkeypatch):
    from paper_2109_11920_amd.api import Context
    rng = np.random.default_rng(0)
    with Context(0) as kept:
        for k in list(range(40)) + [0, 7, 39]:
            for name in SWITCHES:
                monkeypatch.setenv(name, str(int(rng.random() < 0.7)))
            got = _call(kept, k)
            with Context(0) as own:
                for a, b in zip(got, _call(own, k)):
                    np.testing.assert_array_equal(a, b)
