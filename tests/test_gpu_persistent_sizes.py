"""Image sizes whose row bands fill an item's LDS in the persistent schedule to the last kilobyte: with one more
element per staged row they would not fit. 281 and 793 pixels (one image at a time), 279 and 341 (an image pair, in
the reverse sweep): the batch runs, and equals the stream-lane schedule to FP32 rounding."""
import numpy as np
import pytest

from gpu_helpers import cands, geom_pair, report

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,with_grad", [(281, False), (793, False), (279, True), (341, True)])
def test_row_bands_fit_the_executor(n, with_grad):
    from paper_2109_11920_amd.api import Context, SliceBatch
    g, _ = geom_pair(n, 4, 64, (n + 3) // 4 * 4)
    S = torch.as_tensor(np.random.default_rng(n).poisson(20.0, (4, 64)), dtype=torch.float32, device="cuda")
    sb = SliceBatch.make(g, S, torch.as_tensor(cands(n, 2), dtype=torch.float32, device="cuda"), with_grad)
    stream = torch.cuda.Stream()
    out = []
    with Context(0) as ctx:
        for mode in ("lanes", "persistent"):
            ctx.set_batch_mode(mode)
            sb.obj.fill_(-1)
            stream.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(stream):
                ctx.evaluate_batch([sb], 0.8, 2, 2)
            stream.synchronize()
            out.append([x.cpu().numpy().copy() for x in (sb.obj, sb.grad) if x is not None])
    assert np.all(out[1][0] > 0)  # written
    report(f"{n} pixels J", out[1][0], out[0][0], 1e-6)
    if with_grad:
        report(f"{n} pixels dJ", out[1][1], out[0][1], 1e-5)
