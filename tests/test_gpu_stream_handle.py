"""GPU: the stream that a call without one takes is the calling thread's current
torch stream, whichever that is, and its results are ordered on it."""
import threading

import pytest

from test_gpu_parity import agg  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("other", [False, True])
def test_current_stream(agg, other):
    import torch
    side = torch.cuda.Stream() if other else torch.cuda.default_stream()
    x = torch.ones(1 << 20, dtype=torch.int32, device="cuda")
    out = torch.zeros(32, dtype=torch.uint8, device="cuda")
    plan = agg.Plan("i32", "sum", max_n=x.numel())
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        assert agg._stream_handle(None) == torch.cuda.current_stream().cuda_stream == side.cuda_stream
        seen = []
        t = threading.Thread(target=lambda: seen.extend([agg._stream_handle(None),
                                                         torch.cuda.current_stream().cuda_stream]))
        t.start()
        t.join()
        assert seen[0] == seen[1]
        for k in range(2, 5):
            x.add_(1)
            plan.enqueue(x, out)
        assert out.view(torch.int64)[0].item() == 4 * x.numel()
    assert agg._stream_handle(side) == agg._stream_handle(side.cuda_stream) == side.cuda_stream
