"""A device request submitted while the calling thread's stream has unfinished work, or is being
captured, is copied in and out: its outputs stay as they are until it completes (work on that
stream may still use their memory, recycled by an allocator)."""
import pytest
import torch

from paper_1008_2192_amd import _lib, serving
from test_gpu_server_shared import H, W, drain, frame, new_mask, solo, submit

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["busy", "capturing"])
def test_outputs_are_written_at_completion(kind):
    a = frame(11)
    want = solo(a, 4)
    srv = serving.Server(1 << 30, max_slots=8)
    clean, mask = torch.full_like(a, -1.0), new_mask()
    waits = torch.full((1, 64 * 100), 1000.0, device="cuda")  # one actor of 64 lanes: 100 ms
    _lib.work_run(_lib.CRB_WORK_WAITER, waits[:, :1].contiguous(), workers=1)   # (first call)
    tick = torch.zeros(4, device="cuda")
    torch.cuda.synchronize()
    if kind == "busy":
        _lib.work_run(_lib.CRB_WORK_WAITER, waits, workers=1)
        assert not torch.cuda.current_stream().query()
        submit(srv, a, clean, mask, 4)
    else:
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            tick.add_(1)
            submit(srv, a, clean, mask, 4)
        g.replay()
    srv.poll()                                # admitted, its first round launched
    torch.cuda.synchronize()
    assert (clean == -1.0).all() and (mask == 9).all()
    drain(srv)
    assert torch.equal(clean, want[0]) and torch.equal(mask, want[1])
    if kind == "capturing":
        assert (tick == 1).all()
    srv.close()
