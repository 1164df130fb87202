"""Synchronous calls (batched, partitioned) and what else runs on their stream: an asynchronous
call from another thread is not held up, a captured crb_lacosmic or farm run keeps the workspace
it was captured with, and streams that come and go leave no memory behind."""
import threading
import time

import numpy as np
import pytest
import torch

from paper_1008_2192_amd import _lib, synth

pytestmark = pytest.mark.gpu
DEV = "cuda"
P = dict(gain=2.0, readnoise=5.0, niter=4)


def item(H, W, seed):
    img = torch.from_numpy(synth.c1_density_frame(H, W, seed, 2.0, 5.0).img).to(DEV)
    return dict(img=img, out_clean=torch.empty_like(img),
                out_mask=torch.empty(img.shape, dtype=torch.uint8, device=DEV), **P)


@pytest.mark.parametrize("call", ["batched", "partitioned"])
def test_an_asynchronous_call_does_not_wait_for_a_synchronous_one(call):
    s = torch.cuda.Stream()
    waits = torch.full((1, 64 * 15), 1e5, device=DEV)          # one actor of 64 lanes: 1.5 s
    it, other = item(100, 130, 1), item(64, 70, 2)

    def synchronous():
        with torch.cuda.stream(s):
            if call == "batched":
                _lib.lacosmic_batched([it], stream=s)
            else:
                _lib.lacosmic_partitioned(it["img"], ny=2, nx=2, border=-1, stream=s, **P)

    def asynchronous():
        _lib.lacosmic(other["img"], out_clean=other["out_clean"], out_mask=other["out_mask"],
                      stream=s, **P)

    synchronous()
    asynchronous()
    _lib.work_run(_lib.CRB_WORK_WAITER, waits[:, :1].contiguous(), workers=1, stream=s)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    _lib.work_run(_lib.CRB_WORK_WAITER, waits, workers=1, stream=s)
    th = threading.Thread(target=synchronous)
    th.start()
    time.sleep(0.3)                          # it waits for the stream by now
    assert th.is_alive()
    asynchronous()
    took = time.perf_counter() - t0
    th.join()
    torch.cuda.synchronize()
    assert took < 1.0, took


def test_captured_calls_keep_their_workspace():
    s = torch.cuda.Stream()
    small, x = item(64, 70, 3), item(200, 300, 4)["img"]
    srcs = _lib.farm_sources(x, 130.0, capacity=4096)
    want_c, want_m = _lib.lacosmic(small["img"], **P)
    torch.cuda.synchronize()
    want_s = srcs.numpy()
    assert len(want_s) > 10
    out = dict(out_clean=small["out_clean"], out_mask=small["out_mask"], stream=s)
    with torch.cuda.stream(s):
        assert _lib.lib().crb_release_workspace(s.cuda_stream) == 0
        _lib.lacosmic(small["img"], **P, **out)              # the stream's workspace
        lst = _lib.farm_sources(x, 130.0, capacity=4096, stream=s)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            _lib.lacosmic(small["img"], **P, **out)
            _lib.farm_sources(x, 130.0, out=lst, stream=s)
        for rep in range(4):
            big = [item(900, 1200, 10 + i) for i in range(1 + rep)]
            _lib.lacosmic_batched(big, stream=s)
            _lib.lacosmic_partitioned(big[0]["img"], ny=2, nx=3, border=-1, stream=s, **P)
            torch.full((1 << 22,), 77, dtype=torch.int32, device=DEV)   # (memory that was freed)
            small["out_clean"].fill_(-1.0)
            small["out_mask"].fill_(7)
            lst.count.zero_()
            lst.records.zero_()
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(small["out_clean"], want_c), rep
            assert torch.equal(small["out_mask"], want_m), rep
            n = int(lst.count.item())
            got = lst.records[:n * _lib.SOURCE_DTYPE.itemsize].cpu().numpy().view(
                _lib.SOURCE_DTYPE)
            got = got[np.lexsort((got["x"], got["y"]))]
            assert got.tobytes() == want_s.tobytes(), rep


def test_reading_a_list_keeps_captured_workspaces():
    s = torch.cuda.Stream()
    small, sky = item(64, 70, 5), torch.zeros(3000, 3000, device=DEV)   # 1.7 MB to order
    sky.view(-1)[::7001] = 50.0
    want = _lib.lacosmic(small["img"], **P)
    out = dict(out_clean=small["out_clean"], out_mask=small["out_mask"], stream=s)
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        assert _lib.lib().crb_release_workspace(s.cuda_stream) == 0
        _lib.lacosmic(small["img"], **P, **out)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            _lib.lacosmic(small["img"], **P, **out)
        for rep in range(3):
            rec = _lib.farm_sources(sky, 10.0, stream=s).numpy()
            assert len(rec) == -(-sky.numel() // 7001)
            p = rec["y"].astype(np.int64) * 3000 + rec["x"]
            np.testing.assert_array_equal(p, np.arange(len(rec)) * 7001)
            torch.full((1 << 22,), 77, dtype=torch.int32, device=DEV)   # (memory that was freed)
            small["out_clean"].fill_(-1.0)
            small["out_mask"].fill_(7)
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(small["out_clean"], want[0]) and torch.equal(small["out_mask"],
                                                                            want[1])


def taken():
    """Device memory in use beyond what torch's allocator holds."""
    free, total = torch.cuda.mem_get_info()
    return total - free - torch.cuda.memory_reserved()


def test_streams_that_come_and_go_leave_no_memory():
    its = [item(2048, 2048, 20 + i) for i in range(12)]        # 46 MB of state in a call
    streams = [torch.cuda.Stream() for _ in range(6)]
    _lib.lacosmic_batched(its, stream=streams[0])
    torch.cuda.synchronize()
    before = taken()
    for s in streams:
        _lib.lacosmic_batched(its, stream=s)
        with torch.cuda.stream(s):
            _lib.lacosmic_partitioned(its[0]["img"], ny=2, nx=2, border=-1, stream=s, **P)
    torch.cuda.synchronize()
    assert taken() - before < 30 << 20        # (not another block per stream)
    # crb_release_workspace gives back what they keep
    assert _lib.lib().crb_release_workspace(streams[0].cuda_stream) == 0
    assert taken() < before - (30 << 20)


def test_sizes_in_any_order_from_threads():
    rng = np.random.default_rng(2)
    its = [item(int(h), int(w), 40 + i) for i, (h, w) in enumerate(rng.integers(20, 700, (12, 2)))]
    want = [_lib.lacosmic(it["img"], **P) for it in its]
    torch.cuda.synchronize()
    errors = []

    def work(t):
        try:
            s = torch.cuda.Stream()
            with torch.cuda.stream(s):
                for i in range(t, len(its), 4):
                    for _ in range(3):
                        its[i]["out_clean"].fill_(-1.0)
                        _lib.lacosmic_batched([its[i]], stream=s)
                        assert torch.equal(its[i]["out_clean"], want[i][0])
                        assert torch.equal(its[i]["out_mask"], want[i][1])
                    if i % 3 == t % 3:
                        assert _lib.lib().crb_release_workspace(s.cuda_stream) == 0
        except Exception as e:      # noqa: BLE001  (reported by the test's thread)
            errors.append(e)

    ts = [threading.Thread(target=work, args=(t,)) for t in range(4)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not errors, errors
