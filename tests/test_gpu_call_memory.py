"""The synchronous calls keep their memory with the stream: batches and partitions of growing
and shrinking sizes, interleaved with single frames on the same stream, from two threads, and
after the workspace was released, all give crb_lacosmic's results."""
import ctypes
import threading

import torch
import pytest

from paper_1008_2192_amd import _lib, synth

pytestmark = pytest.mark.gpu
DEV = "cuda"
P = dict(gain=2.0, readnoise=5.0, niter=4)


def items(sizes, seed):
    out = []
    for i, (H, W) in enumerate(sizes):
        img = torch.from_numpy(synth.c1_density_frame(H, W, seed + i, 2.0, 5.0).img).to(DEV)
        out.append(dict(img=img, out_clean=torch.full_like(img, -1.0),
                        out_mask=torch.full(img.shape, 7, dtype=torch.uint8, device=DEV), **P))
    return out


def check(its):
    _lib.lacosmic_batched(its)
    for it in its:
        c, m = _lib.lacosmic(it["img"], **P)
        torch.cuda.synchronize()
        assert torch.equal(c, it["out_clean"]) and torch.equal(m, it["out_mask"])


BATCHES = [[(40, 70)], [(300, 417), (64, 64), (33, 97)], [(512, 700)] * 3, [(5, 5), (90, 31)]]


def test_growing_and_shrinking_calls():
    for rep in range(2):
        for b, sizes in enumerate(BATCHES):
            its = items(sizes, 10 * b)
            check(its)
            img = its[0]["img"]
            c, m = _lib.lacosmic_partitioned(img, ny=min(3, img.shape[0]), nx=2, border=-1, **P)
            assert torch.equal(c, its[0]["out_clean"]) and torch.equal(m, its[0]["out_mask"])
        s = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
        assert _lib.lib().crb_release_workspace(s) == 0


def test_two_threads_on_their_streams_and_on_one():
    errors = []

    def work(stream, seed):
        try:
            with torch.cuda.stream(stream):
                for _ in range(3):
                    for sizes in BATCHES[:3]:
                        check(items(sizes, seed))
        except Exception as e:      # noqa: BLE001  (reported by the test's thread)
            errors.append(e)

    one = torch.cuda.Stream()
    for streams in ([torch.cuda.Stream(), torch.cuda.Stream()], [one, one]):
        ts = [threading.Thread(target=work, args=(s, 100 * i)) for i, s in enumerate(streams)]
        for t in ts:
            t.start()
        for t in ts:
            t.join()
        assert not errors, errors
