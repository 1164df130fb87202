"""Device requests are cleaned in the caller's buffers, without copies, unless those overlap one
another (other than in place) or a buffer of another request in the server: those are copied in
and out.  Either way the results are crb_lacosmic's bit for bit."""
import ctypes

import numpy as np
import pytest
import torch

from paper_1008_2192_amd import _lib, serving, synth

pytestmark = pytest.mark.gpu
DEV = "cuda"
P = (5.0, 0.0, 4.5, 0.3, 4.0, 4)


def solo(img, gain):
    return _lib.lacosmic(img.clone(), gain, 5.0, niter=4)


def submit(srv, img, H, W, gain, clean, mask):
    rid = ctypes.c_int64(0)
    _lib.check("crb_server_submit", _lib.lib().crb_server_submit(
        srv.handle, img.data_ptr(), H, W, gain, *P, clean.data_ptr(), mask.data_ptr(),
        ctypes.byref(rid)))
    srv._outs[rid.value] = (img, clean, mask)
    return rid.value


def frame(H, W, seed, gain):
    return torch.from_numpy(synth.c1_density_frame(H, W, seed, gain, 5.0).img).to(DEV)


@pytest.mark.parametrize("kind", ["own", "in_place", "shifted", "one_output", "unaligned"])
def test_buffers(kind):
    H, W = 150, 333
    srv = serving.Server(1 << 30, max_slots=8)
    imgs = [frame(H, W, 70 + i, 1.0 + i) for i in range(3)]
    want = [solo(im, 1.0 + i) for i, im in enumerate(imgs)]
    torch.cuda.synchronize()
    for rep in range(2):
        bufs = []
        shared = (torch.empty(H, W, device=DEV), torch.empty(H, W, dtype=torch.uint8, device=DEV))
        for im in imgs:
            if kind == "shifted":              # the output begins one row into the input
                big = torch.empty(H + 1, W, device=DEV)
                big[:H] = im
                img, clean = big[:H], big[1:]
            elif kind == "unaligned":
                big = torch.empty(H * W + 1, device=DEV)
                img, clean = im.clone(), big[1:].view(H, W)
            else:
                img = im.clone()
                clean = img if kind == "in_place" else torch.empty_like(img)
            mask = torch.empty(H * W + 1, dtype=torch.uint8, device=DEV)[1:].view(H, W)
            bufs.append((img, *shared) if kind == "one_output" else (img, clean, mask))
        torch.cuda.synchronize()
        ids = [submit(srv, b[0], H, W, 1.0 + i, b[1], b[2]) for i, b in enumerate(bufs)]
        done = [r[0] for r in srv.drain()]
        torch.cuda.synchronize()
        assert sorted(done) == sorted(ids)
        if kind == "one_output":               # the requests are copied in and out: one wins whole
            assert any(torch.equal(shared[0], c) and torch.equal(shared[1], m) for c, m in want)
            continue
        for (_, clean, mask), (c, m) in zip(bufs, want):
            assert torch.equal(clean, c) and torch.equal(mask, m)
    srv.close()


def test_rounds_of_many_sizes_with_late_arrivals():
    """Frames of 1 to 200 tiles at different iterations share a round's list."""
    sizes = [(20, 30), (64, 64), (33, 65), (300, 417), (700, 600), (1, 90)]
    frames = [frame(H, W, 90 + i, 1.5) for i, (H, W) in enumerate(sizes)]
    want = [solo(f, 1.5) for f in frames]
    torch.cuda.synchronize()
    srv = serving.Server(1 << 30, max_slots=16)
    rng = np.random.default_rng(3)
    ids, out = {}, []
    for i in rng.permutation(np.repeat(np.arange(len(sizes)), 5)):
        ids[srv.submit(frames[i], 1.5, 5.0, niter=4)] = i
        out += srv.poll()
    out += srv.drain()
    assert len(out) == len(ids)
    for rid, _, clean, mask in out:
        c, m = want[ids[rid]]
        assert torch.equal(clean, c) and torch.equal(mask, m), sizes[ids[rid]]
    srv.close()
