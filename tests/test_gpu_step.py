"""The iteration kernel (grow, mask, replacement and the next codes in one launch) against the
FP64 oracle where its tiling can go wrong: hits on the edges and corners of the 32 x 64 tiles
(whose halos each block recomputes), frames whose last tiles are one row or column, clusters
whose inner pixels have no unflagged neighbour, tiles with more pixels to replace than the
kernel lists, and iterations that keep finding new pixels.  Every entry point takes its own
route through it: one frame (tile lists from iteration 2 on), a plan, a plan with counting on
(every tile, every iteration), the server (frames of one launch at different iterations,
cleaned in place).

Masks and counts are exact; a replaced pixel is an exact FP32 selection or the once-rounded
mean of two, so niter roundings of 2^-24 stay far below the 1e-5 used throughout."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_1008_2192_amd import _lib, serving, synth

pytestmark = pytest.mark.gpu
DEV = "cuda"


def edge_frame(H, W, seed):
    """Noise, with hits along every tile edge and across every tile corner of the frame."""
    rng = np.random.default_rng(seed)
    img = (100.0 + rng.normal(0.0, 11.0, (H, W))).astype(np.float32)
    for y in range(0, H, 32):
        for x in range(0, W, 64):
            for dy, dx in ((0, 0), (-1, -1), (0, -1), (-1, 0), (-4, 5), (5, -4), (16, -2), (-2, 20)):
                a, b = y + dy, x + dx
                n = int(rng.integers(1, 9))
                if rng.random() < 0.5:
                    img[max(a, 0):max(a + n, 0), max(b, 0):max(b + 1, 0)] += rng.uniform(200, 4000)
                else:
                    img[max(a, 0):max(a + 1, 0), max(b, 0):max(b + n, 0)] += rng.uniform(200, 4000)
    return np.ascontiguousarray(img)


DEFAULT = dict(gain=1.0, readnoise=5.0, sky=0.0, sigclip=4.5, sigfrac=0.3125, objlim=4.0)
GREEDY = dict(gain=1.0, readnoise=5.0, sky=0.0, sigclip=0.5, sigfrac=0.0, objlim=0.0625)

CASES = [(H, W, DEFAULT, 4) for H, W in ((33, 65), (64, 128), (65, 129), (95, 191), (160, 257),
                                         (31, 63), (1, 130), (70, 1), (2, 2))]
CASES += [(97, 193, GREEDY, 3), (64, 128, GREEDY, 6), (40, 70, dict(DEFAULT, sigclip=1.5,
                                                                     sigfrac=0.0), 8)]


def check(img, p, niter, early_stop, clean, mask, stats=None):
    r = ref.lacosmic(img, niter=niter, early_stop=early_stop, **p)
    np.testing.assert_array_equal(mask.cpu().numpy(), r["mask"])
    np.testing.assert_allclose(clean.cpu().numpy().astype(np.float64), r["clean"], rtol=1e-5,
                               atol=0)
    if stats:
        assert stats == dict(iters_run=r["iters"], n_flagged=int(r["mask"].sum()))
    return r


@pytest.mark.parametrize("H,W,p,niter", CASES)
def test_single_frame_and_plan(H, W, p, niter):
    img = edge_frame(H, W, 7 * H + W)
    d = torch.from_numpy(img).to(DEV)
    for early in (True, False):
        clean, mask = _lib.lacosmic(d, niter=niter, early_stop=early, **p)
        torch.cuda.synchronize()
        r = check(img, p, niter, early, clean, mask)
        if p is GREEDY and not early:      # more to replace in a tile than the kernel lists
            assert max(r["mask"][y:y + 40, x:x + 72].sum() for y in range(0, H, 32)
                       for x in range(0, W, 64)) > 1024
    inplace = d.clone()
    _lib.lacosmic(inplace, niter=niter, out_clean=inplace, early_stop=False, **p)
    torch.cuda.synchronize()
    assert torch.equal(inplace, clean)


@pytest.mark.parametrize("graph", [False, True])
def test_batch_plain_and_counting(graph):
    frames = [(edge_frame(H, W, 7 * H + W), p, niter) for H, W, p, niter in CASES]
    items = []
    for i, (img, p, niter) in enumerate(frames):
        d = torch.from_numpy(img).to(DEV)
        items.append(dict(img=d, out_clean=torch.empty_like(d), niter=niter, early_stop=i % 2 == 0,
                          out_mask=torch.empty(img.shape, dtype=torch.uint8, device=DEV),
                          incremental=i % 3 == 0, **p))
    plan = _lib.Plan(items, use_graph=graph)
    for counting in (False, True, False):
        plan.set_counting(counting)
        for _ in range(2):
            for it in items:
                it["out_clean"].fill_(-1.0)
                it["out_mask"].fill_(7)
            plan.run()
            stats = plan.stats()
            for i, ((img, p, niter), it) in enumerate(zip(frames, items)):
                check(img, p, niter, i % 2 == 0, it["out_clean"], it["out_mask"], stats[i])
    plan.close()


def test_server_rounds_mix_iterations():
    """Frames large enough that a tile's block starts while its neighbours have already listed
    it for the next iteration, at different iterations in one launch."""
    rng = np.random.default_rng(5)
    frames = [synth.c1_density_frame(1024, 1024, 300 + i, float(np.float32(1.0 + i)), 5.0)
              for i in range(3)] + [synth.c1_density_frame(300, 417, 400, 2.0, 5.0)]
    want = []
    for f in frames:
        d = torch.from_numpy(f.img).to(DEV)
        want.append(_lib.lacosmic(d, f.gain, f.readnoise, niter=4))
    torch.cuda.synchronize()
    srv = serving.Server(1 << 32, max_slots=8)
    for rep in range(3):
        ids, out = {}, []
        for i in rng.permutation(np.repeat(np.arange(len(frames)), 3)):
            f = frames[i]
            ids[srv.submit(torch.from_numpy(f.img).to(DEV), f.gain, f.readnoise, niter=4)] = i
            out += srv.poll()
        out += srv.drain()
        for rid, _, clean, mask in out:
            c, m = want[ids[rid]]
            assert torch.equal(mask, m) and torch.equal(clean, c), (rep, ids[rid])
    srv.close()
