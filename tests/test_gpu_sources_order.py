"""The device ordering of a SOURCES list against numpy's sort of the same records: frames whose
pixel bitmap ends within a word or a chunk of 1024 words, a record on every pixel, on the first
and the last one, and records outside the frame (left out)."""
import numpy as np
import pytest
import torch

from paper_1008_2192_amd import _lib

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("H,W,n", [(1, 1, 1), (1, 65, 65), (7, 9, 63), (256, 256, 65536),
                                   (257, 256, 1000), (1031, 517, 20000), (3, 70000, 777),
                                   (2048, 2048, 5)])
def test_order_equals_sort(H, W, n):
    rng = np.random.default_rng(H * W + n)
    p = rng.permutation(H * W)[:n]
    if n < H * W:
        p[:2] = (0, H * W - 1)[:min(2, n)]
        p = rng.permutation(np.unique(p))
    rec = np.zeros(len(p), _lib.SOURCE_DTYPE)
    rec["y"], rec["x"] = p // W, p % W
    rec["peak"], rec["npix"] = rng.normal(size=len(p)), rng.integers(0, 99, len(p))
    rec["flux"], rec["sy"], rec["sx"] = rng.normal(size=(3, len(p)))
    src = _lib.SourceList(torch.from_numpy(rec.view(np.uint8).copy()).to(DEV),
                          torch.tensor([len(p)], device=DEV), len(p))
    want = src.numpy()                       # no frame shape: sorted on the host
    src.shape = (H, W)
    assert src.numpy().tobytes() == want.tobytes()
    assert want.tobytes() == rec[np.argsort(p)].tobytes()


def test_records_outside_the_frame_are_left_out():
    rec = np.zeros(4, _lib.SOURCE_DTYPE)
    rec["y"], rec["x"], rec["npix"] = [5, -1, 2, 0], [1, 0, 9, 3], [1, 2, 3, 4]
    d = torch.from_numpy(rec.view(np.uint8).copy()).to(DEV)
    out = torch.zeros_like(d)
    _lib.set_stream()
    _lib.check("crb_sources_order", _lib.lib().crb_sources_order(d.data_ptr(), 4, 6, 9,
                                                                 out.data_ptr()))
    torch.cuda.synchronize()
    got = out.cpu().numpy().view(_lib.SOURCE_DTYPE)
    assert got[:2].tobytes() == rec[[3, 0]].tobytes() and not got[2:].tobytes().strip(b"\0")


def test_arguments():
    d = torch.zeros(80, dtype=torch.uint8, device=DEV)
    o = torch.zeros(80, dtype=torch.uint8, device=DEV)
    f = _lib.lib().crb_sources_order
    assert f(d.data_ptr(), 0, 4, 4, None) == 0
    assert f(d.data_ptr(), 17, 4, 4, o.data_ptr()) == -1
    assert f(d.data_ptr(), 2, 0, 4, o.data_ptr()) == -1
    assert f(d.data_ptr(), 1, 4, 4, d.data_ptr() + 8) == -1
    assert f(d.data_ptr(), 1, 4, 4, o.data_ptr() + 4) == -1
