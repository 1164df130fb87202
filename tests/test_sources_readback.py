"""Reading a SOURCES list back: records that were moved to host memory are sorted there, and so
are those of a device without memory to sort them in; lists on either side of the length from
which the device sorts them read the same."""
import numpy as np
import pytest
import torch

from paper_1008_2192_amd import _lib

H, W = 200, 300


def records(n, seed=1):
    rng = np.random.default_rng(seed)
    p = rng.permutation(H * W)[:n]
    rec = np.zeros(n, _lib.SOURCE_DTYPE)
    rec["y"], rec["x"] = p // W, p % W
    rec["peak"], rec["flux"] = rng.normal(size=n), rng.normal(size=n)
    return rec, rec[np.argsort(p)].tobytes()


def source_list(rec, device):
    s = _lib.SourceList(torch.from_numpy(rec.view(np.uint8).copy()).to(device),
                        torch.tensor([len(rec)], device=device), len(rec))
    s.shape = (H, W)
    return s


@pytest.mark.parametrize("n", [0, 1, 5000])
def test_records_in_host_memory(n):
    rec, want = records(n)
    assert source_list(rec, "cpu").numpy().tobytes() == want


@pytest.mark.gpu
@pytest.mark.parametrize("n", [1, 639, 640, 641, 5000])
def test_either_side_of_the_line(n):
    rec, want = records(n)
    assert source_list(rec, "cuda").numpy().tobytes() == want


@pytest.mark.gpu
@pytest.mark.parametrize("what", ["output", "workspace"])
def test_no_device_memory_left(monkeypatch, what):
    rec, want = records(5000)
    s = source_list(rec, "cuda")

    def none_left(*args, **kw):
        if what == "output":
            raise torch.cuda.OutOfMemoryError("none left")
        raise _lib.CrbError("crb_sources_order", _lib.CRB_ENOMEM, "none left")

    if what == "output":
        monkeypatch.setattr(torch, "empty_like", none_left)
    else:
        monkeypatch.setattr(_lib, "check", none_left)
        monkeypatch.setattr(_lib, "set_stream", lambda stream=None: None)
    assert s.numpy().tobytes() == want


@pytest.mark.gpu
@pytest.mark.parametrize("h,w,n", [(1, 1, 1), (1, 65, 65), (7, 9, 63), (2048, 2048, 5)])
def test_short_lists_by_the_device(h, w, n):
    """crb_sources_order itself, at lengths that SourceList leaves to the host."""
    p = np.random.default_rng(n).permutation(h * w)[:n]
    rec = np.zeros(n, _lib.SOURCE_DTYPE)
    rec["y"], rec["x"], rec["sx"] = p // w, p % w, np.arange(n)
    src = torch.from_numpy(rec.view(np.uint8).copy()).cuda()
    out = torch.zeros_like(src)
    _lib.set_stream()
    _lib.check("crb_sources_order", _lib.lib().crb_sources_order(src.data_ptr(), n, h, w,
                                                                 out.data_ptr()))
    torch.cuda.synchronize()
    assert out.cpu().numpy().tobytes() == rec[np.argsort(p)].tobytes()
