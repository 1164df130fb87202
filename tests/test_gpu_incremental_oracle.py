"""Runs with the incremental option (single frame, partitioned with a border that reproduces the
whole frame, batch) against the FP64 oracle: masks and counts exact, cleaned values within a few
FP32 roundings."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_1008_2192_amd import _lib, synth

pytestmark = pytest.mark.gpu
P = dict(gain=1.5, readnoise=5.0, sky=0.0, sigclip=4.5, sigfrac=0.3125, objlim=4.0)


@pytest.mark.parametrize("H,W", [(61, 67), (200, 333)])
@pytest.mark.parametrize("call", ["single", "partitioned", "batched"])
def test_incremental_equals_oracle(H, W, call):
    img = synth.c1_density_frame(H, W, H, 1.5, 5.0).img
    r = ref.lacosmic(img, niter=4, **P)
    d = torch.from_numpy(img).cuda()
    if call == "single":
        clean, mask = _lib.lacosmic(d, niter=4, incremental=True, **P)
    elif call == "partitioned":
        clean, mask = _lib.lacosmic_partitioned(d, ny=2, nx=3, border=-1, niter=4,
                                                incremental=True, **P)
    else:
        clean, mask = torch.empty_like(d), torch.empty((H, W), dtype=torch.uint8, device="cuda")
        stats = _lib.lacosmic_batched([dict(img=d, out_clean=clean, out_mask=mask, niter=4,
                                            incremental=True, **P)])
        assert stats == [dict(iters_run=r["iters"], n_flagged=int(r["mask"].sum()))]
    torch.cuda.synchronize()
    assert r["mask"].any()
    np.testing.assert_array_equal(mask.cpu().numpy(), r["mask"])
    np.testing.assert_allclose(clean.cpu().numpy().astype(np.float64), r["clean"], rtol=1e-5,
                               atol=0)
