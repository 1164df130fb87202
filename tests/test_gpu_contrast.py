"""The contrast test's three routes against the FP64 oracle: one wave per pixel (at most 16
pixels of a tile), med3 shared by the windows (more), and the pixels beyond a tile's list in
their own lanes; on frames whose tiles hold few, many and too many, at the frame's edges, under
each tile height.  Masks are exact; clean values carry at most one FP32 rounding an iteration,
far below 1e-5."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_1008_2192_amd import _lib, synth

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("tile_h", [16, 32, 64])
@pytest.mark.parametrize("H,W,cover", [(40, 70, 0.01), (40, 70, 0.08), (64, 128, 0.05),
                                       (97, 201, 0.03), (97, 201, 0.2), (5, 300, 0.1),
                                       (200, 3, 0.1)])
def test_contrast_routes(tile_h, H, W, cover):
    f = synth.render(H, W, H + W, sky_e=100.0, gain=1.0, readnoise=5.0, n_stars=H * W // 500,
                     star_fwhm=2.0, star_flux="lognormal", hit_coverage=cover, hit_len=(1, 8),
                     hit_amp=(300.0, 5000.0))
    d = torch.from_numpy(f.img).to(DEV)
    try:
        _lib.set_single_tuning(tile_h)
        clean, mask = _lib.lacosmic(d, 1.0, 5.0, niter=3)
        torch.cuda.synchronize()
    finally:
        _lib.set_single_tuning()
    r = ref.lacosmic(f.img, 1.0, 5.0, niter=3)
    np.testing.assert_array_equal(mask.cpu().numpy(), r["mask"])
    np.testing.assert_allclose(clean.cpu().numpy().astype(np.float64), r["clean"], rtol=1e-5, atol=0)
