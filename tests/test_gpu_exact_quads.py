"""The exact pass with four lanes, two lanes and one lane per quad: tiles whose hits need from
about thirty quads to several hundred, under each tile height (the lines lie at a quarter and a
half of the block's threads) and in the re-evaluation.  Masks are the oracle's; clean values
carry at most one FP32 rounding an iteration, far below 1e-5."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_1008_2192_amd import _lib

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile_h", [16, 32, 64])
@pytest.mark.parametrize("hits", [1, 2, 3, 4, 5, 8, 14, 30, 80])
def test_quads(tile_h, hits):
    H, W = 64, 67                       # one tile of columns, and a rest of three
    rng = np.random.default_rng(hits)
    img = rng.normal(100.0, 10.0, (H, W)).astype(np.float32)
    at = rng.choice(H * W, hits, replace=False)
    img.ravel()[at] += rng.uniform(300, 3000, hits).astype(np.float32)
    try:
        _lib.set_single_tuning(tile_h)
        clean, mask = _lib.lacosmic(torch.from_numpy(img).cuda(), 1.0, 5.0, niter=3)
        torch.cuda.synchronize()
    finally:
        _lib.set_single_tuning()
    r = ref.lacosmic(img, 1.0, 5.0, niter=3)
    np.testing.assert_array_equal(mask.cpu().numpy(), r["mask"])
    np.testing.assert_allclose(clean.cpu().numpy().astype(np.float64), r["clean"], rtol=1e-5, atol=0)
