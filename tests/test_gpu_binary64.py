"""The binary64 re-evaluation, forced on every work pixel: fewer pixels than a round holds, full
rounds and a rest, at the frame's edges, under each tile height; the codes are those of the
estimates with their bounds, and the mask after them the oracle's."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_1008_2192_amd import _lib

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile_h", [16, 32, 64])
@pytest.mark.parametrize("hits", [1, 2, 4, 30])
@pytest.mark.parametrize("H,W", [(64, 67), (9, 70), (70, 5)])
def test_codes(tile_h, hits, H, W):
    rng = np.random.default_rng(hits * H)
    img = rng.normal(100.0, 10.0, (H, W)).astype(np.float32)
    at = rng.choice(H * W, hits, replace=False)
    img.ravel()[at] += rng.uniform(60, 3000, hits).astype(np.float32)
    img[0, 0] += 900.0
    d = torch.from_numpy(img).cuda()
    p = dict(gain=1.0, readnoise=5.0)
    try:
        _lib.set_single_tuning(tile_h)
        est = _lib.debug_detect(d, exact=False, **p)
        b64 = _lib.debug_detect(d, exact=True, **p)
        _, mask = _lib.lacosmic(d, niter=2, **p)
        torch.cuda.synchronize()
    finally:
        _lib.set_single_tuning()
    assert int((est & 1).sum()) > 0
    assert torch.equal(est, b64)
    np.testing.assert_array_equal(mask.cpu().numpy(), ref.lacosmic(img, niter=2, **p)["mask"])
