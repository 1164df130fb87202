"""POISSON on tiles whose pixels fill a wave's chunks (16 pixels a lane) partly, exactly and
several times, narrower and wider than a wave, in place and not: the oracle's deviates."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_1008_2192_amd import _lib

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W,th,tw", [(40, 30, 40, 30), (32, 32, 32, 32), (33, 97, 16, 64),
                                       (70, 65, 70, 1), (5, 2100, 1, 2100), (64, 64, 1, 63)])
def test_tiles(H, W, th, tw):
    x = np.random.default_rng(H * W).uniform(0, 30, (H, W)).astype(np.float32)
    d = torch.from_numpy(x).cuda()
    want = ref.poisson(x, 7)
    got = _lib.farm_image(_lib.CRB_WORK_POISSON, d, seed=7, workers=5, tile_h=th, tile_w=tw)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(got.cpu().numpy(), want)
    _lib.farm_image(_lib.CRB_WORK_POISSON, d, seed=7, workers=5, tile_h=th, tile_w=tw, out=d)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(d.cpu().numpy(), want)
