"""The farm's tickets where they can go wrong: fewer and more actors than queues, fewer tiles
than queues or actors, tiles that the actors' first runs take entirely, in part or hardly at
all, and blocks with fewer than four actors: every tile once, every record once."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_1008_2192_amd import _lib

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("workers", [1, 2, 31, 32, 33, 127, 1030, 5000])
@pytest.mark.parametrize("th,tw", [(200, 300), (50, 75), (7, 300), (5, 64), (1, 3)])
def test_every_tile_once(workers, th, tw):
    H, W = 200, 300
    rng = np.random.default_rng(workers)
    x = rng.uniform(0, 6, (H, W)).astype(np.float32)
    d = torch.from_numpy(x).cuda()
    got = _lib.farm_image(_lib.CRB_WORK_POISSON, d, seed=3, workers=workers, tile_h=th, tile_w=tw)
    rec = _lib.farm_sources(d, 5.9, 1.0, 1, 1, workers=workers, tile_h=th, tile_w=tw).numpy()
    torch.cuda.synchronize()
    np.testing.assert_array_equal(got.cpu().numpy(), ref.poisson(x, 3))
    np.testing.assert_array_equal(rec, ref.sources(x, 5.9, 1.0, 1, 1).view(_lib.SOURCE_DTYPE))
