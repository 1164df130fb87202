"""The line between replacement by pairs of lanes and by one lane, 128 pixels to replace in a
tile: frames with exactly that many and one more or less (asserted from the oracle's mask), and
windows with a NaN or an infinity in a tile on either side of it, whose replacement values do not
depend on the side."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_1008_2192_amd import _lib

H, W = 32, 64


def background(seed):
    return (100.0 + np.random.default_rng(seed).normal(0.0, 0.5, (H, W))).astype(np.float32)


def hits(n):
    """n separate hits of one pixel each (a grid of 128, then between its places)."""
    img = background(n)
    grid = [(y, x) for y in range(2, H, 4) for x in range(2, W, 4)]
    between = [(y, x) for y in range(4, H, 4) for x in range(4, W, 4)]
    for y, x in (grid + between)[:n]:
        img[y, x] += 3000.0
    return img


def cleaned(img, niter):
    clean, mask = _lib.lacosmic(torch.from_numpy(img).cuda(), 1.0, 5.0, niter=niter)
    torch.cuda.synchronize()
    return clean.cpu().numpy(), mask.cpu().numpy()


COUNTS = [1, 127, 128, 129, 200]
BAD = [np.nan, np.inf, -np.inf]


@pytest.mark.parametrize("n", COUNTS)
def test_counts_of_the_frames(n):
    assert int(ref.lacosmic(hits(n), 1.0, 5.0, niter=1)["mask"].sum()) == n


@pytest.mark.gpu
@pytest.mark.parametrize("n", COUNTS)
def test_either_side_of_the_line(n):
    img = hits(n)
    for niter in (1, 3):
        clean, mask = cleaned(img, niter)
        r = ref.lacosmic(img, 1.0, 5.0, niter=niter)
        np.testing.assert_array_equal(mask, r["mask"])
        np.testing.assert_allclose(clean.astype(np.float64), r["clean"], rtol=1e-5, atol=0)


def few_and_many(bad):
    """A hit with a bad value two pixels away, alone in its tile and with 150 others far off."""
    few = background(3)
    few[6, 6] += 3000.0
    few[6, 8] = bad
    many = few.copy()
    for i in range(150):
        many[2 + 3 * (i % 10), 20 + 2 * (i // 10) + (i % 2)] += 3000.0
    return few, many


@pytest.mark.gpu
@pytest.mark.parametrize("bad", BAD)
def test_bad_values_on_either_side(bad):
    few, many = few_and_many(bad)
    (ca, ma), (cb, mb) = cleaned(few, 1), cleaned(many, 1)
    near = (slice(0, 14), slice(0, 14))
    assert 1 <= ma.sum() <= 128 < mb.sum()
    windows = [(y, x) for y, x in np.argwhere(ma[near]) if abs(y - 6) <= 2 and abs(x - 8) <= 2]
    assert windows
    np.testing.assert_array_equal(ma[near], mb[near])
    np.testing.assert_array_equal(ca[near].view(np.uint32), cb[near].view(np.uint32))
