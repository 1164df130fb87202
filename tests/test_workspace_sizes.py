"""The workspace a frame is charged (crb_workspace_bytes, which also decides what
crb_lacosmic_noalloc takes and what a server admits): five bytes a pixel and nine a summary tile
of 32 x 64 pixels, whatever the frame's shape, in 256-byte pieces with 12 KiB of counters."""
import pytest

from paper_1008_2192_amd import _lib


def al(x):
    return (x + 255) // 256 * 256


def charged(H, W):
    n, tiles = H * W, ((H + 31) // 32) * ((W + 63) // 64)
    return al(n) + al(4 * n) + al(8 * 1024) + al(4 * 1024) + al(tiles) + 2 * al(4 * tiles)


@pytest.mark.parametrize("side", list(range(1, 18)) + [31, 32, 33, 63, 64, 65, 100])
def test_size_follows_the_pixels(side):
    for other in [1, 2, 5, 31, 32, 33, 64, 65, 127, 128, 129, 255, 256, 257, 500, 1000, 1023, 1024,
                  2047, 2048, 2049, 4096, 5000, 10000, 100000, 1000001, 2000000, 16777216]:
        for H, W in ((side, other), (other, side)):
            assert _lib.workspace_bytes(H, W) == charged(H, W), (H, W)


def test_long_frames_fit_the_fixed_scratch():
    for H, W in ((2000000, 1), (1, 2000000), (19000000, 1), (1, 19000000), (3, 6000000)):
        assert _lib.workspace_bytes(H, W) <= 96 << 20, (H, W)
