"""Integral images of 1 to 3 columns in 32- and 64-row tiles, and of many bands
and segments (the totals of the tiles above and to the left), against numpy's
double cumsum."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def check(H, W):
    import torch

    from paper_2112_10034_amd import cox

    img = np.random.default_rng(H + W).integers(0, 256, size=(H, W), dtype=np.uint8)
    got = cox.integral_image(torch.from_numpy(img).cuda()).cpu().numpy().view(np.uint32)
    want = np.cumsum(np.cumsum(img.astype(np.uint64), 0), 1).astype(np.uint32)
    assert np.array_equal(got, want), (H, W)


# rows per tile change past 64 and 192 tiles of 64 rows
@pytest.mark.parametrize("W", [1, 2, 3])
@pytest.mark.parametrize("H", [4096, 4097, 4129, 12288, 12289, 12343, 70001])
def test_narrow(H, W):
    check(H, W)


# bands x segments: more bands than a batch of the column scan, more segments
# than lanes, in 64-row tiles and in 32-row ones with and without that scan
@pytest.mark.parametrize("H,W", [(64 * 130 + 3, 2 * 1024 + 6), (64 * 259, 1025), (64 * 3, 66 * 1024 + 1),
                                 (70, 66 * 1024 + 5), (64 * 41, 3000), (64 * 40 - 5, 3000), (64 * 9, 64 * 1024)])
def test_bands_and_segments(H, W):
    check(H, W)
