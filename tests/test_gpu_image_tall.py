"""Integral images of 1 to 3 columns in 32- and 64-row tiles, against numpy's
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
