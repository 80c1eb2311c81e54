"""Integral images around the sizes where the height of the scan kernel's
tiles and the kernels of a call change (one segment up to 256 rows, 40
bands, 64 and 192 tiles of 64 rows), at rows that end inside, at and past a
tile, each with random pixels and, for the packed column sums, white ones."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def check(H, W, white=False):
    import torch

    from paper_2112_10034_amd import cox

    rng = np.random.default_rng(H * 10007 + W)
    img = np.full((H, W), 255, np.uint8) if white else rng.integers(0, 256, size=(H, W), dtype=np.uint8)
    out = torch.full((H * W + 4,), -7, dtype=torch.int32, device="cuda")
    print("image", H, W, white, flush=True)
    for _ in range(2):
        cox.integral_image(torch.from_numpy(img).cuda(), out=out[:H * W].view(H, W))
    want = np.cumsum(np.cumsum(img.astype(np.uint64), 0), 1).astype(np.uint32)
    assert np.array_equal(out[:H * W].cpu().numpy().view(np.uint32).reshape(H, W), want), (H, W, white)
    assert (out[H * W:] == -7).all()


@pytest.mark.parametrize("H", [15, 16, 17, 48, 63, 65, 240, 241, 255, 256, 257, 300])
@pytest.mark.parametrize("W", [1, 3, 6, 1000, 1023, 1024, 1025, 2050])
def test_few_rows(H, W):
    check(H, W)


@pytest.mark.parametrize("H,W", [(2559, 2), (2560, 33), (2561, 1001), (2560, 1024), (2625, 1030), (4096, 900),
                                 (4097, 900), (4095, 7), (1025, 3075), (4096, 3000), (4097, 3001), (64, 70000),
                                 (33, 20001)])
def test_bands_and_tiles(H, W):
    check(H, W)


@pytest.mark.parametrize("H,W", [(256, 1024), (256, 1022), (2560, 33), (1000, 1500), (3000, 2000)])
def test_white(H, W):
    check(H, W, white=True)
