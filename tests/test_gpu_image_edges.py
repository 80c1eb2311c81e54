"""Integral images at the widths where the loads change (below 4 and 16
columns, every remainder of a 16-pixel vector and of a 1024-column tile), at
misaligned images and outputs, and at tile counts around a multiple of eight
(the order in which tiles are handed out), against numpy's double cumsum."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def check(H, W, img_shift=0, out_shift=0):
    import torch

    from paper_2112_10034_amd import cox

    rng = np.random.default_rng(H * 10007 + W)
    img = rng.integers(0, 256, size=(H, W), dtype=np.uint8)
    buf = torch.full((img_shift + H * W,), 255, dtype=torch.uint8, device="cuda")
    buf[img_shift:] = torch.from_numpy(img.reshape(-1)).cuda()
    out = torch.full((out_shift + H * W + 4,), -7, dtype=torch.int32, device="cuda")
    view = out[out_shift:out_shift + H * W].view(H, W)
    print("image", H, W, img_shift, out_shift, flush=True)
    cox.integral_image(buf[img_shift:].view(H, W), out=view)
    want = np.cumsum(np.cumsum(img.astype(np.uint64), 0), 1).astype(np.uint32)
    assert np.array_equal(view.cpu().numpy().view(np.uint32), want), (H, W, img_shift, out_shift)
    assert (out[:out_shift] == -7).all() and (out[out_shift + H * W:] == -7).all()


@pytest.mark.parametrize("W", list(range(1, 34)) + [255, 256, 257, 1019, 1023, 1024, 1025, 1039, 1040, 2047, 2063])
def test_every_remainder(W):
    for H in (1, 5, 64, 67, 130):
        check(H, W)
    check(66, W, img_shift=1 + W % 3)
    check(66, W, out_shift=1)


@pytest.mark.parametrize("H,W", [(64 * 7, 1024), (64 * 8, 1024), (64 * 9 + 1, 1024), (64 * 3, 3 * 1024 + 5),
                                 (64 * 5 + 2, 8 * 1024), (64 * 16, 4000)])
def test_tile_counts(H, W):
    check(H, W)
