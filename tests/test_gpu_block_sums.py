"""Block sums and positive counts at the sizes where the kernel's work splits
(groups of 32, 256 and 512 elements, a block of 2048, the two kinds of loads), on
inputs that begin anywhere, with words past the outputs left alone."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shift", [0, 1, 3])
@pytest.mark.parametrize("n", [1, 31, 32, 33, 255, 256, 257, 479, 511, 512, 513, 2047, 2048, 2049, 70001, (1 << 21) - 1,
                               1 << 21, (1 << 21) + 1, (1 << 22) + 513])
def test_sizes(oracle_mod, n, shift):
    import torch

    from paper_2112_10034_amd import cox

    rng = np.random.default_rng(n + shift)
    x = rng.integers(-(1 << 31), 1 << 31, size=n + shift, dtype=np.int64).astype(np.int32)
    x[rng.random(n + shift) < 0.2] = 0
    nb, nw = -(-n // 256), -(-n // 32)
    bs = torch.full((nb + 8,), -7, dtype=torch.int32, device="cuda")
    wc = torch.full((nw + 8,), -7, dtype=torch.int32, device="cuda")
    print("block sums", n, shift, flush=True)
    cox.warp_reduce_blocks_i32(torch.from_numpy(x).cuda()[shift:], bs[:nb], wc[:nw])
    obs, owc = oracle_mod.reduce_blocks_i32(x[shift:])
    assert np.array_equal(bs[:nb].cpu().numpy(), obs) and np.array_equal(wc[:nw].cpu().numpy(), owc)
    assert (bs[nb:] == -7).all() and (wc[nw:] == -7).all()
