"""Group sorts whose last round is cut by n: inside a vector, a row, a block,
and rounds in which some blocks have no keys, for every number of keys per
lane, against numpy's sort of every group."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

FORMS = [(1, 32), (2, 32), (4, 32), (8, 32), (16, 32), (1, 64), (4, 64), (1, 128), (1, 256)]


@pytest.mark.parametrize("k,tile", FORMS)
def test_cut_rounds(k, tile):
    import torch

    from paper_2112_10034_amd import cox

    rng = np.random.default_rng(100 * tile + k)
    round_keys = 256 * k * (1 if k >= 16 else min(16 // k, 4))
    sizes = {1, 2, k + 1, tile - 1, tile + 1, 255 * k + 1, 256 * k - 1, 256 * k + 1, round_keys - 1, round_keys + 1}
    sizes |= {3 * round_keys + r for r in range(2 * k + 1)} | {4 * round_keys + 1}
    for n in sorted(sizes):
        keys = rng.integers(0, 1 << 32, n, dtype=np.uint64).astype(np.uint32)
        keys[rng.random(n) < 0.1] = 0xFFFFFFFF  # the padding's value
        full = n // tile * tile
        want = np.concatenate([np.sort(keys[:full].reshape(-1, tile), axis=1).ravel(), np.sort(keys[full:])])
        for grid in (0, 2):
            d = torch.full((n + 4,), 7, dtype=torch.int32, device="cuda")  # what lies past n stays
            d[:n] = torch.from_numpy(keys.view(np.int32)).cuda()
            out = torch.full((n + 4,), 9, dtype=torch.int32, device="cuda")
            cox.tile_sort(d[:n], tile, cfg=(k, 0, grid), out=out[:n])
            assert np.array_equal(out[:n].cpu().numpy().view(np.uint32), want), (n, grid)
            assert (out[n:] == 9).all(), (n, grid)
            cox.tile_sort(d[:n], tile, cfg=(k, 0, grid), out=d[:n])
            assert np.array_equal(d[:n].cpu().numpy().view(np.uint32), want), (n, grid)
            assert (d[n:] == 7).all(), (n, grid)
