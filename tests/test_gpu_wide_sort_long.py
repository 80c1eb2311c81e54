"""Group sorts on both sides of the length from which the wide-group kernel
takes over (2^21 keys for groups of 128 and 256, 2^20 for 512 and 1024): its
edges (2048 keys a wave, 8192 a block), few blocks, in place, ties with the
padding's value, and 0/1 inputs with every number of ones (a network that sorts
those sorts all), against numpy's sort of every group."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

TILES = [128, 256, 512, 1024]


def check(keys, tile, grid=0, in_place=False):
    import torch

    from paper_2112_10034_amd import cox

    full = keys.size // tile * tile
    want = np.concatenate([np.sort(keys[:full].reshape(-1, tile), axis=1).ravel(), np.sort(keys[full:])])
    d = torch.from_numpy(keys.view(np.int32).copy()).cuda()
    out = cox.tile_sort(d, tile, cfg=(0, 0, grid), out=d if in_place else None)
    assert np.array_equal(out.cpu().numpy().view(np.uint32), want), (keys.size, tile, grid, in_place)


@pytest.mark.parametrize("tile", TILES)
def test_edges(tile):
    least = 1 << (21 if tile <= 256 else 20)
    rng = np.random.default_rng(tile)
    for extra in (-1, 0, 1, tile - 1, tile + 1, 2047, 2049, 8191, 8192, 8193, 5 * 8192 + 1027):
        keys = rng.integers(0, 1 << 32, least + extra, dtype=np.uint64).astype(np.uint32)
        if extra % 2:
            keys = np.where(keys & 1, np.uint32(0xFFFFFFFF), keys & 3).astype(np.uint32)
        check(keys, tile)
    check(keys, tile, grid=2, in_place=True)


@pytest.mark.parametrize("tile", TILES)
def test_every_threshold_input(tile):
    rng = np.random.default_rng(tile)
    rows = []
    while len(rows) * tile <= 1 << 21:
        for ones in range(tile + 1):
            base = np.zeros(tile, np.uint32)
            base[:ones] = 1
            rows += [base, base[::-1], rng.permutation(base), rng.permutation(base)]
    check(np.concatenate(rows), tile)
