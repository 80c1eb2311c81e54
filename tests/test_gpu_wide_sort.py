"""Group sorts at the edges of the wide-group kernel (2048 keys a wave, 8192
a block) and of the 32- and 64-key grids' one-round rule, against numpy's
sort of every group."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def want(keys, tile):
    full = keys.size // tile * tile
    return np.concatenate([np.sort(keys[:full].reshape(-1, tile), axis=1).ravel(), np.sort(keys[full:])])


def run(keys, tile, grid=0, in_place=False):
    import torch

    from paper_2112_10034_amd import cox

    d = torch.from_numpy(keys.view(np.int32).copy()).cuda()
    out = cox.tile_sort(d, tile, cfg=(0, 0, grid), out=d if in_place else None)
    return out.cpu().numpy().view(np.uint32)


@pytest.mark.parametrize("tile", [128, 256, 512, 1024])
def test_wide_groups_at_the_edges(tile):
    rng = np.random.default_rng(tile)
    for n in [1, 31, tile - 1, tile, tile + 1, 2047, 2048, 2049, 8191, 8192, 8193, 5 * 8192 + 1027]:
        for kind in range(3):
            keys = rng.integers(0, 1 << 32, n, dtype=np.uint64).astype(np.uint32)
            if kind == 1:
                keys = np.where(keys & 1, np.uint32(0xFFFFFFFF), keys & 3).astype(np.uint32)  # ties, padding's value
            if kind == 2:
                keys = np.sort(keys)[::-1].copy()
            print("wide", tile, n, kind, flush=True)
            w = want(keys, tile)
            assert np.array_equal(run(keys, tile), w), n
            assert np.array_equal(run(keys, tile, grid=2, in_place=True), w), n


@pytest.mark.parametrize("tile", [128, 256, 512, 1024])
def test_wide_groups_sort_every_threshold_input(tile):
    """0/1 inputs with every number of ones, in shuffled, sorted and reversed
    order: a network that sorts 0/1 inputs sorts all."""
    rng = np.random.default_rng(tile)
    rows = []
    for ones in range(tile + 1):
        base = np.zeros(tile, np.uint32)
        base[:ones] = 1
        rows += [base, base[::-1], rng.permutation(base), rng.permutation(base)]
    keys = np.concatenate(rows)
    assert np.array_equal(run(keys, tile), want(keys, tile))


@pytest.mark.parametrize("tile", [32, 64])
def test_one_round_rule(tile):
    import torch

    cus = torch.cuda.get_device_properties(0).multi_processor_count
    rng = np.random.default_rng(tile)
    for n in (1, 5, 4095, 4097, 6 * cus * 4096, 6 * cus * 4096 + 1):
        keys = rng.integers(0, 1 << 32, n, dtype=np.uint64).astype(np.uint32)
        print("one round", tile, n, flush=True)
        assert np.array_equal(run(keys, tile), want(keys, tile)), n
