"""Float32 dot products with 32 elements per lane, whose chunks are loaded in
two halves: several chunks a block, the block's last one, a ragged tail in
either half, bit for bit against the oracle."""
import numpy as np
import pytest

from paper_2112_10034_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("acc", [0, 1])
@pytest.mark.parametrize("W,G", [(1, 0), (1, 3), (8, 2), (32, 0), (32, 1)])
def test_halves(oracle_mod, acc, W, G):
    import torch

    from paper_2112_10034_amd import cox

    S = 1024 * W
    for n in (S, 2 * S, 5 * S, 5 * S + S // 4 + 3, 4 * S + 3 * S // 4 + 1, 7 * S - 1):
        _, _, x = inputs.primitive_inputs(n, seed=n)
        _, _, y = inputs.primitive_inputs(n, seed=n + 1)
        p, t = oracle_mod.dot(x, y, 32, W, acc)
        tot, part = cox.warp_dot(torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda(), acc, cfg=(32, W, G))
        assert part.cpu().numpy().tobytes() == np.ascontiguousarray(p).tobytes(), n
        assert tot.cpu().numpy().view(np.uint64)[0] == np.float64(t).view(np.uint64), n
