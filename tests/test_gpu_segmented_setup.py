"""The one-kernel setup of a segmented call (at most 15 * 1024 segments) at
its own edges: blocks of 256 segments, the count's rounds of 1024 segments a
block, descriptors written by a wave or by a whole block, every class, and
the first count that takes the three-kernel setup."""
import numpy as np
import pytest

from paper_2112_10034_amd import inputs

pytestmark = pytest.mark.gpu


def layout(nseg, S, seed):
    """Empty, one-element, short and a few long segments; with room for it
    one segment of more than 1024 chunks."""
    rng = np.random.default_rng(seed)
    lens = rng.integers(0, S + 1, size=nseg)
    lens[rng.random(nseg) < 0.1] = 0
    lens[rng.integers(0, nseg, size=1 + nseg // 50)] = rng.integers(S + 1, 6 * S, size=1 + nseg // 50)
    lens[nseg // 2] = 1030 * S + 7
    return np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)


@pytest.mark.parametrize("dtype", ["i32", "f32"])
@pytest.mark.parametrize("nseg,k,W", [(1, 1, 1), (2, 1, 2), (255, 1, 4), (256, 2, 2), (257, 1, 8), (1023, 1, 1),
                                      (1025, 1, 16), (5121, 1, 2), (15360, 1, 1), (15361, 1, 1)])
def test_one_kernel_setup(oracle_mod, dtype, nseg, k, W):
    import torch

    from paper_2112_10034_amd import cox

    off = layout(nseg, 32 * k * W, 7 * nseg + W)
    xi, xf = inputs.segment_values(int(off[-1]), seed=nseg)
    x = xi if dtype == "i32" else xf
    print("setup", dtype, nseg, k, W, "n", off[-1], flush=True)
    want = oracle_mod.segmented(x, off, k, W)
    xg, og = torch.from_numpy(x).cuda(), torch.from_numpy(off).cuda()
    for _ in range(2):  # the second call finds the first one's workspace
        got = cox.segmented(xg, og, 7, cfg=(k, W))
        for g, w, what in zip(got, want, ("totals", "scan", "compaction", "counts")):
            assert g.cpu().numpy().tobytes() == np.ascontiguousarray(w).tobytes(), what


def test_one_kernel_setup_malformed_offsets():
    """Offsets outside [0, n] and reversed ones give what the same offsets,
    clamped, give (a reversed segment is empty)."""
    import torch

    from paper_2112_10034_amd import cox

    n = 5000
    x = torch.arange(1, n + 1, dtype=torch.int32, device="cuda")
    bad = torch.tensor([-7, 100, 40, 40, 3000, 9000, 9000], dtype=torch.int64, device="cuda")
    tot, _, _, cnt = cox.segmented(x, bad, 5, cfg=(1, 2))
    pairs = [(0, 100), (100, 100), (40, 40), (40, 3000), (3000, n), (n, n)]
    assert tot.cpu().tolist() == [sum(range(a + 1, b + 1)) for a, b in pairs]
    assert cnt.cpu().tolist() == [b - a for a, b in pairs]
    cox.workspace(cox.OP_SEGMENTED, cox.I32, n, 6, cfg=(1, 2)).status()
