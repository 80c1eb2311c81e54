"""Look-back scan and compaction with windows of 64 and 32 words: chunk counts
around one window, several windows and the count from which a wait comes
first, every block width (one of half a wave among them), calls in a row on
one workspace, against the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cfg", [(32, 32), (16, 32), (32, 16), (16, 16), (8, 16), (4, 2), (4, 1), (1, 1)])
def test_chunk_counts(oracle_mod, cfg):
    import torch

    from paper_2112_10034_amd import cox

    S = 32 * cfg[0] * cfg[1]
    rng = np.random.default_rng(S)
    for nch in (1, 2, 31, 33, 63, 64, 65, 66, 128, 129, 193):
        n = nch * S - (nch % 3) * 7
        x = rng.integers(-(1 << 31), 1 << 31, size=n, dtype=np.int64).astype(np.int32)
        print("look-back", cfg, nch, n, flush=True)
        d = torch.from_numpy(x).cuda()
        want = np.asarray(oracle_mod.scan_i32(x, *cfg))
        keep = x[x > 0]
        for _ in range(2):
            got = cox.warp_scan(d, cfg=cfg).cpu().numpy()
            out, count = cox.ballot_compact(d, cfg=cfg)
            assert np.array_equal(got, want)
            assert int(count.cpu()[0]) == keep.size
            assert np.array_equal(out.cpu().numpy()[:keep.size], keep)
