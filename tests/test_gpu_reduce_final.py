"""The final combine of a reduction: chunk counts around one batch of a
thread (the block's threads for int32, 256 for floats) and around several,
blocks narrower and wider than 256 threads, many calls in a row on one
workspace, bit for bit against the oracle."""
import pytest

from test_gpu_reduce_edges import check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,acc,dot", [("i32", 0, False), ("f32", 0, False), ("f32", 1, False), ("bf16", 1, True)])
@pytest.mark.parametrize("W", [1, 4, 8, 32])
def test_chunk_counts(oracle_mod, dtype, acc, dot, W):
    from paper_2112_10034_amd import cox

    S = 32 * W
    for nch in (2, 31, 32, 33, 64, 65, 128, 129, 255, 256, 257, 1024, 1025, 2049, 8193):
        check(oracle_mod, cox, dtype, nch * S - (nch & 1) * 5, (1, W), acc, dot)
    for n in (3 * S, 300 * S, 2 * S + 1, 257 * S, 40):
        for _ in range(3):
            check(oracle_mod, cox, dtype, n, (1, W), acc, dot)
