"""The one-kernel setup of a segmented call around its blocks of 32 and 64
segments and the count where one gives way to the other."""
import pytest

from test_gpu_segmented_setup import test_one_kernel_setup as check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["i32", "f32"])
@pytest.mark.parametrize("nseg,k,W", [(31, 1, 2), (32, 1, 4), (33, 2, 1), (63, 1, 8), (65, 1, 1), (4095, 1, 1), (4096, 1, 2),
                                      (4097, 1, 1), (4161, 1, 4)])
def test_blocks(oracle_mod, dtype, nseg, k, W):
    check(oracle_mod, dtype, nseg, k, W)
