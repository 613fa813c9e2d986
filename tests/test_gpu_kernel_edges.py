"""Kernels chosen by a rule on sizes, at the edges of that rule and at shapes that divide into none of their tiles: the parity
checks of tests/test_gpu_kernels.py (same oracle, same bars), with the kernel that ran named."""
import pytest

from tests import test_gpu_kernels as TK

pytestmark = pytest.mark.gpu


# 64 -> 64 channels over at least 65536 pixels: whole rows of one image to a tile.  Rows that fill a tile, rows that leave a part
# of it, a last tile of one row, images lower than a tile, more rounds of loads for the patch; below and beside the rule: the
# kernel that ran before
@pytest.mark.parametrize("case, kernel", [
    ((16, 64, 64, 64, 64, 3, 1), "conv_narrow64_kernel"),
    ((17, 63, 63, 64, 64, 3, 1), "conv_narrow64_kernel"),
    ((22, 55, 56, 64, 64, 3, 1), "conv_narrow64_kernel"),
    ((69, 31, 31, 64, 64, 3, 1), "conv_narrow64_kernel"),
    ((520, 16, 8, 64, 64, 3, 1), "conv_narrow64_kernel"),
    ((1366, 3, 16, 64, 64, 3, 1), "conv_narrow_kernel<64, 2, 2, 4>"),   # 48 pixels an image: less than half a tile
    ((8, 88, 94, 64, 64, 3, 1), "conv_narrow_kernel<64, 2, 2, 4>"),     # the patch takes more rounds than there are
    ((15, 64, 64, 64, 64, 3, 1), "conv_narrow_kernel<64, 2, 2, 2>"),
])
def test_64_channels_over_many_pixels(case, kernel):
    from paper_1906_09108_amd import kernels as K
    for check in (TK.test_conv_fwd, TK.test_conv_dgrad, TK.test_data_gradient_that_feeds_the_layer_below):
        check(case)
        assert K.fdgk_last_kernel() == kernel
