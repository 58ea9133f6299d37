"""Which fp32 layers of a few channels go to the kernel on the bf16 matrix pipe (host only: the kernel search)."""
import ctypes

import pytest

from paper_1910_00078_amd import cvx


@pytest.mark.parametrize("x,w,pad,stride,groups,family", [
    ((32, 64, 56, 56), (64, 64, 3, 3), 1, 1, 1, "tiled_f32_split_"),
    ((11, 7, 11, 5), (15, 7, 5, 5), 2, 1, 1, "tiled_f32_split_"),       # the direct kernel's estimate is three times as long
    ((2, 2, 49, 49), (133, 2, 3, 3), 1, 2, 1, "direct_f32"),            # estimates within their error of each other
    ((41, 8, 5, 11), (208, 2, 3, 3), 1, 3, 4, "direct_f32"),            # groups of a few channels
    ((41, 6, 37, 37), (53, 6, 5, 5), 2, 1, 1, "tiled_f32_128x32_"),     # 5x5 on fewer than half a chunk, several rounds of blocks
    ((30, 5, 25, 25), (69, 5, 5, 5), 2, 1, 1, "tiled_f32_128x32_"),     # 18.5 us, 22.7 split
    ((30, 6, 30, 30), (32, 6, 5, 5), 2, 2, 1, "tiled_f32_split_"),      # one round: 8.9 us, 14.3 tiled
    ((10, 7, 66, 66), (8, 7, 5, 5), 2, 1, 1, "tiled_f32_split_"),       # 17.5 us, 21.1 tiled
])
def test_few_channels_keep_the_kernel_that_is_faster(x, w, pad, stride, groups, family):
    plan = cvx.ConvPlan(cvx.CVX_F32, x, w, (pad, pad), (stride, stride), (1, 1), groups)
    name, ws = ctypes.create_string_buffer(128), ctypes.c_ulonglong()
    status = cvx.lib().cvx_conv_fwd_query(plan.xd, plan.wd, plan.cd, plan.yd, name, 128, ctypes.byref(ws))
    plan.close()
    assert status == 0 and name.value.decode().startswith(family), name.value
