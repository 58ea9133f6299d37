"""The choice between kernels where a measurement drew the line (host logic, no GPU): each layer with the kernels that may
not serve it, because they were measured slower there, and why."""
import pytest

import workloads as wl
from paper_1910_00078_amd import cvx

CODE = {wl.F32: cvx.CVX_F32, wl.F16: cvx.CVX_F16, wl.BF16: cvx.CVX_BF16}


def kernel(w):
    plan = cvx.ConvPlan(CODE[w.dtype], (w.N, w.C, w.H, w.W), (w.K, w.C // w.groups, w.R, w.S), w.pad, w.stride, w.dil, w.groups)
    try:
        return plan.kernel_name()
    finally:
        plan.close()


def _v(**kw):
    return wl.small_variant(wl.WORKLOADS["c2"], **kw)


@pytest.mark.parametrize("w,slow", [
    # a small tile whose only chunk holds all channels pays its prologue for every 32 or 64 pixels
    (_v(N=37, C=16, H=40, W=40, K=5, dtype=wl.F32), "tiled_f32_64x32"),
    (_v(N=13, C=5, H=25, W=25, K=112, R=5, S=5, pad=(2, 2), dtype=wl.F32), "tiled_f32_32x32"),
    (_v(N=44, C=14, H=31, W=31, K=96, dtype=wl.F32), "tiled_f32_32x32"),
    # its chunk does not fit the 16-byte staging
    (_v(N=18, C=15, H=73, W=73, K=129, stride=(2, 2), dtype=wl.F32), "tiled_f32_128x32_c8"),
    # stages of 64 channels by four producer waves, on lines too short for the pointwise kernel
    (_v(N=5, C=521, H=7, W=7, K=48, R=1, S=1, pad=(0, 0), stride=(1, 2)), "igemm_512x64"),
    (_v(N=16, C=41, H=1, W=1, K=640, R=1, S=1, pad=(0, 0), dtype=wl.F16), "igemm_512x64"),
    # few blocks of the wide tile with streamed filters on short runs of pixels
    (_v(N=2, C=1712, H=40, W=40, K=27, R=1, S=1, pad=(0, 0), stride=(3, 1)), "pointwise_lines_256x64_c32_r6_w"),
    # outputs of a few pixels fill a corner of the grouped kernel's pieces
    (_v(N=14, C=168, H=1, W=1, K=10752, R=5, S=5, pad=(2, 2), groups=56), "grouped"),
    (_v(N=16, C=1309, H=1, W=1, K=1309, R=5, S=5, pad=(2, 2), stride=(2, 2), groups=187), "grouped"),
    (_v(N=9, C=126, H=3, W=3, K=126, stride=(2, 2), groups=126), "grouped"),
    (_v(N=7, C=58, H=1, W=1, K=58, groups=29, dtype=wl.F32), "grouped"),
    # small enough for the direct kernel to deal the channels over lanes
    (_v(N=4, C=40, H=17, W=17, K=40, stride=(2, 2), groups=5, dtype=wl.F32), "grouped"),
    # many filters per group in fp32: the matrix pipe, which reads the input once for 32 of them and more
    (_v(N=24, C=336, H=9, W=9, K=2688, R=5, S=5, pad=(2, 2), stride=(2, 2), groups=42, dtype=wl.F32), "grouped"),
    (_v(N=27, C=320, H=6, W=6, K=20480, groups=40, dtype=wl.F32), "grouped"),
], ids=lambda v: getattr(v, "name", v))
def test_measured_slower_elsewhere(w, slow):
    assert not kernel(w).startswith(slow)


@pytest.mark.parametrize("w", [
    _v(N=32, C=128, H=28, W=28, K=128, groups=128), _v(N=3, C=28, H=7, W=7, K=28, groups=7), _v(N=2, C=12, H=3, W=3, K=12, groups=3),
    _v(N=8, C=64, H=28, W=28, K=64, groups=8, dtype=wl.F32), _v(N=8, C=32, H=14, W=14, K=32, R=5, S=5, pad=(2, 2), groups=8, dtype=wl.F32),
], ids=lambda w: "%s_c%d_h%d" % (w.dtype, w.C, w.H))
def test_few_channels_per_group_keep_their_kernel(w):
    assert kernel(w).startswith("grouped")
