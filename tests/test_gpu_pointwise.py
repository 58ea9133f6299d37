"""1x1 layers whose lines are not whole chunks of 8 pixels, whose channels fill no stage, and column stride 2,
against the oracle: the smallest lines of each kind, one past and one short of a chunk, odd widths under a
stride (the last chunk starts a column earlier), rows strided alone, filters past a block, several tiles a block."""
import numpy as np
import pytest

import workloads as wl
from paper_1910_00078_amd import cvx
from parity import run_gpu
from test_gpu_parity import check_case

pytestmark = pytest.mark.gpu


def _c(**kw):
    return wl.small_variant(wl.WORKLOADS["c3a"], **kw)


CASES = [
    _c(name="line8", N=3, C=32, K=32, H=2, W=4),
    _c(name="line9", N=5, C=9, K=33, H=3, W=3),
    _c(name="line49_c339", N=6, C=339, K=65, H=7, W=7),
    _c(name="line121_c8", N=2, C=8, K=130, H=11, W=11),
    _c(name="line63_c1000", N=2, C=1000, K=20, H=7, W=9),
    _c(name="many_tiles", N=40, C=64, K=70, H=29, W=31),
    _c(name="s2_w7", N=3, C=40, K=48, H=8, W=8, stride=(2, 2)),
    _c(name="s2_w9", N=3, C=33, K=100, H=9, W=9, stride=(2, 2)),
    _c(name="s2_w15", N=3, C=64, K=31, H=14, W=15, stride=(2, 2)),
    _c(name="s2_w17", N=9, C=72, K=257, H=17, W=17, stride=(2, 2)),
    _c(name="s2_w16", N=9, C=64, K=64, H=3, W=16, stride=(2, 2)),
    _c(name="s1_2", N=2, C=32, K=32, H=9, W=17, stride=(1, 2)),
    _c(name="s3_1", N=2, C=32, K=32, H=10, W=11, stride=(3, 1)),
    _c(name="s2_1_w8", N=2, C=32, K=32, H=9, W=8, stride=(2, 1)),
]
VARIANTS = ["pointwise_256x64_c32_r5", "pointwise_256x64_c32_r3", "pointwise_128x128_c32_r6", "pointwise_128x256_c32_r6",
            "pointwise_128x64_c32_r6", "pointwise_128x32_c32_r6", "pointwise_128x128_c32_r6_w", "pointwise_256x64_c32_r6_w"]


@pytest.mark.parametrize("dtype", [wl.BF16, wl.F16])
@pytest.mark.parametrize("w", CASES, ids=lambda w: w.name)
def test_lines_channels_strides(w, dtype):
    assert check_case(wl.small_variant(w, dtype=dtype)).startswith("pointwise_")


@pytest.mark.parametrize("stride", [(1, 1), (2, 2)])
@pytest.mark.parametrize("variant", VARIANTS)
def test_every_variant(variant, stride):
    check_case(_c(name="pinned", N=7, C=75, K=150, H=13, W=13, stride=stride), pin=variant, act=cvx.CVX_ACT_LEAKY_RELU, alpha=0.1)


@pytest.mark.parametrize("C", [31, 33, 62, 68, 96, 127, 758])
@pytest.mark.parametrize("variant", VARIANTS[-2:])
def test_streamed_filters_every_remainder(variant, C):
    check_case(_c(name="ws", N=2, C=C, K=70, H=9, W=9), pin=variant)


@pytest.mark.parametrize("pin", [None, VARIANTS[-1]])
def test_infinite_neighbours_stay_out(pin):
    """Ragged channels are not filled from other data: an infinity in the next image or filter must not become a NaN."""
    w = _c(name="inf", N=2, C=33, K=40, H=5, W=5)
    x, wt, b = wl.make_inputs(w)
    clean, _ = run_gpu(w, x, wt, b, pin=pin)
    x, wt = x.copy(), wt.copy()
    inf = 0x7f80                                        # bf16
    x[1] = inf
    wt[1:] = inf
    got, _ = run_gpu(w, x, wt, b, pin=pin)
    np.testing.assert_array_equal(got[0, 0], clean[0, 0])
