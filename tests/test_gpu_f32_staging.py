"""fp32 layers whose image rows are not whole 16-byte pieces and whose channels fill no chunk, against the oracle: rows
of one piece, one past it and one short of the next; one channel past and short of a chunk; filters past a block;
what follows a group's channels being the next group's data."""
import numpy as np
import pytest

import workloads as wl
from parity import run_gpu
from test_gpu_parity import check_case

pytestmark = pytest.mark.gpu


def _c(**kw):
    return wl.small_variant(wl.WORKLOADS["c2"], dtype=wl.F32, **kw)


CASES = [
    _c(name="w4", N=9, C=33, K=40, H=21, W=4),
    _c(name="w5", N=9, C=31, K=65, H=13, W=5),
    _c(name="w7", N=17, C=24, K=64, H=7, W=7),
    _c(name="w13_5x5", N=4, C=19, K=33, H=13, W=13, R=5, S=5, pad=(2, 2)),
    _c(name="w12_5x5", N=3, C=48, K=80, H=12, W=12, R=5, S=5, pad=(2, 2)),
    _c(name="w42_1x1", N=3, C=50, K=94, H=42, W=42, R=1, S=1, pad=(0, 0)),
    _c(name="w31_s2", N=3, C=41, K=70, H=31, W=31, stride=(2, 2)),
    _c(name="w23_1x1_s2", N=5, C=72, K=130, H=23, W=23, R=1, S=1, pad=(0, 0), stride=(2, 2)),
    _c(name="w14_groups", N=5, C=51, K=66, H=14, W=14, groups=3),
    _c(name="w56_c9", N=1, C=9, K=64, H=40, W=56),
    _c(name="one_image", N=1, C=118, K=144, H=25, W=25, R=1, S=1, pad=(0, 0)),
    _c(name="one_image_3x3", N=1, C=67, K=90, H=14, W=14),
]


@pytest.mark.parametrize("w", CASES, ids=lambda w: w.name)
def test_rows_and_channels(w):
    assert check_case(w).startswith("tiled_f32_")


def test_infinite_neighbours_stay_out():
    """An infinity in the next filter or image must not reach a ragged chunk."""
    w = _c(name="inf", N=2, C=33, K=40, H=21, W=21)
    x, wt, b = wl.make_inputs(w)
    clean, _ = run_gpu(w, x, wt, b)
    x, wt = x.copy(), wt.copy()
    x[1] = np.inf
    wt[1:] = np.inf
    got, name = run_gpu(w, x, wt, b)
    assert name.startswith("tiled_f32_")
    np.testing.assert_array_equal(got[0, 0], clean[0, 0])


SMALL = ["tiled_f32_128x32_c4", "tiled_f32_64x32_c16", "tiled_f32_64x32_c8", "tiled_f32_32x32_c16", "tiled_f32_32x32_c8"]


@pytest.mark.parametrize("variant", SMALL + ["tiled_f32_64x32_c16_3x3", "tiled_f32_32x32_c16_3x3"])
@pytest.mark.parametrize("C", [16, 43])
def test_split_reduction_3x3(variant, C):
    check_case(_c(name="small", N=3, C=C, K=50, H=15, W=13), pin=variant)


@pytest.mark.parametrize("variant", ["tiled_f32_128x32_c4", "tiled_f32_64x32_c8", "tiled_f32_32x32_c8"])
def test_split_reduction_5x5(variant):
    check_case(_c(name="small", N=3, C=21, K=40, H=13, W=14, R=5, S=5, pad=(2, 2), stride=(1, 2)), pin=variant)


@pytest.mark.parametrize("variant", SMALL)
def test_split_reduction_1x1(variant):
    check_case(_c(name="small", N=3, C=50, K=33, H=5, W=6, R=1, S=1, pad=(0, 0)), pin=variant)
