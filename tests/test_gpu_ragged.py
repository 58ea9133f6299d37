"""Implicit-GEMM kernels on channel and filter counts that fill neither a stage nor a filter block, against
the oracle: one channel past an octet, past a stage, past a half stage; one filter past a block, one short of
it; the same inside groups, where what follows a group's channels is the next group's data."""
import numpy as np
import pytest

import workloads as wl
from parity import run_gpu
from test_gpu_parity import check_case

pytestmark = pytest.mark.gpu


def _c(**kw):
    return wl.small_variant(wl.WORKLOADS["c2"], **kw)


CASES = [
    _c(name="c9_k65", N=2, C=9, K=65, H=17, W=19),
    _c(name="c31_k63", N=2, C=31, K=63, H=14, W=14),
    _c(name="c33_k64", N=3, C=33, K=64, H=9, W=9),
    _c(name="c65_k129_s2", N=2, C=65, K=129, H=21, W=23, stride=(2, 2)),
    _c(name="c41_groups3", N=2, C=123, K=45, H=13, W=13, groups=3),
    _c(name="c11_5x5", N=2, C=11, K=20, H=12, W=12, R=5, S=5, pad=(2, 2)),
    # pieces that reach over both ends of the tensor: planes smaller than a piece, the last image's and filter's tails
    _c(name="c9_2x2", N=1, C=9, K=9, H=2, W=2),
    _c(name="c8_1x1", N=1, C=8, K=8, H=1, W=1),
    _c(name="c17_3x5_pad3", N=2, C=17, K=33, H=3, W=5, pad=(3, 3)),
    _c(name="c9_groups4", N=2, C=36, K=52, H=12, W=12, groups=4),
    _c(name="c15_5x5_3x3", N=1, C=15, K=7, H=3, W=3, R=5, S=5, pad=(2, 2)),
]


@pytest.mark.parametrize("dtype", [wl.BF16, wl.F16])
@pytest.mark.parametrize("w", CASES, ids=lambda w: w.name)
def test_ragged_channels_and_filters(w, dtype):
    assert check_case(wl.small_variant(w, dtype=dtype)).startswith("igemm_")


@pytest.mark.parametrize("variant", ["igemm_512x64_c32_3x3", "igemm_512x64_c16_3x3", "igemm_256x128_c16_3x3", "igemm_256x64_c32_3x3",
                                     "igemm_256x64_c16_3x3"])
def test_every_3x3_variant(variant):
    check_case(_c(name="pinned", N=3, C=43, K=150, H=12, W=12), pin=variant + ",1,10")


def _f(R, S, **kw):
    return _c(name="%dx%d" % (R, S), R=R, S=S, **kw)


TALL_AND_WIDE = [
    _f(5, 5, N=2, C=16, K=64, H=9, W=40, pad=(2, 2)),
    _f(5, 5, N=3, C=43, K=72, H=35, W=35, pad=(2, 2)),
    _f(5, 5, N=5, C=32, K=33, H=7, W=7, pad=(0, 0)),
    _f(5, 5, N=2, C=48, K=65, H=23, W=21, pad=(4, 4), dil=(2, 2)),
    _f(5, 5, N=2, C=24, K=30, H=20, W=18, pad=(2, 1), stride=(2, 2)),
    _f(5, 5, N=2, C=51, K=42, H=13, W=13, pad=(2, 2), groups=3),
    _f(1, 7, N=2, C=32, K=64, H=17, W=17, pad=(0, 3)),
    _f(1, 7, N=3, C=21, K=70, H=12, W=40, pad=(0, 3)),
    _f(7, 1, N=2, C=64, K=64, H=40, W=12, pad=(3, 0)),
    _f(7, 1, N=3, C=37, K=31, H=15, W=15, pad=(3, 0)),
    _f(7, 1, N=4, C=16, K=48, H=8, W=8, pad=(0, 0)),
    _f(1, 7, N=2, C=48, K=50, H=14, W=30, pad=(1, 6), dil=(1, 2), stride=(2, 1)),
    _f(7, 1, N=2, C=48, K=50, H=30, W=14, pad=(6, 1), dil=(2, 1), stride=(1, 2)),
]


@pytest.mark.parametrize("dtype", [wl.BF16, wl.F16])
@pytest.mark.parametrize("w", TALL_AND_WIDE, ids=lambda w: "%s_c%d_h%d" % (w.name, w.C, w.H))
def test_compiled_filter_sizes(w, dtype):
    assert check_case(wl.small_variant(w, dtype=dtype)).rsplit("_", 1)[1] in ("5x5", "7")


@pytest.mark.parametrize("variant", ["igemm_256x64_c16_7", "igemm_256x64_c32_7", "igemm_64x32_c64_7"])
def test_both_seven_tap_kernels(variant):
    check_case(_f(7, 1, N=3, C=43, K=150, H=12, W=12, pad=(3, 0)), pin=variant + (",1,5" if "64x32" in variant else ",1,10"))


@pytest.mark.parametrize("C", [16, 43, 64])
def test_split_5x5(C):
    check_case(_f(5, 5, N=3, C=C, K=50, H=12, W=14, pad=(2, 2)), pin="igemm_64x32_c32_5x5,1,4")


@pytest.mark.parametrize("dtype", [wl.BF16, wl.F16])
@pytest.mark.parametrize("variant", ["igemm_64x32_c64_3x3", "igemm_64x32_c32_3x3"])
@pytest.mark.parametrize("w,tile", [(_c(name="rows", N=2, C=64, K=32, H=14, W=14), "1,4"), (_c(name="ragged", N=3, C=75, K=33, H=9, W=20), "1,3"),
                                    (_c(name="images", N=5, C=130, K=40, H=5, W=5), "2,5"), (_c(name="one", N=1, C=8, K=9, H=8, W=8), "1,8"),
                                    (_c(name="narrow", N=2, C=96, K=64, H=6, W=3), "1,6"),
                                    (_c(name="s2", N=2, C=70, K=70, H=15, W=13, stride=(2, 2)), "1,8"),
                                    (_c(name="groups", N=2, C=120, K=66, H=7, W=7, groups=3), "1,7")], ids=lambda v: getattr(v, "name", None))
def test_split_reduction(variant, w, tile, dtype):
    check_case(wl.small_variant(w, dtype=dtype), pin=variant + "," + tile)


@pytest.mark.parametrize("pin", ["igemm_256x64_c16_3x3,1,9", "igemm_256x64_c32_3x3,1,9", "igemm_512x64_c16_3x3,1,9", "igemm_64x32_c64_3x3,1,4",
                                 "igemm_256x64_c16_5x5,1,9", "igemm_64x32_c32_5x5,1,4", "igemm_256x64_c16_7,1,9", "igemm_64x32_c64_7,1,4",
                                 "igemm_256x64_c64_1x1,1,9", "igemm_512x64_c32_1x1,1,9", "igemm_256x64_c16_any,1,9"])
def test_infinite_neighbours_stay_out(pin):
    """What is read past a group's channels or a tensor's end must not reach the sum: an infinity in the next group, image or
    filter would turn it into a NaN."""
    R, S = (5, 5) if "5x5" in pin else (7, 1) if "_7" in pin else (1, 1) if "1x1" in pin else (3, 3)
    if "any" in pin:
        R, S = 2, 3
    w = _c(name="inf", N=2, C=78, K=42, H=9, W=9, R=R, S=S, pad=(R // 2, S // 2), groups=2)
    if "any" in pin:
        w = wl.small_variant(w, H=10, pad=(0, 1))
    x, wt, b = wl.make_inputs(w)
    clean, _ = run_gpu(w, x, wt, b, pin=pin)
    x, wt = x.copy(), wt.copy()
    inf = 0x7f80                                        # bf16
    x[1] = inf
    x[0, 39:] = inf
    wt[1:] = inf
    got, _ = run_gpu(w, x, wt, b, pin=pin)
    np.testing.assert_array_equal(got[0, 0], clean[0, 0])
    x2 = x.copy()
    x2[:] = inf
    x2[1, 39:], wt2 = wl.make_inputs(w)[0][1, 39:], wt.copy()
    wt2[:41], wt2[41] = inf, wl.make_inputs(w)[1][41]
    got, _ = run_gpu(w, x2, wt2, b, pin=pin)            # the last image, group and filter, at the tensors' ends
    np.testing.assert_array_equal(got[1, 41], clean[1, 41])
