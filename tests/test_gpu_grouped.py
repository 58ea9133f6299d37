"""The register-tiled kernel for few channels per group against the oracle, where it can go wrong: output
widths around its 16-byte pieces, images smaller than the filter's reach, row counts around its tiles,
depth multipliers, filter blocks that end inside a group, both strides, all types and epilogues."""
import numpy as np
import pytest

import workloads as wl
from paper_1910_00078_amd import cvx
from parity import run_gpu, run_oracle
from test_gpu_parity import check_case

pytestmark = pytest.mark.gpu


def _g(**kw):
    return wl.small_variant(wl.WORKLOADS["c2"], **kw)


CASES = [
    _g(name="wide_padding", N=1, C=6, K=6, H=3, W=5, groups=6, pad=(4, 30)),
    _g(name="narrow_7", N=3, C=12, K=12, H=7, W=7, groups=12),
    _g(name="exact_8", N=2, C=12, K=12, H=9, W=8, groups=12),
    _g(name="shifted_last_piece", N=2, C=9, K=9, H=13, W=17, groups=9),
    _g(name="stride2_odd", N=3, C=10, K=10, H=15, W=31, groups=10, stride=(2, 2)),
    _g(name="no_padding", N=2, C=8, K=8, H=12, W=21, groups=8, pad=(0, 0)),
    _g(name="depth_multiplier_3", N=2, C=6, K=18, H=11, W=19, groups=6),
    _g(name="four_per_group", N=3, C=24, K=24, H=14, W=14, groups=6),
    _g(name="six_of_four_filters", N=2, C=15, K=30, H=10, W=23, groups=5),
    _g(name="seven_per_group_s2", N=2, C=28, K=28, H=19, W=18, groups=4, stride=(2, 2)),
    _g(name="five_by_five", N=2, C=7, K=7, H=16, W=20, R=5, S=5, pad=(2, 2), groups=7),
    _g(name="five_by_five_s2", N=2, C=7, K=7, H=17, W=29, R=5, S=5, pad=(2, 2), groups=7, stride=(2, 2)),
]


@pytest.mark.parametrize("dtype", [wl.BF16, wl.F16, wl.F32])
@pytest.mark.parametrize("w", CASES, ids=lambda w: w.name)
def test_grouped_shapes(w, dtype):
    assert check_case(wl.small_variant(w, dtype=dtype)).startswith("grouped_")


@pytest.mark.parametrize("dtype", [wl.BF16, wl.F16, wl.F32])
@pytest.mark.parametrize("rows", [1, 4])
def test_both_tile_heights(dtype, rows):
    w = _g(name="heights", N=2, C=6, K=6, H=10, W=12, groups=6, dtype=dtype)
    check_case(w, pin="grouped_%s_3x3_s1_k1r%d" % (dtype, rows))


# narrower outputs than the kernel is chosen for: nearly all of a piece lies outside the image
NARROW = [
    _g(name="one_pixel", N=2, C=20, K=20, H=1, W=1, groups=20),
    _g(name="two_columns", N=3, C=12, K=12, H=5, W=2, groups=12),
    _g(name="three_columns", N=1, C=10, K=10, H=3, W=3, groups=5),
]


@pytest.mark.parametrize("dtype", [wl.BF16, wl.F16, wl.F32])
@pytest.mark.parametrize("rows", [1, 4])
@pytest.mark.parametrize("w", NARROW, ids=lambda w: w.name)
def test_narrow_outputs(w, rows, dtype):
    check_case(wl.small_variant(w, dtype=dtype), pin="grouped_%s_3x3_s1_k1r%d" % (dtype, rows))


def test_epilogues_and_unaligned_buffers():
    w = _g(name="epilogues", N=2, C=16, K=16, H=9, W=14, groups=4)
    rng = np.random.default_rng(3)
    bn = (rng.uniform(0.5, 1.5, w.K), rng.uniform(-0.5, 0.5, w.K), rng.uniform(-0.3, 0.3, w.K), rng.uniform(0.5, 2.0, w.K))
    bn = tuple(t.astype(np.float32).astype(np.float64) for t in bn)
    for act, alpha in [(cvx.CVX_ACT_IDENTITY, 0.0), (cvx.CVX_ACT_LEAKY_RELU, 0.1), (cvx.CVX_ACT_TANH, 0.0), (cvx.CVX_ACT_LOGISTIC, 0.0)]:
        check_case(w, act=act, alpha=alpha)
    check_case(w, bn=bn, eps=1e-3)
    check_case(w, use_bias=False)
    check_case(w, bias_f32=True)
    for off in [(1, 0, 0), (0, 1, 0), (0, 0, 1)]:
        assert check_case(w, offsets=off).startswith("grouped_")


INF = {wl.BF16: 0x7f80, wl.F16: np.float16(np.inf), wl.F32: np.float32(np.inf)}


@pytest.mark.parametrize("dtype", [wl.BF16, wl.F16, wl.F32])
@pytest.mark.parametrize("where", ["input", "weight", "both"])
@pytest.mark.parametrize("w", [_g(name="3x3", N=2, C=8, K=8, H=12, W=20, groups=8), _g(name="3x3_s2", N=2, C=8, K=16, H=11, W=19, groups=4, stride=(2, 2)),
                               _g(name="5x5", N=2, C=6, K=6, H=13, W=17, R=5, S=5, pad=(2, 2), groups=6),
                               _g(name="four_filters", N=1, C=8, K=24, H=9, W=10, groups=2)], ids=lambda w: w.name)
def test_an_infinity_reaches_exactly_the_outputs_it_is_part_of(w, where, dtype):
    """Padding and the zeros that fill up a pair of taps are no part of the sum: an infinite input gives infinities of the
    weight's sign, an infinite weight leaves the border outputs finite whose tap lies outside the image."""
    w = wl.small_variant(w, dtype=dtype)
    x, wt, b = wl.make_inputs(w)
    x, wt = x.copy(), wt.copy()
    if where in ("input", "both"):
        x[0, 1, 4, 7] = x[-1, -1, -1, -1] = x[0, 0, 0, 0] = INF[dtype]
    if where in ("weight", "both"):
        wt[1, 0, 0, 0] = wt[-1, -1, -1, -1] = INF[dtype]
    got, name = run_gpu(w, x, wt, b, act=cvx.CVX_ACT_IDENTITY)
    assert "grouped_" in name
    with np.errstate(invalid="ignore"):
        want = run_oracle(w, x, wt, b, act=cvx.CVX_ACT_IDENTITY)
    for test in (np.isnan, np.isposinf, np.isneginf):
        np.testing.assert_array_equal(test(got), test(want))
    ok = np.isfinite(want)
    assert 0 < ok.sum() < ok.size
    # one rounding to the output type of sums of up to 100 products of order one
    rms = np.sqrt(np.mean(want[ok] ** 2))
    assert np.all(np.abs(got[ok] - want[ok]) <= {wl.F32: 1e-5, wl.F16: 2e-3, wl.BF16: 1e-2}[dtype] * (np.abs(want[ok]) + 0.1 * rms))
