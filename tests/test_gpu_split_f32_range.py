"""fp32 layers on the bf16 matrix pipe at the ends of fp32's range: results next to the largest value, and values next to the
smallest, whose parts would fall below bf16's smallest exponent; and infinities and NaNs, which must not make a layer slow either."""
import numpy as np
import pytest

import workloads as wl
from paper_1910_00078_amd import cvx
from parity import run_gpu, run_oracle
from test_gpu_split_f32 import _c, _s1

pytestmark = pytest.mark.gpu

LAYERS = [(_c(N=2, C=20, K=40, H=9, W=9), "64x32_c16_s3"), (_c(N=1, C=16, K=64, H=16, W=16), "256x64_c16_s3"),
          (_s1(N=2, C=40, K=40, H=9, W=8), "128x32_c32_s1"), (_c(N=2, C=20, K=40, H=9, W=9, R=5, S=5, pad=(2, 2)), "32x32_c16_s5")]
IDS = dict(ids=lambda v: v if isinstance(v, str) else "")


@pytest.mark.parametrize("w,pin", LAYERS, **IDS)
@pytest.mark.parametrize("value", [1.8425e19, 1.844e19, 1.9e19])
def test_products_next_to_the_largest_value(w, pin, value):
    """One live product of equal factors for an output: 3.3948e38 is finite, though bf16 rounds its factors to 2^64; the squares
    of larger factors are infinite."""
    x, wt = np.zeros((w.N, w.C, w.H, w.W), np.float32), np.zeros((w.K, w.C, w.R, w.S), np.float32)
    x[:, 3, 4, 4] = value
    x[-1, 3, 2, 5] = -value
    wt[:, 3, w.R // 2, w.S // 2] = value
    wt[5, 3] = 1.0
    got, name = run_gpu(w, x, wt, np.zeros(w.K, np.float32), act=0, pin="tiled_f32_split_" + pin)
    assert name == "tiled_f32_split_" + pin
    with np.errstate(over="ignore"):
        square = float(np.float32(value) * np.float32(value))
    assert got[0, 0, 4, 4] == square and got[-1, 0, 2, 5] == -square and got[0, 5, 4, 4] == float(np.float32(value))
    assert not np.isnan(got).any()


@pytest.mark.parametrize("w,pin", LAYERS, **IDS)
@pytest.mark.parametrize("small,power", [("x", -112), ("x", -119), ("x", -124), ("w", -112), ("w", -119), ("w", -124), ("x", -136), ("w", -136)])
def test_small_values_keep_their_bits(w, pin, small, power):
    """One operand around 2^power, the other so large that results are ordinary.  32-bit sums in any order stay below 1e-6 here
    (the fp32 matrix pipe's error is 3e-7 to 1e-7); below 2^-126 fp32 itself has fewer bits, which the stored inputs already are."""
    x, wt, _ = wl.make_inputs(w)
    x, wt = (np.ldexp(x, power if small == "x" else 100).astype(np.float32), np.ldexp(wt, power if small == "w" else 100).astype(np.float32))
    ref = run_oracle(w, x, wt, np.zeros(w.K, np.float32), act=0, use_bias=False)
    got, name = run_gpu(w, x, wt, None, act=0, use_bias=False, pin="tiled_f32_split_" + pin)
    assert name == "tiled_f32_split_" + pin
    err = np.linalg.norm(got - ref) / np.linalg.norm(ref)
    print("%s %s 2^%d: %.2e" % (pin, small, power, err))
    assert err < 1e-6, err


def _spoil(w, x, wt, what):
    rng = np.random.default_rng(11)
    if what == "x_inf_nan":
        for v in (np.inf, -np.inf, np.nan):
            x[rng.integers(w.N), rng.integers(w.C), rng.integers(w.H), rng.integers(w.W)] = v
    elif what == "w_inf_nan":                      # the padding's zeros are no part of a sum: infinite there, not a NaN
        for v in (np.inf, -np.inf, np.nan):
            wt[rng.integers(w.K), rng.integers(wt.shape[1]), rng.integers(w.R), rng.integers(w.S)] = v
    elif what == "x_large":
        x[:, ::3] *= np.float32(2.0 ** 115)
        wt *= np.float32(2.0 ** -115)
    elif what == "w_large":
        wt[::2] *= np.float32(2.0 ** 120)
        x *= np.float32(2.0 ** -120)
    elif what == "sums_large":
        x *= np.float32(2.0 ** 50)
        wt *= np.float32(2.0 ** 49)
    return x, wt


# pixels and filters short of a tile, an odd channel, waves that split a stage, groups, filters of one column, strides
SPOILT = [(_c(N=2, C=19, K=70, H=13, W=17), "256x64_c16_s3"), (_c(N=3, C=34, K=40, H=7, W=5, groups=2), "64x32_c32_s3"), (_c(N=2, C=33, K=33, H=9, W=11, stride=(2, 2)), "32x32_c32_s3"),
          (_c(N=2, C=16, K=64, H=8, W=9, dil=(2, 2), pad=(2, 2)), "128x32_c16_s3_k2"), (_s1(N=2, C=65, K=70, H=6, W=7), "128x64_c32_s1"), (_s1(N=2, C=37, K=40, H=6, W=5, R=7, pad=(3, 0)), "64x32_c64_s1"),
          (_c(N=2, C=17, K=40, H=9, W=11, R=5, S=5, pad=(2, 2)), "256x32_c16_s5"), (_c(N=2, C=20, K=40, H=9, W=9, R=5, S=5, pad=(2, 2)), "32x32_c16_s5")]


@pytest.mark.parametrize("w,pin", SPOILT, **IDS)
@pytest.mark.parametrize("what", ["x_inf_nan", "w_inf_nan", "x_large", "w_large", "sums_large"])
def test_what_is_not_finite_on_the_bf16_pipe(w, pin, what):
    """As the direct kernel has it, which sums one tap after another and skips the padding."""
    x, wt, b = wl.make_inputs(w)
    x, wt = _spoil(w, x.copy(), wt.copy(), what)
    bn = tuple(np.random.default_rng(5).uniform(lo, hi, w.K).astype(np.float32) for lo, hi in ((0.5, 1.5), (-0.5, 0.5), (-0.3, 0.3), (0.5, 2.0)))
    for kw in (dict(act=cvx.CVX_ACT_IDENTITY), dict(act=cvx.CVX_ACT_LEAKY_RELU, alpha=0.1, bn=bn), dict(act=cvx.CVX_ACT_TANH)):
        got, name = run_gpu(w, x, wt, b, pin="tiled_f32_split_" + pin, **kw)
        want, _ = run_gpu(w, x, wt, b, policy=1, **kw)
        assert name == "tiled_f32_split_" + pin
        np.testing.assert_array_equal(np.isnan(got), np.isnan(want))
        rms = np.sqrt(np.mean(np.square(want[np.isfinite(want)])))
        there = ~np.isnan(want)
        np.testing.assert_allclose(got[there], want[there], rtol=1e-5, atol=1e-5 * rms)


@pytest.mark.parametrize("w", [_c(N=8, C=256, K=256, H=14, W=14), _s1(N=8, C=256, K=256, H=28, W=28)], ids=["3x3", "1x1"])
def test_infinities_and_nans_do_not_make_a_layer_slow(w):
    """A tile with such outputs is summed twice: 2 to 5 times its time.  (Lane by lane and tap by tap it was 60 to 200 times.)"""
    import torch
    x, wt, b = (torch.from_numpy(t).cuda() for t in wl.make_inputs(w))
    y = torch.empty(w.N, w.K, w.Ho, w.Wo, device="cuda")
    plan = cvx.ConvPlan(cvx.CVX_F32, tuple(x.shape), tuple(wt.shape), w.pad, stream=torch.cuda.current_stream().cuda_stream)

    def us():
        marks = [torch.cuda.Event(enable_timing=True) for _ in range(21)]
        for m in marks:
            m.record()
            plan.run(x.data_ptr(), wt.data_ptr(), b.data_ptr(), y.data_ptr())
        torch.cuda.synchronize()
        return sorted(p.elapsed_time(q) for p, q in zip(marks, marks[1:]))[10] * 1e3
    us()
    ordinary = us()
    assert plan.last_kernel().startswith("tiled_f32_split_")
    x[w.N // 2, w.C // 2, 5, 5] = float("inf")
    one = us()
    x.fill_(float("nan"))
    every = us()
    plan.close()
    print("%.1f us, one infinity %.1f, all NaN %.1f" % (ordinary, one, every))
    assert max(one, every) < 15 * ordinary
