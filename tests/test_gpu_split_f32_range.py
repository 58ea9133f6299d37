"""fp32 layers on the bf16 matrix pipe at the ends of fp32's range: results next to the largest value, and values next to the
smallest, whose parts would fall below bf16's smallest exponent."""
import numpy as np
import pytest

import workloads as wl
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
