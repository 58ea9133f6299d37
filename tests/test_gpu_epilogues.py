"""Every epilogue of the 16-bit matrix kernels -- ReLU and identity on rounded pairs, leaky ReLU (also with slopes outside 0..1),
tanh and logistic, each with and without batch-norm -- on each kernel that has one, against the oracle."""
import numpy as np
import pytest

import workloads as wl
from paper_1910_00078_amd import cvx
from parity import run_gpu, run_oracle, tolerance_ok

pytestmark = pytest.mark.gpu

_c2, _c4 = wl.WORKLOADS["c2"], wl.WORKLOADS["c4"]
LAYERS = [
    (wl.small_variant(_c2, N=3, C=40, K=70, H=9, W=11), "igemm_256x64_c16_3x3"),
    (wl.small_variant(_c2, N=2, C=32, K=40, H=8, W=8), "igemm_64x32_c32_3x3"),
    (wl.small_variant(_c2, N=2, C=32, K=72, H=16, W=16, R=1, S=1, pad=(0, 0)), "pointwise_128x64_c32_r6"),
    (wl.small_variant(_c4, N=1, H=40, W=40), "stem_stream_512x64_k11"),
    (wl.small_variant(_c4, N=1, H=40, W=40), "stem_256x64_k11"),
]
ACTS = [(cvx.CVX_ACT_IDENTITY, 0.0), (cvx.CVX_ACT_RELU, 0.0), (cvx.CVX_ACT_LEAKY_RELU, 0.1), (cvx.CVX_ACT_LEAKY_RELU, -0.5),
        (cvx.CVX_ACT_LEAKY_RELU, 2.0), (cvx.CVX_ACT_TANH, 0.0), (cvx.CVX_ACT_LOGISTIC, 0.0)]


@pytest.mark.parametrize("bn", [False, True], ids=["bias", "bn"])
@pytest.mark.parametrize("act,alpha", ACTS)
@pytest.mark.parametrize("w,pin", LAYERS, ids=[p for _, p in LAYERS])
def test_epilogue(w, pin, act, alpha, bn):
    x, wt, b = wl.make_inputs(w)
    rng = np.random.default_rng(7)
    stats = None
    if bn:
        stats = tuple(rng.uniform(lo, hi, w.K).astype(np.float32) for lo, hi in ((-1.5, 1.5), (-0.5, 0.5), (-0.3, 0.3), (0.5, 2.0)))
    got, name = run_gpu(w, x, wt, b, act=act, alpha=alpha, bn=stats, pin=pin)
    assert name == pin
    ref = run_oracle(w, x, wt, b, act=act, alpha=alpha, bn=None if stats is None else tuple(s.astype(np.float64) for s in stats))
    ok, msg = tolerance_ok(got, ref, w.dtype)
    assert ok, msg


@pytest.mark.parametrize("pin", ["stem_stream_512x64_k11", "stem_256x64_k11", "stem_128x64_k11"])
@pytest.mark.parametrize("rows", [1, 4, 99])
@pytest.mark.parametrize("size", [(40, 48), (41, 47), (9, 27)], ids=str)
def test_stem_tile_heights(pin, rows, size):
    """Rows of whole 16-byte pieces and of others, full tiles and tiles of a few rows, the last one cut off."""
    w = wl.small_variant(_c4, N=2, K=40, H=size[0], W=size[1])
    rows = min(rows, w.Ho, int(pin.split("_")[-2].split("x")[0]) // w.Wo)
    x, wt, b = wl.make_inputs(w)
    got, name = run_gpu(w, x, wt, b, pin="%s,%d" % (pin, rows))
    assert name == pin
    ok, msg = tolerance_ok(got, run_oracle(w, x, wt, b), w.dtype)
    assert ok, msg


@pytest.mark.parametrize("bn", [False, True], ids=["bias", "bn"])
@pytest.mark.parametrize("dtype", [wl.BF16, wl.F16])
@pytest.mark.parametrize("w,pin", LAYERS + [(wl.small_variant(_c4, N=1, H=24, W=24), "stem_128x64_k11")], ids=[p for _, p in LAYERS] + ["stem_128x64_k11"])
def test_relu_of_nan_and_infinity(w, pin, dtype, bn):
    """ReLU makes 0 of a NaN of either sign, be it from x, from the bias or from the batch-norm arrays, in the direct kernel and in
    these; and infinities come out as the direct kernel's."""
    w = wl.small_variant(w, dtype=dtype)
    (x, wt, b), (nan, inf) = wl.make_inputs(w), {wl.BF16: (0x7fc0, 0x7f80), wl.F16: (0x7e00, 0x7c00)}[dtype]
    x, b, rng = x.copy(), b.copy(), np.random.default_rng(7)
    stats = [rng.uniform(lo, hi, w.K).astype(np.float32) for lo, hi in ((-1.5, 1.5), (-0.5, 0.5), (-0.3, 0.3), (0.5, 2.0))] if bn else None
    b.view(np.uint16)[[1, 4]] = nan, nan | 0x8000
    if bn:
        stats[0][3], stats[2][5] = np.nan, -np.nan
    for first in (nan, inf) if w.R < 7 else (None,):        # (the stem's zero weights past its filter meet what lies there)
        if first:
            x.view(np.uint16)[0, 1, 1, 1], x.view(np.uint16)[-1, 2, 5, 6] = first, first | 0x8000
        got, name = run_gpu(w, x, wt, b, bn=stats, pin=pin)
        want, _ = run_gpu(w, x, wt, b, bn=stats, policy=1)
        assert name == pin and not np.isnan(want).any() and np.all(want[:, 1] == 0.0)
        np.testing.assert_array_equal(np.isinf(got), np.isinf(want))
        got[np.isinf(got)] = want[np.isinf(want)] = 0.0
        ok, msg = tolerance_ok(got, want, dtype)
        assert ok, msg
