"""The kernels that large layers run, pinned on small tensors against the oracle: on their own, tensors of this size go to
the small tiles.  Every epilogue of each, both 16-bit types, whole images and rows, ragged channels and filters, and the
shapes of the reduced layers."""
import numpy as np
import pytest

import workloads as wl
from paper_1910_00078_amd import cvx
from parity import to_device
from test_gpu_parity import SMALL, check_case

pytestmark = pytest.mark.gpu


def _v(base, **kw):
    return wl.small_variant(wl.WORKLOADS[base], **kw)


def run_pinned(w, variant, **kw):
    """check_case on the largest tile of the variant that takes the problem."""
    if not variant.startswith("igemm_"):
        return check_case(w, pin=variant, **kw)
    pt = int(variant[6:variant.index("x")])
    whole = w.Ho * w.Wo <= pt
    for t in range(min(w.N, pt // (w.Ho * w.Wo)) if whole else min(w.Ho, pt // w.Wo), 0, -1):
        try:
            return check_case(w, pin="%s,%d,%d" % ((variant, t, w.Ho) if whole else (variant, 1, t)), **kw)
        except cvx.CvxError as e:
            assert e.status == cvx.CVX_ERR_UNSUPPORTED
    raise AssertionError("no tile of %s takes the problem" % variant)


def _bn(K):
    rng = np.random.default_rng(9)
    bn = (rng.uniform(0.5, 1.5, K), rng.uniform(-0.5, 0.5, K), rng.uniform(-0.3, 0.3, K), rng.uniform(0.5, 2.0, K))
    return tuple(t.astype(np.float32).astype(np.float64) for t in bn)


EPILOGUES = [dict(act=cvx.CVX_ACT_IDENTITY, use_bias=False), dict(bias_f32=True), dict(act=cvx.CVX_ACT_LEAKY_RELU, alpha=0.1),
             dict(act=cvx.CVX_ACT_TANH), dict(act=cvx.CVX_ACT_LOGISTIC), dict(bn=True, eps=1e-3),
             dict(bn=True, eps=1e-3, act=cvx.CVX_ACT_LOGISTIC, use_bias=False)]

K3 = ["igemm_512x64_c32_3x3", "igemm_512x64_c16_3x3", "igemm_256x128_c16_3x3", "igemm_256x64_c32_3x3", "igemm_256x64_c16_3x3",
      "igemm_256x64_c16_3x3_u2"]
K1 = ["igemm_512x64_c32_1x1", "igemm_512x64_c64_1x1", "igemm_256x64_c32_1x1", "igemm_256x64_c64_1x1", "igemm_128x128_c64_1x1"]
POINTWISE = ["pointwise_256x64_c32_r5", "pointwise_256x64_c32_r3", "pointwise_128x128_c32_r6", "pointwise_128x256_c32_r6"]
F32 = ["tiled_f32_256x64_c8_3x3", "tiled_f32_128x64_c8_3x3", "tiled_f32_256x64_c16_1x1", "tiled_f32_256x64_c8", "tiled_f32_128x64_c8",
       "tiled_f32_128x32_c8"]

ROWS = _v("c2", name="rows", N=2, C=64, K=96, H=20, W=24)
RUNS = _v("c2", name="runs_7x7", N=6, C=32, K=80, H=7, W=7)             # planes of an odd size, staged as runs of y
RUNS4 = _v("c2", name="runs_14x14", N=2, C=43, K=72, H=14, W=14)        # planes of a multiple of 4; ragged channels
ONE = _v("c3a", name="1x1", N=3, C=64, K=96, H=12, W=14)


@pytest.mark.parametrize("dtype", [wl.BF16, wl.F16])
@pytest.mark.parametrize("w", [ROWS, RUNS, RUNS4], ids=lambda w: w.name)
@pytest.mark.parametrize("variant", K3)
def test_every_epilogue_3x3(variant, w, dtype):
    if variant == "igemm_512x64_c32_3x3" and w is ROWS:
        w = wl.small_variant(w, H=8, W=24)                               # two stages of more rows exceed LDS
    for kw in EPILOGUES:
        kw = dict(kw, bn=_bn(w.K)) if kw.get("bn") else kw
        assert run_pinned(wl.small_variant(w, dtype=dtype), variant, **kw) == variant


@pytest.mark.parametrize("dtype", [wl.BF16, wl.F16])
@pytest.mark.parametrize("variant", POINTWISE)
def test_every_epilogue_1x1(variant, dtype):
    for kw in EPILOGUES:
        kw = dict(kw, bn=_bn(ONE.K)) if kw.get("bn") else kw
        check_case(wl.small_variant(ONE, dtype=dtype), pin=variant, **kw)


@pytest.mark.parametrize("variant", F32)
def test_every_epilogue_f32(variant):
    w = wl.small_variant(ONE if variant.endswith("1x1") else ROWS, dtype=wl.F32)
    for kw in EPILOGUES:
        kw = dict(kw, bn=_bn(w.K)) if kw.get("bn") else kw
        assert check_case(w, pin=variant, **kw) == variant


# ---- the reduced layers of the parity tests on the kernels that serve such layers at full size ----
def _is3x3(w):
    return w.dtype != wl.F32 and (w.R, w.S) == (3, 3) and w.C // w.groups >= 8


@pytest.mark.parametrize("w", [w for w in SMALL if _is3x3(w)], ids=lambda w: w.name)
def test_reduced_3x3_layers(w):
    assert run_pinned(w, "igemm_256x64_c16_3x3") == "igemm_256x64_c16_3x3"


@pytest.mark.parametrize("variant", ["pointwise_256x64_c32_r5", "pointwise_128x256_c32_r6"])
@pytest.mark.parametrize("w", [w for w in SMALL if w.dtype != wl.F32 and w.R * w.S == 1 and w.groups == 1 and w.C <= 128], ids=lambda w: w.name)
def test_reduced_1x1_layers(w, variant):
    assert check_case(w, pin=variant).startswith("pointwise_")


@pytest.mark.parametrize("w", [w for w in SMALL if w.dtype == wl.F32 and w.R * w.S < 49 and w.C >= 8], ids=lambda w: w.name)
def test_reduced_f32_layers(w):
    assert check_case(w, pin="tiled_f32_128x32_c8") == "tiled_f32_128x32_c8"


# ---- 1x1 layers that the pointwise kernel does not take: padded, grouped, wide strides, short lines ----
@pytest.mark.parametrize("dtype", [wl.BF16, wl.F16])
@pytest.mark.parametrize("w", [
    _v("c3a", name="padded", N=3, C=64, K=70, H=10, W=11, pad=(1, 1)), _v("c3a", name="padded_c43", N=3, C=43, K=64, H=9, W=9, pad=(0, 2)),
    _v("c3a", name="groups4", N=2, C=256, K=96, H=12, W=12, groups=4), _v("c3a", name="groups3_c75", N=5, C=225, K=99, H=5, W=5, groups=3),
    _v("c3a", name="stride3", N=4, C=96, K=130, H=13, W=16, stride=(3, 3)), _v("c3a", name="plane6_c100", N=9, C=100, K=40, H=2, W=3),
], ids=lambda w: w.name)
@pytest.mark.parametrize("variant", K1)
def test_igemm_1x1(variant, w, dtype):
    assert run_pinned(wl.small_variant(w, dtype=dtype), variant) == variant


@pytest.mark.parametrize("w", [_v("c3a", name="padded", N=2, C=64, K=40, H=28, W=28, pad=(1, 1)), _v("c3a", name="groups4", N=8, C=256, K=64, H=28, W=28, groups=4),
                               _v("c3a", name="plane7", N=40, C=128, K=64, H=1, W=7),
                               _v("c3a", name="w7_s2", N=9, C=72, K=64, H=9, W=7, stride=(2, 2))], ids=lambda w: w.name)
def test_layers_past_the_pointwise_kernels_bounds(w):
    assert check_case(w).startswith("igemm_")


# ---- fp32 rows too short for 16-byte pieces: element-wise staging ----
NARROW = [_v("c2", name="w3", N=9, C=24, K=40, H=17, W=3, dtype=wl.F32), _v("c2", name="w2_c21", N=7, C=21, K=70, H=20, W=2, dtype=wl.F32),
          _v("c2", name="w1", N=16, C=40, K=64, H=9, W=1, dtype=wl.F32), _v("c2", name="w3_groups3", N=4, C=75, K=66, H=12, W=3, groups=3, dtype=wl.F32),
          _v("c2", name="w3_s2", N=9, C=33, K=65, H=19, W=3, stride=(2, 2), dtype=wl.F32)]


@pytest.mark.parametrize("variant", [v for v in F32 if not v.endswith("1x1")])
@pytest.mark.parametrize("w", NARROW, ids=lambda w: w.name)
def test_f32_staged_by_elements(w, variant):
    assert check_case(w, pin=variant) == variant


@pytest.mark.parametrize("variant", ["tiled_f32_256x64_c16_1x1", "tiled_f32_256x64_c8", "tiled_f32_128x64_c8", "tiled_f32_128x32_c8"])
@pytest.mark.parametrize("w", NARROW[:4], ids=lambda w: w.name)
def test_f32_staged_by_elements_1x1(w, variant):
    assert check_case(wl.small_variant(w, R=1, S=1, pad=(0, 0)), pin=variant) == variant


@pytest.mark.parametrize("R", [1, 3])
def test_f32_staged_by_elements_on_its_own(R):
    w = _v("c2", name="64x3", N=64, C=64, K=64, H=64, W=3, R=R, S=R, pad=(R // 2, R // 2), dtype=wl.F32)
    assert check_case(w).startswith("tiled_f32_")


# ---- groups of few channels that only the generic kernel takes ----
@pytest.mark.parametrize("dtype", [wl.BF16, wl.F16, wl.F32])
@pytest.mark.parametrize("w", [_v("c2", name="depthwise_7x7", N=2, C=12, K=12, H=11, W=13, R=7, S=7, pad=(3, 3), groups=12),
                               _v("c2", name="depthwise_dilated", N=2, C=16, K=32, H=14, W=14, pad=(2, 2), dil=(2, 2), groups=16),
                               _v("c2", name="stride_1_2", N=2, C=20, K=15, H=9, W=16, stride=(1, 2), groups=5)], ids=lambda w: w.name)
def test_groups_on_the_generic_kernel(w, dtype):
    assert check_case(wl.small_variant(w, dtype=dtype)) == "direct_" + dtype


def test_repeated_runs_of_the_large_kernels_are_bit_identical():
    import torch
    for w, pin in [(_v("c2", N=2), "igemm_512x64_c16_3x3,1,9"), (_v("c5b", N=2), "igemm_256x128_c16_3x3,1,14"),
                   (_v("c5a", N=10, C=64), "igemm_256x64_c32_3x3,2,7"), (_v("c3a", N=2), "pointwise_256x64_c32_r5"),
                   (_v("c3b", N=2), "pointwise_128x256_c32_r6"), (_v("c2", N=2, dtype=wl.F32), "tiled_f32_256x64_c8_3x3")]:
        x, wt, b = wl.make_inputs(w)
        dx, dw, db = to_device(x, w.dtype), to_device(wt, w.dtype), to_device(b, w.dtype)
        outs = [cvx.conv_fwd_fused(dx, dw, db, pad=w.pad, stride=w.stride, dil=w.dil, pin=pin) for _ in range(3)]
        torch.cuda.synchronize()
        bits = torch.int32 if w.dtype == wl.F32 else torch.int16
        for o in outs[1:]:
            assert torch.equal(o.view(bits), outs[0].view(bits)), pin
