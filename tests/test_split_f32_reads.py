"""The loads of the fp32 kernel on the bf16 matrix pipe stay inside x and w by their own addresses, whatever the hardware's range
check does with the scalar part of one: channels and filters short of a chunk, rows and planes shorter than a 16-byte piece, column strides (host only:
the addresses are computed as the kernel computes them).  And what such pieces hold is right (on the GPU)."""
import pytest

import workloads as wl
from paper_1910_00078_amd import cvx
from test_gpu_parity import check_case
from test_gpu_split_f32 import S1, S3, S5, _c, _s1

SMALL = [(h, q) for h in (1, 2, 5) for q in (1, 2, 3, 4, 5, 6, 7)]
CASES = [(v, _c(N=2, C=c, K=k, H=h, W=q, stride=s)) for v in S3 for c, k in ((17, 33), (16, 32), (1, 5), (34, 40)) for h, q in SMALL for s in ((1, 1), (2, 2)) if c * h * q >= 4]
CASES += [(v, _c(N=1, C=c, K=k, H=9, W=q, dil=(2, 2), pad=(2, 2), groups=g)) for v in S3 for c, k, g in ((38, 66, 2), (19, 7, 1), (9, 9, 3)) for q in (3, 8)]
CASES += [(v, _s1(N=3, C=c, K=k, H=h, W=q, stride=s)) for v in S1 for c, k in ((65, 70), (64, 32), (3, 7), (67, 9)) for h, q in SMALL for s in ((1, 1), (2, 2), (1, 3)) if c * h * q >= 4]
CASES += [(v, _s1(N=2, C=37, K=65, H=6, W=q, R=7, pad=(3, p), stride=s)) for v in S1 for q in (1, 2, 5) for p in (0, 1) for s in ((1, 1), (1, 2))]
CASES += [(v, _c(N=2, C=c, K=k, H=h, W=q, R=5, S=5, pad=(2, 2))) for v in S5 for c, k in ((17, 33), (20, 70), (33, 5)) for h, q in ((1, 1), (3, 2), (6, 3), (9, 11))]


@pytest.mark.parametrize("variant", sorted({v for v, _ in CASES}))
def test_loads_stay_inside(variant):
    served = 0
    for v, w in CASES:
        if v != variant:
            continue
        with cvx.ConvPlan(cvx.CVX_F32, (w.N, w.C, w.H, w.W), (w.K, w.C // w.groups, w.R, w.S), w.pad, w.stride, w.dil, w.groups) as plan:
            try:
                past = cvx.cvx_debug_reads_past_end(plan.xd, plan.wd, plan.cd, plan.yd, "tiled_f32_split_" + v)
            except cvx.CvxError as e:
                assert e.status == cvx.CVX_ERR_UNSUPPORTED             # (the patch does not fit this tile)
                continue
        served += 1
        assert max(past) <= 0, (past, w)
    assert served >= 10


# the last piece of x moved back by 1, 2 and 3 floats, over rows, planes and channels; the last one of w likewise
MOVED = [(v, w) for v in ("64x32_c16_s3", "256x64_c16_s3") for w in (
    _c(N=3, C=17, K=33, H=1, W=1), _c(N=2, C=19, K=40, H=2, W=1), _c(N=2, C=18, K=9, H=3, W=2), _c(N=2, C=21, K=70, H=4, W=3, stride=(1, 2)), _c(N=2, C=34, K=66, H=5, W=7, groups=2))]
MOVED += [(v, w) for v in ("128x64_c32_s1", "32x32_c64_s1") for w in (
    _s1(N=3, C=65, K=70, H=1, W=1), _s1(N=3, C=67, K=9, H=1, W=1), _s1(N=2, C=33, K=40, H=1, W=3), _s1(N=2, C=34, K=40, H=3, W=1), _s1(N=2, C=40, K=40, H=6, W=5, stride=(2, 2)),
    _s1(N=2, C=40, K=40, H=5, W=7, stride=(2, 2)), _s1(N=2, C=37, K=40, H=5, W=6, stride=(1, 2)), _s1(N=2, C=37, K=40, H=5, W=10, stride=(2, 3)))]
MOVED += [("32x32_c16_s5", _c(N=2, C=17, K=33, H=3, W=2, R=5, S=5, pad=(2, 2))), ("256x32_c16_s5", _c(N=2, C=19, K=40, H=6, W=3, R=5, S=5, pad=(2, 2)))]


@pytest.mark.gpu
@pytest.mark.parametrize("variant,w", MOVED, ids=lambda v: v if isinstance(v, str) else "c%d_k%d_%dx%d_s%d" % (v.C, v.K, v.H, v.W, v.stride[1]))
def test_pieces_moved_back(variant, w):
    check_case(w, pin="tiled_f32_split_" + variant)
