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
], ids=lambda v: getattr(v, "name", v))
def test_measured_slower_elsewhere(w, slow):
    assert not kernel(w).startswith(slow)
