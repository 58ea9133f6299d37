"""The separate bias operator on planes that straddle its 16-byte pieces, are just as large as one or smaller, and at
the remainders of a block's pieces, element by element against y + b[k]."""
import numpy as np
import pytest

import workloads as wl
from paper_1910_00078_amd import cvx
from parity import DT_CODE, to_device, to_host_f64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [wl.F32, wl.BF16, wl.F16])
@pytest.mark.parametrize("shape", [(2, 3, 1, 7), (3, 5, 2, 4), (2, 1, 3, 3), (1, 7, 3, 5), (3, 37, 7, 7), (1, 1, 1, 1), (2, 129, 31, 33)])
def test_bias_on_any_plane(dtype, shape):
    import torch
    rng = np.random.default_rng(7)
    quantise = {wl.F32: lambda v: v.astype(np.float32), wl.F16: lambda v: v.astype(np.float16),
                wl.BF16: lambda v: (v.astype(np.float32).view(np.uint32) >> 16).astype(np.uint16)}[dtype]
    y0, b0 = quantise(rng.uniform(-1, 1, shape)), quantise(rng.uniform(-1, 1, shape[1]))
    y, b = to_device(y0, dtype), to_device(b0, dtype)
    h = cvx.cvx_create(torch.cuda.current_stream().cuda_stream)
    yd, bd = cvx.cvx_tensor_desc_create(), cvx.cvx_tensor_desc_create()
    cvx.cvx_tensor_desc_set_4d(yd, DT_CODE[dtype], *shape)
    cvx.cvx_tensor_desc_set_4d(bd, DT_CODE[dtype], 1, shape[1], 1, 1)
    cvx.cvx_bias_add(h, bd, b.data_ptr(), yd, y.data_ptr())
    cvx.cvx_activation_fwd(h, cvx.CVX_ACT_LEAKY_RELU, 0.25, yd, y.data_ptr())
    got = to_host_f64(y, dtype)
    want = wl.to_f64(y0, dtype) + wl.to_f64(b0, dtype)[None, :, None, None]
    want = np.where(want > 0, want, 0.25 * want)
    # two roundings of half an ulp each: 2^-9 (bf16), 2^-12 (fp16), 2^-25 (fp32) of values below 2
    assert np.all(np.abs(got - want) <= 2 * 2 * {wl.F32: 2.0**-25, wl.F16: 2.0**-12, wl.BF16: 2.0**-9}[dtype])
    for d in (yd, bd):
        cvx.cvx_tensor_desc_destroy(d)
    cvx.cvx_destroy(h)
