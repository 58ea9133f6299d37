"""Implicit-GEMM kernels on channel and filter counts that fill neither a stage nor a filter block, against
the oracle: one channel past an octet, past a stage, past a half stage; one filter past a block, one short of
it; the same inside groups, where what follows a group's channels is the next group's data."""
import pytest

import workloads as wl
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
]


@pytest.mark.parametrize("dtype", [wl.BF16, wl.F16])
@pytest.mark.parametrize("w", CASES, ids=lambda w: w.name)
def test_ragged_channels_and_filters(w, dtype):
    assert check_case(wl.small_variant(w, dtype=dtype)).startswith("igemm_")


@pytest.mark.parametrize("variant", ["igemm_512x64_c32_3x3", "igemm_512x64_c16_3x3", "igemm_256x128_c16_3x3", "igemm_256x64_c32_3x3",
                                     "igemm_256x64_c16_3x3"])
def test_every_3x3_variant(variant):
    check_case(_c(name="pinned", N=3, C=43, K=150, H=12, W=12), pin=variant + ",1,10")
