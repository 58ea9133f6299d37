"""The benchmark prices a layer against the peak of the unit that its kernel runs on."""
import pytest

import bench
import workloads as wl


@pytest.mark.parametrize("name,kernel,peak", [
    ("c2", "igemm_512x64_c16_3x3", 2516.6), ("c2f32", "tiled_f32_split_256x64_c16_s3", 2516.6 / 6), ("c2f32", "tiled_f32_256x64_c8_3x3", 157.3),
    ("c1", "direct_f32", 157.3), ("c3a", "pointwise_256x64_c32_r5", 8000.0),
])
def test_peak_is_that_of_the_pipe(name, kernel, peak):
    w = wl.WORKLOADS[name]
    r = bench.roofline(w, name, kernel, 0.1)
    work = w.algorithmic_bytes / 1e-4 / 1e9 if r["unit"] == "GB/s" else w.flops / 1e-4 / 1e12
    assert r["peak"] == pytest.approx(peak) and r["frac"] == pytest.approx(work / peak)
