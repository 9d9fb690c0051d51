"""The benchmark rates each complex64 level kernel by the form of its
products."""
import os
import sys

import pytest

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
import bench  # noqa: E402


def _kernel(name, *steps):
    return f'extern "C" __global__ void __launch_bounds__(256) {name}(C2* mem) {{\n' + "".join(steps) + "}\n"


FP32 = "  // step 3 (matrix cores) b 1 i 5 j 5 k 2\n  mfma\n"
PARTS = "  // step 4 (matrix cores, per item) b 0 i 6 j 6 k 5 fp32\n  S3 x = split3(v);\n"
VECTOR = "  // step 5\n  a0 = cad(a0, v);\n"


def test_peak_of_each_product_form():
    src = _kernel("wc0", VECTOR) + _kernel("wl0", FP32) + _kernel("wl1", PARTS) + _kernel("wl2", VECTOR) + \
        _kernel("wl3", FP32, PARTS)
    fp32, parts = bench.PEAK_FP32_MATRIX_TFLOPS, bench.PEAK_BF16_MATRIX_TFLOPS / 6
    got = bench.c64_peaks(src)
    assert got[:3] == [pytest.approx(fp32), pytest.approx(parts), None]
    assert got[3] == pytest.approx((2 ** 13 + 2 ** 17) / (2 ** 13 / fp32 + 2 ** 17 / parts))
    # one pass of 64 slices in 1 ms at 100 TFLOP/s and few bytes: bound by its own products' peak
    levels = ([1.0, 0.5], [100e12 * 1e-3 / 64, 1.0], [1, 1], 1, 64, [8.0, 8.0], None)
    assert bench.level_roofline(levels, "none", "c64", got)["peak"] == pytest.approx(fp32)
    assert bench.level_roofline(levels, "none", "c64", got[1:])["peak"] == pytest.approx(parts)
