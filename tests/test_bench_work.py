"""The work that bench.py books for each kernel: the unit its sums run on and the
flops it issues (the roofline fractions divide by that unit's peak)."""
import os
import sys

import pytest

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
import bench  # noqa: E402


@pytest.mark.parametrize("level,unit,issued", [
    (2, "f64 valu", 1),           # the 4^3 level, a wave per frequency
    (3, "f64 mfma", 216 / 189),   # octets
    (4, "f64 valu", 1),           # the periodic 16^3 level, whole
    (5, "f64 mfma", 216 / 189),
])
def test_zone_levels_are_booked_on_the_unit_they_run_on(level, unit, issued):
    p, F, nodes = 8, 256 * 9, 8 ** level
    flops = (37 if level == 2 else 189) * 8.0 * F * nodes
    gemm = bench.kernel_work("m2l L%d" % level, 512, 5, p, {"m2l": "gemm", "near": "direct", "precision": "fp32"})
    spec = bench.kernel_work("m2l L%d stencil" % level, 512, 5, p,
                             {"m2l": "spectral", "near": "fft", "precision": "fp32"})
    assert gemm[:2] == (flops, unit) and gemm[3] == issued
    assert spec[:2] == (flops, unit) and spec[3] == issued


def test_other_units():
    r = {"m2l": "spectral", "near": "fft", "precision": "fp32", "zones_fp32_level": 4}
    assert bench.kernel_work("m2l L4 stencil", 256, 4, 8, r)[1] == "f32 valu"
    assert bench.kernel_work("m2l L3 node transforms", 256, 4, 8, r)[1] == "hbm"
    split = bench.kernel_work("m2l L4", 256, 4, 8, {"m2l": "gemm", "near": "direct", "precision": "bf16x3"})
    assert split[1] == "bf16 mfma" and split[3] == 6
