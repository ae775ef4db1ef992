"""bench.py's roofline names the kernel that a variant runs and the rate of the matrix cores as that kernel uses them."""
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402
from paper_2507_17301_amd import binding as nm  # noqa: E402


def test_every_variant_has_a_kernel_of_the_sources():
    csrc = os.path.join(ROOT, "paper_2507_17301_amd", "csrc")
    text = "".join(open(os.path.join(csrc, f)).read() for f in os.listdir(csrc) if f.endswith(".h"))
    for v in range(nm.nm_variant_count()):
        assert f" {bench.kernel_of(nm.nm_variant_name(v))}(const ConvParams p)" in text, nm.nm_variant_name(v)


@pytest.mark.parametrize("variant,dtype,kernel,peak", [
    ("X3S_NB2_WP1_NJ2_S4", "f32", "nm_conv_split_kernel", 2500 / 6), ("X3D_NB4_WP1_NJ1", "f32", "nm_conv_split_kernel", 2500 / 6),
    ("ROWF_R4_NJ2_KS3", "f32", "nm_conv_rows_kernel", 2500 / 6), ("RUN_ROWS8_NJ4_KS3", "bf16", "nm_conv_rows_kernel", 2500),
    ("RUN_NB4_WP1_NJ1_KS3", "bf16", "nm_conv_run16_kernel", 2500), ("NB4_WP1_NJ1_CK32_SPC4_V1", "f32", "nm_conv_kernel", 157.3),
    ("VAR_NB4_WP1_NJ1_CK64_SPC16", "f32", "nm_conv_kernel", 157.3), ("SPR1_NB8_WP1_NJ4_CK64", "bf16", "nm_conv_sp16_kernel", 2500),
    ("SPR1_TAPS_NB7_WP2_NJ4", "bf16", "nm_conv_taps_kernel", 2500), ("SPR0_TAPS_NB5_WP2_NJ4", "bf16", "nm_conv_taps_kernel", 2500),
    ("KW_PB1_NJ2_CK32_SPC4_S16", "f32", "nm_conv_wave_kernel", 157.3),
    ("F8R_NB4_WP1_NJ2_CK128", "f8", "nm_conv_sp16_kernel", 5000), ("F8_NB4_WP1_NJ4", "f8", "nm_conv_f8_kernel", 5000)])
def test_kernel_and_peak(variant, dtype, kernel, peak):
    assert bench.kernel_of(variant) == kernel and bench.matrix_peak(variant, dtype) == peak
