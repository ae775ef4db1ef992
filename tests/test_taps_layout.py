"""The address arithmetic of the tap-staged bf16 kernel, compiled for the CPU from the header that the kernel uses."""
import os

import pytest

from test_sanitizers import ROOT, SAN, ENV, _run


def test_every_tap_finds_its_pixel(tmp_path):
    clang = "/opt/rocm/lib/llvm/bin/clang++"
    if not os.path.exists(clang):
        pytest.skip("no HIP-aware clang++ in this image")
    exe = str(tmp_path / "taps_layout")
    _run([clang, "-x", "hip", "--cuda-host-only", "-std=c++17", "-D__HIP_PLATFORM_AMD__"] + SAN +
         ["-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2507_17301_amd", "csrc"),
          "-I", "/opt/rocm/include", os.path.join(ROOT, "tests", "sanitize", "taps_layout.cpp"), "-o", exe])
    assert "taps layout: ok" in _run([exe], env=ENV)
