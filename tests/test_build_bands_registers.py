"""Registers of the contour-boxplot bands' kernels: at most 128, so that four
waves share a SIMD.  (U8 through a model evaluates 16 points of a chunk in FP64;
eight chunks interleaved once took all 512.)"""
import os
import subprocess

import pytest

from paper_2512_15187_amd import build


def test_bands_registers(tmp_path):
    if not os.path.exists(build.HIPCC):
        pytest.skip("hipcc is not installed")
    r = subprocess.run([build.HIPCC, *build.COMMON, "--cuda-device-only", "-S", "-Rpass-analysis=kernel-resource-usage",
                        os.path.join(build.CSRC, "k_bands.hip"), "-o", str(tmp_path / "k_bands.s")], check=True,
                       capture_output=True, text=True)
    report = build.resource_report(r.stderr)
    assert len(report) == 18
    for name, vgprs, scratch in report:
        assert 0 < vgprs <= 128 and scratch == 0, (name, vgprs, scratch)
