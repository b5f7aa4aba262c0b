"""Registers of the packing pass of the two-pass binary PID-mean: nothing in
scratch, and U8 masks at most 96, so that five waves share a SIMD.  (Its ragged
tile once held byte loads beside vector loads: 130 registers, and scratch for
FP32 and FP64 fields.)"""
import os
import subprocess

import pytest

from paper_2512_15187_amd import build


def test_count_pack_registers(tmp_path):
    if not os.path.exists(build.HIPCC):
        pytest.skip("hipcc is not installed")
    r = subprocess.run([build.HIPCC, *build.COMMON, "--cuda-device-only", "-S", "-Rpass-analysis=kernel-resource-usage",
                        os.path.join(build.CSRC, "k_bits.hip"), "-o", str(tmp_path / "k_bits.s")], check=True,
                       capture_output=True, text=True)
    report = [x for x in build.resource_report(r.stderr) if "count_pack_kernel" in x[0]]
    assert len(report) == 7
    for name, vgprs, scratch in report:
        assert scratch == 0, (name, scratch)
        if "SrcBytes" in name or "SrcValuesIhLb0E" in name:
            assert 0 < vgprs <= 96, (name, vgprs)
