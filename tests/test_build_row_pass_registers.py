"""Registers of the two-pass PID-mean kernels as the last build reported them: the
row pass of FP32 input at most 128 (four waves per SIMD), the column sums of
16-bit input at most 64 (eight).  (Both passes run at the rate of the loads in
flight; the ragged tile's loads once pushed them past these steps.)"""
import os
import re

import pytest

from paper_2512_15187_amd import build


def test_report():
    if not os.path.exists(build.REPORT):
        pytest.skip("no build report")
    rows = colsums = 0
    for line in open(build.REPORT):
        name, vgpr, _ = line.split("\t")
        v = int(vgpr.split("=")[1])
        # <float, MODE, MPW, WEIGHTED, SFROM = true, 8>
        if re.search(r"pidmean_soft_kernelIfLi\dELi\d+ELb\dELb1ELi8E", name):
            rows += 1
            assert v <= 128, (name, v)
        if re.search(r"colsum_part_kernelI(DF16_|NS_6bf16_tE)Li\d", name):
            colsums += 1
            assert v <= 64, (name, v)
    assert rows == 24 and colsums == 14
