"""The build holds no form of the LDS-staged Gram kernel that no call can reach:
without point weights, 16-bit masks are multiplied as they are and FP32 values
through a piecewise-linear model (up to 4 row blocks: 256-byte slabs) are staged
through registers, each by another kernel."""
import os
import re

import pytest

from paper_2512_15187_amd import build


def test_report():
    if not os.path.exists(build.REPORT):
        pytest.skip("no build report")
    # <input, MFMA type, MODE, 3, WEIGHTED, ...>
    names = {line.split("\t")[0] for line in open(build.REPORT) if "gram_dma_kernelI" in line}
    assert names
    masks = [n for n in names if re.search(r"gram_dma_kernelI(DF16_Li0|NS_6bf16_tELi1)ELi0ELi3ELb\dE", n)]
    model = [n for n in names if re.search(r"gram_dma_kernelIfLi0ELi3ELi3ELb\dE.*Li256EE", n)]
    assert len(masks) == 4 and len(model) == 1
    assert all("ELi3ELb1E" in n for n in masks + model)
