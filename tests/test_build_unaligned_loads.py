"""The vector loads of rows at any address promise the compiler the element's
alignment and no more (an alignment attribute is lost on a template argument:
the loads were once declared 16-byte aligned)."""
import os
import re
import subprocess

import pytest

from paper_2512_15187_amd import build

SOURCE = """
#include "%s"
using namespace pidk;
#define K(N, T) __global__ void any_##N(const T* p, uint4* o) { \\
  o[threadIdx.x] = __builtin_bit_cast(uint4, load16_any(p + threadIdx.x)); } \\
  __global__ void nt_##N(const T* p, uint4* o) { \\
  o[threadIdx.x] = __builtin_bit_cast(uint4, load16_nt_any(p + threadIdx.x)); }
K(1, uint8_t) K(2, f16) K(4, float) K(8, double)
"""


def test_alignment_of_loads(tmp_path):
    if not os.path.exists(build.HIPCC):
        pytest.skip("hipcc is not installed")
    src, out = tmp_path / "loads.hip", tmp_path / "loads"
    src.write_text(SOURCE % os.path.join(build.CSRC, "device_common.h"))
    cmd = [build.HIPCC, *build.COMMON, "--cuda-device-only", "-S", str(src), "-o"]
    subprocess.run([*cmd, f"{out}.ll", "-emit-llvm"], check=True, capture_output=True)
    subprocess.run([*cmd, f"{out}.s"], check=True, capture_output=True)
    kernel, seen = None, 0
    for line in open(f"{out}.ll"):
        k = re.search(r"define .*@_Z\d+(any|nt)_(\d)", line)
        if k:
            kernel = int(k.group(2))
        a = re.search(r"= load .* align (\d+)", line)
        if a and kernel:
            seen += 1
            assert int(a.group(1)) == kernel, line
    assert seen >= 8
    asm = open(f"{out}.s").read()
    assert len(re.findall(r"global_load_dwordx4 ", asm)) == 8 and "global_load_ubyte" not in asm
