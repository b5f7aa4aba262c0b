"""The build refuses device code that reads the dispatch packet."""
import os
import subprocess

import pytest

from paper_2512_15187_amd import build


def _asm(tmp_path, text):
    p = tmp_path / "k-hip-amdgcn-amd-amdhsa-gfx950.s"
    p.write_text(text)
    return str(p)


def test_check(tmp_path):
    one = "\t.amdhsa_kernel k{i}\n\t\t.amdhsa_user_sgpr_dispatch_ptr {v}\n\t.end_amdhsa_kernel\n"
    build.check_dispatch_packet(_asm(tmp_path, one.format(i=0, v=0) + one.format(i=1, v=0)))
    with pytest.raises(RuntimeError, match="k1"):
        build.check_dispatch_packet(_asm(tmp_path, one.format(i=0, v=0) + one.format(i=1, v=1)))


def test_bands_kernels(tmp_path):
    """The contour-boxplot bands' U8 kernels once did (an indexed local array)."""
    if not os.path.exists(build.HIPCC):
        pytest.skip("hipcc is not installed")
    out = str(tmp_path / "k_bands.s")
    subprocess.run([build.HIPCC, *build.COMMON, "--cuda-device-only", "-S", os.path.join(build.CSRC, "k_bands.hip"),
                    "-o", out], check=True, capture_output=True)
    build.check_dispatch_packet(out)
