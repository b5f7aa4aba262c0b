"""No source computes a value, keeps a constant or holds a helper function that
nothing uses."""
import os
import re
import subprocess

import pytest

from paper_2512_15187_amd import build


def test_no_unused_names():
    if not os.path.exists(build.HIPCC):
        pytest.skip("hipcc is not installed")
    flags = ["-std=c++17", "--offload-arch=gfx950", "-fsyntax-only", "--cuda-host-only", "-Wunused",
             "-Wno-unused-value", "-Wno-unused-result", "-Wno-unused-command-line-argument"]
    jobs = [subprocess.Popen([build.HIPCC, *flags, os.path.join(build.CSRC, s)], stderr=subprocess.PIPE, text=True)
            for s in build.SOURCES]
    out = "".join(j.communicate()[1] for j in jobs)
    assert all(j.returncode == 0 for j in jobs), out
    found = re.findall(r".*warning: .*", out)
    assert not [f for f in found if "-Wunused" in f], found


def test_no_unused_loads():
    text = "".join(open(os.path.join(build.CSRC, f)).read() for f in sorted(os.listdir(build.CSRC)))
    names = re.findall(r"__device__ __forceinline__ [\w<>:]+ (load\w+)\(", text)
    assert len(names) > 3
    assert not [n for n in names if len(re.findall(rf"\b{n}\b\s*[<(]", text)) < 2]
