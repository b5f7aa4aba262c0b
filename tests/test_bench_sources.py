"""The recorded traffic of the headline kernel counts for the sources that it was
taken on: every file that goes into the build of the two kernel sources."""
import os
import re

import bench

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_kernel_sources_are_complete():
    todo = [os.path.join(ROOT, p) for p in bench.KERNEL_SOURCES if p.endswith(".hip")]
    assert len(todo) == 2
    seen = set()
    while todo:
        p = os.path.normpath(todo.pop())
        if p in seen:
            continue
        seen.add(p)
        with open(p) as fh:
            todo += [os.path.join(os.path.dirname(p), h) for h in re.findall(r'#include "([^"]+)"', fh.read())]
    assert {os.path.relpath(p, ROOT) for p in seen} <= set(bench.KERNEL_SOURCES)
