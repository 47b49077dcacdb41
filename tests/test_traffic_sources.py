"""The counter summary that bench.py quotes is valid for the sources its hash
covers: every device header that those sources include is among them."""
import os
import re

import bench


def test_hash_covers_the_device_headers():
    have = set(bench.KERNEL_SOURCES)
    seen, todo = set(), list(have)
    while todo:
        f = todo.pop()
        if f in seen:
            continue
        seen.add(f)
        text = open(os.path.join(bench.ROOT, f)).read()
        todo += [os.path.join(os.path.dirname(f), h) for h in re.findall(r'#include "([^"]+)"', text)]
    host_only = {"paper_2408_00488_amd/csrc/csl_kernels.hpp"}   # declarations of the launchers
    assert seen - host_only == have
