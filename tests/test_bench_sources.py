"""Profile summaries name the kernel sources that they were taken on by a hash:
it covers every file of the library that the kernels are compiled from."""
import os
import re

import bench


def test_the_hash_covers_what_the_kernels_include():
    csrc = os.path.join(bench.ROOT, "paper_1905_02241_amd", "csrc")
    found, todo = set(), ["mech_kernels.hip"]
    while todo:
        f = todo.pop()
        if f in found or not os.path.exists(os.path.join(csrc, f)):
            continue
        found.add(f)
        todo += re.findall(r'#include "(\w+\.\w+)"', open(os.path.join(csrc, f)).read())
    assert found == set(bench.KERNEL_SOURCES)
