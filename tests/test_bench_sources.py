"""The benchmark's stored counter figures (no GPU): a figure holds only while the sources
of its kernel are those it was taken on, so these have to be all that the kernel's file
includes."""
import os
import re

import pytest

import bench

CSRC = os.path.join(bench.ROOT, "paper_2501_10946_amd", "csrc")


def included(name, seen):
    seen.add(name)
    with open(os.path.join(CSRC, name)) as fh:
        for inc in re.findall(r'^#include "([^"]+)"', fh.read(), re.M):
            if inc not in seen and os.path.exists(os.path.join(CSRC, inc)):
                included(inc, seen)
    return seen


@pytest.mark.parametrize("kernel", sorted(bench.KERNEL_SOURCES))
def test_sources_are_all_that_the_kernel_includes(kernel):
    listed = bench.KERNEL_SOURCES[kernel]
    assert included(listed[0], set()) <= set(listed)
