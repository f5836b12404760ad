"""The sources that the bench's traffic record is tied to: all that a kernel is made of."""
import os
import re

import pytest

import bench

CSRC = os.path.join(bench.ROOT, "paper_2401_13708_amd", "csrc")


def _includes(name, seen):
    for f in re.findall(r'#include "(hts_\w+\.hpp)"', open(os.path.join(CSRC, name)).read()):
        if f not in seen:
            seen.add(f)
            _includes(f, seen)
    return seen


@pytest.mark.parametrize("kernel", sorted(bench.KERNEL_SOURCES))
def test_every_header_is_hashed(kernel):
    files = bench.KERNEL_SOURCES[kernel]
    need = set()
    for f in files:
        _includes(f, need)
    assert need <= set(files)
