"""The server's estimate of a job's device memory against the sizes that the
traversal's workspace is made of (no GPU)."""
import os
import re

import pytest

from paper_2401_13708_amd.serve import footprint_bytes

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2401_13708_amd", "csrc")


def _constant(name):
    for f in ("k_bh.hip", "hts_lists.hpp"):
        m = re.search(r"constexpr int .*\b%s = (\d+)" % name, open(os.path.join(CSRC, f)).read())
        if m:
            return int(m[1])
    raise KeyError(name)


@pytest.mark.parametrize("n", [64, 1000, 100000])
@pytest.mark.parametrize("items", [1, 2, 16, 100, 255, 256, 1000])
def test_a_wave_s_share_of_the_workspace(n, items):
    most = _constant("kListItems")
    chunks = -(-min(items, most) * _constant("kChunks") // most)
    # places in the lists, cells, force and Z partials
    chunk = _constant("kKinds") * 16 + _constant("kCells") * 16 + 64 * 2 * 4 + 8
    waves = 4 * -(-n // 64)
    share = footprint_bytes(n, item_list=items) - footprint_bytes(n, item_list=0)
    assert waves * chunks * chunk <= share <= (waves + 4) * chunks * chunk
