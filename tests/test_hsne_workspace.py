"""The workspace of h-SNE's two traversals, with the rule compiled for the host from the
header that the kernels use: no more than what one traversal takes at the list asked for,
wherever that is large."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2401_13708_amd", "csrc")


def _list_of_both(tmp_path, list_items, size):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text('#include <cstdio>\n#include "hts_lists.hpp"\nint main() { std::printf("%%d", '
                   "hts::list_of_both(%d, (size_t)%dull)); }\n" % (list_items, size))
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                        "-I" + CSRC, str(src), "-o", str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    return int(subprocess.run([str(exe)], capture_output=True, text=True, timeout=60).stdout)


def _bytes(n, list_items, chunk):
    # four waves of 64 queries each, 200 chunks per 256 of the list, rounded up; the forces per slot
    return 4 * (-(-n // 64)) * (-(-min(list_items, 256) * 200 // 256) * chunk + 12) + 80 * n


# points in single precision (696 bytes a chunk) and double (1208), up to what a tree of
# that many levels holds
@pytest.mark.parametrize("n,chunk", [(70000, 696), (3000000, 696), (9500000, 696), (16700000, 696), (9500000, 1208),
                                     (13400000, 1208)])
@pytest.mark.parametrize("list_items", [0, 1, 16, 255, 256, 1000])
def test_two_traversals_fit_where_one_did(tmp_path, n, chunk, list_items):
    one = _bytes(n, list_items, chunk)
    got = _list_of_both(tmp_path, list_items, one)
    if one <= 32 << 30:
        assert got == list_items
    else:
        # (the forces per slot are there twice, and half a list rounds up)
        assert 2 * _bytes(n, got, chunk) <= 1.02 * one
    assert got > 0 or list_items == 0
