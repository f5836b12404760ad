"""Index arithmetic of the lists between the traversal's two phases, compiled for
the host from the header that the kernels use."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2401_13708_amd", "csrc")


def _run(tmp_path, body):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text('#include <cstdio>\n#include <vector>\n#include "hts_lists.hpp"\nusing namespace hts;\n'
                   "int main() {\n" + body + "\nreturn 0;\n}\n")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                        "-I" + os.path.join(ROOT, "include"), "-I" + CSRC, str(src), "-o", str(exe)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout


# query blocks of a layout; chunks a phase-A wave may hand over (200 at the default
# list).  400000 jobs of 7 points are 400000 blocks: 320 million chunks, 2.56
# billion cells.  A chunk's number stays below 2^31 wherever its partials (512
# bytes in single precision) fit a GPU's 288 GB.
@pytest.mark.parametrize("nqb,share", [(1, 200), (1094, 200), (335544, 200), (335545, 200), (400000, 200),
                                       (520000, 200), (16000000, 7)])
def test_a_chunk_is_read_where_its_cells_were_written(tmp_path, nqb, share):
    _run(tmp_path, """
    const long long nqb = %d, share = %d, waves = 4 * nqb;
    for (long long g : {0ll, 1ll, waves / 2, waves - 2, waves - 1}) {
        if (g < 0 || g >= waves) continue;
        const int id0 = (int)(g * share);
        for (long long number : {0ll, 1ll, share / 2, share - 1})
            for (long long start : {number, number * kCells, share * kCells - 1}) {
                if (start < number || start >= share * kCells) continue;
                const Chunk c = chunk_of(id0, (int)number, 5, (int)start, (int)start + 1, 64);
                const long long want = g * share * kCells + start;  // the wave's cells, one after another
                if (wave_cells(id0) + start != want || chunk_cells(c.id, c.first) != want || c.id != g * share + number ||
                    c.cells != 1 || c.cnt != 64 || c.q0 != 5) {
                    std::printf("wave %%lld chunk %%lld cell %%lld: %%lld, read %%lld\\n", g, number, start, want,
                                (long long)chunk_cells(c.id, c.first));
                    return 1;
                }
            }
    }""" % (nqb, share))


# takers: the automatic grids, one per chunk where the list is short, and any
# launch shape that is asked for
@pytest.mark.parametrize("takers", [1, 2, 63, 64, 65, 128, 1000, 4096, 5000, 30632, 40000, 65537])
@pytest.mark.parametrize("most", [0, 1, 9, 504, 3000])
def test_chunks_are_dealt_out_evenly(tmp_path, takers, most):
    _run(tmp_path, """
    const int takers = %d, most = %d;
    int n[kGroups], sum = 0;
    std::vector<std::vector<int>> seen(kGroups);
    for (int p = 0; p < kGroups; ++p) {
        n[p] = (int)((unsigned)(p * 2654435761u) %% (unsigned)(most + 1));
        seen[p].assign(n[p], 0);
        sum += n[p];
    }
    int longest = 0, largest = 0;
    for (int w = 0; w < takers; ++w) {
        int own = 0, part = 0;
        long long last = -1;
        deal(own_parts(takers), w, takers, [&](int p) -> int64_t { return n[p]; }, [&](int p, int64_t i) {
            if (p == part && i <= last) std::printf("order\\n");
            part = p;
            last = i;
            seen[p][i] += 1;
            ++own;
        });
        longest = own > longest ? own : longest;
    }
    for (int p = 0; p < kGroups; ++p) {
        largest = n[p] > largest ? n[p] : largest;
        for (int s : seen[p])
            if (s != 1) { std::printf("part %%d: taken %%d times\\n", p, s); return 1; }
    }
    // no more than a fair share (of the largest part, where the parts have their own)
    const int bound = own_parts(takers) ? (largest + takers / kGroups - 1) / (takers / kGroups)
                                        : (sum + takers - 1) / takers;
    if (longest > bound) { std::printf("%%d of %%d chunks for one, share %%d\\n", longest, sum, bound); return 1; }
    """ % (takers, most))
