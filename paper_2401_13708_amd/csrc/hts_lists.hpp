// hts_lists.hpp -- index arithmetic of the lists between the two phases of the
// Barnes-Hut traversal (also compiled for the host by the tests).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace hts {

// the cells a chunk holds on average at most
constexpr int kCells = 8;

// a cell handed over (its children are walked for the lanes that rejected
// it), and a chunk of cells: its number, the block's first query, its first cell's
// place behind kCells cells for every chunk before it, and its cells and queries.
// Chunks are numbered below 2^31 (512 bytes of partials each), cells are not (2^31
// of them are 335544 query blocks at the default list): places are 64 bits wide,
// and a chunk keeps what distinguishes its own, less than a wave's share.
struct alignas(16) Cell {
    int32_t node, next;
    uint64_t mask;
};
struct alignas(16) Chunk {
    int32_t id, q0, first;
    uint16_t cells, cnt;
};

// Chunk `number` of the phase-A wave whose chunks have the numbers from id0 on; its
// cells are those from `start` on of the wave's.
__host__ __device__ inline Chunk chunk_of(int id0, int number, int q0, int start, int end, int cnt) {
    return Chunk{id0 + number, q0, start - number * kCells, (uint16_t)(end - start), (uint16_t)cnt};
}
// The place of a phase-A wave's first cell, and of a chunk's.
__host__ __device__ inline int64_t wave_cells(int id0) { return (int64_t)id0 * kCells; }
__host__ __device__ inline int64_t chunk_cells(int id, int first) { return (int64_t)id * kCells + first; }

// The list length of each of two traversals side by side, where one's workspace takes
// `bytes` at the length asked for. Two of more than 32 GiB (3.9 million points in single
// precision, 2.2 in double) get half the length each, which nearly halves them: a call
// that fits a card with one workspace has to fit it with both (3 million points in double
// precision 62 GB, as one after the other). Few waves hand over more: 3 million points 41.9
// ms with whole and half lists, 17.3 and 17.4 in single precision.
constexpr size_t kListsWhole = (size_t)32 << 30;
__host__ __device__ inline int list_of_both(int list, size_t bytes) {
    return bytes > kListsWhole ? (list < 256 ? list + 1 : 257) / 2 : list;
}

// The lists are kept in kGroups parts of entries(p) entries: take(p, i) for those
// that taker w of `takers` takes.  own: each part has as many takers of its
// own (own_parts(takers)), and w serves one part.  Else the parts' entries are dealt out one after another, on
// from part to part: were each part's begun with the first taker again, as many
// takers as the longest part has entries would take nearly all of them (n = 70000 near
// the rim: 3.3 ms for the gradient on 1000 workgroups of 4 waves, 1.2 dealt on).
constexpr int kGroups = 64;
__host__ __device__ inline bool own_parts(int64_t takers) { return takers % kGroups == 0; }
template <typename N, typename F>
__host__ __device__ inline void deal(bool own, int64_t w, int64_t takers, N entries, F take) {
    const int p0 = own ? (int)(w % kGroups) : 0, p1 = own ? p0 + 1 : kGroups;
    const int64_t stride = own ? takers / kGroups : takers;
    int64_t i = own ? w / kGroups : w;
    for (int p = p0; p < p1; ++p) {
        const int64_t n = entries(p);
        for (; i < n; i += stride) take(p, i);
        i -= n;
    }
}

}  // namespace hts
