// k_knn.hip -- the exact k nearest neighbours of the input points (Sec. 2-A).
//
// The result is defined by double-precision squared distances, summed over the
// dimensions in ascending order with one fused multiply-add per term, and by
// the order (distance, index).  All n^2 of them in double precision cost
// n^2 d vector operations; here the matrix cores sort out the pairs that can
// matter, with bounds that hold whatever their rounding, and only those get
// their double-precision distance:
//  1. every point, shifted by a centre and scaled by a power of two, is rounded
//     to half precision; its squared norm n^2 and the norm r of what the
//     rounding left out are kept.  With A the distance of two rounded points,
//     the true (scaled) distance D lies in [A - r - r', A + r + r'] (triangle
//     inequality);
//  2. A^2 = n^2 + n'^2 - 2 <x, x'> through MFMA with single-precision
//     accumulation; its error is at most kappa (n^2 + n'^2), kappa = 2 (d + 8)
//     2^-23 (the sum of -n^2 / 2, -n'^2 / 2 and the d products, every addition
//     rounded by at most 2^-23 of the sum of magnitudes), which is folded into
//     the norms: P = (1 + kappa) n^2 for upper bounds, M = (1 - kappa) n^2 for
//     lower ones;
//  3. first pass: per query and group of candidates the smallest upper bound;
//     the (k + 1)-th smallest of a query's group minima bounds its k-th
//     neighbour's distance (k + 1 groups hold k + 1 points, at most one of
//     which is the query itself);
//  4. second pass: the candidates whose lower bound does not exceed it, as a bit
//     matrix (about 1.1 k of them a query);
//  5. their exact distances, sorted.
// A query with more than kCap candidates (many points closer together than the
// rounding resolves, values that are not finite) goes through k_knn_direct,
// which streams all candidates in double precision.
//
// Candidates take their places in the matrix in the order p -> p S mod n, S near
// the golden section of n, so that the points of a group come from all over the
// input (inputs are often sorted by class).
//
// At n = 70000, d = 784 the direct kernel alone took 578 ms (n = 5000, d = 50: 3.1
// ms; n = 1000, d = 32 in double precision: 1.3 ms), bound by the vector rate at
// large n and by the few workgroups at small n.  All of the above takes 12.0 ms
// (0.11 and 0.05 ms): the two passes of products 3.8 ms each (7.6 when every tile
// was formed for both of its blocks; n^2 d / 2 multiply-adds in half precision
// at 1.0 PFLOP/s), the exact distances 3.7 ms (25 GB of candidates' rows, which
// come from beyond the L2).
#include <climits>
#include <cmath>

#include "hts_impl.hpp"
#include "hts_math.hpp"

namespace hts {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef float float16v __attribute__((ext_vector_type(16)));

constexpr int kMaxK = kKnnMaxK;
constexpr int kCap = 512;     // candidates of a query
constexpr int kTileC = 256;   // candidates of a tile of the products
constexpr int kTileQ = 128;   // queries of a tile
constexpr int kStep = 32;     // dimensions of a stage
constexpr int kSample = 64;   // points the centre and the scale are taken from
constexpr int kGroup = 64;    // candidates one lane holds of a tile (a word of the bit matrix)
constexpr int kPick = 1024;   // groups the threshold is picked from, at most
constexpr int64_t kSlabBytes = (int64_t)1 << 30;

__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ascending bitonic sort of P2 (a power of two) (distance, index) pairs held in
// LDS, by the 64 lanes of one wave
__device__ void wave_bitonic(double *sd, int *sj, int P2, int lane) {
    for (int size = 2; size <= P2; size <<= 1) {
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            for (int t = lane; t < (P2 >> 1); t += kWave) {
                int i = 2 * t - (t & (stride - 1));
                int j = i + stride;
                bool up = (i & size) == 0;
                double di = sd[i], dj = sd[j];
                int ji = sj[i], jj = sj[j];
                bool gt = (di > dj) || (di == dj && ji > jj);
                if (gt == up) {
                    sd[i] = dj; sd[j] = di;
                    sj[i] = jj; sj[j] = ji;
                }
            }
            wave_sync();
        }
    }
}

// ---------------------------------------------------------------- 1. halves
// centre of up to kSample points spread over the input, and per block of
// dimensions the largest deviation of those points from it
template <typename XT>
__global__ __launch_bounds__(kBlock) void k_knn_center(const XT *__restrict__ X, int64_t n, int d,
                                                       XT *__restrict__ centre,
                                                       float *__restrict__ spread,
                                                       int32_t *__restrict__ ndirect) {
    __shared__ float s_max[kBlock];
    if (blockIdx.x == 0 && threadIdx.x == 0) *ndirect = 0;
    const int dim = (int)(blockIdx.x * kBlock + threadIdx.x);
    const int m = n < kSample ? (int)n : kSample;
    const int64_t step = n / m;
    float mx = 0.0f;
    if (dim < d) {
        XT v[kSample];
        double sum = 0.0;
#pragma unroll
        for (int a = 0; a < kSample; ++a) v[a] = a < m ? X[a * step * d + dim] : (XT)0;
#pragma unroll
        for (int a = 0; a < kSample; ++a) sum += (double)v[a];
        const XT c = (XT)(sum / m);
        centre[dim] = c;
#pragma unroll
        for (int a = 0; a < kSample; ++a)
            if (a < m) mx = fmaxf(mx, fabsf((float)((double)v[a] - (double)c)));
    }
    s_max[threadIdx.x] = mx;
    __syncthreads();
    for (int o = kBlock / 2; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) s_max[threadIdx.x] = fmaxf(s_max[threadIdx.x], s_max[threadIdx.x + o]);
        __syncthreads();
    }
    if (threadIdx.x == 0) spread[blockIdx.x] = s_max[0];
}

// input index of place p
__device__ __forceinline__ int64_t place(int64_t p, int64_t S, int64_t n) {
    return (int64_t)((uint64_t)(p * S) % (uint64_t)n);
}

// One wave a place: the rounded point in blocks of kStep dimensions
// (H[block][place][kStep], places and dimensions padded with zeros), -P / 2 and
// -M / 2 (minus infinity past n) and r (not less than the truth; infinite when
// the point is not finite).
template <typename XT>
__global__ __launch_bounds__(kBlock) void k_knn_half(const XT *__restrict__ X, int64_t n, int d,
                                                     const XT *__restrict__ centre,
                                                     const float *__restrict__ spread, int nspread,
                                                     int64_t S, int64_t np, int blocks, float kappa,
                                                     _Float16 *__restrict__ H,
                                                     float *__restrict__ hp, float *__restrict__ hm,
                                                     float *__restrict__ r, KnnReverse rev) {
    const int lane = (int)(threadIdx.x & (kWave - 1));
    const int64_t p = ((int64_t)blockIdx.x * kBlock + threadIdx.x) / kWave;
    if (p >= np) return;
    float mx = 0.0f;
    for (int a = lane; a < nspread; a += kWave) mx = fmaxf(mx, spread[a]);
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, kWave));
    // the sample's largest deviation becomes 4 to 8, 2^13 below the largest half
    int e = 0;
    if (mx > 0.0f && mx < __builtin_inff()) e = 2 - ilogbf(mx);
    const double scale = ldexp(1.0, e);
    const bool real = p < n;
    const XT *row = X + (real ? place(p, S, n) : 0) * d;
    double n2 = 0.0, r2 = 0.0, mag2 = 0.0;
    for (int b = lane; b < blocks * (kStep / 8); b += kWave) {
        half8 h;
#pragma unroll
        for (int a = 0; a < 8; ++a) {
            const int dim = 8 * b + a;
            h[a] = (_Float16)0.0f;
            if (real && dim < d) {
                const double x = (double)row[dim], c = (double)centre[dim];
                const double y = scale * (x - c);
                float f = (float)y;
                f = fminf(fmaxf(f, -65504.0f), 65504.0f);
                // (no subnormals, whatever the matrix cores make of them)
                h[a] = (_Float16)(fabsf(f) < 0x1p-14f ? 0.0f : f);
                const double g = (double)(float)h[a], left = y - g;
                n2 += g * g;
                r2 += left * left;
                const double m = scale * (fabs(x) + fabs(c));
                mag2 += m * m;
            }
        }
        *(half8 *)(H + ((int64_t)(b / (kStep / 8)) * np + p) * kStep + (b % (kStep / 8)) * 8) = h;
    }
    n2 = wave_sum(n2);
    r2 = wave_sum(r2);
    mag2 = wave_sum(mag2);
    if (lane == 0) {
        if (real) rev.deg[p * rev.stride] = 0;
        // the differences above and those the distances are summed from are
        // rounded to 2^-53 of the values each
        const float rr = (float)((sqrt(r2) + 0x1p-50 * sqrt(mag2)) * (1.0 + 0x1p-20));
        hp[p] = real ? (float)(-0.5 * n2 * (1.0 + (double)kappa)) : -__builtin_inff();
        hm[p] = real ? (float)(-0.5 * n2 * (1.0 - (double)kappa)) : -__builtin_inff();
        r[p] = !real ? 0.0f : rr < 1e30f ? rr : __builtin_inff();
    }
}

// ---------------------------------------------------------------- 2.-4. products
// Tile (256 candidates x 128 queries) of S = <x', x> - (n^2 + n'^2) / 2, which
// is -1/2 of the squared distance: four waves of 128 x 64, stages of 32 dimensions brought to LDS by direct loads, two stages
// in flight.  A lane ends up with 64 candidates (a group) of each of two
// queries.  16-byte pieces of a row are stored under the exclusive or with bits
// of the row, so that the 16 rows of a read phase lie in different banks.
// FIRST: the smallest upper bound of D - r_query of every group of GS
// candidates, u[group][query].  Else: the candidates within the query's
// reach t as bits, word [group][query].
// With BOTH (many points), two points of the slab meet in one tile only, the one
// with the candidate in the later block of 256, and the wave also stores what
// its candidates learn as queries about its 64 queries: groups of the same
// number, of 64 places in a row.  The largest S over the queries by folding
// registers and lanes, the bits by transposing them between lanes: 7 to 10 %
// of the time of the products.
struct KnnTile {
    const _Float16 *H;
    const float *hq;  // -P / 2 (first pass) or -M / 2, both sides
    const float *r;
    int64_t np;       // places, padded to whole tiles
    int blocks;       // stages
    int64_t q0, nq;   // first query of the slab, queries (whole tiles)
};

// XCD x takes 8 of every 64 query tiles.
constexpr int kBandTiles = 8;
struct TileAt {
    int64_t tq, tc;
};
__device__ __forceinline__ TileAt tile_at(const KnnTile &k, bool both) {
    // workgroups b, b + 8, ... run on one XCD: its query tiles go eight at a
    // time against every candidate tile, so that the 64 or so tiles in flight
    // there share their operands in its L2
    const int64_t ct = k.np / kTileC, qt = k.nq / kTileQ, sb0 = k.q0 / kTileC;
    const int x = (int)(blockIdx.x % 8);
    int64_t in = blockIdx.x / 8;
    for (int64_t band = 0; band * 8 * kBandTiles < qt; ++band) {
        // (the direction changes: with BOTH, later tiles have less to meet)
        const int64_t first = (band * 8 + (band & 1 ? 7 - x : x)) * kBandTiles;
        if (first >= qt) continue;
        const int64_t wide = qt - first < kBandTiles ? qt - first : kBandTiles;
        const int64_t skip = both ? first * kTileQ / kTileC : 0;  // blocks of the slab before these
        const int64_t tiles = wide * (ct - skip);
        if (in < tiles) {
            const int64_t c = in / wide;
            return TileAt{first + in % wide, c < sb0 ? c : c + skip};
        }
        in -= tiles;
    }
    return TileAt{-1, 0};
}
static int64_t tile_count(int64_t np, int64_t nq, bool both) {
    const int64_t ct = np / kTileC, qt = nq / kTileQ;
    int64_t most = 0;
    for (int x = 0; x < 8; ++x) {
        int64_t tiles = 0;
        for (int64_t band = 0; band * 8 * kBandTiles < qt; ++band) {
            const int64_t first = (band * 8 + (band & 1 ? 7 - x : x)) * kBandTiles;
            if (first >= qt) continue;
            const int64_t wide = qt - first < kBandTiles ? qt - first : kBandTiles;
            tiles += wide * (ct - (both ? first * kTileQ / kTileC : 0));
        }
        most = tiles > most ? tiles : most;
    }
    return 8 * most;
}

// a candidate may be near if S = -(lower bound of the squared distance) / 2 is
// not below this (h: the query's -M / 2)
__device__ __forceinline__ float threshold(float reach, float r, float h) {
    const float t2 = (reach + r) * (reach + r);
    return -0.5f * t2 - 1e-6f * (t2 - 2.0f * h);
}

// bit matrix of a half wave (row l in lane l) transposed
template <int O>
__device__ __forceinline__ void transpose_step(uint32_t *v, int lane) {
    // bits whose index lacks O stay in lanes without it, the others in lanes with it
    constexpr uint32_t m = O == 16 ? 0xffffu : O == 8 ? 0xff00ffu : O == 4 ? 0x0f0f0f0fu : O == 2 ? 0x33333333u : 0x55555555u;
    const bool up = (lane & O) != 0;
    const uint32_t stay = up ? ~m : m, by = up ? O : 32 - O;
#pragma unroll
    for (int i = 0; i < 4; ++i)
        v[i] = (v[i] & stay) | (__builtin_rotateright32(lane_xor<O>(v[i]), by) & ~stay);
}

// The largest of each of 64 values over the 32 lanes of a half wave: lane l ends
// up with values 2 l and 2 l + 1. A step halves the values a lane holds.
template <int O, int H>
__device__ __forceinline__ void fold(float *v, int lane) {
#pragma unroll
    for (int i = 0; i < H; ++i) {
        if constexpr (O == 16) {
            const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v[i]), __float_as_uint(v[i + H]), false, false);
            v[i] = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
        } else {
            const bool up = (lane & O) != 0;
            const float keep = up ? v[i + H] : v[i], give = up ? v[i] : v[i + H];
            v[i] = fmaxf(keep, __uint_as_float(lane_xor<O>(__float_as_uint(give))));
        }
    }
}

template <bool FIRST, int GS, bool BOTH>
__global__ __launch_bounds__(kBlock, 2) void k_knn_tile(KnnTile k, float *__restrict__ u,
                                                        const float *__restrict__ reach,
                                                        uint64_t *__restrict__ bits) {
    constexpr int kPieces = kStep / 8;
    constexpr int kSlotsC = kTileC * kPieces, kSlots = (kTileC + kTileQ) * kPieces;
    __shared__ half8 s_x[2][kSlots];
    const int lane = (int)(threadIdx.x & (kWave - 1));
    const int w = uniform((int)(threadIdx.x / kWave));
    const int wc = w >> 1, wq = w & 1;
    const TileAt at = tile_at(k, BOTH);
    const int64_t tq = at.tq, tc = at.tc;
    if (tq < 0) return;
    // the slab's blocks, and the queries' block
    const int64_t sb0 = k.q0 / kTileC, sb1 = (k.q0 + k.nq) / kTileC, qb = sb0 + tq * kTileQ / kTileC;
    if (BOTH && tc >= sb0 && tc < qb) return;
    const bool mirror = BOTH && tc > qb && tc < sb1;
    const int64_t c0 = tc * kTileC, ql = tq * kTileQ, q0 = k.q0 + ql;

    auto stage = [&](int buf, int b) {
        const _Float16 *src = k.H + (int64_t)b * k.np * kStep;
#pragma unroll
        for (int a = 0; a < kSlots / kBlock; ++a) {
            const int s = (a * (kBlock / kWave) + w) * kWave + lane;
            const bool cand = s < kSlotsC;
            const int row = (cand ? s : s - kSlotsC) / kPieces;
            const int piece = (s % kPieces) ^ ((row >> 2) & (kPieces - 1));
            const _Float16 *from = src + ((cand ? c0 : q0) + row) * kStep + piece * 8;
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)from,
                                             (__attribute__((address_space(3))) void *)&s_x[buf][(a * (kBlock / kWave) + w) * kWave],
                                             16, 0, 0);
        }
    };
    const int half = lane >> 5, l = lane & 31;
    float16v acc[4][2];
    const float hq[2] = {k.hq[q0 + wq * 64 + l], k.hq[q0 + wq * 64 + 32 + l]};
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            const float4v v = *(const float4v *)(k.hq + c0 + wc * 128 + 32 * t + 8 * a + 4 * half);
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                acc[t][0][4 * a + b] = v[b] + hq[0];
                acc[t][1][4 * a + b] = v[b] + hq[1];
            }
        }
    stage(0, 0);
    for (int b = 0; b < k.blocks; ++b) {
        const int buf = b & 1;
        // this stage has arrived (every wave waits for its own loads), and the
        // other buffer is free
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (b + 1 < k.blocks) stage(buf ^ 1, b + 1);
#pragma unroll
        for (int s = 0; s < kStep / 16; ++s) {
            half8 fc[4], fq[2];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int row = wc * 128 + 32 * t + l;
                fc[t] = s_x[buf][row * kPieces + ((2 * s + half) ^ ((row >> 2) & (kPieces - 1)))];
            }
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const int row = wq * 64 + 32 * t + l;
                fq[t] = s_x[buf][kSlotsC + row * kPieces + ((2 * s + half) ^ ((row >> 2) & (kPieces - 1)))];
            }
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int a = 0; a < 2; ++a)
                    acc[t][a] = __builtin_amdgcn_mfma_f32_32x32x16_f16(fc[t], fq[a], acc[t][a], 0, 0, 0);
        }
    }
    // the largest r of the lane's 64 candidates (rows 32 t + 8 a + 4 half + b)
    float rg = fmaxf(k.r[c0 + wc * 128 + lane], k.r[c0 + wc * 128 + 64 + lane]);
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1)
        if (o != 4) rg = fmaxf(rg, __shfl_xor(rg, o, kWave));
    rg = __shfl(rg, half * 4, kWave);
    const int64_t group = (tc * 2 + wc) * 2 + half;
#pragma unroll
    for (int a = 0; a < 2; ++a) {
        const int64_t q = ql + wq * 64 + 32 * a + l;
        if (FIRST) {
            constexpr int parts = kGroup / GS;
            float m[parts];
#pragma unroll
            for (int t = 0; t < parts; ++t) m[t] = -__builtin_inff();
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int i = 0; i < 16; ++i) m[(16 * t + i) / GS] = fmaxf(m[(16 * t + i) / GS], acc[t][a][i]);
#pragma unroll
            for (int t = 0; t < parts; ++t)
                u[(group * parts + t) * k.nq + q] =
                    (__builtin_sqrtf(fmaxf(-2.0f * m[t], 0.0f)) + rg) * (1.0f + 1e-6f);
        } else {
            const float thr = threshold(reach[q], rg, hq[a]);
            uint64_t word = 0;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                uint32_t part = 0;
#pragma unroll
                for (int i = 0; i < 16; ++i) part |= (!(acc[t][a][i] < thr) ? 1u : 0u) << i;
                word |= (uint64_t)part << (16 * t);
            }
            bits[group * k.nq + q] = word;
        }
    }
    if (!mirror) return;
    // the wave's candidates as queries: place cq + row of the slab
    const int64_t cq = c0 - k.q0 + wc * 128;
    const int64_t qgroup = (q0 + wq * 64) / kGroup;
    float rw = fmaxf(k.r[q0 + wq * 64 + l], k.r[q0 + wq * 64 + 32 + l]);
#pragma unroll
    for (int o = 16; o >= 1; o >>= 1) rw = fmaxf(rw, __shfl_xor(rw, o, kWave));
    if (FIRST) {
        float v[64];
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int i = 0; i < 16; ++i) v[16 * t + i] = fmaxf(acc[t][0][i], acc[t][1][i]);
        fold<16, 32>(v, lane);
        fold<8, 16>(v, lane);
        fold<4, 8>(v, lane);
        fold<2, 4>(v, lane);
        fold<1, 2>(v, lane);
        // values 2 l and 2 l + 1 are rows 32 t + 8 (i >> 2) + 4 half + (i & 3), i = 2 l % 16
        const int row = 32 * (l >> 3) + 8 * ((l & 7) >> 1) + 4 * half + 2 * (l & 1);
        float2 out;
        out.x = (__builtin_sqrtf(fmaxf(-2.0f * v[0], 0.0f)) + rw) * (1.0f + 1e-6f);
        out.y = (__builtin_sqrtf(fmaxf(-2.0f * v[1], 0.0f)) + rw) * (1.0f + 1e-6f);
        *(float2 *)(u + qgroup * k.nq + cq + row) = out;
    } else {
        __syncthreads();  // the stages' LDS is free
        float *s_t = (float *)s_x + w * 128;
#pragma unroll
        for (int a = 0; a < 2; ++a)
            s_t[64 * a + lane] = threshold(reach[cq + 64 * a + lane], rw, k.hq[c0 + wc * 128 + 64 * a + lane]);
        wave_sync();
        uint32_t v[4] = {};  // values 0-31 and 32-63 of the first query, of the second
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int i4 = 0; i4 < 4; ++i4) {
                const float4v th = *(const float4v *)(s_t + 32 * t + 8 * i4 + 4 * half);
#pragma unroll
                for (int b = 0; b < 4; ++b)
#pragma unroll
                    for (int a = 0; a < 2; ++a)
                        v[2 * a + (t >> 1)] |= (!(acc[t][a][4 * i4 + b] < th[b]) ? 1u : 0u) << (16 * (t & 1) + 4 * i4 + b);
            }
        transpose_step<16>(v, lane);
        transpose_step<8>(v, lane);
        transpose_step<4>(v, lane);
        transpose_step<2>(v, lane);
        transpose_step<1>(v, lane);
        // values l and 32 + l over the lanes
        const int row = 32 * (l >> 4) + 8 * ((l & 15) >> 2) + 4 * half + (l & 3);
#pragma unroll
        for (int a = 0; a < 2; ++a)
            bits[qgroup * k.nq + cq + 64 * a + row] = (uint64_t)v[2 + a] << 32 | v[a];
    }
}

// place of bit b of a group's word
__device__ __forceinline__ int64_t bit_place(int64_t group, int b) {
    const int i = b & 15;
    return (group >> 2) * kTileC + ((group >> 1) & 1) * 128 + 32 * (b >> 4) + 8 * (i >> 2) + 4 * (group & 1) + (i & 3);
}

// The reach of a query: the (k + 1)-th smallest of its groups' bounds (of at
// most kPick groups: neighbouring ones are taken together beyond that) plus twice
// its own r.  Sixteen queries a workgroup (a line of bounds each), which then
// take a wave each: up to kPick / 64 bounds a lane, and the value found bit by
// bit (the bounds are not negative, so their bits are ordered) from counts over
// the wave.  Bound by these counts with few groups: 8 us at n = 1000 (16 when
// all queries took the steps of kPick groups).
constexpr int kReachQ = 16;
// the (k + 1)-th smallest of column q of s_u
template <int N>
__device__ __forceinline__ uint32_t smallest(const uint32_t *s_u, int picked, int q, int lane, int k) {
    uint32_t v[N / kWave];
#pragma unroll
    for (int a = 0; a < N / kWave; ++a) {
        const int g = a * kWave + lane;
        v[a] = g < picked ? s_u[g * kReachQ + q] : 0x7fffffffu;
    }
    uint32_t low = 0;  // the value's bits found so far: at most k bounds lie below
    for (int b = 30; b >= 0; --b) {
        const uint32_t mid = low | (1u << b);
        int c = 0;
#pragma unroll
        for (int a = 0; a < N / kWave; ++a) c += __popcll(__builtin_amdgcn_ballot_w64(v[a] < mid));
        if (c <= k) low = mid;
    }
    return low;
}
__global__ __launch_bounds__(kReachQ * kWave) void k_knn_reach(const float *__restrict__ u, int64_t groups,
                                                               int64_t nq, int64_t q0,
                                                               const float *__restrict__ r, int k,
                                                               float *__restrict__ reach) {
    __shared__ uint32_t s_u[kPick * kReachQ];
    const int64_t per = cdiv(groups, kPick);
    const int picked = (int)cdiv(groups, per);
    const int64_t qa = (int64_t)blockIdx.x * kReachQ;
    const int t = threadIdx.x;
    for (int g = t / kReachQ; g < picked; g += kWave) {
        float m = __builtin_inff();
        for (int64_t a = g * per; a < (g + 1) * per && a < groups; ++a) {
            const float v = u[a * nq + qa + t % kReachQ];
            m = v < m ? v : m;  // a NaN never counts as near
        }
        s_u[g * kReachQ + t % kReachQ] = __float_as_uint(m);
    }
    __syncthreads();
    const int q = uniform(t / kWave), lane = t % kWave;
    uint32_t low = 0;
    if (picked <= kPick / 4) low = smallest<kPick / 4>(s_u, picked, q, lane, k);
    else if (picked <= kPick / 2) low = smallest<kPick / 2>(s_u, picked, q, lane, k);
    else low = smallest<kPick>(s_u, picked, q, lane, k);
    if (lane == 0) {
        // fewer than k + 1 groups: no bound
        const float x = __uint_as_float(low);
        reach[qa + q] = (x < 1e30f ? x + 2.0f * r[q0 + qa + q] : __builtin_inff()) * (1.0f + 1e-6f);
    }
}

// The candidates of sixteen queries, from their words to lists of input
// indices; a query with more than kCap (or fewer than k, which finite values
// rule out) goes to the list of the direct kernel, and the rest of its words are not
// looked at (n = 20000 equal rows: 72 us, 277 for all of them).
__global__ __launch_bounds__(kBlock) void k_knn_lists(const uint64_t *__restrict__ bits, int64_t groups,
                                                      int64_t nq, int64_t q0, int64_t n, int64_t S, int k,
                                                      bool mirrored, int32_t *__restrict__ cand,
                                                      int32_t *__restrict__ ncand,
                                                      int32_t *__restrict__ direct,
                                                      int32_t *__restrict__ ndirect) {
    __shared__ int s_n[16];
    const int64_t qa = (int64_t)blockIdx.x * 16;
    const int t = threadIdx.x, qs = t % 16;
    if (t < 16) s_n[t] = 0;
    __syncthreads();
    const int64_t q = qa + qs;  // in the slab
    // groups of the slab before the query's block: words of 64 places in a row
    const int64_t slab0 = q0 / kGroup, own = (q0 + q) / kTileC * (kTileC / kGroup);
    if (q0 + q < n) {
        int turn = 0;
        for (int64_t g = t / 16; g < groups; g += kBlock / 16) {
            uint64_t word = bits[g * nq + q];
            while (word) {
                const int b = __builtin_ctzll(word);
                word &= word - 1;
                const int64_t p = mirrored && g >= slab0 && g < own ? g * kGroup + b : bit_place(g, b);
                if (p >= n || p == q0 + q) continue;
                const int at = atomicAdd(&s_n[qs], 1);
                if (at < kCap) cand[q * kCap + at] = (int32_t)place(p, S, n);
            }
            if (++turn % 4 == 0 && __hip_atomic_load(&s_n[qs], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) > kCap) break;
        }
    }
    __syncthreads();
    if (t < 16 && q0 + q < n) {
        const int c = s_n[t];
        const bool ok = c >= k && c <= kCap;
        ncand[q] = ok ? c : 0;
        if (!ok) direct[atomicAdd(ndirect, 1)] = (int32_t)place(q0 + q, S, n);
    }
}

// ---------------------------------------------------------------- 5. exact
struct Near {
    uint64_t d;  // bits of a distance, which is not negative
    uint32_t j;
    __device__ __forceinline__ bool operator<(const Near &o) const {
        return d < o.d || (d == o.d && j < o.j);
    }
};
template <int O>
__device__ __forceinline__ Near lane_xor(const Near &v) {
    return Near{lane_xor<O>(v.d), lane_xor<O>(v.j)};
}

// (a choice of whole structs would go through memory)
__device__ __forceinline__ Near pick(bool first, const Near &a, const Near &b) {
    return Near{first ? a.d : b.d, first ? a.j : b.j};
}

// the k smallest of m (distance, index) pairs, in order; by one wave, in registers
template <int R>
__device__ __forceinline__ void nearest(const double *sd, const int *sj, int m, int lane, int k,
                                        double *__restrict__ od, int32_t *__restrict__ oj,
                                        const KnnReverse &rev, int64_t at) {
    Near v[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int u = r * kWave + lane;
        const bool in = u < m;
        v[r].d = in ? (uint64_t)__double_as_longlong(sd[u]) : ~0ull;
        v[r].j = in ? (uint32_t)sj[u] : ~0u;
    }
    bitonic_start(v);
    for (int size = R; size <= kWave * R; size <<= 1)
        bitonic_steps(v, lane, size, ((R * lane) & size) == 0);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (R * lane + r < k) {
            od[R * lane + r] = __longlong_as_double((long long)v[r].d);
            oj[R * lane + r] = (int32_t)v[r].j;
            rev.add((int)v[r].j, at + R * lane + r);
        }
    }
}

// One wave a query: the exact distances of its candidates, a lane each, the
// dimensions in ascending order; their rows pass through LDS in pieces of 32
// dimensions (read as whole lines), the next piece on its way while one is
// summed.  Then the k smallest by (distance, index), sorted in registers (through
// LDS the kernel took 45 us at n = 5000, d = 50 instead of 36, and 15 instead of
// 11 at n = 1000).  A query with a distance
// that is not a number goes to the list of the direct kernel, which leaves such
// candidates out.  Many points with many dimensions are bound by the rows, which
// come from beyond the L2 at 6.7 TB/s (two pieces on their way made no
// difference); the reverse neighbours are counted here because that hides the
// additions to memory, 18 G/s, behind them.
template <typename XT>
__global__ __launch_bounds__(kWave) void k_knn_exact(const XT *__restrict__ X, int64_t n, int d, int k,
                                                     int64_t q0, int64_t S,
                                                     const int32_t *__restrict__ cand,
                                                     const int32_t *__restrict__ ncand,
                                                     int32_t *__restrict__ direct,
                                                     int32_t *__restrict__ ndirect,
                                                     double *__restrict__ ld, int32_t *__restrict__ lj,
                                                     KnnReverse rev) {
    constexpr int kDims = 128 / (int)sizeof(XT);  // of a piece: a line
    constexpr int kPitch = kDims + 1;
    __shared__ XT s_c[kWave][kPitch];
    __shared__ XT s_q[kDims];
    __shared__ double sd[kCap];
    __shared__ int sj[kCap];
    const int lane = (int)threadIdx.x;
    const int64_t ql = blockIdx.x;
    const int m = uniform(ncand[ql]);
    if (m == 0) return;
    const int64_t q = place(q0 + ql, S, n);
    const XT *qr = X + q * d;
    const int32_t *list = cand + ql * kCap;
    for (int t = lane; t < m; t += kWave) sj[t] = list[t];
    wave_sync();
    constexpr int kPer = kWave * kDims / kWave;  // values a lane brings of a piece
    bool nan = false;
    for (int c0 = 0; c0 < m; c0 += kWave) {
        const int rows = m - c0 < kWave ? m - c0 : kWave;
        double acc = 0.0;
        XT v[kPer];
        XT qv = (XT)0;
        // value a of a lane: dimension lane % kDims of row a (64 / kDims) + lane / kDims
        auto fetch = [&](int k0) {
            const int dim = k0 + lane % kDims;
#pragma unroll
            for (int a = 0; a < kPer; ++a) {
                const int row = a * (kWave / kDims) + lane / kDims;
                v[a] = row < rows && dim < d ? X[(int64_t)sj[c0 + row] * d + dim] : (XT)0;
            }
            if (lane < kDims) qv = k0 + lane < d ? qr[k0 + lane] : (XT)0;
        };
        fetch(0);
        for (int k0 = 0; k0 < d; k0 += kDims) {
#pragma unroll
            for (int a = 0; a < kPer; ++a) s_c[a * (kWave / kDims) + lane / kDims][lane % kDims] = v[a];
            if (lane < kDims) s_q[lane] = qv;
            wave_sync();
            if (k0 + kDims < d) fetch(k0 + kDims);
            const int kmax = d - k0 < kDims ? d - k0 : kDims;
            if (kmax == kDims) {
#pragma unroll
                for (int s = 0; s < kDims; ++s) {
                    const double dl = (double)s_q[s] - (double)s_c[lane][s];
                    acc = fma(dl, dl, acc);
                }
            } else {
                for (int s = 0; s < kmax; ++s) {
                    const double dl = (double)s_q[s] - (double)s_c[lane][s];
                    acc = fma(dl, dl, acc);
                }
            }
            wave_sync();
        }
        if (lane < rows) sd[c0 + lane] = acc;
        nan |= lane < rows && acc != acc;
    }
    if (__ballot(nan)) {
        if (lane == 0) direct[atomicAdd(ndirect, 1)] = (int32_t)q;
        return;
    }
    wave_sync();
    double *od = ld + q * k;
    int32_t *oj = lj + q * k;
    if (m <= 2 * kWave) nearest<2>(sd, sj, m, lane, k, od, oj, rev, q * k);
    else if (m <= 4 * kWave) nearest<4>(sd, sj, m, lane, k, od, oj, rev, q * k);
    else nearest<kCap / kWave>(sd, sj, m, lane, k, od, oj, rev, q * k);
}

// ---------------------------------------------------------------- direct
// All candidates in double precision for the listed queries: a block owns 64
// of them and streams the candidates in tiles of 128; each thread accumulates a
// 4 x 8 block of squared distances.  The dimensions come through LDS in stages
// of 16, the next one loaded while one is summed.  A running top-k list per
// query is merged with the candidates that beat its k-th entry by a one-wave
// bitonic sort.  Where it serves all queries (an outlier among the points the scale is
// taken from, many equal rows) the products above come on top of it: n = 70000, d =
// 784 took 598 ms with an outlier and 511 with equal rows, 584 and 491 before there
// were any.  Which distances enter a list is now asked for four queries at once and
// the dimensions are summed by twos: 570 and 476 ms.
constexpr int kQ = 64;     // queries per block
constexpr int kC = 128;    // candidates per tile
constexpr int kD = 16;     // dimensions per LDS stage
constexpr int kSort = 256; // merge buffer per wave (>= kMaxK + kC)
template <typename XT>
__global__ __launch_bounds__(kBlock, 2) void k_knn_direct(const XT *__restrict__ X, int64_t n, int d, int k,
                                                          const int32_t *__restrict__ queries,
                                                          const int32_t *__restrict__ nqueries,
                                                          double *__restrict__ ld,
                                                          int32_t *__restrict__ lj, KnnReverse rev) {
    __shared__ double Qs[kD][kQ];
    __shared__ double Cs[kD][kC];
    __shared__ double thr_d[kQ];
    __shared__ int thr_j[kQ];
    __shared__ int len[kQ];
    __shared__ double sd[kBlock / kWave][kSort];
    __shared__ int sj[kBlock / kWave][kSort];

    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int w = tid / kWave;
    const int tq = tid >> 4, tc = tid & 15;
    const int64_t q0 = (int64_t)blockIdx.x * kQ;
    const int64_t nq = *nqueries;
    if (q0 >= nq) return;
    auto query = [&](int64_t q) -> int64_t { return queries[q < nq ? q : nq - 1]; };
    int64_t rows[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) rows[r] = query(q0 + (threadIdx.x >> 4) + 16 * r);
    if (tid < kQ) {
        thr_d[tid] = __builtin_inf();
        thr_j[tid] = INT_MAX;
        len[tid] = 0;
    }
    __syncthreads();

    // the thread's share of a stage: dimension kk of 4 queries and 8
    // candidates, loaded from clamped (always valid) addresses so that all
    // twelve loads are in flight at once; entries outside the data are zeroed
    // when they are stored to LDS
    const int kk = tid & 15;
    XT qr[4], cr[8];
    auto load_stage = [&](int64_t c0, int k0) {
        const int64_t dim = k0 + kk < d ? k0 + kk : d - 1;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            qr[r] = X[rows[r] * d + dim];
        }
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int64_t c = c0 + (tid >> 4) + 16 * r;
            cr[r] = X[(c < n ? c : n - 1) * d + dim];
        }
    };
    load_stage(0, 0);
    for (int64_t c0 = 0; c0 < n; c0 += kC) {
        double acc[4][8];
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int b = 0; b < 8; ++b) acc[a][b] = 0.0;
        for (int k0 = 0; k0 < d; k0 += kD) {
            const bool din = k0 + kk < d;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                int qq = (tid >> 4) + 16 * r;
                Qs[kk][qq] = (q0 + qq < nq && din) ? (double)qr[r] : 0.0;
            }
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                int cc = (tid >> 4) + 16 * r;
                Cs[kk][cc] = (c0 + cc < n && din) ? (double)cr[r] : 0.0;
            }
            __syncthreads();
            // the next stage (of this tile, else the next tile's first) is
            // loaded while this one is summed
            if (k0 + kD < d) load_stage(c0, k0 + kD);
            else if (c0 + kC < n) load_stage(c0 + kC, 0);
            const int kmax = d - k0 < kD ? d - k0 : kD;
            // (by twos: more would take too many registers for two waves a SIMD)
#pragma unroll 2
            for (int s = 0; s < kmax; ++s) {
                double qv[4], cv[8];
#pragma unroll
                for (int a = 0; a < 4; ++a) qv[a] = Qs[s][tq + 16 * a];
#pragma unroll
                for (int b = 0; b < 8; ++b) cv[b] = Cs[s][tc + 16 * b];
#pragma unroll
                for (int a = 0; a < 4; ++a)
#pragma unroll
                    for (int b = 0; b < 8; ++b) {
                        double dl = qv[a] - cv[b];
                        acc[a][b] = fma(dl, dl, acc[a][b]);
                    }
            }
            __syncthreads();
        }
        // merge the tile into the running lists of this wave's 16 queries
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            // rows[a] is the query of the lane's distances: those that enter its list,
            // for the wave's four queries of this row at once
            const int own = 4 * w + (lane >> 4) + 16 * a;
            const double td = thr_d[own];
            const int tj = thr_j[own];
            const bool real = q0 + own < nq;
            uint64_t near[8], any = 0;
#pragma unroll
            for (int b = 0; b < 8; ++b) {
                const int64_t c = c0 + tc + 16 * b;
                const double dv = acc[a][b];
                near[b] = __ballot(real && c < n && c != rows[a] && (dv < td || (dv == td && c < (int64_t)tj)));
                any |= near[b];
            }
            if (any == 0) continue;
            // one query at a time (not unrolled: the merge's registers then
            // fit two waves per SIMD beside the distance tile)
#pragma unroll 1
            for (int r = 0; r < 4; ++r) {
                const int qq = 4 * w + r + 16 * a;
                uint64_t masks[8];
                int tot = 0;
#pragma unroll
                for (int b = 0; b < 8; ++b) {
                    masks[b] = near[b] & (0xffffull << (16 * r));
                    tot += __popcll(masks[b]);
                }
                if (tot == 0) continue;
                const int64_t q = query(q0 + qq);
                const int L = len[qq];
                double *wd = sd[w];
                int *wj = sj[w];
                for (int t = lane; t < L; t += kWave) {
                    // the list was written by this wave earlier: read it past the L1
                    wd[t] = __hip_atomic_load(&ld[q * k + t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    wj[t] = __hip_atomic_load(&lj[q * k + t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
                int off = L;
                const uint64_t below = lane ? (~0ull >> (64 - lane)) : 0ull;
#pragma unroll
                for (int b = 0; b < 8; ++b) {
                    if ((masks[b] >> lane) & 1ull) {
                        int pos = off + __popcll(masks[b] & below);
                        wd[pos] = acc[a][b];
                        wj[pos] = (int)(c0 + tc + 16 * b);
                    }
                    off += __popcll(masks[b]);
                }
                const int total = L + tot;
                int P2 = kWave;
                while (P2 < total) P2 <<= 1;
                for (int t = total + lane; t < P2; t += kWave) {
                    wd[t] = __builtin_inf();
                    wj[t] = INT_MAX;
                }
                wave_sync();
                wave_bitonic(wd, wj, P2, lane);
                const int nl = total < k ? total : k;
                for (int t = lane; t < nl; t += kWave) {
                    ld[q * k + t] = wd[t];
                    lj[q * k + t] = wj[t];
                }
                if (lane == 0) {
                    len[qq] = nl;
                    if (nl == k) {
                        thr_d[qq] = wd[k - 1];
                        thr_j[qq] = wj[k - 1];
                    }
                }
                wave_sync();
            }
        }
        __syncthreads();
    }
    // fewer than k distances are numbers: the point itself takes the other places
    for (int qq = w; qq < kQ && q0 + qq < nq; qq += kBlock / kWave) {
        const int64_t q = query(q0 + qq);
        for (int t = lane; t < k; t += kWave) {
            int j = (int)q;
            if (t < len[qq]) {
                j = __hip_atomic_load(&lj[q * k + t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            } else {
                ld[q * k + t] = __builtin_inf();
                lj[q * k + t] = j;
            }
            rev.add(j, q * k + t);
        }
    }
}

// ---------------------------------------------------------------- host
static int64_t gcd64(int64_t a, int64_t b) {
    while (b) {
        const int64_t t = a % b;
        a = b;
        b = t;
    }
    return a;
}

// odd pieces of one allocation
struct Carve {
    size_t tot = 0;
    size_t take(size_t bytes) {
        const size_t at = tot;
        tot += (bytes + 255) & ~(size_t)255;
        return at;
    }
};

// The k nearest neighbours of every point (k < n): squared distances ld and
// indices lj, n x k, by (distance, index).
template <typename XT>
hts_status knn(hts_ctx ctx, hipStream_t st, const XT *X, int64_t n, int d, int k, double *ld,
               int32_t *lj, Buffer &ws, KnnReverse rev) {
    TimedScope ts(ctx, st, HTS_K_KNN);
    const int64_t np = cdiv(n, kTileC) * kTileC;
    const int64_t groups = np / kGroup;
    const int blocks = (int)cdiv(d, kStep);
    // fine groups where there are few points: the threshold then lies close
    // above the k-th neighbour (about 1.1 k to 1.6 k points within it).  Whole
    // groups from 12288 points on, where halving the products pays for the
    // candidates they add; whole call with groups of 16 and of 64: d = 784, k = 90,
    // 0.89 and 1.12 ms at n = 8192, 1.55 and 1.35 at 12000, 5.5 and 3.9 at 32000;
    // d = 100, k = 128, 0.64 and 0.62 ms at 12000 (at 8192 the lists overflow)
    const int gs = n < 4096 ? 4 : n < 12288 ? 16 : 64;
    const int parts = kGroup / gs;
    const bool both = gs == kGroup;
    // queries a time: the bit matrix and the bounds of a slab stay within
    // kSlabBytes each
    int64_t slab = kSlabBytes / (groups * 8 > groups * parts * 4 ? groups * 8 : groups * parts * 4);
    slab = slab / kTileC * kTileC;
    if (slab < kTileC) slab = kTileC;
    const int64_t nqp = np;
    if (slab > nqp) slab = nqp;
    const int nspread = (int)cdiv(d, kBlock);
    Carve c;
    const size_t o_h = c.take((size_t)blocks * np * kStep * 2), o_centre = c.take((size_t)d * sizeof(XT));
    const size_t o_spread = c.take((size_t)nspread * 4);
    const size_t o_hp = c.take((size_t)np * 4), o_hm = c.take((size_t)np * 4), o_r = c.take((size_t)np * 4);
    const size_t o_u = c.take((size_t)groups * parts * slab * 4), o_bits = c.take((size_t)groups * slab * 8);
    const size_t o_reach = c.take((size_t)slab * 4);
    const size_t o_cand = c.take((size_t)slab * kCap * 4), o_ncand = c.take((size_t)slab * 4);
    const size_t o_direct = c.take((size_t)n * 4), o_ndirect = c.take(4);
    HTS_OKR(ensure(ws, c.tot));
    char *base = (char *)ws.p;
    _Float16 *H = (_Float16 *)(base + o_h);
    XT *centre = (XT *)(base + o_centre);
    float *spread = (float *)(base + o_spread), *hp = (float *)(base + o_hp), *hm = (float *)(base + o_hm);
    float *r = (float *)(base + o_r), *u = (float *)(base + o_u), *reach = (float *)(base + o_reach);
    uint64_t *bits = (uint64_t *)(base + o_bits);
    int32_t *cand = (int32_t *)(base + o_cand), *ncand = (int32_t *)(base + o_ncand);
    int32_t *direct = (int32_t *)(base + o_direct), *ndirect = (int32_t *)(base + o_ndirect);

    int64_t S = (int64_t)(0.6180339887498949 * (double)n);
    if (S < 1) S = 1;
    while (gcd64(S, n) != 1) ++S;
    const float kappa = 2.0f * (float)(blocks * kStep + 8) * 0x1p-23f;
    hipLaunchKernelGGL(k_knn_center<XT>, dim3(nspread), dim3(kBlock), 0, st, X, n, d, centre, spread,
                       ndirect);
    hipLaunchKernelGGL(k_knn_half<XT>, dim3(cdiv(np * kWave, kBlock)), dim3(kBlock), 0, st, X, n, d, centre,
                       spread, nspread, S, np, blocks, kappa, H, hp, hm, r, rev);
    HTS_HIP(hipGetLastError());
    for (int64_t q0 = 0; q0 < n; q0 += slab) {
        const int64_t nq = nqp - q0 < slab ? nqp - q0 : slab;
        const dim3 tiles((unsigned)tile_count(np, nq, both));
        KnnTile kt{H, hp, r, np, blocks, q0, nq};
        if (gs == 4)
            hipLaunchKernelGGL((k_knn_tile<true, 4, false>), tiles, dim3(kBlock), 0, st, kt, u, nullptr, nullptr);
        else if (gs == 16)
            hipLaunchKernelGGL((k_knn_tile<true, 16, false>), tiles, dim3(kBlock), 0, st, kt, u, nullptr, nullptr);
        else
            hipLaunchKernelGGL((k_knn_tile<true, 64, true>), tiles, dim3(kBlock), 0, st, kt, u, nullptr, nullptr);
        hipLaunchKernelGGL(k_knn_reach, dim3(nq / kReachQ), dim3(kReachQ * kWave), 0, st, u,
                           groups * parts, nq, q0, r, k, reach);
        kt.hq = hm;
        if (both)
            hipLaunchKernelGGL((k_knn_tile<false, 64, true>), tiles, dim3(kBlock), 0, st, kt, nullptr, reach, bits);
        else
            hipLaunchKernelGGL((k_knn_tile<false, 64, false>), tiles, dim3(kBlock), 0, st, kt, nullptr, reach, bits);
        hipLaunchKernelGGL(k_knn_lists, dim3(nq / 16), dim3(kBlock), 0, st, bits, groups, nq, q0, n, S, k, both,
                           cand, ncand, direct, ndirect);
        hipLaunchKernelGGL(k_knn_exact<XT>, dim3(n - q0 < nq ? n - q0 : nq), dim3(kWave), 0, st, X, n, d, k,
                           q0, S, cand, ncand, direct, ndirect, ld, lj, rev);
        HTS_HIP(hipGetLastError());
    }
    hipLaunchKernelGGL(k_knn_direct<XT>, dim3(cdiv(n, kQ)), dim3(kBlock), 0, st, X, n, d, k, direct, ndirect,
                       ld, lj, rev);
    HTS_HIP(hipGetLastError());
    return HTS_OK;
}

template hts_status knn<float>(hts_ctx, hipStream_t, const float *, int64_t, int, int, double *, int32_t *,
                               Buffer &, KnnReverse);
template hts_status knn<double>(hts_ctx, hipStream_t, const double *, int64_t, int, int, double *,
                                int32_t *, Buffer &, KnnReverse);

}  // namespace hts
