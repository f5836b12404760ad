// k_affinity.hip -- input affinities P (Sec. 2-A, eq. (1)), truncated to the
// k nearest neighbours and symmetrised.
//
//  1. exact k-NN (k_knn.hip);
//  2. bandwidth per row: beta = 1 / (2 sigma^2) such that the entropy of
//     p_{j|i} equals ln(perplexity), by Newton's steps within a bracket.
//  3. P = (P_c + P_c^T) / (2 n): row i is the union of i's neighbours and of the
//     points whose neighbour i is. The search for neighbours counts the
//     latter and numbers them as they come; a scan places them, and one wave a row
//     sorts the union by column in registers (whatever the order in
//     which they came) and adds the two values of a pair (at most two: a + b =
//     b + a). A scan of the rows' lengths and a copy make it CSR.
#include "hts_impl.hpp"
#include "hts_math.hpp"

namespace hts {

constexpr int kMaxK = kKnnMaxK;

// ---------------------------------------------------------------- perplexity
// A group of 16 lanes per row; the k sorted squared distances of the row are
// spread over the lanes.  Newton's steps on the entropy H (dH / dbeta = -beta
// Var(D)) from beta = 4 / mean(D), of at most a factor of 4 and by bisection
// instead where one leaves the bracket; a step below 1e-9 of beta is the last
// (the next one would be below the rounding of H).  A row whose entropy cannot
// reach the target ends at 2^100, one that overflows at 2^-100.  A row takes 4
// to 8 evaluations of H, a chain of dependent exponentials, sums, a logarithm and
// divisions; four rows a wave share the instructions of all but the first.
// 11 us at n = 1000, 14 at 5000, 73 at 70000; with a wave a row and doubling from
// beta = 1 (7 to 13 evaluations) 14, 34 and 295.
constexpr int kPerpLanes = 16;
template <int SLOTS>
__global__ __launch_bounds__(kBlock) void k_perplexity(const double *__restrict__ ld, int64_t n,
                                                       int k, double log_perp,
                                                       double *__restrict__ pc,
                                                       const int32_t *__restrict__ lj,
                                                       int32_t *__restrict__ knn_out) {
    const int lane = threadIdx.x & (kPerpLanes - 1);
    const int64_t at = ((int64_t)blockIdx.x * kBlock + threadIdx.x) / kPerpLanes;
    const int64_t row = at < n ? at : n - 1;
    const double *di = ld + row * k;
    const double dmin = di[0];  // the row is sorted
    double D[SLOTS], e[SLOTS];
    double sum = 0.0;
#pragma unroll
    for (int u = 0; u < SLOTS; ++u) {
        const int t = lane + kPerpLanes * u;
        D[u] = t < k ? di[t] - dmin : 0.0;
        sum += D[u];
    }
    sum = group_sum<kPerpLanes>(sum);
    const double most = ldexp(1.0, 100), least = ldexp(1.0, -100);
    double beta = fmin(fmax(4.0 * (double)k / sum, least), most);
    double lo = 0.0, hi = __builtin_inf();
    double s = 0.0;
    bool last = false;  // the row's probabilities are those of this beta
    for (int it = 0; it <= 100; ++it) {
        double ls = 0.0, lsd = 0.0, lsdd = 0.0;
#pragma unroll
        for (int u = 0; u < SLOTS; ++u) {
            const double x = exp(-beta * D[u]);
            e[u] = lane + kPerpLanes * u < k ? x : 0.0;
            const double de = D[u] * e[u];
            ls += e[u];
            lsd += de;
            lsdd += D[u] * de;
        }
        s = group_sum<kPerpLanes>(ls);
        if (it == 100 || !__ballot(!last)) break;
        const double mean = group_sum<kPerpLanes>(lsd) / s;
        const double var = group_sum<kPerpLanes>(lsdd) / s - mean * mean;
        const double over = log(s) + beta * mean - log_perp;
        if (last) continue;
        if (over > 0.0) lo = beta;
        else hi = beta;
        const double step = over / (beta * var);
        double next = beta + step;
        last = fabs(step) <= 1e-9 * beta;
        if (!last) {
            next = fmin(fmax(next, 0.25 * beta), 4.0 * beta);
            if (!(next > lo && next < hi)) {
                if (isinf(hi)) {
                    next = 4.0 * beta;
                } else if (lo == 0.0) {
                    next = 0.25 * beta;
                } else {
                    next = 0.5 * (lo + hi);
                    last = next == lo || next == hi;
                }
            }
            if (next >= most || next <= least) {
                next = next >= most ? most : least;
                last = true;
            }
        }
        beta = next;
    }
    if (at >= n) return;
#pragma unroll
    for (int u = 0; u < SLOTS; ++u) {
        const int t = lane + kPerpLanes * u;
        if (t < k) {
            pc[row * k + t] = e[u] / s;
            if (knn_out) knn_out[row * k + t] = lj[row * k + t];
        }
    }
}

// ---------------------------------------------------------------- scan
// Exclusive prefix sums of n counts (every stride-th word), out[n] their total: tiles of 8192 counts,
// each workgroup adding the totals of the tiles before its own (which a first
// launch leaves in part where there are several).
constexpr int kScanThreads = 1024;
constexpr int kScanItems = 8;
constexpr int kScanTile = kScanThreads * kScanItems;

__device__ __forceinline__ int64_t block_sum(int64_t v, int64_t *s) {
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, kWave);
    if ((threadIdx.x & (kWave - 1)) == 0) s[threadIdx.x / kWave] = v;
    __syncthreads();
    int64_t sum = 0;
#pragma unroll
    for (int a = 0; a < kScanThreads / kWave; ++a) sum += s[a];
    __syncthreads();
    return sum;
}

__global__ __launch_bounds__(kScanThreads) void k_scan_totals(const int32_t *__restrict__ in,
                                                              int stride, int64_t n,
                                                              int64_t *__restrict__ part) {
    __shared__ int64_t s[kScanThreads / kWave];
    const int64_t base = (int64_t)blockIdx.x * kScanTile;
    int64_t v = 0;
#pragma unroll
    for (int a = 0; a < kScanItems; ++a) {
        const int64_t i = base + a * kScanThreads + threadIdx.x;
        v += i < n ? in[i * stride] : 0;
    }
    v = block_sum(v, s);
    if (threadIdx.x == 0) part[blockIdx.x] = v;
}

__global__ __launch_bounds__(kScanThreads) void k_scan_counts(const int32_t *__restrict__ in,
                                                              int stride, int64_t n,
                                                              const int64_t *__restrict__ part,
                                                              int64_t *__restrict__ out) {
    __shared__ int64_t s[kScanThreads / kWave];
    const int t = threadIdx.x, lane = t & (kWave - 1);
    int64_t before = 0;
    if (blockIdx.x > 0) {
        for (int64_t b = t; b < blockIdx.x; b += kScanThreads) before += part[b];
        before = block_sum(before, s);
    }
    const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)t * kScanItems;
    int x[kScanItems];
    int64_t own = 0;
#pragma unroll
    for (int a = 0; a < kScanItems; ++a) {
        x[a] = base + a < n ? in[(base + a) * stride] : 0;
        own += x[a];
    }
    int64_t incl = own;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const int64_t u = __shfl_up(incl, o, kWave);
        incl += lane >= o ? u : 0;
    }
    if (lane == kWave - 1) s[t / kWave] = incl;
    __syncthreads();
    int64_t run = before + incl - own;
#pragma unroll
    for (int a = 0; a < kScanThreads / kWave; ++a) run += a < t / kWave ? s[a] : 0;
#pragma unroll
    for (int a = 0; a < kScanItems; ++a) {
        if (base + a < n) out[base + a] = run;
        run += x[a];
        if (base + a == n - 1) out[n] = run;
    }
}

// ---------------------------------------------------------------- symmetrise
struct __attribute__((aligned(16))) Pair {
    double p;
    int32_t col;
    int32_t pad;
};

// Row i's union has room for its k neighbours and the points it is a
// neighbour of, from place i k + off[i] on; k_reverse puts the latter behind the
// former's room.
__global__ __launch_bounds__(kBlock) void k_reverse(const int32_t *__restrict__ lj,
                                                    const double *__restrict__ pc,
                                                    const int32_t *__restrict__ slot,
                                                    const int64_t *__restrict__ off, int64_t n, int k,
                                                    Pair *__restrict__ in) {
    const int64_t e = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (e >= n * k) return;
    const int64_t j = lj[e];
    Pair v;
    v.p = pc[e];
    v.col = (int32_t)(e / k);
    v.pad = 0;
    in[(j + 1) * k + off[j] + slot[e]] = v;
}

constexpr int kRowBits = 9;  // entries of a row that one wave sorts, as bits
constexpr int kRowMax = 1 << kRowBits;
constexpr int64_t kRowPoints = (int64_t)1 << (32 - kRowBits);

// One wave: the union in registers as column and place, sorted; the values
// wait in LDS. Returns the number of columns.
template <int R, typename Get>
__device__ __forceinline__ int sort_row(Get get, int s, int lane, double *val, Pair *out) {
    uint32_t v[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int u = r * kWave + lane;
        v[r] = ~0u;
        if (u < s) {
            const Pair e = get(u);
            v[r] = (uint32_t)e.col << kRowBits | (uint32_t)u;
            val[u] = e.p;
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    bitonic_start(v);
    for (int size = R; size <= kWave * R; size <<= 1)
        bitonic_steps(v, lane, size, ((R * lane) & size) == 0);
    const uint32_t left = __shfl_up(v[R - 1], 1, kWave), right = __shfl_down(v[0], 1, kWave);
    bool first[R], twice[R];
    int c = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const uint32_t col = v[r] >> kRowBits;
        const bool valid = R * lane + r < s;
        first[r] = valid && (r > 0 ? v[r - 1] >> kRowBits != col : lane == 0 || left >> kRowBits != col);
        twice[r] = R * lane + r + 1 < s && (r + 1 < R ? v[r + 1 < R ? r + 1 : 0] : right) >> kRowBits == col;
        c += first[r] ? 1 : 0;
    }
    int incl = c;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const int u = __shfl_up(incl, o, kWave);
        incl += lane >= o ? u : 0;
    }
    int at = incl - c;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (first[r]) {
            Pair e;
            e.p = val[v[r] & (kRowMax - 1)];
            if (twice[r]) e.p += val[(r + 1 < R ? v[r + 1 < R ? r + 1 : 0] : right) & (kRowMax - 1)];
            e.col = (int32_t)(v[r] >> kRowBits);
            e.pad = 0;
            out[at++] = e;
        }
    }
    return __shfl(incl, kWave - 1, kWave);
}

// A workgroup: rows of any length by stable radix passes over the columns,
// between the row's rooms in a and b (the first pass reads through get and
// writes b), then the sum of equal columns into b. Returns the number of columns.
struct LongRow {
    int count[256];
    int wave[kBlock / kWave][256];
    int last;
};
template <typename Get>
__device__ int sort_long_row(Get get, int64_t s, int bits, Pair *a, Pair *b, LongRow &m) {
    const int t = threadIdx.x, w = t / kWave, lane = t & (kWave - 1);
    const uint64_t below = (1ull << lane) - 1ull;
    Pair *src = nullptr, *dst = b;
    for (int shift = 0; shift < bits; shift += 8) {
        auto entry = [&](int64_t u) { return src ? src[u] : get(u); };
        m.count[t] = 0;
        __syncthreads();
        for (int64_t u = t; u < s; u += kBlock) atomicAdd(&m.count[(entry(u).col >> shift) & 255], 1);
        __syncthreads();
        const int own = m.count[t];
        for (int o = 1; o < 256; o <<= 1) {
            const int v = t >= o ? m.count[t - o] : 0;
            __syncthreads();
            m.count[t] += v;
            __syncthreads();
        }
        m.count[t] -= own;  // where the digit goes on
#pragma unroll
        for (int x = 0; x < kBlock / kWave; ++x) m.wave[x][t] = 0;
        __syncthreads();
        for (int64_t u0 = 0; u0 < s; u0 += kBlock) {
            const bool valid = u0 + t < s;
            Pair e{};
            if (valid) e = entry(u0 + t);
            const int dg = (e.col >> shift) & 255;
            uint64_t peers = __ballot(valid);
#pragma unroll
            for (int x = 0; x < 8; ++x) {
                const uint64_t ones = __ballot(valid && ((dg >> x) & 1));
                peers &= ((dg >> x) & 1) ? ones : ~ones;
            }
            const int rank = __popcll(peers & below);
            if (valid && rank == 0) m.wave[w][dg] = __popcll(peers);
            __syncthreads();
            if (valid) {
                int at = m.count[dg] + rank;
                for (int x = 0; x < w; ++x) at += m.wave[x][dg];
                dst[at] = e;
            }
            __syncthreads();
#pragma unroll
            for (int x = 0; x < kBlock / kWave; ++x) {
                m.count[t] += m.wave[x][t];
                m.wave[x][t] = 0;
            }
            __syncthreads();
        }
        src = dst;
        dst = dst == b ? a : b;
    }
    // a chunk is read whole before its columns go to places at or before it
    int total = 0;
    if (t == 0) m.last = -1;
    __syncthreads();
    for (int64_t u0 = 0; u0 < s; u0 += kBlock) {
        const int64_t u = u0 + t;
        const bool valid = u < s;
        Pair e{}, next{};
        next.col = -1;
        if (valid) e = src[u];
        if (u + 1 < s) next = src[u + 1];
        m.count[t] = valid ? e.col : -1;
        const int last = m.last;
        __syncthreads();
        const int prev = t > 0 ? m.count[t - 1] : last;
        const bool first = valid && prev != e.col;
        if (first && next.col == e.col) e.p += next.p;
        const uint64_t mask = __ballot(first);
        if (lane == 0) m.wave[0][w] = __popcll(mask);
        if (t == kBlock - 1) m.last = e.col;
        __syncthreads();
        int at = total + __popcll(mask & below);
#pragma unroll
        for (int x = 0; x < kBlock / kWave; ++x) {
            at += x < w ? m.wave[0][x] : 0;
            total += m.wave[0][x];
        }
        if (first) b[at] = e;
        __syncthreads();
    }
    return total;
}

// The unions, sorted, from their rooms' starts in `out`, and their lengths. A
// wave a row up to kRowMax entries; a workgroup takes a longer row
// together. Sorting both orientations of all entries by (row, column) in radix
// passes, 15 launches and more, took 1.9 ms of device time at n = 70000 and the
// gathers, flags and scans around it 0.4; the kernels from k_reverse on take 0.33
// (n = 5000, whole call: 346 to 201 us; n = 1000: 190 to 127).
__global__ __launch_bounds__(kBlock) void k_unions(const int32_t *__restrict__ lj,
                                                   const double *__restrict__ pc,
                                                   const int64_t *__restrict__ off, int64_t n, int k,
                                                   int bits, Pair *in, Pair *out,
                                                   int32_t *__restrict__ len) {
    constexpr int kRows = kBlock / kWave;
    __shared__ double s_val[kRows][kRowMax];
    __shared__ LongRow s_long;
    const int w = uniform((int)(threadIdx.x / kWave)), lane = (int)(threadIdx.x & (kWave - 1));
    const int64_t r0 = (int64_t)blockIdx.x * kRows, row = r0 + w;
    const bool fits = n <= kRowPoints;
    // The workgroup's longer rows (which of them, as bits) lie far apart: hubs often
    // follow each other in the input, equal rows above all.  n = 20000 equal rows,
    // whose first 90 have 20000 entries each: 990 us with neighbouring rows, 290 so.
    const int64_t far = blockIdx.x + lane * (int64_t)gridDim.x;
    const bool in_far = lane < kRows && far < n;
    uint64_t longer = __ballot(in_far && !(fits && off[in_far ? far + 1 : 0] - off[in_far ? far : 0] + k <= kRowMax));
    auto get = [&](int64_t i, int64_t room, int64_t u) {
        if (u >= k) return in[room + u];
        Pair e;
        e.p = pc[i * k + u];
        e.col = lj[i * k + u];
        e.pad = 0;
        return e;
    };
    if (row < n) {
        const int64_t room = row * k + off[row], s = off[row + 1] - off[row] + k;
        auto mine = [&](int u) { return get(row, room, u); };
        int c = -1;
        if (fits && s <= kRowMax / 2) c = sort_row<kRowMax / 128>(mine, (int)s, lane, s_val[w], out + room);
        else if (fits && s <= kRowMax) c = sort_row<kRowMax / 64>(mine, (int)s, lane, s_val[w], out + room);
        if (c >= 0 && lane == 0) len[row] = c;
    }
    for (; longer; longer &= longer - 1) {
        const int64_t i = blockIdx.x + __builtin_ctzll(longer) * (int64_t)gridDim.x;
        const int64_t room = i * k + off[i], s = off[i + 1] - off[i] + k;
        __syncthreads();
        const int c = sort_long_row([&](int64_t u) { return get(i, room, u); }, s, bits, in + room,
                                    out + room, s_long);
        if (threadIdx.x == 0) len[i] = c;
    }
}

// One wave a row: the CSR arrays, if they hold all entries; the number of
// entries goes to the host either way.
template <typename PT>
__global__ __launch_bounds__(kBlock) void k_csr(const Pair *__restrict__ rows,
                                                const int64_t *__restrict__ off,
                                                const int64_t *__restrict__ at, int64_t n, int k,
                                                int64_t cap, int64_t *__restrict__ row_ptr,
                                                int32_t *__restrict__ col, PT *__restrict__ pval,
                                                int64_t *__restrict__ nnz) {
    const int lane = (int)(threadIdx.x & (kWave - 1));
    const int64_t row = uniform64(((int64_t)blockIdx.x * kBlock + threadIdx.x) / kWave);
    if (row >= n) return;
    if (row == 0 && lane == 0) *nnz = at[n];
    if (at[n] > cap) return;
    const int64_t a0 = at[row], a1 = at[row + 1];
    const Pair *from = rows + row * k + off[row];
    for (int64_t a = a0 + lane; a < a1; a += kWave) {
        const Pair e = from[a - a0];
        col[a] = e.col;
        pval[a] = (PT)(e.p / (2.0 * (double)n));
    }
    if (lane == 0) {
        row_ptr[row] = a0;
        if (row == n - 1) row_ptr[n] = a1;
    }
}

static hts_status scan_counts(hipStream_t st, const int32_t *in, int stride, int64_t n, int64_t *part,
                              int64_t *out) {
    const int64_t tiles = cdiv(n, kScanTile);
    if (tiles > 1) {
        hipLaunchKernelGGL(k_scan_totals, dim3(tiles), dim3(kScanThreads), 0, st, in, stride, n, part);
        HTS_HIP(hipGetLastError());
    }
    hipLaunchKernelGGL(k_scan_counts, dim3(tiles), dim3(kScanThreads), 0, st, in, stride, n, part, out);
    HTS_HIP(hipGetLastError());
    return HTS_OK;
}

// Additions to one line of memory follow each other: with few points, whose
// queries all end at about the same time, every count has a line of its own.
// Whole call with and without: 97 and 111 us at n = 1000, 181 and 178 at 5000.
constexpr int kSpread = 16;
constexpr int64_t kSpreadPoints = 4096;

hts_status affinities(hts_ctx ctx, hipStream_t st, const void *X, int64_t n, int32_t d,
                      int32_t x_dtype, double perplexity, int32_t k, int32_t *knn_idx,
                      int64_t *row_ptr, int32_t *col_idx, void *p_val, int32_t p_dtype,
                      int64_t cap_nnz, int64_t *nnz_out) {
    if (k > kMaxK) return fail(HTS_EINVAL, "hts_build_affinities: k = %d > %d", k, kMaxK);
    const int64_t nk = n * (int64_t)k, m = 2 * nk;
    HTS_OKR(ensure(ctx->aff[0], (size_t)nk * 8));              // list distances
    HTS_OKR(ensure(ctx->aff[1], (size_t)nk * 4 * 2));          // list indices, reverse numbers
    HTS_OKR(ensure(ctx->aff[2], (size_t)nk * 8));              // conditional p
    HTS_OKR(ensure(ctx->aff[3], (size_t)m * sizeof(Pair)));    // the unions as they come
    HTS_OKR(ensure(ctx->aff[4], (size_t)m * sizeof(Pair)));    // sorted
    const int stride = n < kSpreadPoints ? kSpread : 1;
    HTS_OKR(ensure(ctx->aff[5], (size_t)n * 4 * (stride + 1)));  // in-degrees, lengths
    HTS_OKR(ensure(ctx->aff[6], (size_t)(2 * (n + 1) + cdiv(n, kScanTile)) * 8));  // their scans
    double *ld = (double *)ctx->aff[0].p;
    int32_t *lj = (int32_t *)ctx->aff[1].p, *slot = lj + nk;
    double *pc = (double *)ctx->aff[2].p;
    Pair *in = (Pair *)ctx->aff[3].p, *out = (Pair *)ctx->aff[4].p;
    int32_t *deg = (int32_t *)ctx->aff[5].p, *len = deg + n * stride;
    int64_t *off = (int64_t *)ctx->aff[6].p, *at = off + n + 1, *part = at + n + 1;

    if (x_dtype == HTS_F64)
        HTS_OKR(knn<double>(ctx, st, (const double *)X, n, d, k, ld, lj, ctx->aff[7], KnnReverse{deg, slot, stride}));
    else
        HTS_OKR(knn<float>(ctx, st, (const float *)X, n, d, k, ld, lj, ctx->aff[7], KnnReverse{deg, slot, stride}));
    const int64_t row_wgs = cdiv(n * kWave, kBlock);
    const dim3 perp_wgs(cdiv(n * kPerpLanes, kBlock));
    if (k <= 6 * kPerpLanes)
        hipLaunchKernelGGL(k_perplexity<6>, perp_wgs, dim3(kBlock), 0, st, ld, n, k, std::log(perplexity), pc,
                           lj, knn_idx);
    else
        hipLaunchKernelGGL(k_perplexity<kMaxK / kPerpLanes>, perp_wgs, dim3(kBlock), 0, st, ld, n, k,
                           std::log(perplexity), pc, lj, knn_idx);
    HTS_HIP(hipGetLastError());
    HTS_OKR(scan_counts(st, deg, stride, n, part, off));
    hipLaunchKernelGGL(k_reverse, dim3(cdiv(nk, kBlock)), dim3(kBlock), 0, st, lj, pc, slot, off, n, k, in);
    HTS_HIP(hipGetLastError());
    int bits = 1;
    while ((int64_t)1 << bits < n) ++bits;
    hipLaunchKernelGGL(k_unions, dim3(row_wgs), dim3(kBlock), 0, st, lj, pc, off, n, k, bits, in, out, len);
    HTS_HIP(hipGetLastError());
    HTS_OKR(scan_counts(st, len, 1, n, part, at));
    if (p_dtype == HTS_F64)
        hipLaunchKernelGGL(k_csr<double>, dim3(row_wgs), dim3(kBlock), 0, st, out, off, at, n, k, cap_nnz,
                           row_ptr, col_idx, (double *)p_val, ctx->h_count);
    else
        hipLaunchKernelGGL(k_csr<float>, dim3(row_wgs), dim3(kBlock), 0, st, out, off, at, n, k, cap_nnz,
                           row_ptr, col_idx, (float *)p_val, ctx->h_count);
    HTS_HIP(hipGetLastError());
    HTS_HIP(hipStreamSynchronize(st));
    const int64_t nnz = *ctx->h_count;
    *nnz_out = nnz;
    if (nnz > cap_nnz)
        return fail(HTS_ECAPACITY, "hts_build_affinities: nnz = %lld > cap_nnz = %lld",
                    (long long)nnz, (long long)cap_nnz);
    return HTS_OK;
}

}  // namespace hts
