// k_bh.hip -- Barnes-Hut repulsion over the polar quadtree (eq. (19) and the
// depth-first traversal of Sec. 4-B).
//
// A query block is 64 consecutive points of the key order (spatial
// neighbours), one per lane of a wave.  The block walks the tree depth-first;
// the node index is uniform across the wave and each lane keeps its own
// criterion decision: at an internal node a lane either accepts the cell
// (r_cell / d(y_i, m) < theta, tested as t > cosh(r_cell / theta) - 1 with the
// distance argument t in double) and adds N_cell w^2 d dd/dy, or joins the
// lanes that need the children.  Leaves are evaluated exactly, skipping the
// query.
//
// One wave walking the whole tree for its block is a long serial chain, so the
// walk is split in two phases:
//  A. four waves per query block, one per subtree below the root, walk the
//     nodes that hold more than S points; a smaller cell that some lanes
//     reject is handed over with the mask of those lanes instead of being
//     descended;
//  B. waves walk the cells handed over, in chunks of one large cell or several
//     small ones (about 128 points).  The grid holds several times the waves
//     that fit on the chip, so the hardware hands the next waves (and their
//     chunks) to whichever SIMD frees up; long chunks come first.
//     In single precision with few points the waves of a workgroup share a chunk,
//     unless its leaves hold several points.
// Every chunk writes its own partial force per lane and partial Z at a place
// that depends on its phase-A wave and its number there; the combine adds, per
// query block, its waves' partials and chunks in a fixed order, so the result
// does not depend on scheduling.
//
// Bound: both kernels wait for instruction issue and for the latency of the
// dependent steps of a walk (test, ballot, next record), not for memory.  With
// the loop of walk() below a visit takes about 20 scalar and 39 vector
// instructions where a loop with a mask per depth and separate steps for leaves
// took 30 and 41; at N = 70000, theta = 0.5, clusters near the rim, phase B went
// from 554 to 436 us and from 211 to 173 us at the start of a schedule.
//
// The walk is written once over a metric (Geo<MET>): the Poincare disk for
// the hyperbolic gradient, and the Euclidean Student-t kernel of the disk
// coordinates for the first part of the h-SNE gradient (Sec. 4-C), which walks
// the same tree with Euclidean node records.
#include "hts_impl.hpp"
#include "hts_lists.hpp"
#include "hts_math.hpp"

namespace hts {

constexpr int kStats = kBhStats;
constexpr int kAttractLanes = 16;  // lanes per CSR row of the attractive term
constexpr int64_t kAttractWithTopAt = 131072;  // automatic placement threshold (points of a job)
constexpr int kTopDepth = 1;   // phase A splits each query block's walk at this depth ...
constexpr int kTopSlots = 1 << (2 * kTopDepth);  // ... over this many waves

// Chunks of cells one phase-A wave can hand to phase B at the default
// item-list size (kListItems).
constexpr int kListItems = 256;
constexpr int kChunks = 200;
// a chunk closes at this many points (or at S, when that is less); one of at
// least so many is long
constexpr int kChunkPoints = 128;
constexpr int kLongPoints = 96;
constexpr int kWholePoints = 32;  // of a chunk that goes to the list kWhole
// The chunk lists are kept in kGroups parts (the waves of query block b append
// to part b mod kGroups), long and short chunks apart, each with a counter on
// a cache line of its own: the waves' atomics on one counter would serialise.  A third
// list has the chunks of a job in parts that are walked whole all the same; few
// trees have any, and its counter follows the long ones' on their line, which every
// wave reads (gradients of 64 jobs of 500 to 50000 points 1945 us on a line of its own,
// 1937 so).
constexpr int kLong = 0, kShort = 1, kWhole = 2, kKinds = 3;
static_assert(kBhCounts == 2 * kGroups && kGroups == kWave, "counters; a part a lane");

static inline int chunks_of(int list_items) {
    const int64_t l = list_items < kListItems ? list_items : kListItems;
    return (int)((l * kChunks + kListItems - 1) / kListItems);
}

// The chunk lists between the phases, in parts.  Partials sit at fixed places
// (phase-A wave g owns the chunks from g share on), whatever the order of the
// lists.
struct Lists {
    int share;         // chunks a phase-A wave can hand over
    int64_t part;      // entries of one part of one list
    unsigned *count;   // [long and whole, short][kGroups]
    Chunk *chunks;     // [kKinds][kGroups]
    Cell *cells;
    int *handed;       // per phase-A wave
    __device__ __forceinline__ unsigned &counter(int kind, int p) const {
        return count[((kind == kShort ? kGroups : 0) + p) * kCountStride + (kind == kWhole ? 1 : 0)];
    }
    __device__ __forceinline__ Chunk *list(int kind, int p) const {
        return chunks + (kind * kGroups + p) * part;
    }
    // f(chunk, kind) for the chunks of the lists [K0, K1) that wave w of `waves` takes:
    // long ones first, so that the launch does not end on the longest walks
    // (OWN: the waves are known to be whole sets)
    template <int K0, int K1, bool OWN = false, typename F>
    __device__ __forceinline__ void each(int64_t w, int64_t waves, F f) const {
        // every part's length at once where the wave goes through them all, its own part's
        // of all lists where it has one
        int all[K1 - K0] = {};
        const int lane = (int)(threadIdx.x & (kWave - 1));
        const bool own = OWN || own_parts(waves);
        if (own) {
            if (lane < K1 - K0) all[0] = (int)counter(K0 + lane, (int)(w % kGroups));
        } else {
            for (int kind = K0; kind < K1; ++kind) all[kind - K0] = (int)counter(kind, lane);
        }
        int64_t end[K1 - K0];  // of a part's entries of each list, one after another
        deal(
            own, w, waves,
            [&](int p) {
                int64_t n = 0;
#pragma unroll
                for (int a = 0; a < K1 - K0; ++a) {
                    n += own ? __builtin_amdgcn_readlane(all[0], a) : __builtin_amdgcn_readlane(all[a], p);
                    end[a] = n;
                }
                return n;
            },
            [&](int p, int64_t i) {
                int kind = K0;
                int64_t before = 0;
#pragma unroll
                for (int a = 0; a + 1 < K1 - K0; ++a)
                    if (i >= end[a]) {
                        kind = K0 + a + 1;
                        before = end[a];
                    }
                f(list(kind, p)[i - before], kind);
            });
    }
};

// One traversal: where its lists, partials and results are.  (Its node records
// are a parameter of the kernels: what the compiler knows of them there makes
// their loads scalar.)
template <typename T> struct Walks {
    Lists ls;
    T *part0, *part;           // forces per phase-A wave's query and slot, per chunk
    double *ztop, *zitem, *zq; // Z per phase-A wave, chunk, query block
    T *frep, *fattr;
    uint32_t *stats_top, *stats_items;
    unsigned long long *stats;
};
// The metrics of a launch: kBoth serves h-SNE's two traversals of the same
// tree side by side, the hyperbolic and the Euclidean one, in alternating
// workgroups.  Each is a set of long chains that leaves much of the chip idle: at
// n = 20011 phase A of the two takes 46 us instead of 2 x 42, phase B 135 instead
// of 2 x 103.
constexpr int kBoth = 2;

// What a phase-A wave hands over: cells of at most s points, packed in walk
// order into chunks that close at t points.  A cell of fewer nodes than points has
// leaves of several (depth caps, equal points), which no smaller cell divides: up to
// `most` points are handed over then, for phase A would walk its leaves one after another
// (double, n = 3000 in copies of 128, theta = 0: 163 us with cells of 288 points, 300
// with 64 for all, 94 so; depth cap 8 171, 263 and 113).  And chunks of such cells are not
// walked in parts, which are even in nodes: a leaf is one wave's whatever its points,
// and all the next ones wait for it.  They hold no other cells and close at
// kWholePoints (single, a wave a cell, in parts and so: n = 1000 with depth cap 4 60, 76 and 59; n = 6000 in copies of
// 64, theta = 0, 119, 248 and 122).
// SHARES: with these rules, for trees that have such cells; the other walks, chains of
// dependent steps, are spared them and their registers (phase A of 64 jobs of 500 to
// 50000 points 243 us, 270 with them for all).
template <bool SHARES> struct Emit {
    int s, t;
    Lists ls;
    int id0, q0, cnt, part;
    int most, tw;        // SHARES: as above; where chunks of the list kWhole close (t: there are none)
    int done, n;         // chunks appended to the lists; chunks since
    int total, first;    // cells so far; first cell of the open chunk
    int points, limit;   // of the open chunk; SHARES: where it closes, t or tw
    int starts;          // lane j: first cell of chunk done + j
    uint64_t big, whole; // bit j: chunk done + j is long, goes to the list kWhole
    __device__ __forceinline__ void close() {
        // (a choice of the mask to change would put both in scratch memory: 2 us a launch)
        const uint64_t bit = 1ull << (n - 1);
        const bool to_whole = SHARES && limit != t;
        if (SHARES) whole |= to_whole ? bit : 0;
        big |= !to_whole && points >= kLongPoints ? bit : 0;
    }
    // appends the chunks since the last time (the open one included)
    __device__ __forceinline__ void flush(int lane) {
        if (n == 0) return;
        close();
        int end = __shfl_down(starts, 1, kWave);
        if (lane >= n - 1) end = total;
        const Chunk c = chunk_of(id0, done + lane, q0, starts, end, cnt);
        const uint64_t all = n == kWave ? ~0ull : (1ull << n) - 1, below = (1ull << lane) - 1;
#pragma unroll
        for (int kind = 0; kind < (SHARES ? kKinds : kWhole); ++kind) {
            const uint64_t m = kind == kLong ? big : kind == kWhole ? whole : all & ~(SHARES ? big | whole : big);
            if (m == 0) continue;
            int at = 0;
            if (lane == 0) at = (int)atomicAdd(&ls.counter(kind, part), (unsigned)__popcll(m));
            at = __shfl(at, 0, kWave);
            if ((m >> lane) & 1ull) ls.list(kind, part)[at + __popcll(m & below)] = c;
        }
        done += n;
        n = 0;
        big = whole = 0;
        points = 0;
    }
    // true when the cell was taken; no more will be once the share is full, and
    // the walk ends here (kend) for another to go on
    __device__ __forceinline__ bool take(int lane, int node, int next, uint64_t mask, int count, int &kend) {
        int here = t;
        if constexpr (SHARES) {
            const bool shared = next - node - 1 < count;
            if (count > s && !(shared && count <= most)) return false;
            here = shared ? tw : t;
        } else if (count > s) {
            return false;
        }
        if (n == 0 || points >= (SHARES ? limit : t) || (SHARES && here != limit) || total - first == kWave) {
            if (done + n == ls.share) {
                kend = 0;
                return false;
            }
            if (n == kWave) flush(lane);
            if (n) close();
            starts = lane == n ? total : starts;
            ++n;
            first = total;
            points = 0;
            if (SHARES) limit = here;
        }
        if (lane == 0) ls.cells[wave_cells(id0) + total] = Cell{node, next, mask};
        ++total;
        points += count;
        if (total == ls.share * kCells) kend = 0;
        return true;
    }
};

// Largest cell handed to phase B, for a job of n points (S:
// hts_set_item_points).  In double precision a walk of 288 points is a long
// chain, and cells are as small as leave enough work to each: gradient with 32
// and 64 points at n = 500 92 and 118 us, with 64 and 128 at n = 16000 290 and
// 306, at 30000 560 and 550 (and 380 and 348 early in a schedule).
template <typename T>
__host__ __device__ inline int item_size(int64_t n, int S) {
    if (S != kAutoItemPoints || sizeof(T) == 4) return S;
    return n < 2048 ? 32 : n < 20480 ? 64 : n < 32768 ? 128 : S;
}

// A chunk's forces and Z are summed in parts of kPartNodes nodes when n, the points of
// its job (times the metrics of the launch), is below kPartsBelow: in single
// precision cells keep their 288 points (smaller ones would change the sums
// of Z), and with few of them phase B is as long as the longest walk.  A launch
// that holds nothing else, in the automatic shape, walks the parts of a chunk
// with kManyWaves waves below kManyBelow points in all and kFewWaves from there
// on; any other launch walks them one after another, to the same sums.
// Gradient call near the rim, a wave a chunk and so, us: n = 300 100 and 71, 1000
// 139 and 80, 3000 184 and 106, 5500 227 and 120, 9000 194 and 149, 12000 207
// and 170; over the stages 13000 187-226 and 182-207, 16000 190-210 and 205-220:
// the terms held in LDS keep waves off the chip, which then counts for more than the
// chain.  8 and 4 waves: n = 5003 115-129 and 124-133, 7000 137-156 and 143-149.
// Phase B alone at n = 2000: 84 and 32.  Parts of 16, 32 or 48 nodes and fewer
// terms held were not better.  Parts one after another cost 1 to 2 % of a
// launch (16 jobs of 500 to 20000 points: 305 and 310).
// Where cells may hold more than kPartsCell points (hts_set_item_points) all are
// walked whole: a part goes through the links of its cell's nodes before it, so a
// cell's time grows with the square of its parts (gradient near the rim, n = 12000,
// in parts and whole: cells of 2048 points 459 and 508 us, of 4096 1301 and 623).
constexpr int64_t kPartsBelow = 12288, kManyBelow = 6144;
constexpr int kPartsCell = 2048;
constexpr int kManyWaves = 8, kFewWaves = 4;
constexpr int kPartNodes = 24;
// Workgroups that have a chunk of the list kWhole before any has a second one: few chunks
// have a SIMD of their own, many fill the workgroups that fit on the chip beside their
// LDS (n = 1000 with depth cap 4, n = 6000 in copies of 64 with theta = 0: 59 and 122 us;
// all waves of a workgroup first 76 and 128, all workgroups first 59 and 250).
constexpr int64_t kSpread = 512;
static_assert(kSpread % kGroups == 0, "whole sets");
template <typename T> __host__ __device__ inline bool in_parts(int64_t n) {
    return sizeof(T) == 4 && n < kPartsBelow;
}

// The sums of a chunk's parts up to one, for each lane: Z's terms of the cell that
// goes on in the next, Z of the cells before, forces.  done: parts summed so
// far, counted on over the workgroup's chunks.
constexpr int kHold = 24;  // Z terms a part may hold before it waits
static_assert(kHold <= kWave, "a weight a lane");
struct Sums {
    float zw[kWave], fx[kWave], fy[kWave];
    double z[kWave];
    int done;
};
template <int WAVES> struct PartLds {
    Sums s;
    float w[WAVES][kHold * kWave];
    uint32_t stats[WAVES][kStats];
};

// Z terms of a walk that goes on in a cell: they wait for the sum of the terms
// before them, so that the sum is that of a single walk.
struct Hold {
    Sums &s;
    float *w;       // [kHold][kWave]
    int turn, lane, n;
    bool open;      // terms are added
    float weights;  // lane i: of term i
    __device__ __forceinline__ void add(float weight, float t, float &zw) {
        if (!open) {
            if (n < kHold) {
                w[n * kWave + lane] = t;
                weights = lane == n ? weight : weights;
                ++n;
                return;
            }
            take(zw);
        }
        zw += weight * t;
    }
    // (the waves of the parts before are in this workgroup, and wait for those
    // before them at most)
    __device__ __forceinline__ void wait() const {
        while (__hip_atomic_load(&s.done, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) != turn)
            __builtin_amdgcn_s_sleep(1);
    }
    __device__ __forceinline__ void take(float &zw) {
        if (open) return;
        wait();
        zw = s.zw[lane];
#pragma unroll 8
        for (int i = 0; i < n; ++i)
            zw += __int_as_float(__builtin_amdgcn_readlane(__float_as_int(weights), i)) * w[i * kWave + lane];
        open = true;
    }
};

struct Counters {
    unsigned long long test = 0, acc = 0, pair = 0, step = 0, work = 0, cover = 0;
};

// keeps a value where it was formed (in vector registers)
__device__ __forceinline__ void pin(float &v) { asm volatile("" : "+v"(v)); }
__device__ __forceinline__ void pin(double &v) { asm volatile("" : "+v"(v)); }

// record k (a 32-bit byte offset: kMaxNodes records stay below 4 GiB)
template <typename T>
__device__ __forceinline__ NodeRec<T> node_at(const NodeRec<T> *__restrict__ nodes, int k) {
    static_assert((uint64_t)kMaxNodes * sizeof(NodeRec<T>) <= (1ull << 32), "32-bit offsets");
    return *(const NodeRec<T> *)((const char *)nodes + (uint32_t)k * (uint32_t)sizeof(NodeRec<T>));
}

// Depth-first walk of the pre-order range [k, kend), a subtree or the children
// of a cell, for the lanes in mask0.  With EMIT, internal nodes that some lanes
// reject are offered to em and skipped when it takes them.  The walk's Z terms
// are summed in T, the caller adds the sum to its Z.  at and resume (the nodes from
// which the wave and its lanes go on) are where the walk ended.
// A lane that accepts a node sits out its subtree: it waits for the index
// after it (resume), so the lanes that need node k are those with
// resume <= k, and no mask has to be kept per depth.  A leaf of one point
// needs no step of its own: its record's c makes "t > c" mean "not the query
// itself" (two points of different leaves differ in coordinates, so their t is
// positive), its index after the subtree is k + 1 either way, and the query
// itself, rejecting it, moves on to k + 1 like everybody.
// Node records are read with scalar loads (the index is uniform): the next
// one is under way while the term is formed, whose parts of the current record
// are taken to vector registers before, so the loaded record can replace it.
// The index after the last node is readable (the node arrays hold more than M
// records: their capacity n_max (depth cap + 1) + 1 exceeds any node count).
// THRU marks the walks of phase B, which run among many waves and are bound
// by instruction issue: there the term's wave-uniform choice of branch pays.
template <typename T, int MET, bool STATS, bool EMIT, bool THRU = false, bool HOLD = false, bool SHARES = false>
__device__ __forceinline__ void walk(const NodeRec<T> *__restrict__ nodes,
                                     const PointRec<T> *__restrict__ spts, const PointRec<T> &me,
                                     int64_t q, int lane, int &at, int kend, int &resume, Emit<SHARES> &em, T &fx,
                                     T &fy, T &zw, Counters &c, Hold *held = nullptr) {
    int k = at;
    NodeRec<T> cur = node_at(nodes, k);
    do {
        const uint32_t link = (uint32_t)uniform((int)cur.link);
        const int over = (int)(link & kNextMask);
        const uint64_t m = __builtin_amdgcn_ballot_w64(resume <= k);
        if (STATS) c.step += 1;
        if (link & kManyBit) {  // a leaf of several points
            const bool in = __builtin_amdgcn_inverse_ballot_w64(m);
            const int64_t first = (int64_t)__double_as_longlong(cur.c);
            const int cnt = uniform(cur.count);
            PointRec<T> ahead = spts[first];
            for (int a = 0; a < cnt; ++a) {
                const PointRec<T> o = ahead;
                ahead = spts[first + (a + 1 < cnt ? a + 1 : a)];
                const bool use = in && (first + a) != q;
                auto term = [&]() {
                    double dd;
                    const double t = Geo<MET>::arg(me, o.x, o.y, o.ia, dd);
                    return Geo<MET>::template repel<THRU>(me, part_of<T>(me, o.x, o.y, o.ia, (T)1), t, dd, fx, fy);
                };
                if constexpr (HOLD) {
                    T w = 0;
                    if (use) w = term();
                    held->add((T)1, w, zw);
                } else if (use) {
                    zw += term();
                }
                if (STATS) {
                    const int u = __popcll(__ballot(use));
                    c.pair += u;
                    c.cover += u;
                }
            }
            k = over;
            cur = node_at(nodes, k);
            continue;
        }
        double dd;
        const double t = Geo<MET>::arg(me, cur.mx, cur.my, cur.ib, dd);
        const uint64_t am = __builtin_amdgcn_ballot_w64(!(t <= cur.c)) & m;  // a NaN stays visible
        const uint64_t rej = m & ~am;
        Part<T> p = part_of<T>(me, cur.mx, cur.my, cur.ib, (T)cur.count);
        pin(p.ux);
        pin(p.uy);
        if (MET == 0) pin(p.ib);
        pin(p.weight);
        if (STATS) {
            const int um = __popcll(am);
            if (over == k + 1) {
                c.pair += um;
                c.cover += um;
            } else {
                c.test += __popcll(m);
                c.acc += um;
                c.cover += (unsigned long long)um * (unsigned)cur.count;
            }
            c.work += am != 0;
        }
        int next = rej ? k + 1 : over;
        if (EMIT && rej && over != k + 1 && em.take(lane, k, over, rej, uniform(cur.count), kend))
            next = over;
        k = next;
        cur = node_at(nodes, k);
        asm volatile("" ::: "memory");  // the load stays ahead of the term
        if constexpr (HOLD) {
            T w = 0;
            if (__builtin_amdgcn_inverse_ballot_w64(am)) {
                resume = over;
                w = Geo<MET>::template repel<THRU>(me, p, t, dd, fx, fy);
            }
            if (am) held->add(p.weight, w, zw);
        } else if (__builtin_amdgcn_inverse_ballot_w64(am)) {
            resume = over;
            zw += p.weight * Geo<MET>::template repel<THRU>(me, p, t, dd, fx, fy);
        }
    } while (k < kend);
    at = k;
}
// the lanes of a walk from node k: where they resume
__device__ __forceinline__ int resume_at(uint64_t mask, int k) {
    return __builtin_amdgcn_inverse_ballot_w64(mask) ? k : 0x7fffffff;
}

template <bool STATS>
__device__ __forceinline__ void put_stats(uint32_t *__restrict__ sp, const Counters &c) {
    if (!STATS) return;
    sp[0] = (uint32_t)c.test;
    sp[1] = (uint32_t)c.acc;
    sp[2] = (uint32_t)c.pair;
    sp[3] = (uint32_t)c.step;
    sp[4] = (uint32_t)c.work;
    sp[5] = (uint32_t)c.cover;
}

// the attractive rows of both traversals, row_blocks workgroups each
template <typename T>
__device__ __forceinline__ void both_rows(const Walks<T> &a, const Walks<T> &b, int64_t block,
                                          int64_t row_blocks, const uint32_t *__restrict__ perm,
                                          const PointRec<T> *__restrict__ pts, const int64_t *__restrict__ rp,
                                          const int32_t *__restrict__ col, const T *__restrict__ val,
                                          int64_t n, uint32_t *__restrict__ err) {
    if (block < row_blocks)
        attract_rows<T, kAttractLanes, 0>(block * blockDim.x + threadIdx.x, perm, pts, rp, col, val, n, a.fattr,
                                          err);
    else
        attract_rows<T, kAttractLanes, 1>((block - row_blocks) * blockDim.x + threadIdx.x, perm, pts, rp, col,
                                          val, n, b.fattr, err);
}

// Phase A: the walk of a query block over the nodes of more than S points,
// split over kTopSlots = 4^kTopDepth waves.  Slot s owns one node f of the
// frontier at depth kTopDepth (its base-4 digits pick the child at each level
// below the root; a leaf above that depth belongs to the slot whose remaining
// digits are 0; a slot naming a missing child is idle).  The wave first tests
// the ancestors of f for its lanes -- a lane that accepts one leaves the walk --
// then walks f's subtree, handing over the cells that are small enough.  An
// ancestor's term and counters belong to the one slot whose digits below it are all 0, so every lane meets every cell exactly as in a
// single depth-first walk.  These waves are latency-bound chains.  The
// attractive term (first sum of eq. (15)) runs either in this launch, in the
// workgroups from top_blocks on, where its waves compete with the chains for
// issue and are hidden when the chains are long, or in the last workgroups of
// phase B's launch (hts_set_attract_launch).
template <typename T, int MET, bool STATS>
__device__ __forceinline__ void top_walks(const NodeRec<T> *__restrict__ nodes, const Walks<T> &w, int64_t block,
                                          const int32_t *__restrict__ node_start, const Jobs &jb,
                                          const PointRec<T> *__restrict__ spts, int64_t nqb, int S,
                                          int64_t n, int kinds) {
    const Lists &ls = w.ls;
    T *__restrict__ part0 = w.part0;
    const int64_t g = block * (kBlock / kWave) + uniform((int)(threadIdx.x / kWave));
    const int64_t qb = g / kTopSlots;
    const int slot = (int)(g % kTopSlots);
    if (qb >= nqb) return;
    const int lane = (int)(threadIdx.x & (kWave - 1));
    int64_t q0;
    int cnt, job;
    jb.block(qb, q0, cnt, job);
    q0 = uniform((int)q0);
    cnt = uniform(cnt);
    job = uniform(job);
    const int64_t q = q0 + lane;
    const bool valid = lane < cnt;
    const PointRec<T> me = spts[valid ? q : q0];
    // the job's tree: the pre-order range from its root
    int a = uniform(node_start[jb.off[job]]);
    const int64_t nj = jb.off[job + 1] - jb.off[job];
    const int s = uniform(item_size<T>(nj, S));
    const bool parts = S <= kPartsCell && in_parts<T>(kinds * nj);
    T fx = 0, fy = 0;
    double z = 0.0;
    Counters c;
    uint64_t m = __ballot(valid);
    bool live = true, shares = false;
    for (int d = 0; d < kTopDepth; ++d) {
        const NodeRec<T> A = nodes[a];
        const uint32_t nxd = (uint32_t)uniform((int)A.link);
        const int nx = (int)(nxd & kNextMask);
        // without shared leaves a tree has 1.6 to 2.4 nodes a point
        if (d == 0 && parts) shares = 5 * (nx - a) < 7 * (int64_t)uniform(A.count);
        // this slot owns node a when its digits below depth d are all 0
        const bool owner = (slot & ((1 << (2 * (kTopDepth - d))) - 1)) == 0;
        if (nx == a + 1) {  // a leaf above the frontier depth: its owner walks it
            live = owner;
            break;
        }
        const bool in = (m >> lane) & 1ull;
        bool acc = false;
        if (in) {
            double dd;
            const double t = Geo<MET>::arg(me, A.mx, A.my, A.ib, dd);
            acc = t > A.c;
            if (acc && owner)
                z += (double)((T)A.count *
                              Geo<MET>::repel(me, part_of<T>(me, A.mx, A.my, A.ib, (T)A.count), t, dd, fx, fy));
        }
        const uint64_t rej = __ballot(in && !acc);
        if (STATS && owner) {
            const uint64_t am = __ballot(acc);
            c.test += __popcll(m);
            c.acc += __popcll(am);
            c.step += 1;
            c.work += am != 0;
            c.cover += (unsigned long long)__popcll(am) * (unsigned)A.count;
        }
        m = rej;
        if (!m) break;
        // the child picked by this slot's digit at depth d + 1
        const int digit = (slot >> (2 * (kTopDepth - 1 - d))) & 3;
        int ch = a + 1;
        for (int i = 0; i < digit && ch < nx; ++i)
            ch = (int)((uint32_t)uniform((int)nodes[ch].link) & kNextMask);
        if (ch >= nx) {
            live = false;
            break;
        }
        a = ch;
    }
    int handed = 0;
    if (live && m) {
        const int nxa = (int)((uint32_t)uniform((int)nodes[a].link) & kNextMask);
        T zw = 0;
        int resume = resume_at(m, a);
        if (ls.share > 0) {
            const int t = s < kChunkPoints ? s : kChunkPoints;
            const int tw = !parts ? t : t == kWholePoints ? t + 1 : kWholePoints;
            const int most = S == kAutoItemPoints ? kAutoItemPoints : s;
            auto hand_over = [&](auto em) {
                walk<T, MET, STATS, true>(nodes, spts, me, q, lane, a, nxa, resume, em, fx, fy, zw, c);
                em.flush(lane);
                handed = em.done;
            };
            // (in double precision two walks would take more registers)
            if (sizeof(T) == 8 || shares)
                hand_over(Emit<true>{s, t, ls, (int)(g * ls.share), (int)q0, cnt, (int)(qb % kGroups), most, tw});
            else if constexpr (sizeof(T) == 4)
                hand_over(Emit<false>{s, t, ls, (int)(g * ls.share), (int)q0, cnt, (int)(qb % kGroups)});
        }
        // beyond a full share the walk is one of phase B: with the offers still made,
        // the gradient near the rim at n = 70000 took 2226 us with a list of one, now 1748
        Emit<false> none{};
        if (a < nxa) walk<T, MET, STATS, false, true>(nodes, spts, me, q, lane, a, nxa, resume, none, fx, fy, zw, c);
        z += (double)zw;
    }
    if (valid) {
        part0[((int64_t)slot * n + q) * 2] = fx;
        part0[((int64_t)slot * n + q) * 2 + 1] = fy;
    }
    const double zs = wave_sum(z);
    if (lane == 0) {
        w.ztop[g] = zs;
        ls.handed[g] = handed;
        put_stats<STATS>(w.stats_top + g * kStats, c);
    }
}

template <typename T, int MET, bool STATS>
__global__ __launch_bounds__(kBlock) void k_bh_top(
    const NodeRec<T> *__restrict__ nodes, const NodeRec<T> *__restrict__ enodes, Walks<T> a, Walks<T> b,
    const int32_t *__restrict__ node_start, Jobs jb,
    const PointRec<T> *__restrict__ spts, int64_t nqb, int S, int64_t n, int64_t top_blocks,
    int64_t row_blocks, const uint32_t *__restrict__ perm, const PointRec<T> *__restrict__ pts,
    const int64_t *__restrict__ rp, const int32_t *__restrict__ col, const T *__restrict__ val,
    uint32_t *__restrict__ err) {
    const int64_t at = (int64_t)blockIdx.x;
    if constexpr (MET == kBoth) {
        if (at < 2 * top_blocks) {
            if (at & 1) top_walks<T, 1, STATS>(enodes, b, at >> 1, node_start, jb, spts, nqb, S, n, 2);
            else top_walks<T, 0, STATS>(nodes, a, at >> 1, node_start, jb, spts, nqb, S, n, 2);
        } else {
            both_rows<T>(a, b, at - 2 * top_blocks, row_blocks, perm, pts, rp, col, val, n, err);
        }
    } else {
        if (at < top_blocks) {
            top_walks<T, MET, STATS>(nodes, a, at, node_start, jb, spts, nqb, S, n, 1);
        } else {
            attract_rows<T, kAttractLanes, MET>((at - top_blocks) * kBlock + threadIdx.x, perm, pts, rp, col,
                                                val, n, a.fattr, err);
        }
    }
}

// Before a traversal: clears the item-list counter (a kernel, not a memset,
// so the sequence can be captured in a graph), and as asked writes the point
// records of Y and the criterion thresholds of the internal nodes.
template <typename T>
__global__ __launch_bounds__(kBlock) void k_bh_prepare(const T *__restrict__ Y, int64_t n,
                                                       PointRec<T> *__restrict__ pts, bool points,
                                                       NodeRec<T> *__restrict__ nodes,
                                                       const double *__restrict__ r_cell,
                                                       const int32_t *__restrict__ d_m,
                                                       double theta, bool thresholds,
                                                       unsigned *__restrict__ counts,
                                                       uint32_t *__restrict__ err) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (counts) clear_counts(counts, i);
    if (points && i < n) prep_point<T>(Y, i, pts, err);
    if (thresholds) {
        const int64_t M = *d_m;
        const int64_t G = (int64_t)gridDim.x * kBlock;
        for (int64_t k = i; k < M; k += G) {
            const uint32_t next = nodes[k].link & kNextMask;
            if ((int64_t)next != k + 1) nodes[k].c = node_threshold(r_cell[k], theta);
        }
    }
}

// A chunk as the waves of phase B see it: its cells one after another, node
// by node, and for a chunk in parts the nodes of each part.
template <typename T> struct Work {
    int q0, id, cnt, cells;
    PointRec<T> me;
    int64_t q;
    Cell mine{};  // lane j: cell j
    __device__ __forceinline__ Work(const Chunk &r, const Cell *__restrict__ list,
                                    const PointRec<T> *__restrict__ spts, int lane)
        : q0(uniform(r.q0)), id(uniform(r.id)), cnt(uniform(r.cnt)), cells(uniform(r.cells)) {
        me = spts[lane < cnt ? q0 + lane : q0];
        q = (int64_t)q0 + lane;
        if (lane < cells) mine = list[chunk_cells(id, uniform(r.first)) + lane];
    }
    __device__ __forceinline__ int node(int j) const { return __builtin_amdgcn_readlane(mine.node, j); }
    __device__ __forceinline__ int next(int j) const { return __builtin_amdgcn_readlane(mine.next, j); }
    __device__ __forceinline__ uint64_t mask(int j) const {
        return ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(mine.mask >> 32), j) << 32) |
               (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)mine.mask, j);
    }
};

// A chunk's result: one partial force per lane and one partial Z.
template <typename T, bool STATS>
__device__ __forceinline__ void put_chunk(const Work<T> &k, T fx, T fy, double z, const Counters &c, int lane,
                                          T *__restrict__ part, double *__restrict__ zitem,
                                          uint32_t *__restrict__ stats_items) {
    if (lane < k.cnt) {
        T *o = part + ((int64_t)k.id * kWave + lane) * 2;
        o[0] = fx;
        o[1] = fy;
    }
    const double zs = wave_sum(z);
    if (lane == 0) {
        zitem[k.id] = zs;
        put_stats<STATS>(stats_items + (int64_t)k.id * kStats, c);
    }
}

// A chunk's cells one after another, by one wave.
template <typename T, int MET, bool STATS>
__device__ __forceinline__ void whole_walk(const NodeRec<T> *__restrict__ nodes,
                                           const PointRec<T> *__restrict__ spts, const Work<T> &k, int lane,
                                           T &fx, T &fy, double &z, Counters &c) {
    Emit<false> none{};
    for (int j = 0; j < k.cells; ++j) {
        int at = k.node(j) + 1, resume = resume_at(k.mask(j), at);
        T zw = 0;
        walk<T, MET, STATS, false, true>(nodes, spts, k.me, k.q, lane, at, k.next(j), resume, none, fx, fy, zw, c);
        z += (double)zw;
    }
}

// Phase B: the chunks of small cells.
template <typename T, int MET, bool STATS, bool PARTS>
__device__ __forceinline__ void item_walks(const NodeRec<T> *__restrict__ nodes, const Lists &ls,
                                           T *__restrict__ part, double *__restrict__ zitem,
                                           uint32_t *__restrict__ stats_items, int64_t block,
                                           int64_t item_blocks, const PointRec<T> *__restrict__ spts,
                                           const Jobs &jb, int kinds) {
    const int lane = (int)(threadIdx.x & (kWave - 1));
    const int wpb = (int)(blockDim.x / kWave);
    const int64_t at = block * wpb + uniform((int)(threadIdx.x / kWave));
    ls.each<kLong, PARTS ? kKinds : kWhole>(at, item_blocks * wpb, [&](const Chunk &r, int kind) {
        const Work<T> k(r, ls.cells, spts, lane);
        T fx = 0, fy = 0;
        double z = 0.0;
        Counters c;
        bool parts = false;
        if constexpr (PARTS) {
            const int job = uniform(jb.pjob[k.q0]);
            parts = kind != kWhole && in_parts<T>(kinds * (jb.off[job + 1] - jb.off[job]));
        }
        if (!parts) {
            whole_walk<T, MET, STATS>(nodes, spts, k, lane, fx, fy, z, c);
        } else {
            Emit<false> none{};
            T sx = 0, sy = 0;  // of the parts before
            double sz = 0.0;
            int b = 0, hi = kPartNodes;  // the cell's first node, the part's end
            auto close = [&]() {
                sx += fx;
                sy += fy;
                sz += z;
                fx = fy = 0;
                z = 0.0;
                hi += kPartNodes;
            };
            for (int j = 0; j < k.cells; ++j) {
                const int first = k.node(j) + 1, next = k.next(j);
                int at = first, resume = resume_at(k.mask(j), first);
                T zw = 0;
                do {
                    while (b + (at - first) >= hi) close();
                    const int stop = first + (hi - b) < next ? first + (hi - b) : next;
                    walk<T, MET, STATS, false, true>(nodes, spts, k.me, k.q, lane, at, stop, resume, none, fx, fy,
                                                     zw, c);
                } while (at < next);
                const int e = b + (next - first);
                while (e > hi) close();
                if (b < hi - kPartNodes) sz += (double)zw;  // begun in another part
                else z += (double)zw;
                b = e;
            }
            close();
            fx = sx;
            fy = sy;
            z = sz;
        }
        put_chunk<T, STATS>(k, fx, fy, z, c, lane, part, zitem, stats_items);
    });
}

// The same sums with the parts of a chunk spread over the waves of a workgroup, wave p
// taking parts p, p + WAVES, ...  A part that starts inside a cell looks for its
// first node's ancestors there (the nodes before it that end behind it) and
// takes the lanes through their criteria, whose terms belong to the parts
// before; its Z terms of that cell wait for the sum of those.
template <int MET, bool STATS, int WAVES>
__device__ __forceinline__ void part_walks(PartLds<WAVES> &lds, const NodeRec<float> *__restrict__ nodes,
                                           const Lists &ls, float *__restrict__ part,
                                           double *__restrict__ zitem, uint32_t *__restrict__ stats_items,
                                           int64_t block, int64_t item_blocks,
                                           const PointRec<float> *__restrict__ spts) {
    using T = float;
    constexpr int kLinks = 8;  // 64 links of a cell each, in registers
    const int lane = (int)(threadIdx.x & (kWave - 1)), p = uniform((int)(threadIdx.x / kWave));
    Sums &s = lds.s;
    if (threadIdx.x == 0) s.done = 0;
    __syncthreads();
    int turn = 0;  // of the chunk's first part
    ls.each<kLong, kWhole, true>(block, item_blocks, [&](const Chunk &r, int) {
        const Work<T> k(r, ls.cells, spts, lane);
        int total = 0;
        for (int j = 0; j < k.cells; ++j) total += k.next(j) - k.node(j) - 1;
        const int n = (total + kPartNodes - 1) / kPartNodes;
        Counters c;
        Emit<false> none{};
        int j = 0, b = 0;  // the part's first cell and its first node
        int linked = -1;   // the cell whose links are in
        int links[kLinks];
        for (int i = p; i < n; i += WAVES) {
            const int lo = i * kPartNodes, hi = lo + kPartNodes < total ? lo + kPartNodes : total;
            T fx = 0, fy = 0, zw = 0, zlast = 0;
            double z = 0.0;
            Hold held{s, lds.w[p], turn + i, lane, 0, true, 0.0f};
            bool in = false, ends = false;  // the first cell began before; and ends here
            for (; j < k.cells && b < hi; ++j) {
                const int first = k.node(j) + 1, next = k.next(j), e = b + (next - first);
                if (e > lo) {
                    int at = first, resume = resume_at(k.mask(j), first);
                    const int stop = hi < e ? first + (hi - b) : next;
                    if (lo > b) {
                        in = true;
                        ends = e <= hi;
                        held.open = false;
                        const int from = first + (lo - b);
                        if (linked != j) {
#pragma unroll
                            for (int u = 0; u < kLinks; ++u) {
                                const int o = first + u * kWave + lane;
                                links[u] = o < next ? (int)(nodes[o].link & kNextMask) : 0;
                            }
                            linked = j;
                        }
                        at = from;
                        bool inside = true;
                        auto ancestors = [&](int base, int over_lane) {
                            uint64_t over = __ballot(base + lane < from && over_lane > from);
                            while (over && inside) {
                                const int a = base + __builtin_ctzll(over);
                                over &= over - 1;
                                const NodeRec<T> A = node_at(nodes, a);
                                double dd;
                                const double t = Geo<MET>::arg(k.me, A.mx, A.my, A.ib, dd);
                                const int nx = (int)((uint32_t)uniform((int)A.link) & kNextMask);
                                if (resume <= a && !(t <= A.c)) resume = nx;
                                if (!__ballot(resume <= from)) {
                                    at = nx;
                                    inside = false;
                                }
                            }
                        };
#pragma unroll
                        for (int u = 0; u < kLinks; ++u)
                            if (inside && first + u * kWave < from) ancestors(first + u * kWave, links[u]);
                        for (int o = first + kLinks * kWave; o < from && inside; o += kWave)
                            ancestors(o, o + lane < from ? (int)(nodes[o + lane].link & kNextMask) : 0);
                        if (at < stop)
                            walk<T, MET, STATS, false, true, true>(nodes, spts, k.me, k.q, lane, at, stop, resume,
                                                                   none, fx, fy, zw, c, &held);
                    } else {
                        zlast = 0;
                        walk<T, MET, STATS, false, true>(nodes, spts, k.me, k.q, lane, at, stop, resume, none, fx,
                                                         fy, zlast, c);
                        if (e <= hi) z += (double)zlast;
                    }
                    if (e > hi) break;
                }
                b = e;
            }
            held.wait();
            if (in) held.take(zw);
            T sx = i ? s.fx[lane] : 0, sy = i ? s.fy[lane] : 0;
            double sz = i ? s.z[lane] : 0.0;
            if (ends) sz += (double)zw;
            sx += fx;
            sy += fy;
            sz += z;
            if (i + 1 < n) {
                s.zw[lane] = in && !ends ? zw : zlast;
                s.fx[lane] = sx;
                s.fy[lane] = sy;
                s.z[lane] = sz;
            }
            __hip_atomic_store(&s.done, turn + i + 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
            if (i + 1 < n) continue;
            if (lane < k.cnt) {
                T *o = part + ((int64_t)k.id * kWave + lane) * 2;
                o[0] = sx;
                o[1] = sy;
            }
            const double zs = wave_sum(sz);
            if (lane == 0) zitem[k.id] = zs;
        }
        turn += n;
        if (STATS) {
            if (lane == 0) put_stats<STATS>(lds.stats[p], c);
            __syncthreads();
            if (p == 0 && lane < kStats) {
                uint32_t v = 0;
                for (int a = 0; a < WAVES; ++a) v += lds.stats[a][lane];
                stats_items[(int64_t)k.id * kStats + lane] = v;
            }
            __syncthreads();
        }
    });
    const int64_t b0 = block / kSpread * kSpread, bs = item_blocks - b0 < kSpread ? item_blocks - b0 : kSpread;
    ls.each<kWhole, kKinds, true>(b0 * WAVES + p * bs + (block - b0), item_blocks * WAVES, [&](const Chunk &r, int) {
        const Work<T> k(r, ls.cells, spts, lane);
        T fx = 0, fy = 0;
        double z = 0.0;
        Counters c;
        whole_walk<T, MET, STATS>(nodes, spts, k, lane, fx, fy, z, c);
        put_chunk<T, STATS>(k, fx, fy, z, c, lane, part, zitem, stats_items);
    });
}

// MODE: no chunk of the launch is in parts (kNoParts), some may be (kSomeParts), or
// all are and a workgroup of MODE waves takes a chunk.
constexpr int kNoParts = 0, kSomeParts = 1;
// The workgroups past the chunks' compute the attractive rows when they run
// here: they start last, and fill the chip while the longest walks finish.
template <typename T, int MET, bool STATS, int MODE>
__global__ __launch_bounds__(MODE == kManyWaves ? kManyWaves * kWave : kBlock) void k_bh_items(
    const NodeRec<T> *__restrict__ nodes, const PointRec<T> *__restrict__ spts, Lists ls,
    T *__restrict__ part, double *__restrict__ zitem, uint32_t *__restrict__ stats_items,
    int64_t item_blocks, const uint32_t *__restrict__ perm, const PointRec<T> *__restrict__ pts,
    const int64_t *__restrict__ rp, const int32_t *__restrict__ col, const T *__restrict__ val,
    int64_t n, T *__restrict__ fattr, uint32_t *__restrict__ err,
    const NodeRec<T> *__restrict__ enodes, Walks<T> a, Walks<T> b, int64_t row_blocks, Jobs jb) {
    const int64_t at = (int64_t)blockIdx.x;
    if constexpr (MODE > kSomeParts) {
        __shared__ PartLds<MODE> s;
        constexpr int kinds = MET == kBoth ? 2 : 1;
        if (at < kinds * item_blocks) {
            if (MET == kBoth && (at & 1))
                part_walks<1, STATS>(s, enodes, b.ls, b.part, b.zitem, b.stats_items, at / kinds, item_blocks, spts);
            else
                part_walks<0, STATS>(s, nodes, ls, part, zitem, stats_items, at / kinds, item_blocks, spts);
            return;
        }
    }
    if constexpr (MET == kBoth) {
        if (at < 2 * item_blocks && MODE <= kSomeParts) {
            if (at & 1)
                item_walks<T, 1, STATS, MODE == kSomeParts>(enodes, b.ls, b.part, b.zitem, b.stats_items, at >> 1,
                                                            item_blocks, spts, jb, 2);
            else
                item_walks<T, 0, STATS, MODE == kSomeParts>(nodes, ls, part, zitem, stats_items, at >> 1,
                                                            item_blocks, spts, jb, 2);
        } else {
            both_rows<T>(a, b, at - 2 * item_blocks, row_blocks, perm, pts, rp, col, val, n, err);
        }
    } else {
        if (at < item_blocks && MODE <= kSomeParts) {
            item_walks<T, MET, STATS, MODE == kSomeParts>(nodes, ls, part, zitem, stats_items, at, item_blocks,
                                                          spts, jb, 1);
        } else {
            attract_rows<T, kAttractLanes, MET>((at - item_blocks) * blockDim.x + threadIdx.x, perm, pts, rp,
                                                col, val, n, fattr, err);
        }
    }
}

// Combine, stage 1: one workgroup per query block, one wave per phase-A slot.
// Wave s adds its slot's phase-A partial and then its chunks' partials in
// order (eight loads in flight at a time); the first wave then adds the four
// slot sums in slot order and applies the query's common factor of the terms.
// The order of every sum is fixed, so the result does not depend on
// scheduling.  The counters of the block are added to the caller's totals.
static_assert(kTopSlots == kBlock / kWave, "one wave per phase-A slot");
template <typename T, int MET, bool STATS>
__device__ __forceinline__ void gather_block(const Walks<T> &w, int64_t qb,
                                             const PointRec<T> *__restrict__ spts, const Jobs &jb,
                                             int64_t n) {
    __shared__ T s_f[kTopSlots][2][kWave];
    __shared__ double s_z[kTopSlots];
    const T *__restrict__ part0 = w.part0, *__restrict__ part = w.part;
    const double *__restrict__ zitem = w.zitem;
    const uint32_t *__restrict__ stats_top = w.stats_top, *__restrict__ stats_items = w.stats_items;
    unsigned long long *__restrict__ stats = w.stats;
    const int sl = (int)(threadIdx.x / kWave);
    const int lane = (int)(threadIdx.x & (kWave - 1));
    int64_t q0;
    int cnt, job;
    jb.block(qb, q0, cnt, job);
    const int64_t q = q0 + lane;
    const bool valid = lane < cnt;
    T fx = 0, fy = 0;
    const int64_t g = qb * kTopSlots + sl;
    const int64_t b0 = g * w.ls.share;
    const int ni = uniform(w.ls.handed[g]);
    if (valid) {
        fx = part0[((int64_t)sl * n + q) * 2];
        fy = part0[((int64_t)sl * n + q) * 2 + 1];
        constexpr int U = 8;
        int j = 0;
        for (; j + U <= ni; j += U) {
            T px[U], py[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const T *p = part + ((b0 + j + u) * kWave + lane) * 2;
                px[u] = p[0];
                py[u] = p[1];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                fx += px[u];
                fy += py[u];
            }
        }
        for (; j < ni; ++j) {
            const T *p = part + ((b0 + j) * kWave + lane) * 2;
            fx += p[0];
            fy += p[1];
        }
    }
    double zl = 0.0;
    for (int j = lane; j < ni; j += kWave) zl += zitem[b0 + j];
    const double zs = w.ztop[g] + wave_sum(zl);
    s_f[sl][0][lane] = fx;
    s_f[sl][1][lane] = fy;
    if (lane == 0) s_z[sl] = zs;
    if (STATS) {
        unsigned long long s_it[kStats], s_all[kStats];
#pragma unroll
        for (int a = 0; a < kStats; ++a) s_it[a] = s_all[a] = 0;
        for (int j = lane; j < ni; j += kWave)
#pragma unroll
            for (int a = 0; a < kStats; ++a) s_it[a] += stats_items[(b0 + j) * kStats + a];
        if (lane == 0)
#pragma unroll
            for (int a = 0; a < kStats; ++a) s_all[a] = stats_top[g * kStats + a];
#pragma unroll
        for (int a = 0; a < kStats; ++a) {
            unsigned long long v = s_it[a], u = s_all[a];
#pragma unroll
            for (int o = 32; o >= 1; o >>= 1) {
                v += __shfl_xor(v, o, 64);
                u += __shfl_xor(u, o, 64);
            }
            if (lane == 0) {
                atomicAdd(&stats[a], v + u);
                atomicAdd(&stats[kStats + a], v);
            }
        }
    }
    __syncthreads();
    if (sl != 0) return;
    double zb = s_z[0];
#pragma unroll
    for (int a = 1; a < kTopSlots; ++a) zb += s_z[a];
    if (valid) {
        T sx = s_f[0][0][lane], sy = s_f[0][1][lane];
#pragma unroll
        for (int a = 1; a < kTopSlots; ++a) {
            sx += s_f[a][0][lane];
            sy += s_f[a][1][lane];
        }
        // the query's common factor of the repulsive terms, once
        const double f = Geo<MET>::qfactor(spts[q]);
        w.frep[2 * q] = (T)(f * (double)sx);
        w.frep[2 * q + 1] = (T)(f * (double)sy);
    }
    if (lane == 0) w.zq[qb] = zb;
}

template <typename T, int MET, bool STATS>
__global__ __launch_bounds__(kBlock) void k_bh_gather(Walks<T> a, Walks<T> b,
                                                      const PointRec<T> *__restrict__ spts, Jobs jb,
                                                      int64_t n) {
    const int64_t at = (int64_t)blockIdx.x;
    if constexpr (MET == kBoth) {
        if (at & 1) gather_block<T, 1, STATS>(b, at >> 1, spts, jb, n);
        else gather_block<T, 0, STATS>(a, at >> 1, spts, jb, n);
    } else {
        gather_block<T, MET, STATS>(a, at, spts, jb, n);
    }
}

// Combine, stage 2: g_i = 4 (a F_attr,i - F_rep,i / Z) scattered to input
// order; with BOTH, the Euclidean traversal's gradient plus scale times the
// hyperbolic one's.  Z of a job is the sum of its query blocks'
// totals, formed by every workgroup that holds points of the job the same way
// (one wave: four lane-strided partial sums per lane, then a fixed butterfly), so
// all of them use the same value; the workgroup holding the job's first point
// writes it to z_dev (with BOTH, the Euclidean one first).
__device__ __forceinline__ double job_z(const double *__restrict__ zq, int64_t a0, int64_t a1, int lane) {
    // four partial sums per lane keep four loads in flight
    double z0 = 0.0, z1 = 0.0, z2 = 0.0, z3 = 0.0;
    int64_t a = a0 + lane;
    for (; a + 3 * kWave < a1; a += 4 * kWave) {
        z0 += zq[a];
        z1 += zq[a + kWave];
        z2 += zq[a + 2 * kWave];
        z3 += zq[a + 3 * kWave];
    }
    for (; a < a1; a += kWave) z0 += zq[a];
    return wave_sum((z0 + z1) + (z2 + z3));
}

template <typename T, bool BOTH>
__global__ __launch_bounds__(kBlock) void k_bh_finalize(
    Walks<T> w, Walks<T> euclid, Jobs jb, const uint32_t *__restrict__ perm, int64_t n, double ex,
    const double *__restrict__ ex_job, double scale, T *__restrict__ grad,
    double *__restrict__ z_dev, uint32_t *__restrict__ err) {
    __shared__ double s_z[kBlock];  // a job holds at least one point of the workgroup
    __shared__ double s_e;
    const int64_t b0 = (int64_t)blockIdx.x * kBlock;
    const int64_t bl = (b0 + kBlock < n ? b0 + kBlock : n) - 1;
    const int j0 = jb.pjob[b0], j1 = jb.pjob[bl];
    const int wave = (int)(threadIdx.x / kWave), lane = (int)(threadIdx.x & (kWave - 1));
    for (int j = j0 + wave; j <= j1; j += kBlock / kWave) {
        const double zs = job_z(w.zq, jb.job_qb[j], jb.job_qb[j + 1], lane);
        if (lane == 0) {
            s_z[j - j0] = zs;
            const int64_t f = jb.off[j];
            if (f >= b0 && f <= bl) z_dev[BOTH ? 1 : j] = zs;
        }
    }
    if (BOTH && wave == 1) {  // one job
        const double zs = job_z(euclid.zq, jb.job_qb[0], jb.job_qb[1], lane);
        if (lane == 0) {
            s_e = zs;
            if (b0 == 0) z_dev[0] = zs;
        }
    }
    __syncthreads();
    const int64_t q = b0 + threadIdx.x;
    if (q >= n) return;
    // sorted positions of a job cover the same range as its input points
    const int job = jb.pjob[q];
    const double a = ex_job ? ex_job[job] : ex;
    const uint32_t i = perm[q];
    auto force = [&](const Walks<T> &v, double Z, double &gx, double &gy) {
        const double inv = 1.0 / Z;
        gx = 4.0 * (a * (double)v.fattr[2 * q] - (double)v.frep[2 * q] * inv);
        gy = 4.0 * (a * (double)v.fattr[2 * q + 1] - (double)v.frep[2 * q + 1] * inv);
    };
    double gx, gy;
    force(w, s_z[job - j0], gx, gy);
    if (BOTH) {
        double fx, fy;
        force(euclid, s_e, fx, fy);
        gx = (double)(T)fx + scale * gx;
        gy = (double)(T)fy + scale * gy;
    }
    const T ox = (T)gx, oy = (T)gy;
    if (!isfinite(ox) || !isfinite(oy)) atomicOr(err, HTS_ERR_NONFINITE_GRAD);
    grad[2 * (int64_t)i] = ox;
    grad[2 * (int64_t)i + 1] = oy;
}

// The traversal's workspace (chunk lists, partials, per-block sums) in
// ctx->part: the offsets of its regions and the total, for nqb query blocks
// and n points (with the counters' region when stats are asked).
struct BhLayout {
    enum { Counts, Handed, Part0, Ztop, Chunks, Cells, Part, Zitem, Frep, Zq, Stats, R };
    size_t off[R];
    size_t tot;
};
template <typename T>
static BhLayout bh_layout(int list_items, int64_t nqb, int64_t n, bool stats) {
    const size_t nw = (size_t)nqb * kTopSlots;
    const size_t share = chunks_of(list_items), chunks = nw * share;
    const size_t padded = (size_t)cdiv(nqb, kGroups) * kGroups * kTopSlots;  // waves, whole parts
    size_t sizes[BhLayout::R];
    sizes[BhLayout::Counts] = (size_t)kBhCounts * kCountStride * 4;
    sizes[BhLayout::Handed] = nw * 4;
    sizes[BhLayout::Part0] = (size_t)kTopSlots * n * 2 * sizeof(T);
    sizes[BhLayout::Ztop] = nw * 8;
    sizes[BhLayout::Chunks] = kKinds * padded * share * sizeof(Chunk);
    sizes[BhLayout::Cells] = chunks * kCells * sizeof(Cell);
    sizes[BhLayout::Part] = chunks * kWave * 2 * sizeof(T);
    sizes[BhLayout::Zitem] = chunks * 8;
    sizes[BhLayout::Frep] = (size_t)n * 2 * sizeof(T);
    sizes[BhLayout::Zq] = (size_t)nqb * 8;
    sizes[BhLayout::Stats] = stats ? (nw + chunks) * kStats * 4 : 0;
    BhLayout L;
    L.tot = 0;
    for (int a = 0; a < BhLayout::R; ++a) {
        L.off[a] = L.tot;
        L.tot += (sizes[a] + 255) & ~(size_t)255;
    }
    return L;
}

template <typename T>
hts_status bh_item_counter(hts_ctx ctx, hts_tree t, int64_t n, unsigned **counter) {
    const BhLayout L = bh_layout<T>(ctx->list_items, t->nqb, n, false);
    HTS_OKR(ensure(ctx->part, L.tot));
    *counter = (unsigned *)((char *)ctx->part.p + L.off[BhLayout::Counts]);
    return HTS_OK;
}
template hts_status bh_item_counter<float>(hts_ctx, hts_tree, int64_t, unsigned **);
template hts_status bh_item_counter<double>(hts_ctx, hts_tree, int64_t, unsigned **);

// the places of a traversal in its piece of the workspace
template <typename T>
static Walks<T> walks_at(char *base, const BhLayout &L, int list_items, int64_t nqb, T *fattr,
                         uint64_t *stats) {
    const size_t *off = L.off;
    Walks<T> w;
    w.ls.share = chunks_of(list_items);
    w.ls.part = cdiv(nqb, kGroups) * kTopSlots * w.ls.share;
    w.ls.count = (unsigned *)(base + off[BhLayout::Counts]);
    w.ls.chunks = (Chunk *)(base + off[BhLayout::Chunks]);
    w.ls.cells = (Cell *)(base + off[BhLayout::Cells]);
    w.ls.handed = (int *)(base + off[BhLayout::Handed]);
    w.part0 = (T *)(base + off[BhLayout::Part0]);
    w.part = (T *)(base + off[BhLayout::Part]);
    w.ztop = (double *)(base + off[BhLayout::Ztop]);
    w.zitem = (double *)(base + off[BhLayout::Zitem]);
    w.zq = (double *)(base + off[BhLayout::Zq]);
    w.frep = (T *)(base + off[BhLayout::Frep]);
    w.fattr = fattr;
    w.stats_top = stats ? (uint32_t *)(base + off[BhLayout::Stats]) : nullptr;
    w.stats_items = stats ? w.stats_top + (size_t)nqb * kTopSlots * kStats : nullptr;
    w.stats = (unsigned long long *)stats;
    return w;
}

// the launches of the traversals and their combine, but for the preparation
template <typename T, int MET, bool STATS>
static void launch_walks(hts_ctx ctx, hipStream_t st, hts_tree t, int64_t n, const Walks<T> &a,
                         const Walks<T> &b, PointRec<T> *pts, const int64_t *rp, const int32_t *col,
                         const T *val, double ex, const double *ex_job, double scale, T *grad,
                         double *z_dev) {
    constexpr int kinds = MET == kBoth ? 2 : 1;
    const int64_t nqb = t->nqb, nw = nqb * kTopSlots;  // phase-A waves
    const Jobs jb = jobs_of(t);
    const PointRec<T> *spts = (const PointRec<T> *)t->spts;
    const NodeRec<T> *nodes = (const NodeRec<T> *)t->nodes, *enodes = (const NodeRec<T> *)t->enodes;
    // the attractive rows beside phase A (long chains hide them) or at the end
    // of phase B; automatic: beside phase A for a job of 131072 points or more
    const int64_t largest = t->jobs_set ? t->max_job : n;
    const bool attract_a = ctx->attract_at == 1 || (ctx->attract_at == 0 && largest >= kAttractWithTopAt);
    // phase B: items_grid workgroups of items_waves waves, by default 12
    // waves per phase-A wave (about one per chunk: the hardware hands each
    // freed wave slot the next chunk)
    int mode = kNoParts;
    const bool short_cells = ctx->item_points <= kPartsCell;
    if (short_cells && in_parts<T>(kinds * (t->jobs_set ? t->min_job : n))) mode = kSomeParts;
    // (cells below a part's size leave the other waves of a workgroup without one: n = 3000
    // late in a schedule with cells of 8 points 127 us, 116 so)
    if (short_cells && ctx->item_points >= kPartNodes && ctx->items_grid == 0 && ctx->items_waves == 1 &&
        in_parts<T>(kinds * n))
        mode = kinds * n < kManyBelow ? kManyWaves : kFewWaves;
    const bool parts = mode > kSomeParts;
    const int wpb = parts ? mode : ctx->items_waves;
    const int takers = parts ? 1 : wpb;  // waves of a workgroup that take a chunk each
    int64_t gi = ctx->items_grid > 0 ? (int64_t)ctx->items_grid
                                     : cdiv(cdiv(nqb, kGroups) * kTopSlots * 12, takers) * kGroups;
    // (no more than take a chunk each, in whole sets: a set a part)
    const int64_t most = cdiv(cdiv(nw * a.ls.share, takers), kGroups) * kGroups;
    if (gi > most) gi = most;
    if (gi < 1) gi = ctx->items_grid > 0 ? 1 : kGroups;  // an empty list (nothing can be handed over)
    {
        TimedScope ts(ctx, st, HTS_K_TRAVERSE);
        const int64_t top_blocks = cdiv(nw, kBlock / kWave);
        const int64_t rows = attract_a ? cdiv(n * kAttractLanes, kBlock) : 0;
        hipLaunchKernelGGL((k_bh_top<T, MET, STATS>), dim3(kinds * (top_blocks + rows)), dim3(kBlock), 0, st,
                           nodes, enodes, a, b, t->node_start, jb, spts, nqb, ctx->item_points, n, top_blocks, rows, t->perm, pts, rp,
                           col, val, ctx->d_err);
    }
    {
        TimedScope ts(ctx, st, HTS_K_ITEMS);
        const int64_t rows = attract_a ? 0 : cdiv(n * kAttractLanes, wpb * kWave);
        auto items = k_bh_items<T, MET, STATS, kNoParts>;
        if constexpr (sizeof(T) == 4) {
            if (mode == kSomeParts) items = k_bh_items<T, MET, STATS, kSomeParts>;
            if (mode == kFewWaves) items = k_bh_items<T, MET, STATS, kFewWaves>;
            if (mode == kManyWaves) items = k_bh_items<T, MET, STATS, kManyWaves>;
        }
        hipLaunchKernelGGL(items, dim3(kinds * (gi + rows)), dim3(wpb * kWave), 0, st, nodes, spts, a.ls, a.part,
                           a.zitem, a.stats_items, gi, t->perm, pts, rp, col, val, n, a.fattr, ctx->d_err, enodes, a,
                           b, rows, jb);
    }
    TimedScope ts(ctx, st, HTS_K_FINALIZE);
    hipLaunchKernelGGL((k_bh_gather<T, MET, STATS>), dim3(kinds * nqb), dim3(kBlock), 0, st, a, b, spts, jb, n);
    hipLaunchKernelGGL((k_bh_finalize<T, MET == kBoth>), dim3(cdiv(n, kBlock)), dim3(kBlock), 0, st, a, b, jb,
                       t->perm, n, ex, ex_job, scale, grad, z_dev, ctx->d_err);
}

template <typename T>
hts_status launch_bh_repulsion(hts_ctx ctx, hipStream_t st, hts_tree t, int64_t n,
                               BhPrep<T> prep, PointRec<T> *pts, const int64_t *rp,
                               const int32_t *col, const T *val, T *fattr, double ex,
                               const double *ex_job, T *grad, double *z_dev, uint64_t *stats) {
    const BhLayout L = bh_layout<T>(ctx->list_items, t->nqb, n, stats != nullptr);
    HTS_OKR(ensure(ctx->part, L.tot));
    const Walks<T> w = walks_at<T>((char *)ctx->part.p, L, ctx->list_items, t->nqb, fattr, stats);
    if (prep.points || prep.thresholds || prep.clear) {
        // one thread per point, and the node thresholds strided over the same grid
        const int64_t gp = cdiv(n, kBlock) > 64 ? cdiv(n, kBlock) : 64;
        hipLaunchKernelGGL(k_bh_prepare<T>, dim3(gp), dim3(kBlock), 0, st, prep.Y, n, pts, prep.points,
                           (NodeRec<T> *)t->nodes, t->r_cell, t->d_m, prep.theta, prep.thresholds,
                           prep.clear ? w.ls.count : nullptr, ctx->d_err);
    }
    if (stats)
        launch_walks<T, 0, true>(ctx, st, t, n, w, w, pts, rp, col, val, ex, ex_job, 1.0, grad, z_dev);
    else
        launch_walks<T, 0, false>(ctx, st, t, n, w, w, pts, rp, col, val, ex, ex_job, 1.0, grad, z_dev);
    HTS_HIP(hipGetLastError());
    return HTS_OK;
}

template <typename T>
hts_status launch_bh_hsne(hts_ctx ctx, hipStream_t st, hts_tree t, int64_t n, const T *Y, double theta,
                          PointRec<T> *pts, const int64_t *rp, const int32_t *col, const T *val, T *fattr,
                          T *fattr_euclid, double ex, double lambda, T *grad, double *z_dev, uint64_t *stats) {
    const int list = list_of_both(ctx->list_items, bh_layout<T>(ctx->list_items, t->nqb, n, stats != nullptr).tot);
    const BhLayout L = bh_layout<T>(list, t->nqb, n, stats != nullptr);
    HTS_OKR(ensure(ctx->part, 2 * L.tot));
    char *base = (char *)ctx->part.p;
    const Walks<T> w = walks_at<T>(base, L, list, t->nqb, fattr, stats ? stats + 2 * kBhStats : nullptr);
    const Walks<T> e = walks_at<T>(base + L.tot, L, list, t->nqb, fattr_euclid, stats);
    HTS_OKR(tree_euclid<T>(ctx, st, t, theta, EuclidExtras<T>{Y, pts, w.ls.count, e.ls.count}));
    if (stats)
        launch_walks<T, kBoth, true>(ctx, st, t, n, w, e, pts, rp, col, val, ex, nullptr, lambda, grad, z_dev);
    else
        launch_walks<T, kBoth, false>(ctx, st, t, n, w, e, pts, rp, col, val, ex, nullptr, lambda, grad, z_dev);
    HTS_HIP(hipGetLastError());
    return HTS_OK;
}

#define HTS_INST(T)                                                                                       \
    template hts_status launch_bh_repulsion<T>(hts_ctx, hipStream_t, hts_tree, int64_t, BhPrep<T>,        \
                                               PointRec<T> *, const int64_t *, const int32_t *,           \
                                               const T *, T *, double, const double *, T *, double *,     \
                                               uint64_t *);                                               \
    template hts_status launch_bh_hsne<T>(hts_ctx, hipStream_t, hts_tree, int64_t, const T *, double,     \
                                          PointRec<T> *, const int64_t *, const int32_t *, const T *,     \
                                          T *, T *, double, double, T *, double *, uint64_t *);
HTS_INST(float)
HTS_INST(double)

}  // namespace hts
