// Triangle and k-clique counting/listing on the degree-ordered DAG.
//
// Every k-clique {x_0 < x_1 < ... < x_{k-1}} (in degree order) is found
// exactly once, from x_0, as a path of the DAG: C_1 = N+(x_0), and
// C_{i+1} = C_i ∩ N+(x_i) are the candidates for x_{i+1} (Appendix B.2
// orientation; Appendix B.4 clique pruning; Section 5 local graph).
// Vertices with fewer than k-1 out-neighbours are skipped (degree
// filtering, Section 4.3).
//
// Kernels:
//   k_tc_arcs, k_tc_seg  triangles.  Every arc u -> v belongs to its end of
//                   larger out-degree, x (the root on a tie), and counts the
//                   entries of the other end's out-list that lie in N+(x):
//                   sum over arcs of min(d+(u), d+(v)) tests instead of
//                   sum of d+(v) (RMAT-20: 2.2e9 instead of 5.0e9).  Arcs
//                   between short lists are merged, a lane per arc; for the
//                   other roots x N+(x) sits in LDS as a hash table and x's
//                   neighbours' lists run past it.  Optionally adds 1 to the
//                   triangle count of each of the triangle's three arcs.
//   k_clique_wave   k = 4..9, roots with out-degree <= 64: one wave builds
//                   the local graph on N+(u) as 64-bit adjacency rows in LDS
//                   and counts cliques with AND + popcount.
//   (local_graph.hip) k = 4..9, roots with out-degree 65..1024: workgroup
//                   local graphs in LDS.
//   k_clique_generic  any k in [3, 9] when an out-degree exceeds 1024, and
//                   listing: one wave per root, depth-first with candidate
//                   sets in a per-wave global scratch, wave-cooperative
//                   intersections.
#include "gpm_internal.h"

#include <algorithm>
#include <climits>
#include <cstdlib>

namespace gpm {

gpm_status lg_workspace_bytes(const gpm_graph *g, int32_t k, uint64_t *bytes);
gpm_status lg_cliques(const gpm_graph *g, int32_t k, const int32_t *list_m, const int32_t *cnt_m,
                      const int32_t *list_b, const int32_t *cnt_b, const int64_t *rowoff_b,
                      void *ws, uint64_t ws_bytes, unsigned long long *res,
                      unsigned long long *res3, unsigned long long *res4, const RowEmitter *em,
                      hipStream_t st);

namespace {

constexpr int kBlock = 256;
constexpr int kWPB = kBlock / kWave;   // waves per block

__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// First index i in [0, n) with a[i] >= x (n if none).
__device__ __forceinline__ int lower_bound_i32(const int32_t *a, int n, int32_t x) {
    int lo = 0, hi = n;
    while (lo < hi) {
        int mid = (lo + hi) >> 1;
        if (a[mid] < x) lo = mid + 1; else hi = mid;
    }
    return lo;
}

__device__ __forceinline__ int64_t last_le_i64(const int64_t *a, int64_t n, int64_t x) {
    int64_t lo = 0, hi = n;
    while (hi - lo > 1) {
        int64_t mid = (lo + hi) >> 1;
        if (a[mid] <= x) lo = mid; else hi = mid;
    }
    return lo;
}

// ------------------------------------------------------------ task build --

// Classes of roots by out-degree.
enum RootClass : int { RC_NONE = 0, RC_SMALL = 1, RC_MID = 2, RC_BIG = 3, RC_HUB = 4 };

constexpr int kRootsPer = 4;                      // roots per thread
constexpr int kRootsBlock = kBlock * kRootsPer;   // roots per workgroup

// Block-wide exclusive scan of one 64-bit value per thread (kBlock threads);
// returns the block's total in `total`.  Two barriers.
__device__ __forceinline__ uint64_t block_excl64(uint64_t x, uint64_t *s_sum, uint64_t &total) {
    const int lane = lane_id(), wid = threadIdx.x / kWave;
    const uint64_t inc = wave_incl_scan(x);
    __syncthreads();
    if (lane == 63) s_sum[wid] = inc;
    __syncthreads();
    uint64_t before = inc - x;
    total = 0;
#pragma unroll
    for (int q = 0; q < kWPB; q++) {
        before += q < wid ? s_sum[q] : 0;
        total += s_sum[q];
    }
    return before;
}

// The lists of the roots of every class, in blocks of ascending ids (the
// order of the blocks is that of their arrival): one pass and one atomic per
// workgroup and class, where a flag, scan and compaction per class took ten
// launches a class.
struct RootLists {
    int32_t *list[4];              // small, mid, big, hub
    int32_t *count;                // their lengths (zero on entry)
    int64_t *rowoff;               // big: first word of the root's stored rows (may be null)
    unsigned long long *words;     // big: row words handed out (zero on entry)
    int64_t *hpre;                 // hub: out-arcs of the hubs before this one
    unsigned long long *hub;       // hub: count << 32 | out-arcs (zero on entry)
};

// Words of a stored local graph: d rows of ceil(d / 64), then d vertex ids.
__device__ __forceinline__ int32_t row_words(int32_t d) {
    return d * ((d + 63) >> 6) + (d + 1) / 2;
}

__global__ void __launch_bounds__(kBlock) k_clique_roots(const int32_t *__restrict__ dag_off,
                                                         int32_t n, int32_t min_out,
                                                         int32_t small_max, int32_t mid_max,
                                                         int32_t big_max, RootLists L) {
    __shared__ uint64_t s_sum[kWPB];
    __shared__ uint64_t s_base[6];   // list bases, row words, hub arcs
    for (int64_t r0 = (int64_t)blockIdx.x * kRootsBlock; r0 < n;
         r0 += (int64_t)gridDim.x * kRootsBlock) {
        const int64_t r = r0 + (int64_t)threadIdx.x * kRootsPer;
        int32_t d[kRootsPer], c[kRootsPer];
        uint64_t num = 0, words = 0, arcs = 0;   // num: 16 bits per class
        int32_t at = r < n ? dag_off[r] : 0;
#pragma unroll
        for (int q = 0; q < kRootsPer; q++) {
            const int32_t next = r + q < n ? dag_off[r + q + 1] : at;
            d[q] = next - at;
            at = next;
            c[q] = d[q] < min_out || d[q] == 0 ? RC_NONE
                   : d[q] > big_max ? RC_HUB
                   : d[q] > mid_max ? RC_BIG : (d[q] > small_max ? RC_MID : RC_SMALL);
            if (c[q] != RC_NONE) num += 1ull << (16 * (c[q] - 1));
            if (c[q] == RC_BIG) words += (uint64_t)row_words(d[q]);
            if (c[q] == RC_HUB) arcs += (uint64_t)d[q];
        }
        uint64_t total, wtotal = 0, htotal = 0, wbefore = 0, hbefore = 0;
        const uint64_t before = block_excl64(num, s_sum, total);
        if (total >> 32) {   // big roots or hubs in this block
            wbefore = block_excl64(words, s_sum, wtotal);
            hbefore = block_excl64(arcs, s_sum, htotal);
        }
        if (threadIdx.x < 3) {
            const int32_t t = (int32_t)((total >> (16 * threadIdx.x)) & 0xffffu);
            s_base[threadIdx.x] = t ? (uint64_t)atomicAdd(&L.count[threadIdx.x], t) : 0;
        } else if (threadIdx.x == 3) {
            // a hub's place and its first arc come from one counter, so that
            // the arcs ascend along the list
            const uint64_t t = total >> 48;
            const unsigned long long h =
                t ? atomicAdd(L.hub, (unsigned long long)(t << 32 | htotal)) : 0;
            s_base[3] = h >> 32;
            s_base[5] = h & 0xffffffffull;
        } else if (threadIdx.x == 4) {
            s_base[4] = wtotal && L.words ? atomicAdd(L.words, (unsigned long long)wtotal) : 0;
        }
        __syncthreads();
        uint64_t pos = before;
#pragma unroll
        for (int q = 0; q < kRootsPer; q++) {
            if (c[q] == RC_NONE) continue;
            const int k = c[q] - 1;
            const uint64_t p = s_base[k] + ((pos >> (16 * k)) & 0xffffu);
            L.list[k][p] = (int32_t)(r + q);
            if (c[q] == RC_BIG && L.rowoff) {
                L.rowoff[p] = (int64_t)(s_base[4] + wbefore);
                wbefore += (uint64_t)row_words(d[q]);
            }
            if (c[q] == RC_HUB) {
                L.hpre[p] = (int64_t)(s_base[5] + hbefore);
                hbefore += (uint64_t)d[q];
            }
            pos += 1ull << (16 * k);
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------- triangles ---

// What the triangle kernels do with each triangle (u, v, w), u -> v -> w, u -> w.
enum TcMode : int {
    TC_COUNT = 0,   // count only
    TC_ARCS = 1,    // also +1 on the triangle count of each of its three arcs
    TC_LIST = 2,    // list: emit (u, v, w)
};

// Arcs whose ends both have at most this out-degree are merged by
// k_tc_arcs; roots above it are staged by k_tc_seg, up to kTcMaxD in LDS.
constexpr int32_t kTcArcMax = 32, kTcMaxD = 1024;
constexpr int kTcUnit = 16;   // list entries a 16-lane group tests at once

struct Tau {
    int64_t t[3];   // gpm_graph::tc_tau
};

// Neighbours per task of a staged root of out-degree d: about eight times
// tau / d, since a segment is at most d long, most are shorter, and fewer
// than half of the neighbours have one.
__host__ __device__ inline int32_t tc_task_nbrs(int32_t d, const Tau &tau) {
    const int64_t t = tau.t[d <= 64 ? 0 : (d <= 256 ? 1 : 2)];
    const int64_t k = 8 * t / d / kBlock * kBlock;
    return (int32_t)(k < kBlock ? kBlock : (k > (1 << 20) ? (1 << 20) : k));
}

// A run of tc_task_nbrs neighbours of the staged root x, from the c0-th.
struct TcTask {
    int32_t x, c0;
};

// The tasks of every root of out-degree above kTcArcMax; those of roots
// above kTcMaxD go to `hub`.  num[0], num[1]: their numbers (zero on entry).
__global__ void __launch_bounds__(kBlock) k_tc_tasks(const int32_t *__restrict__ off,
                                                     const int32_t *__restrict__ dag_off,
                                                     int32_t n, Tau tau, TcTask *tasks,
                                                     TcTask *hub, uint32_t *num) {
    __shared__ uint64_t s_sum[kWPB];
    __shared__ uint32_t s_base[2];
    for (int64_t r0 = (int64_t)blockIdx.x * kRootsBlock; r0 < n;
         r0 += (int64_t)gridDim.x * kRootsBlock) {
        const int64_t r = r0 + (int64_t)threadIdx.x * kRootsPer;
        int32_t d[kRootsPer], nt[kRootsPer];
        uint64_t mine = 0;   // tasks, hub tasks << 32
        int32_t at = r < n ? dag_off[r] : 0;
#pragma unroll
        for (int q = 0; q < kRootsPer; q++) {
            const int32_t next = r + q < n ? dag_off[r + q + 1] : at;
            d[q] = next - at;
            at = next;
            nt[q] = 0;
            if (d[q] > kTcArcMax) {
                const int32_t nb = tc_task_nbrs(d[q], tau);
                nt[q] = (off[r + q + 1] - off[r + q] + nb - 1) / nb;
                mine += (uint64_t)nt[q] << (d[q] > kTcMaxD ? 32 : 0);
            }
        }
        uint64_t total;
        uint64_t before = block_excl64(mine, s_sum, total);
        if (threadIdx.x < 2) {
            const uint32_t t = (uint32_t)(total >> (32 * threadIdx.x));
            s_base[threadIdx.x] = t ? atomicAdd(&num[threadIdx.x], t) : 0;
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kRootsPer; q++) {
            if (nt[q] == 0) continue;
            const bool h = d[q] > kTcMaxD;
            const int32_t nb = tc_task_nbrs(d[q], tau);
            TcTask *o = h ? hub + s_base[1] + (uint32_t)(before >> 32)
                          : tasks + s_base[0] + (uint32_t)before;
            for (int32_t i = 0; i < nt[q]; i++) o[i] = {(int32_t)(r + q), i * nb};
            before += (uint64_t)nt[q] << (h ? 32 : 0);
        }
        __syncthreads();
    }
}

// Adds the block's per-wave counts (one per wave, in lane 0) to *result.
template <int NW>
__device__ __forceinline__ void block_add(uint64_t acc, unsigned long long *result) {
    __shared__ unsigned long long s_acc[NW];
    if (lane_id() == 0) s_acc[threadIdx.x / kWave] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long t = 0;
        for (int q = 0; q < NW; q++) t += s_acc[q];
        if (t) atomicAdd(result, t);
    }
}

struct __attribute__((aligned(4))) Int4u {
    int32_t x, y, z, w;
};

// Arcs between short lists, a lane per arc u -> v: the two out-lists
// (d+(u), d+(v) <= kTcArcMax) are merged four entries against four, the
// block with the smaller last entry making way.  Loads of four entries may
// run past a list's end (and past the last list into the arc sources that
// follow it in the graph's storage); what lies there is masked.  Bound by
// the gathers of v's offsets and list, one line each per arc.
//   Per arc (TC_ARCS): a triangle adds to u's arcs, which are the wave's own and
// up to 31 on either side, in LDS, and to v's, of which a lane keeps a mask.
// Where lanes have few hits each adds its own (one line a hit); else half a
// wave adds one lane's, neighbours in one line.  With an atomic per hit on
// either side 5.7e7 triangles of 300,000 vertices joined to the 20 next took
// 3.86 ms, most of it lanes of one row waiting for each other; now 0.40.
constexpr uint32_t kTcOwnHits = 3;
template <int MODE>
__global__ void __launch_bounds__(kBlock) k_tc_arcs(const int32_t *__restrict__ dag_off,
                                                    const int32_t *__restrict__ dag_adj,
                                                    const int32_t *__restrict__ dag_src,
                                                    int64_t m, unsigned long long *result,
                                                    uint32_t *te, RowEmitter em) {
    constexpr int kU = MODE == TC_ARCS ? kWave + 2 * kTcArcMax : 1;
    __shared__ uint32_t s_u[kWPB][kU];   // triangles per arc base - kTcArcMax + i
    uint32_t acc = 0;   // below 2^32: at most kTcArcMax per arc, m < 2^30 over the grid
    uint64_t total = 0;
    const int lane = lane_id(), wib = threadIdx.x / kWave;
    if (MODE == TC_ARCS) {
        for (int i = lane; i < kU; i += kWave) s_u[wib][i] = 0;
        wave_sync();
    }
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    for (int64_t base = (int64_t)blockIdx.x * kBlock + wib * kWave; base < m; base += stride) {
        const int64_t e0 = base + lane;
        int32_t u = 0, v = 0, a = 0, az = 0, b = 0, bz = 0;
        if (e0 < m) {
            u = dag_src[e0];
            a = dag_off[u];
            az = dag_off[u + 1];
            if (az - a <= kTcArcMax && az - a >= 2) {
                v = dag_adj[e0];
                b = dag_off[v];
                bz = dag_off[v + 1];
                if (bz - b > kTcArcMax) bz = b;
            }
        }
        uint32_t mine = 0, found = 0;   // found: the hits' positions, in u's list (TC_LIST) or
        const int32_t a0 = a, b0 = b;   // in v's (TC_ARCS)
        auto load = [&](int32_t at, int32_t end, int32_t pad) {
            Int4u x = *reinterpret_cast<const Int4u *>(dag_adj + at);
            x.y = at + 1 < end ? x.y : pad;
            x.z = at + 2 < end ? x.z : pad;
            x.w = at + 3 < end ? x.w : pad;
            return x;
        };
        Int4u A{}, B{};
        if (b < bz) {
            A = load(a, az, -1);
            B = load(b, bz, -2);
        }
        while (a < az && b < bz) {
            const int32_t x[4] = {A.x, A.y, A.z, A.w}, y[4] = {B.x, B.y, B.z, B.w};
#pragma unroll
            for (int i = 0; i < 4; i++) {
                const bool hit = x[i] == y[0] || x[i] == y[1] || x[i] == y[2] || x[i] == y[3];
                mine += hit ? 1u : 0u;
                if (MODE == TC_ARCS && hit) {
                    const int j = x[i] == y[0] ? 0 : (x[i] == y[1] ? 1 : (x[i] == y[2] ? 2 : 3));
                    atomicAdd(&s_u[wib][a + i - (int32_t)(base - kTcArcMax)], 1u);
                    found |= 1u << (b - b0 + j);
                }
                if (MODE == TC_LIST && hit) found |= 1u << (a - a0 + i);
            }
            const int32_t la = a + 4 < az ? A.w : INT_MAX, lb = b + 4 < bz ? B.w : INT_MAX;
            if (la <= lb) {
                a += 4;
                if (a < az) A = load(a, az, -1);
            }
            if (lb <= la) {
                b += 4;
                if (b < bz) B = load(b, bz, -2);
            }
        }
        if constexpr (MODE == TC_ARCS) {
            uint64_t some = __ballot(mine != 0);
            if (some) {
                wave_sync();
                const int side = lane < kTcArcMax ? lane : lane + kWave;   // the arcs around
                const uint32_t own = s_u[wib][lane + kTcArcMax] + mine, around = s_u[wib][side];
                if (own) atomicAdd(&te[e0], own);
                if (around) atomicAdd(&te[base - kTcArcMax + side], around);
                s_u[wib][lane + kTcArcMax] = 0;
                s_u[wib][side] = 0;
                wave_sync();
                if (!__any(mine > kTcOwnHits)) {
                    for (; found; found &= found - 1u) atomicAdd(&te[b0 + __builtin_ctz(found)], 1u);
                } else {
                    while (some) {
                        const int l0 = __builtin_ctzll(some);
                        some &= some - 1ull;
                        const int l1 = some ? __builtin_ctzll(some) : l0;
                        const int from = lane < 32 ? l0 : l1;
                        const int32_t vb = __shfl(b0, from, 64);
                        uint32_t hits = __shfl(found, from, 64);
                        if (lane >= 32 && !some) hits = 0;
                        some &= some - 1ull;
                        if ((hits >> (lane & 31)) & 1u) atomicAdd(&te[vb + (lane & 31)], 1u);
                    }
                }
            }
        }
        // (emitted after the merge, every lane's next one together: an emission
        // takes as long for one lane as for 64, and at each of the merge's
        // steps it was one for few.  1,000,000 vertices of 8 neighbours among
        // 100: 8.8 ms, now 1.4)
        if (MODE == TC_LIST)
            for (; found; found &= found - 1u) {
                const int32_t tri[3] = {u, v, dag_adj[a0 + __builtin_ctz(found)]};
                emit_vertices<3>(em, tri);
            }
        acc += mine;
    }
    total = wave_sum((uint64_t)acc);
    if (MODE == TC_LIST) {
        row_emitter_flush(em, result);
        return;
    }
    block_add<kWPB>(total, result);
}

// The line between the two: a merge costs a lane up to 16 dependent steps at
// 32 entries a side, and a staged root its table; uniform graphs fall below
// it whole (3,000,001 vertices, 24M edges: 1.1 ms against 2.8 ms for a wave
// per root), and on RMAT-20 99% of the tests lie above it.

// Staged roots.  A workgroup takes a task (x, a run of x's neighbours),
// holds N+(x) in LDS as a hash table (4 to 16 slots per entry, at most 4096)
// and takes 256 neighbours y at a time: y has a segment when the arc between
// x and y is x's (d+(y) < d+(x), or equal and x -> y), namely N+(y), cut
// into units of 16 entries.  A wave looks up the segments of 64 units at
// once, one per lane, and then tests 4 units per step and tile, a 16-lane
// group each: two lane exchanges tell a group its unit, so short and long
// segments cost the same bookkeeping.  With HUB, N+(x) is too long for LDS
// and each entry is searched in it.
//   TC_ARCS: the arc from x to the closing vertex is counted in LDS by its
// position in N+(x), the arc between x and y per segment (found in the table
// when y is an out-neighbour, else by a search for x in N+(y)), both flushed
// after use; the arc from y takes a global atomic.
// RMAT-20: 2.4 ms for 2.2e9 tests (6.1 ms with every arc u -> v at u: 5.0e9).
template <int MODE, bool HUB>
__global__ void __launch_bounds__(kBlock, MODE == TC_COUNT ? 8 : 4)
    k_tc_seg(const int32_t *__restrict__ off, const int32_t *__restrict__ adj,
             const int32_t *__restrict__ okey, const int32_t *__restrict__ dag_off,
             const int32_t *__restrict__ dag_adj, const TcTask *__restrict__ tasks,
             const uint32_t *__restrict__ ntasks_p, Tau tau,
             unsigned long long *cursor, unsigned long long *result, uint32_t *te, RowEmitter em) {
    constexpr int TU = 4;                        // tiles in flight
    constexpr int H = HUB ? 4 : 4096;
    constexpr bool ARCS = MODE == TC_ARCS, VALS = ARCS && !HUB;
    __shared__ __align__(16) int32_t keys[H];
    __shared__ int16_t vals[VALS ? H : 1];
    __shared__ uint32_t cnt[VALS ? kTcMaxD : 1];
    __shared__ int32_t pre[kBlock], sbeg[kBlock], slen[kBlock];
    __shared__ uint32_t scnt[ARCS ? kBlock : 1];
    __shared__ int32_t sy[MODE == TC_LIST ? kBlock : 1];   // y, or ~y for y -> x
    __shared__ int32_t s_sum[kWPB];
    __shared__ int32_t s_task;
    const int tid = threadIdx.x, lane = lane_id();
    const int wid = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int grp = lane / kTcUnit, gl = lane % kTcUnit;
    TaskQueue queue(cursor, *ntasks_p, blockIdx.x, gridDim.x);
    uint64_t acc = 0;   // wave-uniform
    if (VALS)
        for (int i = tid; i < kTcMaxD; i += kBlock) cnt[i] = 0;
    for (;;) {
        if (wid == 0) {
            const int32_t got = (int32_t)queue.next();
            if (lane == 0) s_task = got;
        }
        __syncthreads();
        const int32_t t = s_task;
        if (t < 0) break;
        const int32_t x = tasks[t].x, c0 = tasks[t].c0;
        const int32_t s = dag_off[x], d = dag_off[x + 1] - s;
        const int32_t r0 = off[x], cz = min(off[x + 1] - r0, c0 + tc_task_nbrs(d, tau));
        const int32_t kx = okey[x];
        const int32_t hb = min(12, lds_hash_bits(d, d <= 256 ? 16 : 4));
        const uint32_t bmask = (1u << (hb - 2)) - 1u;
        const int4 *kb = reinterpret_cast<const int4 *>(keys);
        if (!HUB) {
            int4 *k4 = reinterpret_cast<int4 *>(keys);
            for (int i = tid; i < (1 << hb) / 4; i += kBlock) k4[i] = make_int4(-1, -1, -1, -1);
            __syncthreads();
            for (int32_t i = tid; i < d; i += kBlock)
                lds_hash_insert(keys, VALS ? vals : nullptr, hb, dag_adj[s + i], i);
        }
        for (int32_t b0 = c0; b0 < cz; b0 += kBlock) {
            // one neighbour per thread: its segment's units
            int32_t y = 0, ys = 0, dy = 0;
            bool in = false;   // y -> x (known where it matters)
            if (b0 + tid < cz) {
                y = adj[r0 + b0 + tid];
                ys = dag_off[y];
                dy = dag_off[y + 1] - ys;
                if (dy > d) dy = 0;
                if (dy > 0 && (dy == d || MODE == TC_LIST)) {
                    in = !rank_less(kx, x, okey[y], y);
                    if (dy == d && in) dy = 0;
                }
            }
            const int32_t nu = (dy + kTcUnit - 1) / kTcUnit;
            const int32_t inc = wave_incl_scan(nu);
            if (lane == 63) s_sum[wid] = inc;
            sbeg[tid] = ys;
            slen[tid] = dy;
            if (ARCS) scnt[tid] = 0;
            if (MODE == TC_LIST) sy[tid] = in ? ~y : y;
            __syncthreads();
            int32_t before = 0, units = 0;
#pragma unroll
            for (int q = 0; q < kWPB; q++) {
                before += q < wid ? s_sum[q] : 0;
                units += s_sum[q];
            }
            units = __builtin_amdgcn_readfirstlane(units);
            pre[tid] = before + inc - nu;
            __syncthreads();
            for (int32_t ub = wid * kWave; ub < units; ub += kBlock) {
                // this lane's unit of the wave's 64: first arc, entries and segment
                int32_t st = s, ln = 0;
                if (ub + lane < units) {
                    int32_t j = 0;   // last segment starting at or before the unit
#pragma unroll
                    for (int h = kBlock / 2; h > 0; h >>= 1)
                        if (pre[j + h] <= ub + lane) j += h;
                    const int32_t o = (ub + lane - pre[j]) * kTcUnit;
                    st = sbeg[j] + o;
                    ln = min(kTcUnit, slen[j] - o) | (j << 5);
                }
                const int32_t ntile = min(kTcUnit, (units - ub + 3) / 4);
                for (int32_t t0 = 0; t0 < ntile; t0 += TU) {
                    int32_t e[TU], w[TU], us[TU];
                    uint64_t pend[TU];
#pragma unroll
                    for (int q = 0; q < TU; q++) {
                        const int src = (t0 + q) * 4 + grp;   // below 64: TU divides 16
                        us[q] = __shfl(ln, src, 64);
                        e[q] = __shfl(st, src, 64);
                    }
#pragma unroll
                    for (int q = 0; q < TU; q++) {
                        const bool live = gl < (us[q] & 31);
                        pend[q] = __ballot(live);
                        // idle lanes load their unit's first arc
                        e[q] += live ? gl : 0;
                        w[q] = *reinterpret_cast<const int32_t *>(
                            reinterpret_cast<const char *>(dag_adj) + ((uint32_t)e[q] << 2));
                    }
                    if constexpr (MODE == TC_COUNT && !HUB) {
                        uint32_t b[TU];
#pragma unroll
                        for (int q = 0; q < TU; q++) b[q] = lds_hash_slot(w[q], hb) >> 2;
                        for (;;) {
                            int4 kv[TU];
#pragma unroll
                            for (int q = 0; q < TU; q++) kv[q] = kb[b[q]];
                            uint64_t more = 0;
#pragma unroll
                            for (int q = 0; q < TU; q++) {
                                const int4 k = kv[q];
                                const int32_t v = w[q];
                                const uint64_t hit = __ballot(k.x == v) | __ballot(k.y == v) |
                                                     __ballot(k.z == v) | __ballot(k.w == v);
                                const uint64_t empty = __ballot((k.x | k.y | k.z | k.w) < 0);
                                acc += (uint64_t)__popcll(hit & pend[q]);
                                pend[q] &= ~(hit | empty);
                                b[q] = (b[q] + 1u) & bmask;
                                more |= pend[q];
                            }
                            if (!more) break;
                        }
                    } else {
                        int32_t p[TU];   // HUB: last entry of N+(x) up to w, or the first;
                        if constexpr (HUB) {   // the tiles' searches advance together
#pragma unroll
                            for (int q = 0; q < TU; q++) p[q] = 0;
                            for (int32_t len = d; len > 1; len -= len >> 1) {
#pragma unroll
                                for (int q = 0; q < TU; q++)
                                    p[q] += dag_adj[s + p[q] + (len >> 1)] <= w[q] ? len >> 1 : 0;
                            }
                        }
#pragma unroll
                        for (int q = 0; q < TU; q++) {
                            int32_t at = -1;   // slot of w (HUB: position in N+(x))
                            if ((pend[q] >> lane) & 1ull) {
                                if constexpr (HUB) {
                                    at = dag_adj[s + p[q]] == w[q] ? p[q] : -1;
                                } else {
                                    uint32_t h = lds_hash_slot(w[q], hb);
                                    for (;;) {
                                        const int4 k = kb[h >> 2];
                                        const int c = k.x == w[q] ? 0 : k.y == w[q] ? 1
                                                      : k.z == w[q] ? 2 : k.w == w[q] ? 3 : -1;
                                        if (c >= 0) at = (int32_t)h + c;
                                        if (c >= 0 || (k.x | k.y | k.z | k.w) < 0) break;
                                        h = (h + 4) & ((1u << hb) - 1u);
                                    }
                                }
                            }
                            const uint64_t hit = __ballot(at >= 0);
                            acc += (uint64_t)__popcll(hit);
                            if (MODE == TC_COUNT || !hit) continue;
                            const int32_t seg = us[q] >> 5;
                            if (ARCS) {
                                const uint32_t g =
                                    (uint32_t)(hit >> (grp * kTcUnit)) & ((1u << kTcUnit) - 1u);
                                if (gl == 0 && g) atomicAdd(&scnt[seg], (uint32_t)__popc(g));
                                if (at >= 0) {
                                    if (HUB) atomicAdd(&te[s + at], 1u);
                                    else atomicAdd(&cnt[vals[at]], 1u);
                                    atomicAdd(&te[e[q]], 1u);
                                }
                            }
                            if (MODE == TC_LIST && at >= 0) {
                                const int32_t yy = sy[seg];
                                const int32_t tri[3] = {yy < 0 ? ~yy : x, yy < 0 ? x : yy, w[q]};
                                emit_vertices<3>(em, tri);
                            }
                        }
                    }
                }
            }
            __syncthreads();
            if (ARCS) {
                const uint32_t c = scnt[tid];
                if (c) {
                    // the arc between x and y
                    int32_t p = lower_bound_i32(dag_adj + ys, dy, x);
                    if (p < dy && dag_adj[ys + p] == x) {
                        atomicAdd(&te[ys + p], c);
                    } else {
                        p = lower_bound_i32(dag_adj + s, d, y);
                        if (VALS) atomicAdd(&cnt[p], c);
                        else atomicAdd(&te[s + p], c);
                    }
                }
            }
        }
        __syncthreads();
        if (VALS) {
            for (int32_t i = tid; i < d; i += kBlock) {
                const uint32_t c = cnt[i];
                if (c) {
                    atomicAdd(&te[s + i], c);
                    cnt[i] = 0;
                }
            }
        }
    }
    if (MODE == TC_LIST) {
        row_emitter_flush(em, result);
        return;
    }
    block_add<kWPB>(acc, result);
}

// Entries that the triangle kernels look up, the shorter out-list of each arc's
// two, by the kernel that takes the arc: units[0] k_tc_arcs, [1] k_tc_seg, [2]
// its hub form (all zero on entry).  Launched while timing is on only.
__global__ void __launch_bounds__(kBlock) k_tc_units(const int32_t *__restrict__ dag_off,
                                                     const int32_t *__restrict__ dag_adj,
                                                     const int32_t *__restrict__ dag_src,
                                                     int64_t m, unsigned long long *units) {
    uint64_t n[3] = {0, 0, 0};
    for (int64_t e = (int64_t)blockIdx.x * kBlock + threadIdx.x; e < m;
         e += (int64_t)gridDim.x * kBlock) {
        const int32_t u = dag_src[e], v = dag_adj[e];
        const int32_t du = dag_off[u + 1] - dag_off[u], dv = dag_off[v + 1] - dag_off[v];
        const int32_t most = max(du, dv), least = min(du, dv);
        if (most <= kTcArcMax) n[0] += du >= 2 ? least : 0;
        else n[most <= kTcMaxD ? 1 : 2] += least;
    }
#pragma unroll
    for (int q = 0; q < 3; q++) {
        const uint64_t t = wave_sum(n[q]);
        if (lane_id() == 0 && t) atomicAdd(&units[q], (unsigned long long)t);
    }
}

// ------------------------------------------- local-graph k-cliques ---

// Number of D-vertex cliques of the local DAG (rows: 64-bit masks, local
// graph on <= 64 vertices) whose vertices all lie in mask.
template <int D>
__device__ __forceinline__ uint64_t cliques_in64(uint64_t mask, const uint64_t *rows) {
    if constexpr (D == 1) {
        return (uint64_t)__popcll(mask);
    } else if constexpr (D == 2) {
        uint64_t c = 0, m = mask;
        while (m) {
            const int j = __builtin_ctzll(m);
            m &= m - 1;
            c += __popcll(mask & rows[j]);
        }
        return c;
    } else {
        uint64_t c = 0, m = mask;
        while (m) {
            const int j = __builtin_ctzll(m);
            m &= m - 1;
            c += cliques_in64<D - 1>(mask & rows[j], rows);
        }
        return c;
    }
}

// Emits every (K)-clique {u, v_i, ...} through local vertex i (row r): the
// (K-2)-cliques of the local DAG inside r, by nested bit loops.  v holds the
// clique's vertices chosen so far (u, v_i, ...), depth = how many.
template <int K, int DEPTH>
__device__ void list_in64(uint64_t mask, const uint64_t *rows, const int32_t *verts,
                          int32_t (&v)[K], RowEmitter &em) {
    uint64_t m = mask;
    while (m) {
        const int j = __builtin_ctzll(m);
        m &= m - 1;
        v[DEPTH] = verts[j];
        if constexpr (DEPTH + 1 == K) {
            emit_vertices<K>(em, v);
        } else {
            list_in64<K, DEPTH + 1>(mask & rows[j], rows, verts, v, em);
        }
    }
}

// K-cliques of the root through local vertex with row r: (K-2)-cliques of
// the local DAG inside r.
template <int K>
__device__ __forceinline__ uint64_t local_count64(uint64_t r, const uint64_t *rows) {
    return cliques_in64<K - 2>(r, rows);
}

// One 64-thread block (one wave) per root at a time: stages N+(u), sets the
// local rows through the pair walk and the membership hash, then counts.
template <int K, bool LIST>
__global__ void __launch_bounds__(kWave) k_clique_wave(const int32_t *__restrict__ dag_off,
                                                       const int32_t *__restrict__ dag_adj,
                                                       const int32_t *__restrict__ roots,
                                                       const int32_t *__restrict__ nroots_p,
                                                       unsigned long long *result,
                                                       unsigned long long *res3,
                                                       unsigned long long *res4, RowEmitter em) {
    __shared__ uint64_t rows[kWave];
    __shared__ __align__(16) int32_t keys[8 * kWave];
    __shared__ int16_t vals[8 * kWave];
    __shared__ int32_t pre[kWave + 1], offj[kWave];
    __shared__ int32_t verts[LIST ? kWave : 1];
    const int lane = lane_id();
    const int32_t nroots = *nroots_p;
    uint64_t acc = 0, acc3 = 0, acc4 = 0;
    for (int64_t r = blockIdx.x; r < nroots; r += gridDim.x) {
        const int32_t u = roots[r];
        const int32_t s = dag_off[u], d = dag_off[u + 1] - s;
        const int32_t hb = lds_hash_bits(d, 8);
        for (int i = lane; i < (1 << hb); i += kWave) keys[i] = -1;
        rows[lane] = 0;
        stage_root<kWave, 1>(dag_off, dag_adj, s, d, keys, vals, hb, pre, offj, nullptr, nullptr,
                             LIST ? verts : nullptr);
        walk_lookup<2>(pre, offj, dag_adj, d, 0, pre[d], keys, hb,
                [&](int32_t j, int32_t, int32_t w, int32_t slot) {
            if (slot >= 0) atomicOr((unsigned long long *)&rows[j], 1ull << vals[slot]);
        });
        __syncthreads();
        if (lane < d) {
            if constexpr (LIST) {
                int32_t v[K];
                v[0] = u;
                v[1] = verts[lane];
                list_in64<K, 2>(rows[lane], rows, verts, v, em);
            } else {
                acc += local_count64<K>(rows[lane], rows);
                if (res3) acc3 += __popcll(rows[lane]);                 // triangles at u
                if (K == 5 && res4) acc4 += local_count64<4>(rows[lane], rows);
            }
        }
        __syncthreads();
    }
    if (LIST) {
        row_emitter_flush(em, result);
        return;
    }
    acc = wave_sum(acc);
    if (lane == 0 && acc) atomicAdd(result, (unsigned long long)acc);
    if (res3) {
        acc3 = wave_sum(acc3);
        if (lane == 0 && acc3) atomicAdd(res3, (unsigned long long)acc3);
    }
    if (K == 5 && res4) {
        acc4 = wave_sum(acc4);
        if (lane == 0 && acc4) atomicAdd(res4, (unsigned long long)acc4);
    }
}

constexpr int kMidMaxD = 256;

// ------------------------------------------------- generic DFS (k <= 9) ---

constexpr int kGenMaxK = 9;

struct ListOut {
    int32_t *buf;
    uint64_t cap;
};

// Wave-cooperative |A ∩ B| or A ∩ B (ascending, into out) for ascending
// global arrays; lanes walk the shorter list and binary-search the longer.
template <bool WRITE>
__device__ int32_t wave_intersect(const int32_t *a, int32_t na, const int32_t *b, int32_t nb,
                                  int32_t *out) {
    const int lane = lane_id();
    if (na > nb) {
        const int32_t *t = a; a = b; b = t;
        int32_t tn = na; na = nb; nb = tn;
    }
    int32_t cnt = 0;
    for (int32_t i0 = 0; i0 < na; i0 += kWave) {
        const int32_t i = i0 + lane;
        bool hit = false;
        int32_t x = 0;
        if (i < na) {
            x = a[i];
            int32_t p = lower_bound_i32(b, nb, x);
            hit = p < nb && b[p] == x;
        }
        const uint64_t mask = __ballot(hit);
        if (WRITE && hit) out[cnt + lanes_below(mask)] = x;
        cnt += __popcll(mask);
    }
    return cnt;
}

__device__ __forceinline__ void sort_small(uint64_t *k, int len) {
    for (int i = 1; i < len; i++) {
        uint64_t x = k[i];
        int j = i - 1;
        while (j >= 0 && k[j] > x) { k[j + 1] = k[j]; j--; }
        k[j + 1] = x;
    }
}

template <bool LIST>
__global__ void __launch_bounds__(kBlock) k_clique_generic(const int32_t *__restrict__ dag_off,
                                                           const int32_t *__restrict__ dag_adj,
                                                           int32_t n, int32_t k, int32_t maxout,
                                                           int32_t *scratch,
                                                           unsigned long long *result,
                                                           ListOut lo) {
    const int lane = lane_id();
    const int64_t wave_gid = (int64_t)blockIdx.x * kWPB + threadIdx.x / kWave;
    const int64_t nwaves = (int64_t)gridDim.x * kWPB;
    int32_t *mine = scratch + wave_gid * (int64_t)(kGenMaxK - 2) * maxout;
    uint64_t acc = 0, hsum = 0;
    const int last = k - 2;   // level whose intersection is counted/listed
    for (int64_t ur = wave_gid; ur < n; ur += nwaves) {
        const int32_t u = (int32_t)ur;
        const int32_t s = dag_off[u], d = dag_off[u + 1] - s;
        if (d < k - 1) continue;
        const int32_t *cand[kGenMaxK];
        int32_t csz[kGenMaxK], it[kGenMaxK], pv[kGenMaxK];
        cand[1] = dag_adj + s;
        csz[1] = d;
        it[1] = 0;
        pv[0] = u;
        int l = 1;
        while (l >= 1) {
            if (it[l] >= csz[l]) {
                l--;
                if (l >= 1) it[l]++;
                continue;
            }
            const int32_t v = cand[l][it[l]];
            pv[l] = v;
            const int32_t vs = dag_off[v], vd = dag_off[v + 1] - vs;
            if (l == last) {
                if (!LIST) {
                    const int32_t c = wave_intersect<false>(cand[l], csz[l], dag_adj + vs, vd, nullptr);
                    if (lane == 0) acc += (uint64_t)c;   // c is wave-uniform
                } else {
                    // enumerate C_l ∩ N+(v): each element closes a k-clique
                    const int32_t *a = cand[l], *b = dag_adj + vs;
                    int32_t na = csz[l], nb = vd;
                    for (int32_t i0 = 0; i0 < na; i0 += kWave) {
                        const int32_t i = i0 + lane;
                        bool hit = false;
                        int32_t x = 0;
                        if (i < na) {
                            x = a[i];
                            int32_t p = lower_bound_i32(b, nb, x);
                            hit = p < nb && b[p] == x;
                        }
                        const uint64_t mask = __ballot(hit);
                        if (!mask) continue;
                        unsigned long long basei = 0;
                        if (lane == 0) basei = atomicAdd(&result[0], (unsigned long long)__popcll(mask));
                        basei = __shfl(basei, 0, 64);
                        if (hit) {
                            uint64_t key[kGenMaxK];
                            for (int t = 0; t <= last; t++) key[t] = (uint64_t)(uint32_t)pv[t];
                            key[last + 1] = (uint64_t)(uint32_t)x;
                            const uint64_t slot = basei + lanes_below(mask);
                            if (slot < lo.cap) {
                                int32_t *o = lo.buf + slot * (uint64_t)k;
                                for (int t = 0; t <= last; t++) o[t] = pv[t];
                                o[last + 1] = x;
                            }
                            sort_small(key, k);
                            uint64_t h = (uint64_t)k;
                            for (int t = 0; t < k; t++) h = fmix64((h ^ key[t]) + 0x9E3779B97F4A7C15ull);
                            hsum += h;
                        }
                    }
                }
                it[l]++;
            } else {
                int32_t *out = mine + (int64_t)(l - 1) * maxout;
                const int32_t c = wave_intersect<true>(cand[l], csz[l], dag_adj + vs, vd, out);
                wave_sync();
                if (c >= k - 1 - l) {
                    l++;
                    cand[l] = out;
                    csz[l] = c;
                    it[l] = 0;
                } else {
                    it[l]++;
                }
            }
        }
    }
    if (!LIST) {
        acc = wave_sum(acc);
        if (lane == 0 && acc) atomicAdd(&result[0], (unsigned long long)acc);
    } else {
        hsum = wave_sum(hsum);
        if (lane == 0) atomicAdd(&result[2], (unsigned long long)hsum);
    }
}

// written = min(slots handed out, cap)
__global__ void k_finish_rows(unsigned long long *result, const unsigned long long *slot_ctr,
                              uint64_t cap) {
    if (threadIdx.x == 0 && blockIdx.x == 0) result[1] = *slot_ctr < cap ? *slot_ctr : cap;
}

__global__ void k_finish_listing(unsigned long long *result, uint64_t cap) {
    if (threadIdx.x == 0 && blockIdx.x == 0) result[1] = result[0] < cap ? result[0] : cap;
}

// ----------------------------------------------- hub roots (d+ > 1024) ---
//
// Roots whose out-degree exceeds the largest class (their N+(u) does not fit
// the LDS staging of the triangle and local-graph kernels) are split at edge
// granularity (Section 4.1's task model): every arc u -> v of such a root is
// a task of its own, taken by one wave from a flattened index space over the
// hub roots' arcs.  The wave intersects N+(u) and N+(v) (lanes walk the
// shorter list and binary-search the longer) into its scratch and searches
// depth first below the result as k_clique_generic does.

enum HubMode : int {
    HUB_COUNT = 0,   // count K-cliques (and triangles / 4-cliques into res3 / res4)
    HUB_LIST = 1,    // list K-cliques through the row emitter
};

template <int K, int MODE>
__global__ void __launch_bounds__(kBlock) k_clique_hub(const int32_t *__restrict__ dag_off,
                                                       const int32_t *__restrict__ dag_adj,
                                                       const int32_t *__restrict__ hubs,
                                                       const int64_t *__restrict__ hpre,
                                                       const unsigned long long *hub_p,
                                                       int32_t maxout, int32_t *scratch,
                                                       unsigned long long *res,
                                                       unsigned long long *res3,
                                                       unsigned long long *res4,
                                                       RowEmitter em) {
    static_assert(K >= 4 && K <= kGenMaxK, "clique size");
    const int lane = lane_id();
    const int64_t wave_gid = (int64_t)blockIdx.x * kWPB + threadIdx.x / kWave;
    const int64_t nwaves = (int64_t)gridDim.x * kWPB;
    int32_t *mine = scratch + wave_gid * (int64_t)(kGenMaxK - 2) * maxout;
    const int32_t nh = (int32_t)(*hub_p >> 32);
    const int64_t total = (int64_t)(*hub_p & 0xffffffffull);
    // fused counts need every 4-clique below an arc, so only K's own
    // pruning applies when no 4-cliques are asked for
    const int32_t need2 = (res4 && K > 4) ? 2 : K - 2;
    uint64_t acc = 0, acc3 = 0, acc4 = 0;
    for (int64_t t = wave_gid; t < total; t += nwaves) {
        const int32_t r = (int32_t)last_le_i64(hpre, nh, t);
        const int32_t u = hubs[r];
        const int32_t s = dag_off[u], d = dag_off[u + 1] - s;
        const int32_t e = s + (int32_t)(t - hpre[r]);
        const int32_t v = dag_adj[e];
        const int32_t vs = dag_off[v], vd = dag_off[v + 1] - vs;
        // level 1: C = N+(u) ∩ N+(v), the triangles on the arc
        const int32_t c2 = wave_intersect<true>(dag_adj + s, d, dag_adj + vs, vd, mine);
        wave_sync();
        if (res3 && lane == 0) acc3 += (uint64_t)c2;
        if (c2 < need2) continue;
        const int32_t *cand[kGenMaxK];
        int32_t csz[kGenMaxK], it[kGenMaxK], pv[kGenMaxK];
        pv[0] = u;
        pv[1] = v;
        cand[2] = mine;
        csz[2] = c2;
        it[2] = 0;
        constexpr int last = K - 2;   // level whose intersection is counted or listed
        int l = 2;
        while (l >= 2) {
            if (it[l] >= csz[l]) {
                l--;
                if (l >= 2) it[l]++;
                continue;
            }
            const int32_t w = cand[l][it[l]];
            pv[l] = w;
            const int32_t ws = dag_off[w], wd = dag_off[w + 1] - ws;
            if (l == last) {
                if constexpr (MODE == HUB_COUNT) {
                    const int32_t c = wave_intersect<false>(cand[l], csz[l], dag_adj + ws,
                                                            wd, nullptr);
                    if (lane == 0) acc += (uint64_t)c;
                } else {
                    const int32_t *a = cand[l], *b = dag_adj + ws;
                    const int32_t na = csz[l], nb = wd;
                    for (int32_t i0 = 0; i0 < na; i0 += kWave) {
                        const int32_t i = i0 + lane;
                        if (i < na) {
                            const int32_t x = a[i];
                            const int32_t p = lower_bound_i32(b, nb, x);
                            if (p < nb && b[p] == x) {
                                int32_t q[K];
#pragma unroll
                                for (int z = 0; z < K - 1; z++) q[z] = pv[z];
                                q[K - 1] = x;
                                emit_vertices<K>(em, q);
                            }
                        }
                    }
                }
                it[l]++;
            } else {
                int32_t *out = mine + (int64_t)(l - 1) * maxout;
                const int32_t c = wave_intersect<true>(cand[l], csz[l], dag_adj + ws, wd,
                                                       out);
                wave_sync();
                if (res4 && l == 2 && lane == 0) acc4 += (uint64_t)c;
                if (c >= K - 1 - l) {
                    l++;
                    cand[l] = out;
                    csz[l] = c;
                    it[l] = 0;
                } else {
                    it[l]++;
                }
            }
        }
    }
    if constexpr (MODE == HUB_LIST) {
        row_emitter_flush(em, res);
        return;
    }
    acc = wave_sum(acc);
    if (lane == 0 && acc) atomicAdd(res, (unsigned long long)acc);
    if (res3) {
        acc3 = wave_sum(acc3);
        if (lane == 0 && acc3) atomicAdd(res3, (unsigned long long)acc3);
    }
    if (res4) {
        acc4 = wave_sum(acc4);
        if (lane == 0 && acc4) atomicAdd(res4, (unsigned long long)acc4);
    }
}

// ------------------------------------------------------------ host side --

constexpr uint64_t kCtlCur = 32, kCtlWords = kCtlCur + 2 * kCursorWords;

struct CliqueWs {
    unsigned long long *ctr;      // [8]: [0] listing slots, [1] row words, [2] hubs, [3..5]
                                  // triangles' work units, [6..7] unused
    uint32_t *ctl;                // [2..3] triangle tasks, [4..7] class counts, from
                                  // kCtlCur two sets of cursors (triangles)
    int32_t *list_s, *list_m, *list_b, *list_h;
    int64_t *rowoff_b, *hpre;
    TcTask *tasks, *hub_tasks;
    void *lg;                     // local-graph workspace (k >= 4)
    uint64_t lg_bytes;
    int32_t *gen_scratch;
    int gen_waves;
    uint64_t bytes;
};

Tau tau_of(const gpm_graph *g) { return Tau{{g->tc_tau[0], g->tc_tau[1], g->tc_tau[2]}}; }

// Tasks of the staged triangle roots at most: one per root of out-degree
// above kTcArcMax and one per full run of neighbours, runs being shortest at
// the top of a class of tc_tau.
uint64_t tc_task_bound(const gpm_graph *g) {
    const Tau tau = tau_of(g);
    int32_t nb = INT_MAX;
    for (int32_t top : {64, 256, INT_MAX})
        nb = std::min(nb, tc_task_nbrs(std::max(1, std::min(top, g->max_out_degree)), tau));
    const uint64_t roots = (uint64_t)std::min<int64_t>(g->n, g->m / (kTcArcMax + 1));
    return roots + 2 * (uint64_t)g->m / (uint64_t)nb + 1;
}

// The generic DFS (a wave per root) serves listings of k >= 6; every other
// count and listing runs on the triangle and local-graph kernels, with roots
// of out-degree above 1024 split per arc (k_clique_hub).  GPM_LG=0 in the
// environment sends every root of k >= 4 to the per-arc depth-first search
// instead: the search without local graphs, equally load-balanced, for
// comparison.
bool lg_disabled(int32_t k) {
    const char *env = getenv("GPM_LG");
    return k >= 4 && env && env[0] == '0';
}

bool uses_generic(const gpm_graph *g, int32_t k, bool list) {
    (void)g;
    return list && k > 5;
}

// Roots above the largest class go to k_clique_hub (k >= 4).
bool has_hubs(const gpm_graph *g) { return g->max_out_degree > kTcMaxD; }

bool uses_hub_kernel(const gpm_graph *g, int32_t k) { return has_hubs(g) || lg_disabled(k); }

CliqueWs clique_layout(const gpm_graph *g, int32_t k, bool list, void *base) {
    CliqueWs W{};
    Carve c(base, ~0ull);
    const uint64_t n1 = (uint64_t)g->n + 1;
    W.ctr = c.take<unsigned long long>(8);
    W.ctl = c.take<uint32_t>(kCtlWords);
    const bool generic = uses_generic(g, k, list);
    if (!generic && k == 3) {
        if (g->max_out_degree > kTcArcMax) W.tasks = c.take<TcTask>(tc_task_bound(g));
        if (has_hubs(g)) W.hub_tasks = c.take<TcTask>(tc_task_bound(g));
    }
    if (!generic && k >= 4) {
        W.list_s = c.take<int32_t>(n1);
        W.list_m = c.take<int32_t>(n1);
        W.list_b = c.take<int32_t>(n1);
        W.list_h = c.take<int32_t>(n1);
        if (k >= 5) W.rowoff_b = c.take<int64_t>(n1);
        if (uses_hub_kernel(g, k)) W.hpre = c.take<int64_t>(n1);
        if (!lg_disabled(k)) {
            lg_workspace_bytes(g, k, &W.lg_bytes);
            W.lg = c.take<char>(W.lg_bytes);
        }
    }
    if (generic || (k >= 4 && uses_hub_kernel(g, k))) {
        W.gen_waves = persistent_blocks(kWPB, 8) * kWPB;
        W.gen_scratch = c.take<int32_t>((uint64_t)W.gen_waves * (kGenMaxK - 2) *
                                        (uint64_t)std::max(1, g->max_out_degree));
    }
    W.bytes = c.used;
    return W;
}

unsigned grid_for(int64_t items, int per_block, int cap_per_cu) {
    int64_t b = (items + per_block - 1) / per_block;
    int64_t cap = (int64_t)cu_count() * cap_per_cu;
    return (unsigned)std::max<int64_t>(1, std::min<int64_t>(b, cap));
}

// A persistent grid over the roots of out-degree above dmin: no more
// workgroups than the graph can have such roots (each takes dmin + 1 arcs).
unsigned roots_grid(const gpm_graph *g, int32_t dmin, int64_t blocks) {
    const int64_t most = std::min<int64_t>(g->n, g->m / (dmin + 1));
    return (unsigned)std::max<int64_t>(1, std::min(most, blocks));
}

// The class lists of k >= 4 (ctl and ctr zero on entry).
gpm_status clique_roots(const gpm_graph *g, CliqueWs &W, int32_t min_out, int32_t small_max,
                        int32_t mid_max, int32_t big_max, hipStream_t st) {
    RootLists L{{W.list_s, W.list_m, W.list_b, W.list_h}, (int32_t *)(W.ctl + 4), W.rowoff_b,
                W.ctr + 1, W.hpre, W.ctr + 2};
    if (g->n > 0)
        hipLaunchKernelGGL(k_clique_roots, dim3(grid_for(g->n, kRootsBlock, 8)), dim3(kBlock), 0,
                           st, g->dag_off, g->n, min_out, small_max, mid_max, big_max, L);
    GPM_LAUNCH_CHECK("k_clique_roots");
    return GPM_OK;
}

// Cliques rooted at the hub roots, the roots above the largest class, listed
// by clique_roots.  Nothing is launched on graphs without hubs.
template <int K, int MODE>
gpm_status hub_launch(const gpm_graph *g, CliqueWs &W, unsigned long long *res,
                      unsigned long long *res3, unsigned long long *res4, const RowEmitter &em,
                      hipStream_t st, bool all_roots = false) {
    if (!has_hubs(g) && !all_roots) return GPM_OK;
    {
        static const char *const kNames[] = {"k_clique_hub<4>", "k_clique_hub<5>",
                                             "k_clique_hub<6>", "k_clique_hub<7>",
                                             "k_clique_hub<8>", "k_clique_hub<9>"};
        Span sp(kNames[K - 4], st);
        hipLaunchKernelGGL((k_clique_hub<K, MODE>), dim3((unsigned)(W.gen_waves / kWPB)),
                           dim3(kBlock), 0, st, g->dag_off, g->dag_adj, W.list_h,
                           (const int64_t *)W.hpre, W.ctr + 2,
                           std::max(1, g->max_out_degree), W.gen_scratch, res, res3, res4, em);
    }
    GPM_LAUNCH_CHECK("k_clique_hub");
    return GPM_OK;
}

template <int K>
gpm_status launch_local(const gpm_graph *g, CliqueWs &W, unsigned long long *res,
                        unsigned long long *res3, unsigned long long *res4, hipStream_t st,
                        const RowEmitter *em = nullptr) {
    const int32_t *cnt = (const int32_t *)(W.ctl + 4);   // small, mid, big
    gpm_status rc = lg_cliques(g, K, W.list_m, cnt + 1, W.list_b, cnt + 2, W.rowoff_b, W.lg,
                               W.lg_bytes, res, res3, res4, em, st);
    if (rc) return rc;
    {
        static const char *const kNames[] = {"k_clique_wave<4>", "k_clique_wave<5>",
                                             "k_clique_wave<6>", "k_clique_wave<7>",
                                             "k_clique_wave<8>", "k_clique_wave<9>"};
        Span sp(kNames[K - 4], st);
        const dim3 grid(roots_grid(g, 0, (int64_t)cu_count() * g->cw_bpc));
        if (em)
            hipLaunchKernelGGL((k_clique_wave<K, true>), grid, dim3(kWave), 0, st, g->dag_off,
                               g->dag_adj, W.list_s, cnt, res, res3, res4, *em);
        else
            hipLaunchKernelGGL((k_clique_wave<K, false>), grid, dim3(kWave), 0, st, g->dag_off,
                               g->dag_adj, W.list_s, cnt, res, res3, res4, RowEmitter{});
    }
    GPM_LAUNCH_CHECK("k_clique_wave");
    if constexpr (K <= 5) {
        if (em) return hub_launch<K, HUB_LIST>(g, W, res, nullptr, nullptr, *em, st);
    }
    return hub_launch<K, HUB_COUNT>(g, W, res, res3, res4, RowEmitter{}, st);
}

}  // namespace

gpm_status clique_workspace_bytes(const gpm_graph *g, int32_t k, bool list, uint64_t *bytes) {
    if (k < 3 || k > kGenMaxK) return fail(GPM_UNSUPPORTED, "clique size must be in [3, 9]");
    *bytes = clique_layout(g, k, list, nullptr).bytes;
    return GPM_OK;
}

// Triangle count into *res (zero on entry, as are W.ctl and W.ctr); with MODE
// == TC_ARCS also adds 1 to the triangle count of each of the three arcs of
// every triangle (te, m words, zero on entry).  Uses the triangle workspace
// (clique_workspace_bytes(g, 3, false)).
template <int MODE>
static gpm_status tc_launch(const gpm_graph *g, CliqueWs &W, unsigned long long *res,
                            uint32_t *te, hipStream_t st, const RowEmitter &em = RowEmitter{}) {
    if (g->m == 0) return GPM_OK;
    if (timing_on()) {
        hipLaunchKernelGGL(k_tc_units, dim3(grid_for(g->m, kBlock, 8)), dim3(kBlock), 0, st,
                           g->dag_off, g->dag_adj, g->dag_src, g->m, W.ctr + 3);
        GPM_LAUNCH_CHECK("k_tc_units");
    }
    if (g->max_out_degree > kTcArcMax) {
        const Tau tau = tau_of(g);
        hipLaunchKernelGGL(k_tc_tasks, dim3(grid_for(g->n, kRootsBlock, 8)), dim3(kBlock), 0, st,
                           g->off, g->dag_off, g->n, tau, W.tasks, W.hub_tasks, W.ctl + 2);
        GPM_LAUNCH_CHECK("k_tc_tasks");
        const int64_t bpc = std::max(g->tc_bpc[1], g->tc_bpc[2]);
        const dim3 grid((unsigned)std::min<int64_t>((int64_t)tc_task_bound(g), cu_count() * bpc));
        {
            Span sp(MODE == TC_LIST ? "k_tc_seg<list>" : (MODE == TC_ARCS ? "k_tc_seg<arcs>" : "k_tc_seg"), st);
            hipLaunchKernelGGL((k_tc_seg<MODE, false>), grid, dim3(kBlock), 0, st, g->off, g->adj,
                               g->okey, g->dag_off, g->dag_adj, W.tasks, W.ctl + 2, tau,
                               (unsigned long long *)(W.ctl + kCtlCur),
                               res, te, em);
            span_units(W.ctr + 4, st);
        }
        GPM_LAUNCH_CHECK("k_tc_seg");
        if (has_hubs(g)) {
            Span sp("k_tc_seg<hub>", st);
            hipLaunchKernelGGL((k_tc_seg<MODE, true>), grid, dim3(kBlock), 0, st, g->off, g->adj,
                               g->okey, g->dag_off, g->dag_adj, W.hub_tasks, W.ctl + 3, tau,
                               (unsigned long long *)(W.ctl + kCtlCur + kCursorWords), res, te, em);
            span_units(W.ctr + 5, st);
        }
        GPM_LAUNCH_CHECK("k_tc_seg<hub>");
    }
    {
        Span sp(MODE == TC_LIST ? "k_tc_arcs<list>" : (MODE == TC_ARCS ? "k_tc_arcs<arcs>" : "k_tc_arcs"), st);
        hipLaunchKernelGGL(k_tc_arcs<MODE>, dim3(grid_for(g->m, kBlock, g->tc_bpc[0])),
                           dim3(kBlock), 0, st, g->dag_off, g->dag_adj, g->dag_src, g->m, res, te,
                           em);
        span_units(W.ctr + 3, st);
    }
    GPM_LAUNCH_CHECK("k_tc_arcs");
    return GPM_OK;
}

// Clears te (m words), *tri and the words of `also`, then counts.
gpm_status triangle_arc_counts(const gpm_graph *g, void *ws, uint64_t ws_bytes, uint32_t *te,
                               unsigned long long *tri, hipStream_t st, WordRun also) {
    CliqueWs W = clique_layout(g, 3, false, ws);
    if (W.bytes > ws_bytes) return fail(GPM_OUT_OF_MEMORY, "workspace smaller than required");
    GPM_HIP(zero_words(st, {{te, (uint64_t)g->m}, {tri, 2}, {W.ctr, 16}, {W.ctl, kCtlWords}, also}));
    return tc_launch<TC_ARCS>(g, W, tri, te, st);
}

gpm_status clique_run(const gpm_graph *g, int32_t k, bool list, void *ws, uint64_t ws_bytes,
                      unsigned long long *d_count, int32_t *d_buf, uint64_t cap,
                      unsigned long long *d_result, hipStream_t st) {
    CliqueWs W = clique_layout(g, k, list, ws);
    if (W.bytes > ws_bytes) return fail(GPM_OUT_OF_MEMORY, "workspace smaller than required");
    const int32_t n = g->n;
    // counts go straight to the caller's word, listing totals and checksums
    // to its three; the slot counter is in the workspace
    unsigned long long *res = list ? d_result : d_count;
    GPM_HIP(zero_words(st, {{res, list ? 6u : 2u}, {W.ctr, 16}, {W.ctl, kCtlWords},
                            {W.lg, W.lg ? kLgCtlWords : 0}}));
    const bool generic = uses_generic(g, k, list);
    RowEmitter em{W.ctr, d_buf, list ? cap : 0, 0, 0, 0};
    if (generic) {
        ListOut lo{d_buf, list ? cap : 0};
        int blocks = W.gen_waves / kWPB;
        if (list)
            hipLaunchKernelGGL(k_clique_generic<true>, dim3(blocks), dim3(kBlock), 0, st,
                               g->dag_off, g->dag_adj, n, k, std::max(1, g->max_out_degree),
                               W.gen_scratch, res, lo);
        else
            hipLaunchKernelGGL(k_clique_generic<false>, dim3(blocks), dim3(kBlock), 0, st,
                               g->dag_off, g->dag_adj, n, k, std::max(1, g->max_out_degree),
                               W.gen_scratch, res, lo);
        GPM_LAUNCH_CHECK("k_clique_generic");
        if (list) {
            hipLaunchKernelGGL(k_finish_listing, dim3(1), dim3(64), 0, st, res, cap);
            GPM_LAUNCH_CHECK("k_finish_listing");
        }
    } else if (k == 3) {
        gpm_status rc = list ? tc_launch<TC_LIST>(g, W, res, nullptr, st, em)
                             : tc_launch<TC_COUNT>(g, W, res, nullptr, st);
        if (rc) return rc;
    } else if (lg_disabled(k)) {
        // every root with out-degree >= k - 1 is a hub: one task per out-arc
        gpm_status rc = clique_roots(g, W, k - 1, 0, 0, 0, st);
        if (rc) return rc;
        switch (k) {
        case 4: rc = list ? hub_launch<4, HUB_LIST>(g, W, res, nullptr, nullptr, em, st, true)
                          : hub_launch<4, HUB_COUNT>(g, W, res, nullptr, nullptr, em, st, true); break;
        case 5: rc = list ? hub_launch<5, HUB_LIST>(g, W, res, nullptr, nullptr, em, st, true)
                          : hub_launch<5, HUB_COUNT>(g, W, res, nullptr, nullptr, em, st, true); break;
        case 6: rc = hub_launch<6, HUB_COUNT>(g, W, res, nullptr, nullptr, em, st, true); break;
        case 7: rc = hub_launch<7, HUB_COUNT>(g, W, res, nullptr, nullptr, em, st, true); break;
        case 8: rc = hub_launch<8, HUB_COUNT>(g, W, res, nullptr, nullptr, em, st, true); break;
        default: rc = hub_launch<9, HUB_COUNT>(g, W, res, nullptr, nullptr, em, st, true); break;
        }
        if (rc) return rc;
    } else {
        gpm_status rc = clique_roots(g, W, k - 1, 64, kMidMaxD, kTcMaxD, st);
        if (rc) return rc;
        const RowEmitter *pem = list ? &em : nullptr;
        switch (k) {
        case 4: rc = launch_local<4>(g, W, res, nullptr, nullptr, st, pem); break;
        case 5: rc = launch_local<5>(g, W, res, nullptr, nullptr, st, pem); break;
        case 6: rc = launch_local<6>(g, W, res, nullptr, nullptr, st); break;
        case 7: rc = launch_local<7>(g, W, res, nullptr, nullptr, st); break;
        case 8: rc = launch_local<8>(g, W, res, nullptr, nullptr, st); break;
        default: rc = launch_local<9>(g, W, res, nullptr, nullptr, st); break;
        }
        if (rc) return rc;
    }
    if (list && !generic) {
        hipLaunchKernelGGL(k_finish_rows, dim3(1), dim3(64), 0, st, res, W.ctr, cap);
        GPM_LAUNCH_CHECK("k_finish_rows");
    }
    return GPM_OK;
}

// Cliques of every size 3..kmax (kmax = 4 or 5) from one local-graph pass:
// the local graph of root u holds the triangles at u (its edges), the
// 4-cliques at u (its triangles) and the 5-cliques at u (its 4-cliques), so
// one build per root serves all sizes.  Roots need out-degree >= 2.
gpm_status clique_multi_workspace_bytes(const gpm_graph *g, int32_t kmax, uint64_t *bytes) {
    return clique_workspace_bytes(g, kmax, false, bytes);
}

gpm_status clique_multi_run(const gpm_graph *g, int32_t kmax, void *ws, uint64_t ws_bytes,
                            unsigned long long *d_counts, hipStream_t st) {
    if (kmax < 4 || kmax > 5) return fail(GPM_UNSUPPORTED, "kmax must be 4 or 5");
    CliqueWs W = clique_layout(g, kmax, false, ws);
    if (W.bytes > ws_bytes) return fail(GPM_OUT_OF_MEMORY, "workspace smaller than required");
    // d_counts = {triangles, 4-cliques[, 5-cliques]}
    unsigned long long *res = d_counts + (kmax - 3), *res3 = d_counts;
    unsigned long long *res4 = kmax == 5 ? d_counts + 1 : nullptr;
    GPM_HIP(zero_words(st, {{d_counts, (uint64_t)(2 * (kmax - 2))}, {W.ctr, 16}, {W.ctl, kCtlWords},
                            {W.lg, W.lg ? kLgCtlWords : 0}}));
    if (lg_disabled(kmax)) {
        // without local graphs: every root of out-degree >= 2 per arc
        gpm_status rc = clique_roots(g, W, 2, 0, 0, 0, st);
        if (rc) return rc;
        return kmax == 4 ? hub_launch<4, HUB_COUNT>(g, W, res, res3, nullptr, RowEmitter{}, st, true)
                         : hub_launch<5, HUB_COUNT>(g, W, res, res3, res4, RowEmitter{}, st, true);
    }
    gpm_status rc = clique_roots(g, W, 2, 64, kMidMaxD, kTcMaxD, st);
    if (rc) return rc;
    return kmax == 4 ? launch_local<4>(g, W, res, res3, nullptr, st)
                     : launch_local<5>(g, W, res, res3, res4, st);
}

}  // namespace gpm
