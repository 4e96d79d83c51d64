// Local-graph 4- and 5-clique counting for roots of out-degree 65..1024.
//
// For a root u of the degree-ordered DAG the local graph is the subgraph
// induced on N+(u), itself oriented (Section 5, search on a local graph; the
// local graph here is built once per root and kept as bit rows instead of
// being shrunk in place).  Row i holds, as a bit set over local indices, the
// out-neighbours of the i-th out-neighbour v_i that lie in N+(u).  Then
//   4-cliques rooted at u = sum over local edges (i, j) of |row_i & row_j|,
//   5-cliques rooted at u = sum over local edges (i, j), l in row_i & row_j
//                           of |row_i & row_j & row_l|.
// Rows are 64-bit words in LDS (at most 1024 x 16 words = 128 KiB of the
// 160 KiB a gfx950 workgroup may use).
//
// Both sums run as 32 x 32 tiles of pairs on the matrix cores, the rows' bits
// expanded to FP4 in registers (local_tri, lg5_tiles); larger cliques descend
// with AND + population count.
//
// 4-cliques: one workgroup per root builds the rows and counts.
// 5-cliques and larger: counting can cost far more than building on hub roots,
// so above 256 out-neighbours one kernel builds every root's rows once and
// stores them in HBM, and a second splits each root into slices of its local
// vertices (i = s mod S, S proportional to the root's local triangles); a slice
// copies the rows back into LDS and its waves take the vertices as they become
// free.  Roots of 65..256 do both in one kernel.
#include "gpm_internal.h"

#include <algorithm>

namespace gpm {

namespace {

constexpr int kMidMaxD = 256;
constexpr int kBigMaxD = 1024;
constexpr int kMidThreads = 256;
constexpr int kBigThreads = 1024;
// the big class's roots of out-degree 257..512 run at this bound: a third of
// the LDS, three workgroups per CU
constexpr int kHalfMaxD = 512;
constexpr int kHalfThreads = 512;
constexpr int kHalfBlocksPerCu = 3;
// Threads and workgroups per CU of the 5-clique kernel: by registers, 4 waves a
// SIMD for local graphs of up to 8 words a row and 3 up to 16 (RMAT-20: 8.4 ms,
// 9.2 with 2 waves, both before the operands of 10 words and more left scratch
// memory; 6.5 now).  The descents of larger cliques and the listing, whose
// tasks differ more, take one workgroup of 16 waves (6-cliques of RMAT-16: 6.4
// ms in this class; 11.3 with two of 8).
template <int DMAX, bool TILES> struct Lg5Block {
    static constexpr int kThreads = !TILES ? 1024 : (DMAX == 512 ? 512 : 768);
    static constexpr int kWaves = !TILES ? 4 : (DMAX == 512 ? 4 : 3);
    static constexpr int kPerCu = TILES && DMAX == 512 ? 2 : 1;
};
// waves per SIMD of the middle class's 5-clique kernel (RMAT-20: 5.0 ms; 5.4 at
// 5 and 5.2 at 7, for want of waves and for spills)
constexpr int kMidWaves = 6;
constexpr int32_t kMaxSlices = 1024;

__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ int last_le_i32(const int32_t *a, int n, int32_t x) {
    int lo = 0, hi = n;
    while (hi - lo > 1) {
        int mid = (lo + hi) >> 1;
        if (a[mid] <= x) lo = mid; else hi = mid;
    }
    return lo;
}

// Position of the r-th set bit (0-based) of x; x must have more than r bits.
__device__ __forceinline__ int select_bit64(uint64_t x, int r) {
    int pos = 0;
#pragma unroll
    for (int s = 32; s > 0; s >>= 1) {
        const int low = __popcll(x & ((1ull << s) - 1));
        if (r >= low) {
            r -= low;
            x >>= s;
            pos += s;
        }
    }
    return pos;
}

template <int NT>
struct Lds {
    int32_t s_sum[NT / kWave];
    int32_t s_task;
    uint32_t s_next;
    int32_t s_slices;
    uint64_t s_tri;
};

// A 5-clique task: the local vertices slice, slice + slices, ... of the
// r-th root of its class.
struct LgTask {
    int32_t r;
    uint16_t slice, slices;
};

// Hash table of a local-graph block: 4 slots per out-neighbour at the class
// bound (load factor <= 1/4); at the 1024 bound 2 (<= 1/4 up to half the
// bound, <= 1/2 at the bound), so its rows (128 KiB) and the table fit the
// 160 KiB of LDS.
template <int DMAX> struct LgHash {
    static constexpr int kSlots = DMAX >= 1024 ? 2 * DMAX : 4 * DMAX;
    static constexpr int kBits = DMAX >= 1024 ? 11 : (DMAX == 512 ? 11 : (DMAX == 256 ? 10 : 8));
    static_assert((1 << kBits) == kSlots, "slots must be a power of two");
};

// Row words of a class's LDS area, and the rows' stride: odd where it fits, so
// that a column of words is spread over the banks.
template <int DMAX> struct LgRows {
    static constexpr int kWords = DMAX == 256 ? 256 * 5 : DMAX * (DMAX / 64);
    static __device__ __forceinline__ int32_t stride(int32_t d, int32_t W) {
        return d * (W | 1) <= kWords ? W | 1 : W;
    }
};

// Builds the local graph of root u (d out-neighbours, W words per row at
// stride S) in LDS: row a gets bit b for every pair (v, w) of the root with v, w the
// out-neighbours of local indices a and b.  Local indices are positions in
// the out-list, or with RANK positions in the DAG's order, by (okey, id)
// (the graph's orientation key: degrees, or the core-value key); lidx, d
// entries, receives them.  That makes every row hold only bits above its
// own index.
// keys/vals/pre/offj are the root's staging area; ends with a barrier.
template <int DMAX, int NT, bool RANK>
__device__ void build_rows(const int32_t *__restrict__ off, const int32_t *__restrict__ okey,
                           const int32_t *__restrict__ dag_off,
                           const int32_t *__restrict__ dag_adj, int32_t u, int32_t d, int32_t S,
                           uint64_t *rows, int32_t *keys, int16_t *vals, int32_t *pre,
                           int32_t *offj, int16_t *lidx, int32_t *s_sum,
                           int32_t *verts = nullptr) {
    constexpr int PER = (DMAX + NT - 1) / NT;
    constexpr int NW = NT / kWave;
    constexpr int U = DMAX <= 256 ? 2 : 4;
    const int32_t s = dag_off[u];
    if (RANK) {
        // rank of each out-neighbour among the others, by (degree, id); the
        // row area is scratch for the keys until it is cleared below
        uint64_t *key = rows;
        for (int32_t i = threadIdx.x; i < d; i += NT) {
            const int32_t v = dag_adj[s + i];
            key[i] = ((uint64_t)(uint32_t)okey[v] << 32) | (uint32_t)v;
        }
        __syncthreads();
        for (int32_t i = threadIdx.x; i < d; i += NT) {
            const uint64_t k = key[i];
            int32_t c = 0;
            for (int32_t j = 0; j < d; j++) c += key[j] < k;
            lidx[i] = (int16_t)c;
        }
        __syncthreads();
    }
    const int32_t hb = min(lds_hash_bits(d), LgHash<DMAX>::kBits);
    for (int32_t i = threadIdx.x; i < (1 << hb); i += NT) keys[i] = -1;
    for (int32_t i = threadIdx.x; i < d * S; i += NT) rows[i] = 0ull;
    stage_root<NT, PER>(dag_off, dag_adj, s, d, keys, vals, hb, pre, offj, s_sum,
                        RANK ? lidx : nullptr, verts);
    const int32_t npairs = pre[d];
    const int32_t per_wave = ((npairs + NW - 1) / NW + U * kWave - 1) / (U * kWave) * (U * kWave);
    const int32_t qa = min(npairs, (int32_t)(threadIdx.x / kWave) * per_wave);
    const int32_t qz = min(npairs, qa + per_wave);
    walk_lookup<U>(pre, offj, dag_adj, d, qa, qz, keys, hb,
            [&](int32_t j, int32_t, int32_t w, int32_t slot) {
        if (slot >= 0) {
            const int32_t a = RANK ? (int32_t)lidx[j] : j;
            const int32_t b = vals[slot];
            atomicOr((unsigned long long *)&rows[a * S + (b >> 6)], 1ull << (b & 63));
        }
    });
    __syncthreads();
}

// pre[i] = number of local edges in rows 0..i-1; returns the total.
template <int DMAX, int NT>
__device__ int32_t row_prefix(const uint64_t *rows, int32_t d, int32_t W, int32_t S, int32_t *pre,
                              int32_t *s_sum) {
    constexpr int PER = (DMAX + NT - 1) / NT;
    int32_t pc[PER];
#pragma unroll
    for (int q = 0; q < PER; q++) {
        const int32_t i = threadIdx.x * PER + q;
        pc[q] = 0;
        if (i < d)
            for (int32_t w = 0; w < W; w++) pc[q] += __popcll(rows[i * S + w]);
    }
    block_prefix<NT, PER>(pc, d, pre, s_sum);
    return pre[d];
}

// Local edge number e -> (row i, column j).
__device__ __forceinline__ void edge_at(const uint64_t *rows, const int32_t *pre, int32_t d,
                                        int32_t S, int32_t e, int32_t &i, int32_t &j) {
    i = last_le_i32(pre, d + 1, e);
    int32_t rr = e - pre[i];
    const uint64_t *ri = rows + i * S;
    int32_t wj = 0;
    for (;; wj++) {
        const int pc = __popcll(ri[wj]);
        if (rr < pc) break;
        rr -= pc;
    }
    j = wj * 64 + select_bit64(ri[wj], rr);
}

__device__ __forceinline__ uint64_t uniform64(uint64_t x) {
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)x);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(x >> 32));
    return ((uint64_t)hi << 32) | lo;
}

__device__ __forceinline__ uint64_t wave_or64(uint64_t x) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x |= __shfl_xor(x, o, 64);
    return uniform64(x);
}

// part + the sum over the columns b of word q listed in m (wave-uniform) of
// [bit b of X[q]] * sum over w >= q of popc(X[w] & row_b[w]).  The halves of
// the word are walked one after the other, so the lane's bit test is one
// bit-field extract of a 32-bit register and its product with the count one
// 24-bit multiply-add; row_b is a broadcast LDS read.
template <int W, int S>
__device__ __forceinline__ uint32_t pair_sweep(const uint64_t *rows, const uint64_t (&X)[W], int q,
                                               uint64_t m, uint32_t part) {
#pragma unroll
    for (int h = 0; h < 2; h++) {
        const uint32_t x = (uint32_t)(X[q] >> (32 * h));
        uint32_t mh = (uint32_t)(m >> (32 * h));
        while (mh) {
            const int bp = __builtin_ctz(mh);
            mh &= mh - 1u;
            const uint64_t *yb = rows + (q * kWave + h * 32 + bp) * S;
            uint32_t sc = 0;
#pragma unroll
            for (int w = q; w < W; w++) sc += (uint32_t)__popcll(X[w] & yb[w]);
            // written as instructions: the compiler would otherwise turn the
            // 0/1 product into a compare and a select
            uint32_t bit, np;
            asm("v_bfe_u32 %0, %1, %2, 1" : "=v"(bit) : "v"(x), "s"(bp));
            asm("v_mad_u32_u24 %0, %1, %2, %3" : "=v"(np) : "v"(bit), "v"(sc), "v"(part));
            part = np;
        }
    }
    return part;
}

// Units of the products: 2^-16 for counts, and 2^-5, i.e. 2048 of the first.
constexpr int kFp4Count = 0x6f6f6f6f, kFp4Adj = 0x7a7a7a7a;
// sum + a tile's counts at entries whose adjacency bit (2048) is set.
__device__ __forceinline__ uint32_t fp4_masked_sum(const f32x16 &C, uint32_t sum) {
    typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
#pragma unroll
    for (int r = 0; r < 16; r += 2) {
        u16x2 p = __builtin_bit_cast(u16x2, __builtin_amdgcn_cvt_pknorm_u16(C[r], C[r + 1]));
        p = __builtin_elementwise_sub_sat(p, u16x2{2048, 2048});
        sum = __builtin_amdgcn_udot2(p, u16x2{1, 1}, sum, false);
    }
    return sum;
}

// Triangles of a local graph in degree order (d vertices, W words per row at
// stride S, every row holding only bits above its own index): the sum over
// local edges a -> b of |row_a & row_b|, on the matrix cores as in lg5_tiles,
// with consecutive vertices for members and every word for R.  Tiles (ta <=
// tb) are dealt round robin to the nw waves; b's operands are expanded at each
// tile, which keeps the registers of the building phase.  Rows from d on are
// taken as row d - 1, which is empty, and their own bits are beyond every row.
// Returns the calling lane's share.
__device__ __forceinline__ uint64_t local_tri(const uint64_t *rows, int32_t d, int32_t W, int32_t S,
                                              int wib, int nw) {
    const int lane = lane_id(), l32 = lane & 31, half = lane >> 5;
    const uint32_t *rows32 = reinterpret_cast<const uint32_t *>(rows) + half;
    const int32_t T = (d + 31) / 32, tiles = T * (T + 1) / 2;
    uint32_t sum = 0;
    int32_t tb = 0, before = 0;   // the tiles of the columns before tb
    for (int32_t p = __builtin_amdgcn_readfirstlane(wib); p < tiles; p += nw) {
        while (before + tb + 1 <= p) before += ++tb;
        const int32_t ta = p - before;
        const uint32_t *ra = rows32 + min(ta * 32 + l32, d - 1) * (2 * S);
        const uint32_t *rb = rows32 + min(tb * 32 + l32, d - 1) * (2 * S);
        const int32_t q0 = tb >> 1;
        uint32_t aw = ra[2 * (W - 1)], bw = rb[2 * (W - 1)];
        fp4x64 A;
        f32x16 C = {};
        for (int32_t q = W - 1; q >= q0; q--) {
            A = fp4_left(aw);
            const fp4x64 B = fp4_right(bw);
            const int32_t nq = max(q - 1, q0);
            aw = ra[2 * nq];
            bw = rb[2 * nq];
            C = fp4_step(A, B, C, kFp4Count);
        }
        C = fp4_step(A, fp4_right(half == (tb & 1) ? 1u << l32 : 0u), C, kFp4Adj);
        sum = fp4_masked_sum(C, sum);
    }
    return sum;
}

// 4-cliques: workgroup per root (from the work cursors; roots of out-degree
// <= dlo are left to another launch); the root's 4-cliques are the triangles of
// its local graph.  RANK puts the local graph in degree order, in which they are
// counted (local_tri); the listing needs no order.  With LIST every 4-clique
// (u, v_i, v_j, v_x) is emitted instead.  Bound by the building of the rows,
// i.e. the lookups; the sum over local edges that local_tri replaced took
// another 30 to 60 % (RMAT, 100,003 vertices, roots of 65..256: 425 us, now
// 307; out-degrees up to 1,024 at density 0.83: 657 us, now 400).
template <int DMAX, int NT, bool LIST, bool RANK>
__global__ void __launch_bounds__(NT, DMAX == kHalfMaxD ? 6 : (DMAX == kMidMaxD ? 8 : 1))
    k_lg4(const int32_t *__restrict__ off,
                                            const int32_t *__restrict__ okey,
                                            const int32_t *__restrict__ dag_off,
                                            const int32_t *__restrict__ dag_adj,
                                            const int32_t *__restrict__ roots,
                                            const int32_t *__restrict__ nroots_p, int32_t dlo,
                                            unsigned long long *cursor, unsigned long long *result,
                                            unsigned long long *res3, RowEmitter em) {
    __shared__ uint64_t rows[LgRows<DMAX>::kWords];
    __shared__ __align__(16) int32_t keys[LgHash<DMAX>::kSlots];
    __shared__ int16_t vals[LgHash<DMAX>::kSlots];
    __shared__ int32_t offj[DMAX], pre[DMAX + 1];
    __shared__ int32_t verts[LIST ? DMAX : 1];
    __shared__ int16_t lidx[RANK ? DMAX : 1];
    __shared__ Lds<NT> sh;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    TaskQueue queue(cursor, *nroots_p, blockIdx.x, gridDim.x);
    uint64_t acc = 0;
    for (;;) {
        if (wave == 0) {
            const int32_t got = (int32_t)queue.next();
            if (tid == 0) sh.s_task = got;
        }
        __syncthreads();
        const int32_t r = sh.s_task;
        __syncthreads();
        if (r < 0) break;
        const int32_t u = roots[r];
        const int32_t d = dag_off[u + 1] - dag_off[u], W = (d + 63) >> 6;
        if (d <= dlo || d > DMAX) continue;
        const int32_t S = LgRows<DMAX>::stride(d, W);
        build_rows<DMAX, NT, RANK>(off, okey, dag_off, dag_adj, u, d, S, rows, keys, vals, pre, offj,
                                   RANK ? lidx : nullptr, sh.s_sum, LIST ? verts : nullptr);
        const int32_t ne = row_prefix<DMAX, NT>(rows, d, W, S, pre, sh.s_sum);
        if (res3 && tid == 0 && ne) atomicAdd(res3, (unsigned long long)ne);   // triangles at u
        if constexpr (LIST) {
            for (int32_t e = tid; e < ne; e += NT) {
                int32_t i, j;
                edge_at(rows, pre, d, S, e, i, j);
                const uint64_t *ri = rows + i * S, *rj = rows + j * S;
                for (int32_t w = 0; w < W; w++) {
                    uint64_t m = ri[w] & rj[w];
                    while (m) {
                        const int32_t x = w * 64 + __builtin_ctzll(m);
                        m &= m - 1ull;
                        const int32_t q[4] = {u, verts[i], verts[j], verts[x]};
                        emit_vertices<4>(em, q);
                    }
                }
            }
        } else if (ne) {
            acc += local_tri(rows, d, W, S, tid / kWave, NT / kWave);
        }
        __syncthreads();
    }
    if (LIST) {
        row_emitter_flush(em, result);
        return;
    }
    acc = wave_sum(acc);
    if (lane_id() == 0 && acc) atomicAdd(result, (unsigned long long)acc);
}

// 5-cliques, step 1: rows of every root (local indices in degree order) to
// HBM, and local triangle counts for slicing.
template <int DMAX, int NT>
__global__ void __launch_bounds__(NT, DMAX == kHalfMaxD ? 6 : 1) k_lg_build(const int32_t *__restrict__ off,
                                                 const int32_t *__restrict__ okey,
                                                 const int32_t *__restrict__ dag_off,
                                                 const int32_t *__restrict__ dag_adj,
                                                 const int32_t *__restrict__ roots,
                                                 const int32_t *__restrict__ nroots_p, int32_t dlo,
                                                 unsigned long long *cursor, const int64_t *__restrict__ rowoff,
                                                 uint64_t *grows, LgTask *tasks, uint32_t *ntasks,
                                                 unsigned long long *units,
                                                 unsigned long long *res3,
                                                 unsigned long long *res4, uint64_t slice5) {
    __shared__ uint64_t rows[LgRows<DMAX>::kWords];
    __shared__ __align__(16) int32_t keys[LgHash<DMAX>::kSlots];
    __shared__ int16_t vals[LgHash<DMAX>::kSlots];
    __shared__ int16_t lidx[DMAX];
    __shared__ int32_t offj[DMAX], pre[DMAX + 1];
    __shared__ int32_t verts[DMAX];
    __shared__ Lds<NT> sh;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    TaskQueue queue(cursor, *nroots_p, blockIdx.x, gridDim.x);
    if (tid == 0) sh.s_tri = 0;
    for (;;) {
        if (wave == 0) {
            const int32_t got = (int32_t)queue.next();
            if (tid == 0) sh.s_task = got;
        }
        __syncthreads();
        const int32_t r = sh.s_task;
        __syncthreads();
        if (r < 0) break;
        const int32_t u = roots[r];
        const int32_t d = dag_off[u + 1] - dag_off[u], W = (d + 63) >> 6;
        if (d <= dlo || d > DMAX) continue;
        const int32_t S = LgRows<DMAX>::stride(d, W);
        build_rows<DMAX, NT, true>(off, okey, dag_off, dag_adj, u, d, S, rows, keys, vals, pre, offj,
                                   lidx, sh.s_sum, verts);
        uint64_t *dst = grows + rowoff[r];
        for (int32_t i = tid / kWave; i < d; i += NT / kWave)
            if (lane_id() < W) dst[i * W + lane_id()] = rows[i * S + lane_id()];
        // then the out-neighbours in local (degree) order, for listings
        int32_t *dverts = reinterpret_cast<int32_t *>(dst + d * W);
        for (int32_t i = tid; i < d; i += NT) dverts[i] = verts[i];
        const int32_t ne = row_prefix<DMAX, NT>(rows, d, W, S, pre, sh.s_sum);
        if (res3 && tid == 0 && ne) atomicAdd(res3, (unsigned long long)ne);   // triangles at u
        // local triangles (the 4-cliques at u): the 5-clique work
        uint64_t tri = ne ? local_tri(rows, d, W, S, tid / kWave, NT / kWave) : 0;
        tri = wave_sum(tri);
        if (lane_id() == 0 && tri) atomicAdd((unsigned long long *)&sh.s_tri, (unsigned long long)tri);
        __syncthreads();
        if (tid == 0) {
            // slices over local vertices: about slice5 local triangles each
            // (per graph, gpm_graph::lg5_slice), at least 8 local vertices each;
            // none without a local triangle (5-cliques of K_{300,3000}, 3,000
            // such roots: 228 us, now 145)
            const uint64_t s_work = sh.s_tri ? 1 + sh.s_tri / slice5 : 0;
            const uint64_t s_cap = (uint64_t)(d / 8 + 1);
            const int32_t S = (int32_t)std::min<uint64_t>(kMaxSlices, std::min(s_work, s_cap));
            sh.s_slices = S;
            sh.s_next = atomicAdd(ntasks, (uint32_t)S);
            if (sh.s_tri) atomicAdd(units, (unsigned long long)sh.s_tri);
            if (sh.s_tri && res4) atomicAdd(res4, (unsigned long long)sh.s_tri);
            sh.s_tri = 0;
        }
        __syncthreads();
        for (int32_t i = tid; i < sh.s_slices; i += NT)
            tasks[DMAX == kHalfMaxD ? sh.s_next + i : -1 - (int64_t)(sh.s_next + i)] = {r, (uint16_t)i, (uint16_t)sh.s_slices};
        __syncthreads();
    }
}

// 5-cliques and larger, step 2: task (root, slice); rows come back from HBM
// into LDS.  For local vertex i with out-row R (members p_0 < ... < p_{c-1}),
// the 5-cliques {u, v_i, ...} are the triangles a < b < x of the local DAG
// inside R: the sum over members a < b of [a -> b] * |row_a & R & row_b|.
// LDS is dynamic: rows (dmax x row_stride words for the class's largest
// out-degree), then per wave a member list of DMAX int16.

// That sum by population counts, for the leaves of the descents below (k > 5).
// Lanes own a (64 members at a time, row_a & R in registers); b runs over
// R's members in a wave-uniform loop, so row_b is a broadcast LDS read, and
// the AND + population count runs over the words from b's word up (a row
// only holds bits above its own vertex).  Local graphs of hub roots are
// dense, so testing every pair costs little more than following edges and
// keeps all 64 lanes busy.
template <int W, int S>
__device__ __forceinline__ uint64_t lg5_sweep(const uint64_t *rows, const uint64_t *ri, int32_t c,
                                              int16_t *mem) {
    const int lane = lane_id();
    uint64_t R[W];
#pragma unroll
    for (int q = 0; q < W; q++) R[q] = uniform64(ri[q]);
    int32_t base = 0;
#pragma unroll
    for (int q = 0; q < W; q++) {
        if ((R[q] >> lane) & 1ull) mem[base + lanes_below(R[q])] = (int16_t)(q * 64 + lane);
        base += __popcll(R[q]);
    }
    wave_sync();
    uint64_t acc = 0;
    for (int32_t a0 = 0; a0 < c; a0 += kWave) {
        const int32_t a = a0 + lane;
        uint64_t X[W];
        if (a < c) {
            const uint64_t *ra = rows + (int32_t)mem[a] * S;
#pragma unroll
            for (int q = 0; q < W; q++) X[q] = ra[q] & R[q];
        } else {
#pragma unroll
            for (int q = 0; q < W; q++) X[q] = 0ull;
        }
        const int32_t p0 = __builtin_amdgcn_readfirstlane((int32_t)mem[a0]);
        const int32_t q0 = p0 >> 6;
        uint32_t part = 0;
#pragma unroll
        for (int q = 0; q < W; q++) {
            if (q < q0) continue;
            uint64_t m = R[q];
            if (q == q0) m &= ~((2ull << (p0 & 63)) - 1ull);   // members above p0
            part = pair_sweep<W, S>(rows, X, q, m, part);
        }
        acc += part;
    }
    wave_sync();
    return acc;
}

// f(q) for q = Q, Q - 1, .. first, each q a constant, so that the arrays it
// indexes stay in registers.  (As a loop with a break the compiler left the
// product's steps rolled from 10 words on, with the operands in scratch memory:
// 7,000 vertices, out-degrees up to 986, 16.2 ms, now 6.7; RMAT-20 7.7, now 6.4.)
template <int Q, class F>
__device__ __forceinline__ void down_to(int32_t first, F &&f) {
    if constexpr (Q >= 0) {
        if (Q < first) return;
        f(std::integral_constant<int, Q>());
        down_to<Q - 1>(first, f);
    }
}

// The same sum (5-cliques) on the matrix cores.  A tile is 32 members a by 32
// members b, taken by their indices from the list, so the 0/1 product needs
// only c x c / 2 of its d x d entries; its 64-entry steps run over the row
// words from b's up, with R cut out of b's rows.  b's operands stay in registers
// over all a's tiles.  The step that holds b's own bits is taken twice, the
// second time with that bit alone and the weight 2048 (more than any
// count), which puts [a -> b] beside the count: an entry's share is what is
// left above 2048, if anything is.  The unit is 2^-16, so that two entries
// become 16-bit counts by one conversion to fractions of 1 (n - n / 65536 rounds
// to n below 32768) and the rest is a saturating subtraction and a dot product.
// Sums stay whole: an entry is below 2^24 units and a lane adds at most
// 528 tiles x 16 entries x 1021.  The last tile repeats the last member, whose
// row has nothing inside R: it adds nothing on either side.
// Bound by the vector units: about 90 operations a wave and tile of 2.7 steps,
// 85 % of its time; the matrix cores take 28 %.  RMAT-20, 3.7e7 tiles: 6.5 ms; by
// population counts, as lg5_sweep, 15.1.
template <int W, int S>
__device__ __forceinline__ uint64_t lg5_tiles(const uint64_t *rows, const uint64_t *ri, int32_t c,
                                              int16_t *mem) {
    const int lane = lane_id(), l32 = lane & 31, half = lane >> 5;
    uint64_t R[W];
#pragma unroll
    for (int q = 0; q < W; q++) R[q] = uniform64(ri[q]);
    int32_t base = 0;
#pragma unroll
    for (int q = 0; q < W; q++) {
        if ((R[q] >> lane) & 1ull) mem[base + lanes_below(R[q])] = (int16_t)(q * 64 + lane);
        base += __popcll(R[q]);
    }
    wave_sync();
    const uint32_t *rows32 = reinterpret_cast<const uint32_t *>(rows) + half;
    uint32_t sum = 0;
    for (int32_t tb = 0; tb < c; tb += 32) {
        const int32_t pb = mem[min(tb + l32, c - 1)];
        const int32_t q0 = __builtin_amdgcn_readfirstlane((int32_t)mem[tb]) >> 6;
        const int32_t q1 = __builtin_amdgcn_readfirstlane((int32_t)mem[min(tb + 31, c - 1)]) >> 6;
        const int32_t wb = (pb >> 5) - half;   // 2 q of the word that holds b, in this half
        const uint32_t ob = 1u << (pb & 31);
        const fp4x64 O0 = fp4_right(wb == 2 * q0 ? ob : 0u);
        const fp4x64 O1 = fp4_right(wb == 2 * q0 + 2 ? ob : 0u);
        uint32_t bw[W];
#pragma unroll
        for (int q = 0; q < W; q++) bw[q] = rows32[pb * (2 * S) + 2 * q];
        fp4x64 XB[W];
        down_to<W - 1>(q0, [&](auto q) {
            const uint32_t m = half ? (uint32_t)(R[q] >> 32) : (uint32_t)R[q];
            XB[q] = fp4_right(bw[q] & m);
        });
        int32_t pa = mem[min(l32, c - 1)];
        for (int32_t ta = 0; ta <= tb; ta += 32) {
            uint32_t aw[W];
            const uint32_t *ra = rows32 + pa * (2 * S);
            // (opaque, or the compiler keeps a condition per word)
            int32_t first = q0;
            asm volatile("" : "+s"(first));
            down_to<W - 1>(first, [&](auto q) { aw[q] = ra[2 * q]; });
            pa = mem[min(ta + 32 + l32, c - 1)];   // the next tile's
            f32x16 C = {};
            fp4x64 A = fp4_left(aw[W - 1]), A1 = A;
            C = fp4_step(A, XB[W - 1], C, kFp4Count);
            down_to<W - 2>(first, [&](auto q) {
                A1 = A;
                A = fp4_left(aw[q]);
                C = fp4_step(A, XB[q], C, kFp4Count);
            });
            // 2048 where a -> b: b's own bit, in words q0 .. q1
            C = fp4_step(A, O0, C, kFp4Adj);
            if (q1 > first) {
                C = fp4_step(A1, O1, C, kFp4Adj);
                for (int32_t q = first + 2; q <= q1; q++)
                    C = fp4_step(fp4_left(ra[2 * q]), fp4_right(wb == 2 * q ? ob : 0u), C, kFp4Adj);
            }
            sum = fp4_masked_sum(C, sum);
        }
    }
    wave_sync();
    return (uint64_t)sum;
}

// Listing form: emits every 5-clique {u, v_i, a, b, x} with
// a < b < x a triangle inside R (vertex ids from verts, the out-neighbours
// in local order).
template <int W, int S>
__device__ void lg5_list(const uint64_t *rows, const uint64_t *ri, int32_t c, int16_t *mem,
                         const int32_t *verts, int32_t u, int32_t vi, RowEmitter &em) {
    const int lane = lane_id();
    uint64_t R[W];
#pragma unroll
    for (int q = 0; q < W; q++) R[q] = uniform64(ri[q]);
    int32_t base = 0;
#pragma unroll
    for (int q = 0; q < W; q++) {
        if ((R[q] >> lane) & 1ull) mem[base + lanes_below(R[q])] = (int16_t)(q * 64 + lane);
        base += __popcll(R[q]);
    }
    wave_sync();
    for (int32_t a0 = 0; a0 < c; a0 += kWave) {
        const int32_t a = a0 + lane;
        uint64_t X[W];
        int32_t pa = 0;
        if (a < c) {
            pa = mem[a];
            const uint64_t *ra = rows + pa * S;
#pragma unroll
            for (int q = 0; q < W; q++) X[q] = ra[q] & R[q];
        } else {
#pragma unroll
            for (int q = 0; q < W; q++) X[q] = 0ull;
        }
        const int32_t p0 = __builtin_amdgcn_readfirstlane((int32_t)mem[a0]);
        const int32_t q0 = p0 >> 6;
#pragma unroll
        for (int q = 0; q < W; q++) {
            if (q < q0) continue;
            uint64_t m = R[q];
            if (q == q0) m &= ~((2ull << (p0 & 63)) - 1ull);
            while (m) {
                const int bp = __builtin_ctzll(m);
                m &= m - 1ull;
                const int32_t pb = q * 64 + bp;
                if ((X[q] >> bp) & 1ull) {
                    const uint64_t *yb = rows + pb * S;
#pragma unroll
                    for (int w = q; w < W; w++) {
                        uint64_t mm = X[w] & yb[w];
                        while (mm) {
                            const int32_t x = w * 64 + __builtin_ctzll(mm);
                            mm &= mm - 1ull;
                            const int32_t clq[5] = {u, vi, verts[pa], verts[pb], verts[x]};
                            emit_vertices<5>(em, clq);
                        }
                    }
                }
            }
        }
    }
    wave_sync();
}

// The same for the widest rows (the class above 512), read from LDS where they
// are used.  With the words in registers as above, each of the W (W + 1) / 2
// pairs of words holds a copy of the emission: 63 to 187 KB of code from 9 to
// 16 words, more than an instruction cache, and above 128 KB more than a branch
// reaches.  (The compiler then jumped through the register pair of the return
// address, and 14 words never came back.)
__device__ __forceinline__ void lg5_list_wide(const uint64_t *rows, int32_t S, int32_t W,
                                              const uint64_t *ri, int32_t c, int16_t *mem,
                                              const int32_t *verts, int32_t u, int32_t vi,
                                              RowEmitter &em) {
    const int lane = lane_id();
    int32_t base = 0;
    for (int32_t q = 0; q < W; q++) {
        const uint64_t R = uniform64(ri[q]);
        if ((R >> lane) & 1ull) mem[base + lanes_below(R)] = (int16_t)(q * 64 + lane);
        base += __popcll(R);
    }
    wave_sync();
    for (int32_t a0 = 0; a0 < c; a0 += kWave) {
        const int32_t a = a0 + lane, pa = mem[min(a, c - 1)];
        const uint64_t *ra = rows + pa * S;
        for (int32_t b = a0 + 1; b < c; b++) {
            const int32_t pb = __builtin_amdgcn_readfirstlane((int32_t)mem[b]), q = pb >> 6;
            if (a >= c || !((ra[q] >> (pb & 63)) & 1ull)) continue;   // a -> b: b is above a
            const uint64_t *yb = rows + pb * S;
            for (int32_t w = q; w < W; w++) {
                uint64_t mm = ra[w] & yb[w] & ri[w];
                while (mm) {
                    const int32_t x = w * 64 + __builtin_ctzll(mm);
                    mm &= mm - 1ull;
                    const int32_t clq[5] = {u, vi, verts[pa], verts[pb], verts[x]};
                    emit_vertices<5>(em, clq);
                }
            }
        }
    }
    wave_sync();
}

template <int WLO, int WHI>
__device__ __forceinline__ void lg5_list_dispatch(int32_t W, const uint64_t *rows,
                                                  const uint64_t *ri, int32_t c, int16_t *mem,
                                                  const int32_t *verts, int32_t u, int32_t vi,
                                                  RowEmitter &em) {
    if constexpr (WLO <= WHI) {
        if (W == WLO) lg5_list<WLO, (WLO | 1)>(rows, ri, c, mem, verts, u, vi, em);
        else lg5_list_dispatch<WLO + 1, WHI>(W, rows, ri, c, mem, verts, u, vi, em);
    }
}

// (e + 3)-cliques of the local DAG inside the set S (W words, c >= 3
// members): for e = 0 the triangles inside S; for e > 0 the sum over members
// v of S of the (e + 2)-cliques inside S & row_v (rows hold only bits above
// their own index, so each clique is found once, from its lowest member).
// The descent is wave-uniform and iterative: level l keeps its set and the
// members still to visit in the wave's stack area (2 W words per level,
// e + 1 levels), the deepest child set in the last slot.
// (Always inlined: called, as the compiler had it for 9 words, it reads the rows
// by flat loads, and 6-cliques of 5,000 vertices, out-degrees up to 692, took 50
// ms, not 44.)
template <int W, int S>
__device__ __forceinline__ uint64_t lgk_set(const uint64_t *rows, const uint64_t *set0, int32_t c,
                                            int32_t e, int16_t *mem, uint64_t *stack) {
    uint64_t acc = 0;
#pragma unroll
    for (int q = 0; q < W; q++) {
        const uint64_t x = uniform64(set0[q]);
        stack[q] = x;
        stack[W + q] = x;
    }
    wave_sync();
    int32_t lvl = 0;
    while (lvl >= 0) {
        uint64_t *set = stack + lvl * 2 * W, *rem = set + W;
        int32_t v = -1;
#pragma unroll
        for (int q = 0; q < W; q++) {
            const uint64_t r = uniform64(rem[q]);
            if (v < 0 && r) {
                v = q * 64 + __builtin_ctzll(r);
                rem[q] = r & (r - 1ull);
            }
        }
        wave_sync();
        if (v < 0) {
            lvl--;
            continue;
        }
        const uint64_t *rv = rows + v * S;
        uint64_t *child = stack + (lvl + 1) * 2 * W;
        int32_t cnt = 0;
#pragma unroll
        for (int q = 0; q < W; q++) {
            const uint64_t x = uniform64(set[q]) & uniform64(rv[q]);
            child[q] = x;
            child[W + q] = x;
            cnt += __popcll(x);
        }
        wave_sync();
        if (lvl + 1 == e) {
            if (cnt >= 3) acc += lg5_sweep<W, S>(rows, child, cnt, mem);
        } else if (cnt >= e - lvl + 2) {
            lvl++;
        }
    }
    return acc;
}

// Stride of a class's rows in LDS for W words: odd, so that a column of them is
// spread over the banks; but not for the descents above 512, where the room for
// more waves is worth more (6-cliques of 7,000 vertices, out-degrees up to 986:
// 260 ms with 8 waves, 213 with 10), nor up to 256, where they gain nothing by it
// (RMAT-16: 6-cliques 21.8 ms in this class, 20.4 without; 7-cliques 570 and 510;
// from 257 to 512 6.46 and 6.58 ms).
template <int DMAX> __host__ __device__ constexpr int32_t row_stride(int32_t W, bool deep) {
    return deep && DMAX != kHalfMaxD ? W : W | 1;
}

template <int WLO, int WHI, bool DEEP>
__device__ __forceinline__ uint64_t lg5_dispatch(int32_t W, const uint64_t *rows, const uint64_t *ri,
                                                 int32_t c, int32_t e, int16_t *mem,
                                                 uint64_t *stack) {
    if constexpr (WLO > WHI) {
        return 0;
    } else {
        constexpr int S = row_stride<WHI * kWave>(WLO, DEEP);
        if (W == WLO) {
            if constexpr (DEEP) return lgk_set<WLO, S>(rows, ri, c, e, mem, stack);
            else return lg5_tiles<WLO, S>(rows, ri, c, mem);
        }
        return lg5_dispatch<WLO + 1, WHI, DEEP>(W, rows, ri, c, e, mem, stack);
    }
}

template <int DMAX, bool LIST, bool DEEP>
__global__ void __launch_bounds__((Lg5Block<DMAX, !LIST && !DEEP>::kThreads),
                                  (Lg5Block<DMAX, !LIST && !DEEP>::kWaves))
    k_lg5(const int32_t *__restrict__ dag_off,
          const int32_t *__restrict__ roots,
          const LgTask *__restrict__ tasks,
          const uint32_t *__restrict__ ntasks_p,
          const int64_t *__restrict__ rowoff,
          const uint64_t *__restrict__ grows,
          int32_t rows_words, int32_t extra,
          unsigned long long *cursor, unsigned long long *result,
          RowEmitter em) {
    // row widths of the class: out-degrees (DMAX/2, DMAX]
    constexpr int WLO = DMAX / 128 + 1, WHI = DMAX / 64;
    extern __shared__ uint64_t dyn[];
    uint64_t *rows = dyn;
    __shared__ Lds<1024> sh;
    const int tid = threadIdx.x, lane = lane_id(), wib = tid / kWave;
    const int NT = blockDim.x;
    // then the out-neighbours in local order (listing), then per wave: member
    // list (DMAX int16) and the descent stack
    int32_t *verts = reinterpret_cast<int32_t *>(dyn + rows_words);
    uint8_t *wave_area = reinterpret_cast<uint8_t *>(verts + DMAX) +
                         (size_t)wib * (DMAX * 2 + (size_t)(extra + 1) * 2 * (DMAX / 64) * 8);
    int16_t *mem = reinterpret_cast<int16_t *>(wave_area);
    uint64_t *stack = reinterpret_cast<uint64_t *>(wave_area + DMAX * 2);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    TaskQueue queue(cursor, *ntasks_p, blockIdx.x, gridDim.x);
    uint64_t acc = 0;
    for (;;) {
        if (wave == 0) {
            const int32_t got = (int32_t)queue.next();
            if (tid == 0) sh.s_task = got;
        }
        __syncthreads();
        const int32_t t = sh.s_task;
        __syncthreads();
        if (t < 0) break;
        const LgTask T = tasks[DMAX == kHalfMaxD ? t : -1 - t];
        const int32_t r = T.r, slice = T.slice, S = T.slices;
        const int32_t u = roots[r];
        const int32_t d = dag_off[u + 1] - dag_off[u], W = (d + 63) >> 6;
        const uint64_t *src = grows + rowoff[r];
        const int32_t S64 = row_stride<DMAX>(W, DEEP);
        // the words tid, tid + NT, ..., four in flight (a row per wave at a time
        // waited for memory once a row: 5-cliques of 20,000 vertices, out-degrees
        // up to 893, took 20.1 ms, now 16.3)
        {
            constexpr int U = 4;
            const int32_t words = d * W, dr = NT / W, dc = NT - dr * W;
            int32_t row = tid / W, col = tid - row * W;
            for (int32_t i0 = tid; i0 < words; i0 += U * NT) {
                uint64_t x[U];
#pragma unroll
                for (int q = 0; q < U; q++) x[q] = i0 + q * NT < words ? src[i0 + q * NT] : 0ull;
#pragma unroll
                for (int q = 0; q < U; q++) {
                    if (i0 + q * NT < words) rows[row * S64 + col] = x[q];
                    row += dr;
                    col += dc;
                    if (col >= W) {
                        col -= W;
                        row++;
                    }
                }
            }
        }
        if (LIST) {
            const int32_t *sv = reinterpret_cast<const int32_t *>(src + d * W);
            for (int32_t i = tid; i < d; i += NT) verts[i] = sv[i];
        }
        if (tid == 0) sh.s_next = 0;
        __syncthreads();
        // waves take the slice's local vertices i = slice + S * c
        for (;;) {
            uint32_t c = 0;
            if (lane == 0) c = atomicAdd(&sh.s_next, 1u);
            c = __shfl(c, 0, 64);
            const int32_t i = slice + S * (int32_t)c;
            if (i >= d) break;
            const uint64_t *ri = rows + i * S64;
            int32_t cnt = 0;
            for (int32_t w = 0; w < W; w++) cnt += __popcll(ri[w]);
            if (cnt < 3 + extra) continue;
            if constexpr (LIST && DMAX > kHalfMaxD)
                lg5_list_wide(rows, S64, W, ri, cnt, mem, verts, u, verts[i], em);
            else if constexpr (LIST)
                lg5_list_dispatch<WLO, WHI>(W, rows, ri, cnt, mem, verts, u, verts[i], em);
            else
                acc += lg5_dispatch<WLO, WHI, DEEP>(W, rows, ri, cnt, extra, mem, stack);
        }
        __syncthreads();
    }
    if (LIST) {
        row_emitter_flush(em, result);
        return;
    }
    acc = wave_sum(acc);
    if (lane == 0 && acc) atomicAdd(result, (unsigned long long)acc);
}

// k >= 5 for roots of out-degree 65..256, build and count in one kernel: a
// workgroup builds the root's local graph in LDS (degree order), adds its
// local edges (triangles at u) to res3 and its local triangles (4-cliques at
// u) to res4 when asked, then its waves take the level-1 vertices and count
// (or list) as k_lg5 does.  The local graphs are small, so no slicing and no
// trip through HBM.
template <int DMAX, int NT, bool LIST, bool DEEP>
__global__ void __launch_bounds__(NT, DEEP ? 7 : kMidWaves) k_lg5_mid(const int32_t *__restrict__ off,
                                                const int32_t *__restrict__ okey,
                                                const int32_t *__restrict__ dag_off,
                                                const int32_t *__restrict__ dag_adj,
                                                const int32_t *__restrict__ roots,
                                                const int32_t *__restrict__ nroots_p,
                                                int32_t extra, unsigned long long *cursor,
                                                unsigned long long *result,
                                                unsigned long long *res3,
                                                unsigned long long *res4, RowEmitter em) {
    constexpr int NW = NT / kWave;
    constexpr int WMAX = DMAX / 64;
    constexpr int WLO = 2, WHI = WMAX;   // out-degrees 65..DMAX
    constexpr int kMaxExtra = 4;         // k <= 9
    __shared__ uint64_t rows[LgRows<DMAX>::kWords];
    __shared__ __align__(16) int32_t keys[LgHash<DMAX>::kSlots];
    __shared__ int16_t vals[LgHash<DMAX>::kSlots];
    __shared__ int16_t lidx[DMAX];
    __shared__ int32_t offj[DMAX], pre[DMAX + 1];
    __shared__ int32_t verts[DMAX];
    __shared__ int16_t s_mem[NW][DMAX];
    __shared__ uint64_t s_stack[NW][(kMaxExtra + 1) * 2 * WMAX];
    __shared__ Lds<NT> sh;
    const int tid = threadIdx.x, lane = lane_id(), wib = tid / kWave;
    const int32_t nroots = *nroots_p;
    uint64_t acc = 0, acc3 = 0, acc4 = 0;
    for (;;) {
        // (one counter: a root takes about 2 us of a workgroup, and with
        // spread cursors the kernel took 6.2 ms instead of 5.8 on RMAT-20)
        if (tid == 0) sh.s_task = (int32_t)atomicAdd(cursor, 1ull);
        __syncthreads();
        const int32_t r = sh.s_task;
        __syncthreads();
        if (r >= nroots) break;
        const int32_t u = roots[r];
        const int32_t d = dag_off[u + 1] - dag_off[u], W = (d + 63) >> 6;
        const int32_t S = row_stride<DMAX>(W, DEEP);
        build_rows<DMAX, NT, true>(off, okey, dag_off, dag_adj, u, d, S, rows, keys, vals, pre, offj,
                                   lidx, sh.s_sum, verts);
        if (res3 || res4) {
            const int32_t ne = row_prefix<DMAX, NT>(rows, d, W, S, pre, sh.s_sum);
            if (tid == 0) acc3 += ne;
            if (res4 && ne) acc4 += local_tri(rows, d, W, S, wib, NW);
        }
        for (int32_t i = wib; i < d; i += NW) {
            const uint64_t *ri = rows + i * S;
            int32_t cnt = 0;
            for (int32_t w = 0; w < W; w++) cnt += __popcll(ri[w]);
            if (cnt < 3 + extra) continue;
            if constexpr (LIST)
                lg5_list_dispatch<WLO, WHI>(W, rows, ri, cnt, s_mem[wib], verts, u, verts[i], em);
            else
                acc += lg5_dispatch<WLO, WHI, DEEP>(W, rows, ri, cnt, extra, s_mem[wib],
                                                           s_stack[wib]);
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
    if (res4) {
        acc4 = wave_sum(acc4);
        if (lane == 0 && acc4) atomicAdd(res4, (unsigned long long)acc4);
    }
}

struct LgWs {
    unsigned long long *cursor(int i) const {
        return reinterpret_cast<unsigned long long *>(ctl + 64 + i * kCursorWords);
    }
    uint32_t *ctl;                 // [8..9] 5-clique tasks of the two classes, from 64 the sets of cursors
    unsigned long long *units;     // local triangles (5-cliques' work)
    LgTask *tasks, *tasks_end;
    uint64_t *rows_b;
    uint64_t bytes;
};

LgWs lg_layout(const gpm_graph *g, int32_t k, void *base) {
    LgWs L{};
    Carve c(base, ~0ull);
    // the front of the workspace, zero on entry (kLgCtlWords)
    L.ctl = c.take<uint32_t>(kLgCtlWords);
    L.units = reinterpret_cast<unsigned long long *>(L.ctl + 16);
    if (k >= 5) {
        const uint64_t m = (uint64_t)std::max<int64_t>(g->m, 1);
        // at most d / 8 + 1 tasks per root of out-degree d > 256
        // (those of the smaller class from the front, the larger from the end)
        const uint64_t most = m / 8 + m / (kMidMaxD + 1) + 1;
        L.tasks = c.take<LgTask>(most);
        L.tasks_end = L.tasks + most;
        // rows and vertex ids of all roots with out-degree in (256, 1024]: sum of
        // d * ceil(d / 64) + ceil(d / 2) <= m * (ceil(max_out / 64) + 1) words
        const uint64_t wmax = (uint64_t)(std::max(g->max_out_degree, 1) + 63) / 64 + 1;
        const uint64_t words = m * wmax + (uint64_t)g->n;
        L.rows_b = c.take<uint64_t>(words);
    }
    L.bytes = c.used;
    return L;
}

// A persistent grid over the roots of out-degree above dmin: no more
// workgroups than the graph can have such roots (each takes dmin + 1 arcs).
dim3 roots_grid(const gpm_graph *g, int32_t dmin, int blocks_per_cu) {
    const int64_t most = std::min<int64_t>(g->n, g->m / (dmin + 1));
    return dim3((unsigned)std::max<int64_t>(
        1, std::min<int64_t>(most, (int64_t)cu_count() * blocks_per_cu)));
}

// 5-cliques and larger at the big class's roots; nothing is launched when no
// root can be in it.
gpm_status lg5_big(const gpm_graph *g, int32_t k, LgWs &L, const int32_t *list, const int32_t *cnt,
                   const int64_t *rowoff, unsigned long long *res, unsigned long long *res3,
                   unsigned long long *res4, const RowEmitter *em, hipStream_t st) {
    if (g->max_out_degree <= kMidMaxD) return GPM_OK;
    const uint64_t slice5 = (uint64_t)g->lg5_slice;
    uint32_t *ntasks = L.ctl + 8;
    {
        // roots of out-degree up to kHalfMaxD at the smaller bound
        Span sp("k_lg_build<512>", st);
        hipLaunchKernelGGL((k_lg_build<kHalfMaxD, kHalfThreads>),
                           roots_grid(g, kMidMaxD, kHalfBlocksPerCu), dim3(kHalfThreads), 0, st,
                           g->off, g->okey, g->dag_off, g->dag_adj, list, cnt, kMidMaxD,
                           L.cursor(4), rowoff, L.rows_b, L.tasks, ntasks, L.units, res3, res4,
                           slice5);
    }
    GPM_LAUNCH_CHECK("k_lg_build<512>");
    if (g->max_out_degree > kHalfMaxD) {
        Span sp("k_lg_build<1024>", st);
        hipLaunchKernelGGL((k_lg_build<kBigMaxD, kBigThreads>), roots_grid(g, kHalfMaxD, 1),
                           dim3(kBigThreads), 0, st, g->off, g->okey, g->dag_off, g->dag_adj, list,
                           cnt, kHalfMaxD, L.cursor(2), rowoff, L.rows_b, L.tasks_end, ntasks + 1, L.units,
                           res3, res4, slice5);
    }
    GPM_LAUNCH_CHECK("k_lg_build<1024>");
    // step 2, a class at a time.  LDS: rows of the class's largest local graph,
    // the local vertex ids, then per-wave areas, for as many waves as fit
    auto count = [&](auto dmax_class, int cursor, const LgTask *tasks, const uint32_t *nt) -> gpm_status {
        constexpr int DMAX = decltype(dmax_class)::value;
        const int32_t dmax = std::min<int32_t>(DMAX, g->max_out_degree);
        const int32_t extra = k - 5;
        const int32_t rows_words = dmax * row_stride<DMAX>((dmax + 63) / 64, extra > 0);
        const int64_t lds_cap = 160 * 1024 - 1024;
        const int64_t per_wave = (int64_t)DMAX * 2 + (int64_t)(extra + 1) * 2 * (DMAX / 64) * 8;
        const int64_t fixed = (int64_t)rows_words * 8 + (int64_t)DMAX * 4;
        const int threads = em || extra ? Lg5Block<DMAX, false>::kThreads : Lg5Block<DMAX, true>::kThreads;
        int waves = (int)std::min<int64_t>(threads / kWave, (lds_cap - fixed) / per_wave);
        if (waves < 1) return fail(GPM_DEVICE_ERROR, "local graph does not fit in LDS");
        const size_t shmem = (size_t)fixed + (size_t)waves * per_wave;
        const dim3 grid((unsigned)cu_count() *
                        (em || extra ? Lg5Block<DMAX, false>::kPerCu : Lg5Block<DMAX, true>::kPerCu));
        if (em)
            hipLaunchKernelGGL((k_lg5<DMAX, true, false>), grid, dim3(waves * kWave), shmem, st,
                               g->dag_off, list, tasks, nt, rowoff, (const uint64_t *)L.rows_b,
                               rows_words, extra, L.cursor(cursor), res, *em);
        else
            hipLaunchKernelGGL(extra ? (k_lg5<DMAX, false, true>) : (k_lg5<DMAX, false, false>), grid,
                               dim3(waves * kWave), shmem, st, g->dag_off, list, tasks, nt, rowoff,
                               (const uint64_t *)L.rows_b, rows_words, extra, L.cursor(cursor), res,
                               RowEmitter{});
        return GPM_OK;
    };
    Span sp(k == 5 ? "k_lg5<1024>" : "k_lgk<1024>", st);
    if (g->max_out_degree > kHalfMaxD) {
        gpm_status rc = count(std::integral_constant<int, kBigMaxD>(), 3, L.tasks_end, ntasks + 1);
        if (rc) return rc;
    }
    gpm_status rc = count(std::integral_constant<int, kHalfMaxD>(), 5, L.tasks, ntasks);
    if (rc) return rc;
    span_units(L.units, st);
    GPM_LAUNCH_CHECK("k_lg5");
    return GPM_OK;
}

}  // namespace

gpm_status lg_workspace_bytes(const gpm_graph *g, int32_t k, uint64_t *bytes) {
    *bytes = lg_layout(g, k, nullptr).bytes;
    return GPM_OK;
}

// Counts k-cliques (k = 4..9) rooted at the two workgroup classes: list_m
// (out-degree 65..256) and list_b (257..1024), device counts cnt_m, cnt_b,
// into *res.  res3 / res4 (may be null) also receive the triangles and (for
// k = 5) the 4-cliques rooted at the same roots.  rowoff_b (k >= 5): where
// each root of list_b stores its rows.  The workspace's first kLgCtlWords
// words are zero on entry.  A class that no root of the graph can be in is
// not launched.
gpm_status lg_cliques(const gpm_graph *g, int32_t k, const int32_t *list_m, const int32_t *cnt_m,
                      const int32_t *list_b, const int32_t *cnt_b, const int64_t *rowoff_b,
                      void *ws, uint64_t ws_bytes, unsigned long long *res,
                      unsigned long long *res3, unsigned long long *res4, const RowEmitter *em,
                      hipStream_t st) {
    LgWs L = lg_layout(g, k, ws);
    if (L.bytes > ws_bytes) return fail(GPM_OUT_OF_MEMORY, "local-graph workspace too small");
    if (k == 4) {
        const RowEmitter none{};
        if (g->max_out_degree > kHalfMaxD) {
            Span sp("k_lg4<1024>", st);
            const dim3 grid = roots_grid(g, kHalfMaxD, 1);
            if (em)
                hipLaunchKernelGGL((k_lg4<kBigMaxD, kBigThreads, true, true>), grid,
                                   dim3(kBigThreads), 0, st, g->off, g->okey, g->dag_off,
                                   g->dag_adj, list_b, cnt_b, kHalfMaxD, L.cursor(0), res, res3, *em);
            else
                hipLaunchKernelGGL((k_lg4<kBigMaxD, kBigThreads, false, true>), grid,
                                   dim3(kBigThreads), 0, st, g->off, g->okey, g->dag_off,
                                   g->dag_adj, list_b, cnt_b, kHalfMaxD, L.cursor(0), res, res3,
                                   none);
        }
        GPM_LAUNCH_CHECK("k_lg4<1024>");
        if (g->max_out_degree > kMidMaxD) {
            Span sp("k_lg4<512>", st);
            const dim3 grid = roots_grid(g, kMidMaxD, kHalfBlocksPerCu);
            if (em)
                hipLaunchKernelGGL((k_lg4<kHalfMaxD, kHalfThreads, true, true>), grid,
                                   dim3(kHalfThreads), 0, st, g->off, g->okey, g->dag_off, g->dag_adj,
                                   list_b, cnt_b, kMidMaxD, L.cursor(2), res, res3, *em);
            else
                hipLaunchKernelGGL((k_lg4<kHalfMaxD, kHalfThreads, false, true>), grid,
                                   dim3(kHalfThreads), 0, st, g->off, g->okey, g->dag_off, g->dag_adj,
                                   list_b, cnt_b, kMidMaxD, L.cursor(2), res, res3, none);
        }
        GPM_LAUNCH_CHECK("k_lg4<512>");
        if (g->max_out_degree > kWave) {
            Span sp("k_lg4<256>", st);
            const dim3 grid = roots_grid(g, kWave, 8);
            if (em)
                hipLaunchKernelGGL((k_lg4<kMidMaxD, kMidThreads, true, false>), grid,
                                   dim3(kMidThreads), 0, st, g->off, g->okey, g->dag_off, g->dag_adj,
                                   list_m, cnt_m, 0, L.cursor(1), res, res3, *em);
            else
                hipLaunchKernelGGL((k_lg4<kMidMaxD, kMidThreads, false, true>), grid,
                                   dim3(kMidThreads), 0, st, g->off, g->okey, g->dag_off, g->dag_adj,
                                   list_m, cnt_m, 0, L.cursor(1), res, res3, none);
        }
        GPM_LAUNCH_CHECK("k_lg4<256>");
        return GPM_OK;
    }
    gpm_status rc = lg5_big(g, k, L, list_b, cnt_b, rowoff_b, res, res3, res4, em, st);
    if (rc) return rc;
    if (g->max_out_degree > kWave) {
        Span sp(k == 5 ? "k_lg5_mid<256>" : "k_lgk_mid<256>", st);
        const dim3 grid = roots_grid(g, kWave, 8);
        if (em)
            hipLaunchKernelGGL((k_lg5_mid<kMidMaxD, kMidThreads, true, false>), grid, dim3(kMidThreads), 0,
                               st, g->off, g->okey, g->dag_off, g->dag_adj, list_m, cnt_m, k - 5,
                               L.cursor(6), res, res3, res4, *em);
        else
            hipLaunchKernelGGL(k > 5 ? (k_lg5_mid<kMidMaxD, kMidThreads, false, true>)
                                     : (k_lg5_mid<kMidMaxD, kMidThreads, false, false>),
                               grid, dim3(kMidThreads), 0, st, g->off, g->okey, g->dag_off,
                               g->dag_adj, list_m, cnt_m, k - 5, L.cursor(6), res, res3, res4,
                               RowEmitter{});
    }
    GPM_LAUNCH_CHECK("k_lg5_mid");
    return GPM_OK;
}

}  // namespace gpm
