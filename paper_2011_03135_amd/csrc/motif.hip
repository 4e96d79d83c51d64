// Induced 3- and 4-motif counting by local counting (Section 5: the wedge
// equation and the diamond count from per-edge triangle counts; Appendix A:
// the 3-motif and 4-motif local-counting listings, whose elided final step is
// completed here with per-edge identities).
//
// 3-motifs: wedges (open) = sum_v C(d_v, 2) - 3T, triangles = T.
//
// 4-motifs.  For every undirected edge e = (u, v) with T_e triangles,
// S_u = d_u - T_e - 1 and S_v = d_v - T_e - 1 (the local wedge terms of the
// wedge equation), these sums over edges, each edge visited once, equal
// induced counts (I_*):
//   sum C(T_e, 2)                  = I_diamond + 6 I_K4
//   sum T_e (S_u + S_v)            = 2 I_paw + 4 I_diamond
//   sum S_u S_v                    = I_P4 + 4 I_C4
//   sum C(S_u, 2) + C(S_v, 2)      = 3 I_claw + I_paw
// With I_K4 from 4-clique counting and the number of 4-cycles N_C4 (not
// necessarily induced; N_C4 = I_C4 + I_diamond + 3 I_K4) the system solves
// exactly; every division is checked.
//
// N_C4 comes from the 4-cycle counter (c4.hip).
#include "gpm_internal.h"

#include <algorithm>
#include <climits>

namespace gpm {

gpm_status clique_workspace_bytes(const gpm_graph *g, int32_t k, bool list, uint64_t *bytes);
gpm_status clique_run(const gpm_graph *g, int32_t k, bool list, void *ws, uint64_t ws_bytes,
                      unsigned long long *d_count, int32_t *d_buf, uint64_t cap,
                      unsigned long long *d_result, hipStream_t st);
gpm_status triangle_arc_counts(const gpm_graph *g, void *ws, uint64_t ws_bytes, uint32_t *te,
                               unsigned long long *tri, hipStream_t st, WordRun also);
gpm_status c4_workspace_bytes(const gpm_graph *g, bool list, uint64_t *bytes);
gpm_status c4_run(const gpm_graph *g, bool list, void *ws, uint64_t ws_bytes,
                  unsigned long long *out128, int32_t *d_buf, uint64_t cap,
                  unsigned long long *d_result, hipStream_t st,
                  const uint32_t *tsym = nullptr, unsigned long long *cs = nullptr);

namespace {

typedef unsigned __int128 u128;

constexpr int kBlock = 256;

constexpr int kSumBlocks = 1024;   // workgroups of the summing kernels at most

// Adds up N 128-bit values per thread over the workgroup; thread q < N
// writes the q-th total to out[2 q], out[2 q + 1].  One store per workgroup:
// added to one word by an atomic per wave, the four sums of RMAT-18 took
// 0.32 ms, nearly all of it the atomics' queue.
template <int N>
__device__ void block_sums(const u128 (&s)[N], unsigned long long *out) {
    __shared__ u128 sh[kBlock / kWave][N];
#pragma unroll
    for (int q = 0; q < N; q++) {
        const u128 t = wave_sum_u128(s[q]);
        if (lane_id() == 0) sh[threadIdx.x / kWave][q] = t;
    }
    __syncthreads();
    if (threadIdx.x < N) {
        u128 t = 0;
        for (int w = 0; w < kBlock / kWave; w++) t += sh[w][threadIdx.x];
        out[2 * threadIdx.x] = (unsigned long long)t;
        out[2 * threadIdx.x + 1] = (unsigned long long)(t >> 64);
    }
}

// Each workgroup's share of sum_v C(d_v, 2); the degrees too when asked for.
__global__ void __launch_bounds__(kBlock) k_wedge_sum(const int32_t *__restrict__ off, int32_t n,
                                                      int32_t *deg, unsigned long long *part) {
    u128 s[1] = {0};
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * kBlock) {
        const int32_t dv = off[i + 1] - off[i];
        if (deg) deg[i] = dv;
        const uint64_t d = (uint64_t)dv;
        s[0] += (u128)(d * (d - (d > 0)) / 2);
    }
    block_sums<1>(s, part + 2 * blockIdx.x);
}

// Each workgroup's share of the four per-edge local-count sums.
__global__ void __launch_bounds__(kBlock) k_lc_sums(const int32_t *__restrict__ dag_src,
                                                    const int32_t *__restrict__ dag_adj,
                                                    const uint32_t *__restrict__ te,
                                                    const int32_t *__restrict__ deg, int64_t m,
                                                    unsigned long long *part) {
    int64_t e = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    int64_t stride = (int64_t)gridDim.x * kBlock;
    u128 s[4] = {0, 0, 0, 0};
    for (; e < m; e += stride) {
        const uint64_t t = te[e];
        const uint64_t du = (uint64_t)deg[dag_src[e]], dv = (uint64_t)deg[dag_adj[e]];
        const uint64_t su = du - t - 1, sv = dv - t - 1;
        s[0] += (u128)(t * (t - (t > 0)) / 2);
        s[1] += (u128)t * (su + sv);
        s[2] += (u128)su * sv;
        s[3] += (u128)(su * (su - (su > 0)) / 2) + (u128)(sv * (sv - (sv > 0)) / 2);
    }
    block_sums<4>(s, part + 8 * blockIdx.x);
}

// ------------------------------------------------------------- combine ---

struct Sums {
    unsigned long long tri;        // T (triangles)
    unsigned long long k4;         // 4-cliques
    unsigned long long c4[2];      // N_C4
};

__device__ __forceinline__ u128 get128(const unsigned long long *p) {
    return ((u128)p[1] << 64) | p[0];
}

// Total of `blocks` workgroups' shares of N sums.
template <int N>
__device__ void add_parts(const unsigned long long *part, int32_t blocks, u128 (&s)[N]) {
    __shared__ unsigned long long sh[2 * N];
#pragma unroll
    for (int q = 0; q < N; q++) s[q] = 0;
    for (int32_t b = threadIdx.x; b < blocks; b += kBlock)
#pragma unroll
        for (int q = 0; q < N; q++) s[q] += get128(part + 2 * (N * (int64_t)b + q));
    block_sums<N>(s, sh);
    __syncthreads();
#pragma unroll
    for (int q = 0; q < N; q++) s[q] = get128(sh + 2 * q);
}

// One workgroup.
__global__ void __launch_bounds__(kBlock) k_combine(const Sums *S,
                                                    const unsigned long long *wedge,
                                                    int32_t wedge_blocks,
                                                    const unsigned long long *lc,
                                                    int32_t lc_blocks, int32_t k,
                                                    unsigned long long *out) {
    const u128 lim = (u128)1 << 64;
    unsigned long long bad = 0;
    if (k == 3) {
        u128 ws[1];
        add_parts<1>(wedge, wedge_blocks, ws);
        if (threadIdx.x != 0) return;
        const u128 w = ws[0], t3 = (u128)3 * S->tri;
        if (w < t3) bad |= 1;
        const u128 wo = w - t3;
        if (wo >= lim) bad |= 2;
        out[0] = (unsigned long long)wo;
        out[1] = S->tri;
        out[2] = bad;
        return;
    }
    u128 ls[4];
    add_parts<4>(lc, lc_blocks, ls);
    if (threadIdx.x != 0) return;
    const u128 k4 = S->k4;
    const u128 s1 = ls[0], s2 = ls[1], s3 = ls[2], s4 = ls[3], nc4 = get128(S->c4);
    u128 dia = 0, paw = 0, c4 = 0, p4 = 0, claw = 0;
    if (s1 < 6 * k4) bad |= 1; else dia = s1 - 6 * k4;
    if (s2 < 4 * dia || ((s2 - 4 * dia) & 1)) bad |= 2; else paw = (s2 - 4 * dia) / 2;
    if (nc4 < dia + 3 * k4) bad |= 4; else c4 = nc4 - dia - 3 * k4;
    if (s3 < 4 * c4) bad |= 8; else p4 = s3 - 4 * c4;
    if (s4 < paw || (s4 - paw) % 3) bad |= 16; else claw = (s4 - paw) / 3;
    const u128 r[6] = {claw, p4, c4, paw, dia, k4};
    for (int i = 0; i < 6; i++) {
        if (r[i] >= lim) bad |= 32;
        out[i] = (unsigned long long)r[i];
    }
    out[6] = bad;
}

struct MotifWs {
    Sums *sums;
    unsigned long long *part;   // workgroups' shares of the wedge or local-count sums
    uint32_t *te;
    int32_t *deg;
    void *shared;      // clique workspace (k = 3 or 4), reused in sequence
    void *c4ws;        // 4-cycle counting workspace
    uint64_t shared_bytes, c4_bytes, bytes;
};

MotifWs motif_layout(const gpm_graph *g, int32_t k, void *base) {
    MotifWs W{};
    Carve c(base, ~0ull);
    const uint64_t n1 = (uint64_t)g->n + 1;
    W.sums = c.take<Sums>(1);
    W.part = c.take<unsigned long long>((k == 4 ? 8 : 2) * kSumBlocks);
    if (k == 4) {
        W.deg = c.take<int32_t>(n1);
        W.te = c.take<uint32_t>((uint64_t)std::max<int64_t>(g->m, 1));
        c4_workspace_bytes(g, false, &W.c4_bytes);
        W.c4ws = c.take<char>(W.c4_bytes);
    }
    uint64_t b3 = 0, b4 = 0;
    clique_workspace_bytes(g, 3, false, &b3);
    if (k == 4) clique_workspace_bytes(g, 4, false, &b4);
    W.shared_bytes = std::max(b3, b4);
    W.shared = c.take<char>(W.shared_bytes);
    W.bytes = c.used;
    return W;
}

unsigned grid_for(int64_t items, int per_block, int cap_per_cu) {
    int64_t b = (items + per_block - 1) / per_block;
    int64_t cap = (int64_t)cu_count() * cap_per_cu;
    return (unsigned)std::max<int64_t>(1, std::min<int64_t>(b, cap));
}

}  // namespace

gpm_status motif_workspace_bytes(const gpm_graph *g, int32_t k, uint64_t *bytes) {
    *bytes = motif_layout(g, k, nullptr).bytes;
    return GPM_OK;
}

gpm_status motif_run(const gpm_graph *g, int32_t k, void *ws, uint64_t ws_bytes,
                     unsigned long long *d_counts, hipStream_t st) {
    MotifWs W = motif_layout(g, k, ws);
    if (W.bytes > ws_bytes) return fail(GPM_OUT_OF_MEMORY, "workspace smaller than required");
    const int32_t n = g->n;
    const unsigned vb = std::min<unsigned>(grid_for(n, kBlock, 4), kSumBlocks);
    const unsigned eb = std::min<unsigned>(grid_for(g->m, kBlock, 4), kSumBlocks);
    gpm_status rc;
    if (k == 3) {
        hipLaunchKernelGGL(k_wedge_sum, dim3(vb), dim3(kBlock), 0, st, g->off, n, nullptr, W.part);
        GPM_LAUNCH_CHECK("k_wedge_sum");
        rc = clique_run(g, 3, false, W.shared, W.shared_bytes, &W.sums->tri, nullptr, 0, nullptr,
                        st);
        if (rc) return rc;
    } else {
        rc = triangle_arc_counts(g, W.shared, W.shared_bytes, W.te, &W.sums->tri, st,
                                 {W.sums, sizeof(Sums) / 4});
        if (rc) return rc;
        // the degrees; their wedges (here a by-product) are overwritten next
        hipLaunchKernelGGL(k_wedge_sum, dim3(vb), dim3(kBlock), 0, st, g->off, n, W.deg, W.part);
        GPM_LAUNCH_CHECK("k_wedge_sum");
        hipLaunchKernelGGL(k_lc_sums, dim3(eb), dim3(kBlock), 0, st, g->dag_src, g->dag_adj, W.te,
                           W.deg, g->m, W.part);
        GPM_LAUNCH_CHECK("k_lc_sums");
        rc = clique_run(g, 4, false, W.shared, W.shared_bytes, &W.sums->k4, nullptr, 0, nullptr,
                        st);
        if (rc) return rc;
        rc = c4_run(g, false, W.c4ws, W.c4_bytes, W.sums->c4, nullptr, 0, nullptr, st);
        if (rc) return rc;
    }
    hipLaunchKernelGGL(k_combine, dim3(1), dim3(kBlock), 0, st, W.sums, W.part, (int32_t)vb,
                       W.part, (int32_t)eb, k, d_counts);
    GPM_LAUNCH_CHECK("k_combine");
    return GPM_OK;
}

}  // namespace gpm
