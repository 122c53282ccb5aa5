// Streaming edge primitives in full precision: SDDMM-add with on-the-fly
// dequantization + LeakyReLU (Sec. 2.1 step 3, Sec. 3.3), its backward with the
// edge-to-node sums (steps 3', 3''; Sec. 3.3 Fig. 5), edge softmax forward and
// backward (steps 4, 4'; Sec. 3.2 keeps them in fp32).
//
// All of them stream the destination-major edge arrays once or a few times; what bounds them is the chain of
// dependent loads of a row (codes of the other end through its index) rather than bandwidth.  Rows (nodes) are handed
// out in blocks of consecutive rows per wavefront; short rows are processed by groups of GROUP lanes (GROUP ~ the
// mean degree), rows longer than 16*GROUP by the whole wave and rows longer than LONG_ROW by a whole workgroup of the same
// launch, one lane per edge with all heads of that edge, four edges per lane in flight.  Without the last two a hub row
// of some thousand edges is one wave's chain of some hundred round trips: 50 K nodes, 2 M edges of a power-law graph,
// two heads: softmax 131 -> 39 us, its backward 91 -> 26, add 76 -> 26, its backward 96 -> 26 (dD) and 124 -> 52 (dS).
#include <algorithm>
#include <type_traits>

#include "internal.hip.h"
#include "attn_math.hip.h"
#include "rowwalk.hip.h"

namespace {

struct row_split {
    int long_blocks;    // workgroups below this one take the long rows
    int rows_per_wave;  // see walk_rows
    unsigned grid;
};

row_split split_rows(int n, int64_t nnz, int group)
{
    row_split r;
    r.rows_per_wave = pick_rows_per_wave(n, group);
    r.long_blocks = nnz > LONG_ROW ? static_cast<int>(std::min<int64_t>(HUGE_GRID, n)) : 0;  // (no row can be longer otherwise)
    r.grid = row_grid(n, group, r.rows_per_wave) + r.long_blocks;
    return r;
}

template <int GROUP, class Op>
__device__ inline void walk_all_rows(const int32_t *ptr, int n, Op &op, int long_blocks, int rows_per_wave)
{
    __shared__ double scratch[2 * 256 / 64];
    __shared__ int list[256 + 1];
    if (static_cast<int>(blockIdx.x) < long_blocks)
        walk_huge_rows_strided(ptr, n, static_cast<int>(blockIdx.x), long_blocks, op, scratch, list, LONG_ROW);
    else
        walk_rows<GROUP>(ptr, n, op, nullptr, long_blocks, long_blocks > 0, rows_per_wave, LONG_ROW);
}

// The codes of a node; whole: the table is aligned to H bytes (H 2, 4 or 8), one load.
template <int H>
__device__ inline void load_codes(const int8_t *table, int64_t node, bool whole, int (&v)[H])
{
    if (whole) {
        tango_load_heads<H>(table, node, v);
    } else {
#pragma unroll
        for (int h = 0; h < H; ++h) v[h] = static_cast<int>(table[node * H + h]);
    }
}

// body(e0, k): the edges e0, e0 + step, ... (k of them, 4 or 1, k a compile-time constant) of the range [e, t)
template <class Body>
__device__ inline void by_four(int e, int t, int step, Body body)
{
    for (; t - e > 3 * step; e += 4 * step) body(e, std::integral_constant<int, 4>{});
    for (; e < t; e += step) body(e, std::integral_constant<int, 1>{});
}

// ------------------------------------------------------------------ SDDMM-add
template <int H>
struct sddmm_add_op {
    const int32_t *src;
    const int8_t *Sq, *Dq;
    float sS, sD, slope;
    float *E;
    bool whole;
    template <class Team>
    __device__ void run(int row, int b, int t, Team tm)
    {
        float td[H];
#pragma unroll
        for (int h = 0; h < H; ++h) td[h] = sD * static_cast<float>(Dq[static_cast<int64_t>(row) * H + h]);
        by_four(b + tm.rank, t, tm.size(), [&](int e, auto K) __attribute__((always_inline)) {
            constexpr int N = decltype(K)::value;
            int sq[N][H];
            int u[N];
#pragma unroll
            for (int i = 0; i < N; ++i) u[i] = src[e + i * tm.size()];
#pragma unroll
            for (int i = 0; i < N; ++i) load_codes<H>(Sq, u[i], whole, sq[i]);
#pragma unroll
            for (int i = 0; i < N; ++i) {
                float v[H];
#pragma unroll
                for (int h = 0; h < H; ++h) {
                    const float ts = sS * static_cast<float>(sq[i][h]);
                    const float x = ts + td[h];
                    v[h] = x > 0.0f ? x : slope * x;
                }
                store_h<H>(E + static_cast<int64_t>(e + i * tm.size()) * H, v);
            }
        });
    }
};

template <int H, int GROUP>
__global__ __launch_bounds__(256) void k_sddmm_add(int n, const int32_t *ptr, sddmm_add_op<H> op, const float *sS,
                                                   const float *sD, int long_blocks, int rows_per_wave)
{
    op.sS = *sS;
    op.sD = *sD;
    walk_all_rows<GROUP>(ptr, n, op, long_blocks, rows_per_wave);
}

// dD[v][h] = sum over in-edges of dE*lrelu'(t); optional dE_pre.
template <int H>
struct sddmm_add_bwd_dst_op {
    const int32_t *src;
    const int8_t *Sq, *Dq;
    float sS, sD, slope;
    const float *dE;
    float *dEpre, *dD;
    bool whole;
    template <class Team>
    __device__ void run(int row, int b, int t, Team tm)
    {
        float td[H];
        double acc[H];
#pragma unroll
        for (int h = 0; h < H; ++h) {
            td[h] = sD * static_cast<float>(Dq[static_cast<int64_t>(row) * H + h]);
            acc[h] = 0.0;
        }
        by_four(b + tm.rank, t, tm.size(), [&](int e, auto K) __attribute__((always_inline)) {
            constexpr int N = decltype(K)::value;
            int sq[N][H];
            int u[N];
            float g[N][H];
#pragma unroll
            for (int i = 0; i < N; ++i) u[i] = src[e + i * tm.size()];
#pragma unroll
            for (int i = 0; i < N; ++i) load_h<H>(dE + static_cast<int64_t>(e + i * tm.size()) * H, g[i]);
#pragma unroll
            for (int i = 0; i < N; ++i) load_codes<H>(Sq, u[i], whole, sq[i]);
#pragma unroll
            for (int i = 0; i < N; ++i) {
#pragma unroll
                for (int h = 0; h < H; ++h) {
                    const float ts = sS * static_cast<float>(sq[i][h]);
                    const float x = ts + td[h];
                    g[i][h] = g[i][h] * (x > 0.0f ? 1.0f : slope);
                    acc[h] += static_cast<double>(g[i][h]);
                }
                if (dEpre) store_h<H>(dEpre + static_cast<int64_t>(e + i * tm.size()) * H, g[i]);
            }
        });
#pragma unroll
        for (int h = 0; h < H; ++h) {
            const double s = tm.sum(acc[h]);
            if (tm.rank == 0) dD[static_cast<int64_t>(row) * H + h] = static_cast<float>(s);
        }
    }
};

template <int H, int GROUP>
__global__ __launch_bounds__(256) void k_sddmm_add_bwd_dst(int n, const int32_t *ptr, sddmm_add_bwd_dst_op<H> op,
                                                           const float *sS, const float *sD, int long_blocks, int rows_per_wave)
{
    op.sS = *sS;
    op.sD = *sD;
    walk_all_rows<GROUP>(ptr, n, op, long_blocks, rows_per_wave);
}

// dS[u][h] = sum over out-edges of dE[eid]*lrelu'(t), t recomputed from S_q[u], D_q[dst].
template <int H>
struct sddmm_add_bwd_src_op {
    const int32_t *dst, *eid;
    const int8_t *Sq, *Dq;
    float sS, sD, slope;
    const float *dE;
    float *dS;
    bool whole;
    template <class Team>
    __device__ void run(int row, int b, int t, Team tm)
    {
        float ts[H];
        double acc[H];
#pragma unroll
        for (int h = 0; h < H; ++h) {
            ts[h] = sS * static_cast<float>(Sq[static_cast<int64_t>(row) * H + h]);
            acc[h] = 0.0;
        }
        by_four(b + tm.rank, t, tm.size(), [&](int j, auto K) __attribute__((always_inline)) {
            constexpr int N = decltype(K)::value;
            int dq[N][H];
            int v[N], e[N];
            float g[N][H];
#pragma unroll
            for (int i = 0; i < N; ++i) {
                v[i] = dst[j + i * tm.size()];
                e[i] = eid[j + i * tm.size()];
            }
#pragma unroll
            for (int i = 0; i < N; ++i) {
                load_h<H>(dE + static_cast<int64_t>(e[i]) * H, g[i]);
                load_codes<H>(Dq, v[i], whole, dq[i]);
            }
#pragma unroll
            for (int i = 0; i < N; ++i)
#pragma unroll
                for (int h = 0; h < H; ++h) {
                    const float tdv = sD * static_cast<float>(dq[i][h]);
                    const float x = ts[h] + tdv;
                    acc[h] += static_cast<double>(g[i][h] * (x > 0.0f ? 1.0f : slope));
                }
        });
#pragma unroll
        for (int h = 0; h < H; ++h) {
            const double s = tm.sum(acc[h]);
            if (tm.rank == 0) dS[static_cast<int64_t>(row) * H + h] = static_cast<float>(s);
        }
    }
};

template <int H, int GROUP>
__global__ __launch_bounds__(256) void k_sddmm_add_bwd_src(int n, const int32_t *ptr, sddmm_add_bwd_src_op<H> op,
                                                           const float *sS, const float *sD, int long_blocks, int rows_per_wave)
{
    op.sS = *sS;
    op.sD = *sD;
    walk_all_rows<GROUP>(ptr, n, op, long_blocks, rows_per_wave);
}

// ------------------------------------------------------------------ edge softmax
template <int H>
struct softmax_op {
    const float *E;
    float *alpha;
    float amax;
    template <class Team>
    __device__ void run(int /*row*/, int b, int t, Team tm)
    {
        float m[H], s[H];
#pragma unroll
        for (int h = 0; h < H; ++h) {
            m[h] = -INFINITY;
            s[h] = 0.0f;
        }
        constexpr int UE = H >= 8 ? 2 : 4;
        if (t - b <= UE * tm.size()) {  // the row fits the team's registers: one pass over memory
            float v[UE][H];
#pragma unroll
            for (int i = 0; i < UE; ++i) {
#pragma unroll
                for (int h = 0; h < H; ++h) v[i][h] = -INFINITY;
                const int e = b + tm.rank + i * tm.size();
                if (e < t) load_h<H>(E + static_cast<int64_t>(e) * H, v[i]);
            }
#pragma unroll
            for (int h = 0; h < H; ++h) {
#pragma unroll
                for (int i = 0; i < UE; ++i) m[h] = fmaxf(m[h], v[i][h]);
                m[h] = tm.max(m[h]);
            }
#pragma unroll
            for (int i = 0; i < UE; ++i)
                if (b + tm.rank + i * tm.size() < t) {
#pragma unroll
                    for (int h = 0; h < H; ++h) {
                        v[i][h] = expf(v[i][h] - m[h]);
                        s[h] += v[i][h];
                    }
                }
#pragma unroll
            for (int h = 0; h < H; ++h) s[h] = tm.sum(s[h]);
#pragma unroll
            for (int i = 0; i < UE; ++i) {
                const int e = b + tm.rank + i * tm.size();
                if (e >= t) continue;
#pragma unroll
                for (int h = 0; h < H; ++h) {
                    v[i][h] = v[i][h] / s[h];
                    amax = fmaxf(amax, v[i][h]);
                }
                store_h<H>(alpha + static_cast<int64_t>(e) * H, v[i]);
            }
            return;
        }
        by_four(b + tm.rank, t, tm.size(), [&](int e, auto K) __attribute__((always_inline)) {
            constexpr int N = decltype(K)::value;
            float v[N][H];
#pragma unroll
            for (int i = 0; i < N; ++i) load_h<H>(E + static_cast<int64_t>(e + i * tm.size()) * H, v[i]);
#pragma unroll
            for (int i = 0; i < N; ++i)
#pragma unroll
                for (int h = 0; h < H; ++h) m[h] = fmaxf(m[h], v[i][h]);
        });
#pragma unroll
        for (int h = 0; h < H; ++h) m[h] = tm.max(m[h]);
        by_four(b + tm.rank, t, tm.size(), [&](int e, auto K) __attribute__((always_inline)) {
            constexpr int N = decltype(K)::value;
            float v[N][H];
#pragma unroll
            for (int i = 0; i < N; ++i) load_h<H>(E + static_cast<int64_t>(e + i * tm.size()) * H, v[i]);
#pragma unroll
            for (int i = 0; i < N; ++i)
#pragma unroll
                for (int h = 0; h < H; ++h) s[h] += expf(v[i][h] - m[h]);
        });
#pragma unroll
        for (int h = 0; h < H; ++h) s[h] = tm.sum(s[h]);
        by_four(b + tm.rank, t, tm.size(), [&](int e, auto K) __attribute__((always_inline)) {
            constexpr int N = decltype(K)::value;
            float v[N][H];
#pragma unroll
            for (int i = 0; i < N; ++i) load_h<H>(E + static_cast<int64_t>(e + i * tm.size()) * H, v[i]);
#pragma unroll
            for (int i = 0; i < N; ++i) {
#pragma unroll
                for (int h = 0; h < H; ++h) {
                    v[i][h] = expf(v[i][h] - m[h]) / s[h];
                    amax = fmaxf(amax, v[i][h]);
                }
                store_h<H>(alpha + static_cast<int64_t>(e + i * tm.size()) * H, v[i]);
            }
        });
    }
};

template <int H, int GROUP>
__global__ __launch_bounds__(256) void k_edge_softmax(int n, const int32_t *ptr, softmax_op<H> op, float *absmax, int long_blocks,
                                                      int rows_per_wave)
{
    op.amax = 0.0f;
    walk_all_rows<GROUP>(ptr, n, op, long_blocks, rows_per_wave);
    if (absmax) tango_block_max_update(op.amax, absmax);
}

template <int H>
struct softmax_bwd_op {
    const float *alpha, *dalpha;
    float *dE;
    template <class Team>
    __device__ void run(int /*row*/, int b, int t, Team tm)
    {
        double P[H];
#pragma unroll
        for (int h = 0; h < H; ++h) P[h] = 0.0;
        constexpr int UE = H >= 8 ? 1 : 4;
        if (t - b <= UE * tm.size()) {  // the row fits the team's registers
            float a[UE][H], d[UE][H];
#pragma unroll
            for (int i = 0; i < UE; ++i) {
                const int e = b + tm.rank + i * tm.size();
#pragma unroll
                for (int h = 0; h < H; ++h) a[i][h] = d[i][h] = 0.0f;
                if (e < t) {
                    load_h<H>(alpha + static_cast<int64_t>(e) * H, a[i]);
                    load_h<H>(dalpha + static_cast<int64_t>(e) * H, d[i]);
                }
            }
#pragma unroll
            for (int h = 0; h < H; ++h) {
#pragma unroll
                for (int i = 0; i < UE; ++i) P[h] += static_cast<double>(d[i][h]) * static_cast<double>(a[i][h]);
                P[h] = tm.sum(P[h]);
            }
#pragma unroll
            for (int i = 0; i < UE; ++i) {
                const int e = b + tm.rank + i * tm.size();
                if (e >= t) continue;
                float o[H];
#pragma unroll
                for (int h = 0; h < H; ++h)
                    o[h] = static_cast<float>(static_cast<double>(a[i][h]) * (static_cast<double>(d[i][h]) - P[h]));
                store_h<H>(dE + static_cast<int64_t>(e) * H, o);
            }
            return;
        }
        by_four(b + tm.rank, t, tm.size(), [&](int e, auto K) __attribute__((always_inline)) {
            constexpr int N = decltype(K)::value;
            float a[N][H], d[N][H];
#pragma unroll
            for (int i = 0; i < N; ++i) {
                load_h<H>(alpha + static_cast<int64_t>(e + i * tm.size()) * H, a[i]);
                load_h<H>(dalpha + static_cast<int64_t>(e + i * tm.size()) * H, d[i]);
            }
#pragma unroll
            for (int i = 0; i < N; ++i)
#pragma unroll
                for (int h = 0; h < H; ++h) P[h] += static_cast<double>(d[i][h]) * static_cast<double>(a[i][h]);
        });
#pragma unroll
        for (int h = 0; h < H; ++h) P[h] = tm.sum(P[h]);
        by_four(b + tm.rank, t, tm.size(), [&](int e, auto K) __attribute__((always_inline)) {
            constexpr int N = decltype(K)::value;
            float a[N][H], d[N][H];
#pragma unroll
            for (int i = 0; i < N; ++i) {
                load_h<H>(alpha + static_cast<int64_t>(e + i * tm.size()) * H, a[i]);
                load_h<H>(dalpha + static_cast<int64_t>(e + i * tm.size()) * H, d[i]);
            }
#pragma unroll
            for (int i = 0; i < N; ++i) {
                float o[H];
#pragma unroll
                for (int h = 0; h < H; ++h)
                    o[h] = static_cast<float>(static_cast<double>(a[i][h]) * (static_cast<double>(d[i][h]) - P[h]));
                store_h<H>(dE + static_cast<int64_t>(e + i * tm.size()) * H, o);
            }
        });
    }
};

template <int H, int GROUP>
__global__ __launch_bounds__(256) void k_edge_softmax_bwd(int n, const int32_t *ptr, softmax_bwd_op<H> op, int long_blocks, int rows_per_wave)
{
    walk_all_rows<GROUP>(ptr, n, op, long_blocks, rows_per_wave);
}

}  // namespace

int tango_sddmm_add_async(const tango_graph *g, int heads, const int8_t *Sq, const float *sS, const int8_t *Dq,
                          const float *sD, float slope, float *E, hipStream_t st)
{
    const int n = g->n_nodes;
    const int grp = pick_group(n, g->n_edges);
    const row_split sp = split_rows(n, g->n_edges, grp);
#define CALL(HH) \
    { \
        sddmm_add_op<HH> op{g->in_src, Sq, Dq, 0.f, 0.f, slope, E, tango_aligned(Sq, HH)}; \
        k_sddmm_add<HH, GROUP><<<sp.grid, 256, 0, st>>>(n, g->in_ptr, op, sS, sD, sp.long_blocks, sp.rows_per_wave); \
    }
    TANGO_DISPATCH_H(heads, grp, CALL)
#undef CALL
    TANGO_LAUNCH_CHECK();
    return TANGO_OK;
}

int tango_sddmm_add_bwd_async(const tango_graph *g, int heads, const int8_t *Sq, const float *sS, const int8_t *Dq,
                              const float *sD, float slope, const float *dE, float *dEpre, float *dS, float *dD,
                              hipStream_t st)
{
    const int n = g->n_nodes;
    const int grp = pick_group(n, g->n_edges);
    const row_split sp = split_rows(n, g->n_edges, grp);
    if (dD || dEpre) {
#define CALL(HH) \
    { \
        sddmm_add_bwd_dst_op<HH> op{g->in_src, Sq, Dq, 0.f, 0.f, slope, dE, dEpre, dD, tango_aligned(Sq, HH)}; \
        k_sddmm_add_bwd_dst<HH, GROUP><<<sp.grid, 256, 0, st>>>(n, g->in_ptr, op, sS, sD, sp.long_blocks, sp.rows_per_wave); \
    }
        TANGO_DISPATCH_H(heads, grp, CALL)
#undef CALL
        TANGO_LAUNCH_CHECK();
    }
    if (dS) {
#define CALL(HH) \
    { \
        sddmm_add_bwd_src_op<HH> op{g->out_dst, g->out_eid, Sq, Dq, 0.f, 0.f, slope, dE, dS, tango_aligned(Dq, HH)}; \
        k_sddmm_add_bwd_src<HH, GROUP><<<sp.grid, 256, 0, st>>>(n, g->out_ptr, op, sS, sD, sp.long_blocks, sp.rows_per_wave); \
    }
        TANGO_DISPATCH_H(heads, grp, CALL)
#undef CALL
        TANGO_LAUNCH_CHECK();
    }
    return TANGO_OK;
}

int tango_edge_softmax_async(const tango_graph *g, int heads, const float *E, float *alpha, float *absmax,
                             hipStream_t st)
{
    const int n = g->n_nodes;
    const int grp = pick_group(n, g->n_edges);
    const row_split sp = split_rows(n, g->n_edges, grp);
    if (absmax) {
        int rc = tango_fill_u32_async(reinterpret_cast<uint32_t *>(absmax), 0u, 1, st);
        if (rc != TANGO_OK) return rc;
    }
#define CALL(HH) \
    { \
        softmax_op<HH> op{E, alpha, 0.f}; \
        k_edge_softmax<HH, GROUP><<<sp.grid, 256, 0, st>>>(n, g->in_ptr, op, absmax, sp.long_blocks, sp.rows_per_wave); \
    }
    TANGO_DISPATCH_H(heads, grp, CALL)
#undef CALL
    TANGO_LAUNCH_CHECK();
    return TANGO_OK;
}

int tango_edge_softmax_bwd_async(const tango_graph *g, int heads, const float *alpha, const float *dalpha, float *dE,
                                 hipStream_t st)
{
    const int n = g->n_nodes;
    const int grp = pick_group(n, g->n_edges);
    const row_split sp = split_rows(n, g->n_edges, grp);
#define CALL(HH) \
    { \
        softmax_bwd_op<HH> op{alpha, dalpha, dE}; \
        k_edge_softmax_bwd<HH, GROUP><<<sp.grid, 256, 0, st>>>(n, g->in_ptr, op, sp.long_blocks, sp.rows_per_wave); \
    }
    TANGO_DISPATCH_H(heads, grp, CALL)
#undef CALL
    TANGO_LAUNCH_CHECK();
    return TANGO_OK;
}

int tango_sddmm_dot_async(const tango_graph *g, int heads, int dim, const int8_t *X_dst, const float *s_dst,
                          const int8_t *X_src, const float *s_src, float *out, hipStream_t st);
int tango_validate_sddmm_dot_shape(int heads, int dim);

namespace {
int validate_in_graph(const tango_graph *g)
{
    TANGO_REQUIRE(g != nullptr, TANGO_ERR_NULL);
    TANGO_REQUIRE(g->n_nodes > 0 && g->n_edges >= 0 && g->n_edges < (int64_t(1) << 31), TANGO_ERR_BAD_SHAPE);
    TANGO_REQUIRE(g->in_ptr && (g->n_edges == 0 || g->in_src), TANGO_ERR_NULL);
    return TANGO_OK;
}
}  // namespace

extern "C" {

int tango_qsddmm(const tango_graph *g, int op, int heads, int dim, const int8_t *X_src, const float *s_src,
                 const int8_t *X_dst, const float *s_dst, float slope, float *E, void *stream)
{
    TANGO_REQUIRE(op == TANGO_SDDMM_ADD_LEAKYRELU || op == TANGO_SDDMM_DOT, TANGO_ERR_BAD_ENUM);
    int rc = validate_in_graph(g);
    if (rc != TANGO_OK) return rc;
    TANGO_REQUIRE(X_src && X_dst && s_src && s_dst && (g->n_edges == 0 || E), TANGO_ERR_NULL);
    if (op == TANGO_SDDMM_ADD_LEAKYRELU) {
        TANGO_REQUIRE(dim == 1, TANGO_ERR_BAD_SHAPE);
        TANGO_REQUIRE(heads_supported(heads), TANGO_ERR_UNSUPPORTED);
        TANGO_REQUIRE(tango_aligned(E, 16), TANGO_ERR_BAD_SHAPE);
        return tango_sddmm_add_async(g, heads, X_src, s_src, X_dst, s_dst, slope, E, tango_stream(stream));
    }
    rc = tango_validate_sddmm_dot_shape(heads, dim);
    if (rc != TANGO_OK) return rc;
    TANGO_REQUIRE(tango_aligned(X_src, 16) && tango_aligned(X_dst, 16), TANGO_ERR_BAD_SHAPE);
    return tango_sddmm_dot_async(g, heads, dim, X_dst, s_dst, X_src, s_src, E, tango_stream(stream));
}

int tango_qsddmm_bwd(const tango_graph *g, int heads, const int8_t *X_src, const float *s_src, const int8_t *X_dst,
                     const float *s_dst, float slope, const float *dE, float *dE_pre, float *dS, float *dD, void *stream)
{
    int rc = validate_in_graph(g);
    if (rc != TANGO_OK) return rc;
    TANGO_REQUIRE(heads_supported(heads), TANGO_ERR_UNSUPPORTED);
    TANGO_REQUIRE(X_src && X_dst && s_src && s_dst && (g->n_edges == 0 || dE), TANGO_ERR_NULL);
    if (dS) TANGO_REQUIRE(g->out_ptr && (g->n_edges == 0 || (g->out_dst && g->out_eid)), TANGO_ERR_NULL);
    TANGO_REQUIRE(tango_aligned(dE, 16) && tango_aligned(dE_pre, 16), TANGO_ERR_BAD_SHAPE);
    return tango_sddmm_add_bwd_async(g, heads, X_src, s_src, X_dst, s_dst, slope, dE, dE_pre, dS, dD,
                                     tango_stream(stream));
}

int tango_edge_softmax(const tango_graph *g, int heads, const float *E, float *alpha, float *absmax_alpha, void *stream)
{
    int rc = validate_in_graph(g);
    if (rc != TANGO_OK) return rc;
    TANGO_REQUIRE(heads_supported(heads), TANGO_ERR_UNSUPPORTED);
    TANGO_REQUIRE(g->n_edges == 0 || (E && alpha), TANGO_ERR_NULL);
    TANGO_REQUIRE(tango_aligned(E, 16) && tango_aligned(alpha, 16), TANGO_ERR_BAD_SHAPE);
    return tango_edge_softmax_async(g, heads, E, alpha, absmax_alpha, tango_stream(stream));
}

int tango_edge_softmax_bwd(const tango_graph *g, int heads, const float *alpha, const float *dalpha, float *dE,
                           void *stream)
{
    int rc = validate_in_graph(g);
    if (rc != TANGO_OK) return rc;
    TANGO_REQUIRE(heads_supported(heads), TANGO_ERR_UNSUPPORTED);
    TANGO_REQUIRE(g->n_edges == 0 || (alpha && dalpha && dE), TANGO_ERR_NULL);
    TANGO_REQUIRE(tango_aligned(alpha, 16) && tango_aligned(dalpha, 16) && tango_aligned(dE, 16), TANGO_ERR_BAD_SHAPE);
    return tango_edge_softmax_bwd_async(g, heads, alpha, dalpha, dE, tango_stream(stream));
}

}  // extern "C"
