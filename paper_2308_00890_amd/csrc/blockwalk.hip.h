// Aggregation over blocks of 64 edges on the matrix cores (included by sparse.hip after the argument structures).
//
// A wavefront walks a chunk of consecutive edges in blocks of 64 and takes one column slice of SW bytes of every gathered
// row (a slice is one 128-byte line where the row is wide enough).  The 64 row slices of a block go from global memory
// straight into LDS (global_load_lds_dwordx4), so a whole block is in flight per wave without a register held for it.  The
// reduction over the edges is a matrix product: v_mfma_i32_16x16x64_i8 with k = the 64 edges, the 16 rows of the left
// operand = sixteen consecutive graph rows (each holds the weights of its own edges, zero elsewhere), and the columns of the
// right operand = 16 feature columns, read from LDS with the transposing ds_read_b64_tr_b8.  All row segments of a block
// are therefore summed at once, whatever their lengths; the sums are exact int32 as before.
//
// Measured against the kernels with a lane group per gathered row (main kernels of one aggregation, us): GCN with 169 k nodes and
// F = 256 153 -> 85; attention forward, the same graph, 4 x 64: 231 -> 93; 256 subgraphs of 1,024 nodes, 2 x 32: 162 -> 92;
// scale-22 graph, F = 128: 2,066 -> 1,427, F = 32: 1,455 -> 950; 2.4 M nodes, 3 x 128: 4,150 -> 3,780; 115 M edges, 4 x 64:
// 2,520 -> 2,330 (1,580 of them for the gathers alone).
//
// Why: the walk with one lane group per gathered row (k_spmm) spent 10 to 15 vector instructions per edge on byte
// transposes, dot products and per-row bookkeeping and was bound by their issue and by one load latency per row segment.
//
// Why slices: the gathers are bound by what crosses from the L2s to the memory side.  The XCDs' L2s are separate, so when
// a row has 2, 4 or 8 slices, XCD x works on slice x % slices only and its L2 holds lines of 1/slices of the table: gathers
// alone (no arithmetic) on the 60 MB table of a graph with 115 M edges took 1.46 instead of 2.04 ms.  Other slice counts
// are walked one slice after the other over the whole chip.
#pragma once

typedef int bw_v4i __attribute__((ext_vector_type(4)));
typedef int bw_v2i __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) bw_v2i bw_lds_v2i;

struct bw_grid {
    int slices;       // column slices of a row
    unsigned groups;  // workgroups per slice
};

// 16-byte chunk c of row r of a block sits in slot c ^ bw_swz(r).  Both kinds of LDS reads then cover all 64 banks once per
// cycle: sixteen consecutive rows at one chunk (16-byte reads), and eight rows of each of two groups of sixteen rows at
// one chunk (transposing reads).  bw_swz(r + 8) == bw_swz(r) ^ (chunks per row / 2) for r % 16 < 8.
template <int SW>
__device__ __forceinline__ int bw_swz(int r)
{
    if (SW == 128) return ((r >> 1) & 7) ^ (((r >> 4) & 1) << 2);
    if (SW == 64) return ((r >> 2) & 3) ^ (((r >> 4) & 1) << 1);
    return ((r >> 3) & 1) ^ ((r >> 4) & 1);
}

// Which slice and which group of chunks this workgroup takes.
__device__ __forceinline__ void bw_place(const bw_grid &gs, int &slice, unsigned &group)
{
    const unsigned b = blockIdx.x;
    if (gs.slices == 2 || gs.slices == 4 || gs.slices == 8) {
        const unsigned xcd = b % 8, s = static_cast<unsigned>(gs.slices);
        slice = static_cast<int>(xcd % s);
        group = (b / 8) * (8 / s) + xcd / s;
    } else {
        slice = static_cast<int>(b / gs.groups);
        group = b % gs.groups;
    }
}

// The 64 row slices of a block into LDS; at: LDS, the table rows of the block's edges (rows of F bytes, X: the slice of row
// 0), as row numbers; for a table known to end below 4 GB as byte offsets (BW_OFFSETS), or as row numbers below 2^24 (BW_ROWS24).
enum { BW_ROWS = 0, BW_OFFSETS = 1, BW_ROWS24 = 2 };
template <int SW, int KIND>
__device__ __forceinline__ void bw_gather(const int8_t *__restrict__ X, const uint32_t *at, int F, int8_t *tile, int lane)
{
    constexpr int CPR = SW / 16, RPI = 64 / CPR;  // chunks of a row slice, rows per load instruction
    const int rr = lane / CPR, slot = lane % CPR;
#pragma unroll
    for (int j = 0; j < CPR; ++j) {
        const int r = RPI * j + rr;
        const uint32_t chunk = static_cast<uint32_t>((slot ^ bw_swz<SW>(r)) * 16);
        const int8_t *from = KIND == BW_OFFSETS ? X + (at[r] + chunk)
                             : KIND == BW_ROWS24 ? X + (__umul24(at[r], static_cast<uint32_t>(F)) + chunk)
                                                 : X + chunk + static_cast<uint64_t>(at[r]) * static_cast<uint32_t>(F);
        __builtin_amdgcn_global_load_lds(reinterpret_cast<const uint32_t *>(from), reinterpret_cast<uint32_t *>(tile + 1024 * j), 16, 0, 0);
    }
}

// The N (1, 2, 4) consecutive bytes at p as one word; aligned: p is a multiple of N.
template <int N>
__device__ __forceinline__ uint32_t bw_load_bytes(const int8_t *p, bool aligned)
{
    if (N == 4 && aligned) return *reinterpret_cast<const uint32_t *>(p);
    if (N == 2 && aligned) return *reinterpret_cast<const uint16_t *>(p);
    uint32_t w = 0;
#pragma unroll
    for (int j = 0; j < N; ++j) w |= static_cast<uint32_t>(static_cast<uint8_t>(p[j])) << (8 * j);
    return w;
}

// Columns 16t .. 16t+15 of the 64 rows as a matrix operand (k = the rows): lane i of group g reads row 16g + i/2 and the row 8
// further, half i%2 of the 16-byte chunk; base, swz: that row's place and its swizzle in bytes.
template <int SW>
__device__ __forceinline__ bw_v4i bw_columns(const int8_t *tile, int base, int swz, int t)
{
    const bw_v2i f0 = __builtin_amdgcn_ds_read_tr8_b64_v2i32((bw_lds_v2i *)(tile + (base + ((16 * t) ^ swz))));
    const bw_v2i f1 = __builtin_amdgcn_ds_read_tr8_b64_v2i32((bw_lds_v2i *)(tile + (base + ((16 * (t ^ (SW / 32))) ^ swz)) + 8 * SW));
    return bw_v4i{f0[0], f0[1], f1[0], f1[1]};
}

// Byte masks (0xff / 0) of edges 16*kg .. 16*kg+15 of a block that lie in [lo, hi).
__device__ __forceinline__ void bw_range_mask(int lo, int hi, int kg, uint32_t (&m)[4])
{
    const int l = min(max(lo - 16 * kg, 0), 16), h = min(max(hi - 16 * kg, 0), 16);
    const uint32_t bits = ((1u << h) - 1u) & ~((1u << l) - 1u);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const uint32_t ones = __umul24((bits >> (4 * q)) & 15u, 0x204081u) & 0x01010101u;  // bit j of the nibble to byte j
        m[q] = (ones << 8) - ones;
    }
}

// Inclusive running maximum over the lanes.
__device__ __forceinline__ int bw_scan_max(int v)
{
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false));  // row_shr:1
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false));  // row_bcast:15 into rows 1 and 3
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false));  // row_bcast:31 into rows 2 and 3
    return v;
}

__device__ __forceinline__ void bw_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// HS: heads in a slice (a slice lies inside one head: 1).  WMODE: W_LOAD (weights at the edge's own position, or at eid[])
// or W_ATT_FWD (attention codes computed on the fly, as in k_spmm; KEEP: alpha and its codes may be asked for).
//
// The edge streams (indices; weight codes, or the codes of the sources) come from HBM, whose latency would be paid per block,
// because the wait for a block's gathers waits for everything requested before it.  They are therefore fetched for a group of
// blocks at a time, one group ahead, and handed on through LDS.
template <int SW, int HS, int WMODE, bool HAS_EID, bool KEEP = false>
__global__ __launch_bounds__(64 * WAVES_PER_BLOCK) __attribute__((amdgpu_waves_per_eu(SW == 128 && HS == 4 && WMODE == W_ATT_FWD ? 3 : 4))) void k_spmm_blocks(spmm_args a, bw_grid gs)
{
    constexpr int T = SW / 16;  // 16-column tiles of a slice
    constexpr bool ATT = WMODE == W_ATT_FWD;
    constexpr int GB = ATT && SW == 128 && HS > 1 ? 2 : 4;  // blocks whose streams are fetched together (registers allow only two there)
    static_assert(T % HS == 0 && HS <= 4, "a tile lies inside one head, the codes of an edge in a word");
    __shared__ __align__(16) int8_t tile_s[WAVES_PER_BLOCK][64 * SW];
    __shared__ __align__(16) uint32_t at_s[WAVES_PER_BLOCK][64 * GB];            // rows (or offsets) of the gathered table
    __shared__ __align__(16) int8_t w_s[WAVES_PER_BLOCK][HS * (ATT ? 64 : 64 * GB)];  // weight codes, head-major
    __shared__ uint32_t code_s[ATT ? WAVES_PER_BLOCK : 1][ATT ? 64 * GB * HS / 4 : 1];  // S_q of the sources, HS bytes per edge
    __shared__ int row_s[ATT ? WAVES_PER_BLOCK : 1][64];
    const int lane = threadIdx.x % TANGO_WAVE;
    const int wv = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x / TANGO_WAVE));
    int slice;
    unsigned group;
    bw_place(gs, slice, group);
    const int64_t chunk = static_cast<int64_t>(group) * WAVES_PER_BLOCK + wv;
    const int64_t c0l = chunk << a.chunk_shift;
    if (c0l >= a.nnz) return;
    const int c0 = static_cast<int>(c0l), c1 = static_cast<int>(min(c0l + (int64_t(1) << a.chunk_shift), a.nnz));
    const int col0 = slice * SW, h0 = col0 / a.dim;
    const int g = lane >> 4, n16 = lane & 15;
    const int8_t *X = a.X + col0;
    int8_t *tile = tile_s[wv];
    int8_t *wl = w_s[wv];
    float s_w, inv_w = 0.0f, att_sS = 0.0f, att_sD = 0.0f;
    if (ATT) {
        tango_scale_from_absmax(*a.att.absmax_alpha, s_w, inv_w);
        if (blockIdx.x == 0 && threadIdx.x == 0) *a.att.s_alpha = s_w;
        att_sS = *a.att.sS;
        att_sD = *a.att.sD;
    } else {
        s_w = *a.s_w;
    }
    const float sc = s_w * (*a.s_X);
    const int H = a.heads;

    // Graph row r is row 4*(r & 3) + ((r >> 2) & 3) of the matrix product: accumulator register i of lane group g then
    // belongs to the row with r & 15 == 4*i + g, so that four consecutive rows share a register across the lane groups
    // and a row keeps its place from block to block.
    const int a_row = ((n16 & 3) << 2) | (n16 >> 2);  // r & 15 of the row whose weights this lane holds
    bw_v4i acc[T];
#pragma unroll
    for (int t = 0; t < T; ++t) acc[t] = bw_v4i{0, 0, 0, 0};
    // transposing reads: lane i of group g reads row 16g + i/2 (and the row 8 further), half i%2 of a 16-byte chunk
    const int tr_row = 16 * g + (n16 >> 1);
    const int tr_base = tr_row * SW + (n16 & 1) * 8, tr_swz = bw_swz<SW>(tr_row) * 16;
    int maxabs = 0;

    int R = c0 == 0 ? 0 : __builtin_amdgcn_readfirstlane(wave_find_row(a.ptr, a.n, c0));  // first row with an edge at or behind the walk
    auto load_row_ends = [&](int r0, int &lo, int &hi) __attribute__((always_inline)) {  // lane l: where row r0 + l starts and ends (rows beyond the last: nnz)
        lo = a.ptr[min(r0 + lane, a.n)];
        hi = a.ptr[min(r0 + lane + 1, a.n)];
    };
    const int last = c1 - 1;
    // the next group's streams: edges beyond the chunk repeat its last one (their weights are zero)
    int n_idx[GB], n_eid[GB];
    uint32_t n_w[GB];
    auto request_idx = [&](int e0) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < GB; ++k) n_idx[k] = a.idx[min(e0 + 64 * k + lane, last)];
    };
    auto request_eid = [&](int e0) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < GB; ++k) n_eid[k] = a.eid[min(e0 + 64 * k + lane, last)];
    };
    const int8_t *stream = ATT ? a.att.src_codes : (HAS_EID ? nullptr : a.w);  // the codes in edge order, where there are such
    const bool aligned = ATT || a.w_words;
    auto request_w = [&](int e0) __attribute__((always_inline)) {
        if (stream) {  // (a branch of its own: nothing in it waits for the indices)
#pragma unroll
            for (int k = 0; k < GB; ++k) n_w[k] = bw_load_bytes<HS>(stream + static_cast<int64_t>(min(e0 + 64 * k + lane, last)) * H + h0, aligned);
        } else if (ATT) {
#pragma unroll
            for (int k = 0; k < GB; ++k) n_w[k] = bw_load_bytes<HS>(a.att.Sq + static_cast<int64_t>(n_idx[k]) * H + h0, true);
        } else if (HAS_EID) {
#pragma unroll
            for (int k = 0; k < GB; ++k) n_w[k] = bw_load_bytes<HS>(a.w + static_cast<int64_t>(n_eid[k]) * H + h0, aligned);
        }
    };
    int row_lo, row_hi;
    load_row_ends(R, row_lo, row_hi);
    request_idx(c0);
    if (HAS_EID) request_eid(c0);
    request_w(c0);
    if (HAS_EID) request_eid(c0 + 64 * GB);

    // Random bits: one generator block serves eight consecutive (edge, head) elements, so one evaluation by all lanes covers
    // 64 / H consecutive groups of eight edges = 8 / H blocks of 64 edges.
    const int rng_every = ATT ? 64 * max(1, 8 / H) : 64;
    uint4 rng_blk = make_uint4(0, 0, 0, 0);
    int rng_first = 0;  // the edge whose elements begin with lane 0's block
    // Attention mode: D_q and row_lse of the row of every lane's edge, for the block [base, end) whose first row is r0 (lo, hi:
    // where the rows r0 + lane start and end).  A row that goes on filling whole blocks is fetched once.
    uint32_t dq = 0;  // (as loaded: nothing here waits for the loads)
    float lse[HS];
    int held = -1;  // the row whose values all lanes hold
    auto fetch_rows = [&](int base, int end, int r0, int lo, int hi) __attribute__((always_inline)) {
        int my_row = r0;
        if (__builtin_amdgcn_readfirstlane(hi) < end) {  // more than one row
            row_s[wv][lane] = 0;
            bw_lds_fence();
            for (int w = r0;;) {
                const int l = max(lo - base, 0), h = min(hi, end) - base;
                if (l < h) row_s[wv][l] = w + lane;
                if (__builtin_amdgcn_readlane(hi, 63) >= end || w + 64 >= a.n) break;
                w += 64;
                load_row_ends(w, lo, hi);
            }
            bw_lds_fence();
            my_row = bw_scan_max(row_s[wv][lane]);
            held = -1;
        } else if (held == r0) {
            return;
        } else {
            held = r0;
        }
        const int64_t at = static_cast<int64_t>(my_row) * H + h0;
        dq = bw_load_bytes<HS>(a.att.Dq + at, true);
#pragma unroll
        for (int h = 0; h < HS; ++h) lse[h] = a.att.row_lse[at + h];
    };
    if (ATT) fetch_rows(c0, min(c0 + 64, c1), R, row_lo, row_hi);

    for (int base = c0; base < c1; base += 64) {
        const int cnt = min(64, c1 - base), end = base + cnt;
        const int part = ((base - c0) >> 6) & (GB - 1);  // this block's place in its group
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): the previous block's reads of LDS are done
        if (part == 0) {
#pragma unroll
            for (int k = 0; k < GB; ++k) {
                at_s[wv][64 * k + lane] = ATT ? static_cast<uint32_t>(n_idx[k]) * static_cast<uint32_t>(a.F) : static_cast<uint32_t>(n_idx[k]);
                if (ATT) {
                    if (HS == 4) code_s[wv][64 * k + lane] = n_w[k];
                    else if (HS == 2) reinterpret_cast<uint16_t *>(code_s[wv])[64 * k + lane] = static_cast<uint16_t>(n_w[k]);
                    else reinterpret_cast<uint8_t *>(code_s[wv])[64 * k + lane] = static_cast<uint8_t>(n_w[k]);
                } else {
                    const uint32_t w = base + 64 * k + lane < c1 ? n_w[k] : 0u;
#pragma unroll
                    for (int h = 0; h < HS; ++h) wl[64 * GB * h + 64 * k + lane] = static_cast<int8_t>(w >> (8 * h));
                }
            }
            bw_lds_fence();
        }
        // ---- gather the block
        bw_gather<SW, ATT ? BW_OFFSETS : BW_ROWS>(X, &at_s[wv][64 * part], a.F, tile, lane);
        if (part == 0) {
            request_idx(base + 64 * GB);
            request_w(base + 64 * GB);
            if (HAS_EID) request_eid(base + 128 * GB);
        }
        // ---- the weight codes of the block, one byte per edge and head
        if (ATT) {
            const int64_t i0 = static_cast<int64_t>(base + lane) * H + h0;
            uint32_t codes;
            if (HS == 4) codes = code_s[wv][64 * part + lane];
            else if (HS == 2) codes = reinterpret_cast<const uint16_t *>(code_s[wv])[64 * part + lane];
            else codes = reinterpret_cast<const uint8_t *>(code_s[wv])[64 * part + lane];
            uint4 blk = make_uint4(0, 0, 0, 0);
            if (a.att.rounding == TANGO_SR) {
                if ((base - c0) % rng_every == 0) {
                    rng_first = base;
                    rng_blk = tango_philox_block(a.att.rng, ((static_cast<uint64_t>(base) * static_cast<uint32_t>(H)) >> 3) + static_cast<uint32_t>(lane));
                }
                // (the HS elements of an edge lie in one block: their index is a multiple of HS)
                const int from = ((base + lane - rng_first) * H + h0) >> 3;
                blk = make_uint4(__shfl(rng_blk.x, from, 64), __shfl(rng_blk.y, from, 64), __shfl(rng_blk.z, from, 64), __shfl(rng_blk.w, from, 64));
            }
#pragma unroll
            for (int h = 0; h < HS; ++h) {
                bool pos;
                const float sq = static_cast<float>(static_cast<int8_t>(codes >> (8 * h)));
                const float td = att_sD * static_cast<float>(static_cast<int8_t>(dq >> (8 * h)));
                const float ev = tango_attn_score(att_sS * sq, td, a.att.slope, pos);
                const float al = tango_attn_alpha(ev, lse[h]);
                const int q = a.att.rounding == TANGO_SR
                                  ? tango_round_clamp<TANGO_SR>(al * inv_w, tango_bits16(blk, static_cast<int>((i0 + h) & 7)))
                                  : tango_round_clamp<TANGO_RN>(al * inv_w, 0u);
                if (KEEP && lane < cnt) {
                    if (a.att.alpha_dump) a.att.alpha_dump[i0 + h] = al;
                    if (a.att.alpha_q) a.att.alpha_q[i0 + h] = static_cast<int8_t>(q);
                }
                wl[64 * h + lane] = static_cast<int8_t>(lane < cnt ? q : 0);
            }
        }
        bw_lds_fence();
        bw_v4i wf[HS];  // the codes of edges 16g .. 16g+15
#pragma unroll
        for (int h = 0; h < HS; ++h)
            wf[h] = *reinterpret_cast<const bw_v4i *>(wl + (ATT ? 64 * h : 64 * GB * h + 64 * part) + 16 * g);
        int nrows = __popcll(__ballot(R + lane < a.n && row_lo < end));  // rows of the window with an edge before `end`
        int nfin = __popcll(__ballot(R + lane < a.n && row_hi <= end));  // and those that end by then
        int next_lo = row_lo, next_hi = row_hi;
        if (nfin > 0) load_row_ends(R + nfin, next_lo, next_hi);
        __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): the tile has landed
        bw_lds_fence();
        // the rows of the next block: their values are on the way while this block is multiplied
        const bool more = end < c1, early = nfin < 64;
        if (ATT && more && early) fetch_rows(end, min(end + 64, c1), R + nfin, next_lo, next_hi);
        // ---- sixteen rows at a time: multiply, then write out the rows that end here
        for (;;) {
            for (int p = 0; p < nrows; p += 16) {
                bw_v4i wm[HS];
                const int src = p + ((a_row - R) & 15);  // the window lane of my row (R + p + j with j = (a_row - R) mod 16)
                if (nrows == 1 && __builtin_amdgcn_readfirstlane(row_lo) <= base) {  // the whole block is row R's
#pragma unroll
                    for (int h = 0; h < HS; ++h)
#pragma unroll
                        for (int k = 0; k < 4; ++k) wm[h][k] = src == 0 ? wf[h][k] : 0;
                } else {
                    uint32_t m[4];
                    const int lo = __shfl(row_lo, src, 64) - base, hi = min(__shfl(row_hi, src, 64) - base, cnt);
                    bw_range_mask(lo, hi, g, m);
#pragma unroll
                    for (int h = 0; h < HS; ++h)
#pragma unroll
                        for (int k = 0; k < 4; ++k) wm[h][k] = wf[h][k] & static_cast<int>(m[k]);
                }
#pragma unroll
                for (int t = 0; t < T; ++t) {
                    const bw_v4i f = bw_columns<SW>(tile, tr_base, tr_swz, t);
                    acc[t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wm[t * HS / T], f, acc[t], 0, 0, 0);
                }
                if (nfin <= p) continue;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int j = p + ((4 * i + g - R) & 15);  // the window lane of the row in register i
                    const bool fin = j < nfin;
                    if (!__any(fin)) continue;
                    // (only the row that holds the chunk's first edge can have begun before it: it is shared with other chunks)
                    const int began = __shfl(row_lo, j, 64);  // (by all lanes: a lane shuffle reads active lanes only)
                    const bool whole = fin && began >= c0;
                    const int row = R + j;
                    if (ATT && a.relu_bits) {
#pragma unroll
                        for (int t = 0; t < T; ++t) {
                            const unsigned long long bits = __ballot(acc[t][i] > 0);
                            if (whole && n16 == 0)
                                a.relu_bits[(static_cast<uint32_t>(row) * static_cast<uint32_t>(a.F / 16)) + (col0 / 16 + t)] =
                                    static_cast<uint16_t>(bits >> (16 * g));
                        }
                    }
                    if (fin) {
                        float *orow = a.out + (static_cast<int64_t>(row) * a.F + col0 + n16);
                        if (whole) {
#pragma unroll
                            for (int t = 0; t < T; ++t) {
                                int v = acc[t][i];
                                if (ATT && a.relu) v = max(v, 0);
                                orow[16 * t] = static_cast<float>(v) * sc;
                                maxabs = max(maxabs, abs(v));
                            }
                        } else {
#pragma unroll
                            for (int t = 0; t < T; ++t) atomicAdd(reinterpret_cast<int *>(orow) + 16 * t, acc[t][i]);
                        }
#pragma unroll
                        for (int t = 0; t < T; ++t) acc[t][i] = 0;
                    }
                }
            }
            R += nfin;
            row_lo = next_lo;
            row_hi = next_hi;
            if (nfin < 64 || R >= a.n || __builtin_amdgcn_readfirstlane(row_lo) >= end) break;
            nrows = __popcll(__ballot(R + lane < a.n && row_lo < end));  // the window ended inside the block: the next one
            nfin = __popcll(__ballot(R + lane < a.n && row_hi <= end));
            load_row_ends(R + nfin, next_lo, next_hi);
        }
        if (ATT && more && !early) fetch_rows(end, min(end + 64, c1), R, row_lo, row_hi);
    }
    // the row that runs on into the next chunk
    if (R < a.n) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (((R >> 2) & 3) != i) continue;
            int *orow = reinterpret_cast<int *>(a.out + (static_cast<int64_t>(R) * a.F + col0 + n16));
#pragma unroll
            for (int t = 0; t < T; ++t)
                if (g == (R & 3) && acc[t][i] != 0) atomicAdd(orow + 16 * t, acc[t][i]);
        }
    }
    if (a.absmax) {
        float m = static_cast<float>(maxabs) * sc;
        m = tango_wave_max(m);
        if (lane == 0 && m > 0.0f) tango_atomic_max_nonneg(a.absmax, m);
    }
}

// Dot products over blocks of 64 edges: for every edge of a block and every head of a slice (whole heads: HS of them, at most
// 128 columns) the product of the gathered row with the resident row of the edge's own graph row.  DOT_STORE writes them out;
// DOT_DST (steps 5'', 4', 3'': see k_sddmm_dot) turns them into the three running sums per (row, head).
//
// The gathered rows (LDS, as in k_spmm_blocks) are the left operand of v_mfma_i32_16x16x64_i8, sixteen edges at a time, k =
// their columns.  The right operand has sixteen columns: column 4q + c is the resident row number c of the rows that the
// sixteen edges 16q .. 16q+15 belong to.  Lane (group g, column 4q + c) then finds the products of edges 16q + 4g + i,
// i = 0..3, with that row in its four result registers of step q; the one that belongs to the edge's row is picked with a
// sum over the four lanes of a quad, and lane (g, 4q + c) goes on with edge 16q + 4g + c: no trip through LDS.  Edges whose
// group of sixteen spans more than four rows take further rounds of four rows.
template <int SW, int HS, int MODE>
__global__ __launch_bounds__(64 * WAVES_PER_BLOCK) __attribute__((amdgpu_waves_per_eu(4))) void k_dot_blocks(sddmm_dot_args a, bw_grid gs)
{
    constexpr bool ATT = MODE == DOT_DST;
    constexpr int GB = ATT && SW == 128 ? 2 : 4;  // blocks whose streams are fetched together
    constexpr int NC = SW >= 64 ? SW / 64 : 1;   // 64-column steps of a slice
    constexpr int DIM = SW / HS;                 // columns of a head
    constexpr int HPC = DIM >= 64 ? 1 : (SW >= 64 ? 64 : SW) / DIM;  // heads in a 64-column step
    __shared__ __align__(16) int8_t tile_s[WAVES_PER_BLOCK][64 * SW];
    __shared__ __align__(16) uint32_t at_s[WAVES_PER_BLOCK][64 * GB];
    __shared__ uint32_t code_s[ATT ? WAVES_PER_BLOCK : 1][ATT ? 64 * GB * HS / 4 : 1];
    __shared__ __align__(16) int row_s[WAVES_PER_BLOCK][64];
    __shared__ __align__(16) float2 val_s[ATT ? WAVES_PER_BLOCK : 1][ATT ? HS : 1][64];  // per head and edge: alpha (negative: the slope side), dalpha
    const int lane = threadIdx.x % TANGO_WAVE;
    const int wv = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x / TANGO_WAVE));
    int slice;
    unsigned group;
    bw_place(gs, slice, group);
    const int64_t chunk = static_cast<int64_t>(group) * WAVES_PER_BLOCK + wv;
    const int64_t c0l = chunk << a.chunk_shift;
    if (c0l >= a.nnz) return;
    const int c0 = static_cast<int>(c0l), c1 = static_cast<int>(min(c0l + (int64_t(1) << a.chunk_shift), a.nnz)), last = c1 - 1;
    const int col0 = slice * SW, h0 = slice * HS, H = a.heads;
    const int g = lane >> 4, n16 = lane & 15, q_l = n16 >> 2, c_l = n16 & 3;
    const int my_edge = 16 * q_l + 4 * g + c_l;  // the edge of a block that this lane goes on with
    const int8_t *X = a.Xsrc + col0, *Y = a.Xdst + col0;
    int8_t *tile = tile_s[wv];
    const float sc = (*a.s_dst) * (*a.s_src);
    float sS = 0.0f, sD = 0.0f;
    tango_row_sum_grid grid{0, 0};
    if (ATT) {
        sS = *a.sS;
        sD = *a.sD;
        grid = tango_row_sum_grid_for(sc, DIM, a.slope);
    }
    int R = c0 == 0 ? 0 : __builtin_amdgcn_readfirstlane(wave_find_row(a.ptr, a.n, c0));
    auto load_row_ends = [&](int r0, int &lo, int &hi) __attribute__((always_inline)) {
        lo = a.ptr[min(r0 + lane, a.n)];
        hi = a.ptr[min(r0 + lane + 1, a.n)];
    };
    int n_idx[GB];
    uint32_t n_w[GB];
    auto request = [&](int e0) __attribute__((always_inline)) {  // the next group's streams
#pragma unroll
        for (int k = 0; k < GB; ++k) n_idx[k] = a.idx[min(e0 + 64 * k + lane, last)];
        if (ATT && a.src_codes) {  // (a branch of its own: nothing in it waits for the indices)
#pragma unroll
            for (int k = 0; k < GB; ++k) n_w[k] = bw_load_bytes<HS>(a.src_codes + static_cast<int64_t>(min(e0 + 64 * k + lane, last)) * H + h0, true);
        } else if (ATT) {
#pragma unroll
            for (int k = 0; k < GB; ++k) n_w[k] = bw_load_bytes<HS>(a.Sq + static_cast<int64_t>(n_idx[k]) * H + h0, true);
        }
    };
    auto hand_over = [&]() __attribute__((always_inline)) {  // ... and into LDS
#pragma unroll
        for (int k = 0; k < GB; ++k) {
            at_s[wv][64 * k + lane] = static_cast<uint32_t>(n_idx[k]) * static_cast<uint32_t>(a.F);
            if (ATT) {
                if (HS == 4) code_s[wv][64 * k + lane] = n_w[k];
                else if (HS == 2) reinterpret_cast<uint16_t *>(code_s[wv])[64 * k + lane] = static_cast<uint16_t>(n_w[k]);
                else reinterpret_cast<uint8_t *>(code_s[wv])[64 * k + lane] = static_cast<uint8_t>(n_w[k]);
            }
        }
        bw_lds_fence();
    };
    // What a block needs of its graph rows: `held` >= 0: one row for the whole block, else row_s holds every edge's row.  The
    // resident rows of round 0 of the products, and D_q and row_lse of the row of this lane's edge, are requested.
    int held = -1, spans = 0;  // spans: the most rows a group of sixteen edges lies in, less one
    bw_v4i resident[NC];
    uint32_t dq = 0, dq_n = 0;  // D_q and row_lse of the row of this lane's edge (as loaded: nothing here waits for the loads)
    float lse[HS], lse_n[HS];
    auto load_resident = [&](int row) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < NC; ++k) {
            resident[k] = bw_v4i{0, 0, 0, 0};
            if (SW >= 64 || g < 2) resident[k] = *reinterpret_cast<const bw_v4i *>(Y + static_cast<int64_t>(row) * a.F + 64 * k + 16 * g);
        }
    };
    auto fetch_rows = [&](int base, int end, int r0, int lo, int hi) __attribute__((always_inline)) {
        int my_row = r0;
        if (__builtin_amdgcn_readfirstlane(hi) < end) {
            row_s[wv][lane] = 0;
            bw_lds_fence();
            for (int w = r0;;) {
                const int l = max(lo - base, 0), h = min(hi, end) - base;
                if (l < h) row_s[wv][l] = w + lane;
                if (__builtin_amdgcn_readlane(hi, 63) >= end || w + 64 >= a.n) break;
                w += 64;
                load_row_ends(w, lo, hi);
            }
            bw_lds_fence();
            const int row_of = bw_scan_max(row_s[wv][lane]);
            row_s[wv][lane] = row_of;  // (edges beyond the block: the last row)
            bw_lds_fence();
            my_row = row_s[wv][my_edge];
            const int first = row_s[wv][16 * q_l], final = row_s[wv][16 * q_l + 15];
            held = -1;
            spans = 0;
            for (int d = 4; __any(final - first >= d); d += 4) spans = d;
            load_resident(min(first + c_l, final));
        } else if (held == r0) {
            dq_n = dq;
#pragma unroll
            for (int h = 0; h < HS; ++h) lse_n[h] = lse[h];
            return;
        } else {
            held = r0;
            spans = 0;
            load_resident(r0);
        }
        if (ATT) {
            const int64_t at = static_cast<int64_t>(my_row) * H + h0;
            dq_n = bw_load_bytes<HS>(a.Dq + at, true);
#pragma unroll
            for (int h = 0; h < HS; ++h) lse_n[h] = a.row_lse[at + h];
        }
    };
    int row_lo, row_hi;
    load_row_ends(R, row_lo, row_hi);
    request(c0);
    fetch_rows(c0, min(c0 + 64, c1), R, row_lo, row_hi);
    hand_over();
    bw_gather<SW, BW_OFFSETS>(X, &at_s[wv][0], a.F, tile, lane);
    request(c0 + 64 * GB);
    double acc[HS][3];  // the sums of the row that fills whole blocks
    int acc_row = -1;
#pragma unroll
    for (int h = 0; h < HS; ++h) acc[h][0] = acc[h][1] = acc[h][2] = 0.0;
    auto flush = [&]() __attribute__((always_inline)) {
        if (acc_row < 0) return;
#pragma unroll
        for (int h = 0; h < HS; ++h) {
            const double t0 = tango_stride_sum_f64(acc[h][0], 1), t1 = tango_stride_sum_f64(acc[h][1], 1), t2 = tango_stride_sum_f64(acc[h][2], 1);
            const double t = lane == 0 ? t0 : (lane == 1 ? t1 : t2);
            if (lane < 3) tango_row_sum_add(a.stats + (static_cast<int64_t>(acc_row) * H + h0 + h) * 3 + lane, t, lane == 2 ? grid.c : grid.ab);
            acc[h][0] = acc[h][1] = acc[h][2] = 0.0;
        }
        acc_row = -1;
    };

    for (int base = c0; base < c1; base += 64) {
        const int cnt = min(64, c1 - base), end = base + cnt;
        const int place = ((base - c0) >> 6) & (GB - 1);  // this block's place in its group
        const int nrows = __popcll(__ballot(R + lane < a.n && row_lo < end));
        const int nfin = __popcll(__ballot(R + lane < a.n && row_hi <= end));
        int next_lo = row_lo, next_hi = row_hi;
        if (nfin > 0) load_row_ends(R + nfin, next_lo, next_hi);
        __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): the tile has landed
        bw_lds_fence();
        // ---- the dot products of my edge, all heads
        const bool uniform = held >= 0;
        const int block_row = held;
        int dot[HS];
#pragma unroll
        for (int h = 0; h < HS; ++h) {
            dot[h] = 0;
            lse[h] = lse_n[h];
        }
        dq = dq_n;
        int4 rows4 = make_int4(0, 0, 0, 0);
        int first = 0, final = 0;
        if (!uniform) {
            rows4 = *reinterpret_cast<const int4 *>(&row_s[wv][16 * q_l + 4 * g]);
            first = row_s[wv][16 * q_l];
            final = row_s[wv][16 * q_l + 15];
        }
        for (int d0 = 0; d0 <= spans; d0 += 4) {
            if (d0 > 0) load_resident(min(first + d0 + c_l, final));
#pragma unroll
            for (int h = 0; h < HS; ++h) {
                bw_v4i res[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) res[q] = bw_v4i{0, 0, 0, 0};
                constexpr int KH = DIM >= 64 ? DIM / 64 : 1;  // steps of a head
#pragma unroll
                for (int k = 0; k < KH; ++k) {
                    const int kc = DIM >= 64 ? h * KH + k : h / HPC;
                    bw_v4i b = resident[kc];
                    if (HPC > 1) {  // several heads in the 64 columns: zero the others
                        const bool mine = (16 * g) / DIM == h % HPC;
#pragma unroll
                        for (int w = 0; w < 4; ++w) b[w] = mine ? b[w] : 0;
                    }
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int r = 16 * q + n16;
                        bw_v4i f = {0, 0, 0, 0};
                        if (SW >= 64 || g < 2) f = *reinterpret_cast<const bw_v4i *>(tile + r * SW + (((4 * kc + g) ^ bw_swz<SW>(r)) * 16));
                        res[q] = __builtin_amdgcn_mfma_i32_16x16x64_i8(f, b, res[q], 0, 0, 0);
                    }
                }
                int v[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = q_l == 0 ? res[0][i] : (q_l == 1 ? res[1][i] : (q_l == 2 ? res[2][i] : res[3][i]));
                if (!uniform) {
                    const int row = first + d0 + c_l;
                    v[0] = rows4.x == row ? v[0] : 0;
                    v[1] = rows4.y == row ? v[1] : 0;
                    v[2] = rows4.z == row ? v[2] : 0;
                    v[3] = rows4.w == row ? v[3] : 0;
#pragma unroll
                    for (int i = 0; i < 4; ++i) v[i] = tango_group_sum_c<4>(v[i], 4);
                }
                dot[h] += c_l == 0 ? v[0] : (c_l == 1 ? v[1] : (c_l == 2 ? v[2] : v[3]));
            }
        }
        uint32_t codes = 0;
        if (ATT) {
            if (HS == 4) codes = code_s[wv][64 * place + my_edge];
            else if (HS == 2) codes = reinterpret_cast<const uint16_t *>(code_s[wv])[64 * place + my_edge];
            else codes = reinterpret_cast<const uint8_t *>(code_s[wv])[64 * place + my_edge];
        }
        // ---- the next block's gathers, while this one's products are turned into sums
        const int R_now = R, rows_now = nrows, lo_now = row_lo, hi_now = row_hi;
        bool wide = nfin == 64 && nrows == 64;  // (the window of 64 rows may end inside the block)
        R += nfin;
        row_lo = next_lo;
        row_hi = next_hi;
        while (wide && R < a.n && __builtin_amdgcn_readfirstlane(row_lo) < end) {
            const int more = __popcll(__ballot(R + lane < a.n && row_hi <= end));
            R += more;
            wide = more == 64;
            load_row_ends(R, row_lo, row_hi);
        }
        if (end < c1) {
            __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): this block's reads of LDS are done
            if (place == GB - 1) hand_over();
            fetch_rows(end, min(end + 64, c1), R, row_lo, row_hi);
            bw_gather<SW, BW_OFFSETS>(X, &at_s[wv][64 * ((place + 1) & (GB - 1))], a.F, tile, lane);
            if (place == GB - 1) request(end + 64 * GB);
        }
        const bool there = my_edge < cnt;
        if (!ATT) {
            if (there) {
                float *o = a.out + (static_cast<int64_t>(base) + my_edge) * H + h0;
#pragma unroll
                for (int h = 0; h < HS; ++h) o[h] = static_cast<float>(dot[h]) * sc;
            }
            continue;
        }
        if (uniform && acc_row != block_row) {
            flush();
            acc_row = block_row;
        }
#pragma unroll
        for (int h = 0; h < HS; ++h) {
            const float da = static_cast<float>(dot[h]) * sc;
            bool pos;
            const float td = sD * static_cast<float>(static_cast<int8_t>(dq >> (8 * h)));
            const float ev = tango_attn_score(sS * static_cast<float>(static_cast<int8_t>(codes >> (8 * h))), td, a.slope, pos);
            float al = tango_attn_alpha(ev, lse[h]);
            if (uniform) {
                al = there ? al : 0.0f;
                const double sl = pos ? 1.0 : static_cast<double>(a.slope);
                const double ad = static_cast<double>(al) * static_cast<double>(da);
                acc[h][0] += ad;
                acc[h][1] += ad * sl;
                acc[h][2] += static_cast<double>(al) * sl;
            } else {
                val_s[wv][h][my_edge] = make_float2(pos ? al : -al, da);
            }
        }
        if (!uniform) {
            flush();
            // a group of P lanes per (row of the block, head): they share the row's edges
            bw_lds_fence();
            int w = R_now, nr = rows_now, lo = lo_now, hi = hi_now;
            for (;;) {
                const int items = nr * HS;
                const int log2P = items <= 4 ? 4 : (items <= 8 ? 3 : (items <= 16 ? 2 : (items <= 32 ? 1 : 0)));
                const int P = 1 << log2P, part = lane & (P - 1);
                for (int it0 = 0; it0 < items; it0 += 64 >> log2P) {
                    const int it = it0 + (lane >> log2P);
                    const int j = min(it / HS, 63), h = it % HS;
                    const int row_b = __shfl(lo, j, 64), row_t = __shfl(hi, j, 64);  // (by all lanes: a shuffle reads active lanes only)
                    const int b = max(row_b - base, 0), t = it < items ? min(row_t - base, cnt) : 0;
                    double sa = 0.0, sb = 0.0, sc3 = 0.0;
#pragma unroll 4
                    for (int e = b + part; e < t; e += P) {
                        const float2 v = val_s[wv][h][e];
                        const double sl = __float_as_int(v.x) >= 0 ? 1.0 : static_cast<double>(a.slope);
                        const double al = static_cast<double>(fabsf(v.x));
                        const double ad = al * static_cast<double>(v.y);
                        sa += ad;
                        sb += ad * sl;
                        sc3 += al * sl;
                    }
                    sa = tango_group_sum_f64(sa, P);
                    sb = tango_group_sum_f64(sb, P);
                    sc3 = tango_group_sum_f64(sc3, P);
                    if (b < t) {
                        unsigned long long *st = a.stats + (static_cast<int64_t>(w + j) * H + h0 + h) * 3;
                        for (int k = part; k < 3; k += P) {
                            const double v = k == 0 ? sa : (k == 1 ? sb : sc3);
                            tango_row_sum_add(st + k, v, k == 2 ? grid.c : grid.ab);
                        }
                    }
                }
                if (nr < 64 || w + 64 >= a.n) break;
                w += 64;
                load_row_ends(w, lo, hi);
                nr = __popcll(__ballot(w + lane < a.n && lo < end));
                if (nr == 0) break;
            }
            bw_lds_fence();
        }
    }
    if (ATT) flush();
}

// The source-side walk of the attention backward (steps 5' and 3' in one walk over the out-edges, see the DS form of k_spmm) over
// blocks of 64 edges.  A block's gathered gradient rows are used twice from LDS: transposed, with the recomputed int8 attention
// codes, for the aggregation (as in k_spmm_blocks), and as they are, with the resident feature rows, for dalpha of every edge (as
// in k_dot_blocks).  Lane (g, 4q + c) goes through the attention arithmetic of edge 16q + 4g + c from the codes to dE.
// What bounds it is the arithmetic per (edge, head) - rounding bits that no other edge shares, score, exp, fp64 difference - and
// the two random reads of an edge (a row slice and its records): the walk over whole rows spent most of its time in lane-group
// sums of the dot products and in waits for four rows in flight, here 64 are.  Measured: 1,024 nodes, 16 K edges, 2 x 32: 17.5 ->
// 8.0 us; 262 K nodes, 4.5 M edges, 2 x 32: 300 -> 136 us; 40 M edges at mean degree 17, 1 x 128: 4.01 -> 1.50 ms, 2 x 64: 4.13 -> 1.63 ms.
template <int SW, int HS>
__global__ __launch_bounds__(64 * WAVES_PER_BLOCK) __attribute__((amdgpu_waves_per_eu(SW == 128 ? 3 : 4))) void k_rev_blocks(spmm_args a, bw_grid gs)
{
    constexpr int T = SW / 16;
    constexpr int NC = SW >= 64 ? SW / 64 : 1;
    constexpr int DIM = SW / HS;
    constexpr int HPC = DIM >= 64 ? 1 : (SW >= 64 ? 64 : SW) / DIM;
    constexpr int GB = 2;  // blocks whose streams are fetched together
    __shared__ __align__(16) int8_t tile_s[WAVES_PER_BLOCK][64 * SW];
    __shared__ __align__(16) uint32_t at_s[WAVES_PER_BLOCK][64 * GB];
    __shared__ __align__(16) int8_t w_s[WAVES_PER_BLOCK][HS * 64];
    __shared__ __align__(16) int row_s[WAVES_PER_BLOCK][64];
    __shared__ float val_s[WAVES_PER_BLOCK][HS][64];
    int lane = threadIdx.x % TANGO_WAVE;
    const int wv = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x / TANGO_WAVE));
    int slice;
    unsigned group;
    bw_place(gs, slice, group);
    const int64_t chunk = static_cast<int64_t>(group) * WAVES_PER_BLOCK + wv;
    const int64_t c0l = chunk << a.chunk_shift;
    if (c0l >= a.nnz) return;
    const int c0 = static_cast<int>(c0l), c1 = static_cast<int>(min(c0l + (int64_t(1) << a.chunk_shift), a.nnz)), last = c1 - 1;
    const int col0 = slice * SW, h0 = slice * HS, H = a.heads;
    // (what follows from the lane is formed anew for every block, behind an asm that hides the lane from the compiler: hoisted out
    // of the loop the LDS addresses alone are more registers than there are)
    int g, n16, q_l, c_l, my_edge, a_row, tr_base, tr_swz;
    auto from_lane = [&]() __attribute__((always_inline)) {
        asm volatile("" : "+v"(lane));
        g = lane >> 4;
        n16 = lane & 15;
        q_l = n16 >> 2;
        c_l = n16 & 3;
        my_edge = 16 * q_l + 4 * g + c_l;
        a_row = ((n16 & 3) << 2) | (n16 >> 2);  // r & 15 of the row whose weights this lane holds (see k_spmm_blocks)
        const int tr_row = 16 * g + (n16 >> 1);
        tr_base = tr_row * SW + (n16 & 1) * 8;
        tr_swz = bw_swz<SW>(tr_row) * 16;
    };
    from_lane();
    const int8_t *X = a.X + col0, *Y = a.att.Xrow + col0;
    int8_t *tile = tile_s[wv];
    int8_t *wl = w_s[wv];
    float s_w, inv_w;
    tango_scale_from_absmax(*a.att.absmax_alpha, s_w, inv_w);
    const float sS = *a.att.sS, sD = *a.att.sD;
    const float sc = s_w * (*a.s_X), sc_dot = (*a.s_X) * (*a.att.s_Xrow);
    const int HP = tango_rec_heads(H);
    const tango_attn_rec *recs = static_cast<const tango_attn_rec *>(a.att.rec) + h0;

    bw_v4i acc[T];
#pragma unroll
    for (int t = 0; t < T; ++t) acc[t] = bw_v4i{0, 0, 0, 0};
    int maxabs = 0;

    int R = c0 == 0 ? 0 : __builtin_amdgcn_readfirstlane(wave_find_row(a.ptr, a.n, c0));
    auto load_row_ends = [&](int r0, int &lo, int &hi) __attribute__((always_inline)) {
        lo = a.ptr[min(r0 + lane, a.n)];
        hi = a.ptr[min(r0 + lane + 1, a.n)];
    };
    int n_idx[GB], n_eid[GB], c_eid[GB];
    auto request = [&](int e0) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < GB; ++k) {
            n_idx[k] = a.idx[min(e0 + 64 * k + lane, last)];
            n_eid[k] = a.eid[min(e0 + 64 * k + my_edge, last)];
        }
    };
    auto hand_over = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < GB; ++k) {
            at_s[wv][64 * k + lane] = static_cast<uint32_t>(n_idx[k]);
            c_eid[k] = n_eid[k];
        }
        bw_lds_fence();
    };
    int held = -1, spans = 0;  // as in k_dot_blocks
    bw_v4i resident[NC];
    uint32_t sq = 0, sq_n = 0;  // S_q of the row of this lane's edge
    bw_v4i rec_n[HS];           // the records of its neighbour
    auto load_resident = [&](int row) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < NC; ++k) {
            resident[k] = bw_v4i{0, 0, 0, 0};
            if (SW >= 64 || g < 2) resident[k] = *reinterpret_cast<const bw_v4i *>(Y + static_cast<int64_t>(row) * a.F + 64 * k + 16 * g);
        }
    };
    auto fetch_rows = [&](int base, int end, int r0, int lo, int hi, int place) __attribute__((always_inline)) {
        const int64_t v = at_s[wv][64 * place + my_edge];
#pragma unroll
        for (int h = 0; h < HS; ++h) rec_n[h] = *reinterpret_cast<const bw_v4i *>(recs + v * HP + h);
        int my_row = r0;
        if (__builtin_amdgcn_readfirstlane(hi) < end) {
            row_s[wv][lane] = 0;
            bw_lds_fence();
            for (int w = r0;;) {
                const int l = max(lo - base, 0), h = min(hi, end) - base;
                if (l < h) row_s[wv][l] = w + lane;
                if (__builtin_amdgcn_readlane(hi, 63) >= end || w + 64 >= a.n) break;
                w += 64;
                load_row_ends(w, lo, hi);
            }
            bw_lds_fence();
            const int row_of = bw_scan_max(row_s[wv][lane]);
            row_s[wv][lane] = row_of;
            bw_lds_fence();
            my_row = row_s[wv][my_edge];
            const int first = row_s[wv][16 * q_l], final = row_s[wv][16 * q_l + 15];
            held = -1;
            spans = 0;
            for (int d = 4; __any(final - first >= d); d += 4) spans = d;
            load_resident(min(first + c_l, final));
        } else if (held == r0) {
            sq_n = sq;
            return;
        } else {
            held = r0;
            spans = 0;
            load_resident(r0);
        }
        sq_n = bw_load_bytes<HS>(a.att.Sq + static_cast<int64_t>(my_row) * H + h0, true);
    };
    int row_lo, row_hi;
    load_row_ends(R, row_lo, row_hi);
    request(c0);
    hand_over();
    fetch_rows(c0, min(c0 + 64, c1), R, row_lo, row_hi, 0);
    bw_gather<SW, BW_ROWS24>(X, &at_s[wv][0], a.F, tile, lane);
    request(c0 + 64 * GB);
    double run[HS];  // dS of the row that fills whole blocks
    int run_row = -1;
#pragma unroll
    for (int h = 0; h < HS; ++h) run[h] = 0.0;
    auto flush_dS = [&]() __attribute__((always_inline)) {
        if (run_row < 0) return;
#pragma unroll
        for (int h = 0; h < HS; ++h) {
            const double t = tango_stride_sum_f64(run[h], 1);
            if (lane == 0 && t != 0.0) atomicAdd(a.att.dS_acc + static_cast<int64_t>(run_row) * H + h0 + h, t);
            run[h] = 0.0;
        }
        run_row = -1;
    };

    for (int base = c0; base < c1; base += 64) {
        from_lane();
        const int cnt = min(64, c1 - base), end = base + cnt;
        const int place = ((base - c0) >> 6) & (GB - 1);
        const bool uniform = held >= 0, there = my_edge < cnt;
        const int block_row = held;
        sq = sq_n;
        // ---- the attention codes of my edge
        double P[HS];
        float al[HS];  // the sign bit says "score not positive"
        {
            const int64_t i0 = static_cast<int64_t>(place == 0 ? c_eid[0] : c_eid[1]) * H + h0;
            uint4 blk = make_uint4(0, 0, 0, 0);
            if (a.att.rounding == TANGO_SR) blk = tango_philox_block(a.att.rng, static_cast<uint64_t>(i0) >> 3);  // (i0 is a multiple of HS)
#pragma unroll
            for (int h = 0; h < HS; ++h) {
                P[h] = __hiloint2double(rec_n[h][1], rec_n[h][0]);
                bool pos;
                const float ev = tango_attn_score(sS * static_cast<float>(static_cast<int8_t>(sq >> (8 * h))), sD * static_cast<float>(rec_n[h][3]),
                                                  a.att.slope, pos);
                const float alpha = tango_attn_alpha(ev, __int_as_float(rec_n[h][2]));
                al[h] = pos ? alpha : -alpha;
                const int q = a.att.rounding == TANGO_SR
                                  ? tango_round_clamp<TANGO_SR>(alpha * inv_w, tango_bits16(blk, static_cast<int>((i0 + h) & 7)))
                                  : tango_round_clamp<TANGO_RN>(alpha * inv_w, 0u);
                wl[64 * h + my_edge] = static_cast<int8_t>(there ? q : 0);
            }
        }
        int nrows = __popcll(__ballot(R + lane < a.n && row_lo < end));
        int nfin = __popcll(__ballot(R + lane < a.n && row_hi <= end));
        const int R_now = R, rows_now = nrows, lo_now = row_lo, hi_now = row_hi;
        int next_lo = row_lo, next_hi = row_hi;
        if (nfin > 0) load_row_ends(R + nfin, next_lo, next_hi);
        __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): the tile has landed
        bw_lds_fence();
        // ---- dalpha of my edge (see k_dot_blocks)
        int dot[HS];
#pragma unroll
        for (int h = 0; h < HS; ++h) dot[h] = 0;
        int4 rows4 = make_int4(0, 0, 0, 0);
        int first = 0, final = 0;
        if (!uniform) {
            rows4 = *reinterpret_cast<const int4 *>(&row_s[wv][16 * q_l + 4 * g]);
            first = row_s[wv][16 * q_l];
            final = row_s[wv][16 * q_l + 15];
        }
        for (int d0 = 0; d0 <= spans; d0 += 4) {
            if (d0 > 0) load_resident(min(first + d0 + c_l, final));
#pragma unroll
            for (int h = 0; h < HS; ++h) {
                bw_v4i res[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) res[q] = bw_v4i{0, 0, 0, 0};
                constexpr int KH = DIM >= 64 ? DIM / 64 : 1;
#pragma unroll
                for (int k = 0; k < KH; ++k) {
                    const int kc = DIM >= 64 ? h * KH + k : h / HPC;
                    bw_v4i b = resident[kc];
                    if (HPC > 1) {
                        const bool mine = (16 * g) / DIM == h % HPC;
#pragma unroll
                        for (int w = 0; w < 4; ++w) b[w] = mine ? b[w] : 0;
                    }
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int r = 16 * q + n16;
                        bw_v4i f = {0, 0, 0, 0};
                        if (SW >= 64 || g < 2) f = *reinterpret_cast<const bw_v4i *>(tile + r * SW + (((4 * kc + g) ^ bw_swz<SW>(r)) * 16));
                        res[q] = __builtin_amdgcn_mfma_i32_16x16x64_i8(f, b, res[q], 0, 0, 0);
                    }
                }
                int v[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = q_l == 0 ? res[0][i] : (q_l == 1 ? res[1][i] : (q_l == 2 ? res[2][i] : res[3][i]));
                if (!uniform) {
                    const int row = first + d0 + c_l;
                    v[0] = rows4.x == row ? v[0] : 0;
                    v[1] = rows4.y == row ? v[1] : 0;
                    v[2] = rows4.z == row ? v[2] : 0;
                    v[3] = rows4.w == row ? v[3] : 0;
#pragma unroll
                    for (int i = 0; i < 4; ++i) v[i] = tango_group_sum_c<4>(v[i], 4);
                }
                dot[h] += c_l == 0 ? v[0] : (c_l == 1 ? v[1] : (c_l == 2 ? v[2] : v[3]));
            }
        }
        // ---- step 4', LeakyReLU' and step 3' for my edge
        if (uniform && run_row != block_row) {
            flush_dS();
            run_row = block_row;
        }
#pragma unroll
        for (int h = 0; h < HS; ++h) {
            const float da = static_cast<float>(dot[h]) * sc_dot;
            const float dE = static_cast<float>(static_cast<double>(fabsf(al[h])) * (static_cast<double>(da) - P[h]));
            const float d = dE * (__float_as_int(al[h]) < 0 ? a.att.slope : 1.0f);
            if (uniform) run[h] += there ? static_cast<double>(d) : 0.0;
            else val_s[wv][h][my_edge] = d;
        }
        // ---- the aggregation (see k_spmm_blocks)
        bw_v4i wf[HS];
#pragma unroll
        for (int h = 0; h < HS; ++h) wf[h] = *reinterpret_cast<const bw_v4i *>(wl + 64 * h + 16 * g);
        for (;;) {
            for (int p = 0; p < nrows; p += 16) {
                bw_v4i wm[HS];
                const int src = p + ((a_row - R) & 15);
                if (nrows == 1 && __builtin_amdgcn_readfirstlane(row_lo) <= base) {
#pragma unroll
                    for (int h = 0; h < HS; ++h)
#pragma unroll
                        for (int k = 0; k < 4; ++k) wm[h][k] = src == 0 ? wf[h][k] : 0;
                } else {
                    uint32_t m[4];
                    const int lo = __shfl(row_lo, src, 64) - base, hi = min(__shfl(row_hi, src, 64) - base, cnt);
                    bw_range_mask(lo, hi, g, m);
#pragma unroll
                    for (int h = 0; h < HS; ++h)
#pragma unroll
                        for (int k = 0; k < 4; ++k) wm[h][k] = wf[h][k] & static_cast<int>(m[k]);
                }
#pragma unroll
                for (int t = 0; t < T; ++t) {
                    const bw_v4i f = bw_columns<SW>(tile, tr_base, tr_swz, t);
                    acc[t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wm[t * HS / T], f, acc[t], 0, 0, 0);
                }
                if (nfin <= p) continue;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int j = p + ((4 * i + g - R) & 15);
                    const bool fin = j < nfin;
                    if (!__any(fin)) continue;
                    const int began = __shfl(row_lo, j, 64);
                    if (fin) {
                        float *orow = a.out + (static_cast<int64_t>(R + j) * a.F + col0 + n16);
                        if (began >= c0) {
#pragma unroll
                            for (int t = 0; t < T; ++t) {
                                orow[16 * t] = static_cast<float>(acc[t][i]) * sc;
                                maxabs = max(maxabs, abs(acc[t][i]));
                            }
                        } else {
#pragma unroll
                            for (int t = 0; t < T; ++t) atomicAdd(reinterpret_cast<int *>(orow) + 16 * t, acc[t][i]);
                        }
#pragma unroll
                        for (int t = 0; t < T; ++t) acc[t][i] = 0;
                    }
                }
            }
            R += nfin;
            row_lo = next_lo;
            row_hi = next_hi;
            if (nfin < 64 || R >= a.n || __builtin_amdgcn_readfirstlane(row_lo) >= end) break;
            nrows = __popcll(__ballot(R + lane < a.n && row_lo < end));
            nfin = __popcll(__ballot(R + lane < a.n && row_hi <= end));
            load_row_ends(R + nfin, next_lo, next_hi);
        }
        // ---- the next block
        if (end < c1) {
            __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): this block's reads of LDS are done
            if (place == GB - 1) hand_over();
            fetch_rows(end, min(end + 64, c1), R, row_lo, row_hi, (place + 1) & (GB - 1));
            bw_gather<SW, BW_ROWS24>(X, &at_s[wv][64 * ((place + 1) & (GB - 1))], a.F, tile, lane);
            if (place == GB - 1) request(end + 64 * GB);
        }
        // ---- step 3' of a block of several rows, while the next gathers are on their way
        if (!uniform) {
            flush_dS();
            bw_lds_fence();
            int w = R_now, nr = rows_now, lo = lo_now, hi = hi_now;
            for (;;) {
                const int items = nr * HS;
                const int log2P = items <= 4 ? 4 : (items <= 8 ? 3 : (items <= 16 ? 2 : (items <= 32 ? 1 : 0)));
                const int Pn = 1 << log2P, part = lane & (Pn - 1);
                for (int it0 = 0; it0 < items; it0 += 64 >> log2P) {
                    const int it = it0 + (lane >> log2P);
                    const int j = min(it / HS, 63), h = it % HS;
                    const int row_b = __shfl(lo, j, 64), row_t = __shfl(hi, j, 64);
                    const int b = max(row_b - base, 0), t = it < items ? min(row_t - base, cnt) : 0;
                    double sum = 0.0;
#pragma unroll 4
                    for (int e = b + part; e < t; e += Pn) sum += static_cast<double>(val_s[wv][h][e]);
                    sum = tango_group_sum_f64(sum, Pn);
                    if (b < t && part == 0 && sum != 0.0) atomicAdd(a.att.dS_acc + static_cast<int64_t>(w + j) * H + h0 + h, sum);
                }
                if (nr < 64 || w + 64 >= a.n) break;
                w += 64;
                load_row_ends(w, lo, hi);
                nr = __popcll(__ballot(w + lane < a.n && lo < end));
                if (nr == 0) break;
            }
            bw_lds_fence();
        }
    }
    flush_dS();
    if (R < a.n) {  // the row that runs on into the next chunk
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (((R >> 2) & 3) != i) continue;
            int *orow = reinterpret_cast<int *>(a.out + (static_cast<int64_t>(R) * a.F + col0 + n16));
#pragma unroll
            for (int t = 0; t < T; ++t)
                if (g == (R & 3) && acc[t][i] != 0) atomicAdd(orow + 16 * t, acc[t][i]);
        }
    }
    if (a.absmax) {
        float m = static_cast<float>(maxabs) * sc;
        m = tango_wave_max(m);
        if (lane == 0 && m > 0.0f) tango_atomic_max_nonneg(a.absmax, m);
    }
}
