// Fused MaxSim forward for gfx950 (Alg. 1 of the paper, re-designed around 64-wide
// wavefronts and the MFMA result layouts).
//
// Orientation.  Document tokens sit on the MFMA rows (A operand), query tokens on the
// columns (B operand).  A lane of a 32x32 result holds ONE query token (column
// lane % 32) and 16 document tokens, so the max over document tokens (the running row-max step of Alg. 1)
// is an in-lane chain of v_max3 over the accumulator registers and the running row-max is
// one register per lane per 32 query tokens.  The two lane halves are merged once per
// document; the sum over query tokens (the final reduction of Alg. 1) is a butterfly over 32 lanes
// (finish_block).  That is the streaming kernels and the tile kernel with argmax on 16-bit inputs.
// Otherwise the tile kernel, and the packed-window kernel, take the same 32 x 32 tokens as four 16x16
// results (Acc16): two query tokens per lane, eight document tokens of each, two running maxima, and
// four lane quarters to merge, two column blocks at a time (finish_blocks16).
//
// Masking (the -inf step of Alg. 1).  Rows past the end of a document are not set to -inf after
// the product; instead the loads clamp the row index to the document's last token.  A
// duplicated token cannot change a max, and it cannot win the argmax because ties go to the
// lowest index, so the result is the same and the epilogue stays mask-free.
//
// The kernels that share these pieces:
//   fwd_stream_lin_kernel, fwd_stream_split_kernel, fwd_stream_kernel
//                      few query tokens: the corpus read is the cost.  A wavefront holds whole queries and
//                      walks its own run of documents (or half of one document's tiles), tiles read one ahead.
//   fwd_tile_kernel    many query tokens: the contraction is the cost.  A workgroup keeps up
//                      to 1024 query tokens stationary in registers (128 per wavefront) and
//                      streams document tiles through LDS, shared by all its wavefronts.
//   fwd_pack_kernel    the same for queries of one column block, over 32-row windows of the packed corpus.
#pragma once
#include "common.h"

#include <type_traits>

namespace maxsim {

// dispatch_tile<fmt(.., 8), true>, compiled in forward_argmax.hip
hipError_t forward_tile_argmax_f16(const FwdParams &p, int w, int num_cu, hipStream_t s);
hipError_t forward_tile_argmax_bf16(const FwdParams &p, int w, int num_cu, hipStream_t s);

namespace {

// ---------------------------------------------------------------------------------------
// pieces shared by the kernels
// ---------------------------------------------------------------------------------------

// Query fragments of column block `gb` (global block id): column rho of the block is query
// token (gb % bpq) * 32 + rho of query gb / bpq; columns past l_q re-read the last token
// and are dropped from the sum later.
template <int DT>
__device__ __forceinline__ void load_q_block(const FwdParams &p, int gb, int rho, int h,
                                             uint4 (&qf)[Traits<DT>::NU], bool &col_valid)
{
    using TR = Traits<DT>;
    int total_blocks = p.n_q * p.bpq;
    bool active = gb < total_blocks;
    int g = active ? gb : 0;
    int q = g / p.bpq;
    int tok = (g % p.bpq) * BLOCK_COLS + rho;
    col_valid = active && tok < p.l_q;
    if (tok > p.l_q - 1)
        tok = p.l_q - 1;
    const char *row = p.Q + ((int64_t)q * p.l_q + tok) * TR::ROW_BYTES + h * 16;
#pragma unroll
    for (int u = 0; u < TR::NU; ++u)
        qf[u] = *reinterpret_cast<const uint4 *>(row + u * 32);
}

// Fold one 32x32 result tile into the running max (and argmax) of this lane's query token.
template <bool ARGMAX>
__device__ __forceinline__ void fold_tile(const f32x16 &acc, float &m, int &idx, int row_base, int h)
{
    if (ARGMAX) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            bool up = acc[r] > m; // strict: the first occurrence keeps a tie
            m = up ? acc[r] : m;
            idx = up ? row_base + acc_row(r, h) : idx;
        }
    } else {
#pragma unroll
        for (int r = 0; r < 16; r += 2)
            m = fmaxf(fmaxf(m, acc[r]), acc[r + 1]); // one v_max3_f32 per pair
    }
}

// Cross-lane helpers on the VALU (no LDS traffic): v_permlane32_swap exchanges the two lane
// halves, DPP row operations add within a row of 16 lanes.
__device__ __forceinline__ void swap_halves(float x, float &lo_from_hi, float &hi_from_lo)
{
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    hi_from_lo = __uint_as_float(r[0]); // lanes 32..63 now hold lanes 0..31 (lanes 0..31 unchanged)
    lo_from_hi = __uint_as_float(r[1]); // lanes 0..31 now hold lanes 32..63 (lanes 32..63 unchanged)
}

template <int CTRL> __device__ __forceinline__ float dpp_add(float v)
{
    return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}

// Sum over lanes 0..31 (a fixed tree: pairs, quads, eights, sixteens, then the two rows).
__device__ __forceinline__ float sum_low32(float v)
{
    v = dpp_add<0xB1>(v);  // quad_perm [1,0,3,2]
    v = dpp_add<0x4E>(v);  // quad_perm [2,3,0,1]
    v = dpp_add<0x141>(v); // row_half_mirror
    v = dpp_add<0x140>(v); // row_mirror
    float r0 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 0));
    float r1 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 16));
    return r0 + r1;
}

// End of a document for one column block: merge the lane halves, write the argmax of valid
// columns, and return the sum over the block's valid query tokens (same value in all lanes).
template <bool ARGMAX>
__device__ __forceinline__ float finish_block(const FwdParams &p, float m, int idx, bool col_valid,
                                              int gb, int64_t doc, int len, int rho, int h)
{
    float a, b; // a: this lane's value or its partner's, so that max(a, b) is the merged value in every lane
    swap_halves(m, a, b);
    if (ARGMAX) {
        float ia, ib;
        swap_halves(__int_as_float(idx), ia, ib);
        // lanes 0..31: (a, ia) came from the upper half, (b, ib) is the lane's own; upper lanes: the reverse
        int i0 = __float_as_int(ia), i1 = __float_as_int(ib);
        bool take = (a > b) || (a == b && i0 < i1);
        m = take ? a : b;
        idx = take ? i0 : i1;
        if (col_valid && h == 0) {
            // the address is formed here, at the end of a document, from an opaque copy of the lane's
            // column: hoisted out of the tile loop its per-lane 64-bit parts would cost registers there
            int col = rho;
            asm volatile("" : "+v"(col));
            int q = gb / p.bpq;
            int tok = (gb % p.bpq) * BLOCK_COLS + col;
            if (idx > len - 1)
                idx = len - 1;
            p.argmax[((int64_t)q * p.ld + doc) * p.l_q + tok] = idx;
        }
    } else {
        m = fmaxf(a, b);
    }
    return sum_low32(col_valid ? m : 0.0f);
}

// The same two for 16x16 results (Acc16): fragment j * NU / 2 + u of a block is chunk 4 u + g of its query token 16 j + c.
template <int DT> __device__ __forceinline__ void load_q_block16(const FwdParams &p, int gb, int lane, uint4 (&qf)[Traits<DT>::NU])
{
    using TR = Traits<DT>;
    constexpr int S = TR::NU / 2;
    const int total_blocks = p.n_q * p.bpq;
    const int b = gb < total_blocks ? gb : 0;
    const int q = b / p.bpq;
    const int tok = (b % p.bpq) * BLOCK_COLS + (lane & 15);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const char *row = p.Q + ((int64_t)q * p.l_q + min(tok + 16 * j, p.l_q - 1)) * TR::ROW_BYTES + (lane >> 4) * 16;
#pragma unroll
        for (int u = 0; u < S; ++u)
            qf[j * S + u] = *reinterpret_cast<const uint4 *>(row + u * 64);
    }
}

// Byte offset of a lane's u-th document fragment in an LDS tile, from the lane's own (row lane % 16, chunk lane / 16)
template <int DT, int STRIDE> __device__ __forceinline__ constexpr int frag_off16(int u)
{
    constexpr int S = Traits<DT>::NU / 2;
    return u / S * 16 * STRIDE + u % S * 64;
}

// End of a document for NCB column blocks of a wavefront.  m[b] are the lane's maxima for the columns c and 16 + c of block
// b, found in its quarter of the rows.  One swap brings a block's two columns together and merges two quarters, one
// between the blocks 2 k and 2 k + 1 the other two, and the lane then holds column 16 (lane / 32) + c of block
// 2 k + lane / 16 % 2: the sum over columns (the tree of sum_low32) serves two blocks at a time.  A block by itself is some
// thirty dependent instructions, which at four blocks and documents of 180 tokens kept a wavefront busy for a sixth of
// its time.  Returns the sum of block lane / 16 (of lane / 16 % 2 if NCB is 1 or 2).  valid[k]: the column counts.
constexpr int finish_pairs(int ncb) { return (ncb + 1) / 2; }
template <int NCB, bool ARGMAX>
__device__ __forceinline__ float finish_blocks16(const FwdParams &p, const float (&m)[NCB][2], const int (&row)[NCB][2],
                                                 const bool (&valid)[finish_pairs(NCB)], int gb, int64_t doc, int len, int lane)
{
    auto merge = [](auto v, auto i, int &win) {
        const float a = __uint_as_float(v[0]), b = __uint_as_float(v[1]);
        if (ARGMAX) {
            const bool take = a > b || (a == b && (int)i[0] < (int)i[1]);
            win = take ? (int)i[0] : (int)i[1];
            return take ? a : b;
        }
        return fmaxf(a, b);
    };
    float v[finish_pairs(NCB)];
#pragma unroll
    for (int k = 0; k < finish_pairs(NCB); ++k) {
        float x[2];
        int r[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            if (2 * k + e >= NCB) { // an odd last block stands in for its neighbour
                x[e] = x[0];
                r[e] = r[0];
                continue;
            }
            const int b = 2 * k + e;
            x[e] = merge(__builtin_amdgcn_permlane32_swap(__float_as_uint(m[b][0]), __float_as_uint(m[b][1]), false, false),
                         __builtin_amdgcn_permlane32_swap((uint32_t)row[b][0], (uint32_t)row[b][1], false, false), r[e]);
        }
        int win;
        const float best = merge(__builtin_amdgcn_permlane16_swap(__float_as_uint(x[0]), __float_as_uint(x[1]), false, false),
                                 __builtin_amdgcn_permlane16_swap((uint32_t)r[0], (uint32_t)r[1], false, false), win);
        if (ARGMAX && valid[k] && (2 * k + 1 < NCB || (lane & 16) == 0)) {
            int col = ((lane >> 5) << 4) + (lane & 15); // (an opaque copy, as in finish_block)
            asm volatile("" : "+v"(col));
            auto at = [&](int b) { return ((int64_t)(b / p.bpq) * p.ld + doc) * p.l_q + (b % p.bpq) * BLOCK_COLS; };
            p.argmax[((lane & 16) ? at(gb + 2 * k + 1) : at(gb + 2 * k)) + col] = min(win, len - 1);
        }
        v[k] = valid[k] ? best : 0.0f;
        v[k] = dpp_add<0xB1>(v[k]);
        v[k] = dpp_add<0x4E>(v[k]);
        v[k] = dpp_add<0x141>(v[k]);
        v[k] = dpp_add<0x140>(v[k]);
    }
    const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[0]), __float_as_uint(v[finish_pairs(NCB) - 1]), false, false);
    return __uint_as_float(s[0]) + __uint_as_float(s[1]);
}

// Documents of length 0 in [doc0, doc1): score -inf, argmax -1 (ragged corpora only).
__device__ __forceinline__ void write_empty_docs(const FwdParams &p, int64_t doc0, int64_t doc1,
                                                 int tid, int nthreads)
{
    if (!p.offsets)
        return;
    for (int64_t doc = doc0 + tid; doc < doc1; doc += nthreads) {
        if (p.offsets[doc + 1] != p.offsets[doc])
            continue;
        for (int q = 0; q < p.n_q; ++q) {
            p.scores[(int64_t)q * p.ld + doc] = neg_inf();
            if (p.argmax)
                for (int i = 0; i < p.l_q; ++i)
                    p.argmax[((int64_t)q * p.ld + doc) * p.l_q + i] = -1;
        }
    }
}

// ---------------------------------------------------------------------------------------
// streaming kernel: one wavefront per run of documents, all query blocks in registers
// ---------------------------------------------------------------------------------------

template <int DT, int NCB, bool ARGMAX> struct StreamState {
    uint4 qf[NCB][Traits<DT>::NU];
    bool col_valid[NCB];
    float m[NCB];
    int idx[NCB];
};

// The position of a tile: first packed row of its document, the document's length, first row of the tile
struct TilePos {
    int64_t start;
    int32_t len, t0;
};

template <int DT>
__device__ __forceinline__ void stream_load_tile(const FwdParams &p, const TilePos &c, int rho, int h,
                                                 uint4 (&a)[Traits<DT>::NU])
{
    using TR = Traits<DT>;
    int row = c.t0 + rho;
    if (row > c.len - 1)
        row = c.len - 1;
    const char *ptr = p.D + (c.start + row) * TR::ROW_BYTES + h * 16;
#pragma unroll
    for (int u = 0; u < TR::NU; ++u)
        a[u] = *reinterpret_cast<const uint4 *>(ptr + u * 32);
}

// One tile (operands `a`, first row t0 of its document) against the wavefront's column blocks
template <int DT, int NCB, bool ARGMAX>
__device__ __forceinline__ void stream_tile(StreamState<DT, NCB, ARGMAX> &st, const uint4 (&a)[Traits<DT>::NU], int t0, int h)
{
    using TR = Traits<DT>;
    // two column blocks at a time (two accumulator chains in flight); the scheduling barrier keeps
    // the pairs apart so that only two accumulators are live and more wavefronts fit on a SIMD
#pragma unroll
    for (int cb = 0; cb < NCB; cb += 2) {
        f32x16 acc0, acc1;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            acc0[r] = 0.0f;
            acc1[r] = 0.0f;
        }
#pragma unroll
        for (int u = 0; u < TR::NU; ++u) {
            TR::mma(a[u], st.qf[cb][u], acc0);
            if (cb + 1 < NCB)
                TR::mma(a[u], st.qf[cb + 1][u], acc1);
        }
        fold_tile<ARGMAX>(acc0, st.m[cb], st.idx[cb], t0, h);
        if (cb + 1 < NCB)
            fold_tile<ARGMAX>(acc1, st.m[cb + 1], st.idx[cb + 1], t0, h);
        if (cb + 2 < NCB)
            __builtin_amdgcn_sched_barrier(0);
    }
}

template <int DT, int NCB, bool ARGMAX> __device__ __forceinline__ void stream_reset(StreamState<DT, NCB, ARGMAX> &st)
{
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
        st.m[cb] = neg_inf();
        st.idx[cb] = 0;
    }
}

// End of a document: scores (and argmax) of the wavefront's queries
template <int DT, int NCB, bool ARGMAX>
__device__ __forceinline__ void stream_finish(const FwdParams &p, StreamState<DT, NCB, ARGMAX> &st, int gb0, int64_t doc, int len,
                                              int lane, int rho, int h)
{
    float part[NCB];
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb)
        part[cb] = finish_block<ARGMAX>(p, st.m[cb], st.idx[cb], st.col_valid[cb], gb0 + cb, doc, len, rho, h);
    // the wavefront holds whole queries: lane k adds up the blocks of its k-th query in block
    // order and writes the score
    float s = 0.0f;
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb)
        if (cb / p.bpq == lane)
            s += part[cb];
    const int q = gb0 / p.bpq + lane;
    if (lane < NCB / p.bpq && q < p.n_q)
        p.scores[(int64_t)q * p.ld + doc] = s;
}

template <int DT, int NCB, bool ARGMAX>
__device__ __forceinline__ void stream_compute(const FwdParams &p, const Cursor &c,
                                               StreamState<DT, NCB, ARGMAX> &st,
                                               const uint4 (&a)[Traits<DT>::NU], int gb0, int lane, int rho, int h)
{
    if (c.t0 == 0)
        stream_reset(st);
    stream_tile(st, a, c.t0, h);
    if (c.t0 + TILE_ROWS >= c.len) // last tile of the document
        stream_finish(p, st, gb0, c.doc, c.len, lane, rho, h);
}

template <int DT, int NCB, bool ARGMAX>
__global__ void __launch_bounds__(256) fwd_stream_kernel(FwdParams p, OffsetsPtr off)
{
    using TR = Traits<DT>;
    const int lane = threadIdx.x & 63;
    const int rho = lane & 31, h = lane >> 5;
    // p.n_groups (1, 2 or 4) wavefronts of a workgroup share a run of documents, each with its own
    // NCB column blocks (whole queries); they read the same tiles at about the same time, so all
    // but the first read hit in the CU's vector cache.  No LDS and no barrier is involved.
    const int wib = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int group = wib % p.n_groups;
    const int64_t chunk = (int64_t)blockIdx.x * (4 / p.n_groups) + wib / p.n_groups;
    const int gb0 = group * NCB;
    int64_t doc0, doc1;
    chunk_doc_range(p, chunk, doc0, doc1);
    if (doc0 >= doc1)
        return;
    if (group == 0)
        write_empty_docs(p, doc0, doc1, lane, 64);

    StreamState<DT, NCB, ARGMAX> st;
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb)
        load_q_block<DT>(p, gb0 + cb, rho, h, st.qf[cb], st.col_valid[cb]);

    Cursor pc; // prefetch cursor, one tile ahead of the compute cursor
    cursor_init(pc, p, off, doc0, doc1);
    if (!pc.valid)
        return;
    uint4 a0[TR::NU], a1[TR::NU];
    TilePos lp = {pc.start, pc.len, pc.t0}; // where the prefetch reads: pc while it is valid, else the last valid tile
    auto follow = [&]() { // (field by field: a select between whole cursors would put them into memory)
        lp.start = pc.valid ? pc.start : lp.start;
        lp.len = pc.valid ? pc.len : lp.len;
        lp.t0 = pc.valid ? pc.t0 : lp.t0;
    };
    stream_load_tile<DT>(p, lp, rho, h, a0);
    Cursor cc = pc;
    // The prefetch is issued without a condition: past the end of the run the last tile is loaded once more
    // (in bounds, never used).  With `if (pc.valid)` around the loads the compiler has to assume, where the two
    // paths meet, that no load was issued, and makes every MFMA wait for the tile that was only just requested.
    cursor_next_tile(pc, p, off);
    for (;;) {
        follow();
        stream_load_tile<DT>(p, lp, rho, h, a1);
        stream_compute<DT, NCB, ARGMAX>(p, cc, st, a0, gb0, lane, rho, h);
        cc = pc;
        if (!cc.valid)
            break;
        cursor_next_tile(pc, p, off);
        follow();
        stream_load_tile<DT>(p, lp, rho, h, a0);
        stream_compute<DT, NCB, ARGMAX>(p, cc, st, a1, gb0, lane, rho, h);
        cc = pc;
        if (!cc.valid)
            break;
        cursor_next_tile(pc, p, off);
    }
}

// ---------------------------------------------------------------------------------------
// tile kernel: query-stationary workgroup, document tiles staged through LDS
// ---------------------------------------------------------------------------------------

template <int DT> struct LdsTile {
    // rows padded by one 16-byte chunk so that the 32 rows read by one ds_read_b128 of the
    // MFMA operand layout fall into different banks
    static constexpr int ROW_STRIDE = Traits<DT>::ROW_BYTES + 16;
    static constexpr int BYTES = TILE_ROWS * ROW_STRIDE;
    static constexpr int CHUNKS = TILE_ROWS * Traits<DT>::ROW_BYTES / 16;
};

// The streaming kernel with whole-line loads (one wavefront per run, rows of up to 256 bytes).  A tile of 32
// consecutive rows is one contiguous piece of memory: the wavefront reads it with NU instructions of 1 KB each
// (lane l the l-th 16 bytes: sixteen or eight lanes per row), with the non-temporal hint, parks it in its own
// piece of LDS (padded rows, no barrier: nobody else touches it) and reads it back in MFMA operand layout.  The
// direct loads of fwd_stream_kernel take 32 bytes of each of 32 lines per instruction and cannot carry the hint;
// a read stream of this shape measures 6.8 TB/s with it and 6.0 without.
template <int DT> constexpr int lin_waves() { return Traits<DT>::NU <= 8 ? 4 : 2; } // wavefronts per workgroup (LDS tiles of 4 to 17 KB)

template <int DT, int NCB, bool ARGMAX>
__global__ void __launch_bounds__(lin_waves<DT>() * 64) fwd_stream_lin_kernel(FwdParams p, OffsetsPtr off)
{
    using TR = Traits<DT>;
    using LT = LdsTile<DT>;
    constexpr int NU = TR::NU;
    constexpr int WPB = lin_waves<DT>();
    constexpr int CPR = TR::ROW_BYTES / 16; // 16-byte chunks (= lanes) per row
    constexpr int RPI = 64 / CPR;           // rows per load instruction
    static_assert(CPR <= 64 && RPI * NU == TILE_ROWS, "NU instructions of 64 lanes cover a tile");
    __shared__ __attribute__((aligned(16))) char lds_all[WPB][LT::BYTES];
    const int lane = threadIdx.x & 63;
    const int rho = lane & 31, h = lane >> 5;
    const int wib = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    char *lds = lds_all[wib];
    const int64_t chunk = (int64_t)blockIdx.x * WPB + wib;
    const int gb0 = 0;
    int64_t doc0, doc1;
    chunk_doc_range(p, chunk, doc0, doc1);
    if (doc0 >= doc1)
        return;
    write_empty_docs(p, doc0, doc1, lane, 64);

    StreamState<DT, NCB, ARGMAX> st;
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb)
        load_q_block<DT>(p, gb0 + cb, rho, h, st.qf[cb], st.col_valid[cb]);

    Cursor pc; // prefetch cursor, one tile ahead of the compute cursor
    cursor_init(pc, p, off, doc0, doc1);
    if (!pc.valid)
        return;
    TilePos lp = {pc.start, pc.len, pc.t0}; // where the prefetch reads: pc while it is valid, else the last valid tile
    auto follow = [&]() {
        lp.start = pc.valid ? pc.start : lp.start;
        lp.len = pc.valid ? pc.len : lp.len;
        lp.t0 = pc.valid ? pc.t0 : lp.t0;
    };
    const int lrow = lane / CPR, lcol = (lane % CPR) * 16;
    const int st_off = lrow * LT::ROW_STRIDE + lcol;
    const int rd_off = rho * LT::ROW_STRIDE + h * 16;
    uint4 g[NU], a[NU];
    auto load_lin = [&]() { // rows past the document's end repeat its last token
#pragma unroll
        for (int i = 0; i < NU; ++i) {
            int row = lp.t0 + i * RPI + lrow;
            if (row > lp.len - 1)
                row = lp.len - 1;
            g[i] = load_stream16(p.D + (lp.start + row) * TR::ROW_BYTES + lcol);
        }
    };
    load_lin();
    Cursor cc = pc;
    cursor_next_tile(pc, p, off);
    for (;;) {
#pragma unroll
        for (int i = 0; i < NU; ++i)
            *reinterpret_cast<uint4 *>(&lds[st_off + i * RPI * LT::ROW_STRIDE]) = g[i];
        follow();
        load_lin(); // the next tile (past the end of the run: the last one again, in bounds, never used)
#pragma unroll
        for (int u = 0; u < NU; ++u)
            a[u] = *reinterpret_cast<const uint4 *>(&lds[rd_off + u * 32]);
        stream_compute<DT, NCB, ARGMAX>(p, cc, st, a, gb0, lane, rho, h);
        cc = pc;
        if (!cc.valid)
            break;
        cursor_next_tile(pc, p, off);
    }
}

// The streaming kernel for corpora of up to some thousand documents: a workgroup of W wavefronts per document, each
// taking every W-th tile.  With a thousand documents a run of one document per wavefront is a chain of memory round
// trips on a chip that is mostly idle (and the runs of a ragged corpus, equal in tokens, hold up to three documents);
// here more wavefronts have a shorter chain, and nothing is searched for, since a workgroup's document
// is its number.  At the end of a document the sets of maxima (and winners) meet in LDS, lane by lane, and the first
// wavefront finishes it.  A maximum does not depend on how the tiles were shared out, and of equal ones the lower row
// wins, so scores and winners are those of the other kernels.  Two wavefronts; four were no faster (they
// read the queries twice as often): ragged fp16 texts of 64-300 tokens, four queries, 1000 / 4000 documents: 20.8 /
// 52.9 us one wavefront per run, 17.6 / 42.5 here, 18.7 / 46.1 with four; fp32, one query, 1000 x 128 tokens with
// winners: 24.0 -> 18.5 us.
//
// With many queries on few documents (few_documents in forward.hip; there one to four wavefronts) a document has a workgroup
// per column group of NCB blocks: latency and start-up bound it, 16 queries x 16 documents of 128 / 1024 tokens take 4.2 / 8.6 us
// where a workgroup of fwd_tile_kernel per document takes 10.0 / 32.7.
template <int DT, int NCB, bool ARGMAX, int W, bool GROUPS>
__global__ void __launch_bounds__(W * 64) fwd_stream_split_kernel(FwdParams p, OffsetsPtr off)
{
    using TR = Traits<DT>;
    using LT = LdsTile<DT>;
    constexpr int NU = TR::NU;
    constexpr int CPR = TR::ROW_BYTES / 16; // 16-byte chunks (= lanes) per row
    constexpr int RPI = 64 / CPR;           // rows per load instruction
    static_assert((ARGMAX ? 2 : 1) * NCB * 64 * 4 <= LT::BYTES, "a wavefront's maxima fit in its tile");
    __shared__ __attribute__((aligned(16))) char lds_all[W][LT::BYTES];
    const int lane = threadIdx.x & 63;
    const int rho = lane & 31, h = lane >> 5;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    char *lds = lds_all[w];

    int group = 0, first = (int)blockIdx.x, step = (int)gridDim.x;
    if (GROUPS) { // a document's column groups are neighbours on one XCD
        const int v = xcd_grouped(blockIdx.x, gridDim.x);
        group = v % p.n_groups;
        first = v / p.n_groups;
        step = (int)gridDim.x / p.n_groups;
    }
    const int gb0 = group * NCB; // (whole queries)
    StreamState<DT, NCB, ARGMAX> st;
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb)
        load_q_block<DT>(p, gb0 + cb, rho, h, st.qf[cb], st.col_valid[cb]);

    const int lrow = lane / CPR, lcol = (lane % CPR) * 16;
    const int st_off = lrow * LT::ROW_STRIDE + lcol;
    const int rd_off = rho * LT::ROW_STRIDE + h * 16;
    for (int doc = first; doc < p.b; doc += step) {
        int64_t start;
        int len;
        if (p.offsets) {
            start = clamp_offset(off[doc], 0, p.total_tokens);
            len = (int)(clamp_offset(off[doc + 1], start, p.total_tokens) - start);
        } else {
            start = (int64_t)doc * p.l_d;
            len = p.l_d;
        }
        if (len <= 0) {
            if (group == 0)
                write_empty_docs(p, doc, doc + 1, threadIdx.x, W * 64);
            continue;
        }
        const char *base = p.D + start * TR::ROW_BYTES + lcol;
        uint4 g[NU], a[NU];
        auto load_lin = [&](int t0) { // rows past the document's end repeat its last token
#pragma unroll
            for (int i = 0; i < NU; ++i) {
                const int row = min(t0 + i * RPI + lrow, len - 1);
                g[i] = load_stream16(base + (int64_t)row * TR::ROW_BYTES);
            }
        };
        stream_reset(st);
        int t0 = w * TILE_ROWS;
        if (t0 < len) {
            load_lin(t0);
            for (;;) {
#pragma unroll
                for (int i = 0; i < NU; ++i)
                    *reinterpret_cast<uint4 *>(&lds[st_off + i * RPI * LT::ROW_STRIDE]) = g[i];
                const int next = t0 + W * TILE_ROWS;
                if (next < len)
                    load_lin(next);
#pragma unroll
                for (int u = 0; u < NU; ++u)
                    a[u] = *reinterpret_cast<const uint4 *>(&lds[rd_off + u * 32]);
                stream_tile(st, a, t0, h);
                if (next >= len)
                    break;
                t0 = next;
            }
        }
        // the maxima take the place of the wavefront's own tile
        float *mine = reinterpret_cast<float *>(lds);
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) {
            mine[cb * 64 + lane] = st.m[cb];
            if (ARGMAX)
                mine[(NCB + cb) * 64 + lane] = __int_as_float(st.idx[cb]);
        }
        __syncthreads();
        if (w == 0) {
#pragma unroll
            for (int x = 1; x < W; ++x) {
                const float *other = reinterpret_cast<const float *>(lds_all[x]);
#pragma unroll
                for (int cb = 0; cb < NCB; ++cb) {
                    const float mo = other[cb * 64 + lane];
                    if (ARGMAX) {
                        const int io = __float_as_int(other[(NCB + cb) * 64 + lane]);
                        const bool take = mo > st.m[cb] || (mo == st.m[cb] && io < st.idx[cb]);
                        st.idx[cb] = take ? io : st.idx[cb];
                    }
                    st.m[cb] = fmaxf(st.m[cb], mo);
                }
            }
            stream_finish(p, st, gb0, doc, len, lane, rho, h);
        }
        __syncthreads(); // the tiles are overwritten by the next document
    }
}

// The same for fp32 rows of 512 bytes and queries of one or two column blocks.  A tile takes a wavefront's matrix core 1.7 us,
// so the even use of the SIMDs counts: W * C wavefronts share a document, wavefront (x, c) takes every W-th tile against column
// block c, and G documents share a workgroup: the four wavefronts of a workgroup go to the four SIMDs of a CU, where
// workgroups of one or two may meet on one SIMD while others idle (the dispatcher's turn at the launch decides: one query
// x 1000 x 128 right behind a kernel that writes, three documents on one SIMD, 26.2 us, in workgroups of four 20.8).  Operands come
// from LDS chunk by chunk, which leaves the registers of a tile in flight.  What bounds it: the chain of
// a document's tiles (6.8 us of MFMAs for 128 tokens) behind a launch and two loads; two tiles in flight were 5-15 % slower.
template <bool ARGMAX, int W, int C, int G>
__global__ void __launch_bounds__(G * W * C * 64, 2) fwd_f32_split_kernel(FwdParams p, OffsetsPtr off)
{
    constexpr int F = fmt(MAXSIM_F32, 16);
    using TR = Traits<F>;
    using LT = LdsTile<F>;
    constexpr int NU = TR::NU;
    constexpr int CPR = TR::ROW_BYTES / 16; // 16-byte chunks (= lanes) per row
    constexpr int RPI = 64 / CPR;           // rows per load instruction
    __shared__ __attribute__((aligned(16))) char lds_all[G * W * C][LT::BYTES];
    __shared__ float part[G][C];
    const int lane = threadIdx.x & 63;
    const int rho = lane & 31, h = lane >> 5;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int sub = w / (W * C), x = w / C % W, c = w % C;
    char *lds = lds_all[w];

    uint4 qf[NU];
    bool col_valid;
    load_q_block<F>(p, c, rho, h, qf, col_valid);
    const int lrow = lane / CPR, lcol = (lane % CPR) * 16;
    const int st_off = lrow * LT::ROW_STRIDE + lcol;
    const int rd_off = rho * LT::ROW_STRIDE + h * 16;
    auto document = [&](int doc) {
        int64_t start = 0;
        int len = 0;
        if (G == 1 || doc < p.b) {
            if (p.offsets) {
                start = clamp_offset(off[doc], 0, p.total_tokens);
                len = (int)(clamp_offset(off[doc + 1], start, p.total_tokens) - start);
            } else {
                start = (int64_t)doc * p.l_d;
                len = p.l_d;
            }
            if (len <= 0)
                write_empty_docs(p, doc, doc + 1, (int)threadIdx.x - sub * (W * C * 64), W * C * 64);
        }
        // (where documents meet in barriers, those of the workgroup's other documents are kept)
        constexpr bool LEAVE = G == 1 || W * C == 1;
        if (LEAVE && len <= 0)
            return;
        const char *base = p.D + start * TR::ROW_BYTES + lcol;
        uint4 g[NU];
        auto load_lin = [&](int t0) { // rows past the document's end repeat its last token
#pragma unroll
            for (int i = 0; i < NU; ++i) {
                const int row = min(t0 + i * RPI + lrow, len - 1);
                g[i] = load_stream16(base + (int64_t)row * TR::ROW_BYTES);
            }
        };
        float m = neg_inf();
        int idx = 0;
        int t0 = x * TILE_ROWS;
        if (t0 < len) {
            load_lin(t0);
            for (;;) {
#pragma unroll
                for (int i = 0; i < NU; ++i)
                    *reinterpret_cast<uint4 *>(&lds[st_off + i * RPI * LT::ROW_STRIDE]) = g[i];
                const int next = t0 + W * TILE_ROWS;
                if (next < len)
                    load_lin(next);
                uint4 a[4]; // (a ring: three chunks ahead)
                auto read = [&](int u) { a[u & 3] = *reinterpret_cast<const uint4 *>(&lds[rd_off + u * 32]); };
                f32x16 acc;
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    acc[r] = 0.0f;
                read(0);
                read(1);
                read(2);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int u = 0; u < NU; ++u) {
                    if (u + 3 < NU)
                        read(u + 3);
                    TR::mma(a[u & 3], qf[u], acc);
                    __builtin_amdgcn_sched_barrier(0);
                }
                fold_tile<ARGMAX>(acc, m, idx, t0, h);
                if (next >= len)
                    break;
                t0 = next;
            }
        }
        if constexpr (W > 1) { // the maxima take the place of the wavefront's own tile
            float *mine = reinterpret_cast<float *>(lds);
            mine[lane] = m;
            mine[64 + lane] = __int_as_float(idx);
            __syncthreads();
            if (x == 0) {
#pragma unroll
                for (int y = 1; y < W; ++y) {
                    const float *other = reinterpret_cast<const float *>(lds_all[(sub * W + y) * C + c]);
                    const float mo = other[lane];
                    if (ARGMAX) {
                        const int io = __float_as_int(other[64 + lane]);
                        const bool take = mo > m || (mo == m && io < idx); // of equal maxima the lower row
                        idx = take ? io : idx;
                    }
                    m = fmaxf(m, mo);
                }
            }
        }
        if (x == 0 && (LEAVE || len > 0)) {
            const float sum = finish_block<ARGMAX>(p, m, idx, col_valid, c, doc, len, rho, h);
            if (C == 1 || p.bpq == 1) {
                if (lane == 0 && c / p.bpq < p.n_q)
                    p.scores[(int64_t)c * p.ld + doc] = sum;
            } else if (lane == 0) {
                part[sub][c] = sum;
            }
        }
        if constexpr (C == 2) {
            __syncthreads();
            if (p.bpq == 2 && x == 0 && c == 0 && lane == 0 && (LEAVE || len > 0))
                p.scores[doc] = part[sub][0] + part[sub][1];
        }
    };
    const int doc = (int)blockIdx.x * G + sub;
    if constexpr (G > 1 && W * C == 1) // (once; but as a loop the first tiles are asked for a little later, and 1000 x 128 from the caches take 17.2 and not 17.8 us)
        for (int j = doc; j < p.b; j += (int)gridDim.x * G)
            document(j);
    else
        document(doc);
}

// Folds of 16x16 results.  The two cells a v_max3 takes at a time are pair k = 0 .. 7 of an Acc16: result (i, j) =
// (k / 4, k / 2 % 2), registers 2 (k % 2) and the next; a lane's rows grow with k for either j.
//
// Pairs [k0, k1) into the two running maxima.  With ARGMAX (fp32) the winner is kept as a key, the tile's first row (a
// multiple of 32) | 7 - v, v = 4 i + r, and turned into a row at the end of the document.
template <bool ARGMAX>
__device__ __forceinline__ void fold_pairs16(const Acc16 &acc, int k0, int k1, float (&m)[2], int (&key)[2], int row_base)
{
#pragma unroll
    for (int k = k0; k < k1; ++k) {
        const int i = k >> 2, j = (k >> 1) & 1, r = (k & 1) * 2;
        const float x = acc.t[i][j][r], y = acc.t[i][j][r + 1];
        if (ARGMAX) {
            bool up = x > m[j]; // strict: the first occurrence keeps a tie
            m[j] = up ? x : m[j];
            key[j] = up ? (row_base | (7 - 4 * i - r)) : key[j];
            up = y > m[j];
            m[j] = up ? y : m[j];
            key[j] = up ? (row_base | (6 - 4 * i - r)) : key[j];
        } else {
            m[j] = fmaxf(fmaxf(m[j], x), y); // one v_max3_f32
        }
    }
}

// What is folded at step u (of NU) of a column block's chains: the half (i) of four pairs that the chains finished
// last, i.e. half 0 of the block itself during its second half and half 1 of the block before during its first.  Two
// halves of accumulators are live instead of two blocks.  The half's first step folds nothing, so that the MFMAs which
// produced the results have left the matrix pipeline before they are read (no wait states).
template <int NU> __device__ __forceinline__ constexpr int half_pair(int u) // first pair folded at step u (u < NU / 2), four in all
{
    constexpr int S = NU / 2;
    return u < 1 ? 0 : 4 * (u - 1) / (S - 1);
}

// The fold with argmax for 16-bit inputs (the running maximum is an fp32 sum of 128 products).  Compare-and-select
// per cell is three VALU operations against half an operation for the plain maximum, which makes the argmax
// variant VALU-bound.  Here every cell's low four mantissa bits are replaced by 15 - r (r = the accumulator
// register, which grows with the row), one operation per cell, and the tile's maximum is again a v_max3 chain:
// among cells that agree in the upper 28 bits the lowest row wins.  Once per tile and column block the tile's
// maximum, with those four bits cleared, is compared (strictly: an earlier tile keeps a tie) with the running one
// and the row is read back from the four bits.  Consequences: the maxima that enter the score are truncated by at
// most 2^-19 relative (the score tolerance is 2e-3); cells closer than that to each other count as tied and the
// earlier one wins (the argmax rule asks for the exact winner only where the margin exceeds 1e-3).  The ordering
// of the patched values is right among non-negative cells only, which is all that matters once the running
// maximum is non-negative (a negative cell cannot beat it); if any lane of the wavefront has a negative tile
// maximum while its running maximum is still negative, that tile is folded again, exactly, with compare-and-select
// (the first tiles of a document whose similarities with a query token are all negative).  The same exact fold
// takes every tile in which a lane's maximum reaches 512 in magnitude: above that, 2^-19 relative would no longer be
// inside the 1e-3 margin below which the argmax rule lets near-ties go either way.  The running winner is
// kept as a key, the tile's first row (a multiple of 32) | the four bits, and turned into a row at the end of the
// document.
template <int NU>
__device__ __forceinline__ void fold_step_packed(const f32x16 &acc, int u, float &tmax, float &m, int &key, int row_base)
{
    constexpr int LAG = NU >= 4 ? 2 : NU / 2;
    if (u < LAG)
        return;
    const int lo = 2 * (8 * (u - LAG) / (NU - LAG)), hi = 2 * (8 * (u - LAG + 1) / (NU - LAG));
    if (u == LAG)
        tmax = neg_inf();
#pragma unroll
    for (int r = lo; r < hi; r += 2) {
        const float p0 = __uint_as_float((__float_as_uint(acc[r]) & 0xfffffff0u) | (uint32_t)(15 - r));
        const float p1 = __uint_as_float((__float_as_uint(acc[r + 1]) & 0xfffffff0u) | (uint32_t)(14 - r));
        tmax = fmaxf(fmaxf(tmax, p0), p1); // one v_max3_f32
    }
    if (u == NU - 1) {
        const uint32_t tb = __float_as_uint(tmax);
        // one unsigned compare finds the tiles that MAY need the exact fold (a negative maximum has the sign bit set);
        // the precise condition is looked at only then
        bool exact = false;
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(tb >= 0x44000000u /* 512.0f */) != 0, 0))
            exact = __builtin_amdgcn_ballot_w64(((int)tb < 0 && m < 0.0f) || fabsf(tmax) >= 512.0f) != 0;
        if (exact) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const bool up = acc[r] > m; // strict: the first occurrence keeps a tie
                m = up ? acc[r] : m;
                key = up ? (row_base | (15 - r)) : key;
            }
        } else {
            const float ts = __uint_as_float(tb & 0xfffffff0u);
            const bool up = ts > m;
            m = up ? ts : m;
            key = up ? (int)((tb & 15u) | (uint32_t)row_base) : key;
        }
    }
}

// The document-local row behind a key of fold_step_packed in lane half h
__device__ __forceinline__ int packed_key_row(int key, int h)
{
    const int r = 15 - (key & 15);
    return (key & ~31) + h * 4 + (((r & 12) << 1) | (r & 3));
}

// The document-local row behind a key in lane quarter g
__device__ __forceinline__ int key_row16(int key, int g)
{
    const int v = 7 - (key & 7);
    return (key & ~31) + ((v & 4) << 2) + g * 4 + (v & 3);
}
constexpr int KEY_START = 7; // row 0 of the document's first tile

// The main loop is software-pipelined by hand and pinned with scheduling barriers, one operand chunk per step (with
// 16-bit inputs one 32x32 MFMA or two 16x16 ones):
//   * the VALU work of the folds sits under MFMAs whose results it does not need, a slice per step: under the chains of
//     column block cb the previous block's 32x32 result is folded; of 16x16 results the half that was finished last
//     (half_pair: the previous block's second under the block's first, the block's own first under its second);
//   * during the first chain of a tile the wavefront also reads the NEXT tile's A operands from
//     LDS into a second register set, writes the tile after that from registers to LDS and
//     issues the global loads of the tile after that: three LDS buffers rotate (being computed / prefetched
//     into registers / being written), one barrier per tile.  (The argmax variants, 512-byte rows and two
//     wavefronts with four blocks have no registers left for the second operand set; there each operand chunk is
//     replaced by the next tile's right after its last MFMA, during the last chain of the tile.)
//   * with two or three column blocks per wavefront a tile takes too little time for a load issued
//     one tile ahead to have arrived: PFD tiles are then on their way in a ring of registers.  (Less than that
//     in the code: the ring's registers move from slot to slot, and before a move the compiler waits for the load;
//     four wavefronts with two blocks without argmax wait for all of them every second tile.)
template <int DT, int W, int NCB, bool ARGMAX, int PFD = 1>
__global__ void __launch_bounds__(W * 64, Traits<DT>::NU <= 8 ? 2 : 1) fwd_tile_kernel(FwdParams p, OffsetsPtr off)
{
    using TR = Traits<DT>;
    using LT = LdsTile<DT>;
    constexpr int NU = TR::NU;
    constexpr int NT = W * 64;
    constexpr int CPT = (LT::CHUNKS + NT - 1) / NT; // 16-byte chunks each thread moves per tile
    static_assert(LT::CHUNKS % NT == 0 || LT::CHUNKS < NT, "tile must split evenly over the workgroup");
    const bool copies = LT::CHUNKS >= NT || (int)threadIdx.x < LT::CHUNKS; // narrow rows: fewer chunks than threads
    constexpr int CPR = TR::ROW_BYTES / 16; // chunks per row
    constexpr int GROUP_BLOCKS = W * NCB;
    constexpr bool PF = NU <= 8 && !ARGMAX && !(W <= 2 && NCB == 4); // operands of the next tile prefetched into registers (no room for them beside four chunks in flight per thread)

    __shared__ __attribute__((aligned(16))) char lds_tile[3 * LT::BYTES];
    __shared__ float lds_part[2][GROUP_BLOCKS];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);

    // Workgroups are dealt round-robin to the 8 XCDs (each with its own L2).  Renumber so
    // that the column groups sharing a document chunk are neighbours on one XCD and run at
    // the same time: the chunk then comes from HBM once and from L2 for the other groups.
    const int v = xcd_grouped(blockIdx.x, gridDim.x);
    const int group = v % p.n_groups;
    const int chunk = v / p.n_groups;

    int64_t doc0_, doc1_;
    chunk_doc_range(p, chunk, doc0_, doc1_);
    if (doc0_ >= doc1_)
        return;
    const int doc0 = (int)doc0_, doc1 = (int)doc1_;
    if (group == 0)
        write_empty_docs(p, doc0, doc1, tid, NT);

    // this thread's share of a tile copy: chunk ch = tid + i * NT -> (row, 16-byte column)
    int cp_row[CPT], cp_goff[CPT], cp_loff[CPT];
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
        int ch = tid + i * NT;
        cp_row[i] = ch / CPR;
        cp_goff[i] = (ch % CPR) * 16;
        cp_loff[i] = (ch / CPR) * LT::ROW_STRIDE + (ch % CPR) * 16;
    }
    // 16-bit inputs with argmax keep the 32x32 results: their fold takes 1.5 VALU operations per cell, which with twice
    // the MFMA instructions and twice the running maxima fills the issue slots (32 x 1024 x 32 x 1024 through autograd
    // 376 us on 16x16 results, 336 on 32x32)
    constexpr bool PACKED = ARGMAX && TR::DT != MAXSIM_F32;
    const int rho = lane & 31, h = lane >> 5;
    const int a_off = PACKED ? rho * LT::ROW_STRIDE + h * 16 : (lane & 15) * LT::ROW_STRIDE + (lane >> 4) * 16;
    auto a_at = [&](int buf_off, int u) {
        return *reinterpret_cast<const uint4 *>(&lds_tile[buf_off + a_off + (PACKED ? u * 32 : frag_off16<DT, LT::ROW_STRIDE>(u))]);
    };

    for (int pass = 0; pass < p.n_pass; ++pass) {
        // column blocks of this pass: [gb0, gb0 + nb); queries [q_first, q_first + nq)
        int gb0, nb, q_first, nq;
        const bool accumulate = pass > 0;
        if (p.n_pass == 1) {
            q_first = group * p.qpg;
            nq = min(p.qpg, p.n_q - q_first);
            gb0 = q_first * p.bpq;
            nb = nq * p.bpq;
        } else { // one long query per group, GROUP_BLOCKS blocks of it per pass
            q_first = group;
            nq = 1;
            gb0 = group * p.bpq + pass * GROUP_BLOCKS;
            nb = min(GROUP_BLOCKS, p.bpq - pass * GROUP_BLOCKS);
        }
        // a query of one block needs no combination across blocks: its lane writes the score
        const bool direct = p.bpq == 1;

        uint4 qf[NCB][NU];
        bool col_valid[NCB];
        bool pair_valid[finish_pairs(NCB)]; // the same for the columns that finish_blocks16 leaves in the lane
        float m[NCB][2]; // (PACKED: the first of each)
        int key[NCB][2];
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) {
            int lb = w * NCB + cb;
            if constexpr (PACKED)
                load_q_block<DT>(p, gb0 + lb, rho, h, qf[cb], col_valid[cb]);
            else
                load_q_block16<DT>(p, gb0 + lb, lane, qf[cb]);
            col_valid[cb] = PACKED && col_valid[cb] && lb < nb;
            m[cb][0] = m[cb][1] = neg_inf();
            key[cb][0] = key[cb][1] = PACKED ? 0 : KEY_START;
        }

#pragma unroll
        for (int i = 0; i < finish_pairs(NCB); ++i) {
            auto left = [&](int cb) { // query tokens from the block's first on (scalar: the quotient is load_q_block16's)
                const int lb = w * NCB + (cb < NCB ? cb : NCB - 1);
                return lb < nb ? p.l_q - ((gb0 + lb) % p.bpq) * BLOCK_COLS : 0;
            };
            pair_valid[i] = ((lane >> 5) << 4) + (lane & 15) < ((lane & 16) ? left(2 * i + 1) : left(2 * i));
        }
        const bool wave_active = w * NCB < nb;
        TileIter li, ci; // load iterator (three tiles ahead of the compute iterator at steady state)
        it_init(li, p, off, doc0, doc1);
        ci = li;
        if (!it_valid(ci))
            break;

        // tiles in flight from HBM: ring slot 0 is the oldest (next to be stored to LDS), bit s of g_mask says that slot s holds a tile
        static_assert(PFD * CPT <= 8, "at most eight chunks per thread in flight");
        uint4 g0, g1, g2, g3, g4, g5, g6, g7;
        auto g = [&](auto slot, auto i) -> uint4 & { return reg_at<decltype(slot)::value * CPT + decltype(i)::value>(g0, g1, g2, g3, g4, g5, g6, g7); };
        constexpr std::integral_constant<int, 0> OLDEST{};
        constexpr std::integral_constant<int, PFD - 1> NEWEST{};
        unsigned g_mask = 0;
        // HBM -> registers (newest ring slot) for the next tile of the stream
        auto gload = [&]() {
            g_mask &= ~(1u << (PFD - 1));
            if (!it_valid(li))
                return;
            g_mask |= 1u << (PFD - 1);
            if (!copies) {
                it_next(li, p, off);
                return;
            }
            int last_row = li.len - li.t0 - 1; // rows past the document re-read its last token
            const char *base = p.D + (int64_t)li.row0 * TR::ROW_BYTES;
            static_for<CPT>([&](auto i) {
                int row = cp_row[i] < last_row ? cp_row[i] : last_row;
                g(NEWEST, i) = *reinterpret_cast<const uint4 *>(base + row * TR::ROW_BYTES + cp_goff[i]);
            });
            it_next(li, p, off);
        };
        // oldest ring slot -> LDS
        auto lstore = [&](int buf_off) {
            if (!(g_mask & 1u) || !copies)
                return;
            static_for<CPT>([&](auto i) { *reinterpret_cast<uint4 *>(&lds_tile[buf_off + cp_loff[i]]) = g(OLDEST, i); });
        };
        auto rotate = [&]() {
            static_for<PFD - 1>([&](auto slot) {
                static_for<CPT>([&](auto i) { g(slot, i) = g(std::integral_constant<int, decltype(slot)::value + 1>{}, i); });
            });
            g_mask >>= 1;
        };

        // LDS buffers (byte offsets): o_cur holds the tile being computed (already in registers),
        // o_nxt the next one (read into registers during this tile), o_wr receives the one after
        int o_cur = 0, o_nxt = LT::BYTES, o_wr = 2 * LT::BYTES;
        // tiles 0 and 1 go straight to LDS, the next PFD tiles into the ring
#pragma unroll
        for (int s = 0; s < PFD + 2; ++s) {
            rotate();
            gload();
            if (s < 2) { // the tile just loaded sits in the newest slot: pull it to the front and store it
#pragma unroll
                for (int r = 0; r + 1 < PFD; ++r)
                    rotate();
                lstore(s == 0 ? o_cur : o_nxt);
            }
        }
        __syncthreads();
        // a wavefront with a single column block uses every operand chunk once: a ring of four
        // registers, read three steps ahead, replaces the full operand set (the argmax variant with one block of 256-byte rows per wavefront)
        constexpr bool RING = !PF && NCB == 1 && NU >= 8;
        // no registers for a second operand set (fp32, argmax): each chunk is replaced by the next tile's
        // right after its last MFMA, during the last chain
        constexpr bool INPLACE = !PF && !RING;
        uint4 a0[NU], a1[PF ? NU : 1]; // (a0 stays unused when the operand ring is in use)
        if (PF || INPLACE) {
#pragma unroll
            for (int u = 0; u < NU; ++u)
                a0[u] = a_at(o_cur, u);
        }
        int par = 0;

        // one tile: operands in `ac`; the next tile's operands are read into `an` on the way
        auto stage = [&](uint4(&ac)[NU], uint4(&an)[PF ? NU : 1]) {
            const int fin_doc = (ci.t0 + TILE_ROWS >= ci.len) ? ci.doc : -1; // last tile of its document?
            uint4 ring[4];
            if (RING) {
#pragma unroll
                for (int u = 0; u < 3; ++u)
                    ring[u] = a_at(o_cur, u);
            }
            __builtin_amdgcn_sched_barrier(0);
            std::conditional_t<PACKED, f32x16, Acc16> acc[NCB];
            float tmax[NCB]; // PACKED: the tile's maximum per column block
            auto mma = [&](const uint4 &a, int cb, int u) {
                if constexpr (PACKED) {
                    if (u == 0) {
#pragma unroll
                        for (int r = 0; r < 16; ++r)
                            acc[cb][r] = 0.0f;
                    }
                    TR::mma(a, qf[cb][u], acc[cb]);
                } else {
                    mma_step16<DT>(a, qf[cb], u, acc[cb]);
                }
            };
            // what is folded at step u of block cb, and what is left after the last one (cb == NCB)
            auto fold = [&](int cb, int u) {
                if constexpr (PACKED) {
                    if (cb > 0)
                        fold_step_packed<NU>(acc[cb - 1], u, tmax[cb - 1], m[cb - 1][0], key[cb - 1][0], ci.t0);
                } else if (u >= NU / 2) {
                    if (cb < NCB)
                        fold_pairs16<ARGMAX>(acc[cb], half_pair<NU>(u - NU / 2), half_pair<NU>(u - NU / 2 + 1), m[cb], key[cb], ci.t0);
                } else if (cb > 0) {
                    fold_pairs16<ARGMAX>(acc[cb - 1], 4 + half_pair<NU>(u), 4 + half_pair<NU>(u + 1), m[cb - 1], key[cb - 1], ci.t0);
                }
            };
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb) {
#pragma unroll
                for (int u = 0; u < NU; ++u) {
                    if (RING) {
                        if (u + 3 < NU)
                            ring[(u + 3) & 3] = a_at(o_cur, u + 3);
                        mma(ring[u & 3], cb, u);
                    } else {
                        mma(ac[u], cb, u);
                        if (INPLACE && cb == NCB - 1)
                            ac[u] = a_at(o_nxt, u);
                    }
                    if (cb == 0) {
                        if (PF)
                            an[u] = a_at(o_nxt, u);
                        if (u == NU - 1) {
                            lstore(o_wr);
                            rotate();
                            gload();
                        }
                    }
                    fold(cb, u);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
#pragma unroll
            for (int u = 0; u < NU; ++u)
                fold(NCB, u);

            if (fin_doc >= 0) {
                auto put = [&](int lb, float sum) {
                    if (direct) {
                        if (lb < nb)
                            p.scores[(int64_t)(gb0 + lb) * p.ld + ci.doc] = sum;
                    } else {
                        lds_part[par][lb] = sum;
                    }
                };
                if constexpr (PACKED) {
#pragma unroll
                    for (int cb = 0; cb < NCB; ++cb) {
                        const int lb = w * NCB + cb;
                        const float sum = finish_block<ARGMAX>(p, m[cb][0], packed_key_row(key[cb][0], h), col_valid[cb], gb0 + lb, ci.doc, ci.len, rho, h);
                        if (lane == 0)
                            put(lb, sum);
                    }
                } else {
                    int row[NCB][2];
#pragma unroll
                    for (int i = 0; i < 2 * NCB; ++i)
                        row[i >> 1][i & 1] = ARGMAX ? key_row16(key[i >> 1][i & 1], lane >> 4) : 0;
                    const float sum = finish_blocks16<NCB, ARGMAX>(p, m, row, pair_valid, gb0 + w * NCB, ci.doc, ci.len, lane);
                    if ((lane & 15) == 0 && (lane >> 4) < NCB)
                        put(w * NCB + (lane >> 4), sum);
                }
#pragma unroll
                for (int cb = 0; cb < NCB; ++cb) { // the next document starts from nothing
                    m[cb][0] = m[cb][1] = neg_inf();
                    key[cb][0] = key[cb][1] = PACKED ? 0 : KEY_START;
                }
            }
            it_next(ci, p, off);
            __syncthreads();
            if (fin_doc >= 0) {
                if (!direct && tid < nq) { // thread t adds up the blocks of its query in block order
                    float sum = 0.0f;
                    int first_blk = (p.n_pass == 1) ? tid * p.bpq : 0;
                    int cnt = (p.n_pass == 1) ? p.bpq : nb;
                    for (int i = 0; i < cnt; ++i)
                        sum += lds_part[par][first_blk + i];
                    float *dst = p.scores + (int64_t)(q_first + tid) * p.ld + fin_doc;
                    *dst = accumulate ? *dst + sum : sum;
                }
                par ^= 1;
            }
            int t = o_cur;
            o_cur = o_nxt;
            o_nxt = o_wr;
            o_wr = t;
        };

        if (!wave_active) {
            // no column block in this pass: the wavefront only helps moving tiles (same barriers as the others)
            while (it_valid(ci)) {
                lstore(o_wr);
                rotate();
                gload();
                it_next(ci, p, off);
                __syncthreads();
                int t = o_cur;
                o_cur = o_nxt;
                o_nxt = o_wr;
                o_wr = t;
            }
        } else if constexpr (PF) {
            // The loop has one exit.  With a `break` after either stage the compiler joins the two exits in the latch, where
            // it fills the walk's undefined words through v_readfirstlane (eleven per two tiles), and keeps the loading
            // document's length in a vector register: bf16, one query of 130 tokens x 300 documents of 1000 28.0 us instead of
            // 26.7, of 512 tokens 53.1 instead of 50.7, 4 x 1024 tokens x 10 000 of 180 1293 instead of 1250.
            bool more = true;
            while (more) {
                stage(a0, a1);
                more = it_valid(ci);
                if (more) {
                    stage(a1, a0);
                    more = it_valid(ci);
                }
            }
        } else {
            while (it_valid(ci))
                stage(a0, a1);
        }
        __syncthreads(); // LDS is reused by the next pass
    }
}

// ---------------------------------------------------------------------------------------
// packed-window kernel: the tile kernel for ragged corpora and queries of one column block
// ---------------------------------------------------------------------------------------
//
// With documents of 64-300 tokens a sixth of the 32-row tiles is the ragged end of a document, and
// half of such a tile is padding.  Here a 32-row window may hold the last rows of document A and, from
// the next multiple of 4 rows on, the first rows of the next (non-empty) document B; it is cut short
// only where a third document would begin.  The MFMAs are the same.  The boundary sits on a multiple of
// 4 rows because a lane of the 16x16 results keeps rows 16i + 4g .. 16i + 4g + 3 (g = its quarter) in the four
// registers of result i: they then belong to one document, and a window with a boundary folds their maximum into
// A's or B's by two selects, decided once per lane and half of the window (no per-row masks).
// Such a window finishes A and carries B's maximum on.  Everything else (rotating LDS
// buffers, pinned pipeline) is fwd_tile_kernel's.  Queries have one column block here (L_q <= 32), so a
// wavefront's lane writes a score directly and no partial sums are combined.

struct WinIter {
    int doc, doc_end; // document that owns the window's first row; end of the run
    int row0;         // packed row of the window's first token
    int rem;          // tokens of `doc` from row0 on (> 0 while the iterator is valid)
    int end;          // packed row one past `doc`
    int nxt;          // offsets[doc + 2], unclamped, fetched while `doc` is walked
};

struct Window {
    int n_a;   // rows of document A = it.doc
    int pa;    // window row at which B starts: n_a rounded up to a multiple of 4 (rows n_a .. pa-1 repeat A's last)
    int n_b;   // rows of document B (0: no boundary inside the window)
    int doc_b; // next non-empty document (doc_end if there is none); only known when A ends in the window
    int len_b, end_b;
    bool fin_a, fin_b; // A / B end inside this window
};

__device__ __forceinline__ bool win_valid(const WinIter &it) { return it.doc < it.doc_end; }

// offsets[i] (i <= b), or i * l_d for a uniform corpus (UNI: a compile-time choice, so that the ragged case keeps
// its branch-free scalar loads)
template <bool UNI> __device__ __forceinline__ int win_offset(OffsetsPtr off, const FwdParams &p, int i)
{
    if constexpr (UNI)
        return (i < p.b ? i : (int)p.b) * p.l_d;
    else
        return it_offset(off, p, i);
}

// First non-empty document after it.doc within the run: d (doc_end if none) and its end e.  Offsets are
// forced into [previous end, T], so malformed offsets give wrong scores but no address outside D.
// The common case costs no memory access (it.nxt was fetched ahead); only empty documents take the loop,
// whose loads are made scalar values by hand so that the state stays in scalar registers.
template <bool UNI>
__device__ __forceinline__ void win_find_next(const WinIter &it, const FwdParams &p, OffsetsPtr off, int &d, int &e)
{
    const int t_all = (int)p.total_tokens;
    d = it.doc + 1;
    e = min(max(it.nxt, it.end), t_all); // offsets[d + 1]
    if (!UNI && d < it.doc_end && e == it.end) {
        do {
            ++d;
            if (d >= it.doc_end)
                break;
            const int raw = __builtin_amdgcn_readfirstlane(p.offsets[d + 1]);
            e = min(max(raw, it.end), t_all);
        } while (e == it.end);
    }
    if (d > it.doc_end)
        d = it.doc_end;
}

// Makes d (with end e, `used` of its rows already consumed) the current document; no branch around the
// read of the offset after next, so that it stays a scalar load
template <bool UNI>
__device__ __forceinline__ void win_enter(WinIter &it, const FwdParams &p, OffsetsPtr off, int d, int e, int used)
{
    const bool ok = d < it.doc_end;
    it.doc = d;
    it.nxt = win_offset<UNI>(off, p, d + 2);
    it.rem = ok ? e - it.end - used : 0;
    it.end = ok ? e : it.end;
}

template <bool UNI>
__device__ __forceinline__ void win_init(WinIter &it, const FwdParams &p, OffsetsPtr off, int doc0, int doc1)
{
    it.doc = doc0 - 1; // a virtual empty document before the run: its successor is the first real one
    it.doc_end = doc1;
    it.rem = 0;
    it.end = min(max(win_offset<UNI>(off, p, doc0), 0), (int)p.total_tokens);
    it.row0 = it.end;
    it.nxt = win_offset<UNI>(off, p, doc0 + 1);
    int d, e;
    win_find_next<UNI>(it, p, off, d, e);
    win_enter<UNI>(it, p, off, d, e, 0);
}

template <bool UNI>
__device__ __forceinline__ Window win_describe(const WinIter &it, const FwdParams &p, OffsetsPtr off)
{
    Window w;
    w.n_a = min(TILE_ROWS, it.rem);
    w.fin_a = w.n_a == it.rem;
    w.pa = (w.n_a + 3) & ~3;
    w.n_b = 0;
    w.doc_b = it.doc_end;
    w.len_b = 0;
    w.end_b = it.end;
    w.fin_b = false;
    if (w.fin_a) {
        win_find_next<UNI>(it, p, off, w.doc_b, w.end_b);
        if (w.doc_b < it.doc_end) {
            w.len_b = w.end_b - it.end;
            w.n_b = min(w.len_b, TILE_ROWS - w.pa);
            w.fin_b = w.n_b > 0 && w.n_b == w.len_b;
        }
    }
    return w;
}

template <bool UNI>
__device__ __forceinline__ void win_advance(WinIter &it, const Window &w, const FwdParams &p, OffsetsPtr off)
{
    it.row0 += w.n_a + w.n_b;
    if (!w.fin_a) {
        it.rem -= TILE_ROWS;
        return;
    }
    win_enter<UNI>(it, p, off, w.doc_b, w.end_b, w.n_b);
    if (win_valid(it) && it.rem == 0) { // B lay inside the window whole: on to the document after it
        int d, e;
        win_find_next<UNI>(it, p, off, d, e);
        win_enter<UNI>(it, p, off, d, e, 0);
    }
}

// NCB: column blocks (queries) per wavefront, 2 to 4; W: wavefronts per workgroup (8: 16 to 32 queries; 4 and 2 give
//      fewer queries the same 3 or 4 blocks per wavefront, i.e. as many MFMAs per window and barrier)
// UNI: uniform corpus (documents of l_d tokens, no offsets array)
template <int DT, int NCB, bool UNI, int W = 8, bool READ_ONCE>
__global__ void __launch_bounds__(W * 64, 2) fwd_pack_kernel(FwdParams p, OffsetsPtr off)
{
    using TR = Traits<DT>;
    using LT = LdsTile<DT>;
    constexpr int NU = TR::NU;
    constexpr int NT = W * 64;
    static_assert(NU <= 8, "the operand prefetch needs rows of at most 256 bytes");
    constexpr int CPT = (LT::CHUNKS + NT - 1) / NT;
    static_assert(LT::CHUNKS % NT == 0 || LT::CHUNKS < NT, "tile must split evenly over the workgroup");
    const bool copies = LT::CHUNKS >= NT || (int)threadIdx.x < LT::CHUNKS;
    constexpr int CPR = TR::ROW_BYTES / 16;
    constexpr int GROUP_BLOCKS = W * NCB;

    __shared__ __attribute__((aligned(16))) char lds_tile[3 * LT::BYTES];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);

    const int v = xcd_grouped(blockIdx.x, gridDim.x);
    const int group = v % p.n_groups;
    const int chunk = v / p.n_groups;

    int64_t doc0_, doc1_;
    chunk_doc_range(p, chunk, doc0_, doc1_);
    if (doc0_ >= doc1_)
        return;
    const int doc0 = (int)doc0_, doc1 = (int)doc1_;
    if (group == 0)
        write_empty_docs(p, doc0, doc1, tid, NT);

    // this thread's share of a tile copy: chunk ch = tid + i * NT -> (row, 16-byte column); recomputed where it
    // is used (a handful of shifts) rather than kept in registers, which are all taken
    auto cp_row = [&](int i) { return (tid + i * NT) / CPR; };
    auto cp_goff = [&](int i) { return ((tid + i * NT) % CPR) * 16; };
    auto cp_loff = [&](int i) { return ((tid + i * NT) / CPR) * LT::ROW_STRIDE + ((tid + i * NT) % CPR) * 16; };
    const int a_off = (lane & 15) * LT::ROW_STRIDE + (lane >> 4) * 16;
    auto a_at = [&](int buf_off, int u) { return *reinterpret_cast<const uint4 *>(&lds_tile[buf_off + a_off + frag_off16<DT, LT::ROW_STRIDE>(u)]); };

    // one column block = one query: blocks [gb0, gb0 + nb) of this group
    const int gb0 = group * GROUP_BLOCKS;
    const int nb = min(GROUP_BLOCKS, p.n_q - gb0);
    uint4 qf[NCB][NU];
    float m[NCB][2];
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
        int lb = w * NCB + cb;
        load_q_block16<DT>(p, gb0 + lb, lane, qf[cb]);
        m[cb][0] = m[cb][1] = neg_inf();
    }
    const bool wave_active = w * NCB < nb;
    const bool counts = ((lane >> 5) << 4) + (lane & 15) < p.l_q; // (see finish_blocks16; every block is a whole query)
    auto put_scores = [&](const float (&mm)[NCB][2], int doc) {
        bool valid[finish_pairs(NCB)];
#pragma unroll
        for (int i = 0; i < finish_pairs(NCB); ++i)
            valid[i] = counts;
        const int none[NCB][2] = {};
        const float sum = finish_blocks16<NCB, false>(p, mm, none, valid, gb0, doc, 0, lane);
        int b = lane >> 4; // (an opaque copy: the address is formed here and not kept in registers)
        asm volatile("" : "+v"(b));
        const int lb = w * NCB + b;
        if ((lane & 15) == 0 && b < NCB && lb < nb)
            p.scores[(int64_t)(gb0 + lb) * p.ld + doc] = sum;
    };

    // One iterator walks the windows, three ahead of the MFMAs (at load time).  What the stage needs of a window
    // later -- is there one, does it hold a boundary and where, which documents end in it -- travels in three scalar
    // words through a ring of three descriptors, instead of a second iterator that would derive it all again.
    struct WinDesc {
        int flags; // bit 0: the window exists; 1: it holds a boundary; 2: A ends in it; 3: B ends in it; bits 8..: pa
        int doc_a, doc_b;
    };
    WinIter li;
    win_init<UNI>(li, p, off, doc0, doc1);
    if (!win_valid(li))
        return;

    static_assert(CPT <= 4, "a thread moves at most four chunks per window");
    uint4 g0, g1, g2, g3, g4, g5, g6, g7; // the window on its way from HBM (see reg_at); four at most are used
    auto g = [&](auto i) -> uint4 & { return reg_at<decltype(i)::value>(g0, g1, g2, g3, g4, g5, g6, g7); };
    auto gload = [&]() -> WinDesc { // the next window of the stream -> registers; returns its descriptor
        WinDesc d = {0, 0, 0};
        if (!win_valid(li))
            return d;
        const Window lw = win_describe<UNI>(li, p, off);
        d.flags = 1 | (lw.n_b > 0 ? 2 : 0) | (lw.fin_a ? 4 : 0) | (lw.fin_b ? 8 : 0) | (lw.pa << 8);
        d.doc_a = li.doc;
        d.doc_b = lw.doc_b;
        if (copies) {
            // window row i holds A's row min(i, n_a - 1) below pa and B's row min(i - pa, n_b - 1) from pa on
            // (without a B that is A's last row again); A and B are neighbours in the packed corpus
            const char *base = p.D + (int64_t)li.row0 * TR::ROW_BYTES;
            auto at = [&](auto i) {
                const int wr = cp_row(i);
                const int row = wr < lw.pa ? min(wr, lw.n_a - 1) : lw.n_a + min(wr - lw.pa, lw.n_b - 1);
                return base + row * TR::ROW_BYTES + cp_goff(i);
            };
            // A window that repeats no row is a contiguous piece of memory, and its addresses are one addition per
            // thread instead of two clamps and a multiplication per chunk, which the wavefronts spend between their
            // matrix instructions.  Corpora of 100 000 documents of 64 to 300 tokens, 8 queries of 32 tokens 1148 ->
            // 1121 us; 20 000 documents of 8 to 600 tokens, 5 / 8 / 16 queries 324 / 382 / 637 -> 310 / 371 / 621.
            // Where several groups read a window it is a trade: 48 / 64 queries x 100 000 documents of 64 to 300 tokens 5329 /
            // 6645 -> 5176 / 6602, but 33 / 64 x 40 000 of 1 to 30 tokens 293 / 351 -> 301 / 358, also where a rule on the mean
            // length leaves the branch untaken; not there.
            if (READ_ONCE && lw.pa == lw.n_a && lw.n_a + lw.n_b == TILE_ROWS) {
                const char *src = base + tid * 16;
                static_for<CPT>([&](auto i) { g(i) = load_stream16(src + decltype(i)::value * (NT * 16)); });
            } else {
                static_for<CPT>([&](auto i) { g(i) = READ_ONCE ? load_stream16(at(i)) : *reinterpret_cast<const uint4 *>(at(i)); });
            }
        }
        win_advance<UNI>(li, lw, p, off);
        return d;
    };
    WinDesc d_cur, d_n1, d_n2; // the windows being computed, read from LDS next, and on their way from HBM
    auto lstore = [&](int buf_off) { // the window in the registers (d_n2) -> LDS
        if (!(d_n2.flags & 1) || !copies)
            return;
        static_for<CPT>([&](auto i) { *reinterpret_cast<uint4 *>(&lds_tile[buf_off + cp_loff(i)]) = g(i); });
    };

    int o_cur = 0, o_nxt = LT::BYTES, o_wr = 2 * LT::BYTES;
    d_n2 = gload();
    lstore(o_cur);
    d_cur = d_n2;
    d_n2 = gload();
    lstore(o_nxt);
    d_n1 = d_n2;
    d_n2 = gload();
    __syncthreads();
    // One operand set: during the LAST chain of a window every operand chunk is replaced, right after the
    // MFMA that used it last, by the next window's (the second set of fwd_tile_kernel would not fit beside
    // the two maxima of a boundary window).
    uint4 ac[NU];
#pragma unroll
    for (int u = 0; u < NU; ++u)
        ac[u] = a_at(o_cur, u);

    // BND: the window holds rows of two documents
    auto stage = [&](auto bnd_tag) {
        constexpr bool BND = decltype(bnd_tag)::value;
        const int cw_pa = d_cur.flags >> 8;
        const bool cw_fin_a = (d_cur.flags & 4) != 0, cw_fin_b = (d_cur.flags & 8) != 0;
        WinDesc d_new = {0, 0, 0};
        float mb[NCB][2];
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb)
            mb[cb][0] = mb[cb][1] = neg_inf();
        // rows 4 g .. 4 g + 3 of either half of the window belong to A below the boundary, to B from it on
        const bool in_a[2] = {4 * (lane >> 4) < cw_pa, 16 + 4 * (lane >> 4) < cw_pa};
        // what is folded at step u of block cb, and what is left after the last one (cb == NCB): see half_pair
        auto fold = [&](const Acc16 *acc, int cb, int u) {
            const int i = u >= NU / 2 ? 0 : 1, b = cb - i;
            if (b < 0 || b >= NCB)
                return;
            const int k0 = half_pair<NU>(u % (NU / 2)), k1 = half_pair<NU>(u % (NU / 2) + 1);
            if (BND) {
#pragma unroll
                for (int j = k0 / 2; j < k1 / 2; ++j) {
                    const f32x4 &t = acc[b].t[i][j];
                    const float qm = fmaxf(fmaxf(fmaxf(t[0], t[1]), t[2]), t[3]);
                    m[b][j] = fmaxf(m[b][j], in_a[i] ? qm : neg_inf());
                    mb[b][j] = fmaxf(mb[b][j], in_a[i] ? neg_inf() : qm);
                }
            } else {
                int none[2];
                fold_pairs16<false>(acc[b], 4 * i + k0, 4 * i + k1, m[b], none, 0);
            }
        };
        __builtin_amdgcn_sched_barrier(0);
        Acc16 acc[NCB];
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) {
#pragma unroll
            for (int u = 0; u < NU; ++u) {
                mma_step16<DT>(ac[u], qf[cb], u, acc[cb]);
                if (cb == NCB - 1)
                    ac[u] = a_at(o_nxt, u);
                if (cb == 0 && u == NU - 1) {
                    lstore(o_wr);
                    d_new = gload();
                }
                fold(acc, cb, u);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int u = 0; u < NU; ++u)
            fold(acc, NCB, u);

        if (cw_fin_a) {
            put_scores(m, d_cur.doc_a);
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb) {
                m[cb][0] = BND ? mb[cb][0] : neg_inf();
                m[cb][1] = BND ? mb[cb][1] : neg_inf();
            }
            if (BND && cw_fin_b) {
                put_scores(m, d_cur.doc_b);
#pragma unroll
                for (int cb = 0; cb < NCB; ++cb)
                    m[cb][0] = m[cb][1] = neg_inf();
            }
        }
        __syncthreads();
        int t = o_cur;
        o_cur = o_nxt;
        o_nxt = o_wr;
        o_wr = t;
        d_cur = d_n1;
        d_n1 = d_n2;
        d_n2 = d_new;
    };

    if (!wave_active) {
        // fewer than 32 queries in this group: the wavefront only helps moving tiles (same barriers as the others)
        while (d_cur.flags & 1) {
            lstore(o_wr);
            const WinDesc d_new = gload();
            __syncthreads();
            int t = o_cur;
            o_cur = o_nxt;
            o_nxt = o_wr;
            o_wr = t;
            d_cur = d_n1;
            d_n1 = d_n2;
            d_n2 = d_new;
        }
    } else {
        // runs of plain windows, each ended by one boundary window
        for (;;) {
            while (!(d_cur.flags & 2)) {
                stage(std::false_type{});
                if (!(d_cur.flags & 1))
                    return;
            }
            stage(std::true_type{});
            if (!(d_cur.flags & 1))
                return;
        }
    }
}

// ---------------------------------------------------------------------------------------
// host-side launchers (called from the C ABI)
// ---------------------------------------------------------------------------------------

template <int DT, int NCB, bool ARGMAX>
static hipError_t launch_stream(FwdParams p, int grid, hipStream_t stream)
{
    if constexpr (Traits<DT>::NU == 16 && Traits<DT>::DT == MAXSIM_F32) {
        if (p.doc_waves) { // (fp32_shape)
            auto go = [&](auto w, auto g) {
                constexpr int W = decltype(w)::value, G = decltype(g)::value;
                hipLaunchKernelGGL((fwd_f32_split_kernel<ARGMAX, W, NCB, G>), dim3((unsigned)((p.b + G - 1) / G)), dim3(G * W * NCB * 64), 0, stream, p, p.offsets);
                return hipGetLastError();
            };
            constexpr std::integral_constant<int, 1> one{};
            constexpr std::integral_constant<int, 2> two{};
            constexpr std::integral_constant<int, 4> four{};
            if (p.docs_per_wg > 1) { // workgroups of four wavefronts
                if constexpr (NCB == 1)
                    return p.doc_waves == 2 ? go(two, two) : go(one, four);
                else
                    return go(one, two);
            }
            return p.doc_waves == 4 ? go(four, one) : p.doc_waves == 2 ? go(two, one) : go(one, one);
        }
    }
    if (p.doc_waves) { // a workgroup of doc_waves wavefronts per document and qpg queries
        if constexpr (Traits<DT>::NU <= 8 || (NCB == 1 && Traits<DT>::DT != MAXSIM_F32)) {
            p.n_groups = (p.n_q + p.qpg - 1) / p.qpg;
            auto go = [&](auto w, auto groups) {
                constexpr int W = decltype(w)::value;
                constexpr bool G = decltype(groups)::value;
                hipLaunchKernelGGL((fwd_stream_split_kernel<DT, NCB, ARGMAX, W, G>), dim3(grid * p.n_groups), dim3(W * 64), 0, stream, p, p.offsets);
                return hipGetLastError();
            };
            if constexpr (Traits<DT>::NU <= 8 && Traits<DT>::DT != MAXSIM_F32 && ARGMAX && NCB <= 2) { // (few_documents)
                if (p.doc_waves == 1)
                    return go(std::integral_constant<int, 1>{}, std::true_type{});
                if (p.doc_waves == 4)
                    return go(std::integral_constant<int, 4>{}, std::true_type{});
                if (p.n_groups > 1)
                    return go(std::integral_constant<int, 2>{}, std::true_type{});
            }
            return go(std::integral_constant<int, 2>{}, std::false_type{});
        }
        return hipErrorInvalidValue;
    }
    if (p.n_groups == 1) { // one wavefront per run: whole-line loads through LDS
        constexpr int WPB = lin_waves<DT>();
        const int grid_lin = (p.n_chunks + WPB - 1) / WPB;
        hipLaunchKernelGGL((fwd_stream_lin_kernel<DT, NCB, ARGMAX>), dim3(grid_lin), dim3(WPB * 64), 0, stream, p, p.offsets);
        return hipGetLastError();
    }
    if constexpr (Traits<DT>::NU <= 8 || NCB == 1) { // narrow rows: more than four column blocks go to the tile kernel; several groups hold two blocks each
        return hipErrorInvalidValue;
    } else {
        hipLaunchKernelGGL((fwd_stream_kernel<DT, NCB, ARGMAX>), dim3(grid), dim3(256), 0, stream, p, p.offsets);
        return hipGetLastError();
    }
}

// The tile and packed-window kernels: the chunks are cut for the workgroups that are resident at a time, which the
// registers of the instantiation decide: two wavefronts per SIMD with four blocks of 256-byte rows in each, four with
// one block or narrow rows.  (One number for them all left half of the wavefront slots of the others empty: one query
// of 130 tokens x 3000 documents of 100 with argmax 38 us instead of 27, fp32 d = 32 x 20 000 of 70 377 instead of 276.
// Sixteen wavefronts per CU for all of them, in a multiple of eight chunks, left half of the chip idle in a second
// round where documents are few: one query of 130 tokens x 500 documents of 260 23.5 us instead of 13.6, 2 x 1024 x 600
// pages 286 instead of 235.)  The number is a property of the code object, the same on every device the library runs
// on; it is asked for once per instantiation.
template <auto KERNEL> static int resident_workgroups(int threads)
{
    static std::atomic<int> known{0};
    int n = known.load(std::memory_order_relaxed);
    if (n == 0) {
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, KERNEL, threads, 0) != hipSuccess || n < 1)
            return 0;
        known.store(n, std::memory_order_relaxed);
    }
    return n;
}

// HALF: half of the resident workgroups may do (four wavefronts with two blocks each and a ring of tiles: the beginnings
// of all of them cost more than they bring; seven blocks x 1000 documents of 180 tokens of d = 64 9.9 us, 10.4 with all
// of them, ragged 2000 x 8-60 9.8 and 10.8; d = 128, 600 x 64 8.6 and 9.2, but ragged 2000 x 8-60 15.6 and 13.7)
template <auto KERNEL, bool HALF> static hipError_t launch_chunks(FwdParams p, int threads, int num_cu, hipStream_t stream)
{
    const int resident = resident_workgroups<KERNEL>(threads);
    if (resident == 0)
        return hipErrorInvalidValue;
    const ChunkPlan plan = plan_chunks(p, p.n_groups, num_cu, resident, HALF ? (resident + 1) / 2 : resident, true);
    if (plan.n_chunks * p.n_groups >= (int64_t(1) << 31))
        return hipErrorInvalidValue;
    p.unit_per_chunk = plan.per_chunk;
    p.n_chunks = (int)plan.n_chunks;
    hipLaunchKernelGGL(KERNEL, dim3((unsigned)(plan.n_chunks * p.n_groups)), dim3(threads), 0, stream, p, p.offsets);
    return hipGetLastError();
}

template <int DT, int W, int NCB, bool ARGMAX, int PFD = 1>
static hipError_t launch_tile(const FwdParams &p, int num_cu, hipStream_t stream)
{
    return launch_chunks<&fwd_tile_kernel<DT, W, NCB, ARGMAX, PFD>, W == 4 && NCB == 2>(p, W * 64, num_cu, stream);
}

// Windows are read with the non-temporal hint (READ_ONCE) where one workgroup reads each of them and the corpus is
// larger than the 256 MB that the device's last cache holds: 1050 instead of 1118 us for five queries x 100 000 texts,
// 140 instead of 147 for eight x 20 000 x 96 tokens.  A corpus that stays in that cache from one call to the next is
// slower with the hint (five queries x 10 000 x 180 tokens of d = 64 57.5 instead of 52 us, twelve x 3000 texts 59.6
// instead of 57.4), and so are windows that two column groups share (40 queries x 50 000 texts 2054 instead of 1990
// us); fp32 takes the same time either way.
template <int DT, int NCB, int W = 8>
static hipError_t launch_pack(const FwdParams &p, int num_cu, hipStream_t stream)
{
    if constexpr (Traits<DT>::DT != MAXSIM_F32) {
        if (p.n_groups == 1 && p.total_tokens * Traits<DT>::ROW_BYTES > (int64_t(256) << 20))
            return p.offsets ? launch_chunks<&fwd_pack_kernel<DT, NCB, false, W, true>, false>(p, W * 64, num_cu, stream)
                             : launch_chunks<&fwd_pack_kernel<DT, NCB, true, W, true>, false>(p, W * 64, num_cu, stream);
    }
    return p.offsets ? launch_chunks<&fwd_pack_kernel<DT, NCB, false, W, false>, false>(p, W * 64, num_cu, stream)
                     : launch_chunks<&fwd_pack_kernel<DT, NCB, true, W, false>, false>(p, W * 64, num_cu, stream);
}

template <int DT, bool ARGMAX>
static hipError_t dispatch_stream(const FwdParams &p, int ncb, int grid, hipStream_t s)
{
    constexpr int NU = Traits<DT>::NU;
    if constexpr (NU <= 8) {
        switch (ncb) {
        case 1: return launch_stream<DT, 1, ARGMAX>(p, grid, s);
        case 2: return launch_stream<DT, 2, ARGMAX>(p, grid, s);
        case 3: return launch_stream<DT, 3, ARGMAX>(p, grid, s);
        default: return launch_stream<DT, 4, ARGMAX>(p, grid, s);
        }
    } else {
        return ncb == 1 ? launch_stream<DT, 1, ARGMAX>(p, grid, s) : launch_stream<DT, 2, ARGMAX>(p, grid, s);
    }
}

template <int DT, bool ARGMAX>
static hipError_t dispatch_tile(const FwdParams &p, int w, int num_cu, hipStream_t s)
{
    constexpr int NU = Traits<DT>::NU;
    constexpr bool TWO_WAVES = Traits<DT>::DT != MAXSIM_F32; // fp32 takes no shapes of two wavefronts (see forward_launch)
    if constexpr (NU <= 8) {
        switch (w) {
        case 82: return launch_tile<DT, 8, 2, ARGMAX, 3>(p, num_cu, s); // few column blocks
        case 42: return launch_tile<DT, 4, 2, ARGMAX, 4>(p, num_cu, s);
        case 83: return launch_tile<DT, 8, 3, ARGMAX>(p, num_cu, s); // three blocks each
        case 43: return launch_tile<DT, 4, 3, ARGMAX, 2>(p, num_cu, s);
        case 4: return launch_tile<DT, 4, 4, ARGMAX>(p, num_cu, s); // four: query fragments fill 128 registers
        case 8: return launch_tile<DT, 8, 4, ARGMAX>(p, num_cu, s);
        }
        if constexpr (TWO_WAVES) {
            if (w == 23)
                return launch_tile<DT, 2, 3, ARGMAX, 2>(p, num_cu, s);
            if (w == 2)
                return launch_tile<DT, 2, 4, ARGMAX>(p, num_cu, s);
        }
        if constexpr (ARGMAX) { // one long query of five to eight blocks
            if (w == 81)
                return launch_tile<DT, 8, 1, true, 6>(p, num_cu, s);
        } else { // queries of one block on ragged corpora: windows over the packed rows, 3 or 4 queries per wavefront
            switch (w) {
            case 93: return launch_pack<DT, 3>(p, num_cu, s);
            case 94: return launch_pack<DT, 4>(p, num_cu, s);
            case 943: return launch_pack<DT, 3, 4>(p, num_cu, s);
            case 944: return launch_pack<DT, 4, 4>(p, num_cu, s);
            }
            if constexpr (TWO_WAVES) {
                if (w == 923)
                    return launch_pack<DT, 3, 2>(p, num_cu, s);
                if (w == 924)
                    return launch_pack<DT, 4, 2>(p, num_cu, s);
            }
        }
    } else { // 512-byte rows, three to seven blocks: two fill 128 registers
        if (w == 2)
            return launch_tile<DT, 2, 2, ARGMAX>(p, num_cu, s);
        if (w == 4)
            return launch_tile<DT, 4, 2, ARGMAX>(p, num_cu, s);
    }
    return hipErrorInvalidValue;
}

template <int F>
static hipError_t run_format(const FwdParams &p, bool argmax, bool tile, int x, int n, hipStream_t s)
{
    if (tile) {
        if (!argmax)
            return dispatch_tile<F, false>(p, x, n, s);
        if constexpr (F == fmt(MAXSIM_F16, 8))
            return forward_tile_argmax_f16(p, x, n, s);
        else if constexpr (F == fmt(MAXSIM_BF16, 8))
            return forward_tile_argmax_bf16(p, x, n, s);
        else
            return dispatch_tile<F, true>(p, x, n, s);
    }
    return argmax ? dispatch_stream<F, true>(p, x, n, s) : dispatch_stream<F, false>(p, x, n, s);
}

// All widths of one element type: nu = row bytes / 32.  `tile` picks the kernel, x is its shape
// parameter (wavefronts per workgroup for the tile kernel, column blocks per wavefront for the
// streaming kernel) and n the streaming kernel's grid or, for the tile kernel, the device's CUs.
template <int DTYPE>
static hipError_t run_dtype(const FwdParams &p, int nu, bool argmax, bool tile, int x, int n, hipStream_t s)
{
    switch (nu) {
    case 4: return run_format<fmt(DTYPE, 4)>(p, argmax, tile, x, n, s);
    case 8: return run_format<fmt(DTYPE, 8)>(p, argmax, tile, x, n, s);
    case 16: return run_format<fmt(DTYPE, 16)>(p, argmax, tile, x, n, s);
    default: return hipErrorNotSupported;
    }
}

} // namespace
} // namespace maxsim
