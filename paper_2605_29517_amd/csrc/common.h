// Shared device-side vocabulary of the gfx950 MaxSim kernels (not part of the public ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>
#include <cmath>
#include <type_traits>

#include "../../include/maxsim.h"

namespace maxsim {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef int i32x16 __attribute__((ext_vector_type(16)));
typedef int i32x4 __attribute__((ext_vector_type(4)));

constexpr int D_MODEL = 128;  // embedding width of the backward and int8 kernels (the float forward also takes 64, 256, 512)
constexpr int TILE_ROWS = 32; // document tokens per MFMA tile (rows of the 32x32 result)
constexpr int BLOCK_COLS = 32; // query tokens per column block (columns of the 32x32 result)

// A token row is handled in 16-byte chunks.  Lane (rho = lane % 32, h = lane / 32) of a
// wavefront owns chunks 2u + h (u = 0 .. NU-1) of row rho, for documents (MFMA A operand)
// and queries (MFMA B operand) alike, so both sides pair the same k indices.
//
// The float kernels are compiled per "format" F = dtype | (NU << 4): the element type and the
// embedding width (a row is NU * 32 bytes: d = 16 * NU for 16-bit inputs, 8 * NU for fp32).
constexpr int fmt(int dtype, int nu) { return dtype | (nu << 4); }

template <int F> struct Traits {
    static constexpr int DT = F & 15;
    static constexpr int NU = F >> 4;
    static constexpr int ROW_BYTES = NU * 32;
    static __device__ __forceinline__ void mma(const uint4 &a, const uint4 &b, f32x16 &c)
    {
        if constexpr (DT == MAXSIM_F16) {
            c = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
        } else if constexpr (DT == MAXSIM_BF16) {
            c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
        } else {
            // one chunk = 4 floats = 4 rank-2 updates (k = 2 per instruction: halves h = 0, 1)
            c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.x), __uint_as_float(b.x), c, 0, 0, 0);
            c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.y), __uint_as_float(b.y), c, 0, 0, 0);
            c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.z), __uint_as_float(b.z), c, 0, 0, 0);
            c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.w), __uint_as_float(b.w), c, 0, 0, 0);
        }
    }
    // The same on 16 rows x 16 columns (see Acc16): lane quarter g = lane / 16 pairs the g-th of four chunks.
    static __device__ __forceinline__ void mma16(const uint4 &a, const uint4 &b, f32x4 &c)
    {
        if constexpr (DT == MAXSIM_F16) {
            c = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
        } else if constexpr (DT == MAXSIM_BF16) {
            c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
        } else { // four rank-4 updates (k = 4 per instruction: the quarters)
            c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.x), __uint_as_float(b.x), c, 0, 0, 0);
            c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.y), __uint_as_float(b.y), c, 0, 0, 0);
            c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.z), __uint_as_float(b.z), c, 0, 0, 0);
            c = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a.w), __uint_as_float(b.w), c, 0, 0, 0);
        }
    }
};

// 32 document tokens x 32 query tokens as four 16x16 results, for the kernels that are bound by the power limit: on
// operands of unit-norm rows a loop of 16x16x32 MFMAs (operands from LDS, folds in between) sustains 1715-1745 TFLOP/s
// fp16 and 1835-1870 bf16 where one of 32x32x16 MFMAs holds 1500-1525 and 1625-1660 (probe_tile_kernel) -- half as many
// accumulator words travel per product -- and on zero operands, where the clock does not drop, both 2220-2240.
// Lane (c = lane % 16, g = lane / 16) keeps, of result (i, j), query token 16 j + c and document tokens 16 i + 4 g + r,
// r = 0 .. 3.  Operand fragment f = i * NU / 2 + u is chunk 4 u + g of document row 16 i + c, for queries alike.
struct Acc16 {
    f32x4 t[2][2];
};

// Step u (of NU) of the chains of one column block; a is the u-th document fragment, q the block's fragments
template <int F> __device__ __forceinline__ void mma_step16(const uint4 &a, const uint4 (&q)[Traits<F>::NU], int u, Acc16 &acc)
{
    constexpr int S = Traits<F>::NU / 2;
    const int i = u / S, k = u % S;
    if (k == 0) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            acc.t[i][0][r] = 0.0f;
            acc.t[i][1][r] = 0.0f;
        }
    }
    Traits<F>::mma16(a, q[k], acc.t[i][0]);
    Traits<F>::mma16(a, q[S + k], acc.t[i][1]);
}

// Row of the 32x32 MFMA result held in accumulator register r of a lane in half h.
__device__ __forceinline__ int acc_row(int r, int h) { return (r >> 2) * 8 + h * 4 + (r & 3); }

__device__ __forceinline__ float neg_inf() { return -__builtin_huge_valf(); }

// 16-byte load with the non-temporal hint, for streams that are read once by instructions that take whole lines
// (sixteen lanes on 256 contiguous bytes): 6.8 against 6.0 TB/s for a wavefront-per-run read stream.  Not for
// loads that take a part of a line and leave the rest to a neighbour: the hint keeps the caches from merging them.
__device__ __forceinline__ uint4 load_stream16(const void *p)
{
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    const u32x4 t = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(p));
    return make_uint4(t.x, t.y, t.z, t.w);
}

// f(integral_constant<int, 0>) ... f(integral_constant<int, N - 1>), in this order
template <int N, class F> __device__ __forceinline__ void static_for(F &&f)
{
    if constexpr (N > 0) {
        static_for<N - 1>(f);
        f(std::integral_constant<int, N - 1>{});
    }
}

// One of eight named 16-byte registers by compile-time index.  The chunks of a tile on its way from HBM to LDS are
// kept this way: as an array indexed in unrolled loops inside lambdas they stayed in scratch memory whenever a
// thread moves more than one chunk per tile.
template <int I> __device__ __forceinline__ uint4 &reg_at(uint4 &r0, uint4 &r1, uint4 &r2, uint4 &r3, uint4 &r4, uint4 &r5, uint4 &r6, uint4 &r7)
{
    static_assert(I >= 0 && I < 8, "eight registers");
    if constexpr (I == 0)
        return r0;
    else if constexpr (I == 1)
        return r1;
    else if constexpr (I == 2)
        return r2;
    else if constexpr (I == 3)
        return r3;
    else if constexpr (I == 4)
        return r4;
    else if constexpr (I == 5)
        return r5;
    else if constexpr (I == 6)
        return r6;
    else
        return r7;
}

// Arguments of the forward kernels (plain data, passed by value).
struct FwdParams {
    const char *Q;          // [n_q, l_q, d]
    const char *D;          // [b, l_d, d] or packed [T, d]
    const int32_t *offsets; // [b + 1] or nullptr for a uniform corpus
    float *scores;          // [n_q, b]
    int32_t *argmax;        // [n_q, b, l_q] or nullptr
    int64_t b;
    int64_t ld;           // documents per row of scores / argmax (b, or the whole corpus when b is a slice of it)
    int64_t total_tokens; // b * l_d for a uniform corpus
    int n_q, l_q, l_d;
    int bpq;               // column blocks per query = ceil(l_q / 32)
    int n_chunks;          // document chunks (work units along the corpus)
    int64_t unit_per_chunk; // documents (uniform) or tokens (ragged) per chunk
    int n_groups;          // column groups (tile kernel only)
    int qpg;               // queries per column group (tile kernel, bpq <= group size)
    int n_pass;            // passes over the corpus per group (tile kernel, bpq > group size)
    int doc_waves;         // wavefronts that share a document (the split kernels; 0: runs of documents)
    int docs_per_wg;       // documents per workgroup (fwd_f32_split_kernel)
};

// Offsets come from device memory the host cannot check.  Every offset is forced into
// [lo, total_tokens] before it is used (once per document, scalar work), so that offsets which
// are not non-decreasing or run past the corpus give wrong scores but never an address outside D.
__device__ __forceinline__ int64_t clamp_offset(int64_t x, int64_t lo, int64_t hi) { return x < lo ? lo : (x > hi ? hi : x); }

// A kernel that walks a ragged corpus takes the offsets a second time, as a `const int32_t *__restrict__`
// parameter of its own: only then does the compiler know that no store of the kernel can change them and
// reads offsets[uniform index] through the scalar cache, apart from the vector loads in flight.
typedef const int32_t *__restrict__ OffsetsPtr;

// Cursor over the 32-row tiles of a run of documents, identical in every lane of a wavefront.
struct Cursor {
    int64_t doc;     // current document
    int64_t doc_end; // end of the run (exclusive)
    int64_t start;   // first packed row of the current document
    int64_t nxt_end; // offsets[doc + 2], fetched one document ahead (ragged only)
    int32_t len;     // tokens in the current document
    int32_t t0;      // first row (document-local) of the current tile
    bool valid;
};

__device__ __forceinline__ void cursor_next_doc(Cursor &c, const FwdParams &p, OffsetsPtr off)
{
    for (;;) {
        c.doc += 1;
        c.valid = c.doc < c.doc_end;
        if (!c.valid)
            return;
        c.t0 = 0;
        if (p.offsets) {
            c.start += c.len;
            int64_t e = clamp_offset(c.nxt_end, c.start, p.total_tokens);
            c.len = (int32_t)(e - c.start);
            c.nxt_end = (int64_t)off[(c.doc + 2 <= p.b) ? c.doc + 2 : p.b]; // no branch around the load: it stays a scalar load
            if (c.len > 0)
                return;
        } else {
            c.start += p.l_d;
            return;
        }
    }
}

__device__ __forceinline__ void cursor_init(Cursor &c, const FwdParams &p, OffsetsPtr off, int64_t doc0, int64_t doc1)
{
    c.doc = doc0;
    c.doc_end = doc1;
    c.t0 = 0;
    c.valid = doc0 < doc1;
    if (!c.valid)
        return;
    if (p.offsets) {
        c.start = clamp_offset(off[doc0], 0, p.total_tokens);
        int64_t e = clamp_offset(off[doc0 + 1], c.start, p.total_tokens);
        c.len = (int32_t)(e - c.start);
        c.nxt_end = (int64_t)off[(doc0 + 2 <= p.b) ? doc0 + 2 : p.b];
        if (c.len == 0)
            cursor_next_doc(c, p, off);
    } else {
        c.start = doc0 * (int64_t)p.l_d;
        c.len = p.l_d;
        c.nxt_end = 0;
    }
}

__device__ __forceinline__ void cursor_next_tile(Cursor &c, const FwdParams &p, OffsetsPtr off, int rows = TILE_ROWS)
{
    c.t0 += rows;
    if (c.t0 >= c.len)
        cursor_next_doc(c, p, off);
}

// Workgroup ids are dealt round-robin to the 8 XCDs.  This renumbering of n ids gives every XCD a contiguous range.
__device__ __forceinline__ int xcd_grouped(unsigned id, unsigned n)
{
    const unsigned xcd = id & 7;
    return (int)(xcd * (n >> 3) + (xcd < (n & 7) ? xcd : n & 7) + (id >> 3));
}

// Documents [doc0, doc1) of work chunk `chunk`.  Uniform corpus: equal document counts.
// Ragged corpus: the packed token range is cut into equal pieces and a chunk owns every
// document that starts inside its piece (binary search over the offsets).
//
// The search is one of the first things a wavefront does and every step is a memory round trip (a microsecond on a
// busy chip), so a step takes 64 probes, one per lane: three steps for 100 000 documents instead of seventeen, and the
// two ends of a run are searched together.  All 64 lanes must be active and n and the keys uniform.
struct OffsetSearch {
    uint32_t lo, end, step; // the answer is in [lo, end] (n < 2^31: positions up to end + 63 fit)

    __device__ __forceinline__ void begin(int64_t n)
    {
        lo = 0;
        end = (uint32_t)n + 1;
    }
    __device__ __forceinline__ bool open() const { return lo < end; }
    __device__ __forceinline__ uint32_t probe(uint32_t lane) // position this lane looks at; `end` or more: none
    {
        step = (end - lo + 63) >> 6;
        return step ? lo + (lane + 1) * step - 1 : end;
    }
    __device__ __forceinline__ void narrow(uint64_t below) // bit l: lane l's probe is in range and below the key
    {
        lo += (uint32_t)__builtin_popcountll(below) * step;
        const uint32_t hit = lo + step - 1; // the first probe that is not below, if it is in range
        end = hit < end ? hit : end;
    }
};

// smallest i in [0, n] with off[i] >= key (off has n + 1 entries, non-decreasing), n + 1 if there is none; two keys
__device__ __forceinline__ void lower_bound_offsets2(const int32_t *off, int64_t n, int64_t key0, int64_t key1, int64_t &r0, int64_t &r1)
{
    const uint32_t lane = threadIdx.x & 63;
    OffsetSearch a, b;
    a.begin(n);
    b.begin(n);
    while (a.open() || b.open()) {
        const uint32_t pa = a.probe(lane), pb = b.probe(lane);
        const bool ia = pa < a.end, ib = pb < b.end;
        const int32_t va = off[ia ? pa : 0u], vb = off[ib ? pb : 0u];
        a.narrow(__builtin_amdgcn_ballot_w64(ia && (int64_t)va < key0));
        b.narrow(__builtin_amdgcn_ballot_w64(ib && (int64_t)vb < key1));
    }
    r0 = a.lo;
    r1 = b.lo;
}

__device__ __forceinline__ void chunk_doc_range(const FwdParams &p, int64_t chunk, int64_t &doc0, int64_t &doc1)
{
    if (chunk >= p.n_chunks) {
        doc0 = doc1 = 0;
        return;
    }
    if (p.offsets) {
        const int64_t lo = chunk * p.unit_per_chunk;
        const int64_t hi = lo + p.unit_per_chunk;
        lower_bound_offsets2(p.offsets, p.b, lo, hi, doc0, doc1);
        if (chunk == 0)
            doc0 = 0;
        if (chunk == p.n_chunks - 1)
            doc1 = p.b;
        if (doc0 > p.b)
            doc0 = p.b;
        if (doc1 > p.b)
            doc1 = p.b;
    } else {
        doc0 = chunk * p.unit_per_chunk;
        doc1 = doc0 + p.unit_per_chunk;
        if (doc0 > p.b)
            doc0 = p.b;
        if (doc1 > p.b)
            doc1 = p.b;
    }
}

// How a corpus is cut into chunks for `groups` column groups: units (documents, or tokens of a ragged corpus) per
// chunk. A workgroup costs what about 200 tokens do beside its documents (its query fragments and the first loads), a
// chunk of a ragged corpus may be half a document longer than its share, and a CU takes as long as the workgroups that
// fall to it; with fewer than are resident on it at a time it works more slowly, by the square root of the share.
// `time`, in tokens, is what is minimised, over the numbers of workgroups from `fewest` per CU (at most those resident)
// to eight times those resident. With `level`, ragged corpora of 2500 tokens a chunk and more are cut for two rounds at
// least where one or two workgroups are resident, so that CUs whose documents happen to be short take more of them (9
// queries with argmax x 30 000 documents of log-normal length, 98 tokens on average: 425 us instead of 457; with 64-200
// tokens 2-3 % are lost). Several column groups, four resident workgroups and the wide kernel, whose start costs more,
// lose 4-20 % that way.
struct ChunkPlan {
    int64_t per_chunk, n_chunks, time;
};
inline ChunkPlan plan_chunks(const FwdParams &p, int64_t groups, int64_t num_cu, int64_t resident, int64_t fewest, bool level)
{
    const bool ragged = p.offsets != nullptr;
    const int64_t units = ragged ? p.total_tokens : p.b;
    const int64_t mean_len = (p.total_tokens + p.b - 1) / p.b; // (uniform: l_d)
    const bool two_rounds = level && ragged && groups == 1 && resident <= 2 && p.total_tokens >= 2500 * num_cu * resident * 2;
    ChunkPlan best = {1, 1, INT64_MAX};
    for (int64_t k = two_rounds ? 2 * resident : fewest; k <= 8 * resident; ++k) { // workgroups per CU
        int64_t chunks = num_cu * k / groups;
        chunks = chunks < 1 ? 1 : chunks > p.b ? p.b : chunks;
        int64_t per = (units + chunks - 1) / chunks;
        per = per < 1 ? 1 : per;
        const int64_t n = units < 1 ? 1 : (units + per - 1) / per;
        const int64_t tokens = ragged ? (per > mean_len ? per : mean_len) + mean_len / 2 : per * mean_len;
        const int64_t on_cu = (n * groups + num_cu - 1) / num_cu;
        int64_t time = on_cu * (tokens + 200);
        if (on_cu < resident) // (as many as fill the CU, where nothing says that fewer will do)
            time = fewest < resident ? (int64_t)((double)(on_cu * tokens) * std::sqrt((double)resident / (double)on_cu)) + on_cu * 200
                                     : resident * (tokens + 200);
        if (time < best.time)
            best = {per, n, time};
    }
    return best;
}

// Walks the tiles (32 tokens unless told otherwise) of documents [doc, doc_end), the same in every lane.  All
// state is 32-bit and uniform (scalar registers).  For ragged corpora the end of the NEXT document is
// fetched while the current one is walked, so that stepping to the next document waits for no memory.
struct TileIter {
    int doc, doc_end;
    int row0; // packed row of the current tile's first token
    int t0;   // document-local index of that token
    int len;  // tokens in the current document
    int end;  // packed row one past the current document (ragged only)
    int nxt;  // offsets[doc + 2], unclamped, fetched one document ahead (ragged only)
};

__device__ __forceinline__ bool it_valid(const TileIter &it) { return it.doc < it.doc_end; }

__device__ __forceinline__ int it_offset(OffsetsPtr off, const FwdParams &p, int i)
{
    const int64_t j = i < p.b ? (int64_t)i : p.b;
    return off[j];
}

// Enters document it.doc (whose first row is it.end of the previous one and whose unclamped end is it.nxt),
// skipping empty documents.  Offsets are forced into [previous end, T], so that offsets which are not
// non-decreasing or run past the corpus give wrong scores but never an address outside D.
__device__ __forceinline__ void it_enter_ragged(TileIter &it, const FwdParams &p, OffsetsPtr off)
{
    const int t_all = (int)p.total_tokens; // < 2^31
    while (it.doc < it.doc_end) {
        const int s = it.end;
        const int e = min(max(it.nxt, s), t_all);
        it.nxt = it_offset(off, p, it.doc + 2);
        it.row0 = s;
        it.end = e;
        it.len = e - s;
        it.t0 = 0;
        if (it.len > 0)
            return;
        it.doc += 1;
    }
}

__device__ __forceinline__ void it_init(TileIter &it, const FwdParams &p, OffsetsPtr off, int doc0, int doc1)
{
    it.doc = doc0;
    it.doc_end = doc1;
    it.row0 = it.t0 = it.len = it.end = it.nxt = 0;
    if (doc0 >= doc1)
        return;
    if (p.offsets) {
        it.end = min(max(it_offset(off, p, doc0), 0), (int)p.total_tokens);
        it.nxt = it_offset(off, p, doc0 + 1);
        it_enter_ragged(it, p, off);
    } else {
        it.row0 = doc0 * p.l_d;
        it.len = p.l_d;
    }
}

__device__ __forceinline__ void it_next(TileIter &it, const FwdParams &p, OffsetsPtr off, int rows = TILE_ROWS)
{
    it.t0 += rows;
    it.row0 += rows;
    if (it.t0 >= it.len) {
        it.doc += 1;
        if (p.offsets) {
            it_enter_ragged(it, p, off);
        } else {
            it.row0 = it.doc * p.l_d;
            it.t0 = 0;
        }
    }
}

} // namespace maxsim
