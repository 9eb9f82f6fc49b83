// Fused MaxSim forward for any embedding width (the "split-d" forward of the paper's appendix on fat embeddings: an
// inner loop over slabs of the embedding dimension, accumulated in fp32, with the reduction of Alg. 1 unchanged).
//
// The register-stationary kernels of forward_impl.h hold a query block's fragments for the whole embedding width, which
// pays up to rows of 512 bytes.  Here neither operand is stationary: a workgroup of eight wavefronts computes the
// similarities of a MACRO TILE of 256 document tokens x up to 256 query tokens, and both operands go from memory straight
// into LDS (no staging registers) in slabs of 128 bytes per row, a whole cache line.
//
// What bounds it: slabs of half a line, as the slab kernel of forward_splitd.hip has them, fetch every line twice from the
// L2, because the first half's neighbour has left the 32 KB L1 before the next slab asks for it.  Few query tokens: HBM,
// 5.9-6.2 TB/s at one to four blocks and d = 768-1024 (3.3-3.7 before: 1 x 32 tokens x 1000 x 512 rows 290 -> 177 us).  Many: power;
// 4 x 1024 tokens x 500 x 1024 rows of d = 1024 take 2990 us (1.44 PFLOP/s; 2490 on zero operands, where the clock stays up).  On
// 32x32 results, which are kept for fp32, with argmax and for rows of 64 bytes, they took 3300 (2580).  Four wavefronts of 128 x 128 similarities each, which
// read a third less from LDS, took the same time, and so did earlier loads and raised wavefront priorities; rows read
// ahead into the L2 cost 5 %.
//
//   One barrier per slab.  What a slab needs beside MFMAs, loads and operand reads (the next addresses, the end of a document) is
//   done before the barrier, three quarters into the slab's last MFMAs: behind it, where no wavefront has any out, it cost
//   16x16 results 6 % (3140 -> 2960 us; forward without argmax on 16-bit inputs).  The slab's k-steps are read from LDS one step ahead of the MFMAs that use them; the last
//   step's MFMAs run after the next barrier, under the first operand reads of the new slab.  The loads of the slab
//   that takes the place of the one just used go out between the MFMAs; two to four slabs are in LDS, as fit.
//
// The 32-row tiles of a macro tile are dealt to the row wavefronts in turn and tiles past the document's end are skipped,
// so a document costs its length rounded up to 32 tokens.  A macro tile never spans two documents.  When its last slab
// is done the accumulators are folded into the running max (and argmax) of the wavefront's query tokens as in the
// other kernels; at the end of a document the row wavefronts' maxima meet in LDS and the block sums are added in block
// order.  Queries of more than eight blocks take several passes over a document, one after the other, while its rows
// are in the caches.
#pragma once
#include "forward_impl.h"

namespace maxsim {

// per element type (forward_wide_{f16,bf16,f32}.hip)
hipError_t forward_wide_run_f16(const FwdParams &p, int row_bytes, int blocks, int blocks_per_pass, int rows, int grid, hipStream_t stream);
hipError_t forward_wide_allow_f16();
hipError_t forward_wide_run_bf16(const FwdParams &p, int row_bytes, int blocks, int blocks_per_pass, int rows, int grid, hipStream_t stream);
hipError_t forward_wide_allow_bf16();
hipError_t forward_wide_run_f32(const FwdParams &p, int row_bytes, int blocks, int blocks_per_pass, int rows, int grid, hipStream_t stream);
hipError_t forward_wide_allow_f32();

namespace {

constexpr int WD_W = 8;                 // wavefronts per workgroup
constexpr int WD_MAX_BLOCKS = 8;        // column blocks per workgroup (at most one per wavefront: they finish a block each)
constexpr int WD_SLAB = 128;            // bytes of every row in one slab: 8 chunks of 16
constexpr int WD_LDS_MAX = 160 * 1024;

// WR x WC wavefronts, MT tiles of 32 document tokens x NCB blocks of 32 query tokens each
template <int WR_, int WC_, int MT_, int NCB_> struct WideShape {
    static constexpr int WR = WR_, WC = WC_, MT = MT_, NCB = NCB_;
    static constexpr int BLOCKS = WC * NCB;
    static constexpr int COLS = BLOCKS * BLOCK_COLS;
    static constexpr int ROWS = WR * MT * TILE_ROWS; // document tokens per macro tile
    static constexpr int BUF = (ROWS + COLS) * WD_SLAB;
    static constexpr int RED = 2 * (2 * WR * COLS + WD_MAX_BLOCKS) * 4; // two sets of: maxima and winners per row wavefront, block sums
    static constexpr int N_BUF = (WD_LDS_MAX - RED) / BUF < 4 ? (WD_LDS_MAX - RED) / BUF : 4;
    static constexpr int LDS = N_BUF * BUF + RED;
    static constexpr int NA = ROWS / 64;                  // load instructions per wavefront and slab: 8 rows each
    static constexpr int NB = COLS >= 64 ? COLS / 64 : 1;
    static constexpr int NL = NA + NB;
    static_assert(WR * WC == WD_W && ROWS % 64 == 0 && BLOCKS <= WD_MAX_BLOCKS && N_BUF >= 2, "shape");
};

// Results of a kernel: 32x32; or 16x16, for rows of whole lines or with half a line at the end.  16-bit inputs without argmax take
// 16x16 but for rows that are half a line in all.
enum WideResults { WD_32, WD_16, WD_16_HALF };
inline WideResults wide_results(int dtype, bool argmax, int row_bytes)
{
    return argmax || dtype == MAXSIM_F32 || row_bytes < WD_SLAB ? WD_32 : (row_bytes & 64) != 0 ? WD_16_HALF : WD_16;
}

// One MFMA step (k = 16 for 16-bit inputs; a 16-byte chunk of fp32 is four steps of k = 2).
template <int DT> __device__ __forceinline__ void wide_mma(const i32x4 &a, const i32x4 &b, f32x16 &c)
{
    if constexpr (DT == MAXSIM_F16) {
        c = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
    } else if constexpr (DT == MAXSIM_BF16) {
        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            c = __builtin_amdgcn_mfma_f32_32x32x2f32(__int_as_float(a[e]), __int_as_float(b[e]), c, 0, 0, 0);
    }
}

// The same on 16x16 results, k = 32: a lane keeps four document tokens of one query token.  Half as many accumulator words
// travel per product, which the power limit turns into time (see Acc16).  Written as assembly because the compiler does not tie a
// result of four registers to its accumulator, and the largest shape's 32 of them spill.  The waits that the compiler puts in by
// itself elsewhere are written out: results_ready() before anything but an MFMA reads an accumulator, and two cycles between a
// move and an MFMA that reads what it wrote (tests/test_codegen.py looks for both).
template <int DT> __device__ __forceinline__ void wide_mma(const i32x4 &a, const i32x4 &b, f32x4 &c)
{
    if constexpr (DT == MAXSIM_F16)
        asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, %0" : "+v"(c) : "v"(a), "v"(b));
    else
        asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(a), "v"(b));
}
template <int DT, class Acc> __device__ __forceinline__ void wide_mma_first(const i32x4 &a, const i32x4 &b, Acc &c) // on zeros
{
    if constexpr (DT == MAXSIM_F16)
        asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, 0" : "=&v"(c) : "v"(a), "v"(b));
    else
        asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=&v"(c) : "v"(a), "v"(b));
}
// An MFMA's result may be read by other instructions some cycles after it (at most 11 for four passes); the operands keep the reads behind the wait
template <class Acc, int MR, int NR> __device__ __forceinline__ void results_ready(Acc (&acc)[MR][NR])
{
    asm volatile("s_nop 15" ::: "memory");
#pragma unroll
    for (int i = 0; i < MR; ++i)
#pragma unroll
        for (int j = 0; j < NR; ++j)
            asm volatile("" : "+v"(acc[i][j]));
}

// 16 bytes per lane from memory to 1 KB of LDS (lane l's go to dst + 16 l)
__device__ __forceinline__ void load_to_lds16(const char *src, char *dst)
{
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)src, (__attribute__((address_space(3))) void *)dst, 16, 0, 0);
}

// Barrier that waits for this wavefront's LDS operations but, unlike __syncthreads, not for its loads into LDS
__device__ __forceinline__ void lds_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// The position of a macro tile: the document's tile and which pass over the document
struct WidePos {
    TileIter it;
    int pass;
};
__device__ __forceinline__ void wide_next(WidePos &x, const FwdParams &p, OffsetsPtr off, int rows)
{
    if (x.it.t0 + rows >= x.it.len && x.pass + 1 < p.n_pass) { // the document again, for the query's next blocks
        x.pass += 1;
        x.it.row0 -= x.it.t0;
        x.it.t0 = 0;
        return;
    }
    if (x.it.t0 + rows >= x.it.len)
        x.pass = 0;
    it_next(x.it, p, off, rows);
}

// blocks_per_pass: column blocks of a query taken in one pass (n_pass > 1), else unused
template <int DT, class S, bool ARGMAX, WideResults RES>
__global__ void __launch_bounds__(WD_W * 64) fwd_wide_kernel(FwdParams p, OffsetsPtr off, int row_bytes, int blocks_per_pass)
{
    constexpr int WR = S::WR, WC = S::WC, MT = S::MT, NCB = S::NCB;
    constexpr bool R16 = RES != WD_32, HALF = RES == WD_16_HALF;
    // results per wavefront
    constexpr int MR = R16 ? 2 * MT : MT, NR = R16 ? 2 * NCB : NCB;
    extern __shared__ __attribute__((aligned(16))) char lds[];
    float *red_m = reinterpret_cast<float *>(lds + S::N_BUF * S::BUF);  // [2][WR][COLS]
    int *red_i = reinterpret_cast<int *>(red_m + 2 * WR * S::COLS);     // [2][WR][COLS]
    float *part = reinterpret_cast<float *>(red_i + 2 * WR * S::COLS);  // [2][WD_MAX_BLOCKS]

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int rho = lane & 31, h = lane >> 5;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wc = w % WC, wr = w / WC;
    const int n_slabs = (row_bytes + WD_SLAB - 1) / WD_SLAB;
    const bool half_last = R16 ? HALF : (row_bytes & 64) != 0; // the last slab is half a line wide

    // Workgroup ids are dealt round-robin to the 8 XCDs: every XCD takes a contiguous range of (chunk, group), so that
    // the column groups that share a document chunk meet in one L2
    const int v = xcd_grouped(blockIdx.x, gridDim.x);
    const int group = v % p.n_groups;
    const int chunk = v / p.n_groups;

    int64_t doc0_, doc1_;
    chunk_doc_range(p, chunk, doc0_, doc1_);
    if (doc0_ >= doc1_)
        return;
    const int doc0 = (int)doc0_, doc1 = (int)doc1_;
    if (group == 0)
        write_empty_docs(p, doc0, doc1, tid, WD_W * 64);

    const int q_first = p.n_pass == 1 ? group * p.qpg : group;
    const int nq = p.n_pass == 1 ? min(p.qpg, p.n_q - q_first) : 1;

    // Copy role: a load instruction takes 8 rows; this lane chunk cc of row r0 + 64 j.  A row's chunk c sits at position
    // c ^ ((row >> 1) & 7) of its 128 bytes, so that the 16 rows x 16 bytes of an operand read hit all banks once.
    const int r0 = w * 8 + (lane >> 3);
    const int cc = (lane & 7) ^ ((r0 >> 1) & 7);
    const int hi64 = cc >= 4 ? 64 : 0; // what a lane steps back in a slab of half a line (its data is then not used)
    // operand reads: lane (rho, h) takes chunk 2u + h of row rho of a 32-row tile in k-step u
    // (16x16 results: lane (c, g) takes chunk 4u + g of row c of 16)
    const int rd_r = R16 ? lane & 15 : rho, rd_g = R16 ? lane >> 4 : h;
    const int rd_row = rd_r * WD_SLAB, rd_swz = ((rd_r >> 1) & 7) << 4;

    WidePos li, ci; // loader (N_BUF - 1 slabs ahead) and compute position
    it_init(li.it, p, off, doc0, doc1);
    li.pass = 0;
    ci = li;
    if (!it_valid(ci.it))
        return;

    uint32_t a_off[S::NA], b_off[S::NB]; // byte offsets of this lane's chunks within the tile's rows / the group's queries
    const char *q_base = p.Q + (int64_t)q_first * p.l_q * row_bytes; // first query row of the pass
    auto query_rows = [&](int pass) {
        const int tok0 = pass * blocks_per_pass * BLOCK_COLS; // (one pass: 0)
        q_base = p.Q + ((int64_t)q_first * p.l_q + tok0) * row_bytes;
#pragma unroll
        for (int j = 0; j < S::NB; ++j) { // columns past the query or past the group's blocks re-read a valid row and are never summed
            const int r = S::COLS >= 64 ? r0 + 64 * j : (r0 & (S::COLS - 1));
            int q = 0, blk = r >> 5;
            if (p.n_pass == 1) {
                q = blk / p.bpq;
                blk -= q * p.bpq;
                if (q >= nq)
                    q = blk = 0;
            }
            b_off[j] = (uint32_t)((q * p.l_q + min(blk * BLOCK_COLS + (r & 31), p.l_q - 1 - tok0)) * row_bytes + cc * 16);
        }
    };
    int lks = 0;
    const char *l_a = p.D, *l_b = q_base;
    uint32_t l_back = 0;
    auto tile_rows = [&]() { // the loader enters a macro tile: rows past the document's end re-read its last token
        const int last = li.it.len - li.it.t0 - 1;
#pragma unroll
        for (int j = 0; j < S::NA; ++j)
            a_off[j] = (uint32_t)(min(r0 + 64 * j, last) * row_bytes + cc * 16);
        l_a = p.D + (int64_t)li.it.row0 * row_bytes;
        if (p.n_pass > 1)
            query_rows(li.pass);
        l_b = q_base;
    };
    // Addresses of the loader's slab; past the end of the stream the last slab is loaded again (in bounds, never used)
    auto next_slab = [&]() {
        if (!it_valid(li.it))
            return;
        if (lks == n_slabs) {
            wide_next(li, p, off, S::ROWS);
            if (!it_valid(li.it))
                return;
            lks = 0;
        }
        if (lks == 0) {
            tile_rows();
        } else {
            l_a += WD_SLAB;
            l_b += WD_SLAB;
        }
        lks += 1;
        l_back = half_last && lks == n_slabs ? (uint32_t)hi64 : 0u;
    };
    auto load1 = [&](int k, int buf) {
        if (k < S::NA) {
            load_to_lds16(l_a + (a_off[k] - l_back), lds + buf + (w * 8 + 64 * k) * WD_SLAB);
        } else {
            const int j = k - S::NA;
            const int row = S::COLS >= 64 ? w * 8 + 64 * j : ((w * 8) & (S::COLS - 1)); // (32 columns: two wavefronts load the same rows)
            load_to_lds16(l_b + (b_off[j] - l_back), lds + buf + (S::ROWS + row) * WD_SLAB);
        }
    };

    if (p.n_pass == 1)
        query_rows(0);
#pragma unroll
    for (int s = 0; s < S::N_BUF - 1; ++s) {
        next_slab();
#pragma unroll
        for (int k = 0; k < S::NL; ++k)
            load1(k, s * S::BUF);
    }
    if constexpr (R16)
        next_slab();
    int o_cur = 0, o_wr = (S::N_BUF - 1) * S::BUF;

    std::conditional_t<R16, f32x4, f32x16> acc[MR][NR];
    float m[NR];
    int idx[NR];
    float run = 0.0f; // thread 0: sum over the passes of a document so far
#pragma unroll
    for (int c = 0; c < NR; ++c) {
        m[c] = neg_inf();
        idx[c] = 0;
    }

    i32x4 fa[2][MR], fb[2][NR]; // (16x16: rows below MR1 only have the first set)
    auto read1 = [&](auto set, int buf, int u, int i) { // operand i of k-step u: b0, a0, b1, a1, ... in the order of use
        constexpr int X = decltype(set)::value;
        const int at = buf + rd_row + (((2 * u + h) << 4) ^ rd_swz);
        const int pairs = MT < NCB ? MT : NCB;
        const bool is_b = i < 2 * pairs ? (i & 1) == 0 : MT < NCB;
        const int j = i < 2 * pairs ? i >> 1 : i - pairs;
        if (is_b)
            fb[X][j] = *reinterpret_cast<const i32x4 *>(lds + at + (S::ROWS + (wc * NCB + j) * BLOCK_COLS) * WD_SLAB);
        else
            fa[X][j] = *reinterpret_cast<const i32x4 *>(lds + at + (j * WR + wr) * (TILE_ROWS * WD_SLAB));
    };
    // The end of a document takes two barriers, both of them barriers of slabs that follow: behind the first a wavefront per
    // block merges the row wavefronts' maxima, behind the second the blocks are added up.  Two sets of LDS words in turn.
    int par = 0;
    int fin_doc = -1, fin_len = 0, fin_pass = 0; // its maxima are in set `par`
    int sum_doc = -1, sum_pass = 0;              // its block sums are in set `par ^ 1`
    auto finish = [&]() {
        if (sum_doc >= 0) {
            if (tid < nq) { // thread t adds up the blocks of its query in block order
                const int first = p.n_pass == 1 ? tid * p.bpq : 0;
                const int cnt = p.n_pass == 1 ? p.bpq : min(blocks_per_pass, p.bpq - sum_pass * blocks_per_pass);
                float sum = 0.0f;
                for (int i = 0; i < cnt; ++i)
                    sum += part[(par ^ 1) * WD_MAX_BLOCKS + first + i];
                run = sum_pass > 0 ? run + sum : sum;
                if (sum_pass == p.n_pass - 1)
                    p.scores[(int64_t)(q_first + tid) * p.ld + sum_doc] = run;
            }
            sum_doc = -1;
        }
        if (fin_doc >= 0) {
            const int blk0 = p.n_pass == 1 ? 0 : fin_pass * blocks_per_pass;
            const int nb = p.n_pass == 1 ? nq * p.bpq : min(blocks_per_pass, p.bpq - blk0);
            if (w < nb) { // the lower row of equal maxima wins
                const int at = par * WR * S::COLS + w * BLOCK_COLS + rho;
                float mm = red_m[at];
                int win = ARGMAX ? red_i[at] : 0;
#pragma unroll
                for (int x = 1; x < WR; ++x) {
                    const float mo = red_m[at + x * S::COLS];
                    if (ARGMAX) {
                        const int io = red_i[at + x * S::COLS];
                        win = mo > mm || (mo == mm && io < win) ? io : win;
                    }
                    mm = fmaxf(mm, mo);
                }
                const int q = p.n_pass == 1 ? w / p.bpq : 0;
                const int tok = (p.n_pass == 1 ? w - q * p.bpq : blk0 + w) * BLOCK_COLS + rho;
                const bool valid = tok < p.l_q;
                if (ARGMAX && valid && h == 0)
                    p.argmax[((int64_t)(q_first + q) * p.ld + fin_doc) * p.l_q + tok] = min(win, fin_len - 1);
                const float sum = sum_low32(valid ? mm : 0.0f);
                if (lane == 0)
                    part[par * WD_MAX_BLOCKS + w] = sum;
            }
            sum_doc = fin_doc;
            sum_pass = fin_pass;
            fin_doc = -1;
            par ^= 1;
        }
    };

    constexpr int SLOTS = MT * NCB, READS = MT + NCB;
    // MFMAs of a k-step from one register set while the other is read for k-step `u` of buffer `buf` (u < 0: none) and
    // loads [ld0, ld1) of the slab that is due go out.  WHOLE: all MT tiles have rows, else the first `nt`.
    auto step = [&](auto set, auto whole, int nt, auto compute, int buf, int u, auto ld0_tag, auto ld1_tag) {
        constexpr int X = decltype(set)::value;
        constexpr bool WHOLE = decltype(whole)::value, COMPUTE = decltype(compute)::value;
        constexpr int LD0 = decltype(ld0_tag)::value, LD1 = decltype(ld1_tag)::value;
#pragma unroll
        for (int i = 0; i < SLOTS; ++i) {
            const int t = i / NCB, c = i % NCB;
            if constexpr (!R16 && COMPUTE)
                if (WHOLE || t < nt)
                    wide_mma<DT>(fa[X][t], fb[X][c], acc[t][c]);
            if (u >= 0) {
#pragma unroll
                for (int r = 0; r < READS; ++r)
                    if ((r * SLOTS) / READS == i)
                        read1(std::integral_constant<int, X ^ 1>{}, buf, u, r);
            }
            if constexpr (LD1 > LD0) {
#pragma unroll
                for (int k = LD0; k < LD1; ++k)
                    if (((k - LD0) * SLOTS) / (LD1 - LD0) == i)
                        load1(k, o_wr);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // The same for 16x16 results, whose k-steps are twice as long.  The operands of the first MR1 rows are replaced in place once
    // the row's MFMAs are out (two sets of all rows do not fit); the others early, so that the last read is well ahead of the
    // barrier that waits for it.  `tail`: the slab's last k-step.
    constexpr int MR1 = MR <= 4 ? 0 : HALF ? MR : MR - 2; // (HALF: registers)
    auto step16 = [&](auto set, auto whole, int nt, auto compute, int buf, int u, auto ld0_tag, auto ld1_tag, auto tail) {
        constexpr int X = decltype(set)::value;
        constexpr bool WHOLE = decltype(whole)::value;
        constexpr int COMPUTE = decltype(compute)::value; // 0: nothing, 1: yes, 2: the first k-step of a macro tile
        constexpr int LD0 = decltype(ld0_tag)::value, LD1 = decltype(ld1_tag)::value;
        constexpr int SLOT_N = MR * NR, EARLY = SLOT_N * 3 / 4;
        const int at = buf + rd_row + (((4 * u + rd_g) << 4) ^ rd_swz);
        auto read_a = [&](int i) { return *reinterpret_cast<const i32x4 *>(lds + at + ((i / 2) * WR + wr) * (TILE_ROWS * WD_SLAB) + i % 2 * (16 * WD_SLAB)); };
        static_for<SLOT_N>([&](auto slot_tag) {
            constexpr int slot = decltype(slot_tag)::value, i = slot / NR, j = slot % NR;
            auto mma = [&](auto row, auto col) {
                constexpr int y = decltype(row)::value, x = decltype(col)::value;
                if constexpr (R16 && COMPUTE == 1)
                    wide_mma<DT>(fa[y < MR1 ? 0 : X][y], fb[X][x], acc[y][x]);
                else if constexpr (R16 && COMPUTE == 2)
                    wide_mma_first<DT>(fa[y < MR1 ? 0 : X][y], fb[X][x], acc[y][x]);
            };
            if constexpr (WHOLE) {
                mma(std::integral_constant<int, i>{}, std::integral_constant<int, j>{});
            } else if constexpr (i % 2 == 0 && j == 0) { // one branch for a tile of 32 rows
                if (i < 2 * nt)
                    static_for<2 * NR>([&](auto k) {
                        mma(std::integral_constant<int, i + decltype(k)::value / NR>{}, std::integral_constant<int, decltype(k)::value % NR>{});
                    });
            }
            if (u >= 0) {
                if constexpr (i < MR1 && j == NR - 1)
                    fa[0][i] = read_a(i);
#pragma unroll
                for (int r = 0; r < NR + MR - MR1; ++r)
                    if ((r * EARLY) / (NR + MR - MR1) == slot) {
                        if (r < NR)
                            fb[X ^ 1][r] = *reinterpret_cast<const i32x4 *>(lds + at + (S::ROWS + wc * NCB * BLOCK_COLS + r * 16) * WD_SLAB);
                        else
                            fa[X ^ 1][MR1 + r - NR] = read_a(MR1 + r - NR);
                    }
            }
            if constexpr (LD1 > LD0) {
#pragma unroll
                for (int k = LD0; k < LD1; ++k)
                    if (((k - LD0) * EARLY) / (LD1 - LD0) == slot)
                        load1(k, o_wr);
            }
            if constexpr (decltype(tail)::value && slot == EARLY) {
                next_slab();
                finish();
            }
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    constexpr std::integral_constant<int, 0> s0{};
    constexpr std::integral_constant<int, 1> s1{};
    constexpr std::integral_constant<int, 0> L0{};
    constexpr std::integral_constant<int, (S::NL + 1) / 2> L1{};
    constexpr std::integral_constant<int, S::NL> L2{};

    // this slab has landed for every wavefront, and every wavefront has read the one whose place is taken next
    auto enter_slab = [&]() {
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(S::NL * (S::N_BUF - 2)) : "memory");
        lds_barrier();
        if constexpr (!R16) {
            finish();
            next_slab();
        }
    };
    auto leave_slab = [&]() {
        o_wr = o_cur;
        o_cur = o_cur == (S::N_BUF - 1) * S::BUF ? 0 : o_cur + S::BUF;
    };
    auto macro_tile = [&](auto whole, int nt) {
        if constexpr (R16) {
            // (No branch around the MFMAs of a slab: with one, accumulators are copied on both sides of it and take twice the registers.)
            auto slab = [&](auto first) {
                constexpr int FIRST = decltype(first)::value;
                enter_slab();
                step16(s1, whole, nt, std::integral_constant<int, FIRST ? 0 : 1>{}, o_cur, 0, L0, L1, std::false_type{}); // the last step of the slab before
                step16(s0, whole, nt, std::integral_constant<int, FIRST ? 2 : 1>{}, o_cur, 1, L1, L2, std::true_type{});
                leave_slab();
            };
            auto half_slab = [&]() { // one k-step, which is computed where the second one would be
                enter_slab();
                step16(s1, whole, nt, s1, o_cur, 0, L0, L2, std::true_type{});
#pragma unroll
                for (int j = 0; j < NR; ++j)
                    fb[1][j] = fb[0][j];
#pragma unroll
                for (int i = MR1; i < MR; ++i)
                    fa[1][i] = fa[0][i];
                leave_slab();
            };
            if constexpr (HALF) {
                slab(s1); // (there are two slabs at least)
                for (int s = 2; s < n_slabs; ++s)
                    slab(s0);
                half_slab();
            } else {
                slab(s1);
                for (int s = 1; s < n_slabs; ++s)
                    slab(s0);
            }
            asm volatile("s_nop 1" ::: "memory"); // (two cycles between a move and the MFMA that reads what it wrote)
            step16(s1, whole, nt, s1, 0, -1, L0, L0, std::false_type{}); // the last slab's last step
            results_ready(acc);
#pragma unroll
            for (int j = 0; j < NR; ++j)
#pragma unroll
                for (int i = 0; i < MR; ++i)
                    if (decltype(whole)::value || i < 2 * nt) {
                        m[j] = fmaxf(fmaxf(m[j], acc[i][j][0]), acc[i][j][1]);
                        m[j] = fmaxf(fmaxf(m[j], acc[i][j][2]), acc[i][j][3]);
                    }
        } else {
#pragma unroll
            for (int t = 0; t < MT; ++t)
#pragma unroll
                for (int c = 0; c < NCB; ++c)
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        acc[t][c][r] = 0.0f;
            auto slab = [&](auto first, bool half) {
                enter_slab();
                step(s1, whole, nt, std::bool_constant<!decltype(first)::value>{}, o_cur, 0, L0, L1); // the last step of the slab before
                step(s0, whole, nt, std::true_type{}, o_cur, 1, L1, L2);
                if (!half) {
                    step(s1, whole, nt, std::true_type{}, o_cur, 2, L0, L0);
                    step(s0, whole, nt, std::true_type{}, o_cur, 3, L0, L0);
                }
                leave_slab();
            };
            slab(std::true_type{}, half_last && n_slabs == 1);
            for (int s = 1; s < n_slabs; ++s)
                slab(std::false_type{}, half_last && s == n_slabs - 1);
            step(s1, whole, nt, std::true_type{}, 0, -1, L0, L0); // the last slab's last step: k-step 3, or 1 of half a slab
#pragma unroll
            for (int c = 0; c < NCB; ++c)
#pragma unroll
                for (int t = 0; t < MT; ++t)
                    if (decltype(whole)::value || t < nt)
                        fold_tile<ARGMAX>(acc[t][c], m[c], idx[c], ci.it.t0 + (t * WR + wr) * TILE_ROWS, h);
        }
    };

    while (it_valid(ci.it)) {
        // tiles of this wavefront that hold rows of the document
        const int tiles = (ci.it.len - ci.it.t0 + TILE_ROWS - 1) / TILE_ROWS;
        const int nt = tiles <= wr ? 0 : (tiles - wr + WR - 1) / WR;
        if (nt >= MT)
            macro_tile(std::true_type{}, MT);
        else
            macro_tile(std::false_type{}, nt);
        if (ci.it.t0 + S::ROWS >= ci.it.len) { // last macro tile of the document (and pass)
            if constexpr (R16) { // a block's two halves side by side, two quarters of the rows merged; then the other two
#pragma unroll
                for (int c = 0; c < NCB; ++c) {
                    const auto x = __builtin_amdgcn_permlane32_swap(__float_as_uint(m[2 * c]), __float_as_uint(m[2 * c + 1]), false, false);
                    const uint32_t y = __float_as_uint(fmaxf(__uint_as_float(x[0]), __uint_as_float(x[1])));
                    const auto z = __builtin_amdgcn_permlane16_swap(y, y, false, false);
                    if ((lane & 16) == 0)
                        red_m[(par * WR + wr) * S::COLS + (wc * NCB + c) * BLOCK_COLS + (h << 4) + (lane & 15)] = fmaxf(__uint_as_float(z[0]), __uint_as_float(z[1]));
                    m[2 * c] = m[2 * c + 1] = neg_inf();
                }
            }
#pragma unroll
            for (int c = 0; c < (R16 ? 0 : NCB); ++c) {
                const int col = (wc * NCB + c) * BLOCK_COLS + rho;
                float a, b;
                swap_halves(m[c], a, b);
                float mm = fmaxf(a, b);
                if (ARGMAX) {
                    float ia, ib;
                    swap_halves(__int_as_float(idx[c]), ia, ib);
                    const int i0 = __float_as_int(ia), i1 = __float_as_int(ib);
                    const bool take = a > b || (a == b && i0 < i1);
                    if (h == 0)
                        red_i[(par * WR + wr) * S::COLS + col] = take ? i0 : i1;
                }
                if (h == 0)
                    red_m[(par * WR + wr) * S::COLS + col] = mm;
                m[c] = neg_inf();
                idx[c] = 0;
            }
            fin_doc = ci.it.doc;
            fin_len = ci.it.len;
            fin_pass = ci.pass;
        }
        wide_next(ci, p, off, S::ROWS);
    }
    lds_barrier();
    finish();
    lds_barrier();
    finish();
    // the loads past the end of the stream must have landed before this LDS is another workgroup's
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// Shapes by column blocks per workgroup: with fewer of them the wavefronts share the rows instead, so that all eight
// have work, and more slabs fit into LDS.  Short documents (`rows`: their mean length) take macro tiles of 128 or 64 rows, of a
// larger one most loads would repeat the last token.
template <typename F> auto with_shape(int blocks, int rows, F &&f)
{
    if (rows <= 128) {
        if (blocks > 4 && rows <= 64)
            return f(WideShape<2, 4, 1, 2>{});
        if (blocks <= 2)
            return f(WideShape<4, 2, 1, 1>{});
        if (blocks <= 4)
            return f(WideShape<4, 2, 1, 2>{});
        return f(WideShape<2, 4, 2, 2>{});
    }
    if (blocks <= 1)
        return f(WideShape<8, 1, 1, 1>{});
    if (blocks <= 2)
        return f(WideShape<8, 1, 1, 2>{});
    if (blocks <= 4)
        return f(WideShape<4, 2, 2, 2>{});
    if (blocks <= 6)
        return f(WideShape<4, 2, 2, 3>{});
    return f(WideShape<2, 4, 4, 2>{});
}

template <int DT, bool ARGMAX> hipError_t allow_wide_lds()
{
    for (int shape = 0; shape < 9; ++shape) {
        constexpr int blocks[9] = {1, 2, 4, 6, 8, 2, 4, 8, 8}, rows[9] = {256, 256, 256, 256, 256, 128, 128, 128, 64};
        const hipError_t e = with_shape(blocks[shape], rows[shape], [](auto s) {
            using S = decltype(s);
            auto allow = [](auto res) {
                return hipFuncSetAttribute(reinterpret_cast<const void *>(&fwd_wide_kernel<DT, S, ARGMAX, decltype(res)::value>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                           S::LDS);
            };
            hipError_t e = allow(std::integral_constant<WideResults, WD_32>{});
            if constexpr (!ARGMAX && DT != MAXSIM_F32) {
                e = e != hipSuccess ? e : allow(std::integral_constant<WideResults, WD_16>{});
                e = e != hipSuccess ? e : allow(std::integral_constant<WideResults, WD_16_HALF>{});
            }
            return e;
        });
        if (e != hipSuccess)
            return e;
    }
    return hipSuccess;
}

template <int DT, bool ARGMAX> hipError_t launch_wide(const FwdParams &p, int row_bytes, int blocks, int blocks_per_pass, int rows, int grid, hipStream_t stream)
{
    return with_shape(blocks, rows, [&](auto s) {
        using S = decltype(s);
        auto launch = [&](auto res) {
            hipLaunchKernelGGL((fwd_wide_kernel<DT, S, ARGMAX, decltype(res)::value>), dim3(grid), dim3(WD_W * 64), S::LDS, stream, p, p.offsets, row_bytes, blocks_per_pass);
        };
        const WideResults res = wide_results(DT, ARGMAX, row_bytes);
        if constexpr (!ARGMAX && DT != MAXSIM_F32) {
            if (res == WD_16)
                launch(std::integral_constant<WideResults, WD_16>{});
            else if (res == WD_16_HALF)
                launch(std::integral_constant<WideResults, WD_16_HALF>{});
        }
        if (res == WD_32)
            launch(std::integral_constant<WideResults, WD_32>{});
        return hipGetLastError();
    });
}

template <int DT> hipError_t run_wide(const FwdParams &p, int row_bytes, int blocks, int blocks_per_pass, int rows, int grid, hipStream_t stream)
{
    return p.argmax ? launch_wide<DT, true>(p, row_bytes, blocks, blocks_per_pass, rows, grid, stream)
                    : launch_wide<DT, false>(p, row_bytes, blocks, blocks_per_pass, rows, grid, stream);
}
template <int DT> hipError_t allow_wide()
{
    const hipError_t e = allow_wide_lds<DT, false>();
    return e == hipSuccess ? allow_wide_lds<DT, true>() : e;
}

} // namespace
} // namespace maxsim
