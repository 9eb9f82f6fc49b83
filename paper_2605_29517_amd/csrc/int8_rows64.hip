// int8 scoring of many query tokens against documents of equal length: 64 document tokens per step.
//
// Document-stationary like fwd_i8_doc_kernel (int8.hip, where the arithmetic is explained): the query tokens of a group sit in
// LDS, a wavefront keeps a tile of document tokens in registers and walks the column blocks.  That kernel reads 1 KB of query
// operands from LDS per 32x32x32 MFMA; here a tile is 64 tokens high, so an operand serves twice the products, and the results
// are 16x16, of which a lane keeps four document tokens: the scales of its rows take 32 registers where 32x32 results of 64
// rows take 64, and chains of two MFMAs need 32 accumulators instead of 48, which is what lets 64 rows, the next tile and 1024
// query tokens' maxima fit the 256 registers of two wavefronts per SIMD.
//
// What bounds it: power (1024 tokens x 40 000 x 1024: 4504 us, 2385 TOP/s; 4766 by fwd_i8_doc_kernel on the same box; 3306 on zero
// operands), below some thousand documents how evenly they are shared out (1024 x 3000 x 1024 402 -> 355 us, 602 x 1500 x 422
// 94 -> 57), up to four blocks of columns HBM.
#include "int8_impl.h"

namespace maxsim {
namespace {

constexpr int R64_WAVES = 8;
constexpr int R64_ROWS = 64;       // document tokens per tile: four results of 16 rows
constexpr int R64_COLS = 16;       // query tokens per column block
constexpr int R64_MAX_BLOCKS = 64; // column blocks per group (1024 query tokens)

constexpr int R64_HALF_BLOCKS = 36; // with more of them a second walk, over the last 32 tokens of a document, spills registers

constexpr int r64_quads(int nc) { return (nc + 3) / 4; } // registers that hold a document's maxima, four blocks each
// query rows, query scales, and the maxima of the seven wavefronts whose first document another one has begun
constexpr size_t r64_lds(int nc) { return (size_t)nc * R64_COLS * I8_ROW_BYTES + (size_t)R64_WAVES * r64_quads(nc) * 64 * sizeof(float); }

__device__ __forceinline__ float max_pair32(float x, float y) // lanes 0-31: x over both halves, lanes 32-63: y
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float max_pair16(float x, float y) // rows of 16 lanes: x's rows 0+1, y's 0+1, x's 2+3, y's 2+3
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ double sum64(double v)
{
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)b, (uint32_t)b, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(b >> 32), (uint32_t)(b >> 32), false, false);
    return sum32(__builtin_bit_cast(double, (uint64_t)hi[0] << 32 | lo[0]) + __builtin_bit_cast(double, (uint64_t)hi[1] << 32 | lo[1]));
}

// Score of a document.  mm[i] in lane l: the maximum of query token 64 i + l of the group, negative ones halved.  One IEEE
// multiply by the query scale per token, fp64 sums over a query's tokens, one rounding (p.bpq: blocks of 16 per query).
template <int NQUAD>
__device__ __forceinline__ void r64_finish(const I8Params &P, const float (&mm)[NQUAD], const float *q_scale, int nq, int q_first, int doc, int lane)
{
    const FwdParams &p = P.f;
    int l_q = p.l_q, bpq = p.bpq;
    asm volatile("" : "+s"(l_q), "+s"(bpq)); // (else the masks of all registers are formed before the walk and kept)
    double dv = 0.0;
    int j = 0, lo = 0; // query inside the group, its first block
#pragma unroll
    for (int i = 0; i < NQUAD; ++i) {
        float x = mm[i];
        x = x < 0.0f ? x + x : x;
        const float r = q_scale[i * 64 + lane] * x;
        const int blk = 4 * i + (lane >> 4);
        while (j < nq && lo < 4 * i + 4) { // queries that have blocks in this register
            const int tok = (blk - lo) * R64_COLS + (lane & 15);
            dv += tok >= 0 && tok < l_q ? (double)r : 0.0;
            if (lo + bpq > 4 * i + 4)
                break; // goes on in the next one
            dv = sum64(dv);
            if (lane == 0)
                P.scores[(int64_t)(q_first + j) * p.ld + doc] = (float)dv;
            dv = 0.0;
            ++j;
            lo += bpq;
        }
    }
}

// Tiles of a workgroup's documents are dealt to its wavefronts in contiguous shares that may begin and end inside a document,
// so that few documents keep all wavefronts equally busy.  A wavefront's maxima of a document that another one began go to LDS;
// the one that began it adds them in after the only barrier of the walk.  The last tile of a document begins 64 tokens before
// its end: tokens that are seen twice do not change a maximum, and no row index needs a bound.
template <int NC>
__global__ void __launch_bounds__(R64_WAVES * 64) fwd_i8_rows64_kernel(I8Params P)
{
    constexpr int NQUAD = r64_quads(NC);
    const FwdParams &p = P.f;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    float *q_scale = reinterpret_cast<float *>(smem + NC * R64_COLS * I8_ROW_BYTES);
    float *heads = q_scale + NQUAD * 64; // [7][NQUAD * 64]

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int c = lane & 15, g = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);

    const int v = xcd_grouped(blockIdx.x, gridDim.x); // the groups of a chunk meet in one L2
    const int group = v % p.n_groups;
    const int chunk = v / p.n_groups;
    const int q_first = group * p.qpg;
    const int nq = min(p.qpg, p.n_q - q_first);

    // Query rows, padding columns as zeros.  Chunk k of column x sits at k ^ ((x >> 1) & 7): the sixteen rows of an operand read hit all banks.
    for (int i = tid; i < NC * R64_COLS * 8; i += R64_WAVES * 64) {
        const int col = i >> 3, part = i & 7;
        const int blk = col / R64_COLS, q = blk / p.bpq;
        const int tok = (blk - q * p.bpq) * R64_COLS + col % R64_COLS;
        uint4 x = make_uint4(0, 0, 0, 0);
        if (q < nq && tok < p.l_q)
            x = *reinterpret_cast<const uint4 *>(P.Q + ((int64_t)(q_first + q) * p.l_q + tok) * I8_ROW_BYTES + part * 16);
        *reinterpret_cast<uint4 *>(smem + col * I8_ROW_BYTES + (part ^ ((col >> 1) & 7)) * 16) = x;
    }
    for (int col = tid; col < NQUAD * 64; col += R64_WAVES * 64) {
        const int blk = col / R64_COLS, q = blk / p.bpq;
        const int tok = (blk - q * p.bpq) * R64_COLS + col % R64_COLS;
        q_scale[col] = q < nq && tok < p.l_q ? P.qs[(int64_t)(q_first + q) * p.l_q + tok] : 0.0f;
    }
    __syncthreads();

    const int doc0 = (int)min((int64_t)chunk * p.unit_per_chunk, p.b);
    const int doc1 = (int)min((int64_t)doc0 + p.unit_per_chunk, p.b);
    const int per_doc = (p.l_d + R64_ROWS - 1) / R64_ROWS;
    const bool half_last = p.l_d % R64_ROWS != 0 && p.l_d % R64_ROWS <= R64_ROWS / 2;
    const int all = (doc1 - doc0) * per_doc;
    auto share = [&](int i) { return (int)((int64_t)all * i / R64_WAVES); }; // first tile of wavefront i
    const int t_first = share(w), t_end = share(w + 1);

    float mm[NQUAD];
    int open_doc = -1; // the document this wavefront began and did not end
    if (t_first < t_end) {
        int l_doc = doc0 + t_first / per_doc, l_t = t_first % per_doc, l_left = t_end - t_first - 1;
        const char *base = P.D + c * I8_ROW_BYTES + g * 16;
        i32x4 a_n[4][2];
        float s_n;
        auto gload = [&]() { // past the end of the share its last tile again: a load that may not be there would make every wait one for all of them
            const int row = l_doc * p.l_d + min(l_t * R64_ROWS, p.l_d - R64_ROWS);
            const char *src = base + (int64_t)row * I8_ROW_BYTES;
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int u = 0; u < 2; ++u)
                    a_n[s][u] = *reinterpret_cast<const i32x4 *>(src + s * (16 * I8_ROW_BYTES) + u * 64);
            s_n = P.ds[row + lane];
            if (l_left > 0) {
                l_left -= 1;
                l_t += 1;
                if (l_t == per_doc) {
                    l_t = 0;
                    l_doc += 1;
                }
            }
        };
        int doc = l_doc, t = l_t;
        bool begun = t == 0; // this wavefront has the current document from its first tile on
        gload();

        i32x4 seed;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            int x = 0x4B000000;
            asm volatile("" : "+v"(x));
            seed[r] = x;
        }
        float m[4 * NQUAD];
#pragma unroll
        for (int k = 0; k < 4 * NQUAD; ++k)
            m[k] = neg_inf();
        const int swz = (c >> 1) & 7;
        const char *qb0 = smem + c * I8_ROW_BYTES + ((g ^ swz) << 4);
        const char *qb1 = smem + c * I8_ROW_BYTES + (((4 + g) ^ swz) << 4);

        for (int left = t_end - t_first; left > 0; --left) {
            i32x4 a[4][2];
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int u = 0; u < 2; ++u)
                    a[s][u] = a_n[s][u];
            const float s_cur = s_n;
            gload();
            float sc[4][4], bi[4][4]; // of rows 16 s + 4 g + r
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    sc[s][r] = __int_as_float(__builtin_amdgcn_ds_bpermute((16 * s + 4 * g + r) * 4, __float_as_int(s_cur)));
                    bi[s][r] = sc[s][r] * -8388608.0f;
                }

            // Results S0 .. 3 of the tile's rows against all blocks: step by step one MFMA of block k and its part of the fold of block k - 1
            auto walk = [&](auto from) {
                constexpr int S0 = decltype(from)::value, NS = 4 - S0;
                i32x4 acc[2][4], qb[2][2];
                qb[0][0] = *reinterpret_cast<const i32x4 *>(qb0);
                qb[0][1] = *reinterpret_cast<const i32x4 *>(qb1);
                __builtin_amdgcn_sched_barrier(0);
                static_for<NC + 1>([&](auto block) {
                    constexpr int k = decltype(block)::value;
                    constexpr int X = k & 1;
                    static_for<2 * NS>([&](auto step) {
                        constexpr int s = S0 + decltype(step)::value % NS, u = decltype(step)::value / NS;
                        if constexpr (k < NC) {
                            acc[X][s] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[s][u], qb[X][u], u == 0 ? seed : acc[X][s], 0, 0, 0);
                            if constexpr (k + 1 < NC && s == S0)
                                qb[X ^ 1][u] = *reinterpret_cast<const i32x4 *>((u == 0 ? qb0 : qb1) + (k + 1) * (R64_COLS * I8_ROW_BYTES));
                        }
                        if constexpr (k > 0) {
                            constexpr int e = S0 + decltype(step)::value / 2, r = decltype(step)::value % 2 * 2;
                            const float v0 = __builtin_fmaf(__int_as_float(acc[X ^ 1][e][r]), sc[e][r], bi[e][r]);
                            const float v1 = __builtin_fmaf(__int_as_float(acc[X ^ 1][e][r + 1]), sc[e][r + 1], bi[e][r + 1]);
                            m[k - 1] = fmaxf(fmaxf(m[k - 1], v0), v1);
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    });
                });
            };
            if (NC <= R64_HALF_BLOCKS && half_last && t + 1 == per_doc)
                walk(std::integral_constant<int, NC <= R64_HALF_BLOCKS ? 2 : 0>{});
            else
                walk(std::integral_constant<int, 0>{});

            const bool last = t + 1 == per_doc;
            if (last || left == 1) {
#pragma unroll
                for (int i = 0; i < NQUAD; ++i)
                    mm[i] = max_pair16(max_pair32(m[4 * i], m[4 * i + 2]), max_pair32(m[4 * i + 1], m[4 * i + 3]));
                if (!begun) {
#pragma unroll
                    for (int i = 0; i < NQUAD; ++i)
                        heads[((w - 1) * NQUAD + i) * 64 + lane] = mm[i];
                } else if (last) {
                    r64_finish<NQUAD>(P, mm, q_scale, nq, q_first, doc, lane);
                } else {
                    open_doc = doc;
                }
#pragma unroll
                for (int k = 0; k < 4 * NQUAD; ++k)
                    m[k] = neg_inf();
            }
            t += 1;
            if (last) {
                t = 0;
                doc += 1;
                begun = true;
            }
        }
    }
    __syncthreads();
    if (open_doc >= 0) {
        const int doc_end = (open_doc - doc0 + 1) * per_doc;
        for (int x = w + 1; x < R64_WAVES && share(x) < doc_end; ++x) { // (tiles are left, so every such share but an empty one begins with this document)
            if (share(x) == share(x + 1))
                continue;
#pragma unroll
            for (int i = 0; i < NQUAD; ++i)
                mm[i] = fmaxf(mm[i], heads[((x - 1) * NQUAD + i) * 64 + lane]);
        }
        r64_finish<NQUAD>(P, mm, q_scale, nq, q_first, open_doc, lane);
    }
}

// f(integral_constant<int, NC>) for the smallest NC built that holds nc column blocks
template <typename F> hipError_t r64_with_blocks(int nc, F &&f)
{
#define MAXSIM_BLOCKS(N) if (nc <= N) return f(std::integral_constant<int, N>{});
    MAXSIM_BLOCKS(4) MAXSIM_BLOCKS(6) MAXSIM_BLOCKS(8) MAXSIM_BLOCKS(10) MAXSIM_BLOCKS(12) MAXSIM_BLOCKS(14) MAXSIM_BLOCKS(16) MAXSIM_BLOCKS(20) MAXSIM_BLOCKS(24)
    MAXSIM_BLOCKS(28) MAXSIM_BLOCKS(32) MAXSIM_BLOCKS(36) MAXSIM_BLOCKS(40) MAXSIM_BLOCKS(44) MAXSIM_BLOCKS(48) MAXSIM_BLOCKS(52) MAXSIM_BLOCKS(56)
    MAXSIM_BLOCKS(60) MAXSIM_BLOCKS(64)
#undef MAXSIM_BLOCKS
    return hipErrorInvalidValue;
}
// Rows that are multiplied of a document of l_d tokens
int64_t r64_rows(bool whole, int l_d)
{
    const int64_t r = whole ? R64_ROWS : R64_ROWS / 2;
    return (l_d + r - 1) / r * r;
}
int r64_built(int nc)
{
    int n = 0;
    (void)r64_with_blocks(nc, [&](auto k) { n = decltype(k)::value; return hipSuccess; });
    return n;
}

} // namespace

hipError_t forward_i8_rows64_init_device()
{
    for (int nc = 1; nc <= R64_MAX_BLOCKS; ++nc) {
        const hipError_t e = r64_with_blocks(nc, [](auto k) {
            constexpr int NC = decltype(k)::value;
            if constexpr (r64_lds(NC) > 64 * 1024)
                return hipFuncSetAttribute(reinterpret_cast<const void *>(fwd_i8_rows64_kernel<NC>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)r64_lds(NC));
            return hipSuccess;
        });
        if (e != hipSuccess)
            return e;
    }
    return hipSuccess;
}

// Which calls take this kernel, and not fwd_i8_doc_kernel (corpora that give every wavefront of those documents of its own) or the
// kernels for smaller ones.  us there -> here:
//  - up to four blocks of sixteen tokens the corpus read is the cost, and fwd_i8_doc_kernel reads whole lines: 64 tokens x 40 000 x 300
//    241 -> 268, x 4500 x 70 11.6 -> 13.7.  On fewer documents of 256 tokens and more the shares that need not end with a
//    document win, 64 tokens x 1000 x 300 14.2 -> 10.5, x 3000 x 1024 77 -> 72.
//  - many documents of under 128 tokens: the end of a document costs more than a shorter walk saves, 80 tokens x 4500 x 70 12.5 -> 15.2,
//    8 x 32 x 4500 x 70 22.6 -> 24.8, 1024 x 4500 x 96 66.4 -> 77.2.
//  - where the last 32 tokens take a whole tile (r64_rows): 1024 tokens x 4500 x 160 100 -> 102 with 6/5 of the rows, x 224 134 -> 129 with 8/7.
//  - the rest: 80 tokens x 40 000 x 300 282 -> 271, 256 x 9000 x 700 252 -> 226, 1024 x 9000 x 700 777 -> 719, x 40 000 x 1024 4607 -> 4412;
//    602 x 3000 x 1024 401 -> 223, 4 x 310 x 500 x 1000 134 -> 75, 2 x 300 x 2200 x 64 40 -> 19.
bool forward_i8_rows64_takes(int n_q, int l_q, const int32_t *offsets, int64_t b, int l_d, int num_cu)
{
    const int64_t bpq = (l_q + R64_COLS - 1) / R64_COLS, blocks = n_q * bpq;
    if (offsets || l_d < R64_ROWS || bpq > R64_MAX_BLOCKS)
        return false;
    const bool many = b >= (int64_t)num_cu * R64_WAVES * 2;
    if (blocks <= 4)
        return !many && l_d >= 256;
    return !many || (l_d >= 128 && r64_rows(blocks > R64_HALF_BLOCKS, l_d) * 7 <= r64_rows(false, l_d) * 8);
}

namespace {

// Queries per group: what the fullest CU has to do is least.  A workgroup (there is one per CU, whose registers it fills) copies its
// queries first.  Returns the rounds of workgroups, a wavefront's tiles in one and the blocks that are multiplied.
struct R64Plan {
    int64_t rounds, tiles, nc;
};
R64Plan r64_plan(FwdParams &p, int num_cu)
{
    p.bpq = (p.l_q + R64_COLS - 1) / R64_COLS;
    const int most = R64_MAX_BLOCKS / p.bpq;
    int64_t best = INT64_MAX;
    R64Plan plan = {};
    for (int qpg = 1; qpg <= most && qpg <= p.n_q; ++qpg) {
        const int64_t groups = (p.n_q + qpg - 1) / qpg;
        int64_t chunks = num_cu / groups;
        chunks = chunks < 1 ? 1 : chunks > p.b ? p.b : chunks;
        const int64_t docs = (p.b + chunks - 1) / chunks;
        chunks = (p.b + docs - 1) / docs;
        const int64_t rounds = (chunks * groups + num_cu - 1) / num_cu;
        const int64_t nc = r64_built(qpg * p.bpq);
        const int64_t tiles = (docs * r64_rows(nc > R64_HALF_BLOCKS, p.l_d) + R64_WAVES * R64_ROWS - 1) / (R64_WAVES * R64_ROWS);
        const int64_t time = rounds * (tiles * (nc + 4) + nc);
        if (time < best) {
            best = time;
            plan = {rounds, tiles, nc};
            p.qpg = qpg;
            p.n_groups = (int)groups;
            p.n_chunks = (int)chunks;
            p.unit_per_chunk = docs;
        }
    }
    return plan;
}

} // namespace

double forward_i8_rows64_time(I8Params P, int num_cu)
{
    const R64Plan r = r64_plan(P.f, num_cu);
    return -5.9 + 0.056 * (double)r.nc + 0.037 * P.f.n_q + (double)r.rounds * (10.1 + (double)r.tiles * (1.36 + 0.15 * (double)r.nc));
}

hipError_t forward_i8_rows64_launch(I8Params P, int num_cu, hipStream_t stream)
{
    FwdParams &p = P.f;
    (void)r64_plan(p, num_cu);
    const int grid = p.n_chunks * p.n_groups;
    return r64_with_blocks(p.qpg * p.bpq, [&](auto k) {
        constexpr int NC = decltype(k)::value;
        hipLaunchKernelGGL((fwd_i8_rows64_kernel<NC>), dim3(grid), dim3(R64_WAVES * 64), r64_lds(NC), stream, P);
        return hipGetLastError();
    });
}

} // namespace maxsim
