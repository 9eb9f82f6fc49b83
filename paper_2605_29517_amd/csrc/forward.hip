// Fused MaxSim forward for gfx950: choice of kernel and launch shape (the kernels themselves are
// in forward_impl.h, compiled once per element type in forward_{f16,bf16,f32}.hip).
#include "common.h"

namespace maxsim {

hipError_t forward_run_f16(const FwdParams &p, int nu, bool argmax, bool tile, int x, int n, hipStream_t s);
hipError_t forward_run_bf16(const FwdParams &p, int nu, bool argmax, bool tile, int x, int n, hipStream_t s);
hipError_t forward_run_f32(const FwdParams &p, int nu, bool argmax, bool tile, int x, int n, hipStream_t s);

hipError_t forward_splitd_launch(FwdParams p, int dtype, int row_bytes, int num_cu, hipStream_t stream);
hipError_t forward_wide_launch(FwdParams p, int dtype, int row_bytes, int num_cu, hipStream_t stream);
double forward_splitd_time(FwdParams p, int dtype, int row_bytes, int num_cu);
double forward_wide_time(FwdParams p, int num_cu);

constexpr int MAX_ROW_BYTES = 16384; // d = 8192 (16-bit) or 4096 (fp32)

// Rows of 128, 256 or 512 bytes have kernels that keep the queries in registers.  (Such kernels for rows of
// 1024 bytes were measured slower than the slab-streaming kernel at every shape: one column block per
// wavefront leaves one MFMA per LDS operand read.)
static bool register_stationary_width(int row_bytes)
{
    return row_bytes == 128 || row_bytes == 256 || row_bytes == 512;
}

// Embedding widths the float forward takes: rows that are a multiple of 64 bytes (d a multiple of 32 for
// 16-bit inputs, of 16 for fp32), from d = 32 up to MAX_ROW_BYTES.
bool forward_width_supported(int dtype, int d)
{
    const int64_t row_bytes = (int64_t)d * (dtype == MAXSIM_F32 ? 4 : 2);
    return d >= 32 && row_bytes % 64 == 0 && row_bytes <= MAX_ROW_BYTES;
}

// Forward with argmax on 16-bit inputs, fewer documents than CUs.  The tile kernel's workgroups of up to 32 column blocks then leave
// most of the chip idle (16 documents x 16 queries: 16 workgroups).  Smaller column groups make more of them; and the kernel whose
// wavefronts share a document's tiles (fwd_stream_split_kernel) makes most, with one or two blocks per workgroup, of one, two or
// four wavefronts.  The estimate: a start, then what a CU's (a SIMD's) workgroups (wavefronts) have to multiply, or the chain of
// one of them if that is longer.  us, n queries of 32 tokens x n documents, before -> after: n = 16 x 128 tokens 10.0 -> 4.1,
// x 1024 32.7 -> 8.4; 33 x 83-333 24.9 -> 9.7; 50 x 100 16.6 -> 9.4, x 1024 52 -> 33; 64 x 75-300 29 -> 17; 103 queries of 24 x
// 163-653 64 -> 54; from some hundred on the large groups are the best again (128 x 500 70, the others 70-85).
struct FewDocs {
    int shape, blocks; // of the tile kernel and blocks per group, or
    int waves;         // wavefronts per workgroup of the other (0: tile kernel), with `blocks` each
};
static FewDocs few_documents(const FwdParams &p, int num_cu, int shape, int groups)
{
    const double mean_len = (double)p.total_tokens / (double)p.b;
    const double tiles = p.offsets ? mean_len / TILE_ROWS + 0.5 : (double)((p.l_d + TILE_ROWS - 1) / TILE_ROWS);
    const double longest = p.offsets ? 1.5 * tiles : tiles; // (lengths are not known here)
    struct Shape {
        int code, blocks;
        double start, next, one, block; // us: of a workgroup, of one more on a CU; per tile of one by itself, per block where a CU is full
    };
    static const Shape shapes[] = {{81, 8, 4.5, 0.4, 0.62, 0.069}, {42, 8, 4.8, 0.44, 0.67, 0.069}, {43, 12, 5.9, 0.64, 0.81, 0.061}, {82, 16, 6.4, 0.4, 0.9, 0.067},
                                   {4, 16, 6.9, 1.2, 0.96, 0.054}, {83, 24, 7.6, 1.8, 1.3, 0.061}, {8, 32, 9.0, 2.8, 1.8, 0.05}};
    auto tile_time = [&](const Shape &s, int64_t n_groups) {
        const double on_cu = (double)((p.b * n_groups + num_cu - 1) / num_cu);
        const double work = on_cu * s.blocks * s.block;
        return s.start + (on_cu - 1) * s.next + (work > s.one ? work : s.one) * (tiles + (longest - tiles) / on_cu);
    };
    FewDocs best = {shape, 0, 0};
    double least = 1e30;
    for (const Shape &s : shapes)
        if (s.code == shape && groups > 0)
            least = 0.9 * tile_time(s, groups);
    for (const Shape &s : shapes)
        if (p.bpq <= s.blocks) {
            const double t = tile_time(s, (p.n_q + s.blocks / p.bpq - 1) / (s.blocks / p.bpq));
            if (t < least) {
                least = t;
                best = {s.code, s.blocks, 0};
            }
        }
    for (int blocks = p.bpq; blocks <= 2; blocks += p.bpq)
        for (int waves = 1; waves <= 4; waves *= 2) {
            const int64_t n = p.b * ((p.n_q + blocks / p.bpq - 1) / (blocks / p.bpq)) * waves;
            const double chain = std::ceil(longest / waves) * (blocks == 1 ? 0.57 : 0.72);
            const double work = (double)((n + 4 * num_cu - 1) / (4 * num_cu)) * tiles / waves * (blocks == 1 ? 0.43 : 0.66);
            const double t = 2.5 + (double)n / (4.0 * num_cu) * (blocks == 1 ? 0.8 : 1.8) + (work > chain ? work : chain);
            if (t < least) {
                least = t;
                best = {0, blocks, waves};
            }
        }
    return best;
}

// fp32 rows of 512 bytes, queries of one or two column blocks: fwd_f32_split_kernel's wavefronts per document and documents per
// workgroup (0 wavefronts: not that kernel but runs of documents).  `run`: documents of such a run, `runs`: how many there are.
//
// What counts is how many tiles the fullest SIMD has to multiply.  us in a graph (right behind a write of 512 MB), the kernels of
// runs or of two wavefronts per document that were there before -> now, 32 query tokens:
//  - fewer documents than SIMDs: four or two wavefronts on each (100 x 300 tokens 14.7 -> 11.4, 300 x 300 26.6 -> 21.0), from two
//    documents per CU on one (700 x 128 16.9 -> 14.7); with more than three per CU four documents to a workgroup (1000 x 128
//    19.4 -> 17.1 (22.4 -> 20.8; workgroups of one document 26.2), 1000 x 260 35.3 -> 33.5 (37.9 -> 36.0; 49.4); launched one after another by
//    the host workgroups of one are 2 % ahead, 15.1 against 15.5, and 17.0 before).
//  - beyond: one wavefront, but two on each of two documents where that makes the fullest SIMD's share smaller by a tenth, just beyond
//    4, 8, 12 or 16 per CU (1025 x 128 21.0 -> 21.1, one wavefront 23.0; 1400 x 260 55.7 -> 48.5, 51.0; 2300 x 260 72.7 -> 72.8,
//    77; not of three tiles, 1025 x 96 19.5 against 18.3; ragged from six on, 1500 x 200 50.4 against 51.5, x 128 35.2 against 33.4).
// Two blocks (64 tokens): a wavefront on each, with argmax where a SIMD's share is smaller by an eighth than that of a wavefront that holds
// both and reads a tile once, without (of whose runs a SIMD holds one at a time) always (no argmax, 52 tokens x 3098 x 34 68 in runs, 41
// here, 55 x 1575 x 120 69, 47; with: 4000 x 40 equal shares: 48.5 in runs, 56 here; 1536 x 64 three quarters: 27.1 -> 24.5; 2200 x 64 five eighths: 46.8
// -> 34.8).  Two documents to a workgroup with two or six per CU (500 x 300 47.9 -> 34.4, by themselves 49.5; 1536 x 90 35.9 -> 32.3,
// 40.3; but 600 x 100 26.8 against 24.3, 2500 x 20 25.5 against 23.6).
static void fp32_shape(FwdParams &p, int num_cu, int blocks, int64_t run, int64_t runs)
{
    const int64_t mean_len = (p.total_tokens + p.b - 1) / p.b, cus = num_cu, simds = 4 * cus;
    const int64_t tiles = (mean_len + TILE_ROWS - 1) / TILE_ROWS;
    auto rounds = [&](int64_t n) { return (n + simds - 1) / simds; };
    auto set = [&](int waves, int docs) {
        p.doc_waves = waves;
        p.docs_per_wg = docs;
    };
    set(0, 1);
    if (p.b > 64 * cus || (blocks > 1 && ((mean_len >= 4 * TILE_ROWS && p.b > 2 * cus) || (p.argmax && rounds(2 * p.b) * 8 >= rounds(runs) * run * 2 * 7))))
        return;
    if (p.b * blocks <= 2 * cus && tiles > 1)
        return set(tiles >= 4 ? 4 : 2, 1);
    if (blocks > 1) // (with four to a CU the workgroups of two happen to spread well)
        return set(1, (p.b > cus && p.b <= 2 * cus) || (p.b > 5 * cus && p.b <= 6 * cus) ? 2 : 1);
    if (p.b > 4 * cus && tiles >= (p.offsets ? 6 : 4) && rounds(2 * p.b) * 10 <= rounds(p.b) * 2 * 9)
        return set(2, 2);
    set(1, p.b > 3 * cus && p.b <= 4 * cus ? 4 : 1);
}

// Chooses kernel and launch shape from the problem size; `num_cu` is the device's CU count.
hipError_t forward_launch(FwdParams p, int dtype, int d, int num_cu, hipStream_t stream)
{
    if (!forward_width_supported(dtype, d))
        return hipErrorNotSupported;
    const int row_bytes = d * (dtype == MAXSIM_F32 ? 4 : 2);
    // any other width: both operands stream through LDS in slabs of the width; so do rows of 512 bytes from 8 column
    // blocks on (two blocks per wavefront in the register-stationary kernel: measured 3-11 % slower there).  Two
    // kernels: macro tiles of 256 document tokens x 256 query tokens and whole cache lines (forward_wide_impl.h), or of
    // 128 x 512 and half lines (forward_splitd.hip).  Up to 8 blocks the first, except for half lines and documents of
    // up to 128 tokens (8 blocks, d = 32: 121 against 113 us).  Beyond, 512 query tokens at once are ahead where the
    // first would multiply many padded blocks (three queries of 140 tokens x 4000 x 128, d = 512: 72 % of its time) or
    // documents of a few tiles of 256 leave much of one empty: the estimates of both decide.  The other way round, the
    // second's chunks fill the chip badly on some numbers of documents (16 queries x 1500 x 100 tokens, d = 512: 1.35
    // times the first's time).  The estimates are of 32x32 results; on 16x16 ones the first is 5-11 % faster, and where
    // they say 0.86 to 1 it takes 0.77 to 1.0 of the second's time (three queries of 100 tokens x 500 x 1000, d = 256 /
    // 1024: 114 -> 90, 488 -> 376 us; twelve of 32 x 3000 x 97 97 -> 91, 380 -> 346); of 1024 bytes and more than 128
    // tokens from 0.92 on (three of 140 x 1000 x 300, d = 512: 0.90, 215 in the second, 224 in the first).  With argmax the second has narrow rows and 65-128 tokens (20 000 x 100, 16 blocks, d =
    // 256 / 160, before 16x16 results without: 800 / 573 us in the first, 790 / 515 in the second).
    const int64_t all_blocks = (int64_t)p.n_q * ((p.l_q + BLOCK_COLS - 1) / BLOCK_COLS);
    if (!register_stationary_width(row_bytes) || (row_bytes == 512 && all_blocks >= 8)) {
        const int64_t mean_len = (p.total_tokens + p.b - 1) / p.b; // (uniform corpora: total_tokens = b * l_d)
        bool slabs;
        if (all_blocks <= 8)
            slabs = dtype != MAXSIM_F32 && all_blocks == 8 && row_bytes == 64 && mean_len <= 128;
        else if (dtype != MAXSIM_F32 && mean_len <= 128 && (row_bytes == 64 || (p.argmax && row_bytes <= 512 && mean_len > 64)))
            slabs = true;
        else
            slabs = forward_splitd_time(p, dtype, row_bytes, num_cu) <=
                    forward_wide_time(p, num_cu) * (dtype == MAXSIM_F32 || p.argmax || row_bytes == 64 ? 1.0 : mean_len > 128 && row_bytes >= 1024 ? 0.92 : 0.86);
        return slabs ? forward_splitd_launch(p, dtype, row_bytes, num_cu, stream) : forward_wide_launch(p, dtype, row_bytes, num_cu, stream);
    }
    const int nu = row_bytes / 32; // 16-byte chunk pairs per row
    const bool ragged = p.offsets != nullptr;
    const bool am = p.argmax != nullptr;
    p.bpq = (p.l_q + BLOCK_COLS - 1) / BLOCK_COLS;
    if (p.ld == 0)
        p.ld = p.b;
    const int64_t total_blocks = (int64_t)p.n_q * p.bpq;
    const int64_t units = ragged ? p.total_tokens : p.b; // what is split across chunks
    auto run = [&](bool tile, int x, int n) {
        switch (dtype) {
        case MAXSIM_F32: return forward_run_f32(p, nu, am, tile, x, n, stream);
        case MAXSIM_F16: return forward_run_f16(p, nu, am, tile, x, n, stream);
        default: return forward_run_bf16(p, nu, am, tile, x, n, stream);
        }
    };

    // Streaming kernel: every wavefront holds whole queries in as many column blocks as fit beside two
    // document tiles in registers (4 for rows of up to 256 bytes, 2 for 512 bytes), and up
    // to 4 wavefronts share a run of documents.  That covers up to 16 blocks of short queries.
    const int stream_max_blocks = nu <= 8 ? 4 : 2;
    int s_ncb = 0, s_groups = 0;
    if (total_blocks <= stream_max_blocks) {
        s_ncb = (int)total_blocks;
        s_groups = 1;
    } else if (p.bpq <= stream_max_blocks) {
        int qpw = stream_max_blocks / p.bpq; // whole queries per wavefront
        int groups = (p.n_q + qpw - 1) / qpw;
        if (groups <= 4) {
            s_ncb = qpw * p.bpq;
            s_groups = groups == 3 ? 4 : groups;
        }
    }

    // five to sixteen blocks of narrow rows: the tile kernel with two blocks per wavefront is faster than two to
    // four streaming wavefronts per run (measured on the ragged 100K corpus: 1.37 against 1.60 ms at 5 blocks,
    // 2.1-2.6 against 2.7 ms at 9-16; uniform corpora of 50K documents: 10-22 % at 5-8 blocks)
    if (nu <= 8 && total_blocks > 4)
        s_groups = 0;

    const int64_t tokens = ragged ? p.total_tokens : p.b * (int64_t)p.l_d;
    const bool fp32_512 = dtype == MAXSIM_F32 && nu == 16; // (fp32_shape; up to 64 documents per CU with one block, always)
    // Up to 64 documents per CU and two tiles per document on average: a workgroup of two wavefronts per document, four
    // workgroups per CU resident (512 to 2048 workgroups in all were slower).  At one query (fp16, 64-300 tokens) 1000 / 4000 / 16 000 documents take 12.6 / 32.1 /
    // 114.7 us instead of 14.3 / 35.2 / 117.3, four queries 142 instead of 147 us at 16 000; at 32 000 documents and four
    // queries the long runs win (275 against 280 us), with documents of 8-40 tokens already at 20 000 (25.7 against 30.0),
    // and with two blocks of 512-byte rows, which leave room for one wavefront per SIMD, everywhere (53 against 59 us).
    if (s_groups == 1 && p.b <= (int64_t)num_cu * 64 && tokens >= p.b * 2 * TILE_ROWS && (nu <= 8 || s_ncb == 1)) {
        p.n_chunks = 0; // no runs of documents: the kernel takes a document per workgroup
        p.n_groups = 1;
        p.qpg = p.n_q;
        p.n_pass = 1;
        p.doc_waves = 2;
        if (fp32_512)
            fp32_shape(p, num_cu, s_ncb, 1, p.b);
        const int64_t resident = (int64_t)num_cu * 4;
        return run(false, s_ncb, (int)(p.b < resident ? p.b : resident));
    }
    if (s_groups > 0) {
        // one work chunk per group of wavefronts; enough chunks to oversubscribe the chip a few times, but no
        // chunk smaller than about 2K tokens -- unless that leaves wavefront slots empty (a small corpus is a chain
        // of memory latencies per wavefront): then chunks go down to 128 tokens until every slot has one
        int64_t want = (int64_t)num_cu * 16 * 4 / s_groups;
        int64_t by_size = (tokens + 2047) / 2048;
        const int64_t slots = (int64_t)num_cu * 16 / s_groups;
        if (by_size < slots) {
            by_size = (tokens + 127) / 128;
            if (by_size > slots)
                by_size = slots;
        } else if (s_groups == 1) {
            // a large corpus, one wavefront per run: eight long runs per CU, all resident at once, stream 2-5 % faster
            // than more and shorter ones (0.679 against 0.694 ms on the ragged 100K corpus; a read probe shows the same,
            // 7.0 against 6.8 TB/s)
            want = (int64_t)num_cu * 8;
        }
        int64_t n_chunks = want < by_size ? want : by_size;
        if (n_chunks > p.b)
            n_chunks = p.b;
        if (n_chunks < 1)
            n_chunks = 1;
        p.unit_per_chunk = (units + n_chunks - 1) / n_chunks;
        if (p.unit_per_chunk < 1)
            p.unit_per_chunk = 1;
        if (!ragged)
            n_chunks = (units + p.unit_per_chunk - 1) / p.unit_per_chunk;
        p.n_chunks = (int)n_chunks;
        p.n_groups = s_groups;
        p.qpg = p.n_q;
        p.n_pass = 1;
        const int chunks_per_block = 4 / s_groups;
        int grid = (int)((n_chunks + chunks_per_block - 1) / chunks_per_block);
        if (fp32_512 && s_groups == 1)
            fp32_shape(p, num_cu, s_ncb, ragged ? (p.unit_per_chunk * p.b + p.total_tokens - 1) / p.total_tokens : p.unit_per_chunk, n_chunks);
        return run(false, s_ncb, grid);
    }

    // tile kernel: W wavefronts x NCB blocks per group (the query fragments of a wavefront fill 128 registers)
    const int ncb = nu <= 8 ? 4 : 32 / nu;
    int w = 8;
    if (total_blocks <= 1 * ncb)
        w = 1;
    else if (total_blocks <= 2 * ncb)
        w = 2;
    else if (total_blocks <= 4 * ncb)
        w = 4;
    int shape = w, wave_blocks = ncb;
    // Five to sixteen blocks of narrow rows.  What a wavefront spends per tile beside its MFMAs (iterator, copies,
    // barrier) does not depend on how many blocks it holds, so workgroups of two (up to 8 blocks) or four wavefronts
    // with four blocks each beat eight wavefronts with one or two blocks by 6-15 % -- as long as there are documents
    // enough for their many workgroups (at least four per workgroup; a small corpus is a chain of memory latencies
    // per workgroup, and the shapes below keep several tiles in flight for that).
    const int narrow_w = total_blocks <= 8 ? 2 : 4;
    // (fp32 rows carry four times the MFMAs per block: there two wavefronts are 3 % behind four with two blocks each)
    const bool narrow = ncb == 4 && total_blocks > 4 && total_blocks <= 16 && p.b >= 2 * ((int64_t)num_cu * 16 / narrow_w) &&
                        !(dtype == MAXSIM_F32 && narrow_w == 2);
    if (narrow) {
        w = narrow_w;
        shape = w;
    } else if (ncb == 4 && total_blocks <= 16) {
        if (total_blocks <= 8 && !(am && p.bpq > 4)) {
            // four wavefronts with two column blocks each (shape code 42), two workgroups per CU
            wave_blocks = 2;
            w = 4;
            shape = 42;
        } else if (total_blocks > 12 && !am && dtype != MAXSIM_F32 && nu == 8 && !ragged && p.b > num_cu && 2 * p.b <= 3 * (int64_t)num_cu &&
                   p.l_d >= 16 * TILE_ROWS) {
            // 13 to 16 blocks on more documents than CUs, at most three on two of them, of sixteen tiles and more: four
            // wavefronts with four blocks each let a CU that has two documents walk both at once (bf16, one query of 512
            // tokens x 300 documents of 512 / 1000 tokens 29.3 -> 28.2, 51.1 -> 46.3 us, of 400 tokens x 300 x 1000 49.3 ->
            // 46.1).  Shorter documents take 2-17 % longer that way (300 x 300 21.0 against 21.7), as do 13 and 14 blocks
            // from two documents per CU on (512 x 640 5 %), one per CU (150 x 1000 28.6 against 30.5) and ragged corpora
            // (6-40 %).
            w = 4;
            shape = 4;
        } else { // eight wavefronts with one or two column blocks each (shape code 81 / 82)
            wave_blocks = total_blocks <= 8 ? 1 : 2;
            w = 8;
            shape = 80 + wave_blocks;
        }
    }
    // a ragged corpus (or a uniform one whose documents are not a whole number of tiles) scored by many queries of
    // one block: 32-row windows over the packed rows (no padded tiles at the ends of documents)
    // (the windows also serve uniform corpora of whole tiles at 5-16 queries, where their narrow workgroups beat the
    // tile kernel's by 5-17 %)
    const bool rows_32bit = ragged || p.b * (int64_t)p.l_d < ((int64_t)1 << 31); // the window iterator counts packed rows in 32 bits
    const bool ragged_ends = rows_32bit && (ragged || p.l_d % TILE_ROWS != 0 || total_blocks <= 16);
    if (ragged_ends && !am && p.bpq == 1 && narrow) {
        // five to sixteen queries: the same narrow workgroups with 3 or 4 queries per wavefront (7-16 % over eight
        // wavefronts with two queries each, and over the per-document tiles, on the ragged 100K corpus)
        wave_blocks = (total_blocks + w - 1) / w <= 3 ? 3 : 4;
        shape = 900 + w * 10 + wave_blocks;
    }
    if (ragged_ends && !am && ncb == 4 && p.bpq == 1 && total_blocks > 16) {
        // as many workgroups per chunk as 32 queries each would need, then 3 or 4 queries per wavefront so that the
        // queries are spread evenly (48 queries: two workgroups of 24 rather than 32 + 16)
        const int64_t groups = (total_blocks + 31) / 32;
        const int64_t per_group = (total_blocks + groups - 1) / groups;
        wave_blocks = per_group <= 24 ? 3 : 4;
        shape = 90 + wave_blocks;
    }
    auto share = [&](int group_blocks) {
        if (p.bpq <= group_blocks) {
            p.qpg = group_blocks / p.bpq;
            if (p.qpg > p.n_q)
                p.qpg = p.n_q;
            p.n_groups = (p.n_q + p.qpg - 1) / p.qpg;
            // As many queries in each group where that lets the fullest do with three blocks per wavefront (below): four
            // queries of 280 tokens x 1500 x 300 145 -> 116 us.  Elsewhere the wavefronts that equal shares leave half full
            // cost more than a short last group (180 queries of 48 tokens x 180 x 350: eleven groups of 16 and one of 4
            // 158 us, twelve of 15 164).
            const int even = (p.n_q + p.n_groups - 1) / p.n_groups;
            if (p.qpg * p.bpq > 24 && even * p.bpq <= 24)
                p.qpg = even;
            p.n_pass = 1;
        } else {
            p.qpg = 1;
            p.n_groups = p.n_q;
            p.n_pass = (p.bpq + group_blocks - 1) / group_blocks;
        }
    };
    share(w * wave_blocks);
    // Three blocks per wavefront where they hold the group too: wavefronts w and w + 4 share a SIMD, and the one that has
    // most blocks sets the time (19 blocks in fours: 8, 4, 4 and 4, in threes 6, 6, 6 and 3: one query of 600 tokens x 3000 x
    // 300 138 -> 119 us; long queries of 33 to 48 blocks in two passes of 24: 1030 tokens 265 -> 210).
    if (ncb == 4 && shape < 900) {
        const int blocks = p.n_pass == 1 ? p.qpg * p.bpq : 0;
        const int64_t cus = num_cu, mean_len = (p.total_tokens + p.b - 1) / p.b;
        // Five and six blocks on less than sixteen documents per CU: two wavefronts with three blocks each, four such
        // workgroups per CU, instead of two of four wavefronts with two blocks (2000 x 100 / 3000 x 300 tokens, d = 128: 18.3
        // against 18.6 us, 44.4 against 49.6).  The more workgroups, the coarser the shares, which costs more than it gives
        // * on ragged corpora of less than seven documents per CU (1000 x 100-500 tokens 29.4 against 27.6 us; six with argmax,
        //   1500 x 100-500 1.06 times; four of up to 128 tokens: 1000 x 10-200 18.0 against 16.4, 1100 x 10-200 16.8 against 17.4)
        // and on uniform corpora of 256-byte rows
        // * where a workgroup has one document of two tiles (1000 x 60 10.1 against 9.3; not with argmax),
        // * where a few have to take a second one (1200 x 70 20 % slower, 1280 x 150 7 %, but not 1100 x 500; with argmax only
        //   those of three tiles, 9 %),
        // * where up to every other has a second one of 8 to 20 tiles (1500 x 500 46.0 against 41.1).
        bool two = shape == 2;
        if (shape == 42 && dtype != MAXSIM_F32) {
            if (ragged)
                two = p.b >= (mean_len <= 128 ? 4 : am ? 6 : 7) * cus;
            else if (p.b < 3 * cus || nu < 8 || p.b > 6 * cus)
                two = p.b >= 3 * cus;
            else if (p.b > 5 * cus)
                two = mean_len <= 7 * TILE_ROWS || mean_len > 20 * TILE_ROWS;
            else if (p.b > 4 * cus)
                two = mean_len > (am ? 3 : 8) * TILE_ROWS;
            else
                two = am || mean_len > 2 * TILE_ROWS;
        }
        // Nine to twelve blocks: four wavefronts with three blocks each, but for short documents of which a CU has up to
        // three: there eight wavefronts with two blocks each take 2-9 % less (700 x 64 tokens 10.4 against 11.3 us, 600 x 128
        // 0.95 times; 700 x 200 and 400 x 128 the other way, and 128-byte rows from three tiles on)
        const int64_t few_long = nu < 8 ? 64 : p.b > 2 * cus ? 160 : 96;
        const bool four = shape == 4 || (shape == 82 && (dtype == MAXSIM_F32 || ragged || p.b > 3 * cus || mean_len > few_long));
        const int threes = four ? 4 : shape == 8 ? 8 : two ? 2 : 0;
        if (threes && blocks > 0 && blocks <= threes * 3) {
            shape = threes * 10 + 3;
        } else if (shape == 8 && p.n_pass == 2 && p.bpq <= 48) {
            shape = 83;
            share(24);
        }
    }
    // Winners wanted of fewer documents than CUs (a training step on a small batch), which large column groups leave idle: up to three of
    // their workgroups per CU, six of queries of up to six blocks.  Beyond, the small differences of the estimate's long sums are not to
    // be trusted: 54 of 785 shapes (up to 300 queries x 256 documents, d = 64 and 128) were more than 3 % slower by it than in the large
    // groups, up to 1.48 times, with this line 11, up to 1.1 (278 queries of 496 x 256 x 28, d = 64, 351 us, 520 by the estimate; 160 of
    // 399 x 160 x 62 202, 263; but 57 of 58 x 195 x 27, 780 workgroups, 18.9, 13.4).
    if (am && dtype != MAXSIM_F32 && nu <= 8 && p.b <= num_cu && p.b * p.n_groups <= (p.bpq <= 6 ? 6 : 3) * (int64_t)num_cu) {
        const FewDocs few = few_documents(p, num_cu, shape, p.n_pass == 1 ? p.n_groups : 0);
        if (few.waves) { // a document and a column group per workgroup
            p.n_chunks = 0;
            p.qpg = few.blocks / p.bpq;
            p.n_groups = p.n_pass = 1;
            p.doc_waves = few.waves;
            return run(false, few.blocks, (int)p.b);
        }
        if (few.shape != shape) {
            shape = few.shape;
            share(few.blocks);
        }
    }
    return run(true, shape, num_cu); // (the chunks: launch_chunks)
}

} // namespace maxsim
