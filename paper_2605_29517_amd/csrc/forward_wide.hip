// Launch shape of the wide kernel (forward_wide_impl.h, compiled per element type in forward_wide_{f16,bf16,f32}.hip).
#include "forward_wide_impl.h"

namespace maxsim {

// More than 64 KB of dynamic LDS has to be allowed per kernel and device: every instantiation, for the current
// device (called once per device by the library's set-up).
hipError_t forward_wide_init_device()
{
    hipError_t e = forward_wide_allow_f16();
    if (e == hipSuccess)
        e = forward_wide_allow_bf16();
    return e == hipSuccess ? forward_wide_allow_f32() : e;
}

namespace {

// What a slab of 256 rows takes in each shape, in units of 10 ns, taken for all widths and types; only the ratios
// count. Documents that fill little of the lowest macro tile of a shape cost more per row (12 x 32 query tokens x 8000
// x 60, d = 160: 174 us by three groups of 4 blocks, 142 by two of 6).
double wide_weight(int blocks, int rows)
{
    const double w = blocks <= 1 ? 60 : blocks <= 2 ? 65 : blocks <= 4 ? 80 : blocks <= 6 ? 105 : 127;
    return rows <= 64 && blocks <= 4 ? 1.4 * w : rows <= 128 && blocks == 4 ? 1.1 * w : w;
}

struct WidePlan {
    ChunkPlan chunks;
    double time; // of a CU
    int n_groups, qpg, n_pass;
    int blocks; // column blocks of a workgroup, and of a pass where a query takes several
};

// p.bpq is set
WidePlan plan_wide(const FwdParams &p, int num_cu)
{
    const int rows = (int)((p.total_tokens + p.b - 1) / p.b); // the mean length (uniform corpora: total_tokens = b * l_d)
    // a CU's time: the documents of its workgroups, rounded up to tiles, and what 120 tokens take to begin with
    const double tiled = p.offsets ? rows + TILE_ROWS / 2 : (rows + TILE_ROWS - 1) / TILE_ROWS * TILE_ROWS;
    auto time = [&](const ChunkPlan &c, int groups, int n_pass, int blocks) {
        const int64_t on_cu = (c.n_chunks * groups + num_cu - 1) / num_cu;
        const int64_t tokens = p.offsets ? (c.per_chunk > rows ? c.per_chunk : rows) + rows / 2 : c.per_chunk * rows;
        const double padded = rows ? (double)tokens * tiled / rows : 0.0;
        return with_shape(blocks, rows, [&](auto s) { return (double)on_cu * (padded * n_pass + 120) * wide_weight(decltype(s)::BLOCKS, rows); });
    };
    if (p.bpq > WD_MAX_BLOCKS) { // several passes over a document per query
        int n_pass = (p.bpq + WD_MAX_BLOCKS - 1) / WD_MAX_BLOCKS;
        const int blocks = (p.bpq + n_pass - 1) / n_pass;
        n_pass = (p.bpq + blocks - 1) / blocks;
        const ChunkPlan c = plan_chunks(p, p.n_q, num_cu, 1, 1, false);
        return {c, time(c, p.n_q, n_pass, blocks), p.n_q, 1, n_pass, blocks};
    }
    // Whole queries per workgroup.  More of them read a document less often, fewer make more workgroups, which counts where
    // the documents do not fill the chip: the chunks' time decides, at what a slab takes in each shape.
    WidePlan best = {};
    double best_time = 0.0;
    for (int qpg = WD_MAX_BLOCKS / p.bpq < p.n_q ? WD_MAX_BLOCKS / p.bpq : p.n_q; qpg >= 1; --qpg) {
        const int groups = (p.n_q + qpg - 1) / qpg;
        if (qpg > 1 && (p.n_q + groups - 1) / groups < qpg)
            continue; // fewer queries in each of as many groups will do
        const ChunkPlan c = plan_chunks(p, groups, num_cu, 1, 1, false);
        const double t = (double)c.time * with_shape(qpg * p.bpq, rows, [&](auto s) { return wide_weight(decltype(s)::BLOCKS, rows); });
        if (best.n_groups == 0 || t < best_time) {
            best_time = t;
            best = {c, time(c, groups, 1, qpg * p.bpq), groups, qpg, 1, qpg * p.bpq};
        }
    }
    return best;
}

} // namespace

double forward_wide_time(FwdParams p, int num_cu)
{
    p.bpq = (p.l_q + BLOCK_COLS - 1) / BLOCK_COLS;
    return plan_wide(p, num_cu).time;
}

// Any row width that is a multiple of 64 bytes.  `num_cu` is the device's CU count.
hipError_t forward_wide_launch(FwdParams p, int dtype, int row_bytes, int num_cu, hipStream_t stream)
{
    if (row_bytes < 64 || row_bytes % 64 != 0)
        return hipErrorNotSupported;
    p.bpq = (p.l_q + BLOCK_COLS - 1) / BLOCK_COLS;
    if (p.ld == 0)
        p.ld = p.b;
    const WidePlan plan = plan_wide(p, num_cu); // (one workgroup per CU at a time)
    p.n_groups = plan.n_groups;
    p.qpg = plan.qpg;
    p.n_pass = plan.n_pass;
    p.unit_per_chunk = plan.chunks.per_chunk;
    p.n_chunks = (int)plan.chunks.n_chunks;
    if (plan.chunks.n_chunks * p.n_groups >= (int64_t(1) << 31))
        return hipErrorInvalidValue;
    const int grid = (int)(plan.chunks.n_chunks * p.n_groups);
    const int blocks = plan.blocks, blocks_per_pass = plan.n_pass > 1 ? plan.blocks : 0;
    const int rows = (int)((p.total_tokens + p.b - 1) / p.b); // the mean length (uniform corpora: total_tokens = b * l_d)
    switch (dtype) {
    case MAXSIM_F32: return forward_wide_run_f32(p, row_bytes, blocks, blocks_per_pass, rows, grid, stream);
    case MAXSIM_F16: return forward_wide_run_f16(p, row_bytes, blocks, blocks_per_pass, rows, grid, stream);
    default: return forward_wide_run_bf16(p, row_bytes, blocks, blocks_per_pass, rows, grid, stream);
    }
}

} // namespace maxsim
