// The wide kernel for fp32 inputs.
#include "forward_wide_impl.h"

namespace maxsim {

hipError_t forward_wide_run_f32(const FwdParams &p, int row_bytes, int blocks, int blocks_per_pass, int rows, int grid, hipStream_t stream)
{
    return run_wide<MAXSIM_F32>(p, row_bytes, blocks, blocks_per_pass, rows, grid, stream);
}

hipError_t forward_wide_allow_f32() { return allow_wide<MAXSIM_F32>(); }

} // namespace maxsim
