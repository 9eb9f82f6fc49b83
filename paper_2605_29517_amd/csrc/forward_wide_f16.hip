// The wide kernel for fp16 inputs.
#include "forward_wide_impl.h"

namespace maxsim {

hipError_t forward_wide_run_f16(const FwdParams &p, int row_bytes, int blocks, int blocks_per_pass, int rows, int grid, hipStream_t stream)
{
    return run_wide<MAXSIM_F16>(p, row_bytes, blocks, blocks_per_pass, rows, grid, stream);
}

hipError_t forward_wide_allow_f16() { return allow_wide<MAXSIM_F16>(); }

} // namespace maxsim
