// The tile kernels with argmax for rows of 256 bytes (16-bit, d = 128): by themselves because build.py aligns their loops to
// 64 bytes.  Their issue slots are nearly full (the packed fold takes 1.5 VALU operations per cell), and where in a line of
// the instruction cache the stretches between the MFMAs begin then counts: the same 2224 instructions of eight wavefronts
// with four blocks each, 0 .. 60 bytes further on, take 425 to 437 us on 256 x 32 x 256 x 1024 tokens (fp16) and 50.3 to 52.5
// on 64 x 32 x 64 x 1024; with three blocks each 74.9 to 79.4 on 24 queries x 300 x 1000.  Aligned loops give the lower figure
// for every shape.  Other kernels gain nothing and some lose: two blocks of 512-byte rows 61.4 -> 63.8.
#include "forward_impl.h"

namespace maxsim {
hipError_t forward_tile_argmax_f16(const FwdParams &p, int w, int num_cu, hipStream_t s)
{
    return dispatch_tile<fmt(MAXSIM_F16, 8), true>(p, w, num_cu, s);
}
hipError_t forward_tile_argmax_bf16(const FwdParams &p, int w, int num_cu, hipStream_t s)
{
    return dispatch_tile<fmt(MAXSIM_BF16, 8), true>(p, w, num_cu, s);
}
} // namespace maxsim
