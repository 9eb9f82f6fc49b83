// What the int8 kernels of 128-byte rows share.
#pragma once
#include "common.h"

namespace maxsim {

constexpr int I8_ROW_BYTES = 128;

struct I8Params {
    const char *Q;      // [n_q, l_q, 128] int8
    const float *qs;    // [n_q, l_q]
    const char *D;      // [b, l_d, 128] int8
    const float *ds;    // [b, l_d]
    float *scores;      // [n_q, b]
    FwdParams f;        // sizes, optional offsets and the work split
};

// Cross-lane steps on the VALU: a shuffle goes through the LDS, and ten in a row per query at the end of every document
// (five steps of an fp64 butterfly) took longer than the document's MFMAs (4 / 8 queries x 100 000 / 50 000
// texts: 570 -> 533, 440 -> 409 us).
__device__ __forceinline__ float max_halves(float x) // both lane halves get the maximum of the two
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
template <int N> __device__ __forceinline__ double add_rotated(double v) // + the value N lanes on within the row of sixteen
{
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, 0x120 + N, 0xf, 0xf, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), 0x120 + N, 0xf, 0xf, true);
    return v + __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}
// Sum over lanes 0 .. 31 (lanes 32 .. 63 hold the same): a butterfly over distances 16, 8, 4, 2, 1.  Once the lanes repeat with
// period 2N, the lane N away by XOR and the one N away by rotation hold the same value.
__device__ __forceinline__ double sum32(double v)
{
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)b, (uint32_t)b, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)(b >> 32), (uint32_t)(b >> 32), false, false);
    v = __builtin_bit_cast(double, (uint64_t)hi[0] << 32 | lo[0]) + __builtin_bit_cast(double, (uint64_t)hi[1] << 32 | lo[1]);
    v = add_rotated<8>(v);
    v = add_rotated<4>(v);
    v = add_rotated<2>(v);
    return add_rotated<1>(v);
}

// int8_rows64.hip: the calls that forward_i8_rows64_takes
bool forward_i8_rows64_takes(int n_q, int l_q, const int32_t *offsets, int64_t b, int l_d, int num_cu);
hipError_t forward_i8_rows64_launch(I8Params P, int num_cu, hipStream_t stream);
double forward_i8_rows64_time(I8Params P, int num_cu); // an estimate, us, for up to 1024 tokens per query
hipError_t forward_i8_rows64_init_device();

} // namespace maxsim
