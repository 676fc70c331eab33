// Wave-wide scans shared by the HIP translation units.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace dro {

// Wave-wide sums and scans with DPP moves: one VALU instruction a step, where a
// shuffle is a trip through the LDS unit (the 96 shuffles a wave of a prefix
// pass that used them took 9 of its 15 us).
template <int kCtrl, int kRows = 0xf> __device__ __forceinline__ uint32_t dpp0(uint32_t x)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, kCtrl, kRows, 0xf, true);
}
template <int kCtrl, int kRows = 0xf> __device__ __forceinline__ uint64_t dpp0(uint64_t x)
{
    return (uint64_t)dpp0<kCtrl, kRows>((uint32_t)x) |
           ((uint64_t)dpp0<kCtrl, kRows>((uint32_t)(x >> 32)) << 32);
}
// inclusive scan over each row of 16 lanes (lane 15 of a row holds its total)
template <class T> __device__ __forceinline__ T scan_row16(T x)
{
    x += dpp0<0x111>(x);  // row_shr:1
    x += dpp0<0x112>(x);
    x += dpp0<0x114>(x);
    x += dpp0<0x118>(x);
    return x;
}
// inclusive scan over each half of 32 lanes (lanes 31 and 63 hold the totals)
template <class T> __device__ __forceinline__ T scan_half32(T x)
{
    x = scan_row16(x);
    x += dpp0<0x142, 0xa>(x);  // row_bcast:15 into rows 1 and 3
    return x;
}
// inclusive scan over the wave (lane 63 holds the total)
template <class T> __device__ __forceinline__ T scan_wave(T x)
{
    x = scan_half32(x);
    x += dpp0<0x143, 0xc>(x);  // row_bcast:31 into rows 2 and 3
    return x;
}
__device__ __forceinline__ uint32_t lane_value(uint32_t x, int l)
{
    return (uint32_t)__builtin_amdgcn_readlane((int)x, l);
}
__device__ __forceinline__ uint64_t lane_value(uint64_t x, int l)
{
    return (uint64_t)lane_value((uint32_t)x, l) | ((uint64_t)lane_value((uint32_t)(x >> 32), l) << 32);
}

}  // namespace dro
