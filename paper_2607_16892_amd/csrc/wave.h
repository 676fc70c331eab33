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

// x of lane kLane of each group of four lanes (all of them active)
template <int kLane> __device__ __forceinline__ int quad_lane(int x)
{
    return __builtin_amdgcn_update_dpp(0, x, kLane * 0x55, 0xf, 0xf, true);
}

// x of the lane a DPP control names, or the lane's own x where there is none
template <int kCtrl, int kRows = 0xf> __device__ __forceinline__ int dpp_or_own(int x)
{
    return __builtin_amdgcn_update_dpp(x, x, kCtrl, kRows, 0xf, false);
}
template <int kCtrl, int kRows = 0xf> __device__ __forceinline__ double dpp_or_own(double x)
{
    return __hiloint2double(dpp_or_own<kCtrl, kRows>(__double2hiint(x)),
                            dpp_or_own<kCtrl, kRows>(__double2loint(x)));
}
__device__ __forceinline__ double lane_value(double x, int l)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), l),
                            __builtin_amdgcn_readlane(__double2loint(x), l));
}

// Makes what a wave's lanes wrote visible to its other lanes.
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// Minimum over a wave; every lane gets it.  Every lane is active.
__device__ __forceinline__ double wave_min(double x)
{
    auto take = [&](double y) { x = y < x ? y : x; };
    take(dpp_or_own<0x111>(x));
    take(dpp_or_own<0x112>(x));
    take(dpp_or_own<0x114>(x));
    take(dpp_or_own<0x118>(x));
    take(dpp_or_own<0x142, 0xa>(x));
    take(dpp_or_own<0x143, 0xc>(x));
    return lane_value(x, 63);
}

// Lexicographic minimum of (key, idx) over a wave (smallest key, then the
// smallest idx), carrying aux along; every lane gets it.  Every lane is active.
struct KeyIdx {
    double key;
    int idx, aux;
};

__device__ __forceinline__ uint32_t wave_min(uint32_t x)
{
    auto take = [&](int y) { x = (uint32_t)y < x ? (uint32_t)y : x; };
    take(dpp_or_own<0x111>((int)x));  // row_shr:1, 2, 4, 8: lane 15 of a row has its minimum
    take(dpp_or_own<0x112>((int)x));
    take(dpp_or_own<0x114>((int)x));
    take(dpp_or_own<0x118>((int)x));
    take(dpp_or_own<0x142, 0xa>((int)x));  // row_bcast:15 into rows 1 and 3
    take(dpp_or_own<0x143, 0xc>((int)x));  // row_bcast:31 into rows 2 and 3: lane 63 has it all
    return lane_value(x, 63);
}

// The key's bits as an unsigned integer in the key's order (-0 as 0), then three
// 32-bit minima: its high half, the low half among the lanes that hold it, the idx
// among those (idx >= 0).  One fp64 minimum that carries idx and aux along is some
// ninety dependent instructions.
__device__ __forceinline__ KeyIdx wave_min_key(double k, int i, int a)
{
    const long long b = __double_as_longlong(k + 0.0);
    const unsigned long long u = (unsigned long long)b ^ ((unsigned long long)(b >> 63) | (1ull << 63));
    const uint32_t hi = (uint32_t)(u >> 32), lo = (uint32_t)u;
    const uint32_t h = wave_min(hi), l = wave_min(hi == h ? lo : 0xffffffffu);
    const bool least = hi == h && lo == l;
    const uint32_t first = wave_min(least ? (uint32_t)i : 0xffffffffu);
    const int owner = __builtin_ctzll(__ballot(least && (uint32_t)i == first));
    return KeyIdx{lane_value(k, owner), (int)first, __builtin_amdgcn_readlane(a, owner)};
}

}  // namespace dro
