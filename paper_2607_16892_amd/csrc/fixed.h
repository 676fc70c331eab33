// Fixed-point helpers shared by the dense and exact translation units.
//
// Inside the library's limits (integers <= 2^15, binary32 coefficients in
// [2^-10, 2^7]) every candidate of phi (Appendix A, Step 4) is an integer
// multiple of 2^-33 below 2^56.  The helpers below form those integers, divide
// them exactly, and round 128-bit sums of them to double once.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace dro {

// v * 2^33 for a binary32 v in [2^-10, 2^7] (exact integer below 2^41).
__device__ __forceinline__ int64_t fix33(float v)
{
    const uint32_t bits = __float_as_uint(v);
    const int e = (int)((bits >> 23) & 0xffu);
    const int64_t mant = (int64_t)((bits & 0x7fffffu) | 0x800000u);
    const int sh = e - 117;  // e - 127 - 23 + 33
    return sh >= 0 ? (mant << sh) : (mant >> (-sh));
}

// floor(a / b) clamped to [lo, hi] for b > 0 and -2^16 < lo <= hi < 2^16: the
// quotient by the reciprocal instruction (about 2^-26 relative, so within one of
// the floor after the clamp) corrected once with the exact remainder.
__device__ __forceinline__ int floor_div_clamped(int64_t a, int64_t b, double rb, int lo, int hi)
{
    const double q = (double)a * rb;
    int t = (int)floor(fmin(fmax(q, (double)lo), (double)hi));
    const int64_t r = a - b * t;
    t += r < 0 ? -1 : (r >= b ? 1 : 0);
    return t < lo ? lo : (t > hi ? hi : t);
}

__device__ __forceinline__ int floor_div_clamped(int64_t a, int64_t b, int lo, int hi)
{
    return floor_div_clamped(a, b, __builtin_amdgcn_rcp((double)b), lo, hi);
}

// q = RN(S / N) from r = RN(1 / N): q0 = RN(S r) is within one unit of S / N, its
// residual S - q0 N is exact in an fma, and one more fma rounds the quotient
// correctly (Markstein; N is an integer below 2^27, so its significand is not all
// ones; S is finite and far from underflow).
__device__ __forceinline__ double div_by(double S, double N, double rN)
{
    const double q0 = __dmul_rn(S, rN);
    return __fma_rn(__fma_rn(-q0, N, S), rN, q0);
}

// a * b for a of 64 bits and b < 2^31, and for a, b < 2^43, exactly: two and
// four 32-bit multiply-adds where the general 128-bit product takes ten.
__device__ __forceinline__ __int128 mul_i64_u31(int64_t a, uint32_t b)
{
    const uint64_t l = (uint64_t)(uint32_t)a * b;
    const int64_t h = (int64_t)(int32_t)(a >> 32) * (int64_t)(int32_t)b;
    return (__int128)(((unsigned __int128)(__int128)h << 32) + l);
}

__device__ __forceinline__ __int128 mul_u43(uint64_t a, uint64_t b)
{
    const uint32_t al = (uint32_t)a, ah = (uint32_t)(a >> 32), bl = (uint32_t)b,
                   bh = (uint32_t)(b >> 32);
    const uint64_t mid = (uint64_t)ah * bl + (uint64_t)al * bh;  // below 2^44
    return (__int128)(((unsigned __int128)((uint64_t)(ah * bh)) << 64) +
                      ((unsigned __int128)mid << 32) + (uint64_t)al * bl);
}

// Correctly rounded double of the unsigned 128-bit value (hi, lo) times 2^-33.
// The top 64 bits below the leading zeros, with a bit for the rest in the last
// place, round to 53 bits as the whole value does.
__device__ __forceinline__ double fix128_to_double(uint64_t lo, uint64_t hi)
{
    const int s = hi ? __clzll((long long)hi) : 0;
    const unsigned __int128 v = (((unsigned __int128)hi << 64) | lo) << s;
    const uint64_t rest = (uint64_t)v;
    const uint64_t top = hi ? (uint64_t)(v >> 64) | (rest ? 1u : 0u) : lo;
    return ldexp((double)top, hi ? 64 - s - 33 : -33);
}

// Correctly rounded double of a signed 128-bit value times 2^-33.
__device__ __forceinline__ double sfix128_to_double(__int128 v)
{
    const bool neg = v < 0;
    const unsigned __int128 u = neg ? (unsigned __int128)(-v) : (unsigned __int128)v;
    const double d = fix128_to_double((uint64_t)u, (uint64_t)(u >> 64));
    return neg ? -d : d;
}

// The two lines of phi for one (class, grid point, multiplier), in units of
// 2^-33.  For 0 <= x, eta <= L the three candidates of Step 4 reduce to the
// larger of  B - A1 x  and  Cc - A2 (L - x)  with B = c_w eta, Cc = c_p (L - eta),
// A1 = min(g, c_w), A2 = min(g, c_p) (Q(eta, x) is itself the larger of
// c_w (eta - x) and c_p (x - eta), and for x, L - x >= 0 the smaller slope wins
// each pair).  Their difference is  y2 - y1 = De x - Nu  with De = A1 + A2 and
// Nu = B - Cc + A2 L, so the lines cross at x0 = Nu / De.
struct PairLinesFix {
    int64_t B, Cc, A1, A2, Nu, De;
};

__device__ __forceinline__ PairLinesFix pair_lines_fix(int64_t CP, int64_t CW, int64_t G,
                                                       int64_t eta, int64_t L)
{
    PairLinesFix q;
    q.B = CW * eta;
    q.Cc = CP * (L - eta);
    q.A1 = G < CW ? G : CW;
    q.A2 = G < CP ? G : CP;
    q.De = q.A1 + q.A2;
    q.Nu = q.B - q.Cc + q.A2 * L;
    return q;
}

}  // namespace dro
