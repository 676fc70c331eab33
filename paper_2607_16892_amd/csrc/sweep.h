// The Gauss-Seidel reservation sweep under the memory-capacity constraint
// (Sec. 3.4), shared by the block step and by LP2 of Alg. 1.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "wave.h"

namespace dro {

constexpr int kSweepLds = 6144;  // doubles of LDS a sweep may use

// The bound of class c given the reservations res(c') of the others, by one wave:
// a lane per configuration.
template <class F, class Res>
__device__ __forceinline__ double sweep_bound(int c, int C, int G, const F *conc, const F *cap,
                                              double onek, Res &&res)
{
    double bound = INFINITY;
    for (int g = threadIdx.x & 63; g < G; g += 64) {
        const double u = (double)conc[(long long)c * G + g];
        if (!(u > 0.0)) continue;
        double sum = 0.0;
#pragma unroll 4
        for (int c2 = 0; c2 < C; ++c2) {
            const double v = (double)conc[(long long)c2 * G + g] * res(c2);
            sum = c2 != c ? sum + v : sum;
        }
        const double b = ((double)cap[g] - onek * sum) / (onek * u);
        bound = b < bound ? b : bound;
    }
    return wave_min(bound);
}

// For c = 0 .. C-1 in order, with the other classes at their current grid points:
//   bound = min over g with conc[c,g] > 0 of
//           (cap[g] - onek sum_{c' != c} conc[c',g] eta[k[c']]) / (onek conc[c,g])
// (fp64, no contraction, the classes in ascending order), then k[c] = the lowest
// argmin of W[c, .] over the grid points eta[k] <= bound + slack (none: k = 0 and
// not feasible).  best[c, k] is the lowest argmin of W[c, 0 .. k] (launch_best_upto),
// eta ascends, so the argmin is one entry of it.  k_in[C] (clamped into [0, K)) is
// the state entering the sweep, k_out[C] (another array) the one leaving it;
// done(c, k, feasible) is called by one lane per class.
// For one wave: the classes depend on one another, so it is a chain (the operands
// in LDS where they fit, a lane per configuration for the bound, a 64-way search
// for the largest admissible grid point), and a block's barriers and reductions
// would only lengthen it: 8 classes, 6 configurations, K = 1024
// take 15 us and the table 5, 64 before (256 threads, every reservation looked at).
// buf: kSweepLds doubles of LDS.
template <class F, class Done>
__device__ void sweep_wave(const int32_t *best, const int32_t *eta, int C, int K, int G,
                           const F *conc, const F *cap, double onek, double slack,
                           const int32_t *k_in, int32_t *k_out, double *buf, Done &&done)
{
    const int lane = threadIdx.x & 63;
    const long long own = (long long)C * G + C + G;
    const bool lds = own <= kSweepLds / 2, lds_eta = lds && K <= kSweepLds;  // (ints: half a double)
    double *e = buf, *cc = e + C, *cp = cc + C * G;
    int32_t *le = reinterpret_cast<int32_t *>(buf + kSweepLds / 2);
    if (lds_eta)
        for (int k = lane; k < K; k += 64) le[k] = eta[k];
    for (int c = lane; c < C; c += 64) {
        const int k = min(max(k_in[c], 0), K - 1);
        k_out[c] = k;
        if (lds) e[c] = (double)eta[k];
    }
    if (lds) {
        for (int i = lane; i < C * G; i += 64) cc[i] = (double)conc[i];
        for (int g = lane; g < G; g += 64) cp[g] = (double)cap[g];
    }
    wave_sync();
    auto eta_at = [&](int k) { return (double)(lds_eta ? le[k] : eta[k]); };
    for (int c = 0; c < C; ++c) {
        const double top = slack + (lds ? sweep_bound(c, C, G, cc, cp, onek, [&](int c2) { return e[c2]; })
                                        : sweep_bound(c, C, G, conc, cap, onek,
                                                      [&](int c2) { return (double)eta[k_out[c2]]; }));
        // the number of admissible grid points, 64 pieces of [lo, hi) at a time
        int lo = 0, hi = K;
        while (hi > lo) {
            const int step = (hi - lo + 63) >> 6;
            const int k = min(lo + (lane + 1) * step, hi) - 1;  // the last of the lane's piece
            const int n = __popcll(__ballot(eta_at(k) <= top));  // whole pieces admissible
            const int l2 = min(lo + n * step, hi);
            hi = step == 1 ? l2 : min(l2 + step - 1, hi);  // the next piece's last is not admissible
            lo = l2;
        }
        const bool feas = lo > 0;
        const int k = feas ? min(max(best[(long long)c * K + lo - 1], 0), K - 1) : 0;
        if (lane == 0) {
            k_out[c] = k;
            if (lds) e[c] = eta_at(k);
            done(c, k, feas);
        }
        // the next bound reads what lane 0 wrote (a wave's LDS accesses keep their order
        // by themselves)
        if (lds) {
            asm volatile("" ::: "memory");
            __builtin_amdgcn_wave_barrier();
        } else {
            wave_sync();
        }
    }
}

}  // namespace dro
