// Launch plan of the dense evaluation: which of its two kernels runs, with which tile
// shape, over how many slices and blocks.  Host arithmetic on sizes only (no HIP).
#pragma once

#include <stdint.h>

#include <algorithm>
#include <cmath>
#include <utility>
#include <vector>

namespace dro {

// Sizes of the classes' segments, ascending, and how many classes have each.
using SizeCounts = std::vector<std::pair<long long, long long>>;

// The sizes that each(add) reports, add(n, classes) for every segment in use
// (1 <= n <= 2^26): each distinct size while there are at most 64, else bins of an
// eighth of an octave, each by its largest size.  The plan looks the list through some
// hundred times: with one entry per distinct size, 30,000 unequal classes took the host
// 3 ms a call on new segments.
template <class Each> SizeCounts size_counts(Each &&each)
{
    constexpr size_t kMaxSizes = 64;
    SizeCounts v;
    bool exact = true;
    each([&](long long n, long long classes) {
        if (!exact) return;
        const auto it = std::lower_bound(v.begin(), v.end(), n,
                                         [](const auto &z, long long x) { return z.first < x; });
        if (it != v.end() && it->first == n) it->second += classes;
        else if (v.size() < kMaxSizes) v.insert(it, {n, classes});
        else exact = false;
    });
    if (exact) return v;
    v.assign(8 * 25, {0, 0});
    each([&](long long n, long long classes) {
        // n in [2^e, 2^(e + 1)): bins 8 (e - 2) .. 8 (e - 2) + 7; below 8 one a size
        const int e = 31 - __builtin_clz((unsigned)n | 8u);
        auto &z = v[n < 8 ? n : 8 * (e - 2) + ((n >> (e - 3)) & 7)];
        z.first = std::max(z.first, n);
        z.second += classes;
    });
    v.erase(std::remove_if(v.begin(), v.end(), [](const auto &z) { return !z.second; }), v.end());
    return v;
}

// The persistent kernel's tile: a block of kThreads lanes, kTM (grid point, multiplier)
// pairs per lane.
constexpr int kThreads = 256;
constexpr int kTM = 32;

// tile shapes of the one-block-per-slice kernel: pairs per lane, lanes per group
constexpr int kSliceShapes = 5;
constexpr int kSliceTM[kSliceShapes] = {32, 32, 32, 16, 8};
constexpr int kSliceGL[kSliceShapes] = {256, 128, 64, 64, 64};

struct DensePlan {
    int tiles;         // tiles of the K * M pairs of a class, in table order
    int P;             // sample slices per tile (direct: 0 = they differ, slices_of each class's
                       // size and len)
    int direct;        // 1: one block per slice, no claims (smaller problems)
    int shape;         // direct: the tile shape
    int len;           // direct: samples per slice, at most
    bool stored;       // direct: every class has one slice, so the sums are stored, not added
    long long blocks;  // direct: a block per slice; else the persistent grid,
                       // min(resident blocks, C * tiles * P)
};
// slices of n samples (n <= 2^26)
constexpr int slices_of(long long n, int len)
{
    return n <= len ? 1 : (int)(((uint32_t)n + (uint32_t)len - 1u) / (uint32_t)len);
}

// Large problems run the persistent grid that claims slices (dense.hip):
// tiles of kTM pairs per lane, each tile's samples split into P slices.  P
// is the largest of three needs: slices of at most kMaxSliceN samples, so that
// the last ones are short; about kSlicesPerBlock slices per resident block, so
// that the issue priorities keep the blocks of a compute unit in step and the
// blocks still finding work near the end keep every unit full (slices down to
// kBalanceSliceN samples); and one slice for every resident block (slices down
// to kMinSliceN samples).  Measured on 16 x 1e6 samples (K = 2048, M = 256,
// 1024 resident blocks): P = 16 (62,500-sample slices) ran 0.3 % faster than
// the launch of 20,480 short blocks it replaced, P = 31 0.2 % slower and
// P = 8 2.5 % slower.
// Others run one block per slice instead (dense_slices_kernel): a run's set-up
// (its thresholds, claims, the search for work) is then not small beside its
// work.  plan_slices picks its tile shape and slice length, plan_dense between
// the two.
constexpr long long kSlicesPerBlock = 16;
constexpr long long kMaxSliceN = 65536;
constexpr long long kBalanceSliceN = 512;
constexpr long long kMinSliceN = 64;

// Tile shape and slice length of dense_slices_kernel by a model of its time in
// cycles of a compute unit: w passes of the chip's resident blocks (one of 1,024
// threads per compute unit), each as long as a slice's v_sad_u16 (4 waves a SIMD,
// 4 cycles each; kLoop more per step of sixteen samples for its loads, claims and
// branch) and a block's set-up, which grows with its pairs (the first samples,
// thresholds, LDS sums, flush: 31 us for 8,192 pairs from slices of 12,500 and
// 14,286 samples, 5 us for 512).  For every shape and w the shortest slices whose
// blocks fit w passes; a sum split over slices also pays the zero fill of the
// table.  Where the sizes are bins, their largest sizes stand for all; plan_dense
// counts the slices of the true ones.
constexpr int kSliceThreads = 1024;
constexpr long long kMaxDirectBlocks = (1LL << 32) / kSliceThreads - 1;  // below 2^32 work-items
// A block of unequal classes, some of several slices, finds its class by walking them 64
// at a time up to kWalkClasses, else in a table of their first slices that one more
// launch writes: walk against launch and search, 2,048 pairs, 128 classes 28.9 and
// 33.5 us, 512 classes 67.2 and 66.8, 1,000 classes 142 and 116 (512 pairs, 5,000
// classes: 693 and 119).
constexpr int kWalkClasses = 512;
constexpr int kMaxDirectSlice = 65536;
constexpr double kLoop = 8.0, kBlockCycles = 12000.0, kPairCycles = 7.0, kZeroCycles = 6000.0;

inline double plan_slices(const SizeCounts &sizes, int K, int M, int num_cu, DensePlan *best)
{
    const long long KM = (long long)K * M;
    double total = 0.0, best_cost = -1.0;
    for (const auto &z : sizes) total += (double)z.first * z.second;
    for (int sh = 0; sh < kSliceShapes; ++sh) {
        const int TM = kSliceTM[sh], GL = kSliceGL[sh], NG = kSliceThreads / GL;
        const long long tiles = (KM + (long long)TM * GL - 1) / ((long long)TM * GL);
        const double per_sample = (8 * TM + kLoop) / NG;
        const double per_block = kBlockCycles + kPairCycles * TM * GL;
        double least = 0.0;  // blocks of the longest slices
        for (const auto &z : sizes)
            least += (double)tiles * slices_of(z.first, kMaxDirectSlice) * z.second;
        if (least > kMaxDirectBlocks) continue;
        const int w0 = std::max(1, (int)std::ceil(least / num_cu));
        for (int i = 0; i < 12; ++i) {
            const int w = i < 8 ? w0 + i : w0 + 7 + 4 * (i - 7);
            const double room = (double)w * num_cu;
            // (w passes of the longest slices hold all the samples, whatever the lengths)
            const double bound = total * tiles / num_cu * per_sample + w * per_block;
            if (best_cost >= 0.0 && bound > best_cost * (1.0 + 1e-9)) break;
            double len = std::max(16.0, std::ceil(total * tiles / room));
            double blocks = 0.0, longest = 0.0;
            bool one = true, fits = false;
            for (int it = 0; it < 6 && !fits && len <= kMaxDirectSlice; ++it) {
                blocks = longest = 0.0;
                one = true;
                for (const auto &z : sizes) {
                    const int n = slices_of(z.first, (int)len);
                    blocks += (double)n * z.second;
                    longest = std::max(longest, (double)z.first / n);
                    one = one && n == 1;
                }
                blocks *= tiles;
                fits = blocks <= room;
                if (!fits) len = std::ceil(len * std::max(1.02, blocks / room));
            }
            if (!fits || blocks > kMaxDirectBlocks) continue;
            const double cost = w * (longest * per_sample + per_block) + (one ? 0.0 : kZeroCycles);
            if (best_cost < 0.0 || cost < best_cost) {
                best_cost = cost;
                *best = DensePlan{};
                best->tiles = (int)tiles;
                best->direct = 1;
                best->shape = sh;
                best->len = (int)len;
                best->stored = one;
            }
        }
    }
    return best_cost;  // below 0: too many blocks
}

// each: as for size_counts
template <class Each>
DensePlan plan_dense(Each &&each, int C, int K, int M, int num_cu, int bpc)
{
    const SizeCounts sizes = size_counts(each);
    const long long max_n = sizes.back().first;
    DensePlan pl{};
    pl.tiles = (int)(((long long)K * M + kThreads * kTM - 1) / (kThreads * kTM));
    const long long T = (long long)C * pl.tiles;
    const long long slots = (long long)num_cu * std::max(bpc, 1);
    // The claimed slices run at 1.2 % above the v_sad_u16 rate of their padded
    // tiles (16 x 1e6 samples: 108.6 ms), and lose 100 us where the last slices
    // end and some 17 us per tile and compute unit in the runs' set-up (16 x 2e5 samples, K = 1000, M = 200:
    // 8.72 ms, one block per slice 9.03; 8 x 4e5, K = 1024, M = 128: 5.75 and 5.53).
    double total = 0.0;
    for (const auto &z : sizes) total += (double)z.first * z.second;
    const double claimed = total * pl.tiles * (kThreads * kTM) / (128.0 * num_cu) * 1.012 + 2.5e5 +
                           4e4 * (double)T / num_cu;
    DensePlan direct;
    const double cost = plan_slices(sizes, K, M, num_cu, &direct);
    if (cost >= 0.0 && cost <= claimed) {
        long long slices = 0, min_n = max_n;
        each([&](long long n, long long classes) {
            slices += slices_of(n, direct.len) * classes;
            min_n = std::min(min_n, n);
        });
        // (the sizes of one bin can differ in it too)
        direct.P = slices_of(min_n, direct.len) == slices_of(max_n, direct.len)
                       ? slices_of(max_n, direct.len) : 0;
        direct.blocks = slices * direct.tiles;
        return direct;
    }
    const long long by_size = (max_n + kMaxSliceN - 1) / kMaxSliceN;
    const long long by_balance = std::min((kSlicesPerBlock * slots + T - 1) / T, max_n / kBalanceSliceN);
    const long long by_fill = std::min((slots + T - 1) / T, max_n / kMinSliceN);
    long long P = std::max({1LL, by_size, by_balance, by_fill});
    P = std::min(P, std::max(1LL, 0x7fffffffLL / T));  // T P claims fit the 32-bit counters
    pl.P = (int)P;
    pl.direct = 0;
    pl.blocks = std::min(slots, T * P);
    return pl;
}

}  // namespace dro
