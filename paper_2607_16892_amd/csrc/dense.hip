// Dense evaluation of the per-sample worst-case cost and its sums
// (paper, Appendix A, Step 4 closed form and Step 5 sums), plus the minimum
// over the multiplier grid (the Kantorovich dual of Appendix A, Step 3, with
// gamma on a grid).
//
// Work: one (class, grid point, multiplier, sample) term per evaluation,
// C * K * M * N_c terms in all.  This is max-plus arithmetic, not a dense
// contraction, so it runs on the integer VALU; there is no MFMA.
//
// Form of the term.  In units of 2^-33 (fixed.h) the three candidates of
// Step 4 are the larger of two lines, y1 = B - A1 x and y2 = Cc - A2 (L - x),
// whose difference is y2 - y1 = De x - Nu.  With c_w <= c_p
//     phi = y1 + relu(De x - Nu),
// and with t = floor(Nu / De), r = Nu - De t in [0, De), for every integer x
//     relu(De x - Nu) = De relu(x - t) - r [x > t]
// (x > Nu / De exactly when x > t).  With c_w > c_p the mirror image holds
// around t = ceil(Nu / De): phi = y2 + De relu(t - x) - (De t - Nu) [x < t].
// Summed over a class's N samples,
//     S = sum y1 + De sum relu(x - t) - r #{x > t}
// and  sum relu(x - t) = (sum x - N t + sum |x - t|) / 2.
// The per-sample part of every term is |x - t|: that is what this kernel
// evaluates, once per (c, k, m, n).  The line sums need only N and sum x, and
// #{x > t} is one count per (c, k, m), read from the class's value counts in
// the epilogue; every piece is an integer, so S is exact and is rounded to
// double once.
//
// Instruction.  v_sad_u16 adds |a.lo - b.lo| + |a.hi - b.hi| (unsigned 16-bit
// halves) to a 32-bit accumulator: with two samples x + 1 packed in a and the
// threshold t + 1 in both halves of b, it evaluates two terms of one
// (k, m) pair in one single-rate VALU instruction.  Samples are staged in LDS
// as 16-bit x + 1 (x <= 2^15, t clamped to [-1, L] or [0, L + 1], so both
// fit), read back as wave-wide broadcasts of sixteen samples, and every lane
// keeps the thresholds and 32-bit sums of kTM pairs.  Every
// kHalfSadSteps instructions the bit 2^31 of each sum moves into a 16-bit
// carry in LDS, so a sum spans any number of samples without a flush.
//
// Reduction and schedule.  Each tile's samples are split into P slices, and
// a persistent grid (every block resident) claims them with atomic counters:
// a block first drains its own tiles, then the tiles of its XCD with the most
// unclaimed slices, then any tile.  It keeps a tile's sums in registers over
// all the consecutive slices it claims of that tile and adds them to the
// [C][K][M] table with one 64-bit atomic per pair when it moves to another
// tile (a run).  Integer addition is associative, so the table does not
// depend on which block took which slice.  The wave arbiter of a compute unit
// favours its oldest waves, which would let one of its blocks finish its tiles
// far ahead of the others (and then take many short runs elsewhere); so at
// every claim a block sets its waves' issue priority from its lead over the
// average block, read from a counter of all claims.  Within a run, the claim
// of the next slice is issued when a slice starts and read when it ends.
#include <algorithm>

#include "dro_internal.h"
#include "fixed.h"
#include "wave.h"

namespace dro {

__device__ __forceinline__ int seg_of(const int32_t *seg, int c) { return seg ? seg[c] : c; }

// Integer threshold of a pair, clamped to the range a 16-bit sample code can
// meet: [-1, L] when c_w <= c_p (relu(x - t)), [0, L + 1] otherwise
// (relu(t - x)).  Beyond it the sums are linear in the samples, and the epilogue's
// formula holds with the clamped t as it stands.
__device__ __forceinline__ int pair_kink(const PairLinesFix &q, bool upper, int L)
{
    return upper ? floor_div_clamped(q.Nu, q.De, -1, L) : -floor_div_clamped(-q.Nu, q.De, -L - 1, 0);
}

// What the thresholds of one class need.
struct ClassLines {
    int64_t CP, CW;
    int L;
    bool upper;
};

__device__ __forceinline__ ClassLines class_lines(const DenseArgs &a, int c)
{
    const float cpf = a.c_p[c], cwf = a.c_w[c];
    return ClassLines{fix33(cpf), fix33(cwf), a.L[c], cwf <= cpf};
}

// Threshold code t + 1 of pair p of a class (pairs in table order, p = k M + m;
// pairs past the table take its last one, their sums are never stored).
__device__ __forceinline__ uint16_t pair_code(const DenseArgs &a, const ClassLines &cl, uint32_t p)
{
    const uint32_t M = (uint32_t)a.M;
    p = min(p, (uint32_t)a.K * M - 1u);
    const uint32_t k = p / M, m = p - k * M;
    const PairLinesFix q = pair_lines_fix(cl.CP, cl.CW, fix33(a.lam[m]), a.eta[k], cl.L);
    return (uint16_t)(pair_kink(q, cl.upper, cl.L) + 1);
}

// First sample (relative to the segment start) of slice p of P: even offsets,
// so every slice but the last holds whole pairs of samples.
__device__ __forceinline__ long long slice_start(long long N, int p, int P)
{
    return p >= P ? N : 2 * ((N * p) / (2LL * P));
}

__global__ __launch_bounds__(kThreads) void dense_kernel(DenseArgs a)
{
    // two staging buffers of kT samples (kT / kThreads prefetch registers per
    // lane); at the start of a run the same memory passes the tile's
    // thresholds from a rolled loop into registers
    constexpr int kT = 4096;
    __shared__ __attribute__((aligned(16))) uint16_t xs[kTileN];
    __shared__ uint16_t carry[kTM * kThreads];
    __shared__ int s_claim, s_prio;
    __shared__ int s_best[kThreads / 64], s_left[kThreads / 64];
    static_assert(kTileN >= kThreads * kTM, "the threshold table shares the sample buffers");
    static_assert(kT % kThreads == 0 && kT % 16 == 0 && 2 * kT <= kTileN, "staging shape");

    const DensePlan pl = a.plan;
    const int nb = (int)gridDim.x;
    const int T = a.C * pl.tiles;  // tile tau: class tau / tiles, tile tau % tiles of it
    // Workgroups are dispatched to the XCDs in turn (block i to XCD i mod 8), so
    // XCD x is given one contiguous run of logical blocks, whose own tiles are
    // one contiguous range [xt0, xt1): the blocks on an XCD read the samples of
    // a few classes, which stay in its L2.
    const int xcd = (int)(blockIdx.x % kXcds);
    const int qx = nb / kXcds, rx = nb % kXcds;
    const int xb0 = xcd * qx + min(xcd, rx);
    const int xb1 = xb0 + qx + (xcd < rx ? 1 : 0);
    const int b = xb0 + (int)(blockIdx.x / kXcds);
    auto own = [&](int lb) { return (int)(((long long)lb * T) / nb); };
    const int xt0 = own(xb0), xt1 = own(xb1);
    int next_own = own(b);
    const int own_end = own(b + 1);

    const int t = threadIdx.x;

    uint32_t thr[kTM];  // (t + 1) in both 16-bit halves
    uint32_t acc[kTM];
#pragma unroll
    for (int j = 0; j < kTM; ++j) {
        acc[j] = 0u;
        carry[j * kThreads + t] = 0;
    }
    int c = 0, p0 = 0;  // the run's class and this lane's first pair
    // Sample codes 0 pad the end of a slice to whole groups of sixteen; each
    // adds t + 1 to a sum, which the flush takes off again.
    int pads = 0, steps = 0;

    auto normalize = [&]() {
        // (the address is hidden from the optimiser, which would otherwise keep
        // the 32 carry addresses live across the sample loop)
        int te = t;
        asm volatile("" : "+v"(te));
        uint16_t *cp = carry + te;
#pragma unroll
        for (int j = 0; j < kTM; ++j) {
            cp[j * kThreads] += (uint16_t)(acc[j] >> 31);
            acc[j] &= 0x7fffffffu;
        }
        steps = 0;
    };
    auto flush = [&]() {
        int pe = p0, ce = c, te = t;
        asm volatile("" : "+v"(pe), "+v"(ce), "+v"(te));
        const uint32_t KM = (uint32_t)a.K * (uint32_t)a.M;  // below 2^31
        unsigned long long *row = a.R + (long long)ce * KM;
        uint16_t *cp = carry + te;
#pragma unroll
        for (int j = 0; j < kTM; ++j) {
            const uint32_t p = (uint32_t)pe + j * kThreads;
            uint32_t a32 = acc[j];
            asm volatile("" : "+v"(a32));  // keeps the sums 32-bit through the sample loop
            const unsigned long long tot = ((unsigned long long)cp[j * kThreads] << 31) + a32 -
                                           (unsigned long long)pads * (thr[j] & 0xffffu);
            if (p < KM) atomicAdd(row + p, tot);
        }
#pragma unroll
        for (int j = 0; j < kTM; ++j) {
            acc[j] = 0u;
            cp[j * kThreads] = 0;
        }
        pads = 0;
        steps = 0;
    };
    // the thresholds of tile tau: pair j * kThreads + t of its kThreads * kTM
    auto start_run = [&](int tau) {
        c = tau / pl.tiles;
        p0 = (int)((uint32_t)(tau % pl.tiles) * (kThreads * kTM) + t);
        const ClassLines cl = class_lines(a, c);
        // (four at a time: their multiplier loads overlap, and the 64-bit
        // arithmetic of four pairs fits beside the live sums)
#pragma unroll 4
        for (int j = 0; j < kTM; ++j)
            xs[j * kThreads + t] = pair_code(a, cl, (uint32_t)p0 + j * kThreads);
        __syncthreads();
#pragma unroll
        for (int j = 0; j < kTM; ++j) thr[j] = (uint32_t)xs[j * kThreads + t] * 0x10001u;
        __syncthreads();
    };
    // The samples xi[lo, hi) in buffers of kT: the next buffer's samples are
    // loaded into registers while this one is evaluated, then stored; one
    // barrier per buffer.
    constexpr int kPer = kT / kThreads;
    int32_t pf[kPer];
    auto run_slice = [&](long long lo, long long hi) {
        auto fetch = [&](long long base) {
            // a block-uniform base and clamped 32-bit lane offsets: one
            // address register per load and no branches
            const int32_t *tp = a.xi + base;
            const int len = (int)min((long long)kT, hi - base);
#pragma unroll
            for (int r = 0; r < kPer; ++r) {
                const int i = t + r * kThreads;
                const int x = tp[min(i, len - 1)];
                pf[r] = i < len ? x : -1;
            }
        };
        auto put = [&](int buf) {
            uint16_t *dst = xs + buf * kT;
#pragma unroll
            for (int r = 0; r < kPer; ++r) dst[t + r * kThreads] = (uint16_t)(pf[r] + 1);
        };
        const int nbuf = (int)((hi - lo + kT - 1) / kT);
        if (nbuf > 0) {
            fetch(lo);
            put(0);
        }
        __syncthreads();
        for (int i = 0; i < nbuf; ++i) {
            const long long base = lo + (long long)i * kT;
            const int len = (int)min((long long)kT, hi - base);
            const int len16 = (len + 15) & ~15;
            if (steps + len16 / 2 > kHalfSadSteps) normalize();
            if (i + 1 < nbuf) fetch(base + kT);
            pads += len16 - len;
            steps += len16 / 2;
            // sixteen samples (two broadcast LDS reads) per step
            const uint4 *x4 = reinterpret_cast<const uint4 *>(xs + (i & 1) * kT);
            const int n8 = len16 / 16;
            for (int w = 0; w < n8; ++w) {
                const uint4 v = x4[2 * w], u = x4[2 * w + 1];
#pragma unroll
                for (int j = 0; j < kTM; ++j) acc[j] = __builtin_amdgcn_sad_u16(v.x, thr[j], acc[j]);
#pragma unroll
                for (int j = 0; j < kTM; ++j) acc[j] = __builtin_amdgcn_sad_u16(v.y, thr[j], acc[j]);
#pragma unroll
                for (int j = 0; j < kTM; ++j) acc[j] = __builtin_amdgcn_sad_u16(v.z, thr[j], acc[j]);
#pragma unroll
                for (int j = 0; j < kTM; ++j) acc[j] = __builtin_amdgcn_sad_u16(v.w, thr[j], acc[j]);
#pragma unroll
                for (int j = 0; j < kTM; ++j) acc[j] = __builtin_amdgcn_sad_u16(u.x, thr[j], acc[j]);
#pragma unroll
                for (int j = 0; j < kTM; ++j) acc[j] = __builtin_amdgcn_sad_u16(u.y, thr[j], acc[j]);
#pragma unroll
                for (int j = 0; j < kTM; ++j) acc[j] = __builtin_amdgcn_sad_u16(u.z, thr[j], acc[j]);
#pragma unroll
                for (int j = 0; j < kTM; ++j) acc[j] = __builtin_amdgcn_sad_u16(u.w, thr[j], acc[j]);
            }
            if (i + 1 < nbuf) put((i + 1) & 1);
            __syncthreads();
        }
    };
    // Issue priority from this block's lead over the average block: done is
    // the number of slices it has claimed, g the number all blocks had claimed
    // before its latest claim; 0 for a slice or more ahead, 3 for more than a
    // slice behind.
    int done = 0;
    auto prio_of = [&](long long g) {
        const long long lead = (long long)done * nb - g;  // in 1/nb slices
        return lead >= nb ? 0 : (lead >= 0 ? 1 : (lead >= -nb ? 2 : 3));
    };
    auto set_prio = [&](int level) {
        switch (level) {
        case 0: __builtin_amdgcn_s_setprio(0); break;
        case 1: __builtin_amdgcn_s_setprio(1); break;
        case 2: __builtin_amdgcn_s_setprio(2); break;
        default: __builtin_amdgcn_s_setprio(3); break;
        }
    };
    // Claims the next slice of tile tau for the whole block and waits for it
    // (block-uniform result: P or more means the tile is drained).
    auto claim = [&](int tau) {
        __syncthreads();
        if (t == 0) {
            s_claim = (int)atomicAdd(a.claim + tau, 1u);
            s_prio = prio_of((long long)atomicAdd(a.claim + T, 1u));
        }
        __syncthreads();
        return s_claim;
    };
    // The tile of [q0, q1) with the most unclaimed slices (-1 if none): every
    // thread reads some counters, then a block-wide maximum (ties to the
    // higher index).  Counters only grow, and the coherent reads see every
    // completed claim, so a block that finds a tile drained never picks it
    // again: the search ends.
    auto most_left = [&](int q0, int q1) {
        int best = -1, left = 0;
        for (int q = q0 + t; q < q1; q += kThreads) {
            const int r = pl.P - (int)__hip_atomic_load(a.claim + q, __ATOMIC_RELAXED,
                                                        __HIP_MEMORY_SCOPE_AGENT);
            if (r > left) {
                left = r;
                best = q;
            }
        }
        for (int d = 32; d >= 1; d >>= 1) {
            const int ob = __shfl_xor(best, d, 64), ol = __shfl_xor(left, d, 64);
            if (ol > left || (ol == left && ob > best)) {
                left = ol;
                best = ob;
            }
        }
        __syncthreads();
        if ((t & 63) == 0) {
            s_best[t >> 6] = best;
            s_left[t >> 6] = left;
        }
        __syncthreads();
        if (t == 0) {
            int bb = s_best[0], bl = s_left[0];
            for (int w = 1; w < kThreads / 64; ++w)
                if (s_left[w] > bl || (s_left[w] == bl && s_best[w] > bb)) {
                    bl = s_left[w];
                    bb = s_best[w];
                }
            s_claim = bl > 0 ? bb : -1;
        }
        __syncthreads();
        return s_claim;
    };

    // Runs: pick a tile and claim a slice of it; take its thresholds; evaluate
    // its slices while claims on it succeed; add the sums to the table.
    bool any_xcd = xt0 == 0 && xt1 == T;  // search every tile (this XCD's are drained)
    for (;;) {
        int tau = -1, p = pl.P;
        while (p >= pl.P) {
            if (next_own < own_end) {
                tau = next_own++;
            } else {
                tau = any_xcd ? most_left(0, T) : most_left(xt0, xt1);
                if (tau < 0) {
                    if (any_xcd) break;
                    any_xcd = true;
                    continue;
                }
            }
            p = claim(tau);
        }
        if (p >= pl.P) break;  // every slice has been claimed
        ++done;
        set_prio(s_prio);
        start_run(tau);
        const int sg = seg_of(a.seg, c);
        const long long n_beg = a.offsets[sg], N = a.offsets[sg + 1] - n_beg;
        for (;;) {
            run_slice(n_beg + slice_start(N, p, pl.P), n_beg + slice_start(N, p + 1, pl.P));
            p = claim(tau);
            if (p >= pl.P) break;
            ++done;
            set_prio(s_prio);
        }
        flush();
    }
}

// Smaller problems: one block per (class, tile, slice of its samples).  Bound
// by the same v_sad_u16, but a block's fixed cost (thresholds, first samples, the
// sums' way to the table) is no longer small beside its samples, so it is spread
// over 1,024 threads: NG = 1024 / GL groups of GL lanes hold the same tile of
// TM * GL pairs.  Each threshold is then computed once per block (not once per 256
// lanes) and the groups' sums meet in LDS, so the table gets one 64-bit atomic
// per pair and block, a plain store where one block holds all of a class's
// samples.  The waves that hold the same 64 TM pairs claim steps of sixteen
// staged samples from a counter in LDS: with fixed shares the oldest wave of a
// SIMD runs ahead and the last one ends alone, waiting for its reads (8 x 4e5
// samples: 5.68 ms with fixed shares and 4,096 samples a buffer, 5.60 claimed,
// 5.50 with 16,384 a buffer, whose barriers are fewer).
// The tile shape (TM, GL) fits the grid: its pairs are taken in table order, so
// only the last tile of a class is padded.  Slices have one length over all
// classes, so segments of unequal size keep every block equally long.  A slice
// holds at most 65,536 samples: with its padding its sums stay below 2^32, so
// there are no carries.
// dense part of dro_cost_eval before and after, in blocks of 256 threads with
// 32 multipliers a lane before: 4 x 1e5 samples, K = 512, M = 128: 429 -> 375 us
// (344 at this launch's clock of 2.33 GHz; 4.5 % more VALU instructions than
// sads, 99.6 % issue, the rest before the first and after the last wave); six
// segments from 1.2e5 to 7.9e3 samples, K = 333, M = 50: 289 -> 102 us; 1,000
// samples, K = 64, M = 32: 21 -> 5.3 us.
template <int TM, int GL>
__global__ __launch_bounds__(kSliceThreads) void dense_slices_kernel(DenseArgs a)
{
    constexpr int NG = kSliceThreads / GL, kPairs = TM * GL;
    constexpr int kT = 16384, kPer = kT / kSliceThreads;  // samples per staging buffer, per thread
    __shared__ __attribute__((aligned(16))) uint16_t xs[2][kT];
    __shared__ uint16_t code[kPairs];
    __shared__ uint32_t sums[kPairs];
    constexpr int kParts = GL / 64, kChunk = 64 / TM;
    __shared__ uint32_t next[2][kParts];  // next unclaimed step of a buffer, by part of the tile
    const DensePlan pl = a.plan;
    const int t = threadIdx.x, lane = t & 63, gl = t % GL;
    const int part = __builtin_amdgcn_readfirstlane(gl / 64);  // the wave's part of the tile
    // the logical block order gives each XCD one contiguous run of blocks
    const int nb = (int)gridDim.x, xcd = (int)(blockIdx.x % kXcds);
    const int b = xcd * (nb / kXcds) + min(xcd, nb % kXcds) + (int)(blockIdx.x / kXcds);
    // block b: class c, then slice p of its P, then tile
    const int slice = b / pl.tiles, tile = b % pl.tiles;
    int c, p = slice, P = pl.P;
    if (P) {
        c = slice / P;
        p = slice % P;
    } else if (a.C <= kWalkClasses) {  // one or a few steps of 64 classes
        for (c = 0;; c += 64) {
            int n = 0;
            if (c + lane < a.C) {
                const int sg = seg_of(a.seg, c + lane);
                n = slices_of(a.offsets[sg + 1] - a.offsets[sg], pl.len);
            }
            const int incl = (int)scan_wave((uint32_t)n);
            const unsigned long long in = __ballot(p < incl);
            if (in || c + 64 >= a.C) {
                const int l = in ? __ffsll(in) - 1 : 0;
                c += l;
                p -= __builtin_amdgcn_readlane(incl - n, l);
                P = __builtin_amdgcn_readlane(n, l);
                break;
            }
            p -= __builtin_amdgcn_readlane(incl, 63);
        }
    } else {  // the last class that starts at or before the slice, 64 pieces at a time
        const uint32_t *starts = a.claim;
        int hi = a.C;
        for (c = 0; hi - c > 1;) {
            const int step = (hi - c + 63) >> 6, q = c + lane * step;
            const int n = __popcll(__ballot(q < hi && (int)starts[min(q, hi - 1)] <= slice));
            c += (n - 1) * step;  // (starts[c] <= slice, so n >= 1)
            hi = min(c + step, hi);
        }
        p -= (int)starts[c];
        P = (int)starts[c + 1] - (int)starts[c];
    }
    const int sg = seg_of(a.seg, c);
    // slice p of P nearly equal ones (N <= 2^26)
    const long long n_beg = a.offsets[sg];
    const uint32_t N = (uint32_t)(a.offsets[sg + 1] - n_beg);
    const uint32_t each = N / (uint32_t)P, more = N % (uint32_t)P;
    const int len = (int)(each + ((uint32_t)p < more ? 1u : 0u));
    const int32_t *tp = a.xi + n_beg + (uint32_t)p * each + min((uint32_t)p, more);

    int32_t pf[kPer];
    auto fetch = [&](int base) {
#pragma unroll
        for (int r = 0; r < kPer; ++r)
            if (base + r * kSliceThreads < len)
                pf[r] = tp[min(base + r * kSliceThreads + t, len - 1)];
    };
    auto put = [&](int base) {  // codes 0 past the slice's end
#pragma unroll
        for (int r = 0; r < kPer; ++r) {
            const int i = t + r * kSliceThreads;
            if (base + r * kSliceThreads < len)
                xs[(base / kT) & 1][i] = (uint16_t)(base + i < len ? pf[r] + 1 : 0);
        }
    };
    if (len > 0) fetch(0);
    const ClassLines cl = class_lines(a, c);
#pragma unroll  // the multiplier and grid loads of all a thread's pairs in flight
    for (int r = 0; r < (kPairs + kSliceThreads - 1) / kSliceThreads; ++r) {
        const int q = t + r * kSliceThreads;
        if (q < kPairs) {
            code[q] = pair_code(a, cl, (uint32_t)tile * kPairs + q);
            sums[q] = 0u;
        }
    }
    if (len > 0) put(0);
    if (t < kParts) next[0][t] = 0u;
    __syncthreads();
    uint32_t thr[TM], acc[TM];
#pragma unroll
    for (int j = 0; j < TM; ++j) {
        thr[j] = (uint32_t)code[j * GL + gl] * 0x10001u;
        acc[j] = 0u;
    }
    const int nbuf = (len + kT - 1) / kT;
    for (int i = 0; i < nbuf; ++i) {
        const int n16 = (min(kT, len - i * kT) + 15) / 16;
        if (i + 1 < nbuf) fetch((i + 1) * kT);
        const uint4 *x4 = reinterpret_cast<const uint4 *>(xs[i & 1]);
        // the next step's samples are read while this step's are evaluated, in
        // two register sets
        uint4 v0, z0, v1, z1;
        auto read = [&](int w, uint4 &v, uint4 &z) {
            const int q = min(w, n16 - 1);
            v = x4[2 * q];
            z = x4[2 * q + 1];
        };
        auto eval = [&](const uint4 &v, const uint4 &z) {
#pragma unroll
            for (int j = 0; j < TM; ++j) acc[j] = __builtin_amdgcn_sad_u16(v.x, thr[j], acc[j]);
#pragma unroll
            for (int j = 0; j < TM; ++j) acc[j] = __builtin_amdgcn_sad_u16(v.y, thr[j], acc[j]);
#pragma unroll
            for (int j = 0; j < TM; ++j) acc[j] = __builtin_amdgcn_sad_u16(v.z, thr[j], acc[j]);
#pragma unroll
            for (int j = 0; j < TM; ++j) acc[j] = __builtin_amdgcn_sad_u16(v.w, thr[j], acc[j]);
#pragma unroll
            for (int j = 0; j < TM; ++j) acc[j] = __builtin_amdgcn_sad_u16(z.x, thr[j], acc[j]);
#pragma unroll
            for (int j = 0; j < TM; ++j) acc[j] = __builtin_amdgcn_sad_u16(z.y, thr[j], acc[j]);
#pragma unroll
            for (int j = 0; j < TM; ++j) acc[j] = __builtin_amdgcn_sad_u16(z.z, thr[j], acc[j]);
#pragma unroll
            for (int j = 0; j < TM; ++j) acc[j] = __builtin_amdgcn_sad_u16(z.w, thr[j], acc[j]);
        };
        const int ch = max(1, min(kChunk, n16 / (8 * NG)));
        auto claim = [&]() {  // (a register, read when the next chunk starts)
            int w = 0;
            if (lane == 0) w = (int)atomicAdd(&next[i & 1][part], (uint32_t)ch);
            return w;
        };
        if (t < kParts) next[(i + 1) & 1][t] = 0u;
        int w = __builtin_amdgcn_readfirstlane(claim());
        while (w < n16) {
            const int after = claim();
            const int w1 = min(w + ch, n16);
            read(w, v0, z0);
            for (; w < w1; w += 2) {
                read(w + 1, v1, z1);
                eval(v0, z0);
                if (w + 1 >= w1) break;
                read(w + 2, v0, z0);
                eval(v1, z1);
            }
            w = __builtin_amdgcn_readfirstlane(after);
        }
        if (i + 1 < nbuf) put((i + 1) * kT);
        __syncthreads();
    }
#pragma unroll
    for (int j = 0; j < TM; ++j) atomicAdd(&sums[j * GL + gl], acc[j]);
    __syncthreads();
    // codes 0 pad the last buffer to sixteens; each added t + 1
    const uint32_t pads = (uint32_t)((16 - (len & 15)) & 15);
    const int KM = a.K * a.M, q0 = tile * kPairs;  // below 2^31
    unsigned long long *row = a.R + (long long)c * KM + q0;
    const int nq = min(kPairs, KM - q0);
    for (int q = t; q < nq; q += kSliceThreads) {
        const unsigned long long tot = sums[q] - pads * (uint32_t)code[q];
        if (P == 1) row[q] = tot;
        else atomicAdd(row + q, tot);
    }
}

// starts[c] = the first slice of class c (slices of at most len samples, class after
// class), starts[C] = all of them: one block, a run of classes per thread.  Blocks of
// dense_slices_kernel find their class in it where walking the classes would be long.
constexpr int kStartThreads = 1024;

__global__ __launch_bounds__(kStartThreads) void slice_starts_kernel(const int64_t *offsets,
                                                                     const int32_t *seg, int C,
                                                                     int len, uint32_t *starts)
{
    __shared__ uint32_t wsum[kStartThreads / 64];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int per = (C + kStartThreads - 1) / kStartThreads;
    const int c0 = min((long long)t * per, (long long)C), c1 = min(c0 + per, C);
    auto slices = [&](int c) {
        const int sg = seg_of(seg, c);
        return (uint32_t)slices_of(offsets[sg + 1] - offsets[sg], len);
    };
    uint32_t n = 0;
#pragma unroll 4
    for (int c = c0; c < c1; ++c) n += slices(c);
    const uint32_t incl = scan_wave(n);
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    uint32_t at = incl - n;
    for (int w = 0; w < wave; ++w) at += wsum[w];
#pragma unroll 4
    for (int c = c0; c < c1; ++c) {
        starts[c] = at;
        at += slices(c);
    }
    if (t == kStartThreads - 1) starts[C] = at;
}

int dense_blocks_per_cu()
{
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, dense_kernel, kThreads, 0) != hipSuccess || n < 1)
        n = 1;
    return n;
}

// the tile shapes of dense_slices_kernel, by DensePlan::shape
using SlicesKernel = void (*)(DenseArgs);
static const SlicesKernel kSlicesKernels[kSliceShapes] = {
    dense_slices_kernel<32, 256>, dense_slices_kernel<32, 128>, dense_slices_kernel<32, 64>,
    dense_slices_kernel<16, 64>, dense_slices_kernel<8, 64>};

hipError_t launch_dense(const DenseArgs &a, hipStream_t st)
{
    if (a.plan.direct) {
        if (!a.plan.P && a.C > kWalkClasses)
            hipLaunchKernelGGL(slice_starts_kernel, dim3(1), dim3(kStartThreads), 0, st, a.offsets,
                               a.seg, a.C, a.plan.len, a.claim);
        hipLaunchKernelGGL(kSlicesKernels[a.plan.shape], dim3((unsigned)a.plan.blocks),
                           dim3(kSliceThreads), 0, st, a);
    } else
        hipLaunchKernelGGL(dense_kernel, dim3((unsigned)a.plan.blocks), dim3(kThreads), 0, st, a);
    return hipGetLastError();
}

__global__ void zero_u64_u32_kernel(unsigned long long *p, long long n, uint32_t *q, long long nq)
{
    const long long m = n > nq ? n : nq;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < m;
         i += (long long)gridDim.x * blockDim.x) {
        if (i < n) p[i] = 0ull;
        if (i < nq) q[i] = 0u;
    }
}

hipError_t launch_zero_u64_u32(unsigned long long *p, long long n, uint32_t *q, long long nq,
                               hipStream_t st)
{
    const long long m = std::max(n, nq);
    if (m <= 0) return hipSuccess;
    hipLaunchKernelGGL(zero_u64_u32_kernel, dim3((unsigned)std::min((m + 255) / 256, kMaxGridBlocks)),
                       dim3(256), 0, st, p, n, q, nq);
    return hipGetLastError();
}

// #{x <= v} of a segment from its prefix entries (v in [0, 2^15]).
__device__ __forceinline__ long long count_le(const PrefixEntry *pre, long long v, long long N)
{
    if (v < 0) return 0;
    if (v >= kHistBins - 1) return N;
    return (long long)pre[v].cnt;
}

// ---- rows: the exact S and the minimum over the multipliers, in one pass ----
//
// A block takes RB consecutive rows (c, k) of the table, their pairs a chunk of
// kRowPairs at a time (whole rows while M fits): every thread forms q = RN(S / N)
// of its pairs in table order (coalesced, however small M is) and stages them in
// LDS with the multipliers; then the block's 256 lanes split over the (radius,
// row) tasks, lp lanes each (a power of two, at most a wave), lane j of a task
// taking the multipliers j, j + lp, ...  Each lane keeps the smallest J of its
// multipliers (the lowest m among equal values, as it visits them in ascending
// order), then log2(lp) shuffle steps take the task's smallest, ties to the
// lowest m: the same J bits and the same lowest m as a scan over m.
//
// kFinish: S comes from the dense kernels' sums of |x - t| (in the table, u64,
// overwritten in place by S): exactly, in 128-bit integers in units of 2^-33 from
// the segment's N, sample sum and one value count, rounded to double once.
// Otherwise the table already holds S.
// Bound by the integer arithmetic (kFinish) or by reading S; one pass instead of
// the epilogue and the minimum apart saves reading S back: 68 us for the two
// launches' 101 + 21 on 16 x 2048 rows of 256 multipliers, 7.0 for 4.6 + 4.7 on
// 6 x 333 rows of 50 and three radii.  (1,024 pairs a block: 70 us, and 28 for 23
// without kFinish; a resident grid that loads its next rows early: 77 us.)
constexpr int kRowThreads = 256;
constexpr int kRowPairs = 2048;  // pairs staged per block at a time
constexpr int kRowMax = 64;      // rows per block

struct RowInfo {
    int64_t B, Cc, CP, CW, sx;
    double N, rN;  // and RN(1 / N)
    const PrefixEntry *pre;
    int L;
    bool upper;
};

// S of one pair from its sum of |x - t|.  With c_w <= c_p, t = floor(Nu / De)
// and Rt = sum relu(x - t): S = N B - A1 sum x + De Rt - (Nu - De t) #{x > t};
// the mirror image otherwise.
__device__ __forceinline__ double finish_pair(const RowInfo &w, float lam, int64_t sad)
{
    const int64_t G = fix33(lam), N = (int64_t)w.N;
    const int64_t A1 = G < w.CW ? G : w.CW, A2 = G < w.CP ? G : w.CP, De = A1 + A2;
    const int64_t Nu = w.B - w.Cc + A2 * w.L;
    const int64_t t = w.upper ? floor_div_clamped(Nu, De, -1, w.L)
                              : -floor_div_clamped(-Nu, De, -w.L - 1, 0);
    __int128 S;
    if (w.upper) {
        const uint64_t Rt = (uint64_t)(w.sx - N * t + sad) / 2;
        const uint32_t above = (uint32_t)(N - count_le(w.pre, t, N));
        S = mul_i64_u31(w.B, (uint32_t)N) - mul_u43((uint64_t)A1, (uint64_t)w.sx) +
            mul_u43((uint64_t)De, Rt) - mul_i64_u31(Nu - De * t, above);
    } else {
        const uint64_t Rt = (uint64_t)(N * t - w.sx + sad) / 2;
        const uint32_t below = (uint32_t)count_le(w.pre, t - 1, N);
        S = mul_i64_u31(w.Cc - A2 * w.L, (uint32_t)N) + mul_u43((uint64_t)A2, (uint64_t)w.sx) +
            mul_u43((uint64_t)De, Rt) - mul_i64_u31(De * t - Nu, below);
    }
    return sfix128_to_double(S);
}

template <bool kFinish>
__global__ __launch_bounds__(kRowThreads) void row_min_kernel(RowMinArgs a, int RB, int lp)
{
    __shared__ double q[kRowPairs + kRowMax];
    __shared__ float s_lam[kRowPairs];
    __shared__ RowInfo info[kRowMax];
    const int t = threadIdx.x, M = a.M;
    const long long rows = (long long)a.C * a.K;
    for (long long row0 = (long long)blockIdx.x * RB; row0 < rows; row0 += (long long)gridDim.x * RB) {
        const int rb = (int)min((long long)RB, rows - row0);
        // the first chunk's table entries, every load in flight before the rows' data
        constexpr int kPer = kRowPairs / kRowThreads;
        double v[kPer];
        auto load = [&](const double *S, int n) {
#pragma unroll
            for (int u = 0; u < kPer; ++u)
                if (t + u * kRowThreads < n) v[u] = S[t + u * kRowThreads];
        };
        load(a.S + row0 * M, rb * min(M, kRowPairs));
        const int c0 = (int)(row0 / a.K), k0 = (int)(row0 - (long long)c0 * a.K);
        if (t < rb) {
            const int c = c0 + (k0 + t) / a.K, k = (k0 + t) % a.K;
            const int s = seg_of(a.seg, c);
            RowInfo w{};
            w.N = (double)(a.offsets[s + 1] - a.offsets[s]);
            w.rN = __ddiv_rn(1.0, w.N);
            if (kFinish) {
                const float cpf = a.c_p[c], cwf = a.c_w[c];
                w.CP = fix33(cpf);
                w.CW = fix33(cwf);
                w.upper = cwf <= cpf;
                w.L = a.L[c];
                w.B = w.CW * a.eta[k];
                w.Cc = w.CP * (w.L - a.eta[k]);
                w.pre = a.pre + (long long)s * kHistBins;
                w.sx = (int64_t)w.pre[kHistBins - 1].sum();
            }
            info[t] = w;
        }
        __syncthreads();
        const int tasks = rb * a.E, per = kRowThreads / lp;  // tasks at a time
        const int ms = min(M, kRowPairs) | 1;                // odd row stride: no bank conflicts
        // (tasks reaches 2^31 - 1: the loop ends before b0 would pass it)
        for (int b0 = 0;; b0 += per) {
            const int task = b0 + t / lp, part = t % lp;
            const int e = task / rb, rr = task % rb;  // a radius's rows on consecutive lanes
            const int c = c0 + (k0 + rr) / a.K;
            const double ev = task < tasks ? (double)a.eps[(long long)e * a.C + c] : 0.0;
            double best = __builtin_inf();
            int bm = M;  // no multiplier yet: loses every comparison below
            for (int m0 = 0; m0 < M; m0 += kRowPairs) {
                const int mc = min(kRowPairs, M - m0);
                if (b0 == 0 || M > kRowPairs) {  // else the rows are still staged
                    for (int i = t; i < mc; i += kRowThreads) s_lam[i] = a.lam[m0 + i];
                    double *S = a.S + row0 * M + m0;  // (RB = 1 when M > kRowPairs)
                    if (b0 > 0 || m0 > 0) load(S, rb * mc);
                    int r = t / mc, m = t % mc;  // row and multiplier of entry i
                    const int dr = kRowThreads / mc, dm = kRowThreads % mc;
#pragma unroll
                    for (int u = 0; u < kPer; ++u) {
                        const int i = t + u * kRowThreads;
                        if (i >= rb * mc) break;
                        if (kFinish && b0 == 0) {
                            v[u] = finish_pair(info[r], a.lam[m0 + m], __double_as_longlong(v[u]));
                            S[i] = v[u];
                        }
                        // (a table from outside may hold anything: only a plain value takes the
                        // short division)
                        const uint32_t ex = ((uint32_t)__double2hiint(v[u]) >> 20) & 0x7ffu;
                        q[r * ms + m] = kFinish || ex - 100u < 1800u
                                            ? div_by(v[u], info[r].N, info[r].rN)
                                            : __ddiv_rn(v[u], info[r].N);
                        m += dm;
                        r += dr;
                        if (m >= mc) {
                            m -= mc;
                            ++r;
                        }
                    }
                    __syncthreads();
                }
                if (task < tasks)
                    for (int m = part; m < mc; m += lp) {
                        const double J = __dadd_rn(__dmul_rn((double)s_lam[m], ev), q[rr * ms + m]);
                        if (J < best) {
                            best = J;
                            bm = m0 + m;
                        }
                    }
                if (M > kRowPairs) __syncthreads();  // the next chunk overwrites the stage
            }
            for (int d = lp >> 1; d >= 1; d >>= 1) {
                const double ob = __shfl_xor(best, d, 64);
                const int om = __shfl_xor(bm, d, 64);
                if (ob < best || (ob == best && om < bm)) {
                    best = ob;
                    bm = om;
                }
            }
            if (part == 0 && task < tasks) {
                const long long o = ((long long)e * a.C + c) * a.K + (k0 + rr) % a.K;
                a.W[o] = best;
                if (a.m_star) a.m_star[o] = min(bm, M - 1);  // (no J below infinity: the last)
            }
            if (tasks - b0 <= per) break;
        }
        __syncthreads();  // the next rows overwrite the stage
    }
}

// The minimum over the multipliers from an S that is there, one wave per row: the wave
// stages q_m = S / N and lambda_m of a chunk of multipliers, its lanes split over up to 32
// radii, and nothing waits for another wave.  Bound by reading S where the rows are many
// and long.
constexpr int kWaveRows = 4;     // waves (rows) per block
constexpr int kWaveChunk = 256;  // multipliers staged per wave at a time
constexpr int kWaveRadii = 32;   // radii at most

__global__ __launch_bounds__(64 * kWaveRows) void row_min_wave_kernel(RowMinArgs a)
{
    __shared__ double2 st[kWaveRows][kWaveChunk];  // (q_m, lambda_m)
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, M = a.M;
    int lg = 0;  // log2 of the radii's groups of lanes
    while ((1 << lg) < a.E) ++lg;
    const int lp = 64 >> lg, part = lane & (lp - 1), e = lane / lp;
    double2 *q = st[w];
    // rows in a loop of whole waves (no block barrier)
    for (long long ck = (long long)blockIdx.x * kWaveRows + w; ck < (long long)a.C * a.K;
         ck += (long long)gridDim.x * kWaveRows) {
        const int c = (int)(ck / a.K), k = (int)(ck % a.K);
        const int s = seg_of(a.seg, c);
        const double N = (double)(a.offsets[s + 1] - a.offsets[s]);
        const double *row = a.S + ck * M;
        const double ev = e < a.E ? (double)a.eps[(long long)e * a.C + c] : 0.0;
        double best = __builtin_inf();
        int bm = M;  // no multiplier yet: loses every comparison below
        for (int m0 = 0; m0 < M; m0 += kWaveChunk) {
            const int mc = min(kWaveChunk, M - m0);
            __builtin_amdgcn_wave_barrier();  // the last chunk's reads come first
            for (int i = lane; i < mc; i += 64)
                q[i] = make_double2(__ddiv_rn(row[m0 + i], N), (double)a.lam[m0 + i]);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            for (int i = part; i < mc; i += lp) {
                const double2 v = q[i];
                const double J = __dadd_rn(__dmul_rn(v.y, ev), v.x);
                if (J < best) {
                    best = J;
                    bm = m0 + i;
                }
            }
        }
        for (int d = lp >> 1; d >= 1; d >>= 1) {
            const double ob = __shfl_xor(best, d, 64);
            const int om = __shfl_xor(bm, d, 64);
            if (ob < best || (ob == best && om < bm)) {
                best = ob;
                bm = om;
            }
        }
        if (part == 0 && e < a.E) {
            const long long o = ((long long)e * a.C + c) * a.K + k;
            a.W[o] = best;
            if (a.m_star) a.m_star[o] = min(bm, M - 1);  // (no J below infinity: the last)
        }
    }
}

hipError_t launch_row_min(const RowMinArgs &a, bool finish, int num_cu, hipStream_t st)
{
    // A wave per row where the chip has enough rows and few radii share a row: the whole
    // argmin call, row_min_kernel and this one, 32,768 rows of 128 multipliers 37 and 41 us,
    // of 256 47 and 46, of 1,024 107 and 78 (16 radii 243 and 195, 65 radii 1,192 and
    // 1,163); 6,000 rows of 256 31.6 and 31.0, of 2,000 65 and 47; 1,000 rows of 32 29.6 and
    // 28.2, of 512 30.3 and 29.6, of 1,024 31.2 and 31.7, of 4,096 39.5 and 50.7.
    const long long rows = (long long)a.C * a.K;
    if (!finish && a.E <= kWaveRadii &&
        (rows >= 16LL * num_cu ? a.M >= 256 : rows >= 2LL * num_cu && a.M <= 512)) {
        const long long blocks = std::min((rows + kWaveRows - 1) / kWaveRows, kMaxGridBlocks);
        hipLaunchKernelGGL(row_min_wave_kernel, dim3((unsigned)blocks), dim3(64 * kWaveRows), 0, st, a);
        return hipGetLastError();
    }
    // whole rows up to the stage's pairs, but at least two blocks per compute unit (and
    // (radius, row) tasks counted in 32 bits)
    const int RB = (int)std::max(1LL, std::min({(long long)kRowPairs / a.M, (long long)kRowMax,
                                                rows / (2 * num_cu), 0x7fffffffLL / a.E}));
    int lp = 64;
    while (lp > 1 && (long long)RB * a.E * lp > kRowThreads) lp >>= 1;
    const long long blocks = std::min((rows + RB - 1) / RB, kMaxGridBlocks);
    hipLaunchKernelGGL(finish ? row_min_kernel<true> : row_min_kernel<false>,
                       dim3((unsigned)blocks), dim3(kRowThreads), 0, st, a, RB, lp);
    return hipGetLastError();
}

}  // namespace dro
