// Exact parts of the reservation path: the value histograms and prefix sums,
// the exact table (F1) and the argmin over an exact W table, the
// critical-fractile quantile, the block-step sweep and device-data checks.
//
// Compiled with -ffp-contract=off: every double expression below is the
// round-to-nearest-even sequence written, with no fused multiply-add.
//
// Fixed point.  Inside the library's limits (integers <= 2^15, binary32
// coefficients in [2^-10, 2^7]) every candidate of phi (Appendix A, Step 4)
// is an integer multiple of 2^-33 below 2^56, so phi is evaluated exactly in
// 64-bit integers and summed exactly in 128-bit integers.  The reported value
// is J = RN(RN(lam eps) + RN(RN(S) / N)) with RN(S) the correctly rounded
// double of the exact sum.
#include <algorithm>
#include <type_traits>
#include <vector>

#include "dro_internal.h"
#include "fixed.h"
#include "sweep.h"
#include "wave.h"

namespace dro {

__device__ __forceinline__ int seg_of_x(const int32_t *seg, int c) { return seg ? seg[c] : c; }

#define HIPRET(expr)                                 \
    do {                                             \
        const hipError_t e_ = (expr);                \
        if (e_ != hipSuccess) return e_;             \
    } while (0)

__global__ void fill_u32_kernel(uint32_t *p, long long n, uint32_t v)
{
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x)
        p[i] = v;
}

// -------------------------------------------------------------- quantile ----
hipError_t launch_fill_u32(uint32_t *p, long long n, uint32_t v, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(fill_u32_kernel, dim3((unsigned)std::min((n + 255) / 256, kMaxGridBlocks)),
                       dim3(256), 0, st, p, n, v);
    return hipGetLastError();
}

// ------------------------------------------- staging in kernel arguments ----
// One launch for the offsets, the row table and the first kStageClasses classes'
// segments, one more for every further kStageClasses.
constexpr int kStageClasses = 2048;
struct StageArgs {
    int64_t off[kStageSegs + 1];
    int32_t row[kStageSegs + 1];
    uint8_t seg[kStageClasses];
};
static_assert(sizeof(StageArgs) <= 3584 && kStageSegs < 256, "within a launch's 4 KB of arguments");

__global__ void stage_args_kernel(StageArgs a, int entries, int classes, int64_t *offsets,
                                  int64_t *boff, int32_t *seg)
{
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t < entries) {
        offsets[t] = a.off[t];
        if (boff) boff[t] = a.row[t];
    }
    if (t < classes) seg[t] = a.seg[t];
}

hipError_t launch_stage_args(const int64_t *offsets_h, const int64_t *boff_h, int S,
                             const int32_t *seg_h, int C, int64_t *offsets, int64_t *boff,
                             int32_t *seg, hipStream_t st)
{
    if (S > kStageSegs) return hipErrorInvalidValue;
    StageArgs a{};
    for (int s = 0; s <= S; ++s) {
        a.off[s] = offsets_h[s];
        if (boff_h) a.row[s] = (int32_t)boff_h[s];
    }
    int c0 = 0;
    do {
        const int n = seg_h ? std::min(C - c0, kStageClasses) : 0;
        const int entries = c0 == 0 ? S + 1 : 0;
        for (int i = 0; i < n; ++i) a.seg[i] = (uint8_t)seg_h[c0 + i];
        hipLaunchKernelGGL(stage_args_kernel, dim3((unsigned)(std::max(entries, n) + 255) / 256),
                           dim3(256), 0, st, a, entries, n, offsets, boff, seg ? seg + c0 : nullptr);
        HIPRET(hipGetLastError());
        c0 += n;
    } while (seg_h && c0 < C);
    return hipSuccess;
}

// Calls count(x) for every sample of xi[lo, hi) handed to this thread of a
// kThreadsT-thread block: an unaligned head (up to the first 16-byte aligned
// address), a 16-byte body and a tail.  In the body every thread keeps eight
// 16-byte loads in flight, in two register sets of four: the next round's
// loads are issued before this round's samples are counted.  Body vector i
// goes to thread i mod kThreadsT, so even and odd threads see alternate
// vectors.  prologue() (block-wide: every thread calls it) runs once the
// first four loads are in flight and before any count, so the block's set-up
// (clearing its LDS counts) overlaps their latency.
template <int kThreadsT, class F, class G>
__device__ __forceinline__ void for_each_sample(const int32_t *xi, long long lo, long long hi, F &&count,
                                                G &&prologue)
{
    const int t = threadIdx.x;
    const long long mis = (long long)((reinterpret_cast<uintptr_t>(xi + lo) >> 2) & 3u);
    const long long a0 = min(hi, lo + ((4 - mis) & 3));
    const long long a1 = a0 + ((hi - a0) & ~3LL);
    const int4 *v4 = reinterpret_cast<const int4 *>(xi + a0);
    const long long nv = (a1 - a0) / 4;
    constexpr long long kRound = 4LL * kThreadsT;
    int4 qa[4], qb[4];
    // (unconditional loads, clamped to the last vector, so all four issue
    // back to back; tally skips the ones past the end)
    auto load = [&](long long r0, int4 (&d)[4]) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const long long i = r0 + r * kThreadsT + t;
            d[r] = v4[i < nv ? i : nv - 1];
        }
    };
    auto tally = [&](long long r0, const int4 (&d)[4]) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            if (r0 + r * kThreadsT + t >= nv) continue;
            count(d[r].x);
            count(d[r].y);
            count(d[r].z);
            count(d[r].w);
        }
    };
    if (nv > 0) load(0, qa);
    prologue();
    for (long long n = lo + t; n < a0; n += kThreadsT) count(xi[n]);
    for (long long r0 = 0; r0 < nv; r0 += 2 * kRound) {
        load(r0 + kRound, qb);
        tally(r0, qa);
        load(r0 + 2 * kRound, qa);
        tally(r0 + kRound, qb);
    }
    for (long long n = a1 + t; n < hi; n += kThreadsT) count(xi[n]);
}

// Block (segment s, part b of B): a private 32-bit LDS histogram of the values
// 0 .. 2^15 (128 KB) over its 1/B share of the segment, then added into the
// segment's histogram: with plain stores when the block covers the whole
// segment (B == 1), else with one atomic add per non-zero bin into a histogram
// the launch has zeroed (integer adds, so the result does not depend on the
// order).  Only the distinct values of a block cost a global access: about
// 7,800 of the 32,769 bins for a block of 62,500 heavy-tailed lengths.
constexpr int kHistThreads = 1024;

__global__ __launch_bounds__(kHistThreads) void histogram_kernel(const int64_t *offsets,
                                                                 const int32_t *xi, int B,
                                                                 uint32_t *hist)
{
    extern __shared__ uint32_t h[];  // kHistBins words
    const int s = (int)(blockIdx.x / B), b = (int)(blockIdx.x % B);
    const long long n0 = offsets[s], N = offsets[s + 1] - n0;
    const long long lo = n0 + (N * b) / B, hi = n0 + (N * (b + 1)) / B;
    const int t = threadIdx.x;
    for_each_sample<kHistThreads>(
        xi, lo, hi,
        [&](int v) {
            v = v < 0 ? 0 : (v > kHistBins - 1 ? kHistBins - 1 : v);
            atomicAdd(&h[v], 1u);
        },
        [&] {
            for (int i = t; i < kHistBins; i += kHistThreads) h[i] = 0;
            __syncthreads();
        });
    __syncthreads();
    uint32_t *o = hist + (long long)s * kHistBins;
    if (B == 1) {
        for (int i = t; i < kHistBins; i += kHistThreads) o[i] = h[i];
    } else {
        for (int i = t; i < kHistBins; i += kHistThreads) {
            const uint32_t c = h[i];
            if (c) atomicAdd(o + i, c);
        }
    }
}

__device__ int64_t exact_rank(float cp, float cw, int64_t N);

// ---- class_quantile: per-block histograms, then one select per class ----
//
// Block for row r (segment s, part b of its B_s parts, at most kQMaxPart
// samples; rows in a block-uniform loop) counts its share in LDS with 16-bit
// counts packed two to a word (value v < 2^15 in word v mod 2^14, low half
// for v < 2^14, high half above; 2^15 in the low half of word 2^14), in two
// copies: even threads add into one, odd threads into the other, which halves
// the lanes of one wave that meet on one LDS word when short lengths repeat.
// It then stores the two copies' sum (every count fits 16 bits, as the block
// holds at most 65,535 samples) with 16-byte non-temporal stores, as only the
// select reads it, once (on mixture-16x1M 1.4 us less per launch than plain
// stores), and, in the same pass, its counts per coarse bucket of 128 values.
// Segment s owns rows s B .. s B + B - 1 when every segment has B parts, else
// rows boff[s] .. boff[s + 1] - 1 of a table built by the host, in which the
// block finds its segment by bisection.  No global atomics: the select reads
// the segment's rows of the bucket it needs.
//
// kSums: also the sum of the values of each coarse bucket (below 2^31: 65,535
// samples of at most 2^15), which the prefix pass starts its chunks from.
constexpr int kQThreads = 1024;
typedef uint32_t u32x4_nt __attribute__((ext_vector_type(4)));

// The samples [lo, hi) of row r.
struct RowPart {
    long long lo, hi;
};

__device__ __forceinline__ RowPart row_part(const int64_t *offsets, int S, int B,
                                            const int64_t *boff, long long r)
{
    int s;
    long long b, Bs;
    if (boff) {  // the segment whose rows hold r: boff[s] <= r < boff[s + 1]
        int a = 0, z = S;
        while (z - a > 1) {
            const int mid = (a + z) >> 1;
            if (boff[mid] <= r) a = mid;
            else z = mid;
        }
        s = a;
        b = r - boff[s];
        Bs = boff[s + 1] - boff[s];
    } else {
        s = (int)(r / B);
        b = r % B;
        Bs = B;
    }
    const long long n0 = offsets[s], N = offsets[s + 1] - n0;
    return RowPart{n0 + (N * b) / Bs, n0 + (N * (b + 1)) / Bs};
}

template <bool kSums>
__global__ __launch_bounds__(kQThreads) void qhist_kernel(const int64_t *offsets, const int32_t *xi,
                                                          int S, int B, const int64_t *boff,
                                                          long long rows, uint32_t *fine,
                                                          uint32_t *coarse, uint32_t *csum)
{
    extern __shared__ uint32_t h[];  // 2 x kQStride words
    const int t = threadIdx.x;
    for (long long r = blockIdx.x; r < rows; r += gridDim.x) {
        const RowPart rp = row_part(offsets, S, B, boff, r);
        uint32_t *hc = h + (t & 1) * kQStride;
        uint4 *h4 = reinterpret_cast<uint4 *>(h);
        const uint4 *g4 = reinterpret_cast<const uint4 *>(h + kQStride);
        for_each_sample<kQThreads>(
            xi, rp.lo, rp.hi,
            [&](int v) {
                v = v < 0 ? 0 : (v > kQTop ? kQTop : v);
                // bit 14 of v selects the half (v = 2^15 has it clear)
                atomicAdd(&hc[v < kQTop ? (v & (kQTop / 2 - 1)) : kQTop / 2], 1u << ((v >> 10) & 16));
            },
            [&] {
                for (int i = t; i < 2 * kQStride / 4; i += kQThreads) h4[i] = make_uint4(0u, 0u, 0u, 0u);
                __syncthreads();
            });
        __syncthreads();
        // 16-byte word group q = t + 1024 i (i < 4) holds the words 4q .. 4q + 3:
        // the values of coarse bucket q / 32 in its low halves and of bucket
        // 128 + q / 32 in its high halves, so the 32 lanes t mod 32 = 0 .. 31 of a
        // half-wave share both buckets.  The packed words add as plain 32-bit
        // integers: no sum of low halves exceeds the block's 65,535 samples.
        static_assert(kQThreads * 16 == kQTop / 2, "four word groups per thread");
        static_assert(kQStride % 4 == 0 && kQStride >= kQTop / 2 + 4, "row of whole word groups");
        uint4 *out = reinterpret_cast<uint4 *>(fine + r * kQStride);
        uint32_t *co = coarse + r * kQBuckets;
    #pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int q = t + kQThreads * i;
            const uint4 x = h4[q], y = g4[q];
            const uint4 c = make_uint4(x.x + y.x, x.y + y.y, x.z + y.z, x.w + y.w);
            __builtin_nontemporal_store(u32x4_nt{c.x, c.y, c.z, c.w}, reinterpret_cast<u32x4_nt *>(out + q));
            uint32_t p = (c.x + c.y) + (c.z + c.w);
            const int bk = q >> 5;
            // sums of the values less the bucket's first one (below 2^23)
            uint32_t vl = 0, vh = 0;
            if (kSums) {
                const uint32_t o = 4u * (q & 31), pl = p & 0xffffu, ph = p >> 16;
                vl = o * pl + (c.y & 0xffffu) + 2u * (c.z & 0xffffu) + 3u * (c.w & 0xffffu);
                vh = o * ph + (c.y >> 16) + 2u * (c.z >> 16) + 3u * (c.w >> 16);
            }
            p = scan_half32(p);
            if (kSums) {
                vl = scan_half32(vl);
                vh = scan_half32(vh);
            }
            if ((t & 31) == 31) {
                // the last bucket also holds the value 2^15
                const uint32_t top =
                    bk == 127 ? (h[kQTop / 2] + h[kQStride + kQTop / 2]) & 0xffffu : 0u;
                co[bk] = p & 0xffffu;
                co[128 + bk] = (p >> 16) + top;
                if (kSums) {
                    uint32_t *cv = csum + r * kQBuckets;
                    cv[bk] = vl + 128u * bk * (p & 0xffffu);
                    cv[128 + bk] = vh + (kQTop / 2 + 128u * bk) * (p >> 16) + (uint32_t)kQTop * top;
                }
            }
        }
        if (t == 0) {  // the group of the value 2^15 and the padding words
            const uint4 x = h4[kQTop / 8], y = g4[kQTop / 8];
            out[kQTop / 8] = make_uint4(x.x + y.x, x.y + y.y, x.z + y.z, x.w + y.w);
        }
        __syncthreads();  // the next row clears the counts this row has read
    }
}

// The sum of f(p[r stride]) over the rows r = g, g + kStep, ... below B.
template <int kStep, class F>
__device__ __forceinline__ uint32_t sum_rows(const uint32_t *p, int stride, int g, int B, F &&f)
{
    uint32_t a = 0;
    auto take = [&](auto n) {  // n rows, every load in flight
        constexpr int kN = decltype(n)::value;
        for (; g + (kN - 1) * kStep < B; g += kN * kStep) {
            uint32_t x[kN];
#pragma unroll
            for (int i = 0; i < kN; ++i) x[i] = p[(long long)(g + i * kStep) * stride];
#pragma unroll
            for (int i = 0; i < kN; ++i) a += f(x[i]);
        }
    };
    take(std::integral_constant<int, 16>{});
    take(std::integral_constant<int, 4>{});
    take(std::integral_constant<int, 1>{});
    return a;
}

// Class c (segment s, its B rows at s B0 or boff[s]; classes in a
// block-uniform loop): the coarse counts of the rows summed per bucket, the
// bucket holding the exact rank j, then the counts of its values summed over
// the rows, and the value where the cumulative count reaches j.  A thread has 16
// rows' loads in flight, as a class of many rows (763 of 5e7 samples) is a chain of
// round trips else.
__device__ void qselect_class(const int64_t *offsets, const int32_t *seg, const float *c_p,
                              const float *c_w, const uint32_t *fine, const uint32_t *coarse, int B0,
                              const int64_t *boff, int c, int32_t *q_value, int64_t *q_rank)
{
    constexpr int kG = kQThreads / kQBuckets;  // row groups of the coarse sum
    constexpr int kF = 129;                    // values of a bucket (the last adds 2^15)
    constexpr int kFG = kQThreads / 128;       // row groups of the fine sum
    __shared__ uint32_t part[kG][kQBuckets];
    __shared__ uint32_t fpart[kFG][kF];
    __shared__ uint32_t wsum[kQBuckets / 64];
    __shared__ int sel;
    __shared__ long long sel_below;
    __shared__ int64_t s_off[2], s_rank;
    __shared__ float s_cost[2];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int s = seg_of_x(seg, c);
    // the rank's inputs, loaded by every thread from addresses that differ by
    // lane: vector loads in flight with the coarse loads below, not waited for
    // before them as uniform scalar loads would be
    const int64_t r_off = offsets[s + (t & 1)];
    const float r_cost = ((t & 2) ? c_w : c_p)[c];
    // the segment's rows: B0 per segment, or those of the table boff
    const long long row0 = boff ? boff[s] : (long long)s * B0;
    const int B = boff ? (int)(boff[s + 1] - row0) : B0;
    const uint32_t *cs = coarse + row0 * kQBuckets;
    const uint32_t *fs = fine + row0 * kQStride;
    {
        const int q = t % kQBuckets, g = t / kQBuckets;
        part[g][q] = sum_rows<kG>(cs + q, kQBuckets, g, B, [](uint32_t x) { return x; });
    }
    if (t == 0) sel = -1;
    if (t < 2) s_off[t] = r_off;         // offsets[s], offsets[s + 1]
    if ((t | 2) == 2) s_cost[t >> 1] = r_cost;  // t = 0: c_p[c], t = 2: c_w[c]
    __syncthreads();
    // the rank on a wave that has no bucket to scan (with the scans by DPP moves the
    // kernel takes 4.8 us on 16 classes of 1e6 samples, 5.3 with shuffles and thread 0)
    if (t == kQThreads - 64) s_rank = exact_rank(s_cost[0], s_cost[1], s_off[1] - s_off[0]);
    // inclusive scan of the bucket totals (threads 0 .. 255), then the bucket
    // whose range of ranks holds j
    uint32_t tot = 0, incl = 0;
    if (t < kQBuckets) {
#pragma unroll
        for (int g = 0; g < kG; ++g) tot += part[g][t];
        incl = scan_wave(tot);
        if (lane == 63) wsum[wave] = incl;
    }
    __syncthreads();
    const int64_t j = s_rank;
    if (t < kQBuckets) {
        for (int w = 0; w < wave; ++w) incl += wsum[w];
        const int64_t before = (int64_t)(incl - tot);
        if (before < j && j <= (int64_t)incl) {
            sel = t;
            sel_below = before;
        }
    }
    __syncthreads();
    const int bk = sel;  // j is in [1, N] and the totals sum to N, so one bucket holds it
    if (bk < 0) return;
    const int v0 = bk < 128 ? 128 * bk : kQTop / 2 + 128 * (bk - 128);
    {
        // thread t: value v0 + t mod 128 over the rows t / 128, t / 128 + kFG, ...;
        // threads of the first group also count 2^15 in the last bucket
        const int o = t % 128, g = t / 128;
        const int v = v0 + o;
        const int w = v & (kQTop / 2 - 1), sh = (v >> 10) & 16;
        const bool top = bk == kQBuckets - 1 && o == 0;
        fpart[g][o] = sum_rows<kFG>(fs + w, kQStride, g, B,
                                    [&](uint32_t x) { return (x >> sh) & 0xffffu; });
        uint32_t a_top = 0;
        if (top)
            a_top = sum_rows<kFG>(fs + kQTop / 2, kQStride, g, B,
                                  [](uint32_t x) { return x & 0xffffu; });
        if (o == 0) fpart[g][128] = a_top;
    }
    __syncthreads();
    // scan over the bucket's 129 value slots (threads 0 .. 255; slot 128 is 2^15)
    uint32_t f = 0, fin = 0;
    if (t < kQBuckets) {
        if (t < kF)
#pragma unroll
            for (int g = 0; g < kFG; ++g) f += fpart[g][t];
        fin = scan_wave(f);
        if (lane == 63) wsum[wave] = fin;
    }
    __syncthreads();
    if (t < kF) {
        for (int w = 0; w < wave; ++w) fin += wsum[w];
        const int64_t before = sel_below + (int64_t)(fin - f);
        if (before < j && j <= before + (int64_t)f) q_value[c] = t < 128 ? v0 + t : kQTop;
    }
    if (t == 0) q_rank[c] = j;
}

// classes in a block-uniform loop; the barrier lets the next class reuse the LDS
__global__ __launch_bounds__(kQThreads) void qselect_kernel(const int64_t *offsets,
                                                            const int32_t *seg, const float *c_p,
                                                            const float *c_w, const uint32_t *fine,
                                                            const uint32_t *coarse, int B,
                                                            const int64_t *boff, int C,
                                                            int32_t *q_value, int64_t *q_rank)
{
    for (long long c = blockIdx.x; c < C; c += gridDim.x) {
        qselect_class(offsets, seg, c_p, c_w, fine, coarse, B, boff, (int)c, q_value, q_rank);
        __syncthreads();
    }
}

hipError_t qhist_prepare();

hipError_t hist_prepare()
{
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(histogram_kernel),
                                             hipFuncAttributeMaxDynamicSharedMemorySize,
                                             (int)(kHistBins * sizeof(uint32_t)));
    if (e != hipSuccess) return e;
    return qhist_prepare();
}

long long row_part_len(const int64_t *offsets_h, int S, int num_cu)
{
    // The shortest parts whose rows still fit one resident block per compute
    // unit (their LDS counts allow one; a few more rows than units would take a
    // second pass over the chip), at least 16,384 samples, below which a row's
    // fixed cost (clearing and storing its counts) passes its reading time, at
    // least a 128th of the longest segment, whose rows the select and the prefix
    // pass read one after the other (5e6 samples beside two short segments: the
    // quantile 42 us with 254 rows, 38 with 128, the counts 54 and 45), and at most
    // what 16-bit counts hold.
    const long long slots = (long long)num_cu * ((S + num_cu - 1) / num_cu);
    long long max_n = 0;
    for (int s = 0; s < S; ++s) max_n = std::max(max_n, (long long)(offsets_h[s + 1] - offsets_h[s]));
    long long lo = std::min(kQMaxPart, std::max(16384LL, (max_n + 127) / 128)), hi = kQMaxPart;
    // (only segments above the shortest part have more than one row: the search looks
    // those through, not the many short ones of a large problem)
    std::vector<long long> large;
    for (int s = 0; s < S; ++s) {
        const long long n = offsets_h[s + 1] - offsets_h[s];
        if (n > lo) large.push_back(n);
    }
    while (lo < hi) {
        const long long mid = (lo + hi) / 2;
        long long rows = S - (long long)large.size();
        for (size_t i = 0; i < large.size() && rows <= slots; ++i) rows += row_parts(large[i], mid);
        if (rows <= slots) hi = mid;
        else lo = mid + 1;
    }
    return lo;
}

int hist_parts(int S, long long max_seg, int num_cu)
{
    // about one resident block per compute unit, at least 16K samples per block
    long long B = std::max(1LL, (long long)num_cu / std::max(S, 1));
    B = std::min(B, std::max(1LL, max_seg / 16384));
    return (int)B;
}

hipError_t launch_histogram(const int64_t *offsets, const int32_t *xi, int S, int B,
                            uint32_t *hist, hipStream_t st)
{
    if (S <= 0) return hipSuccess;
    if (B > 1) HIPRET(launch_fill_u32(hist, (long long)S * kHistBins, 0u, st));
    hipLaunchKernelGGL(histogram_kernel, dim3((unsigned)((long long)S * B)), dim3(kHistThreads),
                       kHistBins * sizeof(uint32_t), st, offsets, xi, B, hist);
    return hipGetLastError();
}

// Exact rank j = ceil(c_p N / (c_p + c_w)) in [1, N]: estimate in double,
// then correct with exact 128-bit products.
__device__ int64_t exact_rank(float cp, float cw, int64_t N)
{
    const uint64_t P = (uint64_t)fix33(cp), Wc = (uint64_t)fix33(cw);
    const uint64_t den = P + Wc;
    const unsigned __int128 num = (unsigned __int128)P * (uint64_t)N;
    int64_t j = (int64_t)ceil((double)P / (double)den * (double)N);
    if (j < 1) j = 1;
    if (j > N) j = N;
    while (j > 1 && (unsigned __int128)(uint64_t)(j - 1) * den >= num) --j;
    while (j < N && (unsigned __int128)(uint64_t)j * den < num) ++j;
    return j;
}

// One wave per class: the j-th smallest sample is the first value whose prefix
// count reaches j, found in three 64-way steps (513 values a lane, then 9, then
// one).
constexpr int kSelWaves = 4;  // classes per block

__global__ __launch_bounds__(64 * kSelWaves) void prefix_select_kernel(
    const int64_t *offsets, const int32_t *seg, const float *c_p, const float *c_w,
    const PrefixEntry *pre, int C, int32_t *q_value)
{
    const int lane = threadIdx.x & 63;
    // classes in a loop of whole waves (no block barrier)
    for (long long c = (long long)blockIdx.x * kSelWaves + (threadIdx.x >> 6); c < C;
         c += (long long)gridDim.x * kSelWaves) {
        const int s = seg_of_x(seg, (int)c);
        const int64_t j = exact_rank(c_p[c], c_w[c], offsets[s + 1] - offsets[s]);
        const PrefixEntry *pc = pre + (long long)s * kHistBins;
        int v0 = 0;  // the answer is in [v0, v0 + 64 step)
        for (int step = 513; step >= 1; step = step == 513 ? 9 : (step == 9 ? 1 : 0)) {
            const int v = min(v0 + (lane + 1) * step - 1, kHistBins - 1);
            const unsigned long long reach = __ballot((int64_t)pc[v].cnt >= j);
            // the last lane's value is 2^15 or past the answer, so some lane reaches j <= N
            v0 += (reach ? __ffsll(reach) - 1 : 63) * step;
        }
        if (lane == 0) q_value[c] = min(v0, kHistBins - 1);
    }
}

hipError_t launch_prefix_select(const int64_t *offsets, const int32_t *seg, const float *c_p,
                                const float *c_w, const PrefixEntry *pre, int C, int32_t *q_value,
                                hipStream_t st)
{
    const long long blocks = std::min(((long long)C + kSelWaves - 1) / kSelWaves, kMaxGridBlocks);
    hipLaunchKernelGGL(prefix_select_kernel, dim3((unsigned)blocks), dim3(64 * kSelWaves), 0, st,
                       offsets, seg, c_p, c_w, pre, C, q_value);
    return hipGetLastError();
}

hipError_t qhist_prepare()
{
    const int bytes = (int)(2 * kQStride * sizeof(uint32_t));
    HIPRET(hipFuncSetAttribute(reinterpret_cast<const void *>(qhist_kernel<false>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, bytes));
    return hipFuncSetAttribute(reinterpret_cast<const void *>(qhist_kernel<true>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
}

hipError_t launch_class_quantile(const int64_t *offsets, const int32_t *seg, const int32_t *xi,
                                 const float *c_p, const float *c_w, int S, int C, const RowPlan &pl,
                                 uint32_t *fine, uint32_t *coarse, int32_t *q_value,
                                 int64_t *q_rank, hipStream_t st)
{
    hipLaunchKernelGGL(qhist_kernel<false>, dim3((unsigned)std::min(pl.rows, kMaxGridBlocks)),
                       dim3(kQThreads), 2 * kQStride * sizeof(uint32_t), st, offsets, xi, S, pl.B,
                       pl.boff, pl.rows, fine, coarse, (uint32_t *)nullptr);
    HIPRET(hipGetLastError());
    hipLaunchKernelGGL(qselect_kernel, dim3((unsigned)std::min((long long)C, kMaxGridBlocks)),
                       dim3(kQThreads), 0, st, offsets, seg, c_p, c_w, fine, coarse, pl.B, pl.boff,
                       C, q_value, q_rank);
    return hipGetLastError();
}

// ------------------------------------------------------------ block step ----
// best[c, k] = the lowest k' <= k with the smallest W[c, k'] (k where no value is
// below infinity): one block per class, a run of consecutive points per thread,
// the runs' minima scanned over the block.
constexpr int kBestThreads = 256;

__global__ __launch_bounds__(kBestThreads) void best_upto_kernel(const double *W, int K,
                                                                 int32_t *best)
{
    __shared__ double sw[kBestThreads / 64];
    __shared__ int sk[kBestThreads / 64];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const double *w = W + (long long)blockIdx.x * K;
    int32_t *o = best + (long long)blockIdx.x * K;
    const int per = (K + kBestThreads - 1) / kBestThreads;
    const int k0 = min(t * per, K), k1 = min(k0 + per, K);
    double bw = __builtin_inf();
    int bk = 0x7fffffff;
    for (int k = k0; k < k1; ++k)
        if (w[k] < bw) {
            bw = w[k];
            bk = k;
        }
    // the minimum of the runs before this one, the earlier among equals
    for (int d = 1; d < 64; d <<= 1) {
        const double w2 = __shfl_up(bw, d, 64);
        const int k2 = __shfl_up(bk, d, 64);
        if (lane >= d && !(bw < w2)) {
            bw = w2;
            bk = k2;
        }
    }
    if (lane == 63) {
        sw[wave] = bw;
        sk[wave] = bk;
    }
    const double ew = __shfl_up(bw, 1, 64);
    const int ek = __shfl_up(bk, 1, 64);
    __syncthreads();
    double cw = __builtin_inf();
    int ck = 0x7fffffff;
    for (int i = 0; i < wave; ++i)
        if (sw[i] < cw) {
            cw = sw[i];
            ck = sk[i];
        }
    if (lane > 0 && ew < cw) {
        cw = ew;
        ck = ek;
    }
    for (int k = k0; k < k1; ++k) {
        if (w[k] < cw) {
            cw = w[k];
            ck = k;
        }
        o[k] = min(ck, k);
    }
}

hipError_t launch_best_upto(const double *W, int C, int K, int32_t *best, hipStream_t st)
{
    hipLaunchKernelGGL(best_upto_kernel, dim3((unsigned)C), dim3(kBestThreads), 0, st, W, K, best);
    return hipGetLastError();
}

// The Gauss-Seidel sweep of the block step, one wave (sweep.h), then the values at
// the new grid points and every group's usage.
__global__ __launch_bounds__(64) void bcd_sweep_kernel(const double *W, const int32_t *best,
                                                       const int32_t *eta, int C, int K, int G,
                                                       const float *cap, const float *conc,
                                                       float kappa, const int32_t *k_prev,
                                                       int32_t *kcur, int32_t *k_next,
                                                       double *W_star, uint8_t *feasible,
                                                       double *usage)
{
    __shared__ double lds[kSweepLds];
    const int t = threadIdx.x;
    const double onek = __dadd_rn(1.0, (double)kappa);
    sweep_wave(best, eta, C, K, G, conc, cap, onek, 0.0, k_prev, kcur, lds,
               [&](int c, int, bool feas) { feasible[c] = feas ? 1 : 0; });
    wave_sync();
    for (int g = t; g < G; g += 64) {
        double sum = 0.0;
        for (int c = 0; c < C; ++c)
            sum = __dadd_rn(sum, __dmul_rn((double)conc[(long long)c * G + g], (double)eta[kcur[c]]));
        usage[g] = __dmul_rn(onek, sum);
    }
    for (int c = t; c < C; c += 64) {
        k_next[c] = kcur[c];
        W_star[c] = W[(long long)c * K + kcur[c]];
    }
}

hipError_t launch_bcd_sweep(const double *W, const int32_t *best, const int32_t *eta, int C, int K,
                            int G, const float *cap, const float *conc, float kappa,
                            const int32_t *k_prev, int32_t *kcur, int32_t *k_next, double *W_star,
                            uint8_t *feasible, double *usage, hipStream_t st)
{
    hipLaunchKernelGGL(bcd_sweep_kernel, dim3(1), dim3(64), 0, st, W, best, eta, C, K, G, cap, conc,
                       kappa, k_prev, kcur, k_next, W_star, feasible, usage);
    return hipGetLastError();
}

// ------------------------------------------------------------ validation ----
// Block (segment s, part b of B): the smallest and largest sample of its share
// of the segment, merged into mn[s] / mx[s] with atomic min / max (which the
// caller sets to INT_MAX / INT_MIN first); the result does not depend on order.
__global__ __launch_bounds__(256) void seg_minmax_kernel(const int64_t *offsets, const int32_t *xi,
                                                         int B, int32_t *mn, int32_t *mx)
{
    const int s = (int)(blockIdx.x / B), b = (int)(blockIdx.x % B), t = threadIdx.x;
    const long long n0 = offsets[s], N = offsets[s + 1] - n0;
    const long long lo = n0 + (N * b) / B, hi = n0 + (N * (b + 1)) / B;
    int a = 0x7fffffff, c = -0x7fffffff - 1;
    for (long long n = lo + t; n < hi; n += 256) {
        const int v = xi[n];
        a = v < a ? v : a;
        c = v > c ? v : c;
    }
    __shared__ int sa[256], sb[256];
    sa[t] = a;
    sb[t] = c;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (t < w) {
            sa[t] = sa[t + w] < sa[t] ? sa[t + w] : sa[t];
            sb[t] = sb[t + w] > sb[t] ? sb[t + w] : sb[t];
        }
        __syncthreads();
    }
    if (t == 0 && hi > lo) {
        atomicMin(&mn[s], sa[0]);
        atomicMax(&mx[s], sb[0]);
    }
}

hipError_t launch_seg_minmax(const int64_t *offsets, const int32_t *xi, int S, long long max_seg,
                             int32_t *mn, int32_t *mx, hipStream_t st)
{
    // about 16K samples per block, at most 4096 blocks in all
    const long long B = std::max(1LL, std::min(std::max(1LL, 4096LL / S), (max_seg + 16383) / 16384));
    HIPRET(launch_fill_u32(reinterpret_cast<uint32_t *>(mn), S, 0x7fffffffu, st));
    HIPRET(launch_fill_u32(reinterpret_cast<uint32_t *>(mx), S, 0x80000000u, st));
    hipLaunchKernelGGL(seg_minmax_kernel, dim3((unsigned)(S * B)), dim3(256), 0, st, offsets, xi,
                       (int)B, mn, mx);
    return hipGetLastError();
}

}  // namespace dro

namespace dro {

// ============================================================ exact table ====
// The whole table from value counts (the production alternative to the dense
// pass when only results are needed; it does not evaluate per-sample terms).
// For 0 <= x, eta <= L the three candidates of Step 4 reduce to the larger of
// two lines, phi = max(B - a1 x, C - a2 (L - x)) with B = c_w eta,
// C = c_p (L - eta), a1 = min(g, c_w), a2 = min(g, c_p); the first wins exactly
// for (a1 + a2) x <= B - C + a2 L.  With the counts cnt(v) = #{x <= v} and sums
// sum(v) = sum{x : x <= v} of the segment, and t the last sample value on the
// first line's side,
//   S = B cnt(t) - a1 sum(t) + (C - a2 L)(N - cnt(t)) + a2 (sum_all - sum(t)),
// evaluated in 128-bit integers in units of 2^-33: exact.

// Per segment: cnt[v] = #{x <= v} (u32) and sum[v] = sum of the samples <= v
// (u64), from the value histogram, in two passes over blocks of (segment,
// chunk of 4096 bins): the chunk totals, then per chunk the sum of the totals
// before it, the chunk staged in LDS (padded to spread the per-thread runs over
// the banks) and scanned (16 consecutive bins per thread, then across threads),
// and each thread's run of prefixes stored.
constexpr int kPrefixThreads = 256;
constexpr int kPrefixPer = kPrefixChunk / kPrefixThreads;  // 16

__device__ __forceinline__ int pad32(int j) { return j + (j >> 5); }

// Per (segment, chunk): the count and the value-weighted sum of the chunk's
// bins, tot[(s * kPrefixChunks + ch) * 2 + {0, 1}].
__global__ __launch_bounds__(kPrefixThreads) void chunk_total_kernel(const uint32_t *hist,
                                                                     uint64_t *tot)
{
    __shared__ uint64_t rc[kPrefixThreads], rs[kPrefixThreads];
    const int ch = (int)(blockIdx.x % kPrefixChunks), s = (int)(blockIdx.x / kPrefixChunks);
    const int t = threadIdx.x;
    const uint32_t *h = hist + (long long)s * kHistBins;
    const int v0 = ch * kPrefixChunk, v1 = min(kHistBins, v0 + kPrefixChunk);
    uint64_t bc = 0, bs = 0;
    for (int v = v0 + t; v < v1; v += kPrefixThreads) {
        const uint64_t x = h[v];
        bc += x;
        bs += x * (uint64_t)v;
    }
    rc[t] = bc;
    rs[t] = bs;
    __syncthreads();
    for (int w = kPrefixThreads / 2; w > 0; w >>= 1) {
        if (t < w) {
            rc[t] += rc[t + w];
            rs[t] += rs[t + w];
        }
        __syncthreads();
    }
    if (t == 0) {
        tot[(long long)blockIdx.x * 2] = rc[0];
        tot[(long long)blockIdx.x * 2 + 1] = rs[0];
    }
}

__global__ __launch_bounds__(kPrefixThreads) void prefix_kernel(const uint32_t *hist,
                                                                const uint64_t *tot,
                                                                PrefixEntry *pre)
{
    __shared__ uint32_t hc[kPrefixChunk + kPrefixChunk / 32];
    __shared__ uint64_t rc[kPrefixThreads / 64], rs[kPrefixThreads / 64];
    const int ch = (int)(blockIdx.x % kPrefixChunks), s = (int)(blockIdx.x / kPrefixChunks);
    const int t = threadIdx.x;
    const uint32_t *h = hist + (long long)s * kHistBins;
    const int v0 = ch * kPrefixChunk, v1 = min(kHistBins, v0 + kPrefixChunk), n = v1 - v0;
    for (int j = t; j < n; j += kPrefixThreads) hc[pad32(j)] = h[v0 + j];
    uint64_t base_c = 0, base_s = 0;  // everything before the chunk, in chunk order
    const uint64_t *tt = tot + (long long)s * kPrefixChunks * 2;
    for (int i = 0; i < ch; ++i) {
        base_c += tt[2 * i];
        base_s += tt[2 * i + 1];
    }
    __syncthreads();
    const int a = t * kPrefixPer;
    uint64_t lc = 0, ls = 0;
    for (int i = 0; i < kPrefixPer; ++i) {
        const int j = a + i;
        if (j < n) {
            const uint64_t x = hc[pad32(j)];
            lc += x;
            ls += x * (uint64_t)(v0 + j);
        }
    }
    // inclusive scans of the thread totals: shuffles within each wave, then
    // the totals of the waves before
    const int lane = t & 63, wave = t >> 6;
    uint64_t ic = lc, is = ls;
    for (int d = 1; d < 64; d <<= 1) {
        const uint64_t oc = __shfl_up(ic, d, 64), os = __shfl_up(is, d, 64);
        if (lane >= d) {
            ic += oc;
            is += os;
        }
    }
    if (lane == 63) {
        rc[wave] = ic;
        rs[wave] = is;
    }
    __syncthreads();
    for (int w = 0; w < wave; ++w) {
        ic += rc[w];
        is += rs[w];
    }
    uint64_t c = base_c + ic - lc, x = base_s + is - ls;
    PrefixEntry *gp = pre + (long long)s * kHistBins + v0;
    for (int i = 0; i < kPrefixPer; ++i) {
        const int j = a + i;
        if (j < n) {
            const uint64_t hv = hc[pad32(j)];
            c += hv;
            x += hv * (uint64_t)(v0 + j);
            gp[j] = PrefixEntry::of((uint32_t)c, x);
        }
    }
}

// Prefix counts and sums straight from the per-block packed rows of
// qhist_kernel<true>, in one pass and without a merged histogram.  Block
// (segment s, chunk ch of 32): the 512 words ch * 512 .. of a row hold the
// values 512 ch .. 512 ch + 511 in their low halves and the same plus 2^14 in
// their high halves, so the block owns two runs of 512 values.  Wave g takes
// the segment's rows g, g + 16, ...: four 16-byte loads a lane and row, the
// chunk's counts and the row's coarse counts and sums (a run starts on a bucket,
// so the totals before it are sums of whole buckets).  The waves' counts meet in
// LDS; then thread t scans value t of the low run (t < 512) or t - 512 of the
// high run and stores its entry, consecutive threads consecutive entries.  The
// sums are scanned relative to the wave's first value: 63 * 2^26 fits 32 bits.
// Bound by latency (a block's loads are one round trip for up to 16 rows).  On
// 16 x 1e6 samples the rows and this pass take 14.0 + 9.2 us; the zero fill,
// the merged histogram (2e6 global atomics), the chunk totals and the chunk
// scans they replaced took 4.9 + 22.1 + 6.3 + 12.3 us.
constexpr int kPreThreads = 1024;
constexpr int kPreWaves = kPreThreads / 64;
constexpr int kPreWords = kPreThreads / 2;         // packed words per chunk
constexpr int kPreChunks = kQTop / 2 / kPreWords;  // 32 per segment

__global__ __launch_bounds__(kPreThreads) void prefix_rows_kernel(const uint32_t *fine,
                                                                  const uint32_t *coarse,
                                                                  const uint32_t *csum,
                                                                  const int64_t *offsets, int S,
                                                                  int B0, const int64_t *boff,
                                                                  PrefixEntry *pre)
{
    __shared__ __attribute__((aligned(16))) uint32_t part[kPreWaves][2 * kPreWords];
    __shared__ uint32_t base_c[2][16], tot_c[16];  // before the low and the high run, by wave
    __shared__ uint64_t base_s[2][16], tot_s[16];
    static_assert(kPreWaves == 16 && kQBuckets == 4 * 64, "a row of 16 lanes per wave table");
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    for (long long u = blockIdx.x; u < (long long)S * kPreChunks; u += gridDim.x) {
        const int s = (int)(u / kPreChunks), ch = (int)(u % kPreChunks);
        const long long row0 = boff ? boff[s] : (long long)s * B0;
        const int B = boff ? (int)(boff[s + 1] - row0) : B0;
        const int parts = min(B, kPreWaves);
        if (wave < parts) {
            uint32_t lo[8] = {0, 0, 0, 0, 0, 0, 0, 0}, hi[8] = {0, 0, 0, 0, 0, 0, 0, 0};
            uint32_t bc[4] = {0, 0, 0, 0};
            uint64_t bs[4] = {0, 0, 0, 0};
            auto add = [&](const uint4 &w, int o) {
                lo[o] += w.x & 0xffffu;
                lo[o + 1] += w.y & 0xffffu;
                lo[o + 2] += w.z & 0xffffu;
                lo[o + 3] += w.w & 0xffffu;
                hi[o] += w.x >> 16;
                hi[o + 1] += w.y >> 16;
                hi[o + 2] += w.z >> 16;
                hi[o + 3] += w.w >> 16;
            };
#pragma unroll 2
            for (int r = wave; r < B; r += kPreWaves) {
                const uint4 *f = reinterpret_cast<const uint4 *>(fine + (row0 + r) * kQStride) +
                                 ch * (kPreWords / 4) + lane;
                const long long cr = (row0 + r) * (kQBuckets / 4) + lane;
                const uint4 a = f[0], b = f[64];
                const uint4 c = reinterpret_cast<const uint4 *>(coarse)[cr];
                const uint4 v = reinterpret_cast<const uint4 *>(csum)[cr];
                add(a, 0);
                add(b, 4);
                bc[0] += c.x;
                bc[1] += c.y;
                bc[2] += c.z;
                bc[3] += c.w;
                bs[0] += v.x;
                bs[1] += v.y;
                bs[2] += v.z;
                bs[3] += v.w;
            }
            uint4 *pw = reinterpret_cast<uint4 *>(part[wave]);
            pw[lane] = make_uint4(lo[0], lo[1], lo[2], lo[3]);
            pw[64 + lane] = make_uint4(lo[4], lo[5], lo[6], lo[7]);
            pw[kPreWords / 4 + lane] = make_uint4(hi[0], hi[1], hi[2], hi[3]);
            pw[kPreWords / 4 + 64 + lane] = make_uint4(hi[4], hi[5], hi[6], hi[7]);
            // lane's buckets 4 lane .. 4 lane + 3; a run starts at a multiple of 4
            // buckets: the low one after lane ch, the high one after lane 32 + ch
            const uint32_t c4 = (bc[0] + bc[1]) + (bc[2] + bc[3]);
            const uint64_t s4 = (bs[0] + bs[1]) + (bs[2] + bs[3]);
            static_assert(kPreWords == 4 * 128, "four buckets per run");
            // (the lanes are read outside the branch: every lane is active there)
            const uint32_t cs = scan_wave(c4);
            const uint64_t ss = scan_wave(s4);
            const uint32_t c_hi = lane_value(cs, 31 + ch), c_lo = lane_value(cs, max(ch, 1) - 1);
            const uint64_t s_hi = lane_value(ss, 31 + ch), s_lo = lane_value(ss, max(ch, 1) - 1);
            if (lane == 0) {
                base_c[0][wave] = ch ? c_lo : 0u;
                base_s[0][wave] = ch ? s_lo : 0ull;
                base_c[1][wave] = c_hi;
                base_s[1][wave] = s_hi;
            }
        }
        __syncthreads();
        uint32_t c = 0;
        for (int g = 0; g < parts; ++g) c += part[g][t];
        const uint32_t cs = scan_wave(c), rs = scan_wave(c * (uint32_t)lane);
        const int run = wave >> 3;
        const int v = ch * kPreWords + (t & (kPreWords - 1)) + run * (kQTop / 2);
        if (lane == 63) {
            tot_c[wave] = cs;
            tot_s[wave] = (uint64_t)cs * (uint32_t)(v - 63) + rs;
        }
        __syncthreads();
        // before this wave: the totals before its run and those of the run's waves before it
        uint32_t bc = 0;
        uint64_t bs = 0;
        if (lane < parts) {
            bc = base_c[run][lane];
            bs = base_s[run][lane];
        }
        if (lane < (wave & 7)) {
            bc += tot_c[run * 8 + lane];
            bs += tot_s[run * 8 + lane];
        }
        bc = lane_value(scan_row16(bc), 15) + cs;
        bs = lane_value(scan_row16(bs), 15) + (uint64_t)cs * (uint32_t)(v - lane) + rs;
        PrefixEntry *o = pre + (long long)s * kHistBins;
        o[v] = PrefixEntry::of(bc, bs);
        if (v == kQTop - 1) {  // the value 2^15 (one thread of the last chunk)
            const uint64_t N = (uint64_t)(offsets[s + 1] - offsets[s]);
            o[kQTop] = PrefixEntry::of((uint32_t)N, bs + (N - bc) * (uint64_t)kQTop);
        }
        __syncthreads();  // the next chunk reuses the LDS
    }
}

hipError_t launch_counts(const int64_t *offsets, const int32_t *xi, int S, const CountBufs &b,
                         hipStream_t st)
{
    if (!b.hist) {
        hipLaunchKernelGGL(qhist_kernel<true>, dim3((unsigned)std::min(b.plan.rows, kMaxGridBlocks)),
                           dim3(kQThreads), 2 * kQStride * sizeof(uint32_t), st, offsets, xi, S, b.plan.B,
                           b.plan.boff, b.plan.rows, b.fine, b.coarse, b.csum);
        HIPRET(hipGetLastError());
        const long long units = (long long)S * kPreChunks;
        hipLaunchKernelGGL(prefix_rows_kernel, dim3((unsigned)std::min(units, kMaxGridBlocks)),
                           dim3(kPreThreads), 0, st, (const uint32_t *)b.fine,
                           (const uint32_t *)b.coarse, (const uint32_t *)b.csum, offsets, S, b.plan.B,
                           b.plan.boff, b.pre);
        return hipGetLastError();
    }
    HIPRET(launch_histogram(offsets, xi, S, b.plan.B, b.hist, st));
    // chunk totals first, then each chunk's scan starts from the totals of the
    // chunks before it
    const long long blocks = (long long)S * kPrefixChunks;
    hipLaunchKernelGGL(chunk_total_kernel, dim3((unsigned)blocks), dim3(kPrefixThreads), 0, st,
                       (const uint32_t *)b.hist, b.tot);
    hipLaunchKernelGGL(prefix_kernel, dim3((unsigned)blocks), dim3(kPrefixThreads), 0, st,
                       (const uint32_t *)b.hist, (const uint64_t *)b.tot, b.pre);
    return hipGetLastError();
}

// One (class, grid point) of the exact table.  For 0 <= x, eta <= L the three
// candidates of Step 4 reduce to the larger of two lines, B - a1 x and
// C - a2 (L - x) with B = c_w eta, C = c_p (L - eta), a1 = min(g, c_w),
// a2 = min(g, c_p); the first is the larger up to t = floor((B - C + a2 L) /
// (a1 + a2)).  All integers in units of 2^-33.
struct TableRow {
    const PrefixEntry *pre;  // of the class's segment
    int64_t B, C, CP, CW;
    uint64_t SX;             // sum of the samples
    uint32_t N;
    int L, tmax;
    double Nd, rN;           // N and RN(1 / N)
};

// What a row needs of one multiplier, the same for every grid point of a class.
struct __attribute__((aligned(16))) TableLam {
    int64_t A2L, A12;  // a2 L and a1 + a2
    double rcp;        // an estimate of 1 / (a1 + a2)
    int64_t A2;
};

__device__ __forceinline__ TableLam table_lam(int64_t G, int64_t CP, int64_t CW, int L)
{
    const int64_t A1 = G < CW ? G : CW, A2 = G < CP ? G : CP;
    return TableLam{A2 * L, A1 + A2, __builtin_amdgcn_rcp((double)(A1 + A2)), A2};
}

// the prefix entry at t
__device__ __forceinline__ PrefixEntry row_split(const TableRow &r, const TableLam &g)
{
    const int t = floor_div_clamped(r.B - r.C + g.A2L, g.A12, g.rcp, -1, r.tmax);
    const PrefixEntry e = r.pre[max(t, 0)];
    return t >= 0 ? e : PrefixEntry::of(0u, 0ull);
}

// RN(RN(S) / N) at a multiplier: with cnt and sum over the samples <= t,
//   S = B cnt - a1 sum + (C - a2 L)(N - cnt) + a2 (sum_all - sum),
// every term an exact integer (the sum is non-negative, as phi is).
__device__ __forceinline__ double row_mean(const TableRow &r, const TableLam &g,
                                           const PrefixEntry &e)
{
    const __int128 S = mul_i64_u31(r.B, e.cnt) + mul_i64_u31(r.C - g.A2L, r.N - e.cnt) +
                       mul_u43((uint64_t)g.A2, r.SX) - mul_u43((uint64_t)g.A12, e.sum());
    return div_by(fix128_to_double((uint64_t)S, (uint64_t)((unsigned __int128)S >> 64)), r.Nd, r.rN);
}

// The slopes of the active lines of S at a multiplier: less RN(eps N), it is N
// times a subgradient of gamma -> gamma eps + S(gamma) / N, with the sign changed;
// an exact integer below 2^42 (a sample where the lines meet may take either
// line's slope), not increasing in the multiplier.
__device__ __forceinline__ double row_lines(const TableRow &r, bool below_cw, bool below_cp,
                                            const PrefixEntry &e)
{
    const int64_t below = below_cw ? (int64_t)e.sum() : 0;
    const int64_t above = below_cp ? (int64_t)(r.N - e.cnt) * r.L - (int64_t)(r.SX - e.sum()) : 0;
    return (double)(below + above);
}

// One thread per (c, k), for `per` radii: W = min over m of J_m = RN(RN(lam_m eps) +
// RN(RN(S_m) / N)) and the lowest m attaining it, without evaluating every m.
// J without its roundings, j(gamma) = gamma eps + S(gamma) / N, is convex (Step 4
// is a supremum of lines in gamma), so a binary search on the sign of its
// subgradient at the grid's multipliers finds the first m = b where it is not
// negative; the smallest j on the grid is at b or at a = b - 1.  J_a and J_b are
// evaluated exactly.  Any other m is ruled out by convexity: left of a, j is at
// least j_a + |slope_a| (lam_a - lam_(a-1)), right of b at least j_b + slope_b
// (lam_(b+1) - lam_b); three roundings move J by less than 4 * 2^-53 of j, so a
// rise above 2^-44 of J settles it (and the slope itself must exceed its own
// rounding, 2^-50 eps N).  At eps = 0 the slope right of b is exactly zero and S
// the same integer, so J ties and b is the lower index.  Where the rise is too
// small the neighbours are evaluated, one after the other, until it is not: the
// same W and the same lowest m as a scan over all m.
// About 9 subgradients and 2 values of S instead of M values.  A block holds one
// class: what depends on class and multiplier (the fixed-point slopes, a2 L, the
// reciprocal of the division) is staged in LDS once, the prefix entry met by a
// subgradient serves the value there, and the next radius starts from the bracket
// of the one before (its two subgradients less their own eps N) in doubling steps.
// Bound by the search's chain of dependent loads and instructions and, with many
// rows, by the gathers of prefix entries (64 lines a wave) and the 64-bit integer
// arithmetic: 128 classes x 1024 points x 16 radii (M = 128) 45 us, 73 with one
// radius a block, 82 with a thread per (e, c, k) and nothing staged; 16 x 2048
// points of 1e6 samples (M = 256, one radius) 10 us, as before.
// kStaged: M <= kTableLam; beyond, those terms are computed where they are used.
// A grid of multipliers that is not ascending (outside the contract) is scanned.
constexpr int kTableThreads = 128;
constexpr int kTableLam = 1024;  // multipliers staged per block (36 KB)
// a block takes as many radii as leave this many blocks (16 radii on 1,024 blocks'
// worth of rows: 69 us with 1,024, 53 with 2,048, 52 with 4,096, 55 with 8,192)
constexpr int kTableBlocks = 4096;

template <bool kStaged>
__global__ __launch_bounds__(kTableThreads) void exact_table_kernel(
    const int64_t *offsets, const int32_t *seg, const int32_t *L_, const int32_t *eta_,
    const float *lam, const float *c_p, const float *c_w, const float *eps,
    const PrefixEntry *pre, long long units, int per, int E, int C, int K, int M, double *W,
    int32_t *m_star)
{
    extern __shared__ __attribute__((aligned(16))) char table_lds[];
    TableLam *const s_tab = reinterpret_cast<TableLam *>(table_lds);
    float *const s_lam = reinterpret_cast<float *>(s_tab + (kStaged ? M : 0));
    __shared__ int s_mw, s_mp;  // the multipliers below c_w and below c_p
    const int t = threadIdx.x, chunks = (K + kTableThreads - 1) / kTableThreads;
    for (long long unit = blockIdx.x; unit < units; unit += gridDim.x) {
        const long long rest = unit / chunks;
        const int k = (int)(unit - rest * chunks) * kTableThreads + t;
        const int eg = (int)(rest / C), c = (int)(rest - (long long)eg * C);
        const int s = seg_of_x(seg, c);
        TableRow r;
        r.pre = pre + (long long)s * kHistBins;
        r.SX = r.pre[kHistBins - 1].sum();
        r.N = (uint32_t)(offsets[s + 1] - offsets[s]);
        r.L = L_[c];
        r.tmax = min(r.L, kHistBins - 1);
        r.CP = fix33(c_p[c]);
        r.CW = fix33(c_w[c]);
        r.Nd = (double)r.N;
        r.rN = __ddiv_rn(1.0, r.Nd);
        if (t == 0) s_mw = s_mp = 0;
        __syncthreads();
        bool up = true;
        for (int m = t; m < M; m += kTableThreads) {
            const float l = lam[m], next = m + 1 < M ? lam[m + 1] : INFINITY;
            if (!(l < next)) up = false;
            const int64_t G = fix33(l);
            if (kStaged) {
                s_lam[m] = l;
                s_tab[m] = table_lam(G, r.CP, r.CW, r.L);
            }
            const int64_t G1 = m + 1 < M ? fix33(next) : INT64_MAX;
            if (G < r.CW && G1 >= r.CW) s_mw = m + 1;
            if (G < r.CP && G1 >= r.CP) s_mp = m + 1;
        }
        const bool ascending = __syncthreads_and(up);
        const int mw = s_mw, mp = s_mp;
        __syncthreads();  // (the next unit sets them again)
        if (k < K) {
            const int64_t eta = eta_[k];
            r.B = r.CW * eta;
            r.C = r.CP * (r.L - eta);
            auto lam_at = [&](int m) { return kStaged ? s_lam[m] : lam[m]; };
            auto tab_at = [&](int m) {
                return kStaged ? s_tab[m] : table_lam(fix33(lam[m]), r.CP, r.CW, r.L);
            };
            auto lines = [&](int m, const PrefixEntry &p) { return row_lines(r, m < mw, m < mp, p); };
            int a = -1, b = M;  // the slope is negative at a, not at b
            double da = 0.0, db = 0.0, qa = 0.0, qb = 0.0;  // their lines and means
            PrefixEntry pa{}, pb{};
            int step = 1;
            const int e1 = (int)min((long long)(eg + 1) * per, (long long)E);
            for (int e = eg * per; e < e1; ++e) {
                const long long ec = (long long)e * C + c;
                const double ev = (double)eps[ec], eN = __dmul_rn(ev, r.Nd);
                auto J_of = [&](int m, double q) {
                    return __dadd_rn(__dmul_rn((double)lam_at(m), ev), q);
                };
                // m and all beyond it are settled: the rise over the gap to the next
                // multiplier, of slope h at a point of value J
                auto clear = [&](double h, double J, int m0) {
                    const double gap = (double)lam_at(m0 + 1) - (double)lam_at(m0);
                    return h * gap > r.Nd * fabs(J) * 0x1p-44 && h > fabs(eN) * 0x1p-50;
                };
                double best = __builtin_inf();
                int bm = M;
                if (ascending) {
                    bool na = false, nb = false;
                    const int a0 = a;
                    int dir = 0;
                    if (a >= 0 && !(eN - da < 0.0)) {
                        b = a;
                        db = da;
                        qb = qa;
                        a = -1;
                        dir = -1;
                    } else if (b < M && eN - db < 0.0) {
                        a = b;
                        da = db;
                        qa = qb;
                        b = M;
                        dir = 1;
                    }
                    while (b - a > 1) {
                        const int mid = dir == 0 ? (a + b) >> 1
                                                 : (dir < 0 ? max(b - step, a + 1) : min(a + step, b - 1));
                        const PrefixEntry p = row_split(r, tab_at(mid));
                        const double d = lines(mid, p);
                        if (eN - d < 0.0) {
                            a = mid;
                            da = d;
                            pa = p;
                            na = true;
                            if (dir < 0) dir = 0;
                            else step *= 2;
                        } else {
                            b = mid;
                            db = d;
                            pb = p;
                            nb = true;
                            if (dir > 0) dir = 0;
                            else step *= 2;
                        }
                    }
                    step = max(abs(a - a0), 1);
                    double Ja = 0.0, Jb = 0.0;
                    if (b < M) {
                        if (nb) qb = row_mean(r, tab_at(b), pb);
                        Jb = J_of(b, qb);
                        if (Jb < best) {
                            best = Jb;
                            bm = b;
                        }
                    }
                    if (a >= 0) {
                        if (na) qa = row_mean(r, tab_at(a), pa);
                        Ja = J_of(a, qa);
                        if (Ja <= best) {
                            best = Ja;
                            bm = a;
                        }
                    }
                    double h = eN - da;
                    for (int m = a; m > 0 && !clear(-h, Ja, m - 1);) {
                        const PrefixEntry p = row_split(r, tab_at(--m));
                        h = eN - lines(m, p);
                        Ja = J_of(m, row_mean(r, tab_at(m), p));
                        if (Ja <= best) {
                            best = Ja;
                            bm = m;
                        }
                    }
                    h = eN - db;
                    for (int m = b; m < M - 1 && ev != 0.0 && !clear(h, Jb, m);) {
                        const PrefixEntry p = row_split(r, tab_at(++m));
                        h = eN - lines(m, p);
                        Jb = J_of(m, row_mean(r, tab_at(m), p));
                        if (Jb < best) {
                            best = Jb;
                            bm = m;
                        }
                    }
                } else {
                    for (int m = 0; m < M; ++m) {
                        const TableLam g = tab_at(m);
                        const double J = J_of(m, row_mean(r, g, row_split(r, g)));
                        if (J < best) {
                            best = J;
                            bm = m;
                        }
                    }
                }
                W[ec * K + k] = best;
                m_star[ec * K + k] = min(bm, M - 1);  // (no J below infinity: the last)
            }
        }
        __syncthreads();  // the next unit reuses the LDS
    }
}

// Block per (e, c): lowest k <= kmax with the smallest W, and the values there
// (the exact optimum over a W table whose entries are exact-spec values; kmax where
// no entry is below infinity).  Bound
// by latency: each thread loads four values at a time, then 32-bit minima within the
// waves and one pass over their results (8,193 points of 42 rows: 5.6 us, 7.9 with
// fp64 shuffles).
constexpr int kArgThreads = 256;

__device__ void table_argmin_row(const double *W, const int32_t *m_star, const int32_t *k_max,
                                int C, int K, int ec, int32_t *k_star, double *W_star,
                                int32_t *m_at_star)
{
    const int c = ec % C, t = threadIdx.x;
    int kmax = K - 1;
    if (k_max) {
        kmax = k_max[c];
        kmax = kmax < 0 ? 0 : (kmax > K - 1 ? K - 1 : kmax);
    }
    const double *w = W + (long long)ec * K;
    double bw = __builtin_inf();
    int bk = 0x7fffffff;
    for (int k0 = t; k0 <= kmax; k0 += 4 * kArgThreads) {
        double v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = w[min(k0 + q * kArgThreads, kmax)];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int k = k0 + q * kArgThreads;
            if (k <= kmax && v[q] < bw) {
                bw = v[q];
                bk = k;
            }
        }
    }
    const KeyIdx least = wave_min_key(bw, bk, 0);
    bw = least.key;
    bk = least.idx;
    __shared__ double sw[kArgThreads / 64];
    __shared__ int sk[kArgThreads / 64];
    if ((t & 63) == 0) {
        sw[t >> 6] = bw;
        sk[t >> 6] = bk;
    }
    __syncthreads();
    if (t == 0) {
        for (int i = 1; i < kArgThreads / 64; ++i)
            if (sw[i] < bw || (sw[i] == bw && sk[i] < bk)) {
                bw = sw[i];
                bk = sk[i];
            }
        bk = min(bk, kmax);  // no W below infinity: the last point
        k_star[ec] = bk;
        W_star[ec] = bw;
        if (m_at_star) m_at_star[ec] = m_star[(long long)ec * K + bk];
    }
}

// rows (e, c) in a block-uniform loop; the barrier lets the next row reuse the LDS
__global__ __launch_bounds__(kArgThreads) void table_argmin_kernel(
    const double *W, const int32_t *m_star, const int32_t *k_max, int C, int K, int rows,
    int32_t *k_star, double *W_star, int32_t *m_at_star)
{
    // (rows reaches 2^31 - 1: the last step would pass the 32-bit range)
    for (long long ec = blockIdx.x; ec < rows; ec += gridDim.x) {
        table_argmin_row(W, m_star, k_max, C, K, (int)ec, k_star, W_star, m_at_star);
        __syncthreads();
    }
}

hipError_t launch_table_argmin(const double *W, const int32_t *m_star, const int32_t *k_max,
                               int E, int C, int K, int32_t *k_star, double *W_star,
                               int32_t *m_at_star, hipStream_t st)
{
    const long long rows = (long long)E * C;  // below 2^31: checked by the entry points
    hipLaunchKernelGGL(table_argmin_kernel, dim3((unsigned)std::min(rows, kMaxGridBlocks)),
                       dim3(kArgThreads), 0, st, W, m_star, k_max, C, K, (int)rows, k_star, W_star, m_at_star);
    return hipGetLastError();
}

hipError_t launch_exact_table(const int64_t *offsets, const int32_t *seg, const int32_t *L,
                              const int32_t *eta, const float *lam, const float *c_p,
                              const float *c_w, const float *eps, const int32_t *k_max,
                              const PrefixEntry *pre, int E, int C, int K, int M, double *W,
                              int32_t *m_star, int32_t *k_star, double *W_star, int32_t *m_at_star,
                              hipStream_t st)
{
    // radii per block: blocks enough to fill the chip come first
    const long long groups = (long long)C * ((K + kTableThreads - 1) / kTableThreads);
    const int per = (int)std::min<long long>(E, std::max(1LL, groups * E / kTableBlocks));
    const long long units = groups * (((long long)E + per - 1) / per);
    const bool staged = M <= kTableLam;
    hipLaunchKernelGGL(staged ? exact_table_kernel<true> : exact_table_kernel<false>,
                       dim3((unsigned)std::min(units, kMaxGridBlocks)), dim3(kTableThreads),
                       staged ? (size_t)M * (sizeof(TableLam) + sizeof(float)) : 0, st, offsets, seg, L,
                       eta, lam, c_p, c_w, eps, pre, units, per, E, C, K, M, W, m_star);
    HIPRET(hipGetLastError());
    if (k_star) HIPRET(launch_table_argmin(W, m_star, k_max, E, C, K, k_star, W_star, m_at_star, st));
    return hipGetLastError();
}

}  // namespace dro

namespace dro {

// ================================================== baseline reservations ====
// The moment-based and block-aligned baselines of the policy comparison
// (Sec. 5.1: the mean and the block-aligned P95; Sec. 5.4: mean + k sigma), one
// thread per class, exactly in integers:
//   mean_r        = ceil(s / n)
//   lp_r[i]       = min(L, the least integer r with r n - s >= k_i sqrt(n ss - s^2)),
//                   i.e. ceil((s + ceil(sqrt(k_i^2 (n ss - s^2)))) / n)
//   block_r       = q rounded up to a multiple of `block`
// with n, s, ss the count, sum and sum of squares of the class samples.

// ceil(sqrt(d)) for d < 2^100: a double estimate corrected with exact products
__device__ uint64_t ceil_sqrt_u128(unsigned __int128 d)
{
    uint64_t r = (uint64_t)sqrt((double)d);
    while (r > 0 && (unsigned __int128)r * r > d) --r;
    while ((unsigned __int128)(r + 1) * (r + 1) <= d) ++r;
    return r + ((unsigned __int128)r * r < d ? 1u : 0u);
}

__device__ __forceinline__ int64_t ceil_div_pos(__int128 a, int64_t b)
{
    return (int64_t)((a + b - 1) / b);  // a >= 0, b >= 1
}

__global__ void baseline_kernel(int C, const int64_t *count, const int64_t *sum,
                                const int64_t *sumsq, const int32_t *L, BaselineKs ks,
                                const int32_t *q, int block, int32_t *mean_r, int32_t *lp_r,
                                int32_t *block_r)
{
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= C) return;
    const int64_t n = count[c] > 0 ? count[c] : 1, s = sum[c], ss = sumsq[c];
    mean_r[c] = (int32_t)ceil_div_pos(s, n);
    const __int128 v = (__int128)n * ss - (__int128)s * s;  // n^2 times the population variance
    const unsigned __int128 var = v > 0 ? (unsigned __int128)v : 0;
    for (int i = 0; i < ks.n; ++i) {
        const uint64_t k = (uint64_t)ks.k[i];
        const uint64_t r = ceil_sqrt_u128(var * (k * k));
        const int64_t lp = ceil_div_pos((__int128)s + r, n);
        lp_r[(long long)i * C + c] = (int32_t)(lp < L[c] ? lp : L[c]);
    }
    if (q && block_r) {
        const int64_t v0 = q[c] > 0 ? q[c] : 0;
        block_r[c] = (int32_t)(((v0 + block - 1) / block) * block);
    }
}

hipError_t launch_baselines(int C, const int64_t *count, const int64_t *sum, const int64_t *sumsq,
                            const int32_t *L, const BaselineKs &ks, const int32_t *q, int block,
                            int32_t *mean_r, int32_t *lp_r, int32_t *block_r, hipStream_t st)
{
    hipLaunchKernelGGL(baseline_kernel, dim3((C + 255) / 256), dim3(256), 0, st, C, count, sum,
                       sumsq, L, ks, q, block, mean_r, lp_r, block_r);
    return hipGetLastError();
}

// ====================================================== continuous dual ====
// W(eta) = min over gamma >= 0 of gamma eps + S(gamma) / N, the Kantorovich
// dual (Appendix A, Step 3) with gamma continuous (= the LP of Step 5 by
// strong duality).  With a1 = min(g, c_w), a2 = min(g, c_p) the per-sample sup
// is max(B - a1 x, C - a2 (L - x)): convex and piecewise linear in g, so J is
// too, and its right derivative at any g follows from the value counts:
//   dS/dg = -[g < c_w] sum_{x < x0} x - [g < c_p] sum_{x > x0} (L - x)
//           + (#{x = x0}) max(-[g < c_w] x0, -[g < c_p] (L - x0)).
// Bisection on [0, max(c_p, c_w)] (where J' = eps >= 0) finds the smallest g
// with J'(g+) >= 0, i.e. the smallest minimiser; J is evaluated there in fp64.

struct DualRow {
    const PrefixEntry *pre;
    double N, rN, SX;  // count, RN(1 / N), sum
    int tmax;
    double B, C, L, cw, cp, ev;
};

// Where a multiplier splits the samples: x0, its floor t (clamped to [-2, L + 2])
// and whether x0 is a sample value, t.
struct DualSplit {
    double a1, a2, tf;
    int t;
    bool tie;
};

__device__ __forceinline__ DualSplit dual_split(const DualRow &r, double g)
{
    DualSplit d;
    d.a1 = g < r.cw ? g : r.cw;
    d.a2 = g < r.cp ? g : r.cp;
    const double s12 = d.a1 + d.a2;
    const double q = (r.B - r.C + d.a2 * r.L) / (s12 > 0.0 ? s12 : 1.0);
    const double x0 = s12 > 0.0 ? q : (r.B >= r.C ? 1e300 : -1e300);
    d.tf = floor(x0 < -2.0 ? -2.0 : (x0 > r.L + 2.0 ? r.L + 2.0 : x0));
    d.t = (int)d.tf;
    d.tie = d.tf == x0 && d.t >= 0 && d.t <= r.tmax;
    return d;
}

// count and sum of the samples x <= t, and of those below t (both loads in flight)
struct DualCounts {
    double n1, s1, n0, s0;
};

__device__ __forceinline__ DualCounts dual_counts(const DualRow &r, int t)
{
    const PrefixEntry *p = r.pre + min(max(t, 0), r.tmax);
    const PrefixEntry *p0 = r.pre + min(max(t - 1, 0), r.tmax);
    const PrefixEntry e = *p, e0 = *p0;
    const bool in = t >= 0, in0 = t >= 1;
    return DualCounts{in ? (double)e.cnt : 0.0, in ? (double)e.sum() : 0.0,
                      in0 ? (double)e0.cnt : 0.0, in0 ? (double)e0.sum() : 0.0};
}

// J(g): line 1 for x <= t, line 2 above (equal at a tie, so ties do not matter)
__device__ __forceinline__ double dual_value(const DualRow &r, const DualSplit &d,
                                             const DualCounts &k, double g)
{
    const double S = r.B * k.n1 - d.a1 * k.s1 + (r.C - d.a2 * r.L) * (r.N - k.n1) +
                     d.a2 * (r.SX - k.s1);
    return g * r.ev + S / r.N;
}

// the right derivative J'(g+): ties exactly at x0 take the larger slope
__device__ __forceinline__ double dual_slope(const DualRow &r, const DualSplit &d,
                                             const DualCounts &k, double g)
{
    const double nt = d.tie ? k.n1 - k.n0 : 0.0, xt = d.tie ? (double)d.t : 0.0;
    const double n1 = d.tie ? k.n0 : k.n1, s1 = d.tie ? k.s0 : k.s1;
    const double w1 = g < r.cw ? 1.0 : 0.0, w2 = g < r.cp ? 1.0 : 0.0;
    const double n2 = r.N - n1 - nt, s2 = r.SX - s1 - nt * xt;
    const double d1 = -w1 * xt, d2 = -w2 * (r.L - xt);
    double dS = -w1 * s1 - w2 * (r.L * n2 - s2);
    dS = nt > 0.0 ? dS + nt * (d1 > d2 ? d1 : d2) : dS;
    return r.ev + div_by(dS, r.N, r.rN);
}

// The bisection is a chain of some 55 halvings, each a division, a lookup and a
// dozen dependent fp64 operations, and a table of a few ten thousand rows leaves
// most of the chip idle.  So kLanes = 4 lanes share a row and take two halvings a
// step: three of them evaluate the middle and the middles of both halves, a ballot
// tells which two count, and the brackets are those of one halving after the other.
// Once the bracket's ends lie at the same or neighbouring t, the sign of J' is known
// for every (t, tie, g >= the smaller cost) inside and only the split is computed.
// 32,768 rows of 1e6 samples 27 us, 36 before (a lane a row, two lookups and two
// divisions a halving); 1,048,576 rows of 1e4 samples, with the counts, 236 us, 385
// before.
// The line: four lanes a row up to two waves a SIMD (32,768 rows: 44 us with the
// counts against 49; 65,536 rows: 64 against 57).
constexpr long long kDualFew = 1 << 15;

template <int kLanes>
__global__ __launch_bounds__(256) void continuous_dual_kernel(
    const int64_t *offsets, const int32_t *seg, const int32_t *L_, const int32_t *eta_,
    const float *c_p, const float *c_w, const float *eps, const PrefixEntry *pre, int E, int C,
    int K, double *W, double *gamma)
{
    const long long n = (long long)E * C * K;
    const int lane = threadIdx.x & 63, sub = lane & (kLanes - 1), base = lane - sub;
    // (a group's lanes leave together; a ballot reads its own lanes' bits only)
    for (long long i = ((long long)blockIdx.x * blockDim.x + threadIdx.x) / kLanes; i < n;
         i += (long long)gridDim.x * blockDim.x / kLanes) {
        const int ec = n <= 0x7fffffffLL ? (int)((uint32_t)i / (uint32_t)K) : (int)(i / K);
        const int k = (int)(i - (long long)ec * K), c = ec % C;
        const int s = seg_of_x(seg, c);
        DualRow r;
        r.pre = pre + (long long)s * kHistBins;
        r.N = (double)(offsets[s + 1] - offsets[s]);
        r.rN = 1.0 / r.N;
        r.SX = (double)r.pre[kHistBins - 1].sum();
        const int Li = L_[c];
        r.tmax = min(max(Li, 0), kHistBins - 1);  // (L is not checked: stays inside the entries)
        const double eta = (double)eta_[k];
        r.L = (double)Li;
        r.cw = (double)c_w[c];
        r.cp = (double)c_p[c];
        r.B = r.cw * eta;
        r.C = r.cp * (r.L - eta);
        r.ev = (double)eps[ec];
        const double kink = r.cw < r.cp ? r.cw : r.cp;
        double lo = 0.0, hi = r.cw > r.cp ? r.cw : r.cp, at = 0.0;
        const DualSplit d0 = dual_split(r, 0.0);
        if (!(dual_slope(r, d0, dual_counts(r, d0.t), 0.0) >= 0.0)) {
            int tlo = d0.t, thi = dual_split(r, hi).t;
            // `known`: the sign of J' where t is near or near + 1, by (t, tie, g >= kink)
            int near = -9;
            uint32_t known = 0;
            // J'(g+) >= 0 and t at g, 0 < g < max(c_p, c_w)
            auto rises = [&](double g, int &t) {
                const DualSplit d = dual_split(r, g);
                const int state = 2 * (d.t - near) + (d.tie ? 0 : 1);
                t = d.t;
                bool up = (known >> ((state + (g < kink ? 0 : 4)) & 7)) & 1;
                if ((uint32_t)state >= 4u) up = dual_slope(r, d, dual_counts(r, d.t), g) >= 0.0;
                return up;
            };
            for (int it = 0; it < 200;) {
                const double mid = 0.5 * (lo + hi);
                if (mid <= lo || mid >= hi) break;
                const int low = min(tlo, thi), high = max(tlo, thi);
                if (high - low <= 1 && (low < near || high > near + 1)) {
                    near = low;
                    known = 0;
                    for (int q = 0; q < 2; ++q) {
                        const DualCounts k2 = dual_counts(r, low + q);
                        DualSplit d{};
                        d.t = low + q;
                        for (int tie = 0; tie < 2; ++tie) {
                            d.tie = tie;
                            const int bit = 2 * q + 1 - tie;
                            if (dual_slope(r, d, k2, lo) >= 0.0) known |= 1u << bit;
                            if (dual_slope(r, d, k2, kink) >= 0.0) known |= 16u << bit;
                        }
                    }
                }
                bool up, up2 = false;
                int t, t2 = 0;
                double m2 = 0.0;
                if (kLanes == 1) {
                    up = rises(mid, t);
                } else {
                    const double ml = 0.5 * (lo + mid), mh = 0.5 * (mid + hi);
                    const bool u = rises(sub == 1 ? ml : (sub == 2 ? mh : mid), t);
                    const uint32_t bits = (uint32_t)(__ballot(u) >> base);
                    up = bits & 1;
                    m2 = up ? ml : mh;
                    up2 = (up ? bits >> 1 : bits >> 2) & 1;
                    const int t1 = quad_lane<1>(t), t3 = quad_lane<2>(t);
                    t2 = up ? t1 : t3;
                    t = quad_lane<0>(t);
                }
                ++it;
                hi = up ? mid : hi;
                thi = up ? t : thi;
                lo = up ? lo : mid;
                tlo = up ? tlo : t;
                if (kLanes > 1) {
                    if (it >= 200 || m2 <= lo || m2 >= hi) break;
                    ++it;
                    hi = up2 ? m2 : hi;
                    thi = up2 ? t2 : thi;
                    lo = up2 ? lo : m2;
                    tlo = up2 ? tlo : t2;
                }
            }
            at = hi;
        }
        if (sub == 0) {
            const DualSplit d = dual_split(r, at);
            W[i] = dual_value(r, d, dual_counts(r, d.t), at);
            gamma[i] = at;
        }
    }
}

hipError_t launch_continuous_dual(const int64_t *offsets, const int32_t *seg, const int32_t *L,
                                  const int32_t *eta, const float *c_p, const float *c_w,
                                  const float *eps, const PrefixEntry *pre, int E, int C, int K,
                                  double *W, double *gamma, hipStream_t st)
{
    const long long n = (long long)E * C * K;
    const bool few = n <= kDualFew;
    const long long blocks = ((few ? 4 : 1) * n + 255) / 256;
    hipLaunchKernelGGL(few ? continuous_dual_kernel<4> : continuous_dual_kernel<1>,
                       dim3((unsigned)std::min(blocks, kMaxGridBlocks)), dim3(256), 0, st, offsets,
                       seg, L, eta, c_p, c_w, eps, pre, E, C, K, W, gamma);
    return hipGetLastError();
}

}  // namespace dro

namespace dro {

// ===================================================== reservation cost ====
// The stochastic cost of Sec. 3.3, Q(eta, x) = c_p (x - eta)^+ + c_w (eta - x)^+,
// averaged over a class's samples for any given reservations, and the class
// moments from which mean- and spread-based reservations are formed.  With
// cnt(v) = #{x <= v} and sum(v) the sum of those samples, for an integer eta
//   sum_n Q(eta, x_n) = c_p ((SX - sum(eta)) - eta (N - cnt(eta)))
//                     + c_w (eta cnt(eta) - sum(eta)),
// evaluated in 128-bit integers in units of 2^-33: exact for every eta.

// Block for row r (segment s, part b, as the quantile's rows): the sum of its
// samples, the same sum, the sum of squares and the largest with every sample
// clamped to the histogram's values 0 .. 2^15 (equal for validated samples).
// One wave a row where no row is longer than kMomShort samples, else four: bcd_init_state
// on 8,000 segments of 100 samples 35 us and 46 (128 with 16 waves a row), on 500 of
// 16,000 32 and 28, on one of 400,000 30 and 26.
constexpr long long kMomShort = 4096;

// The wave's totals (every lane active; the largest lies in [0, 2^15]).
__device__ __forceinline__ RowMoments wave_moments(const RowMoments &m)
{
    return RowMoments{(long long)lane_value(scan_wave((uint64_t)m.raw), 63),
                      (long long)lane_value(scan_wave((uint64_t)m.sum), 63),
                      lane_value(scan_wave((uint64_t)m.sq), 63),
                      (long long)~wave_min(~(uint32_t)m.mx)};
}

template <int kMomThreads>
__global__ __launch_bounds__(kMomThreads) void row_moments_kernel(const int64_t *offsets,
                                                                  const int32_t *xi, int S, int B,
                                                                  const int64_t *boff,
                                                                  long long rows, RowMoments *out)
{
    __shared__ RowMoments red[kMomThreads / 64];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    for (long long r = blockIdx.x; r < rows; r += gridDim.x) {
        const RowPart rp = row_part(offsets, S, B, boff, r);
        RowMoments m{0, 0, 0, 0};
        for_each_sample<kMomThreads>(
            xi, rp.lo, rp.hi,
            [&](int x) {
                m.raw += x;
                const int v = x < 0 ? 0 : (x > kHistBins - 1 ? kHistBins - 1 : x);
                m.sum += v;
                m.sq += (unsigned long long)((uint32_t)v * (uint32_t)v);
                m.mx = v > m.mx ? v : m.mx;
            },
            [] {});
        m = wave_moments(m);
        if (lane == 0) red[wave] = m;
        __syncthreads();
        if (t == 0) {
            for (int w = 1; w < kMomThreads / 64; ++w) {
                m.raw += red[w].raw;
                m.sum += red[w].sum;
                m.sq += red[w].sq;
                m.mx = red[w].mx > m.mx ? red[w].mx : m.mx;
            }
            out[r] = m;
        }
        __syncthreads();  // the next row reuses red
    }
}

// One wave per class: the rows of its segment combined.  count .. xmax are
// written when count is given; k0, the largest k with eta[k] N <= the sum of
// the samples (0 if none), when eta is.
constexpr int kMomWaves = 4;  // classes per block

__global__ __launch_bounds__(64 * kMomWaves) void class_moments_kernel(
    const int64_t *offsets, const int32_t *seg, const RowMoments *rows, int B0,
    const int64_t *boff, int C, int64_t *count, int64_t *sum, int64_t *sumsq, int32_t *xmax,
    const int32_t *eta, int K, int32_t *k0)
{
    const int lane = threadIdx.x & 63;
    // classes in a loop of whole waves (no block barrier)
    for (long long c = (long long)blockIdx.x * kMomWaves + (threadIdx.x >> 6); c < C;
         c += (long long)gridDim.x * kMomWaves) {
        const int s = seg_of_x(seg, (int)c);
        const long long row0 = boff ? boff[s] : (long long)s * B0;
        const int B = boff ? (int)(boff[s + 1] - row0) : B0;
        RowMoments m{0, 0, 0, 0};
        for (int r = lane; r < B; r += 64) {
            const RowMoments x = rows[row0 + r];
            m.raw += x.raw;
            m.sum += x.sum;
            m.sq += x.sq;
            m.mx = x.mx > m.mx ? x.mx : m.mx;
        }
        m = wave_moments(m);
        if (lane != 0) continue;
        const long long N = offsets[s + 1] - offsets[s];
        if (count) {
            count[c] = N;
            sum[c] = m.sum;
            sumsq[c] = (int64_t)m.sq;
            xmax[c] = (int32_t)m.mx;
        }
        if (eta) {
            int lo = 0, hi = K - 1;  // eta ascending
            while (lo < hi) {
                const int mid = (lo + hi + 1) / 2;
                if ((long long)eta[mid] * N <= m.raw) lo = mid;
                else hi = mid - 1;
            }
            k0[c] = lo;
        }
    }
}

// Thread per (row r, class c): cost = RN(RN(S) / N) and cover = cnt(eta).
__global__ __launch_bounds__(256) void reservation_cost_kernel(
    const int64_t *offsets, const int32_t *seg, const float *c_p, const float *c_w,
    const PrefixEntry *pre, int C, long long RC, const int32_t *eta_r, double *cost, int64_t *cover)
{
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= RC) return;
    const int c = (int)(i % C);
    const int s = seg_of_x(seg, c);
    const int64_t N = offsets[s + 1] - offsets[s];
    const PrefixEntry *pc = pre + (long long)s * kHistBins;
    const __int128 SX = (__int128)pc[kHistBins - 1].sum();
    const int64_t eta = eta_r[i];
    int64_t nle;
    __int128 sle;
    if (eta < 0) {
        nle = 0;
        sle = 0;
    } else if (eta >= kHistBins - 1) {
        nle = N;
        sle = SX;
    } else {
        const PrefixEntry e = pc[eta];
        nle = (int64_t)e.cnt;
        sle = (__int128)e.sum();
    }
    const __int128 CP = fix33(c_p[c]), CW = fix33(c_w[c]);
    const __int128 S = CP * ((SX - sle) - (__int128)eta * (__int128)(N - nle)) +
                       CW * ((__int128)eta * (__int128)nle - sle);
    const unsigned __int128 u = (unsigned __int128)S;  // S >= 0
    cost[i] = __ddiv_rn(fix128_to_double((uint64_t)u, (uint64_t)(u >> 64)), (double)N);
    cover[i] = nle;
}

hipError_t launch_moments(const int64_t *offsets, const int32_t *seg, const int32_t *xi, int S,
                          int C, const RowPlan &pl, RowMoments *rows, int64_t *count, int64_t *sum,
                          int64_t *sumsq, int32_t *xmax, const int32_t *eta, int K, int32_t *k0,
                          hipStream_t st)
{
    const bool small = pl.longest <= kMomShort;
    hipLaunchKernelGGL(small ? row_moments_kernel<64> : row_moments_kernel<256>,
                       dim3((unsigned)std::min(pl.rows, kMaxGridBlocks)), dim3(small ? 64 : 256), 0,
                       st, offsets, xi, S, pl.B, pl.boff, pl.rows, rows);
    HIPRET(hipGetLastError());
    const long long blocks = std::min(((long long)C + kMomWaves - 1) / kMomWaves, kMaxGridBlocks);
    hipLaunchKernelGGL(class_moments_kernel, dim3((unsigned)blocks), dim3(64 * kMomWaves), 0, st,
                       offsets, seg, (const RowMoments *)rows, pl.B, pl.boff, C, count, sum, sumsq,
                       xmax, eta, K, k0);
    return hipGetLastError();
}

hipError_t launch_reservation_cost(const int64_t *offsets, const int32_t *seg, const float *c_p,
                                   const float *c_w, const PrefixEntry *pre, int C, int R,
                                   const int32_t *eta_r, double *cost, int64_t *cover,
                                   hipStream_t st)
{
    const long long n = (long long)R * C;
    hipLaunchKernelGGL(reservation_cost_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0,
                       st, offsets, seg, c_p, c_w, pre, C, n, eta_r, cost, cover);
    return hipGetLastError();
}

}  // namespace dro
