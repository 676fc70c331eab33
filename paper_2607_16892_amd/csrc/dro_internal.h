// Internal declarations shared by the HIP translation units of libdro.
// Not part of the public ABI (include/dro.h is).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "dro.h"
#include "plan.h"

namespace dro {

// ---- dense evaluation -------------------------------------------------------
// A 256-lane block covers a tile of 256 kTM (grid point, multiplier) pairs of one
// class, kTM per lane, taken in table order.  The samples of each tile are split
// into P slices.  A persistent grid of blocks claims slices
// (its own tiles first, then other tiles' unclaimed slices) and keeps a
// tile's sums in registers over consecutive slices of that tile.
constexpr int kTileN = 8192;          // 16-bit LDS words of the staging buffers and the thresholds
constexpr int kHalfSadSteps = 32766;  // v_sad_u16 steps between carries: a sum kept below 2^31
                                      // takes 32766 more steps of at most 2 * 32770 below 2^32
constexpr int kXcds = 8;              // accelerator complex dies of one MI355X (one L2 each)

struct DenseArgs {
    const int64_t *offsets;
    const int32_t *seg;
    const int32_t *xi;
    const int32_t *L;
    const int32_t *eta;
    const float *lam;
    const float *c_p;
    const float *c_w;
    int C, K, M;
    DensePlan plan;
    unsigned long long *R;  // [C][K][M] sums of |x - t| over the class's samples, zeroed first
                            // unless plan.stored
    uint32_t *claim;        // dense_claim_words: slice counters per tile, then the total, zeroed
                            // first; direct: the classes' first slices (slice_starts_kernel)
};

hipError_t launch_dense(const DenseArgs &a, hipStream_t st);
// resident dense blocks per compute unit (occupancy of dense_kernel)
int dense_blocks_per_cu();
// Launches whose block count grows with the problem loop over their items or
// rows with at most kMaxGridBlocks blocks, so a grid stays below 2^32
// work-items whatever the sizes.
constexpr long long kMaxGridBlocks = 1LL << 20;

// zeroes p[0, n) and q[0, nq)
hipError_t launch_zero_u64_u32(unsigned long long *p, long long n, uint32_t *q, long long nq,
                               hipStream_t st);

// ---- value counts ------------------------------------------------------------
constexpr int kHistBins = 32769;  // values 0 .. 2^15
// Prefix count #{x <= v} and sum of those samples of one segment: one entry per
// value v, read with one 12-byte load.
struct PrefixEntry {
    uint32_t cnt, sum_lo, sum_hi;
    __host__ __device__ static PrefixEntry of(uint32_t c, uint64_t s)
    {
        return PrefixEntry{c, (uint32_t)s, (uint32_t)(s >> 32)};
    }
    __host__ __device__ uint64_t sum() const { return (uint64_t)sum_lo | ((uint64_t)sum_hi << 32); }
};

// ---- dense epilogue ------------------------------------------------------------
// W[e,c,k] = min_m RN(RN(lam_m eps[e,c]) + RN(S[c,k,m] / N_c)) and the lowest m
// (m_star may be null), for the table's rows.  With `finish`, S holds the dense
// kernel's sums and is overwritten by the exact S from them and the segments'
// prefix entries (pre: [S][kHistBins], from launch_counts); without it S is read
// only and L, eta, c_p, c_w and pre are not used.
struct RowMinArgs {
    const int64_t *offsets;
    const int32_t *seg;
    const int32_t *L;
    const int32_t *eta;
    const float *lam;
    const float *c_p;
    const float *c_w;
    const float *eps;
    const PrefixEntry *pre;
    int E, C, K, M;
    double *S;
    double *W;
    int32_t *m_star;
};
hipError_t launch_row_min(const RowMinArgs &a, bool finish, int num_cu, hipStream_t st);

// ---- rows: the parts the samples are counted in ---------------------------------
constexpr int kQTop = 32768;              // largest sample value, 2^15
constexpr int kQWords = kQTop / 2 + 1;    // packed 16-bit counts of the values 0 .. 2^15
constexpr int kQStride = kQWords + 3;     // words per stored row and LDS copy (16-byte multiple)
constexpr int kQBuckets = 256;            // coarse buckets of 128 values (the last also holds 2^15)
constexpr long long kQMaxPart = 65535;    // samples per row, so every 16-bit count fits
// Every segment is cut into parts of about one length, one row each: B rows per
// segment when boff is null (rows = S B), else boff[s] .. boff[s+1] are segment
// s's rows (device int64 [S+1], rows = boff[S]).
struct RowPlan {
    long long rows;
    int B;
    const int64_t *boff;
    long long longest;  // samples of the longest row, at most
    long long most;     // rows of the segment with the most
};
// samples per part: about one part per compute unit over all segments (host offsets)
long long row_part_len(const int64_t *offsets_h, int S, int num_cu);
inline long long row_parts(long long n, long long len) { return n <= len ? 1 : (n + len - 1) / len; }

hipError_t launch_fill_u32(uint32_t *p, long long n, uint32_t v, hipStream_t st);
// Writes offsets [S+1], the row table [S+1] (both pointers null: none) and the segment
// map [C] (null: none) to the device, taking them from host memory in kernel arguments
// before it returns.  S <= kStageSegs.
constexpr int kStageSegs = 63;
hipError_t launch_stage_args(const int64_t *offsets_h, const int64_t *boff_h, int S,
                             const int32_t *seg_h, int C, int64_t *offsets, int64_t *boff,
                             int32_t *seg, hipStream_t st);
// allows the histogram and quantile kernels their 128 KB of dynamic LDS (once per device)
hipError_t hist_prepare();

// ---- class_quantile (per-block packed histograms, then a select per class) ----
// fine: [rows][kQStride] u32, coarse: [rows][kQBuckets] u32 (scratch, fully written)
hipError_t launch_class_quantile(const int64_t *offsets, const int32_t *seg, const int32_t *xi,
                                 const float *c_p, const float *c_w, int S, int C, const RowPlan &pl,
                                 uint32_t *fine, uint32_t *coarse, int32_t *q_value,
                                 int64_t *q_rank, hipStream_t st);

// ---- prefix counts and sums of every segment -----------------------------------
// From packed rows (fine, coarse and csum, the sums per coarse bucket: [rows]
// each) or, where their scratch does not fit, from a merged histogram (hist
// non-null: [S][kHistBins], plan.B blocks per segment; tot: the chunk totals).
constexpr int kPrefixChunk = 4096;  // bins per chunk of the merged histogram's prefix pass
constexpr int kPrefixChunks = (kHistBins + kPrefixChunk - 1) / kPrefixChunk;
struct CountBufs {
    RowPlan plan;
    uint32_t *fine, *coarse, *csum;
    uint32_t *hist;
    uint64_t *tot;     // [S][kPrefixChunks][2]
    PrefixEntry *pre;  // [S][kHistBins]
};
// blocks per segment of the merged histogram
int hist_parts(int S, long long max_seg, int num_cu);
hipError_t launch_counts(const int64_t *offsets, const int32_t *xi, int S, const CountBufs &b,
                         hipStream_t st);
// the critical-fractile quantile of every class from the prefix entries
hipError_t launch_prefix_select(const int64_t *offsets, const int32_t *seg, const float *c_p,
                                const float *c_w, const PrefixEntry *pre, int C, int32_t *q_value,
                                hipStream_t st);

// ---- exact table (value counts and prefix sums) -------------------------------
// k_star == null skips the argmin.
hipError_t launch_exact_table(const int64_t *offsets, const int32_t *seg, const int32_t *L,
                              const int32_t *eta, const float *lam, const float *c_p,
                              const float *c_w, const float *eps, const int32_t *k_max,
                              const PrefixEntry *pre, int E, int C, int K, int M, double *W,
                              int32_t *m_star, int32_t *k_star, double *W_star, int32_t *m_at_star,
                              hipStream_t st);
// Per (e, c): the lowest k <= k_max[c] (k_max may be null: K - 1) with the
// smallest W[e,c,k], W there, and m_star there (m_at_star may be null).
hipError_t launch_table_argmin(const double *W, const int32_t *m_star, const int32_t *k_max,
                               int E, int C, int K, int32_t *k_star, double *W_star,
                               int32_t *m_at_star, hipStream_t st);

// continuous-multiplier dual over the same prefix counts (gamma: the smallest minimiser)
hipError_t launch_continuous_dual(const int64_t *offsets, const int32_t *seg, const int32_t *L,
                                  const int32_t *eta, const float *c_p, const float *c_w,
                                  const float *eps, const PrefixEntry *pre, int E, int C, int K,
                                  double *W, double *gamma, hipStream_t st);

// ---- reservation cost and class moments ----------------------------------------
struct RowMoments {
    long long raw, sum;     // sum of the samples as they are, and clamped to 0 .. 2^15
    unsigned long long sq;  // sum of squares and largest of the clamped samples
    long long mx;
};
// rows: [plan.rows] scratch.  count .. xmax (may all be null) and, with eta, the
// initial state of Alg. 1, r0 = L_in + E[xi]: k0[c] = the largest k with
// eta[k] N <= the sum of the samples.
hipError_t launch_moments(const int64_t *offsets, const int32_t *seg, const int32_t *xi, int S,
                          int C, const RowPlan &pl, RowMoments *rows, int64_t *count, int64_t *sum,
                          int64_t *sumsq, int32_t *xmax, const int32_t *eta, int K, int32_t *k0,
                          hipStream_t st);
hipError_t launch_reservation_cost(const int64_t *offsets, const int32_t *seg, const float *c_p,
                                   const float *c_w, const PrefixEntry *pre, int C, int R,
                                   const int32_t *eta_r, double *cost, int64_t *cover,
                                   hipStream_t st);

// ---- baseline reservations (policy comparison) ---------------------------------
constexpr int kMaxBaselineKs = 8;
struct BaselineKs {
    int n;                    // number of multiples k of the standard deviation
    int k[kMaxBaselineKs];    // each in [0, 64]
};
hipError_t launch_baselines(int C, const int64_t *count, const int64_t *sum, const int64_t *sumsq,
                            const int32_t *L, const BaselineKs &ks, const int32_t *q, int block,
                            int32_t *mean_r, int32_t *lp_r, int32_t *block_r, hipStream_t st);

// ---- block step ----------------------------------------------------------------
// best[c,k] = the lowest argmin of W[c, 0 .. k] (int32 [C][K])
hipError_t launch_best_upto(const double *W, int C, int K, int32_t *best, hipStream_t st);
// The block step's Gauss-Seidel sweep over the exact W [C][K] (one radius row) and
// its best_upto, k_prev [C] the state entering it; kcur: [C] scratch.
hipError_t launch_bcd_sweep(const double *W, const int32_t *best, const int32_t *eta, int C, int K,
                            int G, const float *cap, const float *conc, float kappa,
                            const int32_t *k_prev, int32_t *kcur, int32_t *k_next, double *W_star,
                            uint8_t *feasible, double *usage, hipStream_t st);

// ---- serving model: routing LP, prefix caching, configuration search -------------
struct SvcArgs {
    int C, G;
    const int32_t *tau, *pp;
    const float *Mcap, *Cc, *Bc;
    const float *lam;
    const int32_t *Lin, *Lpre;
    const float *D;
    double alpha, beta, t_ar, NL, c_gpu, c_slo, c_rej, kappa, u_max;
    int J;
};

hipError_t launch_service_times(const SvcArgs &s, const int64_t *count, const int64_t *sum,
                                const int64_t *sumsq, double *T, double *ET2, hipStream_t st);
hipError_t launch_state(const SvcArgs &s, const double *T, const double *ET2, const double *pi,
                        const int32_t *z, const int32_t *eta_c, const uint8_t *delta, double *Wq,
                        double *cap, double *conc, double *mem, hipStream_t st);
hipError_t launch_cache(const double *conc, int n, uint8_t *delta, hipStream_t st);
// doubles of the LP1 work area (tableau, pivot column and row, basis)
size_t lp1_work_doubles(int C, int G);
// allow lp1_kernel its dynamic LDS (once per device)
hipError_t lp1_prepare();
hipError_t launch_lp1(const SvcArgs &s, const double *Wc, const double *T, const double *Wq,
                      const int32_t *z, const int32_t *eta_c, const uint8_t *delta, double *work,
                      int max_pivots, double *pi_out, double *obj_out, int32_t *info,
                      hipStream_t st);
hipError_t launch_sweep(const double *W, const int32_t *eta, int C, int K, int G,
                        const double *conc, const double *cap, double kappa, const int32_t *k_in,
                        int32_t *k_out, uint8_t *feasible, hipStream_t st);
// Scratch of the configuration search: the z-independent sums and routing entries,
// the waits per configuration and count, the count table of the ranks and the
// blocks' results.
struct ConfigBufs {
    double *pre_d;   // [config_pre_doubles]
    int32_t *pre_i;  // [config_pre_ints]
    double *wt;      // [G][J + 1]
    int32_t *gpus;   // [G] tau pp
    long long *ways; // [G + 1][J + 1]
    double *part_obj;
    long long *part_rank, *part_feas;  // [config_parts] each
    double *best_obj;
    long long *best_rank, *n_feas;
};
size_t config_pre_doubles(int C, int G);
size_t config_pre_ints(int C, int G);
// blocks of the search over nz configurations
long long config_parts(long long nz);
hipError_t launch_config_prep(const SvcArgs &s, const double *T, const double *ET2, const double *pi,
                              const int32_t *eta_c, const uint8_t *delta, const ConfigBufs &b,
                              hipStream_t st);
// after launch_config_prep (or launch_block1) on the same buffers
hipError_t launch_config_search(const SvcArgs &s, long long nz, const double *Wc,
                                const ConfigBufs &b, int32_t *z, const uint8_t *delta_new,
                                uint8_t *delta, double *best_obj, long long *best_rank,
                                long long *n_feasible, int32_t *flag, hipStream_t st);
// Blocks 1 and 2 of one outer iteration of Alg. 1 and the sums of Block 3.
struct Block1Args {
    const double *W;      // [C][K]
    const int32_t *best;  // its launch_best_upto
    const int32_t *eta;   // [K]
    int K;
    const double *T, *ET2;
    int32_t *k;           // [C] in and out
    double *pi;           // [C * G] in and out
    const int32_t *z;
    uint8_t *delta;       // [C * G] the caching entering (zeroed with pi when first)
    uint8_t *d_new;       // the caching of Block 2
    double *pi_new;
    int32_t *k_new;
    double *Wc;           // W and eta at the reservations leaving
    int32_t *eta_c;
    double *Wq, *cap, *conc;
    double *work;         // [lp1_work_doubles]
    ConfigBufs b;
    int32_t *ctl;         // out: rounds, pivots, status bits (1, 2, 4, 16 of dro_bcd_solve),
                          // 1 if the last sweep found every class a feasible reservation
    int max_inner, max_pivots, first;
    double tol;
};
hipError_t launch_block1(const SvcArgs &s, const Block1Args &a, hipStream_t st);
hipError_t launch_state_objective(const SvcArgs &s, const double *T, const double *ET2,
                                  const double *pi, const int32_t *z, const int32_t *eta_c,
                                  const uint8_t *delta, const double *Wc, const ConfigBufs &b,
                                  double *out, hipStream_t st);

// ---- validation ----------------------------------------------------------------
hipError_t launch_seg_minmax(const int64_t *offsets, const int32_t *xi, int S, long long max_seg,
                             int32_t *mn, int32_t *mx, hipStream_t st);

}  // namespace dro
