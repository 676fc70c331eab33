// The rest of Alg. 1 around the reservation update: the routing LP (LP1 of
// Block 1), prefix caching (Block 2) and the configuration search (Block 3),
// over the serving model of Sec. 3.1-3.4.
//
// Compiled with -ffp-contract=off: every double expression is evaluated in the
// order written, one rounding per operation, so that the decisions taken on
// its values (capacity bounds, the caching threshold, the configuration
// objective) are reproducible bit for bit.
//
// Model (per class c and configuration g; z_g groups of configuration g):
//   T[c,g]    = pp_g alpha Lin_c / Cc_g + NL tau_g t_ar + beta E[xi_c] / Bc_g
//   conc[c,g] = lam_c T_cg pi_cg / z_g                      (Little's law)
//   mem[g]    = (1 + kappa) (sum_c lam_c T_cg pi_cg (Lin_c + eta_c - delta_cg Lpre_c)) / z_g
//               + sum_c delta_cg Lpre_c                      (KV tokens in use)
//   Wq[g]     = u (1 + Cs2) / (2 (1 - u)) Tbar with u = mem_g / Mcap_g
//               (Pollaczek-Khinchin at the memory utilisation)
//   objective = sum_c lam_c (a_c W_c + sum_g pi_cg c_gpu tau_g pp_g T_cg + c_slo s_c
//               + (1 - a_c) c_rej),  s_c = max(0, sum_g pi_cg (Wq_g + T_cg) - a_c D_c)
//   feasible  : sum_g z_g tau_g pp_g <= J, pi_cg > 0 only where z_g > 0,
//               mem_g <= u_max Mcap_g (1 + 1e-9): the slack makes a routing that
//               the LP leaves exactly at its memory bound count as feasible.
#include <algorithm>
#include <cmath>

#include "dro_internal.h"
#include "sweep.h"
#include "wave.h"

namespace dro {

namespace {

constexpr int kSvcThreads = 256;
constexpr double kMemSlack = 1.0 + 1e-9;  // relative slack of a configuration's memory check
constexpr double kEtaSlack = 1e-6;        // tokens of slack of the sweep's reservation bound
constexpr int kLpDegenerateRun = 20;      // degenerate pivots before the simplex turns to Bland's rule

// The z-independent sums of the configuration search (config_prep_block) and the
// routing's non-zero entries: entries start[c] .. start[c + 1] - 1 of g, pi, T.
struct ConfigPre {
    double *a, *gpu;                      // [C]
    double *used, *pre, *load, *X, *m2;   // [G]
    double *pi, *T;                       // entries
    int32_t *start, *g, *route;           // [C + 1], entries, [G] some pi_cg > 0
};

}  // namespace

// ------------------------------------------------------------ service times --
__global__ void service_times_kernel(SvcArgs s, const int64_t *count, const int64_t *sum,
                                     const int64_t *sumsq, double *T, double *ET2)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= s.C * s.G) return;
    const int c = i / s.G, g = i % s.G;
    const double n = (double)count[c];
    const double mean = (double)sum[c] / n;
    const double ex2 = (double)sumsq[c] / n;
    double A = (double)s.pp[g] * s.alpha * (double)s.Lin[c] / (double)s.Cc[g];
    A = A + s.NL * (double)s.tau[g] * s.t_ar;
    const double B = s.beta / (double)s.Bc[g];
    T[i] = A + B * mean;
    ET2[i] = A * A + 2.0 * A * B * mean + B * B * ex2;
}

// ---------------------------------------------------------------- state -----
// Per configuration g: the waiting time at the current state, the memory left
// for the reservations (cap) and conc[c, g] (Wq and mem_out may be null).  One
// wave per configuration: a lane forms a class's six terms, six lanes then add
// them up in class order from LDS.
constexpr int kBlockThreads = 1024;
constexpr int kStateLds = 6 * kBlockThreads;  // doubles

__device__ void state_block(const SvcArgs &s, const double *T, const double *ET2, const double *pi,
                            const int32_t *z, const int32_t *eta_c, const uint8_t *delta,
                            double *Wq, double *cap, double *conc, double *mem_out, double *lds)
{
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, C = s.C, G = s.G;
    double *sc = lds + wave * 6 * 64;
    for (int g = wave; g < G; g += kBlockThreads / 64) {
        if (z[g] <= 0) {
            for (int c = lane; c < C; c += 64) conc[c * G + g] = 0.0;
            if (lane == 0) {
                if (Wq) Wq[g] = 0.0;
                cap[g] = INFINITY;
                if (mem_out) mem_out[g] = 0.0;
            }
            continue;
        }
        const double zg = (double)z[g];
        double acc = 0.0;  // lanes 0 .. 5: used, fixed, pre, load, X, m2
        for (int c0 = 0; c0 < C; c0 += 64) {
            const int c = c0 + lane;
            if (c < C) {
                const int i = c * G + g;
                const int dl = delta[i] ? s.Lpre[c] : 0;
                const double lTp = (double)s.lam[c] * T[i] * pi[i];
                const double wgt = (double)s.lam[c] * pi[i];
                sc[lane] = lTp * (double)(s.Lin[c] + eta_c[c] - dl);
                sc[64 + lane] = lTp * (double)(s.Lin[c] - dl);
                sc[128 + lane] = (double)dl;
                sc[192 + lane] = wgt * T[i];
                sc[256 + lane] = wgt;
                sc[320 + lane] = wgt * ET2[i];
                conc[i] = lTp / zg;
            }
            wave_sync();
            if (lane < 6)
                for (int i = 0; i < min(64, C - c0); ++i) acc = acc + sc[lane * 64 + i];
            wave_sync();
        }
        const double used = __shfl(acc, 0), fixed = __shfl(acc, 1), pre = __shfl(acc, 2);
        const double load = __shfl(acc, 3), X = __shfl(acc, 4), m2 = __shfl(acc, 5);
        if (lane != 0) continue;
        const double kap = 1.0 + s.kappa;
        const double mem = kap * (used / zg) + pre;
        double w = 0.0;
        if (X > 0.0) {
            const double u = mem / (double)s.Mcap[g];
            const double tb = load / X;
            const double cs2 = (m2 / X) / (tb * tb) - 1.0;
            w = u < 1.0 ? u * (1.0 + cs2) / (2.0 * (1.0 - u)) * tb : INFINITY;
        }
        if (Wq) Wq[g] = w;
        cap[g] = s.u_max * (double)s.Mcap[g] - pre - kap * (fixed / zg);
        if (mem_out) mem_out[g] = mem;
    }
}

__global__ __launch_bounds__(kBlockThreads) void state_kernel(
    SvcArgs s, const double *T, const double *ET2, const double *pi, const int32_t *z,
    const int32_t *eta_c, const uint8_t *delta, double *Wq, double *cap, double *conc,
    double *mem_out)
{
    __shared__ double lds[kStateLds];
    state_block(s, T, ET2, pi, z, eta_c, delta, Wq, cap, conc, mem_out, lds);
}

// Block 2: delta = 1[conc > 1]
__global__ void cache_kernel(const double *conc, int n, uint8_t *delta)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) delta[i] = conc[i] > 1.0 ? 1 : 0;
}

// ------------------------------------------------------------------- LP1 ----
// min c^T x over x >= 0 with A x <= b, b >= 0, by the simplex method on a
// dense tableau.  The entering column has the most negative reduced cost;
// after 20 degenerate pivots in a row the rule becomes Bland's (smallest
// entering index) until a pivot moves the objective, so the method cannot
// cycle.  Ties of the ratio test go to the smallest basic index.  Variables: pi[c,g]
// at c*G + g (fixed at 0 where z_g = 0: an empty column of cost 0), then s_c.
// Rows: sum_g pi_cg <= 1; sum_g pi_cg (Wq_g + T_cg - D_c) - s_c <= 0; memory of
// every g with z_g > 0 (empty rows otherwise).  Each row is scaled by its largest
// coefficient, the objective by its largest cost.  One block of 1,024 threads;
// the tableau ((m + 1) x (n + m + 1) doubles, in LDS when it fits), the pivot
// column, the scaled pivot row and the basis lie in `work`.
// A pivot is latency: the first wave alone finds the entering column and the
// leaving row (four reduced costs in flight per lane, a ratio or two, then 32-bit
// minima; a block-wide reduction costs two barriers and a pass over the waves
// each), all threads copy the pivot's column and scale its row once, then update a
// column of every fourth row each.  15 pivots on 15 x 12 routings (43 x 238
// doubles) took 62 us with the rest of the kernel, 159 before (256 threads,
// block-wide reductions, basis and configuration counts read from memory at every
// pivot, row scaling and the objective on one thread per row); 32-bit minima for
// fp64 ones took another 5 us off.
constexpr int kLpThreads = kBlockThreads;
constexpr int kLpMaxG = 32;

struct LpShared {
    int jin, rsel, status, pivots;
    double scale;
    double red[kLpThreads / 64];
    unsigned long long pre[kLpMaxG];
};

// doubles of the work area
__host__ __device__ inline long long lp1_doubles(int C, int G)
{
    const long long nv = (long long)C * G + C, m = 2LL * C + G, w = nv + m + 1;
    return (m + 1) * w + (m + 1) + w + (m + 1) / 2 + 1;
}

// (kLds: `work` is the kernel's dynamic LDS, known as such to the compiler: through
// a pointer that may be either, every access is a flat one, at a third of the rate)
template <bool kLds>
__device__ __forceinline__ void lp1_block(const SvcArgs &s, const double *Wc, const double *T,
                                          const double *Wq, const int32_t *z, const int32_t *eta_c,
                                          const uint8_t *delta, double *work_g, int max_pivots,
                                          double *pi_out, double *obj_out, LpShared &sh)
{
    extern __shared__ double dyn[];
    double *work = kLds ? dyn : work_g;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, nt = kLpThreads;
    const int C = s.C, G = s.G, CG = C * G;
    const int nv = CG + C, m = 2 * C + G, w = nv + m + 1;
    const double kap = 1.0 + s.kappa;
    double *tab = work, *col = tab + (long long)(m + 1) * w, *prow = col + (m + 1);
    int32_t *basis = reinterpret_cast<int32_t *>(prow + w);

    // build: constraint rows, slack identity, right-hand sides
    for (long long e = t; e < (long long)(m + 1) * w; e += nt) tab[e] = 0.0;
    if (t < G) sh.pre[t] = 0ull;
    if (t == 0) sh.status = sh.pivots = 0;
    __syncthreads();
    double lmx = 0.0;  // the objective row's costs and their largest
    for (int i = t; i < CG; i += nt) {
        const int c = i / G, g = i % G;
        if (z[g] <= 0) continue;
        const int dl = delta[i] ? s.Lpre[c] : 0;
        if (dl) atomicAdd(&sh.pre[g], (unsigned long long)(long long)dl);  // exact in any order
        const double rt = (double)(s.Lin[c] + eta_c[c] - dl);
        tab[(long long)c * w + i] = 1.0;
        tab[(long long)(C + c) * w + i] = Wq[g] + T[i] - (double)s.D[c];
        tab[(long long)(2 * C + g) * w + i] = kap * ((double)s.lam[c] * T[i] / (double)z[g]) * rt;
        const double cj =
            (double)s.lam[c] * (Wc[c] + s.c_gpu * (double)(s.tau[g] * s.pp[g]) * T[i] - s.c_rej);
        tab[(long long)m * w + i] = cj;
        lmx = fmax(lmx, fabs(cj));
    }
    for (int c = t; c < C; c += nt) {
        tab[(long long)(C + c) * w + CG + c] = -1.0;
        const double cj = (double)s.lam[c] * s.c_slo;
        tab[(long long)m * w + CG + c] = cj;
        lmx = fmax(lmx, fabs(cj));
    }
    for (int off = 32; off > 0; off >>= 1) lmx = fmax(lmx, __shfl_xor(lmx, off));
    if (lane == 0) sh.red[wave] = lmx;
    __syncthreads();
    // one wave per row: its largest coefficient, the scaled row, the slack, the bound
    for (int r = wave; r < m; r += nt / 64) {
        double *row = tab + (long long)r * w;
        double mx = 0.0;
        for (int j = lane; j < nv; j += 64) mx = fmax(mx, fabs(row[j]));
        for (int off = 32; off > 0; off >>= 1) mx = fmax(mx, __shfl_xor(mx, off));
        const double sc = mx > 0.0 ? 1.0 / mx : 1.0;
        for (int j = lane; j < nv; j += 64) row[j] *= sc;
        if (lane == 0) {
            double rhs = 0.0;
            if (r < C) rhs = 1.0;
            else if (r >= 2 * C && z[r - 2 * C] > 0)
                rhs = s.u_max * (double)s.Mcap[r - 2 * C] - (double)(long long)sh.pre[r - 2 * C];
            if (rhs < 0.0) sh.status = 2;  // infeasible start
            row[nv + r] = 1.0;
            row[w - 1] = rhs * sc;
            basis[r] = nv + r;
        }
    }
    double cmx = 0.0;
    for (int q = 0; q < nt / 64; ++q) cmx = fmax(cmx, sh.red[q]);
    const double scale = cmx > 0.0 ? 1.0 / cmx : 1.0;
    for (int j = t; j < nv; j += nt) tab[(long long)m * w + j] *= scale;
    __syncthreads();

    // status: 0 optimal, 1 pivot limit, 2 infeasible start, 3 unbounded
    const double tol_d = 1e-12, tol_p = 1e-11;
    int degenerate = 0;  // (the first wave's)
    bool run = sh.status == 0;
    __syncthreads();
    while (run) {
        if (wave == 0) {
            // entering column: the most negative reduced cost (lowest index on ties);
            // after a run of degenerate pivots, the lowest index with a negative
            // reduced cost (Bland's rule, which cannot cycle) until the objective moves
            const bool bland = degenerate >= kLpDegenerateRun;
            double dmin = 0.0;
            int cand = 0x7fffffff;
            for (int j0 = lane; j0 < nv + m; j0 += 256) {  // four loads in flight
                double d[4];
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    d[q] = tab[(long long)m * w + min(j0 + 64 * q, nv + m - 1)];
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (j0 + 64 * q < nv + m && d[q] < -tol_d &&
                        (bland ? cand == 0x7fffffff : d[q] < dmin)) {
                        dmin = d[q];
                        cand = j0 + 64 * q;
                    }
            }
            const int jin = wave_min_key(bland ? 0.0 : dmin, cand, 0).idx;
            int rsel = -1;
            if (jin == 0x7fffffff) {
                // optimal
            } else if (sh.pivots >= max_pivots) {
                if (lane == 0) sh.status = 1;
            } else {
                // ratio test: smallest b_i / a_ij over a_ij > 0, ties to the smallest basic index
                double best = INFINITY;
                int bb = 0x7fffffff, brow = -1;
                for (int r = lane; r < m; r += 64) {
                    const double a = tab[(long long)r * w + jin];
                    if (a > tol_p) {
                        const double q = tab[(long long)r * w + w - 1] / a;
                        const int bs = basis[r];
                        if (q < best || (q == best && bs < bb)) {
                            best = q;
                            bb = bs;
                            brow = r;
                        }
                    }
                }
                const KeyIdx lv = wave_min_key(best, bb, brow);
                if (lv.idx == 0x7fffffff) {
                    if (lane == 0) sh.status = 3;
                } else {
                    rsel = lv.aux;  // the row of the leaving basic variable
                    degenerate = lv.key == 0.0 ? degenerate + 1 : 0;
                    if (lane == 0) {
                        basis[rsel] = jin;
                        ++sh.pivots;
                    }
                }
            }
            if (lane == 0) {
                sh.jin = jin;
                sh.rsel = rsel;
            }
        }
        __syncthreads();
        const int jin = sh.jin, rsel = sh.rsel;
        if (rsel < 0) break;
        // pivot on (rsel, jin)
        const double piv = tab[(long long)rsel * w + jin];
        for (int r = t; r <= m; r += nt) col[r] = tab[(long long)r * w + jin];
        for (int j = t; j < w; j += nt) prow[j] = tab[(long long)rsel * w + j] / piv;
        __syncthreads();
        for (int j = t & 255; j < w; j += 256) {
            const double pj = prow[j];
            for (int r0 = t >> 8; r0 <= m; r0 += 16) {
                double v[4], f[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int r = min(r0 + 4 * q, m);
                    v[q] = tab[(long long)r * w + j];
                    f[q] = col[r];
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int r = r0 + 4 * q;
                    if (r > m) continue;
                    if (r == rsel) tab[(long long)r * w + j] = pj;
                    else if (f[q] != 0.0) tab[(long long)r * w + j] = v[q] - f[q] * pj;
                }
            }
        }
        __syncthreads();
    }
    // solution
    for (int j = t; j < CG; j += nt) pi_out[j] = 0.0;
    __syncthreads();
    for (int r = t; r < m; r += nt) {
        const int j = basis[r];
        if (j < CG) {
            const double v = tab[(long long)r * w + w - 1];
            pi_out[j] = v > 0.0 ? v : 0.0;
        }
    }
    __syncthreads();
    if (obj_out && wave == 0) {
        // objective of the routing: sum_c lam_c (sum_g pi_cg (W_c + c_gpu tau pp T - c_rej)
        // + c_slo s_c + c_rej) with s_c at its optimum max(0, sum_g pi_cg h_cg), the
        // classes in order (a lane computes a class's term)
        double obj = 0.0;
        for (int c0 = 0; c0 < C; c0 += 64) {
            const int c = c0 + lane;
            double term = 0.0;
            if (c < C) {
                double lin = 0.0, h = 0.0;
                for (int g = 0; g < G; ++g) {
                    const double p = pi_out[c * G + g];
                    if (z[g] <= 0) continue;
                    lin = lin + p * (Wc[c] + s.c_gpu * (double)(s.tau[g] * s.pp[g]) * T[c * G + g] - s.c_rej);
                    h = h + p * (Wq[g] + T[c * G + g] - (double)s.D[c]);
                }
                term = (double)s.lam[c] * (lin + s.c_slo * (h > 0.0 ? h : 0.0) + s.c_rej);
            }
            for (int i = 0; i < min(64, C - c0); ++i) obj = obj + __shfl(term, i);
        }
        if (lane == 0) obj_out[0] = obj;
    }
}

template <bool kLds>
__global__ __launch_bounds__(kLpThreads) void lp1_kernel(SvcArgs s, const double *Wc,
                                                         const double *T, const double *Wq,
                                                         const int32_t *z, const int32_t *eta_c,
                                                         const uint8_t *delta, double *work,
                                                         int max_pivots, double *pi_out,
                                                         double *obj_out, int32_t *info)
{
    __shared__ LpShared sh;
    lp1_block<kLds>(s, Wc, T, Wq, z, eta_c, delta, work, max_pivots, pi_out, obj_out, sh);
    if (threadIdx.x == 0) {
        info[0] = sh.pivots;
        info[1] = sh.status;
    }
}

// ------------------------------------------------------------------- LP2 ----
// The reservation sweep of the block step over a fixed W table: for c in
// order, the largest admissible grid point given the others, then the lowest
// argmin of W[c, 0..kmax], with 1e-6 tokens of slack on the bound so that a
// reservation at which the LP left the memory exactly full stays admissible.
// One block.  Incoming grid indices are clamped into [0, K).
// The call has no scratch, so this kernel takes each class's minimum over its
// admissible points directly (the loop of Alg. 1 keeps the table of sweep_wave).
__global__ __launch_bounds__(kBlockThreads) void sweep_kernel(
    const double *W, const int32_t *eta, int C, int K, int G, const double *conc,
    const double *cap, double kappa, const int32_t *k_in, int32_t *k_out, uint8_t *feasible)
{
    __shared__ double s_top, sw[kBlockThreads / 64];
    __shared__ int sk[kBlockThreads / 64];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    for (int c = t; c < C; c += kBlockThreads) k_out[c] = min(max(k_in[c], 0), K - 1);
    __syncthreads();
    for (int c = 0; c < C; ++c) {
        if (wave == 0) {
            const double b = sweep_bound(c, C, G, conc, cap, 1.0 + kappa,
                                         [&](int c2) { return (double)eta[k_out[c2]]; });
            if (lane == 0) s_top = b + kEtaSlack;
        }
        __syncthreads();
        const double top = s_top;
        double bw = INFINITY;
        int bk = 0x7fffffff;
        for (int k = t; k < K; k += kBlockThreads) {  // ascending: a thread's first minimiser
            const double v = W[(long long)c * K + k];
            if ((double)eta[k] <= top && v < bw) {
                bw = v;
                bk = k;
            }
        }
        const KeyIdx m = wave_min_key(bw, bk, 0);
        if (lane == 0) {
            sw[wave] = m.key;
            sk[wave] = m.idx;
        }
        __syncthreads();
        if (wave == 0) {
            const KeyIdx r = wave_min_key(lane < kBlockThreads / 64 ? sw[lane] : INFINITY,
                                          lane < kBlockThreads / 64 ? sk[lane] : 0x7fffffff, 0);
            if (lane == 0) {
                const bool feas = (double)eta[0] <= top;
                int k = r.idx;
                if (k > K - 1)  // no W below infinity: the last admissible point
                    for (k = K - 1; k > 0 && !((double)eta[k] <= top);) --k;
                k_out[c] = feas ? k : 0;
                if (feasible) feasible[c] = feas ? 1 : 0;
            }
        }
        __syncthreads();
    }
}

// --------------------------------------------------------------- Block 3 ----
// The objective at a given z with the routing, reservations and caching
// fixed, from sums that do not depend on z: per class a (routed share) and its
// GPU cost, per configuration the memory, load and service-time sums; and the
// routing's non-zero entries, class after class (a zero entry adds nothing to a
// class's response).
constexpr int kMaxG = 32;

__device__ ConfigPre config_view(const ConfigBufs &b, int C, int G)
{
    ConfigPre q;
    q.a = b.pre_d;
    q.gpu = q.a + C;
    q.used = q.gpu + C;
    q.pre = q.used + G;
    q.load = q.pre + G;
    q.X = q.load + G;
    q.m2 = q.X + G;
    q.pi = q.m2 + G;
    q.T = q.pi + (long long)C * G;
    q.start = b.pre_i;
    q.g = q.start + C + 1;
    q.route = q.g + (long long)C * G;
    return q;
}

// One block of kBlockThreads; lds: kStateLds doubles.  G <= 32, so the five sums of every
// configuration have a thread each.
__device__ void config_prep_block(const SvcArgs &s, const double *T, const double *ET2,
                                  const double *pi, const int32_t *eta_c, const uint8_t *delta,
                                  const ConfigPre &q, double *lds)
{
    constexpr int nt = kBlockThreads;
    static_assert(5 * nt + kLpMaxG <= kStateLds && 5 * kLpMaxG <= nt, "a tile; a thread per sum");
    const int t = threadIdx.x, C = s.C, G = s.G;
    // calls f(g, pi, T) for the configurations of class c, in order
    auto routing = [&](int c, auto &&f) {
        for (int g0 = 0; g0 < G; g0 += 8) {
            double p[8], w[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int j = c * G + min(g0 + i, G - 1);
                p[i] = pi[j];
                w[i] = T[j];
            }
#pragma unroll
            for (int i = 0; i < 8; ++i)
                if (g0 + i < G) f(g0 + i, p[i], w[i]);
        }
    };
    auto kept = [](double p, double w) { return p != 0.0 || !(fabs(w) < INFINITY); };
    for (int c = t; c < C; c += nt) {
        double a = 0.0, gpu = 0.0;
        int n = 0;
        routing(c, [&](int g, double p, double w) {
            a = a + p;
            gpu = gpu + p * (s.c_gpu * (double)(s.tau[g] * s.pp[g]) * w);
            n += kept(p, w) ? 1 : 0;
        });
        q.a[c] = a;
        q.gpu[c] = gpu;
        q.start[c + 1] = n;
    }
    // a tile of classes at a time: a thread per (class, configuration) forms its five terms,
    // then a thread per (sum, configuration) adds them up in class order (one thread per
    // configuration, each class a round trip, took 52 us for 200 classes and 12
    // configurations, this takes 16; 88 and 45 for 250 and 32)
    const int tile = nt / G, sum = t / G, g1 = t % G;
    int *any = reinterpret_cast<int *>(lds + 5 * nt);  // [G] some pi_cg > 0
    if (t < G) any[t] = 0;
    double acc = 0.0;
    bool route = false;
    for (int c0 = 0; c0 < C; c0 += tile) {
        const int n = min(tile, C - c0);
        if (sum < n) {  // (t = class of the tile, configuration)
            const int c = c0 + sum, j = c * G + g1;
            const double p = pi[j], w = T[j], w2 = ET2[j], lam = (double)s.lam[c];
            const int pre = s.Lpre[c], res = s.Lin[c] + eta_c[c], dl = delta[j] ? pre : 0;
            const double wgt = lam * p;
            lds[t] = lam * w * p * (double)(res - dl);
            lds[nt + t] = (double)dl;
            lds[2 * nt + t] = wgt * w;
            lds[3 * nt + t] = wgt;
            lds[4 * nt + t] = wgt * w2;
            route = route || p > 0.0;
        }
        __syncthreads();
        if (route) any[g1] = 1;
        if (sum < 5) {
            const double *v = lds + sum * nt + g1;
            int i = 0;
            for (; i + 8 <= n; i += 8) {
                double x[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) x[k] = v[(i + k) * G];
#pragma unroll
                for (int k = 0; k < 8; ++k) acc = acc + x[k];
            }
            for (; i < n; ++i) acc = acc + v[i * G];
        }
        __syncthreads();
    }
    if (sum < 5) (sum == 0 ? q.used : (sum == 1 ? q.pre : (sum == 2 ? q.load : (sum == 3 ? q.X : q.m2))))[g1] = acc;
    if (t < G) q.route[t] = any[t];
    __syncthreads();
    if (t < 64) {  // the classes' entry counts to starts, by one wave
        int base = 0;
        for (int c0 = 0; c0 < C; c0 += 64) {
            const int c = c0 + t;
            const int n = c < C ? q.start[c + 1] : 0;
            const int incl = (int)scan_wave((uint32_t)n);
            if (c < C) q.start[c + 1] = base + incl;
            base += __builtin_amdgcn_readlane(incl, 63);
        }
        if (t == 0) q.start[0] = 0;
    }
    __syncthreads();
    for (int c = t; c < C; c += nt) {
        int o = q.start[c];
        routing(c, [&](int g, double p, double w) {
            if (!kept(p, w)) return;
            q.g[o] = g;
            q.pi[o] = p;
            q.T[o] = w;
            ++o;
        });
    }
}

// Marks a wait that z does not allow: routed traffic without a group, or too
// little memory (a NaN of its own; arithmetic makes none with this payload).
__device__ __forceinline__ double no_wait() { return __longlong_as_double(0x7ff8dead00000000LL); }
__device__ __forceinline__ bool is_no_wait(double w) { return __double2hiint(w) == 0x7ff8dead; }

// The wait of configuration g with z groups.
__device__ __forceinline__ double config_wait(const SvcArgs &s, const ConfigPre &q, int g, int z)
{
    if (z <= 0) return q.route[g] ? no_wait() : 0.0;
    const double kap = 1.0 + s.kappa;
    const double mem = kap * (q.used[g] / (double)z) + q.pre[g];
    if (!(mem <= s.u_max * (double)s.Mcap[g] * kMemSlack)) return no_wait();
    if (!(q.X[g] > 0.0)) return 0.0;
    const double u = mem / (double)s.Mcap[g];
    const double tb = q.load[g] / q.X[g];
    const double cs2 = (q.m2[g] / q.X[g]) / (tb * tb) - 1.0;
    return u < 1.0 ? u * (1.0 + cs2) / (2.0 * (1.0 - u)) * tb : INFINITY;
}

// What the objective needs of the classes: in memory, or staged in LDS.
struct ClassCosts {
    const double *a, *gpu, *Wc, *pi, *T;
    const int32_t *start, *g;
    const double *lam, *D;  // staged; else null and the service's floats are read
};

__device__ __forceinline__ ClassCosts class_costs(const ConfigPre &q, const double *Wc)
{
    return ClassCosts{q.a, q.gpu, Wc, q.pi, q.T, q.start, q.g, nullptr, nullptr};
}

// Class c's share of the objective with the waits wq(g).
template <bool kStaged, class F>
__device__ __forceinline__ double class_cost(const SvcArgs &s, const ClassCosts &q, int c, F &&wq)
{
    double resp = 0.0;
    for (int o = q.start[c]; o < q.start[c + 1]; ++o) resp = resp + q.pi[o] * (wq(q.g[o]) + q.T[o]);
    const double a = q.a[c];
    double sl = resp - a * (kStaged ? q.D[c] : (double)s.D[c]);
    if (sl < 0.0) sl = 0.0;
    return (kStaged ? q.lam[c] : (double)s.lam[c]) *
           (a * q.Wc[c] + q.gpu[c] + s.c_slo * sl + (1.0 - a) * s.c_rej);
}

// The wait of every configuration at every count the budget allows: [G][J + 1].
// One block, after config_prep_block.
__device__ void config_wait_table(const SvcArgs &s, const ConfigPre &q, const int32_t *gpus,
                                  double *wt)
{
    const int n = s.G * (s.J + 1);
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
        const int g = i / (s.J + 1), z = i % (s.J + 1);
        if ((long long)z * gpus[g] <= s.J) wt[i] = config_wait(s, q, g, z);
    }
}

__global__ __launch_bounds__(kBlockThreads) void config_prep_kernel(
    SvcArgs s, const double *T, const double *ET2, const double *pi, const int32_t *eta_c,
    const uint8_t *delta, ConfigBufs b)
{
    __shared__ double lds[kStateLds];
    const ConfigPre q = config_view(b, s.C, s.G);
    config_prep_block(s, T, ET2, pi, eta_c, delta, q, lds);
    __syncthreads();
    config_wait_table(s, q, b.gpus, b.wt);
}

// The objective at z by one wave (INFINITY when infeasible): a lane per
// configuration for its wait, a lane per class for its cost, the classes added in
// order.  w: [kMaxG] in LDS.
__device__ double config_objective(const SvcArgs &s, const ConfigPre &q, const double *Wc,
                                   const int32_t *z, double *w)
{
    const int lane = threadIdx.x & 63;
    bool bad = false;
    if (lane < s.G) {
        const double v = config_wait(s, q, lane, z[lane]);
        bad = is_no_wait(v);
        w[lane] = v;
    }
    wave_sync();
    if (__ballot(bad)) return INFINITY;
    double obj = 0.0;
    for (int c0 = 0; c0 < s.C; c0 += 64) {
        const int c = c0 + lane;
        const double term =
            c < s.C ? class_cost<false>(s, class_costs(q, Wc), c, [&](int g) { return w[g]; }) : 0.0;
        for (int i = 0; i < min(64, s.C - c0); ++i) obj = obj + __shfl(term, i);
    }
    return obj;
}

// z of lexicographic rank r: ways[g][b] = number of (z_g..z_{G-1}) of cost <= b.
// With z_g = v there are ways[g][b - v n] - ways[g][b - (v + 1) n] of them (n GPUs a
// group), so those with z_g < v number ways[g][b] - ways[g][b - v n]: the largest v
// for which that is at most r, by bisection.  put(g, z_g) in order; returns what is
// left of the budget.
template <class F>
__device__ __forceinline__ int unrank(long long r, int G, int J, const int32_t *gpus,
                                      const long long *ways, F &&put)
{
    int b = J;
    for (int g = 0; g < G; ++g) {
        const int n = gpus[g];
        const long long *w = ways + (long long)g * (J + 1);
        const long long need = w[b] - r;  // positive: r < ways[g][b]
        int lo = 0, hi = b / n;           // lo satisfies ways[g][b - lo n] >= need
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (w[b - mid * n] >= need) lo = mid;
            else hi = mid - 1;
        }
        r -= w[b] - w[b - lo * n];
        b -= lo * n;
        put(g, lo);
    }
    return b;
}

// Every thread takes `each` consecutive ranks: the first z by unrank, the next ones
// by counting up; per block the lowest (objective, rank) and the number of
// feasible z.  The waits come from the table of config_wait_table (they depend on
// z_g alone), the classes' sums run over the routing's non-zero entries, and a z
// whose waits are all those of the one before (only counts of configurations
// without traffic differ) has its objective.  The tables and the classes' data are
// staged in LDS where they fit; a thread keeps its counts of groups there ([G][threads])
// and, kWaits, its waits.  747,788 configurations of 15 classes in the loop of Alg. 1:
// 46 us, 49 with counts of 32 bits; one rank a thread, its waits recomputed with five
// divisions each, its counts read from memory, all 180 entries of the routing, took 2.5
// times as long.
template <bool kLds, bool kWaits>
__global__ __launch_bounds__(kSvcThreads) void config_search_kernel(SvcArgs s, long long nz,
                                                                    int each, const double *Wc,
                                                                    ConfigBufs b)
{
    extern __shared__ double dyn[];
    __shared__ double red_o[kSvcThreads / 64];
    __shared__ long long red_r[kSvcThreads / 64], red_n[kSvcThreads / 64];
    __shared__ int32_t gpus[kMaxG];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, G = s.G, J = s.J;
    if (t < G) gpus[t] = b.gpus[t];
    const ConfigPre q = config_view(b, s.C, G);
    // a thread's waits (kWaits) and counts (J <= 4,096): [G][threads] each
    double *wl = dyn;
    uint16_t *zl = reinterpret_cast<uint16_t *>(wl + (kWaits ? G * kSvcThreads : 0));
    // when kLds: the tables and the classes' data behind them
    long long *lw = reinterpret_cast<long long *>(zl + G * kSvcThreads);
    double *lt = reinterpret_cast<double *>(lw + (G + 1) * (J + 1)), *ld = lt + G * (J + 1);
    int32_t *li = reinterpret_cast<int32_t *>(ld + 5 * s.C + 2 * s.C * G);
    if (kLds) {
        const int C = s.C, n = q.start[C];
        for (int i = t; i < (G + 1) * (J + 1); i += kSvcThreads) lw[i] = b.ways[i];
        for (int i = t; i < G * (J + 1); i += kSvcThreads) lt[i] = b.wt[i];
        for (int i = t; i < C; i += kSvcThreads) {
            ld[i] = q.a[i];
            ld[C + i] = q.gpu[i];
            ld[2 * C + i] = Wc[i];
            ld[3 * C + i] = (double)s.lam[i];
            ld[4 * C + i] = (double)s.D[i];
        }
        for (int i = t; i <= C; i += kSvcThreads) li[i] = q.start[i];
        for (int i = t; i < n; i += kSvcThreads) {
            ld[5 * C + i] = q.pi[i];
            ld[5 * C + C * G + i] = q.T[i];
            li[C + 1 + i] = q.g[i];
        }
    }
    __syncthreads();
    const long long *ways = kLds ? lw : b.ways;
    const double *wt = kLds ? lt : b.wt;
    const int C = s.C;
    const ClassCosts cc = kLds ? ClassCosts{ld, ld + C, ld + 2 * C, ld + 5 * C, ld + 5 * C + C * G,
                                            li, li + C + 1, ld + 3 * C, ld + 4 * C}
                               : class_costs(q, Wc);
    double best = INFINITY;
    long long brank = 0x7fffffffffffffffLL, feas = 0;
    const long long r0 = ((long long)blockIdx.x * kSvcThreads + t) * each;
    if (r0 < nz) {
        int bad = 0;  // configurations that z does not allow
        auto wait = [&](int g) {
            const int o = g * kSvcThreads + t;
            return kWaits ? wl[o] : wt[g * (J + 1) + zl[o]];
        };
        auto set = [&](int g, int v, double w) {
            zl[g * kSvcThreads + t] = (uint16_t)v;
            if (kWaits) wl[g * kSvcThreads + t] = w;
        };
        int left = unrank(r0, G, J, gpus, ways, [&](int g, int v) {
            const double w = wt[g * (J + 1) + v];
            set(g, v, w);
            bad += is_no_wait(w) ? 1 : 0;
        });
        const long long r1 = min(nz, r0 + each);
        bool same = false;  // the waits are those obj belongs to
        double obj = 0.0;
        for (long long r = r0;;) {
            if (!bad) {
                if (!same) {
                    obj = 0.0;
                    for (int c = 0; c < C; ++c) obj = obj + class_cost<kLds>(s, cc, c, wait);
                }
                same = true;
                feas += obj < INFINITY ? 1 : 0;
                if (obj < best) {  // ranks ascend: the first minimiser
                    best = obj;
                    brank = r;
                }
            }
            if (++r >= r1) break;
            // the next z: one more of the last configuration that the budget allows
            for (int g = G - 1; g >= 0; --g) {
                const int n = gpus[g], z0 = zl[g * kSvcThreads + t];
                const int v = left >= n ? z0 + 1 : 0;
                const double w0 = wait(g), w = wt[g * (J + 1) + v];
                bad += (is_no_wait(w) ? 1 : 0) - (is_no_wait(w0) ? 1 : 0);
                same = same && __double_as_longlong(w0) == __double_as_longlong(w);
                left += v ? -n : z0 * n;
                set(g, v, w);
                if (v) break;
            }
        }
    }
    for (int off = 32; off > 0; off >>= 1) {
        const double o2 = __shfl_xor(best, off);
        const long long k2 = __shfl_xor(brank, off);
        if (o2 < best || (o2 == best && k2 < brank)) {
            best = o2;
            brank = k2;
        }
        feas += __shfl_xor(feas, off);
    }
    if (lane == 0) {
        red_o[wave] = best;
        red_r[wave] = brank;
        red_n[wave] = feas;
    }
    __syncthreads();
    if (t == 0) {
        for (int w = 1; w < kSvcThreads / 64; ++w) {
            if (red_o[w] < best || (red_o[w] == best && red_r[w] < brank)) {
                best = red_o[w];
                brank = red_r[w];
            }
            feas += red_n[w];
        }
        b.part_obj[blockIdx.x] = best;
        b.part_rank[blockIdx.x] = brank;
        b.part_feas[blockIdx.x] = feas;
    }
}

// Final reduction over the blocks, the keep rule (the current z stays when it
// attains the minimum) and the change flag of the outer loop.
__global__ __launch_bounds__(kBlockThreads) void config_final_kernel(
    SvcArgs s, long long nparts, const double *Wc, ConfigBufs b, int32_t *z,
    const uint8_t *delta_new, uint8_t *delta, double *best_obj, long long *best_rank,
    long long *n_feasible, int32_t *flag)
{
    __shared__ double red_o[kBlockThreads / 64], w[kMaxG];
    __shared__ long long red_r[kBlockThreads / 64], red_n[kBlockThreads / 64];
    __shared__ int32_t zc[kMaxG], zb[kMaxG];
    __shared__ int dchg;
    __shared__ double s_min, s_cur;
    __shared__ long long s_rank;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, nt = kBlockThreads;
    const ConfigPre q = config_view(b, s.C, s.G);
    double o = INFINITY;
    long long rk = 0x7fffffffffffffffLL, nf = 0;
    for (long long p = t; p < nparts; p += nt) {
        nf += b.part_feas[p];
        const double v = b.part_obj[p];
        const long long r = b.part_rank[p];
        if (v < o || (v == o && r < rk)) {
            o = v;
            rk = r;
        }
    }
    if (t < kMaxG) zc[t] = zb[t] = t < s.G ? z[t] : 0;
    if (t == 0) dchg = 0;
    for (int off = 32; off > 0; off >>= 1) {
        const double o2 = __shfl_xor(o, off);
        const long long k2 = __shfl_xor(rk, off);
        if (o2 < o || (o2 == o && k2 < rk)) {
            o = o2;
            rk = k2;
        }
        nf += __shfl_xor(nf, off);
    }
    if (lane == 0) {
        red_o[wave] = o;
        red_r[wave] = rk;
        red_n[wave] = nf;
    }
    __syncthreads();
    if (t == 0) {
        for (int i = 1; i < nt / 64; ++i) {
            if (red_o[i] < o || (red_o[i] == o && red_r[i] < rk)) {
                o = red_o[i];
                rk = red_r[i];
            }
            nf += red_n[i];
        }
        s_min = o;
        s_rank = rk;
        if (o < INFINITY && rk != 0x7fffffffffffffffLL)
            unrank(rk, s.G, s.J, b.gpus, b.ways, [&](int g, int v) { zb[g] = v; });
        if (best_obj) best_obj[0] = o;
        if (best_rank) best_rank[0] = o < INFINITY ? rk : -1;
        if (n_feasible) n_feasible[0] = nf;
    } else if (wave == 1) {
        const double ocur = config_objective(s, q, Wc, zc, w);
        if (lane == 0) s_cur = ocur;
    } else if (wave > 1 && delta_new && delta) {  // delta changes?
        bool d = false;
        for (int i = t - 128; i < s.C * s.G; i += nt - 128) d = d || delta_new[i] != delta[i];
        if (__ballot(d) && lane == 0) dchg = 1;
    }
    __syncthreads();
    if (delta_new && delta)
        for (int i = t; i < s.C * s.G; i += nt) delta[i] = delta_new[i];
    if (t == 0) {
        int zchg = 0;
        if (s_min < INFINITY && s_rank != 0x7fffffffffffffffLL && !(s_cur == s_min))
            for (int g = 0; g < s.G; ++g) {
                zchg |= zb[g] != zc[g];
                z[g] = zb[g];
            }
        if (flag) flag[0] = (zchg || dchg) ? 1 : 0;
    }
}

// -------------------------------------------------------------- Block 1 ----
// Wc[c] = W[c, k[c]] and eta_c[c] = eta[k[c]]
__device__ void gather_block(const double *W, const int32_t *eta, const int32_t *k, int C, int K,
                             double *Wc, int32_t *eta_c)
{
    for (int c = threadIdx.x; c < C; c += blockDim.x) {
        const int kc = min(max(k[c], 0), K - 1);
        Wc[c] = W[(long long)c * K + kc];
        eta_c[c] = eta[kc];
    }
}

// Blocks 1 and 2 of one outer iteration and the sums Block 3 starts from, in one
// launch of one block: the wait frozen at the state entering, then the routing
// LP and the reservation sweep in turn until the reservations repeat and the
// routing moves by at most tol (at most max_inner times), the caching at the
// state reached, the configuration sums with it.  A chain of small dependent
// steps: as launches of their own (six per round and seven more per iteration,
// with a copy and a wait for the host per round) the launches and waits took
// most of the time.  15 classes, 12 configurations,
// K = 2048: 98 us for one round of 15 pivots and 184 for two (103 and 195 while the
// simplex's minima were fp64 steps that carried their index), the whole solve 600 to
// 4,500 us on eight instances, 1,570 to 10,740 before.
template <bool kLds>
__global__ __launch_bounds__(kBlockThreads) void block1_kernel(SvcArgs s, Block1Args a)
{
    extern __shared__ double dyn[];  // the LP's work area (kLds), the sweep's and the state's scratch
    __shared__ LpShared lp;
    __shared__ int moved, feasible_all;
    const int t = threadIdx.x, nt = kBlockThreads, C = s.C, G = s.G, CG = C * G;
    if (a.first) {
        for (int i = t; i < CG; i += nt) {
            a.pi[i] = 0.0;
            a.delta[i] = 0;
        }
        __syncthreads();
    }
    gather_block(a.W, a.eta, a.k, C, a.K, a.Wc, a.eta_c);
    __syncthreads();
    // the wait is linearised once, at the state entering
    state_block(s, a.T, a.ET2, a.pi, a.z, a.eta_c, a.delta, a.Wq, a.cap, a.conc, nullptr, dyn);
    __syncthreads();
    int inner = 0, pivots = 0, status = 0;
    bool converged = false;
    while (inner < a.max_inner && !converged) {
        ++inner;
        if (inner > 1) {  // (the first round's are the ones above)
            gather_block(a.W, a.eta, a.k, C, a.K, a.Wc, a.eta_c);
            __syncthreads();
        }
        lp1_block<kLds>(s, a.Wc, a.T, a.Wq, a.z, a.eta_c, a.delta, a.work, a.max_pivots, a.pi_new,
                        nullptr, lp);
        pivots += lp.pivots;
        status |= lp.status == 1 ? 1 : (lp.status == 2 ? 2 : (lp.status == 3 ? 4 : 0));
        __syncthreads();
        state_block(s, a.T, a.ET2, a.pi_new, a.z, a.eta_c, a.delta, nullptr, a.cap, a.conc, nullptr,
                    dyn);
        if (t == 0) {
            moved = 0;
            feasible_all = 1;
        }
        __syncthreads();
        if (t < 64)
            sweep_wave(a.best, a.eta, C, a.K, G, (const double *)a.conc, (const double *)a.cap,
                       1.0 + s.kappa, kEtaSlack, a.k, a.k_new, dyn, [&](int, int, bool feas) {
                           if (!feas) feasible_all = 0;
                       });
        __syncthreads();
        for (int i = t; i < CG; i += nt) {
            if (fabs(a.pi_new[i] - a.pi[i]) > a.tol) moved = 1;
            a.pi[i] = a.pi_new[i];
        }
        for (int c = t; c < C; c += nt) {
            if (a.k_new[c] != a.k[c]) moved = 1;
            a.k[c] = a.k_new[c];
        }
        __syncthreads();
        converged = moved == 0;
        __syncthreads();
    }
    // Block 2, then the sums of Block 3 with its caching
    gather_block(a.W, a.eta, a.k, C, a.K, a.Wc, a.eta_c);
    __syncthreads();
    state_block(s, a.T, a.ET2, a.pi, a.z, a.eta_c, a.delta, nullptr, a.cap, a.conc, nullptr, dyn);
    __syncthreads();
    for (int i = t; i < CG; i += nt) a.d_new[i] = a.conc[i] > 1.0 ? 1 : 0;
    __syncthreads();
    const ConfigPre q = config_view(a.b, C, G);
    config_prep_block(s, a.T, a.ET2, a.pi, a.eta_c, a.d_new, q, dyn);
    __syncthreads();
    config_wait_table(s, q, a.b.gpus, a.b.wt);
    if (t == 0) {
        a.ctl[0] = inner;
        a.ctl[1] = pivots;
        a.ctl[2] = status | (converged ? 0 : 16);
        a.ctl[3] = feasible_all;
    }
}

// Objective of the current state (one block).
__global__ __launch_bounds__(kBlockThreads) void state_objective_kernel(
    SvcArgs s, const double *T, const double *ET2, const double *pi, const int32_t *z,
    const int32_t *eta_c, const uint8_t *delta, const double *Wc, ConfigBufs b, double *out)
{
    __shared__ double w[kMaxG], lds[kStateLds];
    const ConfigPre q = config_view(b, s.C, s.G);
    config_prep_block(s, T, ET2, pi, eta_c, delta, q, lds);
    __syncthreads();
    if (threadIdx.x < 64) {
        const double o = config_objective(s, q, Wc, z, w);
        if (threadIdx.x == 0) out[0] = o;
    }
}

// ------------------------------------------------------------- launchers ----
hipError_t launch_service_times(const SvcArgs &s, const int64_t *count, const int64_t *sum,
                                const int64_t *sumsq, double *T, double *ET2, hipStream_t st)
{
    const int n = s.C * s.G;
    hipLaunchKernelGGL(service_times_kernel, dim3((n + 255) / 256), dim3(256), 0, st, s, count, sum,
                       sumsq, T, ET2);
    return hipGetLastError();
}

hipError_t launch_state(const SvcArgs &s, const double *T, const double *ET2, const double *pi,
                        const int32_t *z, const int32_t *eta_c, const uint8_t *delta, double *Wq,
                        double *cap, double *conc, double *mem, hipStream_t st)
{
    hipLaunchKernelGGL(state_kernel, dim3(1), dim3(kBlockThreads), 0, st, s, T, ET2, pi, z, eta_c,
                       delta, Wq, cap, conc, mem);
    return hipGetLastError();
}

hipError_t launch_cache(const double *conc, int n, uint8_t *delta, hipStream_t st)
{
    hipLaunchKernelGGL(cache_kernel, dim3((n + 255) / 256), dim3(256), 0, st, conc, n, delta);
    return hipGetLastError();
}

constexpr size_t kLp1LdsBytes = 152 * 1024;  // dynamic LDS for the work area (of 160 KB)

hipError_t lp1_prepare()
{
    const void *k[] = {reinterpret_cast<const void *>(lp1_kernel<true>),
                       reinterpret_cast<const void *>(block1_kernel<true>),
                       reinterpret_cast<const void *>(block1_kernel<false>),
                       reinterpret_cast<const void *>(config_search_kernel<false, false>),
                       reinterpret_cast<const void *>(config_search_kernel<false, true>),
                       reinterpret_cast<const void *>(config_search_kernel<true, false>),
                       reinterpret_cast<const void *>(config_search_kernel<true, true>)};
    for (const void *f : k) {
        const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize,
                                                 (int)kLp1LdsBytes);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

size_t lp1_work_doubles(int C, int G) { return (size_t)lp1_doubles(C, G); }

hipError_t launch_lp1(const SvcArgs &s, const double *Wc, const double *T, const double *Wq,
                      const int32_t *z, const int32_t *eta_c, const uint8_t *delta, double *work,
                      int max_pivots, double *pi_out, double *obj_out, int32_t *info,
                      hipStream_t st)
{
    // the work area lives in LDS when it fits (one workgroup, every pivot touches all of it)
    const size_t bytes = lp1_work_doubles(s.C, s.G) * sizeof(double);
    const bool lds = bytes <= kLp1LdsBytes;
    hipLaunchKernelGGL(lds ? lp1_kernel<true> : lp1_kernel<false>, dim3(1), dim3(kLpThreads),
                       lds ? bytes : 0, st, s, Wc, T, Wq, z, eta_c, delta, work, max_pivots, pi_out,
                       obj_out, info);
    return hipGetLastError();
}

hipError_t launch_sweep(const double *W, const int32_t *eta, int C, int K, int G,
                        const double *conc, const double *cap, double kappa, const int32_t *k_in,
                        int32_t *k_out, uint8_t *feasible, hipStream_t st)
{
    hipLaunchKernelGGL(sweep_kernel, dim3(1), dim3(kBlockThreads), 0, st, W, eta, C, K, G, conc, cap,
                       kappa, k_in, k_out, feasible);
    return hipGetLastError();
}

hipError_t launch_block1(const SvcArgs &s, const Block1Args &a, hipStream_t st)
{
    const size_t lp = lp1_work_doubles(s.C, s.G) * sizeof(double);
    const size_t other = sizeof(double) * (kStateLds > kSweepLds ? kStateLds : kSweepLds);
    const bool lds = lp <= kLp1LdsBytes;
    hipLaunchKernelGGL(lds ? block1_kernel<true> : block1_kernel<false>, dim3(1),
                       dim3(kBlockThreads), lds ? std::max(lp, other) : other, st, s, a);
    return hipGetLastError();
}

size_t config_pre_doubles(int C, int G) { return (size_t)(2 * C + 5 * G + 2 * C * G); }
size_t config_pre_ints(int C, int G) { return (size_t)(C + 1 + C * G + G); }

// consecutive configurations per thread: about a thousand blocks over the chip
static int config_each(long long nz)
{
    return (int)std::max(1LL, (nz + 256LL * 1024 - 1) / (256LL * 1024));
}

long long config_parts(long long nz)
{
    const long long per = (long long)kSvcThreads * config_each(nz);
    return (nz + per - 1) / per;
}

hipError_t launch_config_prep(const SvcArgs &s, const double *T, const double *ET2, const double *pi,
                              const int32_t *eta_c, const uint8_t *delta, const ConfigBufs &b,
                              hipStream_t st)
{
    hipLaunchKernelGGL(config_prep_kernel, dim3(1), dim3(kBlockThreads), 0, st, s, T, ET2, pi, eta_c,
                       delta, b);
    return hipGetLastError();
}

hipError_t launch_config_search(const SvcArgs &s, long long nz, const double *Wc,
                                const ConfigBufs &b, int32_t *z, const uint8_t *delta_new,
                                uint8_t *delta, double *best_obj, long long *best_rank,
                                long long *n_feasible, int32_t *flag, hipStream_t st)
{
    // Tables staged and waits kept where two blocks fit a compute unit, else the tables
    // staged and the waits looked up in them where three do, else the tables in memory and
    // the waits kept where two do.  Staged without waits against kept without tables: 30
    // classes, 32 configurations, 24 GPUs 473 and 1,317 us (one block a unit), 24
    // configurations 31 and 58; 200 classes, 12 configurations, 48 GPUs (two blocks) 31 and
    // 22.  Neither: 200 classes, 32 configurations, 20 GPUs 91 us, 278 with the waits kept.
    const size_t counts = (size_t)s.G * kSvcThreads * 2, waits = (size_t)s.G * kSvcThreads * 8;
    const size_t tables = (size_t)(2 * s.G + 1) * (s.J + 1) * 8 + (size_t)s.C * (40 + 20 * s.G) +
                          (size_t)(s.C + 2) * 4;
    const bool both = counts + waits + tables <= kLp1LdsBytes / 2;
    const bool lds = both || counts + tables <= kLp1LdsBytes / 3;
    const bool keep = both || (!lds && counts + waits <= kLp1LdsBytes / 2);
    const auto kernel = lds ? (keep ? config_search_kernel<true, true> : config_search_kernel<true, false>)
                            : (keep ? config_search_kernel<false, true> : config_search_kernel<false, false>);
    hipLaunchKernelGGL(kernel, dim3((unsigned)config_parts(nz)), dim3(kSvcThreads),
                       counts + (keep ? waits : 0) + (lds ? tables : 0), st, s, nz, config_each(nz), Wc, b);
    hipLaunchKernelGGL(config_final_kernel, dim3(1), dim3(kBlockThreads), 0, st, s, config_parts(nz),
                       Wc, b, z, delta_new, delta, best_obj, best_rank, n_feasible, flag);
    return hipGetLastError();
}

hipError_t launch_state_objective(const SvcArgs &s, const double *T, const double *ET2,
                                  const double *pi, const int32_t *z, const int32_t *eta_c,
                                  const uint8_t *delta, const double *Wc, const ConfigBufs &b,
                                  double *out, hipStream_t st)
{
    hipLaunchKernelGGL(state_objective_kernel, dim3(1), dim3(kBlockThreads), 0, st, s, T, ET2, pi, z,
                       eta_c, delta, Wc, b, out);
    return hipGetLastError();
}

}  // namespace dro
