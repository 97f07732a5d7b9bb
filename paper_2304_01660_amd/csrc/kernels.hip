// HIP kernels (gfx950) of the range-discord search.
//
// Method (paper): for each length m, per-subsequence mean/sigma by the
// recurrences of Eq. (7)-(8) (Sec. 3.1.1); a selection pass that drops every
// subsequence having a non-self match closer than r, scanning to the right of
// each row tile (Sec. 3.2, after phase 1 of Alg. 2); a refinement pass that
// computes the exact nearest-neighbour distance of the survivors and drops
// those closer than r (Sec. 3.3, phase 2 of Alg. 2); MERLIN's choice of r per
// length (Alg. 1).  Distances use the Pearson form of Eq. (6):
// ED^2 = 2m(1 - rho), rho = C_ij / (m sigma_i sigma_j) with C_ij the centred
// covariance of the two windows.
//
// MI355X mapping:
//   * A sweep work item is one wavefront owning a tile of R = 64*Q
//     consecutive rows (Q per lane) and a run of columns.  Along a column
//     step every row takes the value of its upper-left neighbour (Eq. (10)'s
//     diagonal update, here on the centred covariance:
//     C(i,j) = C(i-1,j-1) + df[i-1]*dg[j-1] + df[j-1]*dg[i-1]), so a lane's
//     Q rows shift inside registers and one DPP wave_shr moves the last row
//     into the next lane.  Lane 0's top row is taken from exact FP64 dot
//     products computed 64 columns at a time, so every value is at most R
//     recurrence steps from an exact one.
//   * Each block of 64 columns is staged in LDS with one burst of loads: the
//     T segment (for the boundary dot products) and, per step, the column
//     helpers df, dg, 1/(sqrt(m) sigma) and the boundary value, all read as
//     one broadcast record.
//   * Row and column prunes are lane masks; a column prune is one ballot per
//     step, flushed to the candidate bitmap every 64 columns with one atomic.
//   * Long scans are split into column chunks fed from a device work list in
//     nearest-first order, so the critical path is one chunk, not one row.
//   * Most range searches sweep nothing: every row carries the neighbour that
//     pruned it to the next length (k_advance, k_rescue), and the few rows left
//     are bounded against every column on the FP16 matrix cores (k_screen) and
//     decided in FP64 (k_exact).  Where thousands of rows are left, k_dense
//     bounds them in the same way.
//   * Every kernel serves a batch of series: flat block indices map to
//     (series, block) through host-built prefix tables, the queued passes
//     drain each series' work list in turn, and all per-series geometry and
//     MERLIN state is read from device descriptors.
#include "engine.h"

#include <math.h>

#include <algorithm>
#include <type_traits>

namespace palmad {

// ---------------------------------------------------------------------------
// small helpers
// ---------------------------------------------------------------------------
constexpr int DPP_WAVE_SHR1 = 0x138;  // lane l <- lane l-1
constexpr int DPP_WAVE_ROL1 = 0x134;  // lane l <- lane l+1 (63 <- 0)

template <typename F>
__device__ __forceinline__ F f_inf();
template <>
__device__ __forceinline__ float f_inf<float>() { return __int_as_float(0x7f800000); }
template <>
__device__ __forceinline__ double f_inf<double>() { return __longlong_as_double(0x7ff0000000000000ll); }

// A margin no pair reaches (finite, so that its low bits can carry a step
// index: infinity with low bits set would be a NaN).
template <typename F>
__device__ __forceinline__ F f_low();
template <>
__device__ __forceinline__ float f_low<float>() { return -3.0e38f; }
template <>
__device__ __forceinline__ double f_low<double>() { return -1.0e300; }

// v with its six lowest mantissa bits replaced by the step index s < 64: the
// largest such value of a block tells the step it came from, for one extra
// instruction per pair.
__device__ __forceinline__ float pack_step(float v, int s)
{
    return __int_as_float((__float_as_int(v) & ~63) | s);
}
__device__ __forceinline__ double pack_step(double v, int s)
{
    return __longlong_as_double((__double_as_longlong(v) & ~63ll) | (long long)s);
}
__device__ __forceinline__ int step_of(float v) { return __float_as_int(v) & 63; }
__device__ __forceinline__ int step_of(double v) { return (int)(__double_as_longlong(v) & 63ll); }

__device__ __forceinline__ float f_fma(float a, float b, float c) { return fmaf(a, b, c); }
__device__ __forceinline__ double f_fma(double a, double b, double c) { return fma(a, b, c); }

// lane l <- src of lane l-1; lane 0 <- old of lane 0
__device__ __forceinline__ float dpp_shr1(float old, float src)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(old), __float_as_int(src),
                                                      DPP_WAVE_SHR1, 0xf, 0xf, false));
}
__device__ __forceinline__ double dpp_shr1(double old, double src)
{
    const long long o = __double_as_longlong(old), s = __double_as_longlong(src);
    const int lo = __builtin_amdgcn_update_dpp((int)o, (int)s, DPP_WAVE_SHR1, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp((int)(o >> 32), (int)(s >> 32), DPP_WAVE_SHR1, 0xf,
                                               0xf, false);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
// lane l <- lane l+1, lane 63 <- lane 0
__device__ __forceinline__ float dpp_rol1(float v)
{
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), DPP_WAVE_ROL1, 0xf, 0xf, false));
}
__device__ __forceinline__ double dpp_rol1(double v)
{
    const long long s = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_mov_dpp((int)s, DPP_WAVE_ROL1, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_mov_dpp((int)(s >> 32), DPP_WAVE_ROL1, 0xf, 0xf, false);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

__device__ __forceinline__ unsigned long long ord_of(double d)
{
    const unsigned long long u = (unsigned long long)__double_as_longlong(d);
    return (u >> 63) ? ~u : (u | 0x8000000000000000ull);
}
__device__ __forceinline__ double dbl_of(unsigned long long u)
{
    return (u >> 63) ? __longlong_as_double((long long)(u & 0x7fffffffffffffffull))
                     : __longlong_as_double((long long)~u);
}

// Values identical in every lane, made explicit so the compiler keeps them
// (and everything derived from them) in scalar registers.
__device__ __forceinline__ unsigned long long uniform64(unsigned long long v)
{
    const unsigned int lo = __builtin_amdgcn_readfirstlane((unsigned int)v);
    const unsigned int hi = __builtin_amdgcn_readfirstlane((unsigned int)(v >> 32));
    return ((unsigned long long)hi << 32) | lo;
}
__device__ __forceinline__ int64_t uniform_i64(int64_t v) { return (int64_t)uniform64((unsigned long long)v); }

__device__ __forceinline__ unsigned long long load_word(const unsigned long long* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ unsigned int load_flag(const uint32_t* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

__device__ double block_sum(double v, double* sh)
{
    v = wave_sum(v);
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    if (l == 0) sh[w] = v;
    __syncthreads();
    double t = 0.0;
    if (threadIdx.x == 0)
        for (int i = 0; i < (int)(blockDim.x >> 6); ++i) t += sh[i];
    __syncthreads();
    return t;  // valid in thread 0
}

// Number of (row, column) pairs with rows in [ilo, ihi) and columns in
// [j0, j0+ns) that are non-self matches on the given side:
//   right side: j >= i + m;   left side: j <= i - m.
__device__ __forceinline__ unsigned long long pair_count(long long ilo, long long ihi, long long j0,
                                                         long long ns, long long m, bool left)
{
    if (ihi <= ilo || ns <= 0) return 0;
    unsigned long long tot = 0;
    if (!left) {
        // row i sees clamp(E - i, 0, ns) columns, E = j0 + ns - m
        const long long E = j0 + ns - m;
        const long long full_hi = min(ihi, E - ns + 1);  // i <= E - ns  -> ns columns
        if (full_hi > ilo) tot += (unsigned long long)(full_hi - ilo) * (unsigned long long)ns;
        const long long p = max(ilo, E - ns + 1), q = min(ihi, E);
        if (q > p) tot += (unsigned long long)((2 * E - p - q + 1) * (q - p) / 2);
    } else {
        // row i sees clamp(i - G, 0, ns) columns, G = j0 + m - 1
        const long long G = j0 + m - 1;
        const long long full_lo = max(ilo, G + ns);      // i >= G + ns -> ns columns
        if (ihi > full_lo) tot += (unsigned long long)(ihi - full_lo) * (unsigned long long)ns;
        const long long p = max(ilo, G + 1), q = min(ihi, G + ns);
        if (q > p) tot += (unsigned long long)((p + q - 1 - 2 * G) * (q - p) / 2);
    }
    return tot;
}

// ---------------------------------------------------------------------------
// round preparation: MERLIN's walk over the lengths and its choice of r
// (Alg. 1)
// ---------------------------------------------------------------------------
// Guard band of the FP32 selection sweep.  An FP32 correlation drifts from
// the exact one by rounding: the centred recurrence accumulates one rounding
// of the covariance per step over chains of at most R_MAX - 1 steps, and a
// pair's covariance is divided by m sigma_i sigma_j, so windows with a small
// spread next to windows with a large one (within the R_MAX windows a chain
// passes) amplify the covariance's absolute error.  With gamma the largest
// ratio of the nearby largest spread to a window's own spread, the drift
// measured on the device (k_drift, thousands of sampled 512-row tiles, and
// every tile of the smaller series) over the configured workloads stays
// below
//     2^-24 * sqrt(R_MAX) * gamma^2
// (random walks, ECG-like series; ECG-like beats between quiet baselines
// come closest); the band is four times that, and never below the caller's
// guard (default 1.25e-4).  A series with an extreme spread contrast thus
// gets a wide band (the selection sweep prunes less, the FP64 refinement
// decides), never an unsound one.
constexpr double WIDE_BAND = 0.01;  // more rows within it of the k-th best than are candidates
constexpr double GUARD_PER_CONTRAST2 = 4.0 * 0x1p-24 * 22.62741699796952;  // 4 u sqrt(512)

__device__ __forceinline__ double sel_guard(const Ctrl* c, float guard)
{
    if (guard <= 0.0f) return 0.0;  // FP64 selection sweep: no band
    const double gc = GUARD_PER_CONTRAST2 * c->gam2;
    return gc > (double)guard ? gc : (double)guard;
}

__device__ __forceinline__ void set_sel_thresholds(Ctrl* c, float guard)
{
    c->thr_sel = c->thr64 + sel_guard(c, guard);
    // round up: an FP32 threshold must never prune more than thr_sel
    c->thr32 = __double2float_ru(c->thr_sel);
}

// A round that bounds every row left, by a short first pass (DENSE_SWEEP) or by
// the witnesses (DENSE_LEFT), instead of sweeping on (see k_dense).
// DENSE_OFF: not at this length; DENSE_NEVER: not again in this call (the bounds
// of this series decide too little).
enum { DENSE_NO = 0, DENSE_SWEEP, DENSE_OFF, DENSE_LEFT, DENSE_NEVER };
__device__ __forceinline__ bool dense_round(const Ctrl* c)
{
    return c->dense == DENSE_SWEEP || c->dense == DENSE_LEFT;
}
__device__ __forceinline__ bool dense_off(const Ctrl* c)
{
    return c->dense == DENSE_OFF || c->dense == DENSE_NEVER;
}
// Columns of the short first pass: most rows of the second range (r = sqrt(m))
// fall within a few thousand columns where they fall at all; from the third
// range on a good part never does.
__device__ __forceinline__ int dense_near(const Ctrl* c) { return c->attempt == 1 ? DENSE_NEAR : 2048; }
// Rows x columns x m above which rows left by the witnesses get a first pass
// before they are bounded (about half a millisecond of k_dense; a million
// points took 48.9 ms without this rule, 28.7 without dense rounds, 25.6 so).
constexpr double DENSE_LEFT_WORK = 2.5e11;
constexpr double DENSE_MIN_THR = 0.2;  // smallest threshold of a dense round

// Candidates of a dense round: those whose bounds do not tell them from the k
// best, usually some hundred, on a noisy series a few thousand.  More than
// CAND_MAX go through the exact pass in parts, each with the k best so far; a
// part costs 0.1 ms at 20,000 points and 0.4 at 500,000, the same range again
// with sweeps 0.5 and 20 to 90.
__device__ __forceinline__ unsigned int dense_cands(int64_t N)
{
    return (unsigned int)CAND_MAX * (unsigned int)std::min<int64_t>(16, std::max<int64_t>(2, N / 32768));
}
// The round goes on with the next part of its candidates, and does nothing else.
__device__ __forceinline__ bool taking_parts(const Ctrl* c) { return c->cand_at > 0; }

__device__ void begin_range(const SeriesDev& s, Ctrl* c, float guard)
{
    const int li = c->li;
    const int32_t m = c->m;
    if (c->attempt == 0 && c->mode != 3) {
        if (li == 0) {
            c->mode = 0;
            c->r = 2.0 * sqrt((double)s.minL);
        } else if (li <= 4) {
            c->mode = 1;
            c->r = 0.99 * s.hist[li - 1];
        } else {
            double mean = 0.0;
            for (int q = 1; q <= 5; ++q) mean += s.hist[li - q];
            mean /= 5.0;
            double v = 0.0;
            for (int q = 1; q <= 5; ++q) {
                const double d = s.hist[li - q] - mean;
                v += d * d;
            }
            c->step = sqrt(v / 5.0);
            c->r = mean - 2.0 * c->step;
            c->mode = 2;
        }
    }
    const double r = c->r;
    c->prune = r > 0.0 ? 1 : 0;
    c->thr64 = r > 0.0 ? 1.0 - r * r / (2.0 * (double)m) : 2.0;
    // a new length's contrast is measured by k_helpers and k_guard, which
    // then resets the selection thresholds; a repeat keeps the current length's
    if (c->new_len) c->gam2 = 0.0;
    set_sel_thresholds(c, guard);
    c->nlive_sel = c->maxc_sel = 0;
    c->nlive_ref = c->maxc_ref = 0;
    c->nsurv = 0;
    c->ncand = 0;
    c->live_ref = 0;
    c->nlive = 0;
    c->band_over = 0;
    // Most rows the exact pass takes without a sweep: its screening costs
    // about 4e-12 s per row and column (1e6 columns: 4 us per row), a round of
    // sweeps 250-400 us.
    const int64_t N = s.n - m + 1;
    c->lean_max = (uint32_t)std::min<int64_t>(CAND_MAX, std::max<int64_t>(128, LEAN_PAIRS / N));
    if (c->new_len) {
        c->flat_min = 0x7fffffffffffffffll;
        c->flat_max = -1;
        if (c->dense != DENSE_NEVER) c->dense = DENSE_NO;
    }
    c->handled = 0;
    // from the second range of the first length on (long series: the third;
    // there the second leaves few rows to sweep and many columns to bound)
    if (!dense_off(c))
        c->dense = c->mode == 0 && c->attempt >= (N <= DENSE_NEAR_MAXN ? 1 : 2) &&
                           s.heat == nullptr && m <= DENSE_MAXM && c->thr64 >= DENSE_MIN_THR
                       ? DENSE_SWEEP
                       : DENSE_NO;
}

// A length whose rows left are too many for the exact pass, and for which a
// dense round is no choice (dense_allowed), is followed by others of its kind
// (heatmaps of noisy series, windows past 256 points): its series asks for
// sweeps at once instead of waiting for them in a round that can only find that
// out.  SWEEPS_MANY: the range discords alone were too many (for a dense round,
// where that is possible, half of all rows), so that neither second chances nor
// fresh witnesses can make the next round one without sweeps, and its sweeps,
// for which a witness is 1.5 operations more per pair, keep
// none; SWEEPS_AGAIN: the one before swept too, and the host issues several
// such rounds at once.  (Heatmap of 14,098 points, eleven lengths, 1,675 to
// 2,275 range discords at six of them: 4.2 ms, so 3.5; white noise, 300,000
// points, m = 50 to 53, 1,600 to 3,000 range discords: 82 ms with witnesses throughout, so 76.)
enum { SWEEPS_NO = 0, SWEEPS_FEW = 1, SWEEPS_MANY = 2, SWEEPS_AGAIN = 4 };

// The next range search of a series (one thread): the first length, the next
// one after a success, or the same length again with the r that k_round_end
// lowered.
__device__ void next_range(const SeriesDev& s, Ctrl* c, float guard, int max_attempts, int32_t* rem)
{
    if (!c->started) {
        c->started = 1;
        c->m = s.minL;
        c->li = 0;
        c->attempt = 0;
        c->new_len = 2;
    } else if (c->done) {
        if (c->m >= s.maxL) {
            c->finished = 1;
            c->active = 0;
            return;
        }
        c->m += 1;
        c->li += 1;
        c->attempt = 0;
        c->new_len = 1;
    } else {
        c->attempt += 1;
        c->new_len = 0;
        if (c->attempt >= max_attempts) {
            c->error = 1;
            c->finished = 1;
            c->active = 0;
            atomicAdd(&rem[REM_ERROR], 1);
            return;
        }
    }
    c->done = 0;
    c->active = 1;
    begin_range(s, c, guard);
    // (read before the first atomic: after one each would be a load of its own)
    const int left = s.maxL - c->m + 1, sweeps = c->li == 0 ? (int)SWEEPS_FEW : c->sweeps;
    const bool dense = dense_round(c);
    atomicMax(&rem[REM_LEFT], left);
    if (sweeps) atomicAdd(&rem[REM_SWEEP], 1);
    if (sweeps & SWEEPS_FEW) atomicAdd(&rem[REM_WITNESS], 1);
    if (sweeps & SWEEPS_AGAIN) atomicAdd(&rem[REM_STEADY], 1);
    if (dense) atomicAdd(&rem[REM_DENSE], 1);
}

// Before the first round of a search.
__global__ void k_start(SeriesDev* S, int B, float guard, int max_attempts, int32_t* rem)
{
    if (rem[REM_BAD] > 0) return;  // a series holds NaN or Inf: no range search starts
    for (int b = blockIdx.x * blockDim.x + threadIdx.x; b < B; b += gridDim.x * blockDim.x)
        next_range(S[b], S[b].ctrl, guard, max_attempts, rem);
}

// ---------------------------------------------------------------------------
// per-length statistics (Eq. (4) at minL, Eq. (7)-(8) after), the column and
// row helpers, and the per-round reset of the bitmap and row maxima
// ---------------------------------------------------------------------------
// Statistics live in two buffers used alternately from one length to the
// next (mu/var for even m - minL, mu2/var2 for odd), so every thread can
// read the previous length's values of its own window and of the next one.
__device__ __forceinline__ const double* cur_mu(const SeriesDev& s, const Ctrl* c)
{
    return (c->li & 1) ? s.mu2 : s.mu;
}
__device__ __forceinline__ const double* cur_var(const SeriesDev& s, const Ctrl* c)
{
    return (c->li & 1) ? s.var2 : s.var;
}

// A round whose selection left at most DIRECT_MAX live subsequences: the
// refinement sweep is skipped and the exact pass evaluates every one of them.
__device__ __forceinline__ bool direct_round(const Ctrl* c) { return c->live_ref <= DIRECT_MAX; }
// Few enough rows left by the witnesses for the exact pass without a sweep.
__device__ __forceinline__ bool lean_round(const Ctrl* c) { return c->nlive <= c->lean_max; }

// Mean and variance of window p at length m: two passes (Eq. (4)).
__device__ __forceinline__ void direct_stats(const double* T, int64_t p, int32_t m, double& mean,
                                             double& var)
{
    double acc = 0.0;
#pragma unroll 8
    for (int k = 0; k < m; ++k) acc += T[p + k];
    mean = acc / (double)m;
    double q = 0.0;
#pragma unroll 8
    for (int k = 0; k < m; ++k) {
        const double d = T[p + k] - mean;
        q += d * d;
    }
    var = q / (double)m;
}

// a / d from rd = 1 / d (correctly rounded): the residual of the first
// quotient corrects it to the correctly rounded one (Markstein), in three
// operations instead of a division's dozen.
__device__ __forceinline__ double div_by(double a, double d, double rd)
{
    const double q = a * rd;
    return fma(fma(-q, d, a), rd, q);
}

// Constants of one length's update: m, 1/m, (m-1)/m.
struct GrowBy {
    double m, rm, fm;
};
__device__ __forceinline__ GrowBy grow_by(int32_t m)
{
    GrowBy g;
    g.m = (double)m;
    g.rm = 1.0 / g.m;
    g.fm = (double)(m - 1) / g.m;
    return g;
}

// Eq. (7)-(8): a window from length m-1 (mean mu0, variance v0) to m, t its
// new last value.
__device__ __forceinline__ void grow_stats(double t, const GrowBy& g, double mu0, double v0,
                                           double& mean, double& var)
{
    const double d = mu0 - t;
    mean = div_by(fma(g.m - 1.0, mu0, t), g.m, g.rm);
    var = g.fm * (v0 + div_by(d * d, g.m, g.rm));
}

// Block extremes of the window spreads (every block of k_helpers, and of
// k_length in the diagnostics): the largest and smallest sigma of the block's non-flat windows.
__device__ void spread_extremes(const SeriesDev& s, int64_t lb, double smax, double smin)
{
    __shared__ double rmax[4], rmin[4];
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        smax = fmax(smax, __shfl_xor(smax, o));
        smin = fmin(smin, __shfl_xor(smin, o));
    }
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        rmax[w] = smax;
        rmin[w] = smin;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double a = rmax[0], z = rmin[0];
        for (int q = 1; q < (int)(blockDim.x >> 6); ++q) {
            a = fmax(a, rmax[q]);
            z = fmin(z, rmin[q]);
        }
        s.sgm[2 * lb] = a;
        s.sgm[2 * lb + 1] = z;
    }
}

// The spread contrast of a new length and the round's selection thresholds
// (one block per series, after k_helpers): over every block of 256 windows,
// the largest spread of the two blocks on either side (a superset of the
// R_MAX - 1 windows a recurrence chain passes on each side) over the block's
// smallest spread, squared (see sel_guard).
constexpr int GUARD_BLOCK = 1024;
__global__ __launch_bounds__(GUARD_BLOCK) void k_guard(SeriesDev* S, float guard)
{
    const SeriesDev& s = S[blockIdx.x];
    Ctrl* c = s.ctrl;
    if (!c->active || lean_round(c) || guard <= 0.0f) return;
    __shared__ double red[GUARD_BLOCK / 64];
    const int64_t nb = (s.n - c->m + 1 + 255) / 256;
    double g = 0.0;
    for (int64_t q = threadIdx.x; q < nb; q += blockDim.x) {
        const double lo = s.sgm[2 * q + 1];
        double hi = 0.0;
        for (int64_t e = (q >= 2 ? q - 2 : 0); e <= q + 2 && e < nb; ++e) hi = fmax(hi, s.sgm[2 * e]);
        if (lo < f_inf<double>()) {  // not a block of flat windows only
            const double rt = hi / lo;
            g = fmax(g, rt * rt);
        }
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) g = fmax(g, __shfl_xor(g, o));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = g;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int q = 1; q < GUARD_BLOCK / 64; ++q) g = fmax(g, red[q]);
        c->gam2 = g;
        set_sel_thresholds(c, guard);
    }
}

// df[i] = (t_{i+m} - t_i)/2, dg[i] = (t_{i+m} - mu_{i+1}) + (t_i - mu_i) for
// i < N-1 (zero beyond), inv[i] = 1/(sqrt(m) sigma_i) for non-flat i < N.
//
// At a new length every block also records the largest and smallest window
// sigma of its 256 windows, from which k_guard sets the FP32 guard band.
__global__ void k_length(SeriesDev* S, int B, const int64_t* __restrict__ pfx)
{
    const int b = series_of(pfx, B, blockIdx.x);
    const SeriesDev& s = S[b];
    Ctrl* c = s.ctrl;
    if (!c->active) return;
    const int64_t lb = blockIdx.x - pfx[b];
    const int64_t i = lb * (int64_t)blockDim.x + threadIdx.x;
    const int32_t m = c->m;
    const int64_t N = s.n - m + 1;
    double smax = 0.0, smin = f_inf<double>();  // spread extremes of this thread's window
    if (c->new_len && i < s.Npad + 64) {
        const double* __restrict__ T = s.T;
        const bool odd = (c->li & 1) != 0;
        double* mu_n = odd ? s.mu2 : s.mu;
        double* var_n = odd ? s.var2 : s.var;
        const double* mu_o = odd ? s.mu : s.mu2;
        const double* var_o = odd ? s.var : s.var2;
        double m0 = 0.0, v0 = 0.0, m1 = 0.0, v1 = 0.0;
        if (i < N) {
            if (c->new_len == 2) {
                direct_stats(T, i, m, m0, v0);
                if (i + 1 < N) direct_stats(T, i + 1, m, m1, v1);
            } else {
                const GrowBy g = grow_by(m);
                grow_stats(T[i + m - 1], g, mu_o[i], var_o[i], m0, v0);
                if (i + 1 < N) grow_stats(T[i + m], g, mu_o[i + 1], var_o[i + 1], m1, v1);
            }
        }
        mu_n[i] = m0;
        var_n[i] = v0;
        double df = 0.0, dg = 0.0, inv = 0.0;
        if (i < N - 1) {
            const double a = T[i + m], e = T[i];
            df = (a - e) * 0.5;
            dg = (a - m1) + (e - m0);
        }
        if (i < N) {
            const double sg = sqrt(v0);
            if (sg <= c->flat_eps) {
                atomicMin((long long*)&c->flat_min, (long long)i);
                atomicMax((long long*)&c->flat_max, (long long)i);
            } else {
                inv = 1.0 / (sqrt((double)m) * sg);
                smax = smin = sg;
            }
        }
        s.df64[i] = df;
        s.dg64[i] = dg;
        s.inv64[i] = inv;
        s.df32[i] = (float)df;
        s.dg32[i] = (float)dg;
        s.inv32[i] = (float)inv;
    }
    if (c->new_len) spread_extremes(s, lb, smax, smin);
    // every round: all N subsequences start alive, row maxima at -inf
    if (i < s.nwords) {
        const int64_t lo = i * 64;
        unsigned long long bits = 0ull;
        if (lo + 64 <= N) bits = ~0ull;
        else if (lo < N) bits = (1ull << (N - lo)) - 1ull;
        s.alive[i] = bits;
        s.unc[i] = 0ull;
    }
    if (i < s.Npad) {
        s.rho[i] = 0x000fffffffffffffull;  // ordered bits of -inf
        s.rhs[i] = 0x000fffffffffffffull;
    }
}

// ---------------------------------------------------------------------------
// witnesses: the per-length step of a search
// ---------------------------------------------------------------------------
// A subsequence pruned at one length by a neighbour closer than r is almost
// always pruned by the same neighbour at the next length: distances and r
// both move slowly with m.  Every row therefore keeps its last witness j and
// the centred covariance C of the pair in FP64.  From length m - 1 to m,
//     C += (m-1)/m (t[i+m-1] - mu_i) (t[j+m-1] - mu_j)      (means at m - 1),
// the two-window form of Eq. (8), so a row costs a few operations instead of
// the hundreds to thousands of pairs a selection sweep evaluates before it
// prunes the row (k_advance).  A row whose witness fails tries its witness's
// witness and the diagonal extensions of its nearest pruned neighbours'
// (k_rescue).  What is left, a handful to a few hundred rows, goes to the
// exact pass; only when more than Ctrl::lean_max rows are left (the first
// length, mostly) does a round sweep.
//
// Soundness: a row is pruned only by an FP64 correlation above thr64 by more
// than a guard; rows nearer to the threshold are left to the exact pass.  C
// starts from a direct dot product (or the exact pass's value).  The chain adds
// what its means are off by, to first order: after S lengths a mean of values
// up to M is off by at most e = (m + 2 S) u M (u = 2^-53; the first sum, then two
// roundings per length), and as the products' other factors are the deviations
// that make up m sigma^2, rho is off by at most e_i / sigma_i + e_j / sigma_j for
// S <= m.  With M <= |mu| + sqrt(m) sigma that is
//     3 m u (|mu_i| / sigma_i + |mu_j| / sigma_j + 2 sqrt(m)),
// 1e-11 for a walk of 10^6 steps, but past 1e-9 where the series lies 10^4 to 10^5
// times its windows' deviations from zero (windows of 128 points at 4e7 times
// were seen 6e-8 off): WIT_GUARD, or that where it is more.  A direct product's
// error is of second order in e, far below either.
constexpr double WIT_GUARD = 1e-9;
constexpr double WIT_DRIFT = 3.0;
constexpr int32_t WIT_NONE = (int32_t)0x80000000;  // j >= 0: C known; ~j: C to be computed

__device__ __forceinline__ double inv_of(double var, double sqm, double feps)
{
    const double sg = sqrt(var);
    return sg <= feps ? 0.0 : 1.0 / (sqm * sg);
}

// Correlation of a pair (R11: flat windows correlate 1 with each other, 0 with others).
__device__ __forceinline__ double pair_rho(double C, double ii, double ij)
{
    if (ii == 0.0 || ij == 0.0) return (ii == 0.0 && ij == 0.0) ? 1.0 : 0.0;
    return C * ii * ij;
}

// Direct centred dot product of windows i and j.
__device__ __forceinline__ double direct_cov(const double* __restrict__ T, int64_t i, int64_t j,
                                             int32_t m, double mi, double mj)
{
    const double* __restrict__ x = T + i;
    const double* __restrict__ y = T + j;
    double a0 = 0.0, a1 = 0.0;
    int k = 0;
    for (; k + 8 <= m; k += 8) {
        double u[8], v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            u[e] = x[k + e];
            v[e] = y[k + e];
        }
#pragma unroll
        for (int e = 0; e < 8; e += 2) {
            a0 = fma(u[e] - mi, v[e] - mj, a0);
            a1 = fma(u[e + 1] - mi, v[e + 1] - mj, a1);
        }
    }
    for (; k < m; ++k) a0 = fma(x[k] - mi, y[k] - mj, a0);
    return a0 + a1;
}

// Statistics of a new length (Eq. (4) at minL, Eq. (7)-(8) after), the
// witness test, the bitmap of live rows and the lists of those whose witness
// failed.  One thread per subsequence, one wave per bitmap word.  Bound by
// HBM: about 90 bytes per subsequence and length.  A repeat of the same
// length at a smaller r only repeats the test.  rem: the round's host
// counters restart.
constexpr int ADV_BLOCK = 256;
__global__ __launch_bounds__(ADV_BLOCK, 8) void k_advance(SeriesDev* S, int B,
                                                       const int64_t* __restrict__ pfx, int32_t* rem)
{
    extern __shared__ double ts[];  // ADV_BLOCK + maxL values
    __shared__ unsigned int wcnt[ADV_BLOCK / 64];
    __shared__ unsigned int base_s;
    if (blockIdx.x == 0 && threadIdx.x < REM_COUNT) rem[threadIdx.x] = 0;
    const int b = B == 1 ? 0 : series_of(pfx, B, blockIdx.x);
    const SeriesDev& s = S[b];
    Ctrl* c = s.ctrl;
    if (!c->active || c->pending) return;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t lb = blockIdx.x - (B == 1 ? 0 : pfx[b]);
    if (lb == 0 && threadIdx.x < CAND_GROUPS) c->pcnt[threadIdx.x] = 0;
    const int64_t i = lb * (int64_t)ADV_BLOCK + threadIdx.x;
    const int32_t m = c->m;
    const int64_t N = s.n - m + 1;
    const int new_len = c->new_len;
    const bool prune = c->prune != 0;
    const double feps = c->flat_eps, sqm = sqrt((double)m);
    const double kill = c->thr64 + WIT_GUARD;
    const double* __restrict__ T = s.T;
    const bool odd = (c->li & 1) != 0;
    double* mu_n = odd ? s.mu2 : s.mu;
    double* var_n = odd ? s.var2 : s.var;
    const double* __restrict__ mu_o = odd ? s.mu : s.mu2;
    const double* __restrict__ var_o = odd ? s.var : s.var2;
    const bool in = i < N;
    const int32_t w0 = in && new_len != 2 ? s.wit[i] : WIT_NONE;
    const GrowBy gb = grow_by(m);
    if (new_len == 2) {  // the block's stretch of the series, for the direct sums
        const int64_t e = std::min<int64_t>(s.Tlen - (i - threadIdx.x), ADV_BLOCK + m);
        for (int t = threadIdx.x; t < e; t += ADV_BLOCK) ts[t] = T[i - threadIdx.x + t];
        __syncthreads();
    }
    double mi = 0.0, vi = 0.0, ii = 0.0, moi = 0.0, ti = 0.0;
    if (new_len) {
        if (in) {
            if (new_len == 2) {
                direct_stats(ts, threadIdx.x, m, mi, vi);
            } else {
                moi = mu_o[i];
                ti = T[i + m - 1];
                grow_stats(ti, gb, moi, var_o[i], mi, vi);
            }
            ii = inv_of(vi, sqm, feps);
            if (ii == 0.0) {
                atomicMin((long long*)&c->flat_min, (long long)i);
                atomicMax((long long*)&c->flat_max, (long long)i);
            }
        }
        if (i < s.Npad + 64) {
            mu_n[i] = mi;
            var_n[i] = vi;
            s.inv64[i] = ii;
        }
    } else if (in) {
        mi = mu_n[i];
        ii = s.inv64[i];
    }
    bool dead = false;
    if (new_len == 2) {
        if (in) s.wit[i] = WIT_NONE;
    } else if (w0 != WIT_NONE) {
        const bool fresh = w0 < 0;
        const int64_t j = fresh ? ~w0 : w0;
        if (j < N && (j - i >= m || i - j >= m)) {
            double mj, ij, moj = 0.0, tj = 0.0;
            if (new_len) {
                double vj;
                moj = mu_o[j];
                tj = T[j + m - 1];
                grow_stats(tj, gb, moj, var_o[j], mj, vj);
                ij = inv_of(vj, sqm, feps);
            } else {
                mj = mu_n[j];
                ij = s.inv64[j];
            }
            double C;
            if (fresh) {
                C = direct_cov(T, i, j, m, mi, mj);
                s.wit[i] = (int32_t)j;
                s.wc[i] = C;
            } else {
                C = s.wc[i];
                if (new_len) {
                    C += gb.fm * (ti - moi) * (tj - moj);
                    s.wc[i] = C;
                }
            }
            const double rho = pair_rho(C, ii, ij);
            const double drift = fma(fabs(mi), ii, fma(fabs(mj), ij, 2.0)) * (WIT_DRIFT * 0x1p-53);
            dead = prune && rho > kill && rho - c->thr64 > drift * (gb.m * sqm);
        } else {  // no longer a window, or now a self match
            s.wit[i] = WIT_NONE;
        }
    }
    const unsigned long long live = __ballot(in && !dead);
    if (lane == 0 && (i >> 6) < s.nwords) s.alive[i >> 6] = live;
    if (s.heat) {  // range discords are written by k_round_end and k_heat
        double* hrow = s.heat + (int64_t)c->li * s.heat_ld;
        for (int64_t q = i; q < s.heat_ld; q += s.Npad + 64) hrow[q] = 0.0;
    }
    if (new_len == 2 || !prune) {
        if (i == 0) c->nlive = 0x7fffffffu;
        return;
    }
    if (lane == 0) wcnt[wv] = (unsigned int)__popcll(live);
    __syncthreads();
    const int list = (int)(lb & (fail_lists(s.Npad) - 1));
    if (threadIdx.x == 0) {
        unsigned int tot = 0;
        for (int q = 0; q < ADV_BLOCK / 64; ++q) tot += wcnt[q];
        base_s = tot ? atomicAdd(&c->nfail[list], tot) : 0u;
    }
    __syncthreads();
    if (in && !dead) {
        unsigned int p = base_s + (unsigned int)__popcll(live & ((1ull << lane) - 1ull));
        for (int q = 0; q < wv; ++q) p += wcnt[q];
        s.fail[list * fail_cap(s.Npad) + p] = (int32_t)i;
    }
}

// Second chances for the rows whose witness failed, one wave per row: up to
// RESCUE_TRIES batches of eight candidates, eight lanes each, compared by
// direct FP64 dot products; the best one above the threshold prunes the row
// and becomes its witness.  Candidates: the witness's witness and that one's,
// the diagonal extensions of the nearest pruned rows' witnesses on either
// side, and the witnesses' witnesses of rows a little further off; then those
// of rows at growing distance.  (ECG-like series at lengths past one beat,
// where r falls and up to a fifth of the witnesses fail in one length: all but
// about one row in a thousand of them are pruned here, most by the first
// batch.)  Rows that stay are the round's candidates.  Bound by latency: a
// chain of dependent loads per batch, which is why a batch is wide.
constexpr int RESCUE_TRIES = 2;
// Too many failures for second chances (a new threshold altogether, e.g. the
// first length's next r), or too many range discords among them.
__device__ __forceinline__ bool rescue_hopeless(const Ctrl* c, unsigned int total, int64_t N)
{
    return ((int64_t)total * 2 > N || (c->sweeps & SWEEPS_MANY)) && total > c->lean_max;
}

// The waves of k_rescue that each series of a batch gets (one block, a thread
// per series): one, and its part of the others by its rows.  wpfx[b]: first
// wave of series b.  (64 series of 10,000 to 200,000 points, per round: an even
// share, waves bound to one list, 267 us; this share and the rows of all lists
// in turn, 96.)
constexpr int FAIL_ITEMS_MAXB = 1024;
__global__ __launch_bounds__(FAIL_ITEMS_MAXB) void k_fail_items(SeriesDev* S, int B, int64_t waves,
                                                               int64_t* wpfx)
{
    __shared__ long long ws[2][FAIL_ITEMS_MAXB / 64];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    long long rows = 0, any = 0;
    if (tid < B) {
        const SeriesDev& s = S[tid];
        const Ctrl* c = s.ctrl;
        if (c->active && !c->pending && c->new_len != 2 && c->prune) {
            unsigned int total = 0;
#pragma unroll 16
            for (int q = 0; q < FAIL_LISTS; ++q) total += c->nfail[q];
            any = total > 0 ? 1 : 0;
            rows = rescue_hopeless(c, total, s.n - c->m + 1) ? 0 : total;
        }
    }
    auto scan = [&](long long v, int at, long long& before) {
        long long x = v;
        for (int o = 1; o < 64; o <<= 1) {
            const long long y = __shfl_up(x, o);
            if (lane >= o) x += y;
        }
        if (lane == 63) ws[at][w] = x;
        __syncthreads();
        long long tot = 0;
        before = x - v;
        for (int e = 0; e < FAIL_ITEMS_MAXB / 64; ++e) {
            before += e < w ? ws[at][e] : 0;
            tot += ws[at][e];
        }
        return tot;
    };
    long long before;
    const long long all = scan(rows, 0, before);
    const long long mine = any ? 1 + (all ? rows * (waves - B) / all : 0) : 0;
    const long long used = scan(mine, 1, before);
    if (tid < B) wpfx[tid] = before;
    if (tid == 0) wpfx[B] = used;
}

__global__ __launch_bounds__(RESCUE_BLOCK) void k_rescue(SeriesDev* S, int B,
                                                         const int64_t* __restrict__ wpfx)
{
    const int lane = threadIdx.x & 63;
    const int sub = lane & 7, cq = lane >> 3;
    const int64_t wave = (int64_t)blockIdx.x * (RESCUE_BLOCK / 64) + (threadIdx.x >> 6);
    const int64_t nwaves = (int64_t)gridDim.x * (RESCUE_BLOCK / 64);
    // the waves are shared out by k_fail_items, without its table evenly
    if (wpfx && wave >= wpfx[B]) return;
    const int64_t own = wpfx ? series_of(wpfx, B, wave) : 0;
    const int64_t nper = wpfx ? wpfx[own + 1] - wpfx[own] : std::max<int64_t>(1, nwaves / B);
    const int64_t w = wpfx ? wave - wpfx[own] : wave % nper;
    for (int64_t b = wpfx ? own : wave / nper; b < B; b += wpfx ? (int64_t)B : nwaves / nper) {
        const SeriesDev& s = S[b];
        Ctrl* c = s.ctrl;
        const unsigned int mine = c->nfail[lane];
        if (!c->active || c->pending || c->new_len == 2 || !c->prune) continue;
        const int32_t m = c->m;
        const int64_t N = s.n - m + 1;
        unsigned int total = mine;
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) total += __shfl_xor(total, o);
        if (rescue_hopeless(c, total, N)) {
            if (w == 0 && lane == 0) c->nlive = 0x7fffffffu;
            continue;
        }
        const int64_t cap = fail_cap(s.Npad);
        const double* __restrict__ T = s.T;
        const double* __restrict__ mu = cur_mu(s, c);
        const double* __restrict__ inv = s.inv64;
        const double kill = c->thr64 + WIT_GUARD;
        // the waves take the rows in turn, numbered through the lists (lane l
        // holds list l's end)
        unsigned int end = mine;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const unsigned int y = __shfl_up(end, o);
            if (lane >= o) end += y;
        }
        {
            for (int64_t p = w; p < (int64_t)total; p += nper) {
                const int list = __popcll(__ballot((int64_t)end <= p));
                const int64_t at = p - (list ? __builtin_amdgcn_readlane((int)end, list - 1) : 0);
                const int64_t i = s.fail[list * cap + at];
                const double mi = mu[i], ii = inv[i];
                // a row's witness, whatever its state (a candidate is always recomputed)
                auto wit_of = [&](int64_t q) -> int64_t {
                    if (q < 0 || q >= N) return -1;
                    const int32_t v =
                        __hip_atomic_load(&s.wit[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    return v == WIT_NONE ? -1 : v < 0 ? (int64_t)~v : (int64_t)v;
                };
                bool done = false;
                for (int t = 0; t < RESCUE_TRIES && !done; ++t) {
                    // this lane's candidate: row q's witness (hops = 1) or that
                    // one's witness (2, 3), shifted along the diagonal to row i
                    int64_t q = i;
                    int hops = 2;
                    if (t == 0) {
                        if (cq == 1) hops = 3;
                        if (cq == 2 || cq == 3) {
                            // the nearest pruned row on the left (2) or right (3),
                            // within 63 rows
                            hops = 1;
                            const int64_t base = cq == 2 ? i - 63 : i;
                            q = -1;
                            if (base >= 0) {
                                const int off = (int)(base & 63);
                                unsigned long long bits = load_word(&s.alive[base >> 6]) >> off;
                                if (off) bits |= load_word(&s.alive[(base >> 6) + 1]) << (64 - off);
                                // bit e: row base + e is pruned (or past the end)
                                const unsigned long long z = ~bits;
                                if (z)
                                    q = base + (cq == 2 ? 63 - __clzll((long long)z)
                                                        : __ffsll((long long)z) - 1);
                            }
                        }
                        if (cq >= 4) q = i + (cq == 4 ? -4 : cq == 5 ? 4 : cq == 6 ? -16 : 16);
                    } else {
                        const int64_t d = (int64_t)32 << (cq >> 1);  // 32 .. 256 rows away
                        q = (cq & 1) ? i + d : i - d;
                    }
                    int64_t j = wit_of(q);
                    if (hops > 1) j = wit_of(j);
                    if (hops > 2) j = wit_of(j);
                    if (j >= 0) j += i - q;
                    if (j < 0 || j >= N || (j < i + m && j > i - m)) j = -1;
                    double rho = -4.0, C = 0.0;
                    if (j >= 0) {
                        const double mj = mu[j], ij = inv[j];
                        const double* __restrict__ x = T + i;
                        const double* __restrict__ y = T + j;
                        int k = sub;
                        for (; k + 24 < m; k += 32) {
                            double u[4], v[4];
#pragma unroll
                            for (int z = 0; z < 4; ++z) {
                                u[z] = x[k + 8 * z];
                                v[z] = y[k + 8 * z];
                            }
#pragma unroll
                            for (int z = 0; z < 4; ++z) C = fma(u[z] - mi, v[z] - mj, C);
                        }
                        for (; k < m; k += 8) C = fma(x[k] - mi, y[k] - mj, C);
                        rho = ij;
                    }
#pragma unroll
                    for (int o = 4; o >= 1; o >>= 1) C += __shfl_xor(C, o);
                    if (j >= 0) rho = pair_rho(C, ii, rho);
                    // the best of the eight
                    double br = rho;
                    int bq = cq;
#pragma unroll
                    for (int o = 8; o <= 32; o <<= 1) {
                        const double r2 = __shfl_xor(br, o);
                        const int q2 = __shfl_xor(bq, o);
                        if (r2 > br || (r2 == br && q2 < bq)) {
                            br = r2;
                            bq = q2;
                        }
                    }
                    done = __builtin_amdgcn_readfirstlane((int)(br > kill)) != 0;
                    if (done && sub == 0 && cq == bq) {
                        __hip_atomic_store(&s.wit[i], (int32_t)j, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
                        s.wc[i] = C;
                        atomicAnd(&s.alive[i >> 6], ~(1ull << (i & 63)));
                    }
                }
                if (!done && lane == 0) {
                    const unsigned int have =
                        __hip_atomic_load(&c->nlive, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if (have <= (unsigned int)CAND_MAX) {  // abandoned once it overflows
                        const unsigned int slot = atomicAdd(&c->nlive, 1u);
                        if (slot < (unsigned int)CAND_MAX) s.cand[slot] = i;
                    }
                }
            }
        }
    }
}

// Helpers of a round that sweeps (Eq. (10)'s centred form): df[i] =
// (t_{i+m} - t_i)/2, dg[i] = (t_{i+m} - mu_{i+1}) + (t_i - mu_i) for i < N-1
// (zero beyond) in both precisions, the spread extremes that set the FP32
// guard band, and the resets of the row maxima.
__global__ __launch_bounds__(ADV_BLOCK) void k_helpers(SeriesDev* S, int B,
                                                       const int64_t* __restrict__ pfx)
{
    const int b = series_of(pfx, B, blockIdx.x);
    const SeriesDev& s = S[b];
    Ctrl* c = s.ctrl;
    if (!c->active || lean_round(c) || taking_parts(c)) return;  // (the candidates stand in s.fail)
    const int64_t lb = blockIdx.x - pfx[b];
    const int64_t i = lb * (int64_t)ADV_BLOCK + threadIdx.x;
    const int32_t m = c->m;
    const int64_t N = s.n - m + 1;
    const double* __restrict__ mu = cur_mu(s, c);
    double smax = 0.0, smin = f_inf<double>();
    if (i < s.Npad + 64) {
        double df = 0.0, dg = 0.0, inv = 0.0;
        if (i < N - 1) {
            const double a = s.T[i + m], e = s.T[i];
            df = (a - e) * 0.5;
            dg = (a - mu[i + 1]) + (e - mu[i]);
        }
        if (i < N) {
            inv = s.inv64[i];
            if (inv > 0.0) smax = smin = sqrt(cur_var(s, c)[i]);
        }
        s.df64[i] = df;
        s.dg64[i] = dg;
        s.df32[i] = (float)df;
        s.dg32[i] = (float)dg;
        s.inv32[i] = (float)inv;
    }
    spread_extremes(s, lb, smax, smin);
    if (i < s.nwords) s.unc[i] = 0ull;
    if (i < s.Npad) {
        s.rho[i] = 0x000fffffffffffffull;  // ordered bits of -inf
        s.rhs[i] = 0x000fffffffffffffull;
    }
}

// ---------------------------------------------------------------------------
// the sweeps
// ---------------------------------------------------------------------------
template <typename F>
struct SweepArgs {
    const double* __restrict__ T;
    const double* __restrict__ mu;
    const F* __restrict__ df;
    const F* __restrict__ dg;
    const F* __restrict__ inv;
    unsigned long long* alive;
    unsigned long long* rho;
    unsigned long long* rhs;
    unsigned long long* unc;
    uint32_t* twork;
    int32_t* wit;  // witnesses of the rows this item prunes
    Ctrl* ctrl;
    int64_t N;
    int32_t m;
};

// Copy count doubles from global memory to LDS (the whole workgroup): groups
// of eight loads per thread are issued before their stores, so one memory
// latency covers 8 x blockDim values.
__device__ __forceinline__ void lds_fill(double* dst, const double* __restrict__ src, int count)
{
    const int tid = threadIdx.x, nt = blockDim.x;
    for (int base = 0; base < count; base += nt * 8) {
        double v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int t = base + tid + nt * u;
            v[u] = t < count ? src[t] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int t = base + tid + nt * u;
            if (t < count) dst[t] = v[u];
        }
    }
}

// ----- exact values from the FP64 matrix cores -----
// A sweep needs exact FP64 centred dot products in two places: the first
// column of a work item (one per row of the tile) and the top row of the
// tile at every later column (the boundary that feeds the recurrence).
// Both are correlations of one short centred window v (m values) with a
// stretch of the series w:
//     D(p) = sum_k v[k] w[p + k],   p = 0 .. 255,
// which is one 16 x 16 tile of V_MFMA_F64_16X16X4F64 with the Toeplitz
// operand A[r][k] = v[k - r] and the Hankel operand B[k][c] = w[16 c + k]:
// D[r][c] = D(16 c + r).  Lane l supplies A[l % 16][k0 + l / 16] and
// B[k0 + l / 16][l % 16] and receives D[l / 16 + 4 q][l % 16], q < 4, i.e.
// D(p) for p = 16 (l % 16) + l / 16 + 4 q.  Two LDS reads per matrix
// instruction (1024 multiply-adds) replace the two reads per multiply-add of
// a vector loop, which left the sweeps bound by LDS bandwidth.
typedef double pm_acc_t __attribute__((ext_vector_type(4)));
constexpr int HK_PAD = 16;    // zeros before v (k - r >= -15)
constexpr int HK_TILE = 256;  // values D(p) per Hankel tile
// Columns per boundary batch: a whole tile for the FP32 sweeps; half a tile
// for FP64 records, whose smaller staging lets more refinement items stay
// resident (the FP32 sweeps measured slower at half a tile).
__host__ __device__ constexpr int bcols_of(int fbytes) { return fbytes == 8 ? HK_TILE / 2 : HK_TILE; }
template <typename F>
__host__ __device__ constexpr int batch_cols() { return bcols_of((int)sizeof(F)); }
// w is staged skewed (value p at p + p / 16), so that the 16 lanes reading
// w[16 c + k] for c = 0..15 hit distinct LDS banks.
__host__ __device__ constexpr int hk_skew(int p) { return p + (p >> 4); }
// k < 4 hk_steps(m) covers every k - r < m for r < 16
__host__ __device__ constexpr int hk_steps(int m) { return (m + 15 + 3) >> 2; }
// v with HK_PAD zeros before and zeros after: HK_PAD + 4 hk_steps(m) values
__host__ __device__ constexpr int hk_vp_doubles(int m) { return (HK_PAD + 4 * hk_steps(m) + 3) & ~3; }

__device__ __forceinline__ int hk_offset(int q)
{
    const int lane = threadIdx.x;
    return 16 * (lane & 15) + (lane >> 4) + 4 * q;
}

// D(p) for p < ncols (a multiple of 16, at most 256; see above): vp = v
// after HK_PAD zeros, zero beyond m; w = skewed LDS stretch starting at value
// wbase, at least wbase + ncols + m + 16 values.  Lanes of the columns
// c >= ncols / 16 read the stretch's first column instead: their D values
// are not meaningful.  One accumulator (the matrix core chains dependent
// accumulations), so the sweep keeps its registers.
__device__ __forceinline__ pm_acc_t hankel16(const double* vp, const double* w, int wbase, int m,
                                             int ncols = HK_TILE)
{
    const int lane = threadIdx.x;
    const int ca = lane & 15, ka = lane >> 4;
    const int K4 = hk_steps(m);
    const double* va = vp + HK_PAD + ka - ca;
    const int wb = wbase + 16 * (16 * ca < ncols ? ca : 0) + ka;
    pm_acc_t d = {0.0, 0.0, 0.0, 0.0};
    for (int s = 0; s < K4; ++s)
        d = __builtin_amdgcn_mfma_f64_16x16x4f64(va[4 * s], w[hk_skew(wb + 4 * s)], d, 0, 0, 0);
    return d;
}

// Copy count doubles from src into the skewed LDS stretch w (the whole
// wave: four loads in flight per lane before their stores).
__device__ __forceinline__ void stage_skewed(double* w, const double* __restrict__ src, int count)
{
    const int lane = threadIdx.x;
    for (int base = 0; base < count; base += 64 * 4) {
        double v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int t = base + lane + 64 * u;
            v[u] = t < count ? src[t] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int t = base + lane + 64 * u;
            if (t < count) w[hk_skew(t)] = v[u];
        }
    }
}

// Column helpers of one step, staged in LDS per batch of columns.
template <typename F>
struct alignas(4 * sizeof(F)) H4 {
    F df, dg, inv;  // df[j-1], dg[j-1], 1/(sqrt(m) sigma_j)
    F B;            // C(i0, j): exact value of the tile's top row at column j
};

// LDS of a sweep work item with R-row tiles, in doubles:
//   xp   [hk_vp_doubles(m)]  the first column's centred window, then the
//                            tile's top-row centred window (padded for the
//                            Toeplitz operand)
//   ws   [sweep_ws_doubles]  skewed series stretch: the rows' windows while
//                            the first column is computed, then each batch's
//                            columns
//   hs   [batch records]     per-step helpers and boundary values of a batch
//                            (the first column's R row values before that)
//   rowv [R]                 refinement only: per-row 1/(sqrt(m) sigma_i)
// (fbytes: bytes of the sweep's float type; nc: columns per batch)
__host__ __device__ constexpr int sweep_ws_count(int m, int R, int nc) { return (R > nc ? R : nc) + m + 16; }
__host__ __device__ constexpr int sweep_ws_doubles(int m, int R, int nc)
{
    return (hk_skew(sweep_ws_count(m, R, nc) - 1) + 1 + 3) & ~3;
}
__host__ __device__ constexpr int sweep_hs_offset(int m, int R, int nc)
{
    return hk_vp_doubles(m) + sweep_ws_doubles(m, R, nc);
}
// (the region first holds the R first-column values of an item, as doubles)
__host__ __device__ constexpr int sweep_hs_doubles(int R, int fbytes, int nc)
{
    return nc * 4 * fbytes / 8 > R ? nc * 4 * fbytes / 8 : R;
}
__host__ __device__ constexpr int sweep_rowv_offset(int m, int R, int fbytes, int nc)
{
    return sweep_hs_offset(m, R, nc) + sweep_hs_doubles(R, fbytes, nc);
}
__host__ __device__ constexpr size_t sweep_lds_doubles(int m, int R, int fbytes, bool rowv, int nc)
{
    return (size_t)(sweep_rowv_offset(m, R, fbytes, nc) + (rowv ? R : 0));
}
__host__ __device__ constexpr size_t sweep_lds_doubles(int m, int R, int fbytes, bool rowv)
{
    return sweep_lds_doubles(m, R, fbytes, rowv, bcols_of(fbytes));
}

// Start of a sweep work item (one wavefront, row tile of R = 64 Q rows from
// i0, first column jbeg): acc[q] = C(rbase + q, jbeg), rbase = i0 + Q lane,
// the centred dot products sum_k t_{i+k} y_k - mu_i Sy with y the centred
// window of column jbeg, from R / 256 Hankel tiles (the rows' values pass
// through the hs region); then xp holds the tile's top-row centred window
// x with sum Sx (zero up to rounding) for the boundary values.
template <int Q>
__device__ void item_start(const double* __restrict__ T, const double* __restrict__ mu, int32_t m,
                           int64_t i0, int64_t jbeg, double* xp, double* ws, double* rowc,
                           double& Sx, double& Sy, double (&acc)[Q])
{
    constexpr int R = 64 * Q;
    const int lane = threadIdx.x;
    const int nvp = hk_vp_doubles(m);
    const double muj = mu[jbeg], mui0 = mu[i0];
    double mr[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) mr[q] = mu[i0 + Q * lane + q];
    // the column window (xp, zero padded) and the rows' stretch (ws)
    for (int t = lane; t < nvp; t += 64) {
        const int k = t - HK_PAD;
        xp[t] = (k >= 0 && k < m) ? T[jbeg + k] : 0.0;
    }
    stage_skewed(ws, T + i0, R + m + 16);
    __syncthreads();
    double sy = 0.0;
    for (int k = lane; k < m; k += 64) {
        const double v = xp[HK_PAD + k] - muj;
        xp[HK_PAD + k] = v;
        sy += v;
    }
    Sy = wave_sum(sy);
    __syncthreads();
#pragma unroll
    for (int h = 0; h < (R + 255) / 256; ++h) {
        const pm_acc_t D = hankel16(xp, ws, 256 * h, m, R - 256 * h < 256 ? R - 256 * h : 256);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int p = 256 * h + hk_offset(q);
            if (p < R) rowc[p] = D[q];
        }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < Q; ++q) acc[q] = rowc[Q * lane + q] - mr[q] * Sy;
    // the top row's centred window
    double sx = 0.0;
    for (int k = lane; k < m; k += 64) {
        const double v = ws[hk_skew(k)] - mui0;
        xp[HK_PAD + k] = v;
        sx += v;
    }
    Sx = wave_sum(sx);
    __syncthreads();
}

// One batch of up to NC columns from j0: the series stretch t[j0 ..
// j0 + NC + m + 16) staged skewed, then hs[p] = {df[j0+p-1], dg[j0+p-1],
// inv[j0+p], B(j0+p)} with the exact top-row values B(j) = sum_k x_k t_{j+k}
// - mu_j Sx from one Hankel tile.  Reads stay inside the padded buffers
// (their padding exceeds one 512-row tile beyond the last subsequence).
template <typename F, int NC = batch_cols<F>()>
__device__ void stage_batch(const double* __restrict__ T, const double* __restrict__ mu,
                            const F* __restrict__ df, const F* __restrict__ dg,
                            const F* __restrict__ inv, int32_t m, int64_t j0, const double* xp,
                            double Sx, double* ws, H4<F>* hs)
{
    const int lane = threadIdx.x;
    __syncthreads();  // the previous batch is consumed
#pragma unroll
    for (int u = 0; u < NC / 64; ++u) {
        const int64_t j = j0 + lane + 64 * u;
        H4<F>& h = hs[lane + 64 * u];
        h.df = df[j - 1];
        h.dg = dg[j - 1];
        h.inv = inv[j];
    }
    stage_skewed(ws, T + j0, NC + m + 16);
    __syncthreads();
    const pm_acc_t D = hankel16(xp, ws, 0, m, NC);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int p = hk_offset(q);
        if (p < NC) hs[p].B = (F)(D[q] - mu[j0 + p] * Sx);
    }
    __syncthreads();
}

// ----- sweep machinery shared by selection and refinement -----

// Column helpers are read-only during a sweep and wave-uniform per step:
// reading them through the constant address space lets the compiler use
// scalar loads.
template <typename T>
using cptr = const __attribute__((address_space(4))) T*;
template <typename T>
__device__ __forceinline__ cptr<T> as_const(const T* p)
{
    return (cptr<T>)p;
}

// Row state is kept as wave-uniform lane masks: bit l of dm[q] is set when
// the row of lane l, slot q is dead (pruned, invalid or past the end).
template <int Q>
__device__ __forceinline__ void rows_from_bitmap(const unsigned long long* alive, int64_t rbase,
                                                 unsigned long long (&dm)[Q])
{
    const unsigned int msk = (Q >= 32) ? 0xffffffffu : ((1u << Q) - 1u);
    const unsigned int live = (unsigned int)(load_word(&alive[rbase >> 6]) >> (rbase & 63)) & msk;
#pragma unroll
    for (int q = 0; q < Q; ++q) dm[q] = uniform64(__ballot(!((live >> q) & 1u)));
}

// Publish rows dead locally but still set in the bitmap; absorb rows the
// bitmap says are dead (`word`: the lane's bitmap word, loaded earlier so
// that its latency overlaps the sweep).  Returns true while some row of the
// tile is alive.
template <int Q>
__device__ __forceinline__ bool sync_rows_with(unsigned long long* alive, int64_t rbase,
                                               unsigned long long word,
                                               unsigned long long (&dm)[Q])
{
    const int lane = threadIdx.x;
    unsigned long long* wp = &alive[rbase >> 6];
    const int off = (int)(rbase & 63);
    const unsigned int msk = (Q >= 32) ? 0xffffffffu : ((1u << Q) - 1u);
    const unsigned int live = (unsigned int)(word >> off) & msk;
    unsigned int mine = 0;
#pragma unroll
    for (int q = 0; q < Q; ++q) mine |= (unsigned int)((dm[q] >> lane) & 1ull) << q;
    const unsigned int pub = live & mine;
    if (pub) atomicAnd(wp, ~((unsigned long long)pub << off));
    unsigned long long all = ~0ull;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        dm[q] = uniform64(dm[q] | __ballot(!((live >> q) & 1u)));
        all &= dm[q];
    }
    return __builtin_amdgcn_readfirstlane((int)(all != ~0ull)) != 0;
}

template <int Q>
__device__ __forceinline__ bool sync_rows(unsigned long long* alive, int64_t rbase,
                                          unsigned long long (&dm)[Q])
{
    return sync_rows_with<Q>(alive, rbase, load_word(&alive[rbase >> 6]), dm);
}

__device__ __forceinline__ void kill_columns(unsigned long long* alive, int64_t j0,
                                             unsigned long long bits)
{
    if (bits == 0ull) return;
    if (threadIdx.x == 0) {
        const int64_t w0 = j0 >> 6;
        const int off = (int)(j0 & 63);
        atomicAnd(&alive[w0], ~(bits << off));
        if (off) atomicAnd(&alive[w0 + 1], ~(bits >> (64 - off)));
    }
}

// The alive bits of columns j0 .. j0 + 63.
__device__ __forceinline__ unsigned long long live_columns(const unsigned long long* alive, int64_t j0)
{
    const int64_t w0 = j0 >> 6;
    const int off = (int)(j0 & 63);
    const unsigned long long lo = load_word(&alive[w0]) >> off;
    return uniform64(off ? lo | (load_word(&alive[w0 + 1]) << (64 - off)) : lo);
}

// One step of the diagonal recurrence for all Q slots of every lane.
// Registers rotate: before step u of a group of Q steps, slot q lives in
// C[(q - u) mod Q]; each register is updated in place, so the shift from
// slot q-1 to slot q costs nothing and only slot 0 needs the DPP move from
// the previous lane.  Lane 0 keeps the DPP's old operand instead: Bv, the
// exact boundary value of this step (identical in every lane).
template <typename F, int Q, int U>
__device__ __forceinline__ void advance(F (&C)[Q], const F (&a)[Q], const F (&b)[Q], F dfj, F dgj,
                                        F Bv)
{
#pragma unroll
    for (int q = 1; q < Q; ++q) {
        F& r = C[(q - 1 - U + 2 * Q) % Q];
        r = f_fma(a[q], dgj, f_fma(dfj, b[q], r));
    }
    F& r0 = C[(Q - 1 - U + 2 * Q) % Q];
    r0 = f_fma(a[0], dgj, f_fma(dfj, b[0], dpp_shr1(Bv, r0)));
}
template <int Q, int U>
__device__ __forceinline__ int slot_reg(int q)
{
    return (q - U - 1 + 2 * Q) % Q;  // register of slot q after step U
}

// ----- selection sweep -----
// A pair closer than r prunes both of its subsequences, and each remembers
// the other as its witness (SeriesDev::wit, stored as ~index: the pair's
// covariance is not known in FP64 yet).  At the next lengths k_advance tests
// a subsequence against its witness first, which prunes nearly all of them
// again without a sweep.
//
// Witness of a column hit in step s: the row of the lowest hit lane (mg: that
// lane's margins), kept in lane s of wcol until the block ends.
template <typename F, int Q>
__device__ __forceinline__ void col_witness(unsigned long long bal, const F (&mg)[Q], int32_t row0,
                                            int s, int32_t& wcol)
{
    const int l = __ffsll((long long)bal) - 1;
    int slot = 0;
#pragma unroll
    for (int q = 1; q < Q; ++q)
        if ((__ballot(mg[q] > F(0)) >> l) & 1ull) slot = q;
    wcol = (int)threadIdx.x == s ? row0 + Q * l + slot : wcol;
}

// One step U of a group: advance, then the pruning margin of every slot,
// C * inv_j - th = (rho - thr) / inv_i, which is > 0 exactly when the pair is
// closer than r.  The row keeps its largest margin (rm) and the block's
// largest with its step (bm; folded into the dead masks once per block); the
// column is hit when any slot's margin is > 0.
// MASK: only pairs with j >= i + m count (the triangle next to the band).
template <typename F, int Q, int U, bool MASK, bool WIT>
__device__ __forceinline__ void sel_step(F (&C)[Q], const F (&a)[Q], const F (&b)[Q],
                                         const F (&nth)[Q], F (&rm)[Q], F (&bm)[Q],
                                         const int32_t (&ri)[Q], F dfj, F dgj, F invj, F Bv,
                                         int32_t jm, int32_t row0, unsigned long long& colbits,
                                         int32_t& wcol, int s)
{
    advance<F, Q, U>(C, a, b, dfj, dgj, Bv);
    F mg[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        mg[q] = f_fma(C[slot_reg<Q, U>(q)], invj, nth[q]);
        if (MASK) mg[q] = (jm >= ri[q]) ? mg[q] : f_low<F>();
        rm[q] = fmax(rm[q], mg[q]);
        if (WIT) bm[q] = fmax(bm[q], pack_step(mg[q], s));
    }
    F cm = mg[0];
#pragma unroll
    for (int q = 1; q < Q; ++q) cm = fmax(cm, mg[q]);
    const unsigned long long bal = uniform64(__ballot(cm > F(0)));
    if (bal != 0ull) {
        colbits |= 1ull << s;
        if (WIT) col_witness<F, Q>(bal, mg, row0, s, wcol);
    }
}

template <typename F, int Q, bool MASK, bool WIT>
__device__ __forceinline__ void sel_block(const SweepArgs<F>& A, int64_t j0, int nst, F (&C)[Q],
                                          const F (&a)[Q], const F (&b)[Q], const F (&nth)[Q],
                                          F (&rm)[Q], F (&bm)[Q], const int32_t (&ri)[Q],
                                          const H4<F>* hs, int32_t row0,
                                          unsigned long long& colbits, int32_t& wcol)
{
    for (int s0 = 0; s0 < nst; s0 += Q) {
        const int64_t jg = j0 + s0;
        H4<F> hv[Q];
#pragma unroll
        for (int u = 0; u < Q; ++u) hv[u] = hs[s0 + u];
        const int32_t jm = (int32_t)(jg - A.m);
        const int left = nst - s0;
#define SEL_STEP(U)                                                                            \
    if ((U) < left)                                                                            \
        sel_step<F, Q, ((U) < Q ? (U) : 0), MASK, WIT>(                                       \
            C, a, b, nth, rm, bm, ri, hv[(U) % Q].df, hv[(U) % Q].dg, hv[(U) % Q].inv,         \
            hv[(U) % Q].B, jm + (U), row0, colbits, wcol, s0 + (U));
        static_assert(Q == 2 || Q == 4 || Q == 8, "Q must be 2, 4 or 8");
        SEL_STEP(0)
        SEL_STEP(1)
        if (Q > 2) {
            SEL_STEP(2)
            SEL_STEP(3)
        }
        if (Q > 4) {
            SEL_STEP(4)
            SEL_STEP(5)
            SEL_STEP(6)
            SEL_STEP(7)
        }
#undef SEL_STEP
    }
}

// Margins of every slot after one step of a full block (no masks); returns
// the lane's largest margin (the column test).
template <typename F, int Q, int U>
__device__ __forceinline__ F sel_margins(F (&C)[Q], const F (&a)[Q], const F (&b)[Q],
                                         const F (&nth)[Q], const H4<F>& h, F (&mg)[Q])
{
    advance<F, Q, U>(C, a, b, h.df, h.dg, h.B);
#pragma unroll
    for (int q = 0; q < Q; ++q) mg[q] = f_fma(C[slot_reg<Q, U>(q)], h.inv, nth[q]);
    F cm = mg[0];
#pragma unroll
    for (int q = 1; q < Q; ++q) cm = fmax(cm, mg[q]);
    return cm;
}

template <typename F, int Q, bool WIT>
__device__ __forceinline__ void sel_group(F (&C)[Q], const F (&a)[Q], const F (&b)[Q],
                                          const F (&nth)[Q], F (&rm)[Q], F (&bm)[Q],
                                          const H4<F> (&hv)[Q], int32_t row0,
                                          unsigned long long& colbits, int32_t& wcol, int s0)
{
    unsigned long long bal[Q];
#define SEL_PAIR(U)                                                                    \
    {                                                                                  \
        F m0[Q], m1[Q];                                                                \
        const F c0 = sel_margins<F, Q, (U)>(C, a, b, nth, hv[(U)], m0);                \
        const unsigned long long b0 = uniform64(__ballot(c0 > F(0)));                  \
        const F c1 = sel_margins<F, Q, (U) + 1>(C, a, b, nth, hv[(U) + 1], m1);        \
        const unsigned long long b1 = uniform64(__ballot(c1 > F(0)));                  \
        _Pragma("unroll") for (int q = 0; q < Q; ++q) {                                \
            rm[q] = fmax(rm[q], fmax(m0[q], m1[q]));                                   \
            if (WIT)                                                                   \
                bm[q] = fmax(bm[q], fmax(pack_step(m0[q], s0 + (U)), pack_step(m1[q], s0 + (U) + 1))); \
        }                                                                              \
        if (WIT) {                                                                     \
            if (b0 != 0ull) {                                                          \
                colbits |= 1ull << (s0 + (U));                                         \
                col_witness<F, Q>(b0, m0, row0, s0 + (U), wcol);                       \
            }                                                                          \
            if (b1 != 0ull) {                                                          \
                colbits |= 1ull << (s0 + (U) + 1);                                     \
                col_witness<F, Q>(b1, m1, row0, s0 + (U) + 1, wcol);                   \
            }                                                                          \
        } else {                                                                       \
            bal[(U)] = b0;                                                             \
            bal[(U) + 1] = b1;                                                         \
        }                                                                              \
    }
    static_assert(Q == 2 || Q == 4 || Q == 8, "Q must be 2, 4 or 8");
    SEL_PAIR(0)
    if (Q > 2) SEL_PAIR((Q > 2 ? 2 : 0))
    if (Q > 4) {
        SEL_PAIR((Q > 4 ? 4 : 0))
        SEL_PAIR((Q > 4 ? 6 : 0))
    }
#undef SEL_PAIR
    if (!WIT) {
        unsigned long long g = 0ull;
#pragma unroll
        for (int u = 0; u < Q; ++u)
            if (bal[u] != 0ull) g |= 1ull << u;
        colbits |= g << s0;
    }
}

// A full block of 64 steps with every pair a non-self match, in groups of Q
// steps without per-step tests: row maxima fold two steps per max.  (Reading
// the next group's helpers ahead costs registers, hence occupancy, and
// measured slower.)
template <typename F, int Q, bool WIT>
__device__ __forceinline__ void sel_block_full(F (&C)[Q], const F (&a)[Q], const F (&b)[Q],
                                               const F (&nth)[Q], F (&rm)[Q], F (&bm)[Q],
                                               const H4<F>* hs, int32_t row0,
                                               unsigned long long& colbits, int32_t& wcol)
{
    for (int s0 = 0; s0 < 64; s0 += Q) {
        H4<F> hv[Q];
#pragma unroll
        for (int u = 0; u < Q; ++u) hv[u] = hs[s0 + u];
        sel_group<F, Q, WIT>(C, a, b, nth, rm, bm, hv, row0, colbits, wcol, s0);
    }
}

// WIT: keep the witnesses of the rows and columns it prunes (a search; a bare
// range search has no next length and saves the instructions): WIT_INLINE with
// every pair, 1.5 operations on four, for the first pass, where most blocks
// prune; WIT_REPLAY by a second run over a block in which something fell, for the
// split pass, where few do.  (Split pass of a first length, 300,000 points: white
// noise, m = 50, 13.4 ms inline, 9.1 so; a periodic signal whose level jumps, of
// which the FP32 sweeps prune nothing, m = 64, 16.0 and 9.9.)
enum { WIT_OFF = 0, WIT_INLINE, WIT_REPLAY };
template <typename F, int Q, int WIT>
__device__ void sel_item(const SweepArgs<F>& A, int64_t i0, int64_t jbeg, int64_t jend, F thr,
                         double* lds, unsigned long long& evals, uint32_t* work)
{
    constexpr int R = 64 * Q;
    constexpr bool INL = WIT == WIT_INLINE;
    i0 = uniform_i64(i0);
    jbeg = uniform_i64(jbeg);
    jend = uniform_i64(jend);
    const int lane = threadIdx.x;
    const int32_t m = A.m;
    const int64_t N = A.N;
    const int64_t rbase = i0 + (int64_t)Q * lane;
    const int32_t row0 = (int32_t)i0;

    unsigned long long dm[Q];
    rows_from_bitmap<Q>(A.alive, rbase, dm);
    {
        unsigned long long all = ~0ull;
#pragma unroll
        for (int q = 0; q < Q; ++q) all &= dm[q];
        if (all == ~0ull) return;
    }
    double* xp = lds;
    double* ws = lds + hk_vp_doubles(m);
    H4<F>* hs = (H4<F>*)(lds + sweep_hs_offset(m, R, batch_cols<F>()));
    double Sx, Sy;
    F C[Q];
    {
        double acc[Q];
        item_start<Q>(A.T, A.mu, m, i0, jbeg, xp, ws, (double*)hs, Sx, Sy, acc);
#pragma unroll
        for (int q = 0; q < Q; ++q) C[q] = (F)acc[q];
    }
    F a[Q], b[Q], nth[Q], rm[Q];
    int32_t ri[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int64_t i = rbase + q;
        const bool top = (lane == 0) && (q == 0);
        const int64_t ip = top ? i : i - 1;
        a[q] = top ? F(0) : A.df[ip];
        b[q] = top ? F(0) : A.dg[ip];
        const F invi = A.inv[i];
        // margin offset: C * inv_j - thr / inv_i > 0  <=>  rho > thr
        nth[q] = (i < N && invi > F(0)) ? -(thr / invi) : f_low<F>();
        ri[q] = (int32_t)i;
        rm[q] = f_low<F>();
    }
    // Rows of block [j0, j0 + 64) that fell in it keep the step as witness.
    auto row_witness = [&](const F (&bm)[Q], int64_t j0) {
#pragma unroll
        for (int q = 0; q < Q; ++q)
            if (bm[q] > F(0) && !((dm[q] >> lane) & 1ull))
                A.wit[rbase + q] = ~(int32_t)(j0 + step_of(bm[q]));
    };
    // column jbeg
    {
        const F invj = A.inv[jbeg];
        F mg[Q], bm[Q];
        F cm = f_low<F>();
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            mg[q] = f_fma(C[q], invj, nth[q]);
            mg[q] = ((int32_t)(jbeg - m) >= ri[q]) ? mg[q] : f_low<F>();
            rm[q] = fmax(rm[q], mg[q]);
            bm[q] = pack_step(mg[q], 0);
            cm = fmax(cm, mg[q]);
        }
        const unsigned long long bal = uniform64(__ballot(cm > F(0)));
        if (WIT == WIT_OFF) {
            kill_columns(A.alive, jbeg, bal ? 1ull : 0ull);
        } else if (bal != 0ull) {
            int32_t wcol = 0;
            col_witness<F, Q>(bal, mg, row0, 0, wcol);
            if (live_columns(A.alive, jbeg) & 1ull) {
                if (lane == 0) A.wit[jbeg] = ~wcol;
                kill_columns(A.alive, jbeg, 1ull);
            }
            row_witness(bm, jbeg);
        }
#pragma unroll
        for (int q = 0; q < Q; ++q) dm[q] |= uniform64(__ballot(rm[q] > F(0)));
    }
    unsigned long long ev = pair_count(i0, std::min<int64_t>(i0 + R, N), jbeg, 1, m, false);
    bool go = sync_rows<Q>(A.alive, rbase, dm);
    uint32_t nblk = 0;
    int64_t j = jbeg + 1;
    while (go && j < jend) {
        // a batch of up to batch_cols columns (boundary values from one
        // Hankel tile), swept in blocks of 64 with the bitmap synchronised after
        // each
        stage_batch<F>(A.T, A.mu, A.df, A.dg, A.inv, m, j, xp, Sx, ws, hs);
        const int64_t jb_end = std::min<int64_t>(jend, j + batch_cols<F>());
        for (int sb = 0; go && j < jb_end; ++sb) {
            const int nst = (int)std::min<int64_t>(64, jb_end - j);
            const H4<F>* hb = hs + 64 * sb;
            const unsigned long long word = load_word(&A.alive[rbase >> 6]);
            unsigned long long colbits = 0ull;
            int32_t wcol = 0;
            F bm[Q], C0[Q];
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                bm[q] = f_low<F>();
                C0[q] = C[q];
            }
            const bool full = (j - (i0 + R - 1)) >= m;
            if (Q <= 4 && full && nst == 64)  // taller tiles: the general path keeps fewer registers
                sel_block_full<F, Q, INL>(C, a, b, nth, rm, bm, hb, row0, colbits, wcol);
            else if (full)
                sel_block<F, Q, false, INL>(A, j, nst, C, a, b, nth, rm, bm, ri, hb, row0, colbits, wcol);
            else
                sel_block<F, Q, true, INL>(A, j, nst, C, a, b, nth, rm, bm, ri, hb, row0, colbits, wcol);
            if (WIT == WIT_OFF) {
                kill_columns(A.alive, j, colbits);
            } else if (colbits != 0ull) {
                // only columns still alive: the others keep the witness they have
                colbits &= live_columns(A.alive, j);
                unsigned long long fell = colbits;
                if (WIT == WIT_REPLAY) {
#pragma unroll
                    for (int q = 0; q < Q; ++q) fell |= uniform64(__ballot(rm[q] > F(0))) & ~dm[q];
                }
                if (WIT == WIT_REPLAY && fell != 0ull) {
                    F rm0[Q];
                    unsigned long long cb = 0ull;
#pragma unroll
                    for (int q = 0; q < Q; ++q) rm0[q] = f_low<F>();
                    sel_block<F, Q, true, true>(A, j, nst, C0, a, b, nth, rm0, bm, ri, hb, row0, cb, wcol);
                }
                if ((colbits >> lane) & 1ull) A.wit[j + lane] = ~wcol;
                row_witness(bm, j);
                kill_columns(A.alive, j, colbits);
            }
#pragma unroll
            for (int q = 0; q < Q; ++q) dm[q] |= uniform64(__ballot(rm[q] > F(0)));
            ev += pair_count(i0, std::min<int64_t>(i0 + R, N), j, nst, m, false);
            j += nst;
            go = sync_rows_with<Q>(A.alive, rbase, word, dm);
            ++nblk;
        }
    }
    if (work && lane == 0 && nblk) atomicAdd(work, nblk);
    // rows still alive: their largest correlation over this item's columns
    // (rho - thr = margin * inv_i), for the refinement that sweeps only the
    // left side of tiles whose rows are all clearly below the threshold;
    // rows above thr64 - guard are marked in unc
    const double ulim = 2.0 * A.ctrl->thr64 - A.ctrl->thr_sel;
    unsigned long long ub[Q];
    unsigned long long uany = 0ull;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int64_t i = rbase + q;
        bool u = false;
        if (!((dm[q] >> lane) & 1ull) && i < N && rm[q] > F(0.5) * f_low<F>()) {
            const double rt = (double)rm[q] * (double)A.inv[i] + (double)thr;
            atomicMax(&A.rhs[i], ord_of(rt));
            u = rt > ulim;
        }
        ub[q] = uniform64(__ballot(u));
        uany |= ub[q];
    }
    // one atomic per bitmap word: lane l's slot q is row Q l + q of the tile
    if (uany != 0ull && lane == 0) {
        constexpr int LPW = 64 / Q;  // lanes per bitmap word
#pragma unroll
        for (int wd = 0; wd < Q; ++wd) {
            unsigned long long mask = 0ull;
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                unsigned long long lb = (ub[q] >> (wd * LPW)) & ((LPW == 64) ? ~0ull : ((1ull << LPW) - 1ull));
                while (lb) {
                    const int l = __ffsll((long long)lb) - 1;
                    lb &= lb - 1ull;
                    mask |= 1ull << (Q * l + q);
                }
            }
            if (mask) atomicOr(&A.unc[(i0 >> 6) + wd], mask);
        }
    }
    evals += ev;
}

template <typename F>
__device__ __forceinline__ F sel_threshold(const Ctrl* c);
template <>
__device__ __forceinline__ float sel_threshold<float>(const Ctrl* c) { return c->thr32; }
template <>
__device__ __forceinline__ double sel_threshold<double>(const Ctrl* c) { return c->thr_sel; }

template <typename F>
__device__ __forceinline__ SweepArgs<F> args_of(const SeriesDev& s, Ctrl* c);
template <>
__device__ __forceinline__ SweepArgs<float> args_of<float>(const SeriesDev& s, Ctrl* c)
{
    SweepArgs<float> A;
    A.T = s.T;
    A.mu = cur_mu(s, c);
    A.df = s.df32;
    A.dg = s.dg32;
    A.inv = s.inv32;
    A.alive = s.alive;
    A.rho = s.rho;
    A.rhs = s.rhs;
    A.unc = s.unc;
    A.twork = s.twork;
    A.wit = s.wit;
    A.ctrl = c;
    A.m = c->m;
    A.N = s.n - A.m + 1;
    return A;
}
template <>
__device__ __forceinline__ SweepArgs<double> args_of<double>(const SeriesDev& s, Ctrl* c)
{
    SweepArgs<double> A;
    A.T = s.T;
    A.mu = cur_mu(s, c);
    A.df = s.df64;
    A.dg = s.dg64;
    A.inv = s.inv64;
    A.alive = s.alive;
    A.rho = s.rho;
    A.rhs = s.rhs;
    A.unc = s.unc;
    A.twork = s.twork;
    A.wit = s.wit;
    A.ctrl = c;
    A.m = c->m;
    A.N = s.n - A.m + 1;
    return A;
}

// ----- refinement sweep (FP64) -----
// MASK 0: all pairs valid; 1: right side (j >= i + m); 2: left side (j <= i - m).
template <int Q, int U, int MASK>
__device__ __forceinline__ void ref_step(double (&C)[Q], const double (&a)[Q], const double (&b)[Q],
                                         double (&mx)[Q], const int32_t (&ri)[Q], double dfj,
                                         double dgj, double invj, double Bv, int32_t jm,
                                         int32_t jp)
{
    advance<double, Q, U>(C, a, b, dfj, dgj, Bv);
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        double v = C[slot_reg<Q, U>(q)] * invj;
        if (MASK == 1) v = (jm >= ri[q]) ? v : -f_inf<double>();
        if (MASK == 2) v = (jp <= ri[q]) ? v : -f_inf<double>();
        mx[q] = fmax(mx[q], v);
    }
}

template <int Q, int MASK>
__device__ __forceinline__ void ref_block(const SweepArgs<double>& A, int64_t j0, int nst,
                                          double (&C)[Q], const double (&a)[Q],
                                          const double (&b)[Q], double (&mx)[Q],
                                          const int32_t (&ri)[Q], const H4<double>* hs)
{
    for (int s0 = 0; s0 < nst; s0 += Q) {
        const int64_t jg = j0 + s0;
        H4<double> hv[Q];
#pragma unroll
        for (int u = 0; u < Q; ++u) hv[u] = hs[s0 + u];
        const int32_t jm = (int32_t)(jg - A.m), jp = (int32_t)(jg + A.m);
        const int left = nst - s0;
#define REF_STEP(U)                                                                             \
    if ((U) < left)                                                                             \
        ref_step<Q, ((U) < Q ? (U) : 0), MASK>(C, a, b, mx, ri, hv[(U) % Q].df, hv[(U) % Q].dg, \
                                               hv[(U) % Q].inv, hv[(U) % Q].B, jm + (U),        \
                                               jp + (U));
        static_assert(Q == 2 || Q == 4 || Q == 8, "Q must be 2, 4 or 8");
        REF_STEP(0)
        REF_STEP(1)
        if (Q > 2) {
            REF_STEP(2)
            REF_STEP(3)
        }
        if (Q > 4) {
            REF_STEP(4)
            REF_STEP(5)
            REF_STEP(6)
            REF_STEP(7)
        }
#undef REF_STEP
    }
}

// A full refinement block of 64 steps (every pair valid) in groups of Q
// steps without per-step tests; row maxima fold two steps per max.
template <int Q>
__device__ __forceinline__ void ref_block_full(double (&C)[Q], const double (&a)[Q],
                                               const double (&b)[Q], double (&mx)[Q],
                                               const H4<double>* hs)
{
    for (int s0 = 0; s0 < 64; s0 += Q) {
        H4<double> hv[Q];
#pragma unroll
        for (int u = 0; u < Q; ++u) hv[u] = hs[s0 + u];
#define REF_PAIR(U)                                                                        \
    {                                                                                      \
        double v0[Q], v1[Q];                                                               \
        advance<double, Q, (U)>(C, a, b, hv[(U)].df, hv[(U)].dg, hv[(U)].B);               \
        _Pragma("unroll") for (int q = 0; q < Q; ++q) v0[q] =                              \
            C[slot_reg<Q, (U)>(q)] * hv[(U)].inv;                                          \
        advance<double, Q, (U) + 1>(C, a, b, hv[(U) + 1].df, hv[(U) + 1].dg, hv[(U) + 1].B); \
        _Pragma("unroll") for (int q = 0; q < Q; ++q) v1[q] =                              \
            C[slot_reg<Q, (U) + 1>(q)] * hv[(U) + 1].inv;                                  \
        _Pragma("unroll") for (int q = 0; q < Q; ++q) mx[q] = fmax(mx[q], fmax(v0[q], v1[q])); \
    }
        static_assert(Q == 2 || Q == 4 || Q == 8, "Q must be 2, 4 or 8");
        REF_PAIR(0)
        if (Q > 2) REF_PAIR((Q > 2 ? 2 : 0))
        if (Q > 4) {
            REF_PAIR((Q > 4 ? 4 : 0))
            REF_PAIR((Q > 4 ? 6 : 0))
        }
#undef REF_PAIR
    }
}

// The block of nst steps from j0 again (same operations, same values): every
// slot keeps the first column of the block that prunes it.
template <int Q>
__device__ __forceinline__ void ref_replay(const SweepArgs<double>& A, int64_t j0, int nst, bool left,
                                           double (&C)[Q], const double (&a)[Q],
                                           const double (&b)[Q], const double (&iv)[Q],
                                           const int32_t (&ri)[Q], double thr,
                                           const H4<double>* hs, int32_t (&wj)[Q])
{
    for (int s0 = 0; s0 < nst; s0 += Q) {
        auto step = [&](auto U) {
            constexpr int u = decltype(U)::value;
            if (u < Q && s0 + u < nst) {
                const H4<double> h = hs[s0 + u];
                advance<double, Q, (u < Q ? u : 0)>(C, a, b, h.df, h.dg, h.B);
                const int32_t j = (int32_t)(j0 + s0 + u);
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    const double v = C[slot_reg<Q, (u < Q ? u : 0)>(q)] * h.inv;
                    const bool ok = left ? j + A.m <= ri[q] : j - A.m >= ri[q];
                    if (ok && v * iv[q] > thr && wj[q] < 0) wj[q] = j;
                }
            }
        };
        step(std::integral_constant<int, 0>());
        step(std::integral_constant<int, 1>());
        if (Q > 2) {
            step(std::integral_constant<int, 2>());
            step(std::integral_constant<int, 3>());
        }
        if (Q > 4) {
            step(std::integral_constant<int, 4>());
            step(std::integral_constant<int, 5>());
            step(std::integral_constant<int, 6>());
            step(std::integral_constant<int, 7>());
        }
    }
}

template <int Q, int NC = batch_cols<double>(), bool WIT = false>
__device__ void ref_item(const SweepArgs<double>& A, int64_t i0, int64_t jbeg, int64_t jend,
                         bool left, double thr, int prune, double* lds, unsigned long long& evals)
{
    constexpr int R = 64 * Q;
    i0 = uniform_i64(i0);
    jbeg = uniform_i64(jbeg);
    jend = uniform_i64(jend);
    const int lane = threadIdx.x;
    const int32_t m = A.m;
    const int64_t N = A.N;
    const int64_t rbase = i0 + (int64_t)Q * lane;
    const Ctrl* c = A.ctrl;

    unsigned long long dm[Q];
    rows_from_bitmap<Q>(A.alive, rbase, dm);
    {
        unsigned long long all = ~0ull;
#pragma unroll
        for (int q = 0; q < Q; ++q) all &= dm[q];
        if (all == ~0ull) return;
    }
    double* xp = lds;
    double* ws = lds + hk_vp_doubles(m);
    H4<double>* hs = (H4<double>*)(lds + sweep_hs_offset(m, R, NC));
    double Sx, Sy;
    double C[Q];
    item_start<Q>(A.T, A.mu, m, i0, jbeg, xp, ws, (double*)hs, Sx, Sy, C);
    double a[Q], b[Q], mx[Q];
    int32_t ri[Q];
    // 1/(sqrt(m) sigma_i) of the lane's rows
    double* rowinv = lds + sweep_rowv_offset(m, R, 8, NC);
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int64_t i = rbase + q;
        const bool top = (lane == 0) && (q == 0);
        const int64_t ip = top ? i : i - 1;
        a[q] = top ? 0.0 : A.df[ip];
        b[q] = top ? 0.0 : A.dg[ip];
        rowinv[Q * lane + q] = A.inv[i];
        mx[q] = -f_inf<double>();
        ri[q] = (int32_t)i;
    }
    {
        const double invj = A.inv[jbeg];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const bool ok = left ? ((int32_t)(jbeg + m) <= ri[q]) : ((int32_t)(jbeg - m) >= ri[q]);
            if (ok) mx[q] = fmax(mx[q], C[q] * invj);
        }
    }
    unsigned long long ev = pair_count(i0, std::min<int64_t>(i0 + R, N), jbeg, 1, m, left);
    int64_t j = jbeg + 1;
    bool go = true;
    while (go && j < jend) {
        stage_batch<double, NC>(A.T, A.mu, A.df, A.dg, A.inv, m, j, xp, Sx, ws, hs);
        const int64_t jb_end = std::min<int64_t>(jend, j + NC);
        for (int sb = 0; go && j < jb_end; ++sb) {
            const int nst = (int)std::min<int64_t>(64, jb_end - j);
            const H4<double>* hb = hs + 64 * sb;
            const unsigned long long word = load_word(&A.alive[rbase >> 6]);
            double C0[Q];
            if (WIT) {
#pragma unroll
                for (int q = 0; q < Q; ++q) C0[q] = C[q];
            }
            bool full;
            if (left) full = (i0 - (j + nst - 1)) >= m;
            else full = (j - (i0 + R - 1)) >= m;
            if (full && nst == 64) ref_block_full<Q>(C, a, b, mx, hb);
            else if (full) ref_block<Q, 0>(A, j, nst, C, a, b, mx, ri, hb);
            else if (left) ref_block<Q, 2>(A, j, nst, C, a, b, mx, ri, hb);
            else ref_block<Q, 1>(A, j, nst, C, a, b, mx, ri, hb);
            ev += pair_count(i0, std::min<int64_t>(i0 + R, N), j, nst, m, left);
            j += nst;
            if (prune) {
                unsigned long long fell = 0ull;
                double iv[Q];
                bool now[Q];
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    iv[q] = rowinv[Q * lane + q];
                    now[q] = iv[q] > 0.0 && mx[q] * iv[q] > thr && !((dm[q] >> lane) & 1ull);
                    const unsigned long long k = uniform64(__ballot(now[q]));
                    fell |= k;
                    dm[q] |= k;
                }
                if (WIT && fell != 0ull) {
                    // the rows that fell in this block: their witnesses
                    // (one found in the item's first column falls here too)
                    int32_t wj[Q];
#pragma unroll
                    for (int q = 0; q < Q; ++q) wj[q] = -1;
                    ref_replay<Q>(A, j - nst, nst, left, C0, a, b, iv, ri, thr, hb, wj);
#pragma unroll
                    for (int q = 0; q < Q; ++q)
                        if (now[q]) A.wit[rbase + q] = ~(wj[q] >= 0 ? wj[q] : (int32_t)jbeg);
                }
            }
            go = sync_rows_with<Q>(A.alive, rbase, word, dm);
        }
    }
    double invi[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) invi[q] = rowinv[Q * lane + q];
    if (prune && jend == jbeg + 1) {  // the only column: no block tested it
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const bool now = invi[q] > 0.0 && mx[q] * invi[q] > thr && !((dm[q] >> lane) & 1ull);
            if (WIT && now) A.wit[rbase + q] = ~(int32_t)jbeg;
            dm[q] |= uniform64(__ballot(now));
        }
    }
    // flat rows: correlation 1 with another flat window, 0 with any other
    const int64_t flo = c->flat_min, fhi = c->flat_max;
    bool flat[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int64_t i = rbase + q;
        flat[q] = (i < N) && !(invi[q] > 0.0);
        if (flat[q]) {
            const bool lo_ok = flo >= 0 && flo <= i - m, hi_ok = fhi >= 0 && fhi >= i + m;
            const bool partner = lo_ok || hi_ok;
            mx[q] = partner ? 1.0 : 0.0;
            if (WIT && prune && mx[q] > thr)
                A.wit[i] = ~(int32_t)(lo_ok ? flo : hi_ok ? fhi : i + m < N ? i + m : i - m);
        }
        if (prune) dm[q] |= uniform64(__ballot(flat[q] && mx[q] > thr));
    }
    sync_rows<Q>(A.alive, rbase, dm);
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int64_t i = rbase + q;
        const bool dead = (dm[q] >> lane) & 1ull;
        if (!dead && i < N && mx[q] > -f_inf<double>()) {
            const double rho = flat[q] ? mx[q] : mx[q] * invi[q];
            atomicMax(&A.rho[i], ord_of(rho));
        }
    }
    evals += ev;
}

// The first local item of this workgroup in a series whose items start at
// global number cum: the smallest it >= 0 with (cum + it) mod G = g.
__device__ __forceinline__ unsigned long long first_item(unsigned long long cum)
{
    const unsigned long long G = gridDim.x;
    return ((unsigned long long)blockIdx.x + G - cum % G) % G;
}

// ----- diagonal band pre-pass of the first selection pass -----
// The pairs (i, i + d), d in [m, m + BAND_D), of every subsequence — its
// nearest non-self matches on the right — swept down the diagonals.  A work
// item is one wavefront owning BAND_D consecutive diagonals (BAND_Q per
// lane, consecutive) over BAND_S consecutive rows.  Each lane carries its
// diagonals' values from row to row with the centred recurrence (R23) in
// the selection precision, started from exact FP64 values of the item's top
// row (one Hankel tile on the matrix cores), so every value is at most
// BAND_S steps from an exact one, as in the row-tile sweeps.  A pair that
// passes the selection test kills both subsequences: the row through the
// wave's ballot of the step, the column through per-lane bit histories
// (one add-with-carry per pair) merged in LDS and published once per item.
// No tile straddles the exclusion zone, so every pair evaluated counts.
// The pass only prunes: the row-tile passes after it still sweep each tile
// with a live row from its first non-self column, which keeps the recorded
// right-side maxima of the surviving rows complete.
constexpr int BAND_Q = 4;
constexpr int BAND_D = 64 * BAND_Q;      // diagonals per item
constexpr int BAND_S = 256;              // rows per item (a multiple of 64)
constexpr int BAND_C = BAND_S + BAND_D;  // column records per item (the last one is padding)
constexpr int BAND_W32 = (BAND_C + 64) / 32;  // column-kill words, aligned to the bitmap
static_assert(BAND_D == HK_TILE, "one Hankel tile gives the top row's values");

__host__ __device__ constexpr size_t band_lds_bytes(int m, int fbytes)
{
    // phase 1: top-row window + skewed series stretch for the Hankel tile
    // phase 2: column records, row records, column-kill bits
    return (size_t)8 * (hk_vp_doubles(m) + ((hk_skew(HK_TILE + m + 16 - 1) + 1 + 3) & ~3)) >
                   (size_t)4 * fbytes * (BAND_C + BAND_S) + 4 * BAND_W32
               ? (size_t)8 * (hk_vp_doubles(m) + ((hk_skew(HK_TILE + m + 16 - 1) + 1 + 3) & ~3))
               : (size_t)4 * fbytes * (BAND_C + BAND_S) + 4 * BAND_W32;
}

// One row step's kill tests, for the BAND_Q pairs of every lane: per slot
// km = 2 km + (mg > 0) (the lane's column history, newest step in bit 0) as
// one compare and one add-with-carry, and the row's history rh = 2 rh +
// (some pair of the wave has mg > 0) in scalar instructions.  (Written as C,
// the compiler reassociates the unrolled histories into sums of selected
// powers of two and keeps every step's masks alive until the end.)
#define BAND_CMP_F32 "v_cmp_lt_f32_e64"
#define BAND_CMP_F64 "v_cmp_lt_f64_e64"
#define BAND_HIT_ASM(CMP)                                                                   \
    CMP " %[m0], 0, %[g0]\n\t"                                                              \
        "v_addc_co_u32_e64 %[k0], %[co], %[k0], %[k0], %[m0]\n\t" CMP " %[m1], 0, %[g1]\n\t" \
        "v_addc_co_u32_e64 %[k1], %[co], %[k1], %[k1], %[m1]\n\t" CMP " %[m2], 0, %[g2]\n\t" \
        "v_addc_co_u32_e64 %[k2], %[co], %[k2], %[k2], %[m2]\n\t" CMP " %[m3], 0, %[g3]\n\t" \
        "v_addc_co_u32_e64 %[k3], %[co], %[k3], %[k3], %[m3]\n\t"                           \
        "s_or_b64 %[m0], %[m0], %[m1]\n\t"                                                   \
        "s_or_b64 %[m2], %[m2], %[m3]\n\t"                                                   \
        "s_or_b64 %[m0], %[m0], %[m2]\n\t"                                                   \
        "s_cmp_lg_u64 %[m0], 0\n\t"                                                          \
        "s_addc_u32 %[rh], %[rh], %[rh]"
template <typename F>
__device__ __forceinline__ void band_hits(const F (&mg)[BAND_Q], unsigned int (&km)[BAND_Q],
                                          unsigned int& rh)
{
    static_assert(BAND_Q == 4, "four slots per lane");
    unsigned long long m0, m1, m2, m3, co;
    if constexpr (sizeof(F) == 4) {
        asm(BAND_HIT_ASM(BAND_CMP_F32)
            : [k0] "+v"(km[0]), [k1] "+v"(km[1]), [k2] "+v"(km[2]), [k3] "+v"(km[3]),
              [rh] "+s"(rh), [m0] "=&s"(m0), [m1] "=&s"(m1), [m2] "=&s"(m2), [m3] "=&s"(m3),
              [co] "=&s"(co)
            : [g0] "v"(mg[0]), [g1] "v"(mg[1]), [g2] "v"(mg[2]), [g3] "v"(mg[3])
            : "scc");
    } else {
        asm(BAND_HIT_ASM(BAND_CMP_F64)
            : [k0] "+v"(km[0]), [k1] "+v"(km[1]), [k2] "+v"(km[2]), [k3] "+v"(km[3]),
              [rh] "+s"(rh), [m0] "=&s"(m0), [m1] "=&s"(m1), [m2] "=&s"(m2), [m3] "=&s"(m3),
              [co] "=&s"(co)
            : [g0] "v"(mg[0]), [g1] "v"(mg[1]), [g2] "v"(mg[2]), [g3] "v"(mg[3])
            : "scc");
    }
}

template <typename F>
__global__ __launch_bounds__(64) void k_select_band(SeriesDev* S, int B, const int64_t* __restrict__ pfx,
                                                   int wit)
{
    extern __shared__ double lds[];
    const int b = series_of(pfx, B, blockIdx.x);
    const SeriesDev& s = S[b];
    Ctrl* c = s.ctrl;
    if (!c->active || !c->prune || lean_round(c) || taking_parts(c)) return;
    const SweepArgs<F> A = args_of<F>(s, c);
    const int32_t m = A.m;
    const int64_t i0 = (int64_t)(blockIdx.x - pfx[b]) * BAND_S;
    const int64_t j0 = i0 + m;  // column of the top row on the first diagonal
    // every column of the item inside the series (the tail is left to the
    // row-tile passes)
    if (j0 + BAND_C - 1 > A.N) return;
    const int lane = threadIdx.x;
    const F thr = sel_threshold<F>(c);

    // exact top-row values C(i0, j0 + p), p < 256
    F C[BAND_Q];
    {
        double* xp = lds;
        double* ws = lds + hk_vp_doubles(m);
        const double mui0 = A.mu[i0];
        const int nvp = hk_vp_doubles(m);
        double sx = 0.0;
        for (int t = lane; t < nvp; t += 64) {
            const int k = t - HK_PAD;
            double v = 0.0;
            if (k >= 0 && k < m) {
                v = A.T[i0 + k] - mui0;
                sx += v;
            }
            xp[t] = v;
        }
        const double Sx = wave_sum(sx);
        stage_skewed(ws, A.T + j0, HK_TILE + m + 16);
        __syncthreads();
        const pm_acc_t D = hankel16(xp, ws, 0, m);
        __syncthreads();  // the stretch is consumed: its space takes the values
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int p = hk_offset(q);
            ws[p] = D[q] - A.mu[j0 + p] * Sx;
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < BAND_Q; ++q) C[q] = (F)ws[BAND_Q * lane + q];
        __syncthreads();  // phase 1 is over
    }

    // column records (helpers of column j0 + e: df[j-1], dg[j-1], inv[j])
    // and row records (df[i-1], dg[i-1], -thr / inv_i: the margin offset)
    H4<F>* colh = (H4<F>*)lds;
    H4<F>* rowh = colh + BAND_C;
    uint32_t* kb = (uint32_t*)(rowh + BAND_S);
    {
        constexpr int NE = BAND_C / 64, NT = BAND_S / 64;
        F v[NE][3];
#pragma unroll
        for (int u = 0; u < NE; ++u) {
            const int64_t j = j0 + lane + 64 * u;
            v[u][0] = A.df[j - 1];
            v[u][1] = A.dg[j - 1];
            v[u][2] = A.inv[j];
        }
#pragma unroll
        for (int u = 0; u < NE; ++u) {
            H4<F> h;
            h.df = v[u][0];
            h.dg = v[u][1];
            h.inv = v[u][2];
            h.B = F(0);
            colh[lane + 64 * u] = h;
        }
        F r[NT][3];
#pragma unroll
        for (int u = 0; u < NT; ++u) {
            const int t = lane + 64 * u;
            const int64_t ip = i0 + t - (t > 0 ? 1 : 0);  // row 0 takes no step
            r[u][0] = A.df[ip];
            r[u][1] = A.dg[ip];
            r[u][2] = A.inv[i0 + t];
        }
#pragma unroll
        for (int u = 0; u < NT; ++u) {
            H4<F> h;
            h.df = r[u][0];
            h.dg = r[u][1];
            h.inv = r[u][2] > F(0) ? -(thr / r[u][2]) : -f_inf<F>();
            h.B = F(0);
            rowh[lane + 64 * u] = h;
        }
        if (lane < BAND_W32) kb[lane] = 0u;
    }
    __syncthreads();

    // row i0 + t, slot q of the lane: diagonal m + BAND_Q lane + q, column
    // record t + BAND_Q lane + q, held in hv[(q + t) % BAND_Q] (the records
    // shift down one slot per row; the top slot is read from LDS)
    const int off = (int)(j0 & 63);
    H4<F> hv[BAND_Q];
#pragma unroll
    for (int q = 0; q < BAND_Q; ++q) hv[q] = colh[BAND_Q * lane + q];
    unsigned int km[BAND_Q];
#pragma unroll
    for (int q = 0; q < BAND_Q; ++q) km[q] = 0u;
    unsigned long long rowbits = 0ull;
    unsigned int rhist = 0u;
    for (int t0 = 0; t0 < BAND_S; t0 += 32) {
#pragma unroll
        for (int u = 0; u < 32; ++u) {
            const int t = t0 + u;
            const H4<F> rh = rowh[t];
            if (u != 0 || t0 != 0) {
                hv[(BAND_Q - 1 + u) % BAND_Q] = colh[t + BAND_Q * lane + BAND_Q - 1];
#pragma unroll
                for (int q = 0; q < BAND_Q; ++q) {
                    const H4<F>& h = hv[(q + u) % BAND_Q];
                    C[q] = f_fma(rh.df, h.dg, f_fma(h.df, rh.dg, C[q]));
                }
            }
            F mg[BAND_Q];
#pragma unroll
            for (int q = 0; q < BAND_Q; ++q) mg[q] = f_fma(C[q], hv[(q + u) % BAND_Q].inv, rh.inv);
            band_hits<F>(mg, km, rhist);
        }
        // bit 31 - u of rhist: row i0 + t0 + u; of km[q]: column record
        // t0 + u + BAND_Q lane + q
        rowbits |= (unsigned long long)__builtin_bitreverse32(rhist) << (t0 & 32);
        rhist = 0u;
#pragma unroll
        for (int q = 0; q < BAND_Q; ++q) {
            const unsigned int v = __builtin_bitreverse32(km[q]);
            // every hit is a witness of both its subsequences
            for (unsigned int h = wit ? v : 0u; h; h &= h - 1u) {
                const int32_t t = t0 + __ffs((int)h) - 1;
                const int32_t i = (int32_t)i0 + t, j = (int32_t)j0 + t + BAND_Q * lane + q;
                A.wit[i] = ~j;
                A.wit[j] = ~i;
            }
            if (v) {
                const int cb = off + t0 + BAND_Q * lane + q;
                atomicOr(&kb[cb >> 5], v << (cb & 31));
                if (cb & 31) atomicOr(&kb[(cb >> 5) + 1], v >> (32 - (cb & 31)));
            }
            km[q] = 0u;
        }
        if ((t0 & 63) == 32) {
            if (lane == 0 && rowbits) atomicAnd(&A.alive[(i0 + t0 - 32) >> 6], ~rowbits);
            rowbits = 0ull;
        }
    }
    __syncthreads();
    // the killed columns, one bitmap word per lane (kb bit off + e: column j0 + e)
    if (lane < BAND_W32 / 2) {
        const unsigned long long bits =
            (unsigned long long)kb[2 * lane] | ((unsigned long long)kb[2 * lane + 1] << 32);
        if (bits) atomicAnd(&A.alive[(j0 >> 6) + lane], ~bits);
    }
    if (lane == 0)
        atomicAdd(&s.evc[EV_BAND * EV_SLOTS + (blockIdx.x & (EV_SLOTS - 1))],
                  (unsigned long long)BAND_S * BAND_D);
}

// First selection pass: every row tile's nearest near_cols columns, split
// into chunks of `chunk` columns that run concurrently; each stops as soon
// as the whole tile is dead.
template <typename F, int Q, int WIT>
__global__ __launch_bounds__(64) void k_select_near(SeriesDev* S, int B,
                                                    const int64_t* __restrict__ pfx, int near_cols,
                                                    int chunk)
{
    extern __shared__ double lds[];
    const int b = series_of(pfx, B, blockIdx.x);
    const SeriesDev& s = S[b];
    Ctrl* c = s.ctrl;
    if (!c->active || !c->prune || lean_round(c)) return;
    constexpr int R = 64 * Q;
    const int64_t lb = blockIdx.x - pfx[b];
    const SweepArgs<F> A = args_of<F>(s, c);
    // The series' blocks enumerate (tile, chunk) pairs: first every chunk of
    // the hot tiles (those that held survivors after the last round), then
    // the other tiles; both parts chunk-major, so that every tile's nearest
    // chunk is dispatched before its later ones, which then find the rows
    // their neighbours already pruned.
    const int64_t ntiles = (s.Nmax + R - 1) / R;
    const int64_t nsub = (pfx[b + 1] - pfx[b]) / ntiles;
    const unsigned int nhot = c->hot_r == R ? c->nhot : 0u;
    int64_t tile, cc;
    if (nhot == 0u) {
        tile = lb % ntiles;
        cc = lb / ntiles;
    } else {
        const int lane = threadIdx.x;
        const int hv = lane < (int)nhot ? s.hot[lane] : 0x7fffffff;
        const int64_t nh = (int64_t)nhot * nsub;
        if (lb < nh) {
            // rotated by the chunk so that one tile's chunks do not all fall
            // on the same XCD when nhot is a multiple of the XCD count
            cc = lb / nhot;
            tile = __builtin_amdgcn_readlane(hv, (int)((lb + cc) % nhot));
        } else {
            // the r-th tile that is not hot is r + #{i : hot[i] - i <= r}
            const int64_t x = lb - nh;
            const int64_t rest = ntiles - nhot;
            if (rest <= 0) return;
            const int64_t r = x % rest;
            cc = x / rest;
            tile = r + __popcll(__ballot(lane < (int)nhot && (int64_t)(hv - lane) <= r));
        }
    }
    const int64_t i0 = tile * R;
    if (i0 >= A.N) return;
    const int64_t j00 = i0 + A.m;
    const int64_t jbeg = j00 + cc * chunk;
    if (c->dense == DENSE_LEFT) return;
    const int64_t width = c->dense == DENSE_SWEEP ? dense_near(c) : near_cols;
    if (jbeg >= A.N || jbeg >= j00 + width) return;
    const int64_t jend = std::min<int64_t>(std::min<int64_t>(A.N, jbeg + chunk), j00 + width);
    const F thr = sel_threshold<F>(c);
    unsigned long long ev = 0;
    sel_item<F, Q, WIT>(A, i0, jbeg, jend, thr, lds, ev, &A.twork[tile]);
    if (threadIdx.x == 0 && ev) {
        atomicAdd(&s.evc[EV_NEAR * EV_SLOTS + (blockIdx.x & (EV_SLOTS - 1))], ev);
    }
}

// Remaining selection work: items (live tile, chunk) drawn nearest-first
// from each series' counter; a workgroup drains the series in rotated order.
// The FP32 two-row tile fits 128 registers, so four waves share a SIMD
// (three otherwise): the pass is bound by how many items are resident.
template <typename F, int Q, int WIT>
__global__ __launch_bounds__(64, (sizeof(F) == 4 && Q <= 2) ? 4 : 1) void k_select_far(
    SeriesDev* S, int B, int near_cols, int chunk, int near_rows)
{
    extern __shared__ double lds[];
    constexpr int R = 64 * Q;
    // Items are dealt out statically: the items of series b get the global
    // numbers cum_b + it (cum_b = items of the series before it) and
    // workgroup g takes the global numbers g, g + G, ...  (a shared queue
    // counter would cost one serialised device-scope atomic per item).
    unsigned long long cum = 0;
    for (int b = 0; b < B; ++b) {
        const SeriesDev& s = S[b];
        Ctrl* c = s.ctrl;
        if (!c->active || !c->prune || lean_round(c) || dense_round(c)) continue;
        const unsigned int nlive = c->nlive_sel;
        const unsigned long long total = (unsigned long long)nlive * c->maxc_sel;
        if (total == 0) continue;
        const unsigned long long first = first_item(cum);
        cum += total;
        const SweepArgs<F> A = args_of<F>(s, c);
        const F thr = sel_threshold<F>(c);
        const int32_t* __restrict__ tiles = s.tsel;
        unsigned long long ev = 0;
        for (unsigned long long it = first; it < total; it += gridDim.x) {
            const unsigned long long cc = it / nlive;
            const unsigned int p = (unsigned int)(it % nlive);
            const int64_t i0 = (int64_t)tiles[p] * R;
            // continue where the first pass (tiles of near_rows rows) ended,
            // so that every row's right side is covered completely
            const int64_t jbeg = (i0 / near_rows) * near_rows + A.m + near_cols + (int64_t)cc * chunk;
            if (jbeg >= A.N) continue;
            const int64_t jend = std::min<int64_t>(A.N, jbeg + chunk);
            sel_item<F, Q, WIT>(A, i0, jbeg, jend, thr, lds, ev, nullptr);
        }
        if (threadIdx.x == 0 && ev) {
            atomicAdd(&s.evc[EV_FAR * EV_SLOTS + (blockIdx.x & (EV_SLOTS - 1))], ev);
        }
    }
}

// Live-tile lists.  mode 0: selection tiles (R rows), chunks to the right
// beyond the first pass; mode 1: refinement tiles, chunks on both sides.
// One thread per tile; the block's live tiles are compacted with wave
// ballots and a prefix over the block's waves, so each block makes one
// atomic per counter (device-scope atomics on one address serialise).
constexpr int TILES_BLOCK = 256;
__global__ __launch_bounds__(TILES_BLOCK) void k_tiles(SeriesDev* S, int B,
                                                       const int64_t* __restrict__ pfx, int R,
                                                       int mode, int near_cols, int chunk,
                                                       int near_rows)
{
    constexpr int NW = TILES_BLOCK / 64;
    __shared__ unsigned int wn[NW], wmax[NW];
    __shared__ unsigned long long wrows[NW];
    __shared__ unsigned int base_s;
    const int b = series_of(pfx, B, blockIdx.x);
    const SeriesDev& s = S[b];
    Ctrl* c = s.ctrl;
    if (!c->active || lean_round(c) || dense_round(c)) return;
    if (mode == 0 && !c->prune) return;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t t = (blockIdx.x - pfx[b]) * (int64_t)TILES_BLOCK + threadIdx.x;
    const int32_t m = c->m;
    const int64_t N = s.n - m + 1;
    const int64_t ntiles = (N + R - 1) / R;
    const int words = R / 64;
    unsigned int cnt = 0;
    int64_t nch = 0;
    bool both = true;
    if (t < ntiles) {
        unsigned long long any = 0ull;
        for (int q = 0; q < words; ++q) {
            const unsigned long long v = s.alive[t * words + q];
            any |= v;
            cnt += (unsigned int)__popcll(v);
        }
        const int64_t i0 = t * R;
        if (any == 0ull) {
            nch = 0;
        } else if (mode == 0) {
            // the first pass covered near_cols columns from its own tile's start
            const int64_t j0 = (i0 / near_rows) * near_rows + m + near_cols;
            nch = j0 >= N ? 0 : (N - j0 + chunk - 1) / chunk;
        } else {
            const int64_t lend = std::min<int64_t>(N, i0 + R - m);
            const int64_t nl = lend > 0 ? (lend + chunk - 1) / chunk : 0;
            const int64_t jr = i0 + m;
            const int64_t nr = jr < N ? (N - jr + chunk - 1) / chunk : 0;
            // The selection sweep covered the right side of every live row in
            // FP32; a row's exact maximum there is within the guard g of the
            // recorded one, so the right side needs the exact sweep only when
            // some live row's recorded maximum is above thr64 - g (or when
            // there was no selection sweep, or the round is an exact repeat,
            // or a bare range search or a heatmap, which report every
            // survivor's exact maximum).
            both = !c->prune || c->exact_ref || c->mode == 3 || s.heat != nullptr;
            if (!both) {
                unsigned long long u = 0ull;
                for (int q = 0; q < words; ++q) u |= s.alive[t * words + q] & s.unc[t * words + q];
                both = u != 0ull;
            }
            nch = nl + (both ? nr : 0);
        }
    }
    const bool entry = nch > 0;
    // live rows and entries of the wave, then of the block
    unsigned long long rows = cnt;
    unsigned int mx = (unsigned int)nch;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        rows += __shfl_xor(rows, o);
        mx = max(mx, (unsigned int)__shfl_xor((int)mx, o));
    }
    const unsigned long long bal = __ballot(entry);
    if (lane == 0) {
        wn[w] = (unsigned int)__popcll(bal);
        wrows[w] = rows;
        wmax[w] = mx;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned int tot = 0, mxb = 0;
        unsigned long long rb = 0ull;
        for (int q = 0; q < NW; ++q) {
            tot += wn[q];
            rb += wrows[q];
            mxb = max(mxb, wmax[q]);
        }
        if (rb) {
            atomicAdd(mode == 0 ? &c->rows_near : &c->rows_far, rb);
            if (mode == 1) atomicAdd(&c->live_ref, (unsigned int)rb);
        }
        base_s = tot ? atomicAdd(mode == 0 ? &c->nlive_sel : &c->nlive_ref, tot) : 0u;
        if (tot) atomicMax(mode == 0 ? &c->maxc_sel : &c->maxc_ref, mxb);
    }
    __syncthreads();
    if (entry) {
        unsigned int before = 0;
        for (int q = 0; q < w; ++q) before += wn[q];
        const unsigned int slot =
            base_s + before + (unsigned int)__popcll(bal & ((1ull << lane) - 1ull));
        // refinement entries carry bit 31 when only the left side is swept
        (mode == 0 ? s.tsel : s.tref)[slot] =
            both ? (int32_t)t : (int32_t)((uint32_t)t | 0x80000000u);
    }
}

// Refinement: exact FP64 row maximum of rho over both sides for every tile
// holding survivors; items drawn nearest-first, alternating right and left.
// WIT: the rows it prunes keep their witnesses (a search); a bare range
// search has no next length.
template <int Q, bool WIT>
__global__ __launch_bounds__(64, (Q <= 4 ? 3 : 1)) void k_refine(SeriesDev* S, int B,
                                                                         int chunk)
{
    extern __shared__ double lds[];
    constexpr int R = 64 * Q;
    unsigned long long cum = 0;  // items dealt out as in k_select_far
    for (int b = 0; b < B; ++b) {
        const SeriesDev& s = S[b];
        Ctrl* c = s.ctrl;
        if (!c->active || lean_round(c) || dense_round(c) || direct_round(c)) continue;
        const unsigned int nlive = c->nlive_ref;
        const unsigned long long total = (unsigned long long)nlive * c->maxc_ref;
        if (total == 0) continue;
        const unsigned long long first = first_item(cum);
        cum += total;
        const SweepArgs<double> A = args_of<double>(s, c);
        const double thr = c->thr64;
        const int prune = c->prune;
        const int32_t* __restrict__ tiles = s.tref;
        unsigned long long ev = 0;
        for (unsigned long long it = first; it < total; it += gridDim.x) {
            const unsigned long long cc = it / nlive;
            const unsigned int p = (unsigned int)(it % nlive);
            const int32_t e = tiles[p];
            const int64_t i0 = (int64_t)(e & 0x7fffffff) * R;
            const int64_t lend = std::min<int64_t>(A.N, i0 + R - A.m);
            const int64_t nl = lend > 0 ? (lend + chunk - 1) / chunk : 0;
            const int64_t jr = i0 + A.m;
            const int64_t nr = (e >= 0 && jr < A.N) ? (A.N - jr + chunk - 1) / chunk : 0;
            if ((int64_t)cc >= nl + nr) continue;
            const int64_t mn = std::min(nl, nr);
            bool left;
            int64_t q;
            if ((int64_t)cc < 2 * mn) {
                left = (cc & 1u) != 0u;
                q = cc >> 1;
            } else {
                q = mn + ((int64_t)cc - 2 * mn);
                left = nl > nr;
            }
            int64_t jbeg, jend;
            if (left) {
                jend = lend - q * chunk;
                jbeg = std::max<int64_t>(0, jend - chunk);
            } else {
                jbeg = jr + q * chunk;
                jend = std::min<int64_t>(A.N, jbeg + chunk);
            }
            if (jbeg >= jend) continue;
            ref_item<Q, batch_cols<double>(), WIT>(A, i0, jbeg, jend, left, thr, prune, lds, ev);
        }
        if (threadIdx.x == 0 && ev)
            atomicAdd(&s.evc[EV_REF * EV_SLOTS + (blockIdx.x & (EV_SLOTS - 1))], ev);
    }
}

struct Key {
    unsigned long long u;  // ordered bits of rho (ascending rho = descending nnDist)
    long long i;
};
constexpr long long KEY_NONE = 0x7fffffffffffffffll;
__device__ __forceinline__ bool key_less(const Key& x, const Key& y)
{
    return x.u < y.u || (x.u == y.u && x.i < y.i);
}
__device__ __forceinline__ Key wave_min_key(Key k)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        Key y;
        y.u = __shfl_xor(k.u, o);
        y.i = __shfl_xor(k.i, o);
        if (key_less(y, k)) k = y;
    }
    return k;
}

// The round's range discords and the exact pass's candidates (one block per
// series).  After a refinement sweep: count the subsequences still alive
// (the range discords of this range search), pick the k + KP_EXTRA with the
// smallest refined correlation (largest distance; ties: smaller index).  Each
// wave first extracts the best of the bitmap words it owns by rounds of
// wave-wide minimum (no block barriers), then wave 0 extracts the best of
// the pooled per-wave lists.  In a direct round (no refinement sweep) every
// live subsequence becomes a candidate.
// fn(q, word) for every nonzero word q of the bitmap taken by this thread
// (q = threadIdx.x + TOPK_BLOCK j): sixteen words are loaded before any is
// scanned, so one memory latency covers them.
template <typename Fn>
__device__ __forceinline__ void scan_words(const unsigned long long* __restrict__ alive, int64_t nw,
                                           Fn&& fn)
{
    constexpr int U = 16;
    for (int64_t q0 = threadIdx.x; q0 < nw; q0 += (int64_t)U * TOPK_BLOCK) {
        unsigned long long wv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t q = q0 + (int64_t)u * TOPK_BLOCK;
            wv[u] = q < nw ? alive[q] : 0ull;
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (wv[u]) fn(q0 + (int64_t)u * TOPK_BLOCK, wv[u]);
    }
}

__global__ __launch_bounds__(TOPK_BLOCK) void k_select_top(SeriesDev* S)
{
    constexpr int NW = TOPK_BLOCK / 64;
    __shared__ unsigned long long pu[NW][KP_MAX];
    __shared__ long long pi[NW][KP_MAX];
    __shared__ unsigned int cnt_s[NW];
    __shared__ long long cand_s[KP_MAX];
    __shared__ unsigned int nc_s;
    __shared__ unsigned long long kth_s;
    __shared__ int kp_s;
    const SeriesDev& s = S[blockIdx.x];
    Ctrl* c = s.ctrl;
    if (!c->active || lean_round(c) || dense_round(c)) return;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int64_t N = s.n - c->m + 1;
    const int64_t nw = (N + 63) / 64;
    const unsigned long long* __restrict__ alive = s.alive;
    const unsigned long long* __restrict__ rho = s.rho;
    const unsigned long long* __restrict__ rhs = s.rhs;
    const int k = s.k;
    // ranking key of a live row: its refined maximum, or, where refinement
    // swept only the left side, the larger of that and the selection sweep's
    // (within the guard of exact); an exact repeat ranks by exact values
    const bool exact = c->exact_ref || !c->prune || c->mode == 3 || s.heat != nullptr;
    auto key_of = [&](long long i) -> unsigned long long {
        return exact ? rho[i] : (rho[i] > rhs[i] ? rho[i] : rhs[i]);
    };
    int kp;
    if (direct_round(c)) {
        if (tid == 0) nc_s = 0;
        __syncthreads();
        scan_words(alive, nw, [&](int64_t q, unsigned long long bits) {
            while (bits) {
                const int t = __ffsll((long long)bits) - 1;
                bits &= bits - 1ull;
                const unsigned int slot = atomicAdd(&nc_s, 1u);
                if (slot < (unsigned int)CAND_MAX) s.cand[slot] = q * 64 + t;
            }
        });
        __syncthreads();
        kp = (int)min(nc_s, (unsigned int)CAND_MAX);
        if (tid == 0) {
            c->nsurv = (unsigned int)kp;  // refined by k_round_end
            c->ncand = kp < k ? 0u : (unsigned int)kp;
        }
    } else {
        unsigned int cnt = 0;
        scan_words(alive, nw, [&](int64_t, unsigned long long bits) { cnt += (unsigned int)__popcll(bits); });
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) cnt += __shfl_xor(cnt, o);
        if (lane == 0) cnt_s[w] = cnt;
        __syncthreads();
        unsigned int ns = 0;
        for (int q = 0; q < NW; ++q) ns += cnt_s[q];
        // (a bare range search wants the count only)
        if (ns < (unsigned int)k || (c->mode == 3 && s.idx == nullptr)) {
            if (tid == 0) {
                c->nsurv = ns;
                c->ncand = 0;
            }
            return;
        }
        kp = (int)min(ns, (unsigned int)(k + KP_EXTRA));
        // per-wave best kp
        {
            Key last = {0ull, -1};
            for (int r = 0; r < kp; ++r) {
                Key best = {~0ull, KEY_NONE};
                scan_words(alive, nw, [&](int64_t q, unsigned long long bits) {
                    while (bits) {
                        const int t = __ffsll((long long)bits) - 1;
                        bits &= bits - 1ull;
                        const long long i = q * 64 + t;
                        const Key x = {key_of(i), i};
                        if ((r == 0 || key_less(last, x)) && key_less(x, best)) best = x;
                    }
                });
                best = wave_min_key(best);
                if (lane == 0) {
                    pu[w][r] = best.u;
                    pi[w][r] = best.i;
                }
                last = best;
                if (__builtin_amdgcn_readfirstlane((int)(best.i == KEY_NONE))) {
                    for (int q = r + 1 + lane; q < kp; q += 64) {
                        pu[w][q] = ~0ull;
                        pi[w][q] = KEY_NONE;
                    }
                    break;
                }
            }
        }
        __syncthreads();
        if (w == 0) {
            Key last = {0ull, -1};
            for (int r = 0; r < kp; ++r) {
                Key best = {~0ull, KEY_NONE};
                for (int e = lane; e < NW * kp; e += 64) {
                    const int ww = e / kp, rr = e - ww * kp;
                    const Key x = {pu[ww][rr], pi[ww][rr]};
                    if (x.i == KEY_NONE) continue;
                    if (r > 0 && !key_less(last, x)) continue;
                    if (key_less(x, best)) best = x;
                }
                best = wave_min_key(best);
                if (lane == 0) {
                    cand_s[r] = best.i;
                    s.cand[r] = best.i;
                    if (r == k - 1) kth_s = best.u;
                }
                last = best;
            }
        }
        if (tid == 0) kp_s = kp;
        __syncthreads();
        if (!exact) {
            // Every row whose key is within 2g of the k-th smallest may hold
            // one of the k smallest exact values (keys are within g of
            // exact): all of them are evaluated, up to KP_MAX; beyond that
            // the round is repeated with exact refinement.
            const double g = c->thr_sel - c->thr64;
            const unsigned long long ub = ord_of(dbl_of(kth_s) + 2.0 * g);
            if (tid == 0) nc_s = 0;
            __syncthreads();
            unsigned int nb = 0;
            scan_words(alive, nw, [&](int64_t q, unsigned long long bits) {
                while (bits) {
                    const int t = __ffsll((long long)bits) - 1;
                    bits &= bits - 1ull;
                    nb += key_of(q * 64 + t) <= ub ? 1u : 0u;
                }
            });
            if (nb) atomicAdd(&nc_s, nb);
            __syncthreads();
            const unsigned int nband = nc_s;
            __syncthreads();
            if (nband > (unsigned int)KP_MAX) {
                if (tid == 0) {
                    c->band_over = 1;
                    c->nsurv = ns;
                    c->ncand = 0;
                }
                return;
            }
            if (nband > (unsigned int)kp) {
                if (tid == 0) nc_s = 0;
                __syncthreads();
                scan_words(alive, nw, [&](int64_t q, unsigned long long bits) {
                    while (bits) {
                        const int t = __ffsll((long long)bits) - 1;
                        bits &= bits - 1ull;
                        const long long i = q * 64 + t;
                        if (key_of(i) <= ub) {
                            const unsigned int slot = atomicAdd(&nc_s, 1u);
                            cand_s[slot] = i;
                            s.cand[slot] = i;
                        }
                    }
                });
                if (tid == 0) kp_s = (int)nband;
                __syncthreads();
            }
        }
        kp = kp_s;
        if (tid == 0) {
            c->nsurv = ns;
            c->ncand = (unsigned int)kp;
        }
    }
}

// ---------------------------------------------------------------------------
// the exact pass: nearest neighbours of the candidate rows over every column
// ---------------------------------------------------------------------------
// Candidates are taken in groups of PM_G = 16.  The reported values come from
// direct centred FP64 dot products on the FP64 matrix cores (k_exact); a
// screening pass (k_screen) first bounds every pair's correlation on the FP16
// matrix cores and leaves to k_exact only the blocks of EX_COLS columns that
// can hold a candidate's largest correlation.
constexpr int PM_G = 16;       // candidates per group
constexpr int EX_COLS = EXACT_COLS;  // columns per exact block
constexpr int EX_WAVES = 4;    // waves per workgroup, EX_COLS / EX_WAVES columns each
constexpr int EX_CT = EX_COLS / EX_WAVES / 16;  // 16-column tiles per wave
constexpr int EX_STEPS = 8;    // matrix steps (of 4 offsets) read ahead
constexpr int PM_KC = 256;     // window offsets per LDS chunk
constexpr int PM_XS = PM_KC + 1;  // LDS row stride of a candidate window (odd: no bank conflicts)
constexpr int SC_WAVES = 4;
constexpr int SC_COLS = SCREEN_COLS;  // columns per screening chunk, EX_COLS per wave
static_assert(SC_COLS == SC_WAVES * EX_COLS, "a wave screens one exact block");
// (below any product: those of a stretch with a spike are off by its e_j)
constexpr float SC_NONE = -1e30f;
constexpr int SC_AS = PM_KC + 8;  // LDS row stride of a screened window, in halves
constexpr int SC_SLOTS = (SC_COLS + PM_KC) / 8;  // 16-byte slots of one shifted copy
// LDS row stride of a whole window, in halves
__host__ __device__ constexpr int dense_stride(int m) { return ((m + 31) & ~31) + 8; }

// Candidates of a series in this round (0: nothing to evaluate).
__device__ __forceinline__ int cand_count(const SeriesDev& s, const Ctrl* c, int full)
{
    if (!c->active) return 0;
    if (lean_round(c)) return c->nlive >= (uint32_t)s.k ? (int)c->nlive : 0;
    return full || c->handled ? (int)c->ncand : 0;
}
__device__ __forceinline__ int64_t exact_blocks(int64_t N) { return (N + EX_COLS - 1) / EX_COLS; }
__device__ __forceinline__ int64_t screen_chunks(int64_t N) { return (N + SC_COLS - 1) / SC_COLS; }

// Candidate groups of a screening item.  Four share a chunk's operands where
// there are items enough, in the series or in the batch (staging costs as much
// as the products of three groups), else one, whose items are shorter and more
// (12,000 points: 11.5 us per round, with four always 26; batches of two to
// sixteen series of 12,000 to 30,000 points, m = 120: 3 to 10 % less time than
// with four in every batch); windows past PM_KC are staged in parts, a
// group at a time.
constexpr int SC_GS = SCREEN_GROUPS;
__device__ __forceinline__ int screen_groups(int large, int32_t m, int64_t ng, int64_t nch)
{
    return m <= PM_KC && (large || ng * nch > 2 * SCREEN_GRID) ? SC_GS : 1;
}

// Work items of the two kernels: (candidate groups, chunk) or (group, block)
// of every series, group-major, numbered across the batch; each workgroup
// takes one contiguous range, so that it stays with a group's windows.
// ipfx[b]: first item of series b (one series needs no table).
__device__ __forceinline__ int64_t items_of(const SeriesDev& s, int large, int full, bool screen)
{
    const Ctrl* c = s.ctrl;
    const int64_t ng = (cand_count(s, c, full) + PM_G - 1) / PM_G;
    const int64_t N = s.n - c->m + 1;
    const int64_t nch = screen_chunks(N);
    const int gs = screen_groups(large, c->m, ng, nch);
    return screen ? (ng + gs - 1) / gs * nch : ng * exact_blocks(N);
}
constexpr int ITEMS_BLOCK = 1024;
__global__ __launch_bounds__(ITEMS_BLOCK) void k_items(SeriesDev* S, int B, int large, int full, int64_t* ipfx_s,
                                                       int64_t* ipfx_e)
{
    __shared__ long long ws[2][ITEMS_BLOCK / 64];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    long long base[2] = {0, 0};
    for (int b0 = 0; b0 < B; b0 += ITEMS_BLOCK) {
        const int b = b0 + tid;
        long long v[2] = {0, 0}, x[2];
        if (b < B) {
            v[0] = items_of(S[b], large, full, true);
            v[1] = items_of(S[b], large, full, false);
        }
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            x[q] = v[q];
            for (int o = 1; o < 64; o <<= 1) {
                const long long y = __shfl_up(x[q], o);
                if (lane >= o) x[q] += y;
            }
            if (lane == 63) ws[q][w] = x[q];
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            long long before = 0, tot = 0;
            for (int e = 0; e < ITEMS_BLOCK / 64; ++e) {
                before += e < w ? ws[q][e] : 0;
                tot += ws[q][e];
            }
            if (b < B) (q ? ipfx_e : ipfx_s)[b] = base[q] + before + x[q] - v[q];
            base[q] += tot;
        }
        __syncthreads();
    }
    if (tid == 0) {
        ipfx_s[B] = base[0];
        ipfx_e[B] = base[1];
    }
}

// The share of a workgroup: items [lo, hi) of total, per items each.
struct Share {
    int64_t lo, hi, per;
};
__device__ __forceinline__ Share share_of(int64_t total)
{
    Share r;
    r.per = (total + gridDim.x - 1) / gridDim.x;
    r.lo = std::min<int64_t>(total, r.per * blockIdx.x);
    r.hi = std::min<int64_t>(total, r.lo + r.per);
    return r;
}

// Partials of a series: a workgroup that evaluated something for group g
// leaves one, in one of the slots from part_base(g) on (as many as there are
// workgroups whose share meets the group).
__device__ __forceinline__ int64_t part_base(int64_t per, int64_t first, int64_t nblk, int g)
{
    return (first + g * nblk) / per - first / per + g;
}

typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef float acc4f_t __attribute__((ext_vector_type(4)));

// Screening.  Every candidate window x (centred, scaled to unit norm) and
// every stretch of the series w (offset and scaled by a power of two per
// chunk) is rounded to FP16 and x.w accumulated in FP32 by
// V_MFMA_F32_16X16X32_F16, 32 times the rate of the FP64 instruction.  The
// values only bound the correlation; every value that is reported or decides
// anything comes from k_exact.  The Hankel operand B[k][c] = w[c' + k] is read
// in aligned groups of eight values: tile u of a wave holds the columns
// 8 c + u (c < 16) and reads the copy of w shifted by u, so eight copies of
// the stretch stand in LDS.
//
// Bound: |rho~ - rho| <= e_j = e0 sqrt(1 + m ((mu_j - off) inv_j)^2) + floor,
// by Cauchy-Schwarz on |x| = 1 and |w_j - off|: e0 holds the two roundings
// (2^-11 each) and the FP32 accumulation (one rounding of 2^-23 per product),
// floor the smallest normal FP16 value (should the matrix cores flush
// subnormals), all rounded up.  (Measured on the device: the instruction's sums
// of 32 to 512 products of random, cancelling, offset, widely spread and
// subnormal values are off by at most 4.7 x 2^-23 of the products' absolute
// sum, where the bound allows the number of products + 32; subnormal values are
// kept.)  A candidate's lower bound is the largest
// rho~ - e_j over all columns; only blocks whose largest rho~ + e_j reaches
// it can hold its maximum, so k_exact finds the same value and the same
// smallest argmax as over all columns.  (A split into two FP16 values per
// operand, 2^-22 instead of 2^-11, takes three times the matrix work and
// leaves few blocks fewer.)  Eight columns of a lane share their largest e_j,
// so that a product costs two vector operations.
//
// Bound by latency where a workgroup has one chunk (two loads in a chain, the
// operands, the products), else by the LDS reads and the 64 x 512 products'
// maxima.  The next chunk's values are fetched during the products.  (One group per item and a bound per product: 64 series 216 us
// per round, 1,000,000 points 50 us; so 110 and 33.)

// One group after the other of G (for G = 4 half the columns at a time, so
// that the accumulators stay at 64 registers): the largest product of every
// row over the lane's eight columns.
template <int G, int NU>
__device__ __forceinline__ void screen_products(const _Float16* ap, int stride, int steps,
                                                const half8_t (*wcopy)[SC_SLOTS], int slot,
                                                const float (&gj)[8], const int32_t* rows, int ka,
                                                int32_t jl, int64_t N, int32_t m,
                                                unsigned int edge, float (&mx)[4 * SC_GS])
{
#pragma unroll
    for (int q = 0; q < 4 * G; ++q) mx[q] = SC_NONE;
#pragma unroll
    for (int hf = 0; hf < 8 / NU; ++hf) {
        acc4f_t acc[G][NU];
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int u = 0; u < NU; ++u) acc[g][u] = (acc4f_t){0.f, 0.f, 0.f, 0.f};
        for (int st = 0; st < steps; ++st) {
            half8_t av[G];
#pragma unroll
            for (int g = 0; g < G; ++g) av[g] = *(const half8_t*)(ap + 16 * g * stride + 32 * st);
#pragma unroll
            for (int u = 0; u < NU; ++u) {
                const half8_t bv = wcopy[NU * hf + u][slot + 4 * st];
#pragma unroll
                for (int g = 0; g < G; ++g)
                    acc[g][u] = __builtin_amdgcn_mfma_f32_16x16x32_f16(av[g], bv, acc[g][u], 0, 0, 0);
            }
        }
#pragma unroll
        for (int g = 0; g < G; ++g) {
            if (!((edge >> g) & 1u)) {
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int u = 0; u < NU; ++u)
                        mx[4 * g + r] = fmaxf(mx[4 * g + r], acc[g][u][r] * gj[NU * hf + u]);
            } else {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int32_t i = rows[16 * g + 4 * ka + r];
#pragma unroll
                    for (int u = 0; u < NU; ++u) {
                        const int32_t j = jl + NU * hf + u;
                        const bool ok = (int64_t)j < N && (j <= i - m || j >= i + m);
                        mx[4 * g + r] = fmaxf(mx[4 * g + r], ok ? acc[g][u][r] * gj[NU * hf + u] : SC_NONE);
                    }
                }
            }
        }
    }
}

// A chunk's stretch in FP16, converted once per series (k_half): the values
// less the chunk's offset, times its power of two, and what the wave's two
// columns per lane need.
struct ChunkRegs {
    uint2 h[3];
    double off, usw;
    double cm[2], ci[2];
};
__device__ __forceinline__ void fetch_chunk(const SeriesDev& s, const double* __restrict__ mu,
                                            const double* __restrict__ inv, int64_t ch, ChunkRegs& R)
{
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const uint2* __restrict__ src = (const uint2*)(s.half + ch * HALF_STRIDE) + min(tid, 2 * SC_SLOTS - 1);
#pragma unroll
    for (int q = 0; q < 3; ++q) R.h[q] = src[q];
    R.off = s.chunk_scale[2 * ch];
    R.usw = s.chunk_scale[2 * ch + 1];
    const int64_t j = ch * SC_COLS + w * EX_COLS + lane;  // (inside the padded buffers)
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        R.cm[q] = mu[j + 64 * q];
        R.ci[q] = inv[j + 64 * q];
    }
}
// Thread tid has values 4 tid .. 4 tid + 11: slot t = tid / 2 of four copies
// (slot t of copy u: w[8 t + u .. 8 t + u + 7]).
__device__ __forceinline__ void stage_chunk(const ChunkRegs& R, half8_t (*wcopy)[SC_SLOTS])
{
    const int tid = threadIdx.x;
    if (tid >= 2 * SC_SLOTS) return;
    const int t = tid >> 1, u0 = (tid & 1) * 4;
    const uint32_t d[6] = {R.h[0].x, R.h[0].y, R.h[1].x, R.h[1].y, R.h[2].x, R.h[2].y};
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        uint32_t p[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int b = e + (u >> 1);
            p[e] = (u & 1) ? __builtin_amdgcn_alignbit(d[b + 1], d[b], 16) : d[b];
        }
        *(uint4*)&wcopy[u0 + u][t] = make_uint4(p[0], p[1], p[2], p[3]);
    }
}
// Product to correlation, and its error bound, of column q of the lane's two.
__device__ __forceinline__ float2 chunk_column(const ChunkRegs& R, int q, int32_t m, float e0, float fl)
{
    const float iv = (float)(R.ci[q] * R.usw);
    const float dn = (float)((R.cm[q] - R.off) * R.ci[q]);
    return make_float2(iv * 0x1p-10f, 1.02f * (e0 * sqrtf(1.0f + (float)m * dn * dn) + fl * iv) + 1e-6f);
}

// The chunks of every series (blocks past a series' last one exit), so that a
// round copies its chunks instead of scaling and converting them again
// (k_dense of 51,000 rows, m = 96, 200,000 points: 8.3 -> 6.5 ms).  Bound by
// the copy; 1,000,000 points 8.8 us.
__global__ __launch_bounds__(256) void k_half(SeriesDev* S)
{
    __shared__ double rlo[4], rhi[4];
    const SeriesDev& s = S[blockIdx.y];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int64_t nch = screen_chunks(s.n - s.minL + 1);
    for (int64_t ch = blockIdx.x; ch < nch; ch += gridDim.x) {
        constexpr int NV = (HALF_STRIDE + 255) / 256;
        const int64_t j0 = ch * SC_COLS;
        const int span = (int)std::min<int64_t>(SC_COLS + PM_KC, s.n - j0);
        double v[NV], lo = f_inf<double>(), hi = -f_inf<double>();
#pragma unroll
        for (int q = 0; q < NV; ++q) {
            const int t = tid + 256 * q;
            v[q] = t < span ? s.T[j0 + t] : 0.0;
            lo = t < span ? fmin(lo, v[q]) : lo;
            hi = t < span ? fmax(hi, v[q]) : hi;
        }
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) {
            lo = fmin(lo, __shfl_xor(lo, o));
            hi = fmax(hi, __shfl_xor(hi, o));
        }
        __syncthreads();
        if (lane == 0) {
            rlo[w] = lo;
            rhi[w] = hi;
        }
        __syncthreads();
        for (int q = 0; q < 4; ++q) {
            lo = fmin(lo, rlo[q]);
            hi = fmax(hi, rhi[q]);
        }
        const double off = 0.5 * (lo + hi);
        const double range = 0.5 * (hi - lo);
        // power of two with range * sw in (512, 1024] (1 for a constant stretch)
        int ex = 0;
        if (range > 0.0) (void)frexp(range, &ex);
        const double sw = range > 0.0 ? ldexp(1.0, min(10 - ex, 900)) : 1.0;
        _Float16* out = (_Float16*)s.half + ch * HALF_STRIDE;
#pragma unroll
        for (int q = 0; q < NV; ++q) {
            const int t = tid + 256 * q;
            if (t < HALF_STRIDE) out[t] = t < span ? (_Float16)(float)((v[q] - off) * sw) : (_Float16)0.0f;
        }
        if (tid == 0) {
            s.chunk_scale[2 * ch] = off;
            s.chunk_scale[2 * ch + 1] = 1.0 / sw;
        }
    }
}

hipError_t launch_half(const Batch& bt, int series, hipStream_t st)
{
    const int64_t nch = (bt.Nmax_all + SC_COLS - 1) / SC_COLS;
    hipLaunchKernelGGL(k_half, dim3((unsigned int)std::min<int64_t>(2048, nch), series), dim3(256), 0, st,
                       bt.s);
    return hipGetLastError();
}

__global__ __launch_bounds__(64 * SC_WAVES, 2) void k_screen(SeriesDev* S, int B, int large, int full,
                                                          const int64_t* __restrict__ ipfx)
{
    extern __shared__ __align__(16) _Float16 xa[];  // [PM_G SC_GS][dense_stride(m)]
    __shared__ half8_t wcopy[8][SC_SLOTS];
    __shared__ float gjs[SC_COLS], ejs[SC_COLS];
    __shared__ double cmu[PM_G * SC_GS], cinv[PM_G * SC_GS];
    __shared__ int32_t rows[PM_G * SC_GS];
    __shared__ float lbw[SC_WAVES][PM_G * SC_GS];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int ca = lane & 15, ka = lane >> 4;
    const int64_t total = B == 1 ? items_of(S[0], 0, full, true) : ipfx[B];
    const Share sh = share_of(total);
    for (int64_t it = sh.lo; it < sh.hi;) {
        const int b = B == 1 ? 0 : series_of(ipfx, B, it);
        const int64_t first = B == 1 ? 0 : ipfx[b];
        const SeriesDev& s = S[b];
        const Ctrl* c = s.ctrl;
        const int ncand = cand_count(s, c, full);
        const int32_t m = c->m;
        const int64_t N = s.n - m + 1;
        const int64_t nch = screen_chunks(N), nblk = exact_blocks(N);
        const int g = (int)((it - first) / nch);  // (of SC_GS groups, or the group)
        const int64_t c0 = (it - first) - g * nch;
        const int64_t c1 = std::min<int64_t>(nch, c0 + (sh.hi - it));
        it += c1 - c0;
        const double* __restrict__ T = s.T;
        const double* __restrict__ mu = cur_mu(s, c);
        const double* __restrict__ inv = s.inv64;
        if (m > PM_KC) continue;
        const int gs = screen_groups(large, m, (ncand + PM_G - 1) / PM_G, nch);
        const int ng = min(gs, (ncand + PM_G - 1) / PM_G - gs * g);
        const int nr = PM_G * ng;
        const int stride = dense_stride(m);
        ChunkRegs R;
        fetch_chunk(s, mu, inv, c0, R);
        __syncthreads();  // (the previous item is consumed)
        if (tid < PM_G * SC_GS) {
            const int64_t i = s.cand[min(PM_G * gs * g + tid, ncand - 1)];
            rows[tid] = (int32_t)i;
            cmu[tid] = mu[i];
            cinv[tid] = inv[i];
        }
        __syncthreads();
        // the candidates' windows, centred and scaled to norm 1024 (of three
        // groups the fourth's products are left over)
        const int nst = ng == 3 ? PM_G * SC_GS : nr;
#pragma unroll 1
        for (int r0 = w; r0 < nst; r0 += 4 * SC_WAVES) {
            constexpr int NQ = PM_KC / 64 + 1;
            double v[4][NQ];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int64_t i = rows[r0 + SC_WAVES * u];
#pragma unroll
                for (int q = 0; q < NQ; ++q) {
                    const int k = lane + 64 * q;
                    v[u][q] = k < m ? T[i + k] : 0.0;
                }
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int r = r0 + SC_WAVES * u;
                const double mi = cmu[r], sc = cinv[r] * 1024.0;
#pragma unroll
                for (int q = 0; q < NQ; ++q) {
                    const int k = lane + 64 * q;
                    if (k < stride)
                        xa[r * stride + k] =
                            k < m ? (_Float16)(float)((v[u][q] - mi) * sc) : (_Float16)0.0f;
                }
            }
        }
        unsigned int flat = 0u;  // bit 4 g + r: row 16 g + 4 ka + r is flat
        float lbr[4 * SC_GS];
#pragma unroll
        for (int q = 0; q < 4 * SC_GS; ++q) lbr[q] = -4.0f;
#pragma unroll
        for (int q = 0; q < 4 * SC_GS; ++q) {
            if ((q >> 2) >= ng) break;
            flat |= cinv[16 * (q >> 2) + 4 * ka + (q & 3)] == 0.0 ? 1u << q : 0u;
        }
        const float e0 = 1.05f * (2.0f * 0x1p-11f + 0x1p-22f + (float)(m + 32) * 0x1p-23f +
                                  sqrtf((float)m) * 0x1p-23f);
        const float fl = sqrtf((float)m) * 0x1p-13f;
        const int steps = (m + 31) >> 5;
        const _Float16* ap = xa + ca * stride + 8 * ka;
        for (int64_t ch = c0; ch < c1; ++ch) {
            const int64_t j0 = ch * SC_COLS, jb = j0 + w * EX_COLS;
            __syncthreads();  // (the previous chunk's operands are consumed)
            stage_chunk(R, wcopy);
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const float2 x = chunk_column(R, q, m, e0, fl);
                gjs[w * EX_COLS + lane + 64 * q] = x.x;
                ejs[w * EX_COLS + lane + 64 * q] = x.y;
            }
            __syncthreads();
            if (ch + 1 < c1) fetch_chunk(s, mu, inv, ch + 1, R);
            const int64_t blk = ch * SC_WAVES + w;
            if (blk >= nblk) continue;  // (the next barrier is the loop's first)
            float gj[8], em = 0.0f;
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                gj[u] = gjs[w * EX_COLS + 8 * ca + u];
                em = fmaxf(em, ejs[w * EX_COLS + 8 * ca + u]);
            }
            unsigned int edge = 0u;  // groups with a row at its exclusion zone
#pragma unroll
            for (int q = 0; q < 4 * SC_GS; ++q) {
                if ((q >> 2) >= ng) break;
                const int32_t i = rows[16 * (q >> 2) + 4 * ka + (q & 3)];
                if (jb + EX_COLS > N || (jb < (int64_t)i + m && jb + EX_COLS > (int64_t)i - m))
                    edge |= 1u << (q >> 2);
            }
#pragma unroll
            for (int o = 32; o >= 16; o >>= 1) edge |= (unsigned int)__shfl_xor((int)edge, o);
            edge = (unsigned int)__builtin_amdgcn_readfirstlane((int)edge);
            const int slot = w * (EX_COLS / 8) + ca + ka;
            const int32_t jl = (int32_t)jb + 8 * ca;
            float mx[4 * SC_GS];
            if (ng == 1)
                screen_products<1, 8>(ap, stride, steps, wcopy, slot, gj, rows, ka, jl, N, m, edge, mx);
            else if (ng == 2)
                screen_products<2, 8>(ap, stride, steps, wcopy, slot, gj, rows, ka, jl, N, m, edge, mx);
            else
                screen_products<4, 4>(ap, stride, steps, wcopy, slot, gj, rows, ka, jl, N, m, edge, mx);
#pragma unroll
            for (int gi = 0; gi < SC_GS; ++gi) {
                if (gi >= ng) break;
                float ub[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float v = mx[4 * gi + r];
                    lbr[4 * gi + r] = fmaxf(lbr[4 * gi + r], v - em);
                    ub[r] = v + em;
#pragma unroll
                    for (int o = 8; o >= 1; o >>= 1) ub[r] = fmaxf(ub[r], __shfl_xor(ub[r], o));
                    if ((flat >> (4 * gi + r)) & 1u) ub[r] = 4.0f;  // every block is evaluated
                }
                if (ca == 0)
                    *(float4*)(s.ub + ((int64_t)(gs * g + gi) * nblk + blk) * PM_G + 4 * ka) =
                        make_float4(ub[0], ub[1], ub[2], ub[3]);
            }
        }
        // the workgroup's lower bounds of these groups
#pragma unroll
        for (int q = 0; q < 4 * SC_GS; ++q) {
            if ((q >> 2) >= ng) break;
#pragma unroll
            for (int o = 8; o >= 1; o >>= 1) lbr[q] = fmaxf(lbr[q], __shfl_xor(lbr[q], o));
            if (ca == 0)
                lbw[w][16 * (q >> 2) + 4 * ka + (q & 3)] = (flat >> q) & 1u ? -4.0f : lbr[q];
        }
        __syncthreads();
        if (tid < nr) {
            float v = lbw[0][tid];
            for (int q = 1; q < SC_WAVES; ++q) v = fmaxf(v, lbw[q][tid]);
            const int64_t e = (int64_t)blockIdx.x - first / sh.per + g;
            s.lbp[e * gs * PM_G + tid] = v;
        }
    }
}

// Windows past PM_KC points: staged in parts, a group at a time.
__global__ __launch_bounds__(64 * SC_WAVES, 2) void k_screen_long(SeriesDev* S, int B, int large, int full,
                                                          const int64_t* __restrict__ ipfx)
{
    __shared__ __align__(16) _Float16 xa[PM_G * SC_AS];
    __shared__ half8_t wcopy[8][SC_SLOTS];
    __shared__ double cmu[PM_G], cinv[PM_G];
    __shared__ int64_t cidx[PM_G];
    __shared__ double rlo[SC_WAVES], rhi[SC_WAVES];
    __shared__ float lbw[SC_WAVES][PM_G];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int ca = lane & 15, ka = lane >> 4;
    const int64_t total = B == 1 ? items_of(S[0], 0, full, true) : ipfx[B];
    const Share sh = share_of(total);
    for (int64_t it = sh.lo; it < sh.hi;) {
        const int b = B == 1 ? 0 : series_of(ipfx, B, it);
        const int64_t first = B == 1 ? 0 : ipfx[b];
        const SeriesDev& s = S[b];
        const Ctrl* c = s.ctrl;
        const int ncand = cand_count(s, c, full);
        const int32_t m = c->m;
        const int64_t N = s.n - m + 1;
        const int64_t nch = screen_chunks(N), nblk = exact_blocks(N);
        const int g = (int)((it - first) / nch);  // (of SC_GS groups, or the group)
        const int64_t c0 = (it - first) - g * nch;
        const int64_t c1 = std::min<int64_t>(nch, c0 + (sh.hi - it));
        it += c1 - c0;
        const double* __restrict__ T = s.T;
        const double* __restrict__ mu = cur_mu(s, c);
        const double* __restrict__ inv = s.inv64;
        if (m <= PM_KC) continue;
        __syncthreads();
        if (tid < PM_G) {
            const int cid = PM_G * g + tid;
            const int64_t i = s.cand[min(cid, ncand - 1)];
            cidx[tid] = i;
            cmu[tid] = mu[i];
            cinv[tid] = inv[i];
        }
        __syncthreads();
        int64_t ci[4];
        bool flat[4];
        float lbr[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            ci[r] = cidx[4 * ka + r];
            flat[r] = cinv[4 * ka + r] == 0.0;
            lbr[r] = -4.0f;
        }
        const float e0 = 1.05f * (2.0f * 0x1p-11f + 0x1p-22f + (float)(m + 32) * 0x1p-23f +
                                  sqrtf((float)m) * 0x1p-23f);
        auto stage_windows = [&](int kb, int kn) {
            for (int gq = w; gq < PM_G; gq += SC_WAVES) {
                const int64_t i = cidx[gq];
                const double mi = cmu[gq], sc = cinv[gq] * 1024.0;
                double v[(SC_AS + 63) / 64];
#pragma unroll
                for (int q = 0; q < (SC_AS + 63) / 64; ++q) {
                    const int k = lane + 64 * q;
                    v[q] = k < kn ? T[i + kb + k] : mi;
                }
#pragma unroll
                for (int q = 0; q < (SC_AS + 63) / 64; ++q) {
                    const int k = lane + 64 * q;
                    if (k < SC_AS) xa[gq * SC_AS + k] = (_Float16)(float)((v[q] - mi) * sc);
                }
            }
        };
        for (int64_t ch = c0; ch < c1; ++ch) {
            const int64_t j0 = ch * SC_COLS;
            // offset and scale of the chunk's stretch
            double lo = f_inf<double>(), hi = -f_inf<double>();
            const int span = (int)std::min<int64_t>(SC_COLS + m, s.n - j0);
            for (int t0 = tid; t0 < span; t0 += 4 * 64 * SC_WAVES) {
                double v[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int t = t0 + q * 64 * SC_WAVES;
                    v[q] = T[j0 + (t < span ? t : t0)];
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    lo = fmin(lo, v[q]);
                    hi = fmax(hi, v[q]);
                }
            }
#pragma unroll
            for (int o = 32; o >= 1; o >>= 1) {
                lo = fmin(lo, __shfl_xor(lo, o));
                hi = fmax(hi, __shfl_xor(hi, o));
            }
            if (lane == 0) {
                rlo[w] = lo;
                rhi[w] = hi;
            }
            __syncthreads();  // (the previous chunk's operands are consumed)
            for (int q = 0; q < SC_WAVES; ++q) {
                lo = fmin(lo, rlo[q]);
                hi = fmax(hi, rhi[q]);
            }
            const double off = 0.5 * (lo + hi);
            const double range = 0.5 * (hi - lo);
            // power of two with range * sw in (512, 1024] (1 for a constant stretch)
            int ex = 0;
            if (range > 0.0) (void)frexp(range, &ex);
            const double sw = range > 0.0 ? ldexp(1.0, min(10 - ex, 900)) : 1.0;
            acc4f_t acc[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) acc[u] = (acc4f_t){0.f, 0.f, 0.f, 0.f};
            for (int kb = 0; kb < m; kb += PM_KC) {
                const int kn = min(PM_KC, m - kb);
                if (kb) __syncthreads();
                // slot t of copy u: w[8 t + u .. 8 t + u + 7]
                for (int e = tid; e < 2 * SC_SLOTS; e += 64 * SC_WAVES) {
                    const int t = e >> 1, u0 = (e & 1) * 4;
                    const double* __restrict__ src = T + j0 + kb + 8 * t + u0;
                    _Float16 h[11];
#pragma unroll
                    for (int q = 0; q < 11; ++q) {
                        const double v = (src[q] - off) * sw;
                        // values past the windows of this chunk may exceed the scale
                        h[q] = (_Float16)(float)fmin(2048.0, fmax(-2048.0, v));
                    }
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        half8_t ph;
#pragma unroll
                        for (int q = 0; q < 8; ++q) ph[q] = h[u + q];
                        wcopy[u0 + u][t] = ph;
                    }
                }
                stage_windows(kb, kn);
                __syncthreads();
                const int steps = (kn + 31) >> 5;
                const _Float16* ah = &xa[ca * SC_AS + 8 * ka];
                const int slot = w * (EX_COLS / 8) + ca + ka;
                for (int st = 0; st < steps; ++st) {
                    const half8_t vh = *(const half8_t*)(ah + 32 * st);
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const half8_t bh = wcopy[u][slot + 4 * st];
                        acc[u] = __builtin_amdgcn_mfma_f32_16x16x32_f16(vh, bh, acc[u], 0, 0, 0);
                    }
                }
            }
            // epilogue: lane holds candidate 4 ka + r, columns jb + 8 ca + u
            const int64_t jb = j0 + w * EX_COLS;
            bool edge = jb + EX_COLS > N;
#pragma unroll
            for (int r = 0; r < 4; ++r) edge = edge || (jb < ci[r] + m && jb + EX_COLS > ci[r] - m);
            const bool masked = __ballot(edge) != 0ull;
            const double usw = 1.0 / sw;
            const float fl = sqrtf((float)m) * 0x1p-13f;
            float ubm[4], lbm[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) ubm[r] = lbm[r] = -4.0f;
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int64_t j = jb + 8 * ca + u;
                const double ivd = inv[j];
                const float iv = (float)(ivd * usw);
                const float dn = (float)((mu[j] - off) * ivd);
                const float ej = 1.02f * (e0 * sqrtf(1.0f + (float)m * dn * dn) + fl * iv) + 1e-12f;
                const float gj = iv * 0x1p-10f;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float t = acc[u][r] * gj;
                    const bool ok = !masked || (j < N && (j <= ci[r] - m || j >= ci[r] + m));
                    ubm[r] = fmaxf(ubm[r], ok ? t + ej : -4.0f);
                    lbm[r] = fmaxf(lbm[r], ok ? t - ej : -4.0f);
                }
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                lbr[r] = fmaxf(lbr[r], lbm[r]);
#pragma unroll
                for (int o = 8; o >= 1; o >>= 1) ubm[r] = fmaxf(ubm[r], __shfl_xor(ubm[r], o));
                if (flat[r]) ubm[r] = 4.0f;  // every block of a flat candidate is evaluated
            }
            const int64_t blk = ch * SC_WAVES + w;
            if (ca == 0 && blk < nblk)
                *(float4*)(s.ub + ((int64_t)g * nblk + blk) * PM_G + 4 * ka) =
                    make_float4(ubm[0], ubm[1], ubm[2], ubm[3]);
        }
        // the workgroup's lower bounds of this group
#pragma unroll
        for (int r = 0; r < 4; ++r) {
#pragma unroll
            for (int o = 8; o >= 1; o >>= 1) lbr[r] = fmaxf(lbr[r], __shfl_xor(lbr[r], o));
            if (ca == 0) lbw[w][4 * ka + r] = flat[r] ? -4.0f : lbr[r];
        }
        __syncthreads();
        if (tid < PM_G) {
            float v = lbw[0][tid];
            for (int q = 1; q < SC_WAVES; ++q) v = fmaxf(v, lbw[q][tid]);
            const int64_t e = (int64_t)blockIdx.x - first / sh.per + g;
            s.lbp[e * PM_G + tid] = v;
        }
    }
}

// Exact FP64 nearest-neighbour correlation of the candidate rows: direct
// centred dot products (no recurrence), the reference the reported distances
// and neighbour indices come from.  X (candidates x m) . H (m x columns) with
// H[k][j] = t_{j+k} on the FP64 matrix cores: V_MFMA_F64_16X16X4F64
// multiplies a 16 x 4 block of candidate values by a 4 x 16 block of the
// series, lane l supplying X[l % 16][l / 16] and H[l / 16][l % 16] and
// receiving D[l / 16 + 4 r][l % 16], r < 4.  A block is EX_COLS columns, EX_CT
// tiles per wave: small, because after the screening a group has a few blocks
// and their latency counts.  With `screened` only the marked blocks run.  One
// (max rho, argmax j) partial per candidate, group and workgroup, in the
// order the workgroups finish (slots from one counter per group).
__global__ __launch_bounds__(64 * EX_WAVES) void k_exact(SeriesDev* S, int B, int large, int full, int screened,
                                                         int screen_grid,
                                                         const int64_t* __restrict__ ipfx_s,
                                                         const int64_t* __restrict__ ipfx_e)
{
    extern __shared__ double lds[];
    __shared__ double red_v[EX_WAVES][PM_G];
    __shared__ long long red_j[EX_WAVES][PM_G];
    __shared__ double sxs[PM_G], civ[PM_G], cmu[PM_G];
    __shared__ int64_t cidx[PM_G];
    __shared__ float lbs[EX_WAVES * 4][PM_G];
    __shared__ unsigned long long mark_s[EX_WAVES];
    __shared__ unsigned int slot_s;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int ca = lane & 15, ka = lane >> 4;
    double* xg = lds;                 // [PM_G][PM_XS] candidate window chunk
    double* ts = lds + PM_G * PM_XS;  // t[j0 .. j0 + EX_COLS + m + 4 EX_STEPS)
    const int64_t total = B == 1 ? items_of(S[0], 0, full, false) : ipfx_e[B];
    const Share sh = share_of(total);
    for (int64_t it = sh.lo; it < sh.hi;) {
        const int b = B == 1 ? 0 : series_of(ipfx_e, B, it);
        const int64_t first = B == 1 ? 0 : ipfx_e[b];
        const SeriesDev& s = S[b];
        Ctrl* c = s.ctrl;
        const int ncand = cand_count(s, c, full);
        const int32_t m = c->m;
        const int64_t N = s.n - m + 1;
        const int64_t nblk = exact_blocks(N);
        const int g = (int)((it - first) / nblk);
        const int64_t b0 = (it - first) - g * nblk;
        const int64_t b1 = std::min<int64_t>(nblk, b0 + (sh.hi - it));
        it += b1 - b0;
        const int g0 = PM_G * g;
        const double* __restrict__ T = s.T;
        const double* __restrict__ mu = cur_mu(s, c);
        const double* __restrict__ inv = s.inv64;  // 1/(sqrt(m) sigma), 0 for a flat window
        const bool single = m <= PM_KC;
        bool loaded = false, any = false;
        double best[4];
        long long bj[4];
        unsigned int evb = 0;
        int64_t ci[4];
        double sxv[4], ivi[4];
        __syncthreads();
        // the group's indices, means and spreads, fetched while the bounds are
        if (tid < PM_G) {
            const int64_t i = s.cand[min(g0 + tid, ncand - 1)];
            cidx[tid] = i;
            cmu[tid] = mu[i];
            civ[tid] = inv[i];
        }
        float lb = -8.0f;  // lower bound of candidate tid % 16
        if (screened) {
            // the lower bounds the screening's workgroups left
            const int64_t nch = screen_chunks(N);
            const int64_t firsts = B == 1 ? 0 : ipfx_s[b];
            const int64_t tots = B == 1 ? items_of(s, 0, full, true) : ipfx_s[B];
            const int64_t pers = (tots + screen_grid - 1) / screen_grid;
            const int64_t w0 = firsts / pers;
            const int gs = screen_groups(large, m, (ncand + PM_G - 1) / PM_G, nch), sg = g / gs;
            const int64_t e0 = (firsts + sg * nch) / pers - w0 + sg;
            const int64_t e1 = (firsts + (sg + 1) * nch - 1) / pers - w0 + sg;
            const float* lbg = s.lbp + (g - sg * gs) * PM_G + (tid & 15);
            constexpr int EN = EX_WAVES * 4;  // entries per pass of the workgroup
            for (int64_t e = e0 + (tid >> 4); e <= e1; e += 8 * EN) {
                float v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    v[u] = e + u * EN <= e1 ? lbg[(e + u * EN) * gs * PM_G] : -8.0f;
#pragma unroll
                for (int u = 0; u < 8; ++u) lb = fmaxf(lb, v[u]);
            }
            lbs[tid >> 4][tid & 15] = lb;
        }
        __syncthreads();
        if (screened)
            for (int q = 0; q < EX_WAVES * 4; ++q) lb = fmaxf(lb, lbs[q][tid & 15]);
        for (int64_t bb = b0; bb < b1; bb += EX_WAVES * 4) {
            // sixteen blocks at a time: which of them hold a column that counts
            {
                const int64_t q = bb + (tid >> 4);
                const int cid = tid & 15;
                bool mk = q < b1 && g0 + cid < ncand;
                if (mk && screened) mk = s.ub[((int64_t)g * nblk + q) * PM_G + cid] >= lb;
                const unsigned long long bal = __ballot(mk);
                __syncthreads();
                if (lane == 0) mark_s[w] = bal;
                __syncthreads();
            }
            for (int e = 0; e < EX_WAVES * 4; ++e) {
                if (((mark_s[e >> 2] >> (16 * (e & 3))) & 0xffffull) == 0ull) continue;
                const int64_t blk = bb + e;
                const int64_t j0 = blk * EX_COLS;
                const int colbase = w * (EX_COLS / EX_WAVES);
                // the columns' spreads and means, in flight during the products
                double ivj[EX_CT], muj[EX_CT];
#pragma unroll
                for (int ct = 0; ct < EX_CT; ++ct) {
                    const int64_t j = j0 + colbase + 16 * ct + ca;  // (inside the padded buffers)
                    ivj[ct] = inv[j];
                    muj[ct] = mu[j];
                }
                pm_acc_t acc[EX_CT];
#pragma unroll
                for (int ct = 0; ct < EX_CT; ++ct) acc[ct] = (pm_acc_t){0.0, 0.0, 0.0, 0.0};
                for (int kb = 0; kb < m; kb += PM_KC) {
                    const int kn = min(PM_KC, m - kb);
                    __syncthreads();  // the previous chunk and block are consumed
                    const bool fill = !single || !loaded;
                    if (fill) {
                        // every load of the chunk's windows before its stores
                        constexpr int NG = PM_G / EX_WAVES, NQ = PM_KC / 64;
                        double v[NG][NQ];
#pragma unroll
                        for (int u = 0; u < NG; ++u) {
                            const double* __restrict__ x = T + cidx[w + EX_WAVES * u] + kb;
#pragma unroll
                            for (int q = 0; q < NQ; ++q)
                                v[u][q] = lane + 64 * q < kn ? x[lane + 64 * q] : 0.0;
                        }
                        if (kb == 0) lds_fill(ts, T + j0, EX_COLS + m + 4 * EX_STEPS);
#pragma unroll
                        for (int u = 0; u < NG; ++u) {
                            const int gq = w + EX_WAVES * u;
                            const double mi = cmu[gq];
                            double sx = 0.0;
#pragma unroll
                            for (int q = 0; q < NQ; ++q) {
                                const int k = lane + 64 * q;
                                const double d = k < kn ? v[u][q] - mi : 0.0;
                                xg[gq * PM_XS + k] = d;
                                sx += d;
                            }
                            if (!any) {  // the windows' sums (zero up to rounding)
                                sx = wave_sum(sx);
                                if (lane == 0) sxs[gq] = kb ? sxs[gq] + sx : sx;
                            }
                        }
                        loaded = true;
                    } else if (kb == 0) {
                        lds_fill(ts, T + j0, EX_COLS + m + 4 * EX_STEPS);
                    }
                    __syncthreads();
                    const double* xp = xg + ca * PM_XS + ka;
                    const double* tb = ts + colbase + kb + ka + ca;
                    // eight steps' operands are read before their products (one
                    // wave per SIMD: nothing else hides the LDS latency); the
                    // window is zero past kn, the stretch finite
                    for (int k8 = 0; k8 < kn; k8 += 4 * EX_STEPS) {
                        double av[EX_STEPS], bv[EX_STEPS][EX_CT];
#pragma unroll
                        for (int u = 0; u < EX_STEPS; ++u) {
                            av[u] = xp[k8 + 4 * u];
#pragma unroll
                            for (int ct = 0; ct < EX_CT; ++ct) bv[u][ct] = tb[k8 + 4 * u + 16 * ct];
                        }
#pragma unroll
                        for (int u = 0; u < EX_STEPS; ++u)
#pragma unroll
                            for (int ct = 0; ct < EX_CT; ++ct)
                                acc[ct] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[u], bv[u][ct],
                                                                               acc[ct], 0, 0, 0);
                    }
                }
                if (!any) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        ci[r] = cidx[ka + 4 * r];
                        sxv[r] = sxs[ka + 4 * r];
                        ivi[r] = civ[ka + 4 * r];
                        best[r] = -f_inf<double>();
                        bj[r] = 0x7fffffffffffffffll;
                    }
                    any = true;
                }
                // epilogue: lane holds D[ka + 4 r][16 ct + ca]; rho = C inv_i inv_j
#pragma unroll
                for (int ct = 0; ct < EX_CT; ++ct) {
                    const int64_t j = j0 + colbase + 16 * ct + ca;
                    if (j >= N) continue;
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        if (j <= ci[r] - m || j >= ci[r] + m) {
                            double rh;
                            if (ivi[r] == 0.0 || ivj[ct] == 0.0) {  // a flat window (R11)
                                rh = (ivi[r] == 0.0 && ivj[ct] == 0.0) ? 1.0 : 0.0;
                            } else {
                                const double Cv = acc[ct][r] - muj[ct] * sxv[r];
                                rh = fmin(1.0, fmax(-1.0, Cv * ivi[r] * ivj[ct]));
                            }
                            if (rh > best[r]) {  // a lane's columns ascend with ct and with the block
                                best[r] = rh;
                                bj[r] = j;
                            }
                            if (g0 + ka + 4 * r < ncand) ++evb;
                        }
                    }
                }
            }
        }
        if (!any) continue;  // (uniform over the workgroup)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
#pragma unroll
            for (int o = 8; o >= 1; o >>= 1) {  // the 16 lanes of one candidate row
                const double v = __shfl_xor(best[r], o);
                const long long jj = __shfl_xor(bj[r], o);
                if (v > best[r] || (v == best[r] && jj < bj[r])) {
                    best[r] = v;
                    bj[r] = jj;
                }
            }
            if (ca == 0) {
                red_v[w][ka + 4 * r] = best[r];
                red_j[w][ka + 4 * r] = bj[r];
            }
        }
        if (tid == 0) slot_s = atomicAdd(&c->pcnt[g], 1u);
        __syncthreads();
        if (tid < PM_G) {
            double bv = red_v[0][tid];
            long long bjj = red_j[0][tid];
            for (int q = 1; q < EX_WAVES; ++q)
                if (red_v[q][tid] > bv || (red_v[q][tid] == bv && red_j[q][tid] < bjj)) {
                    bv = red_v[q][tid];
                    bjj = red_j[q][tid];
                }
            const int64_t p = ((part_base(sh.per, first, nblk, g) + slot_s) * PM_G + tid) * 2;
            s.part[p] = bv;
            s.part[p + 1] = (double)bjj;
        }
        const unsigned long long e = (unsigned long long)wave_sum((double)evb);
        if (lane == 0 && e)
            atomicAdd(&s.evc[EV_POL * EV_SLOTS + ((blockIdx.x + w) & (EV_SLOTS - 1))], e);
    }
}

// ---------------------------------------------------------------------------
// dense rounds: many range discords
// ---------------------------------------------------------------------------
// The first length halves r until k range discords are found, and the last
// of these ranges can lie far below the k-th distance: a quarter of all
// subsequences may be range discords, each to be proved against every column;
// later lengths can have thousands of them as well.  The sweeps would scan
// nearly every tile against every column, on the right in FP32 and on the
// left in FP64.  Instead such a round runs the first selection pass over a
// part of its columns (dense_near; not at all where the witnesses already
// pruned what falls), lists the rows left (k_dense_list) and bounds each of
// them against all columns on the FP16 matrix cores as k_screen does
// (k_dense, the same operands and error bound): rows with a pair above the
// threshold, or within the error of it, are decided by FP64 dot products
// (k_pairs), and a row without one is a range discord.  Only rows whose
// largest correlation may be among the k smallest go to the exact pass
// (k_dense_top).  Heatmaps report every range discord's exact maximum, and
// windows past 256 points leave no room for the operands: both sweep.
// Measured against sweeps: 200,000 points, m = 96, 51,000 range discords: the
// round's sweeps 14 ms, this 5.7 ms (620 TFLOP/s); 64 series of 10,000 to
// 200,000 points: the search 480 ms, with dense rounds 175; 100,000 points,
// lengths 64-128: 8.4 ms, then 7.2.
constexpr int DN_ROWS = DENSE_ROWS;      // rows per item, DN_G groups of 16
constexpr int DN_G = DN_ROWS / 16;
constexpr int DN_BUF = 512;              // entries buffered per workgroup

// The rows left, ascending (one block per series); few enough of them are
// candidates at once.  In a round without sweeps (full = 0) every series with
// too many rows left for that is taken here, unless its witnesses failed
// altogether.
__device__ __forceinline__ bool dense_possible(const SeriesDev& s, const Ctrl* c)
{
    return c->prune && s.heat == nullptr && c->m <= DENSE_MAXM && c->thr64 >= DENSE_MIN_THR &&
           !dense_off(c);
}
__device__ __forceinline__ bool dense_allowed(const SeriesDev& s, const Ctrl* c)
{
    return c->nlive != 0x7fffffffu && dense_possible(s, c);
}
__global__ __launch_bounds__(TOPK_BLOCK) void k_dense_list(SeriesDev* S, int full)
{
    __shared__ unsigned int wsum[TOPK_BLOCK / 64];
    const SeriesDev& s = S[blockIdx.x];
    Ctrl* c = s.ctrl;
    if (!c->active || lean_round(c) || taking_parts(c)) return;
    if (!dense_round(c) && (full || !dense_allowed(s, c))) return;
    if (!full && c->dense == DENSE_SWEEP) return;  // its first pass has not run
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int64_t nw = (s.n - c->m + 1 + 63) / 64;
    const unsigned int lean_max = c->lean_max;
    unsigned int base = 0;
    for (int64_t q0 = 0; q0 < nw; q0 += TOPK_BLOCK) {
        const int64_t q = q0 + tid;
        unsigned long long bits = q < nw ? s.alive[q] : 0ull;
        const unsigned int cnt = (unsigned int)__popcll(bits);
        unsigned int x = cnt;
        for (int o = 1; o < 64; o <<= 1) {
            const unsigned int y = __shfl_up(x, o);
            if (lane >= o) x += y;
        }
        __syncthreads();
        if (lane == 63) wsum[w] = x;
        __syncthreads();
        unsigned int before = 0, tot = 0;
        for (int e = 0; e < TOPK_BLOCK / 64; ++e) {
            before += e < w ? wsum[e] : 0u;
            tot += wsum[e];
        }
        unsigned int p = base + before + x - cnt;
        while (bits) {
            const int t = __ffsll((long long)bits) - 1;
            bits &= bits - 1ull;
            const int64_t i = q * 64 + t;
            if (p < lean_max) s.cand[p] = i;
            s.fail[p++] = (int32_t)i;
            s.rho[i] = 0x000fffffffffffffull;  // ordered bits of -inf
            s.rhs[i] = 0x000fffffffffffffull;
        }
        base += tot;
    }
    __syncthreads();  // (the control block is read until here)
    // many rows of a long series: a first pass over some columns prunes most of
    // them for less than bounding them all costs
    if (!full && (double)base * (double)(s.n - c->m + 1) * (double)c->m > DENSE_LEFT_WORK) {
        if (tid == 0) c->dense = DENSE_SWEEP;
        return;
    }
    if (tid == 0) {
        c->handled = 1;
        c->rows_near += base;
        c->npairs = 0;
        c->lost = 0;
        c->cand_total = 0;
        if (base <= lean_max) {
            c->dense = DENSE_NO;
            c->live_ref = base;  // a direct round
            c->rows_far += base;
            c->nsurv = base;
            c->ncand = base < (unsigned int)s.k ? 0u : base;
        } else {
            c->dense = DENSE_LEFT;
            c->ndense = base;
        }
    }
}

// One item: DN_ROWS listed rows against one segment of the columns, four waves
// of 128 columns each per chunk of 512.  A wave computes a 64 x 128 tile of
// products in parts (128 accumulators do not fit two waves per SIMD); for
// windows of 33 to 128 points (STEPS operand steps of 32) the rows' operands
// stay in registers for the whole item, as many as the window needs, so that
// eight matrix instructions take two LDS reads (200,000 points, m = 96: four
// steps kept for every window 6.5 ms, three 5.7);
// from LDS (STEPS = 0, every other window) they take six, which is as long as
// the products.  The next chunk's series values are fetched during the
// products.  Bound by the matrix cores (2 m flops per pair) and, for short
// windows, by the 1.5 vector operations per product that fold it into its
// row's maximum.  A row with a product that may exceed the threshold hands the
// lane's eight columns to k_pairs; if it surely does, the row is out of the
// item.  A workgroup that hands an entry over past the end of the list ends its
// item, and every later item ends at once: the round has given up.  (20,000
// points whose level jumps by 3000 deviations of the noise, 17 lengths: 45 ms
// with an addition to the counter per lane, 4.6 with one per wave and the
// end; always sweeping 3.7.)  (Workgroups take the items in turn, two of this
// size per CU: a launch of all items of 64 series measured 2 ms with nothing to
// do, this 0.1.  Registers over the budget spill outside the loop over the
// products.)
template <int STEPS>
__device__ __forceinline__ void dense_item(const SeriesDev& s, Ctrl* c, int64_t tile, int seg, int segs,
                                           _Float16* dxa, half8_t (*wcopy)[SC_SLOTS], float* gjs,
                                           int32_t* rows,
                                           float (*bnd)[SC_WAVES][DN_ROWS],
                                           unsigned long long* dead_p, unsigned int* npair_p,
                                           unsigned int* gbase_p, int2* buf)
{
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int ca = lane & 15, ka = lane >> 4;
    const int32_t m = c->m;
    const int64_t N = s.n - m + 1;
    const unsigned int nrow = c->ndense;
    const double* __restrict__ T = s.T;
    const double* __restrict__ mu = cur_mu(s, c);
    const double* __restrict__ inv = s.inv64;
    const float thr = (float)c->thr64;
    const int stride = dense_stride(m);
    __syncthreads();  // (the previous item is consumed)
    if (tid == 0) *npair_p = 0u;
    if (tid < DN_ROWS)
        rows[tid] = s.fail[std::min<int64_t>(tile * DN_ROWS + tid, (int64_t)nrow - 1)];
    __syncthreads();
    // the rows' windows, centred and scaled to norm 1024
#pragma unroll 1
    for (int r0 = w; r0 < DN_ROWS; r0 += 4 * SC_WAVES) {
        constexpr int NQ = (DENSE_MAXM + 63) / 64 + 1;
        double v[4][NQ], mi[4], sc[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t i = rows[r0 + SC_WAVES * u];
            mi[u] = mu[i];
            sc[u] = inv[i] * 1024.0;
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                const int k = lane + 64 * q;
                v[u][q] = k < m ? T[i + k] : 0.0;
            }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                const int k = lane + 64 * q;
                if (k < stride)
                    dxa[(r0 + SC_WAVES * u) * stride + k] =
                        k < m ? (_Float16)(float)((v[u][q] - mi[u]) * sc[u]) : (_Float16)0.0f;
            }
    }
    // rows past the list, rows pruned meanwhile, and flat rows (R11:
    // correlation 1 with another flat window, 0 with any other, so a partner
    // decides)
    if (tid < DN_ROWS) {
        const int64_t i = rows[tid];
        bool off = tile * DN_ROWS + tid >= (int64_t)nrow ||
                   !((load_word(&s.alive[i >> 6]) >> (i & 63)) & 1ull);
        if (!off && inv[i] == 0.0) {
            const int64_t flo = c->flat_min, fhi = c->flat_max;
            const bool lo_ok = flo >= 0 && flo <= i - m, hi_ok = fhi >= 0 && fhi >= i + m;
            if (lo_ok || hi_ok) {
                off = true;
                s.wit[i] = ~(int32_t)(lo_ok ? flo : fhi);
                atomicAnd(&s.alive[i >> 6], ~(1ull << (i & 63)));
            }
        }
        // (a round that has given up: no row of the item is left)
        const unsigned long long d = __ballot(off || load_flag(&c->lost) != 0u);
        if (tid == 0) *dead_p = d;
    }
    __syncthreads();
    int32_t rmin = 0x7fffffff, rmax = -1;
#pragma unroll
    for (int q = 0; q < 4 * DN_G; ++q) {
        const int32_t i = rows[16 * (q >> 2) + 4 * ka + (q & 3)];
        rmin = min(rmin, i);
        rmax = max(rmax, i);
    }
    const _Float16* ap = dxa + ca * stride + 8 * ka;
    half8_t areg[STEPS ? STEPS : 1][DN_G];
    float ubr[4 * DN_G];
#pragma unroll
    for (int q = 0; q < 4 * DN_G; ++q) ubr[q] = -4.0f;
    float em_max = 0.0f;
    unsigned long long seen = 0ull;
    bool fresh = true;  // the rows' operands changed
    const float e0 = 1.05f * (2.0f * 0x1p-11f + 0x1p-22f + (float)(m + 32) * 0x1p-23f +
                              sqrtf((float)m) * 0x1p-23f);
    const float fl = sqrtf((float)m) * 0x1p-13f;
    const int64_t nch = screen_chunks(N);
    const int64_t ch0 = nch * seg / segs, ch1 = nch * (seg + 1) / segs;
    const int steps = (m + 31) >> 5;
    ChunkRegs R;
    auto flush = [&]() {  // hand the listed entries over (whole workgroup)
        const unsigned int np = min(*npair_p, (unsigned int)DN_BUF);
        if (tid == 0 && np) {
            *gbase_p = atomicAdd(&c->npairs, np);
            if ((int64_t)*gbase_p + np > dense_pairs(s.Npad)) {
                atomicOr(&c->lost, 1u);
                *dead_p = ~0ull;  // the item ends
            }
        }
        __syncthreads();
        for (unsigned int q = tid; q < np; q += 64 * SC_WAVES)
            if ((int64_t)*gbase_p + q < dense_pairs(s.Npad)) s.pairs[*gbase_p + q] = buf[q];
        __syncthreads();
        if (tid == 0) *npair_p = 0u;
    };
    unsigned int ev = 0, left = DN_ROWS;  // rows times blocks, rows not dead
    fetch_chunk(s, mu, inv, ch0, R);
    for (int64_t ch = ch0; ch < ch1; ++ch) {
        const int64_t j0 = ch * SC_COLS;
        const int64_t jb = j0 + w * EX_COLS;
        __syncthreads();  // the previous chunk's operands are consumed
        const unsigned long long dead = *dead_p;  // (written only between the next barrier and this one)
        if (dead == ~0ull) break;
        if (*npair_p > DN_BUF / 2) {
            __syncthreads();
            flush();
        }
        stage_chunk(R, wcopy);
        float em = 0.0f;  // largest error bound of the wave's columns
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const float2 x = chunk_column(R, q, m, e0, fl);
            if (jb + lane + 64 * q < N) em = fmaxf(em, x.y);
            gjs[w * EX_COLS + lane + 64 * q] = x.x;
        }
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) em = fmaxf(em, __shfl_xor(em, o));
        // a dead row's window becomes zero: its products then stay below the
        // threshold (positive by DENSE_MIN_THR); with a wide bound they pass the
        // test below all the same, which leaves the dead rows out
        if (dead != seen) {
            for (unsigned long long d = (dead & ~seen) & (0x1111111111111111ull << w); d; d &= d - 1ull) {
                const int r = __ffsll((long long)d) - 1;
                for (int k = lane; k < stride; k += 64) dxa[r * stride + k] = (_Float16)0.0f;
            }
            seen = dead;
            left = (unsigned int)(DN_ROWS - __popcll(uniform64(dead)));
            fresh = true;
        }
        __syncthreads();
        if (STEPS && fresh) {
#pragma unroll
            for (int st = 0; st < STEPS; ++st)
#pragma unroll
                for (int g = 0; g < DN_G; ++g)
                    areg[st][g] = *(const half8_t*)(ap + 16 * g * stride + 32 * st);
            fresh = false;
        }
        if (ch + 1 < ch1) fetch_chunk(s, mu, inv, ch + 1, R);
        if (jb >= N) continue;  // (the next barrier is the loop's first)
        const int slot = w * (EX_COLS / 8) + ca + ka;
        const bool edge = __ballot(jb + EX_COLS > N ||
                                   ((int64_t)rmin < jb + EX_COLS + m && (int64_t)rmax > jb - m)) != 0ull;
        float mx[4 * DN_G];
#pragma unroll
        for (int q = 0; q < 4 * DN_G; ++q) mx[q] = -4.0f;
        // NU of the eight shifts at a time
        constexpr int NU = STEPS ? 2 : 4;
#pragma unroll 1
        for (int hf = 0; hf < 8 / NU; ++hf) {
            acc4f_t acc[DN_G][NU];
#pragma unroll
            for (int g = 0; g < DN_G; ++g)
#pragma unroll
                for (int u = 0; u < NU; ++u) acc[g][u] = (acc4f_t){0.f, 0.f, 0.f, 0.f};
            if (STEPS) {
#pragma unroll
                for (int st = 0; st < STEPS; ++st) {
#pragma unroll
                    for (int u = 0; u < NU; ++u) {
                        const half8_t bv = wcopy[NU * hf + u][slot + 4 * st];
#pragma unroll
                        for (int g = 0; g < DN_G; ++g)
                            acc[g][u] = __builtin_amdgcn_mfma_f32_16x16x32_f16(areg[st][g], bv,
                                                                               acc[g][u], 0, 0, 0);
                    }
                }
            } else {
                for (int st = 0; st < steps; ++st) {
                    half8_t av[DN_G];
#pragma unroll
                    for (int g = 0; g < DN_G; ++g)
                        av[g] = *(const half8_t*)(ap + 16 * g * stride + 32 * st);
#pragma unroll
                    for (int u = 0; u < NU; ++u) {
                        const half8_t bv = wcopy[NU * hf + u][slot + 4 * st];
#pragma unroll
                        for (int g = 0; g < DN_G; ++g)
                            acc[g][u] = __builtin_amdgcn_mfma_f32_16x16x32_f16(av[g], bv, acc[g][u],
                                                                               0, 0, 0);
                    }
                }
            }
            // lane: rows 16 g + 4 ka + r, columns jl + u
            float gj[NU];
#pragma unroll
            for (int u = 0; u < NU; ++u) gj[u] = gjs[w * EX_COLS + 8 * ca + NU * hf + u];
            if (!edge) {
#pragma unroll
                for (int g = 0; g < DN_G; ++g)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        float v = mx[4 * g + r];
#pragma unroll
                        for (int u = 0; u < NU; ++u) v = fmaxf(v, acc[g][u][r] * gj[u]);
                        mx[4 * g + r] = v;
                    }
            } else {
                const int32_t jl = (int32_t)jb + 8 * ca + NU * hf;
#pragma unroll
                for (int g = 0; g < DN_G; ++g)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int32_t i = rows[16 * g + 4 * ka + r];
#pragma unroll
                        for (int u = 0; u < NU; ++u) {
                            const int32_t j = jl + u;
                            const bool ok = (int64_t)j < N && (j <= i - m || j >= i + m);
                            mx[4 * g + r] = fmaxf(mx[4 * g + r], ok ? acc[g][u][r] * gj[u] : -4.0f);
                        }
                    }
            }
        }
        em_max = fmaxf(em_max, em);
        float any = -4.0f;
#pragma unroll
        for (int q = 0; q < 4 * DN_G; ++q) {
            ubr[q] = fmaxf(ubr[q], mx[q] + em);  // (-4 + em: no pair yet)
            any = fmaxf(any, mx[q]);
        }
        if (__ballot(any + em > thr) != 0ull) {
            bool room = true;  // in the list (uniform over the wave)
#pragma unroll 1
            for (int q = 0; q < 4 * DN_G; ++q) {
                float v = mx[0];
#pragma unroll
                for (int e = 1; e < 4 * DN_G; ++e) v = q == e ? mx[e] : v;
                const int rr = 16 * (q >> 2) + 4 * ka + (q & 3);
                const bool hand = v + em > thr && !((seen >> rr) & 1ull);
                const unsigned long long bal = __ballot(hand);
                if (bal == 0ull) continue;
                // one reservation per wave: a counter takes one addition at a time
                const int lead = __ffsll((long long)bal) - 1;
                const unsigned int cnt = (unsigned int)__popcll(bal);
                const unsigned int at = (unsigned int)__popcll(bal & ((1ull << lane) - 1ull));
                const int2 pr = make_int2(rows[rr], (int32_t)jb + 8 * ca);
                unsigned int p = 0;
                if (lane == lead) p = atomicAdd(npair_p, cnt);
                p = (unsigned int)__builtin_amdgcn_readlane((int)p, lead);
                const unsigned int fit =
                    min(cnt, p < (unsigned int)DN_BUF ? (unsigned int)DN_BUF - p : 0u);
                if (hand && at < fit) buf[p + at] = pr;
                if (fit < cnt && room) {  // (buffer full)
                    unsigned int gp = 0;
                    if (lane == lead) gp = atomicAdd(&c->npairs, cnt - fit);
                    gp = (unsigned int)__builtin_amdgcn_readlane((int)gp, lead);
                    const int64_t end = dense_pairs(s.Npad);
                    if (hand && at >= fit && (int64_t)gp + (at - fit) < end) s.pairs[gp + (at - fit)] = pr;
                    room = (int64_t)gp + (cnt - fit) <= end;
                    if (!room && lane == lead) {
                        atomicOr(&c->lost, 1u);
                        atomicOr(dead_p, ~0ull);  // the item ends
                    }
                }
                if (hand && v - em > thr) atomicOr(dead_p, 1ull << rr);  // surely closer than r
            }
        }
        ev += left;
    }
    __syncthreads();
    flush();
    // the rows' upper bounds over this segment; a row's largest correlation is
    // at least that less twice the error of the block that gave it
#pragma unroll
    for (int q = 0; q < 4 * DN_G; ++q) {
#pragma unroll
        for (int o = 8; o >= 1; o >>= 1) ubr[q] = fmaxf(ubr[q], __shfl_xor(ubr[q], o));
        if (ca == 0) {
            bnd[0][w][16 * (q >> 2) + 4 * ka + (q & 3)] = ubr[q];
            bnd[1][w][16 * (q >> 2) + 4 * ka + (q & 3)] = ubr[q] - 2.01f * em_max;
        }
    }
    __syncthreads();
    if (tid < DN_ROWS && !((*dead_p >> tid) & 1ull)) {
        float u = -4.0f, l = -4.0f;
        for (int q = 0; q < SC_WAVES; ++q) {
            u = fmaxf(u, bnd[0][q][tid]);
            l = fmaxf(l, bnd[1][q][tid]);
        }
        const int64_t i = rows[tid];
        if (u > -2.0f) {
            atomicMax(&s.rhs[i], ord_of((double)u));
            atomicMax(&s.rho[i], ord_of((double)l));
        }
    }
    if (lane == 0 && ev)
        atomicAdd(&s.evc[EV_DENSE * EV_SLOTS + ((blockIdx.x + w) & (EV_SLOTS - 1))],
                  (unsigned long long)ev * EX_COLS);
}

// Row tiles of a series' list.
__device__ __forceinline__ int64_t dense_tiles(const Ctrl* c)
{
    return c->active && !lean_round(c) && dense_round(c) && c->handled && !taking_parts(c)
               ? ((int64_t)c->ndense + DN_ROWS - 1) / DN_ROWS
               : 0;
}

// First row tile of every series (one block; one series needs no table).
__global__ __launch_bounds__(ITEMS_BLOCK) void k_dense_items(SeriesDev* S, int B, int64_t* pfx)
{
    __shared__ long long ws[ITEMS_BLOCK / 64];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    long long base = 0;
    for (int b0 = 0; b0 < B; b0 += ITEMS_BLOCK) {
        const int b = b0 + tid;
        const long long v = b < B ? dense_tiles(S[b].ctrl) : 0;
        long long x = v;
        for (int o = 1; o < 64; o <<= 1) {
            const long long y = __shfl_up(x, o);
            if (lane >= o) x += y;
        }
        if (lane == 63) ws[w] = x;
        __syncthreads();
        long long before = 0, tot = 0;
        for (int e = 0; e < ITEMS_BLOCK / 64; ++e) {
            before += e < w ? ws[e] : 0;
            tot += ws[e];
        }
        if (b < B) pfx[b] = base + before + x - v;
        base += tot;
        __syncthreads();
    }
    if (tid == 0) pfx[B] = base;
}

__global__ __launch_bounds__(64 * SC_WAVES, 2) void k_dense(SeriesDev* S, int B,
                                                            const int64_t* __restrict__ pfx)
{
    extern __shared__ __align__(16) _Float16 dxa[];  // [DN_ROWS][dense_stride(m)]
    __shared__ half8_t wcopy[8][SC_SLOTS];
    __shared__ float gjs[SC_COLS];
    __shared__ int32_t rows[DN_ROWS];
    __shared__ float bnd[2][SC_WAVES][DN_ROWS];
    __shared__ unsigned long long dead_s;
    __shared__ unsigned int npair_s, gbase_s;
    __shared__ int2 buf[DN_BUF];
    const int64_t tiles = B == 1 ? dense_tiles(S[0].ctrl) : pfx[B];
    if (tiles == 0) return;
    // column segments: a few items per workgroup
    const int segs = (int)std::min<int64_t>(16, std::max<int64_t>(1, 3 * (int64_t)gridDim.x / tiles));
    for (int64_t it = blockIdx.x; it < tiles * segs; it += gridDim.x) {
        const int64_t t = it % tiles;
        const int seg = (int)(it / tiles);
        const int b = B == 1 ? 0 : series_of(pfx, B, t);
        const SeriesDev& s = S[b];
        Ctrl* c = s.ctrl;
        const int64_t tile = t - (B == 1 ? 0 : pfx[b]);
#define DENSE_ITEM(ST)                                                                        \
    dense_item<ST>(s, c, tile, seg, segs, dxa, wcopy, gjs, rows, bnd, &dead_s, &npair_s, &gbase_s, buf)
        switch ((c->m + 31) >> 5) {
        case 2: DENSE_ITEM(2); break;
        case 3: DENSE_ITEM(3); break;
        case 4: DENSE_ITEM(4); break;
        default: DENSE_ITEM(0); break;
        }
#undef DENSE_ITEM
    }
}

// The rows handed over, by direct FP64 dot products with the eight columns of
// each entry, eight lanes per column, one wave per entry: the best one above
// the threshold prunes the row and becomes its witness.
__global__ __launch_bounds__(RESCUE_BLOCK) void k_pairs(SeriesDev* S, int B,
                                                        const int64_t* __restrict__ pfx)
{
    const int lane = threadIdx.x & 63;
    const int sub = lane & 7, cq = lane >> 3;
    const int64_t wave = (int64_t)blockIdx.x * (RESCUE_BLOCK / 64) + (threadIdx.x >> 6);
    const int64_t nwaves = (int64_t)gridDim.x * (RESCUE_BLOCK / 64);
    // a batch: the waves lie evenly over its row tiles (k_dense_items), and a
    // series has those that meet its tiles (64 series: an even share 190 us
    // per round, this 65)
    const int64_t tiles = B == 1 ? 1 : pfx[B];
    if (tiles == 0) return;
    for (int64_t b = B == 1 ? 0 : series_of(pfx, B, wave * tiles / nwaves); b < B; ++b) {
        const int64_t t0 = B == 1 ? 0 : pfx[b], t1 = B == 1 ? 1 : pfx[b + 1];
        const int64_t first = t0 * nwaves / tiles;
        if (first > wave) break;
        const SeriesDev& s = S[b];
        Ctrl* c = s.ctrl;
        if (t0 == t1 || !c->active || lean_round(c) || !dense_round(c) || !c->handled) continue;
        if (taking_parts(c) || c->lost) continue;
        const int64_t nper = (t1 * nwaves - 1) / tiles - first + 1, w = wave - first;
        const int32_t m = c->m;
        const int64_t N = s.n - m + 1;
        const int64_t np = std::min<int64_t>(c->npairs, dense_pairs(s.Npad));
        const double* __restrict__ T = s.T;
        const double* __restrict__ mu = cur_mu(s, c);
        const double* __restrict__ inv = s.inv64;
        const double thr = c->thr64;
        for (int64_t p = w; p < np; p += nper) {
            const int2 pr = s.pairs[p];
            const int64_t i = pr.x, j = (int64_t)pr.y + cq;
            if (!((load_word(&s.alive[i >> 6]) >> (i & 63)) & 1ull)) continue;
            const bool ok = j < N && (j <= i - m || j >= i + m);
            double C = 0.0, rho = -4.0;
            if (ok) {
                const double mi = mu[i], mj = mu[j];
                for (int k = sub; k < m; k += 8) C = fma(T[i + k] - mi, T[j + k] - mj, C);
            }
#pragma unroll
            for (int o = 4; o >= 1; o >>= 1) C += __shfl_xor(C, o);
            if (ok) rho = pair_rho(C, inv[i], inv[j]);
            double br = rho;
            int bq = cq;
#pragma unroll
            for (int o = 8; o <= 32; o <<= 1) {
                const double r2 = __shfl_xor(br, o);
                const int q2 = __shfl_xor(bq, o);
                if (r2 > br || (r2 == br && q2 < bq)) {
                    br = r2;
                    bq = q2;
                }
            }
            if (br > thr && sub == 0 && cq == bq) {
                // (~j: several entries of a row may land here at once, and an index
                // and a covariance stored apart could come from different ones)
                s.wit[i] = ~(int32_t)j;
                atomicAnd(&s.alive[i >> 6], ~(1ull << (i & 63)));
            }
        }
    }
}

// After a dense round (one block per series): the number of range discords,
// and as candidates every one whose lower bound does not exceed the k-th
// smallest upper bound (rhs, rho: upper and lower bounds of the largest
// correlation); more than an exact pass takes are listed in s.fail, as the
// bounds do not outlive the screening.  The k-th smallest by k rounds of the block's minimum, each
// thread holding its own; only the winner looks for its next.
__global__ __launch_bounds__(TOPK_BLOCK) void k_dense_top(SeriesDev* S)
{
    constexpr int NW = TOPK_BLOCK / 64;
    __shared__ unsigned long long wu[NW];
    __shared__ long long wi[NW];
    __shared__ unsigned int cnt_s, nc_s;
    const SeriesDev& s = S[blockIdx.x];
    Ctrl* c = s.ctrl;
    if (!c->active || lean_round(c) || !dense_round(c) || !c->handled || taking_parts(c)) return;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int64_t nw = (s.n - c->m + 1 + 63) / 64;
    const int k = s.k;
    if (tid == 0) cnt_s = nc_s = 0;
    __syncthreads();
    unsigned int cnt = 0;
    // this thread's smallest key after `last`
    auto next_of = [&](const Key& last, bool count) {
        Key best = {~0ull, KEY_NONE};
        scan_words(s.alive, nw, [&](int64_t q, unsigned long long bits) {
            if (count) cnt += (unsigned int)__popcll(bits);
            while (bits) {
                const int t = __ffsll((long long)bits) - 1;
                bits &= bits - 1ull;
                const Key x = {s.rhs[q * 64 + t], q * 64 + t};
                if (key_less(last, x) && key_less(x, best)) best = x;
            }
        });
        return best;
    };
    Key mine = next_of(Key{0ull, -1}, true);
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) cnt += __shfl_xor(cnt, o);
    if (lane == 0) atomicAdd(&cnt_s, cnt);
    __syncthreads();
    const unsigned int ns = cnt_s;
    if (tid == 0) {
        c->live_ref = 0xffffffffu;  // not a direct round: every live row is a range discord
        c->rows_far += ns;
        c->nsurv = ns;
        c->ncand = 0;
    }
    const bool lost = c->lost != 0;
    if (ns < (unsigned int)k && !lost) return;
    Key kth = {0ull, -1};
    for (int r = 0; r < k && !lost; ++r) {
        const Key v = wave_min_key(mine);
        if (lane == 0) {
            wu[w] = v.u;
            wi[w] = v.i;
        }
        __syncthreads();
        kth = Key{wu[0], wi[0]};
        for (int q = 1; q < NW; ++q) {
            const Key x = {wu[q], wi[q]};
            if (key_less(x, kth)) kth = x;
        }
        __syncthreads();
        if (mine.i == kth.i && r + 1 < k) mine = next_of(kth, false);
    }
    if (!lost)
        scan_words(s.alive, nw, [&](int64_t q, unsigned long long bits) {
            while (bits) {
                const int t = __ffsll((long long)bits) - 1;
                bits &= bits - 1ull;
                const int64_t i = q * 64 + t;
                if (s.rho[i] <= kth.u) {
                    const unsigned int slot = atomicAdd(&nc_s, 1u);
                    if (slot < (unsigned int)CAND_MAX) s.cand[slot] = i;
                    s.fail[slot] = (int32_t)i;
                }
            }
        });
    __syncthreads();
    if (tid == 0) {
        if (lost || nc_s > dense_cands(s.n - c->m + 1)) {
            c->band_over = 1;  // the range again, with sweeps
            c->dense = lost || c->thrown ? DENSE_NEVER : DENSE_OFF;
            c->thrown = 1;
        } else {
            c->ncand = min(nc_s, (unsigned int)CAND_MAX);
            if (nc_s > (unsigned int)CAND_MAX) {
                c->cand_total = nc_s;
                c->cand_at = CAND_MAX;
            }
        }
    }
}

// Close the round of every series (one block each): reduce the exact pass's
// partials to each candidate's (rho, j), rank the candidates, write the
// length's top-k rows when the round found at least k range discords, lower
// MERLIN's r otherwise, and set up the series' next range search.  A round
// without sweeps (full = 0) that turned out to need them is left pending.
constexpr int END_BLOCK = 1024;
static_assert(END_BLOCK >= CAND_MAX, "a thread per candidate");
// Candidates per reported row above which the k largest are found in k rounds
// of the block's maximum instead of by every candidate's rank: a round costs
// two barriers and a reduction, a rank two LDS reads per candidate.  (64
// series with up to a thousand candidates each: k_round_end 41 us per round
// by ranks, so 15; 12,000 points 18.6, so 17.)
constexpr int RANK_PER_ROUND = 64;
__global__ __launch_bounds__(END_BLOCK) void k_round_end(SeriesDev* S, int32_t* rem, int hot_rows,
                                                          int full, int more, float guard,
                                                          int max_attempts, int B, int large,
                                                          const int64_t* __restrict__ ipfx_e)
{
    // the valid candidates, nvalid_s of them
    __shared__ double nn_s[CAND_MAX];
    __shared__ long long id_s[CAND_MAX];
    __shared__ long long jj_s[CAND_MAX];
    __shared__ unsigned long long ku_s[END_BLOCK / 64];
    __shared__ long long ki_s[END_BLOCK / 64];
    __shared__ unsigned int nvalid_s;
    __shared__ long long next_s[K_MAX];
    const SeriesDev& s = S[blockIdx.x];
    Ctrl* c = s.ctrl;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    if (!c->active) {
        if (tid == 0 && c->error) atomicAdd(&rem[REM_ERROR], 1);  // stays visible in later rounds
        if (tid == 0) c->heat_m = 0;
        return;
    }
    // the round's kind, read before any barrier: next_range rewrites the control
    // block at the end, and a wave that read it there could take another branch
    // (with barriers in it) than the thread that runs next_range
    const bool lean = lean_round(c), handled = c->handled != 0;
    const unsigned int cand_at = c->cand_at, cand_total = c->cand_total;
    const bool parts_left = handled && cand_at > 0 && cand_at < cand_total;
    const bool lost = c->lost != 0;
    // (what the tail needs too: each load there would be a memory latency more)
    const bool may_dense = dense_possible(s, c), hopeless = c->nlive == 0x7fffffffu;
    const bool wide = c->thr_sel - c->thr64 > WIDE_BAND;
    const unsigned int lean_max = c->lean_max;
    const int swept_before = c->sweeps;
    // (a dense round in a launch without dense kernels waits too)
    const bool swept = full && !dense_round(c);
    if (!swept && !lean && !handled) {
        if (tid == 0) {
            c->pending = 1;
            if (c->dense == DENSE_NO && dense_allowed(s, c)) c->dense = DENSE_LEFT;
            atomicMax(&rem[REM_LEFT], s.maxL - c->m + 1);
            if (c->dense != DENSE_LEFT) {
                atomicAdd(&rem[REM_SWEEP], 1);
                atomicAdd(&rem[REM_WITNESS], 1);
            }
            if (dense_round(c)) atomicAdd(&rem[REM_DENSE], 1);
        }
        return;
    }
    const int k = s.k;
    const int32_t m = c->m;
    const int li = c->li;
    const int kp = lean ? (int)c->nlive : (int)c->ncand;
    const bool direct = direct_round(c);
    if (tid == 0) nvalid_s = 0;
    __syncthreads();
    if (tid < FAIL_LISTS) c->nfail[tid] = 0;  // read by k_rescue only
    if (kp >= k) {
        // tpc threads per candidate (all candidates at once, tpc as large as
        // the block allows, at most a wave): strided partials loaded eight at
        // a time before they are compared (they come from other XCDs' caches,
        // so each batch costs a full memory latency), then a reduction over
        // the tpc threads.
        int tpc = 64;
        while (tpc > 1 && tpc * kp > END_BLOCK) tpc >>= 1;
        const int sub = tid & (tpc - 1);
        const int64_t nblk = exact_blocks(s.n - m + 1);
        const int64_t first = B == 1 ? 0 : ipfx_e[blockIdx.x];
        const int64_t total =
            B == 1 ? (int64_t)((kp + CAND_GROUP - 1) / CAND_GROUP) * nblk : ipfx_e[B];
        const int64_t per = (total + exact_grid(large) - 1) / exact_grid(large);
        for (int cid = tid / tpc; cid < kp; cid += END_BLOCK / tpc) {
            double best = -f_inf<double>(), bj = 1e300;
            const int g = cid / CAND_GROUP;
            const long long i = s.cand[cid];
            const double ii = s.inv64[i];
            const int np = (int)c->pcnt[g];
            const double* pc =
                s.part + (part_base(per, first, nblk, g) * CAND_GROUP + cid % CAND_GROUP) * 2;
            for (int p0 = sub; p0 < np; p0 += 8 * tpc) {
                double v[8], jj[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int64_t p = p0 + u * tpc;
                    v[u] = p < np ? pc[p * 2 * CAND_GROUP] : -f_inf<double>();
                    jj[u] = p < np ? pc[p * 2 * CAND_GROUP + 1] : 1e300;
                }
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    if (v[u] > best || (v[u] == best && jj[u] < bj)) {
                        best = v[u];
                        bj = jj[u];
                    }
            }
            for (int o = tpc >> 1; o >= 1; o >>= 1) {
                const double v = __shfl_xor(best, o);
                const double jj = __shfl_xor(bj, o);
                if (v > best || (v == best && jj < bj)) {
                    best = v;
                    bj = jj;
                }
            }
            if (sub == 0) {
                const double d2 = 2.0 * (double)m * (1.0 - best);
                const long long j = bj < 1e299 ? (long long)bj : -1;  // every candidate has a neighbour
                // a direct round decides here which live subsequences are range
                // discords (distance >= r, i.e. rho <= thr64), as refinement would
                int ok_i = 1;
                if (direct) {
                    ok_i = !(c->prune && best > c->thr64);
                    if (ok_i) s.rho[i] = ord_of(best);
                    else atomicAnd(&s.alive[i >> 6], ~(1ull << (i & 63)));
                    if (s.heat && ok_i)
                        s.heat[(int64_t)li * s.heat_ld + i] = fmin(2.0, fmax(0.0, 1.0 - best));
                }
                if (ok_i) {
                    const unsigned int v = atomicAdd(&nvalid_s, 1u);
                    nn_s[v] = sqrt(fmin(4.0 * (double)m, fmax(0.0, d2)));
                    id_s[v] = i;
                    jj_s[v] = j;
                }
                if (more && j >= 0) {  // the nearest neighbour is the best witness
                    const double ij = s.inv64[j];
                    // (a flat window's correlation is a convention, not its
                    // covariance: ~j has that computed at the next length)
                    const bool known = ii > 0.0 && ij > 0.0;
                    s.wit[i] = known ? (int32_t)j : ~(int32_t)j;
                    if (known) s.wc[i] = best / (ii * ij);
                }
            }
        }
    }
    __syncthreads();
    const unsigned int ns = direct ? (kp >= k ? nvalid_s : (lean ? c->nlive : c->nsurv)) : c->nsurv;
    // the candidates could not be narrowed: same r again, after sweeps with
    // both sides of every tile refined exactly, after a dense round with sweeps
    // (exactly too where the FP32 guard band is wide, as level jumps make it
    // that also lose a dense round: its sweeps would be repeated in turn.  300,000
    // points with jumps 160 -> 109 ms; refining both sides where the band is
    // narrow costs as much again: 600,000 points without jumps 65 ms, 46 on the
    // left alone)
    const bool redo = !lean && c->band_over != 0;
    const bool ok = ns >= (unsigned int)k && kp >= k && !redo;
    const int nv = kp >= k ? (int)nvalid_s : 0;
    auto write_row = [&](int t, int rank) {
        const int64_t row = (int64_t)li * k + rank;
        if (parts_left) {
            next_s[rank] = id_s[t];
            return;
        }
        if (s.idx) {
            s.idx[row] = id_s[t];
            s.len[row] = m;
            s.nn[row] = nn_s[t];
            s.nnidx[row] = jj_s[t];
        }
        if (rank == k - 1) s.hist[li] = nn_s[t];
    };
    if (ok && RANK_PER_ROUND * k < nv) {
        // the largest distance (ties: smallest index) k times; distances are not
        // negative, so their bits order as they do
        Key mine = {~0ull, KEY_NONE};
        if (tid < nv) mine = Key{~(unsigned long long)__double_as_longlong(nn_s[tid]), id_s[tid]};
        for (int r = 0; r < k; ++r) {
            const Key v = wave_min_key(mine);
            if (lane == 0) {
                ku_s[w] = v.u;
                ki_s[w] = v.i;
            }
            __syncthreads();
            Key first = {ku_s[0], ki_s[0]};
            for (int q = 1; q < END_BLOCK / 64; ++q) {
                const Key x = {ku_s[q], ki_s[q]};
                if (key_less(x, first)) first = x;
            }
            if (mine.i == first.i) {
                write_row(tid, r);
                mine = Key{~0ull, KEY_NONE};
            }
            __syncthreads();
        }
    } else if (ok && tid < nv) {
        const double nt = nn_s[tid];
        const long long it = id_s[tid];
        int rank = 0;
#pragma unroll 8
        for (int e = 0; e < nv; ++e) {
            const double ne = nn_s[e];
            const long long ie = id_s[e];
            rank += (ne > nt || (ne == nt && ie < it)) ? 1 : 0;
        }
        if (rank < k) write_row(tid, rank);
    }
    __syncthreads();
    if (parts_left) {  // the k best so far and the next part of the candidates
        const unsigned int take = min(cand_total - cand_at, (unsigned int)(CAND_MAX - k));
        for (unsigned int e = tid; e < k + take; e += END_BLOCK)
            s.cand[e] = e < (unsigned int)k ? next_s[e] : (long long)s.fail[cand_at + e - k];
        if (tid < CAND_GROUPS) c->pcnt[tid] = 0;
        if (tid == 0) {
            c->ncand = k + take;
            c->cand_at = cand_at + take;
            c->pending = 1;
            atomicMax(&rem[REM_LEFT], s.maxL - m + 1);
        }
        return;
    }
    if (tid == 0) {
        c->cand_at = 0;
        c->rounds += 1;
        c->nsurv = ns;
        if (lean) {
            c->rows_near += c->nlive;
            c->rows_far += c->nlive;
        }
        c->exact_ref = redo && (!handled || (lost && wide)) ? 1 : 0;
        c->pending = 0;
        const bool many = may_dense ? (int64_t)ns * 2 > s.n - m + 1 : ns > lean_max;
        c->sweeps = li == 0 || lean || handled || (may_dense && !hopeless)
                        ? SWEEPS_NO
                        : (swept_before ? SWEEPS_AGAIN : 0) | (many ? SWEEPS_MANY : SWEEPS_FEW);
        // (a heatmap row of a round that refined: the bitmap's rows, by k_heat)
        c->heat_m = ok && !direct ? m : 0;
        if (ok) {
            c->done = 1;
            c->survivors += ns;
            if (s.count) s.count[li] = (int32_t)ns;
            if (s.rlen) s.rlen[li] = c->r;
        } else if (!redo) {
            c->done = 0;
            if (c->mode == 0) c->r *= 0.5;
            else if (c->mode == 1) c->r *= 0.99;
            else if (c->mode == 2) c->r = (c->step > 0.0) ? c->r - c->step : 0.99 * c->r;
        } else {
            c->done = 0;
        }
    }
    if (swept && !lean && !handled) {
        // Hot tiles of hot_rows rows, in ascending order (the first HOT_MAX of
        // them): those that still hold survivors or whose first-pass items swept
        // at least N / HOT_FRAC columns this round.  The next sweep's first
        // selection pass dispatches all their chunks before any other tile's, so
        // that the longest work items of the pass start first.  The per-tile
        // work counters restart.
        __shared__ unsigned int wcnt_s[END_BLOCK / 64];
        __shared__ unsigned int base_s;
        // (the bitmap atomics of this block completed before the barrier; the
        // scan reads the bitmap with agent-scope loads)
        __syncthreads();
        if (tid == 0) base_s = 0;
        const int64_t ntl = (s.n - m + 1 + hot_rows - 1) / hot_rows;
        const int wpt = hot_rows / 64;
        const uint32_t hot_work = (uint32_t)((s.n - m + 1 + 64 * HOT_FRAC - 1) / (64 * HOT_FRAC));
        for (int64_t t0 = 0; t0 < ntl; t0 += END_BLOCK) {
            __syncthreads();
            const unsigned int base = base_s;
            const int64_t t = t0 + tid;
            bool hot = false;
            if (t < ntl) {
                unsigned long long any = 0ull;
                for (int w2 = 0; w2 < wpt; ++w2) any |= load_word(&s.alive[t * wpt + w2]);
                hot = any != 0ull || s.twork[t] >= hot_work;
                s.twork[t] = 0u;
            }
            const unsigned long long bal = __ballot(hot);
            if (lane == 0) wcnt_s[w] = (unsigned int)__popcll(bal);
            __syncthreads();
            unsigned int before = 0, total = 0;
            for (int q = 0; q < END_BLOCK / 64; ++q) {
                before += (q < w) ? wcnt_s[q] : 0u;
                total += wcnt_s[q];
            }
            const unsigned int pos =
                base + before + (unsigned int)__popcll(bal & ((1ull << lane) - 1ull));
            if (hot && pos < (unsigned int)HOT_MAX) s.hot[pos] = (int32_t)t;
            __syncthreads();
            if (tid == 0) base_s = base + total;
        }
        __syncthreads();
        if (tid == 0) {
            c->nhot = base_s < (unsigned int)HOT_MAX ? base_s : (unsigned int)HOT_MAX;
            c->hot_r = hot_rows;
        }
    }
    // (the other waves read nothing of the control block after the barrier above
    // thread 0's part; one more here would wait for its stores)
    if (more && tid == 0) next_range(s, c, guard, max_attempts, rem);
}

// The heatmap row (Eq. (11)) of a successful round that refined: every range
// discord (the alive bits) with its exact nearest-neighbour correlation, as
// ED^2 / (2m) = 1 - rho; k_advance cleared the row.  (Launched after
// k_round_end: the control block already holds the next range search.)
__global__ void k_heat(SeriesDev* S, int B, const int64_t* __restrict__ pfx)
{
    const int b = series_of(pfx, B, blockIdx.x);
    const SeriesDev& s = S[b];
    const int32_t m = s.ctrl->heat_m;
    if (s.heat == nullptr || m == 0) return;
    const int64_t i = (blockIdx.x - pfx[b]) * (int64_t)ADV_BLOCK + threadIdx.x;
    if (i >= s.n - m + 1) return;
    if (!((s.alive[i >> 6] >> (i & 63)) & 1ull)) return;
    s.heat[(int64_t)(m - s.minL) * s.heat_ld + i] = fmin(2.0, fmax(0.0, 1.0 - dbl_of(s.rho[i])));
}

// ---------------------------------------------------------------------------
// diagnostic: drift of the FP32 selection recurrence from FP64
// ---------------------------------------------------------------------------
// Items of 512-row tiles (the longest recurrence chains any sweep runs) and
// `chunk` columns to their right, spread over the series (tiles evenly,
// columns at varying distance): the centred diagonal recurrence is run in
// FP32 exactly as the selection sweep runs it (FP32 helpers, exact
// boundary values rounded to FP32) and in FP64 (the refinement sweep's
// arithmetic), side by side from the same exact first column.  The largest
// |rho32 - rho64| over the items' non-self pairs (rho = C inv_i inv_j) goes
// to out[0] (ordered bits, atomicMax).
template <int U>
__device__ __forceinline__ void drift_step(float (&C32)[8], double (&C64)[8], const float (&a32)[8],
                                           const float (&b32)[8], const double (&a64)[8],
                                           const double (&b64)[8], const H4<float>& h32,
                                           const H4<double>& h64, const float (&iv32)[8],
                                           const double (&iv64)[8], const int64_t (&ri)[8],
                                           int64_t j, int32_t m, int64_t N, double& mx)
{
    advance<float, 8, U>(C32, a32, b32, h32.df, h32.dg, h32.B);
    advance<double, 8, U>(C64, a64, b64, h64.df, h64.dg, h64.B);
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        if (j - m >= ri[q] && ri[q] < N && j < N) {
            const float r32 = C32[slot_reg<8, U>(q)] * h32.inv * iv32[q];
            const double r64 = C64[slot_reg<8, U>(q)] * h64.inv * iv64[q];
            mx = fmax(mx, fabs((double)r32 - r64));
        }
    }
}

__global__ __launch_bounds__(64) void k_drift(SeriesDev* S, int64_t nitems, int chunk,
                                              unsigned long long* out)
{
    constexpr int Q = 8, R = 64 * Q;
    extern __shared__ double lds[];
    const SeriesDev& s = S[0];
    Ctrl* c = s.ctrl;
    const SweepArgs<float> A32 = args_of<float>(s, c);
    const SweepArgs<double> A64 = args_of<double>(s, c);
    const int32_t m = A64.m;
    const int64_t N = A64.N;
    const int lane = threadIdx.x;
    double* xp = lds;
    double* ws = lds + hk_vp_doubles(m);
    constexpr int NC = batch_cols<double>();  // both precisions in batches of the FP64 width
    H4<double>* hs64 = (H4<double>*)(lds + sweep_hs_offset(m, R, NC));
    H4<float>* hs32 = (H4<float>*)(lds + sweep_hs_offset(m, R, NC) + sweep_hs_doubles(R, 8, NC));
    const int64_t ntiles = (N + R - 1) / R;
    // nitems <= 0: every (tile, chunk) of the right side, chunk-major
    const int64_t nchall = (N + chunk - 1) / chunk;
    const bool all = nitems <= 0;
    const int64_t total = all ? ntiles * nchall : nitems;
    double mx = 0.0;
    for (int64_t it = blockIdx.x; it < total; it += gridDim.x) {
        const int64_t i0 = uniform_i64(all ? (it % ntiles) * R : ((it * ntiles) / nitems) * R);
        const int64_t span = N - (i0 + m);
        if (span <= 0) continue;
        const int64_t nch = std::max<int64_t>(1, span / chunk);
        const int64_t cc = all ? it / ntiles : (it * 37) % nch;
        if (all && cc * chunk >= span) continue;
        const int64_t jbeg = uniform_i64(i0 + m + cc * chunk);
        const int64_t jend = std::min<int64_t>(N, jbeg + 1 + chunk);
        double Sx, Sy, acc[Q];
        item_start<Q>(A64.T, A64.mu, m, i0, jbeg, xp, ws, (double*)hs64, Sx, Sy, acc);
        float C32[Q], a32[Q], b32[Q], iv32[Q];
        double C64[Q], a64[Q], b64[Q], iv64[Q];
        int64_t ri[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int64_t i = i0 + Q * lane + q;
            const bool top = (lane == 0) && (q == 0);
            const int64_t ip = top ? i : i - 1;
            C64[q] = acc[q];
            C32[q] = (float)acc[q];
            a32[q] = top ? 0.0f : A32.df[ip];
            b32[q] = top ? 0.0f : A32.dg[ip];
            a64[q] = top ? 0.0 : A64.df[ip];
            b64[q] = top ? 0.0 : A64.dg[ip];
            iv32[q] = A32.inv[i];
            iv64[q] = A64.inv[i];
            ri[q] = i;
        }
        for (int64_t j = jbeg + 1; j + Q <= jend; ) {
            stage_batch<double, NC>(A64.T, A64.mu, A64.df, A64.dg, A64.inv, m, j, xp, Sx, ws, hs64);
            stage_batch<float, NC>(A32.T, A32.mu, A32.df, A32.dg, A32.inv, m, j, xp, Sx, ws, hs32);
            const int64_t jb_end = std::min<int64_t>(jend, j + NC);
            for (int s0 = 0; j + Q <= jb_end; s0 += Q, j += Q) {
#define DRIFT_STEP(U)                                                                          \
    drift_step<U>(C32, C64, a32, b32, a64, b64, hs32[s0 + (U)], hs64[s0 + (U)], iv32, iv64, ri, \
                  j + (U), m, N, mx);
                DRIFT_STEP(0) DRIFT_STEP(1) DRIFT_STEP(2) DRIFT_STEP(3)
                DRIFT_STEP(4) DRIFT_STEP(5) DRIFT_STEP(6) DRIFT_STEP(7)
#undef DRIFT_STEP
            }
        }
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) mx = fmax(mx, __shfl_xor(mx, o));
    if (lane == 0) atomicMax(out, ord_of(mx));
}

// The guard band the selection sweep uses at the current length (after
// k_guard), as a double in out[1].
__global__ void k_drift_band(SeriesDev* S, float guard, double* out)
{
    out[1] = sel_guard(S[0].ctrl, guard);
}

// ---------------------------------------------------------------------------
// streaming series: exact nearest-neighbour profiles per length, updated by
// the pairs each append adds (the discord definition, Sec. 2.1, applied to a
// series that grows; the top-k of a length are then those of its profile)
// ---------------------------------------------------------------------------
// After an append from n_old to n points, the subsequences of length m that
// start at i >= N_old = n_old - m + 1 are new; each reaches back over at most
// m - 1 points that were already there (the halo).  The pairs the append
// adds are (new row, any column) and (old row, new column):
//   part A  the row tiles from the one holding N_old sweep every column,
//           both sides (left-side and right-side chunks alternate, nearest
//           first);
//   part B  the row tiles holding old rows sweep the new columns (right
//           side only: every new column is to the right of every old row).
// Rows of part A's first tile below N_old are swept again in full, which
// only re-derives their maxima.  The refinement sweep does the work with
// pruning off; every row's running maximum of rho stays in its length's
// profile (ordered bits, prof[(m - minL) Npad + i]).
//
// One length of a series of tens of thousands of points does not fill the
// machine (30,000 points: 3,500 items of 128 rows and 1,024 columns), and a
// kernel per length and step costs as much as its work, so `lanes` lengths go
// together: the batch holds one descriptor per lane, which share the series,
// lane b at length m0 + b.  (30,000 points, 33 lengths, three appends and
// queries: a length at a time 36 ms, nine 10.9.  The profile update takes 175
// us per length alone and 93 of nine, of which its FP64 operations, four per
// pair and side, are 31.)

// The lanes' lengths m0, m0 + 1, ... up to maxL (one block).
__global__ void k_stream_group(SeriesDev* S, int lanes, int32_t m0, int32_t maxL)
{
    const int b = threadIdx.x;
    if (b >= lanes) return;
    const SeriesDev& s = S[b];
    Ctrl* c = s.ctrl;
    const double eps = S[0].ctrl->flat_eps;
    c->m = m0 + b;
    c->li = c->m - s.minL;
    c->active = c->m <= maxL ? 1 : 0;
    c->flat_eps = eps;
    c->flat_min = 0x7fffffffffffffffll;
    c->flat_max = -1;
    // a round without pruning whose candidates k_stream_pick chooses
    c->mode = 3;
    c->r = 0.0;
    c->prune = 0;
    c->thr64 = c->thr_sel = 2.0;
    c->thr32 = 2.0f;
    c->exact_ref = 0;
    c->band_over = 0;
    c->live_ref = 0xffffffffu;  // not a direct round
    c->nlive = 0xffffffffu;
    c->handled = 1;
    c->nsurv = c->ncand = 0;
    c->done = 0;
    for (int g = 0; g < CAND_GROUPS; ++g) c->pcnt[g] = 0;
}

// Statistics and helpers of the lanes' lengths, as k_length computes them one
// length at a time: a thread carries window i and its right neighbour through
// the lengths.  The group before left its last length's mean and variance
// with the last lane (`lanes` is odd, so that its two buffers alternate).
__global__ __launch_bounds__(256) void k_stream_stats(SeriesDev* S, int lanes, int32_t m0,
                                                      int32_t maxL)
{
    const SeriesDev& s = S[0];
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    const double* __restrict__ T = s.T;
    const double feps = s.ctrl->flat_eps;
    double mean0 = 0.0, v0 = 0.0, mean1 = 0.0, v1 = 0.0;
    if (m0 > s.minL && i < s.n - m0 + 2) {  // (length m0 - 1)
        const SeriesDev& p = S[lanes - 1];
        const bool odd = ((m0 - 1 - s.minL) & 1) != 0;
        const double* mu_o = odd ? p.mu2 : p.mu;
        const double* var_o = odd ? p.var2 : p.var;
        mean0 = mu_o[i];
        v0 = var_o[i];
        if (i + 1 < s.n - m0 + 2) {
            mean1 = mu_o[i + 1];
            v1 = var_o[i + 1];
        }
    }
    for (int b = 0; b < lanes && m0 + b <= maxL; ++b) {
        const SeriesDev& sb = S[b];
        Ctrl* c = sb.ctrl;
        const int32_t m = m0 + b;
        const int64_t N = s.n - m + 1;
        if (i < sb.Npad + 64) {
            double a0 = 0.0, q0 = 0.0, a1 = 0.0, q1 = 0.0;
            if (i < N) {
                if (m == s.minL) {
                    direct_stats(T, i, m, a0, q0);
                    if (i + 1 < N) direct_stats(T, i + 1, m, a1, q1);
                } else {
                    const GrowBy g = grow_by(m);
                    grow_stats(T[i + m - 1], g, mean0, v0, a0, q0);
                    if (i + 1 < N) grow_stats(T[i + m], g, mean1, v1, a1, q1);
                }
            }
            mean0 = a0;
            v0 = q0;
            mean1 = a1;
            v1 = q1;
            const bool odd = ((m - s.minL) & 1) != 0;
            (odd ? sb.mu2 : sb.mu)[i] = mean0;
            if (b == lanes - 1) (odd ? sb.var2 : sb.var)[i] = v0;
            double df = 0.0, dg = 0.0, inv = 0.0;
            if (i < N - 1) {
                const double a = T[i + m], e = T[i];
                df = (a - e) * 0.5;
                dg = (a - mean1) + (e - mean0);
            }
            if (i < N) {
                const double sg = sqrt(v0);
                if (sg <= feps) {
                    atomicMin((long long*)&c->flat_min, (long long)i);
                    atomicMax((long long*)&c->flat_max, (long long)i);
                } else {
                    inv = 1.0 / (sqrt((double)m) * sg);
                }
            }
            sb.df64[i] = df;
            sb.dg64[i] = dg;
            sb.inv64[i] = inv;
        }
        if (i < sb.nwords) {
            const int64_t lo = i * 64;
            sb.alive[i] = lo + 64 <= N ? ~0ull : lo < N ? (1ull << (N - lo)) - 1ull : 0ull;
        }
    }
}

template <int Q>
__global__ __launch_bounds__(64, (Q <= 4 ? 3 : 1)) void k_stream_band(SeriesDev* S, int lanes,
                                                                      unsigned long long* prof,
                                                                      int64_t n_old, int chunk)
{
    extern __shared__ double lds[];
    constexpr int R = 64 * Q;
    unsigned long long cum = 0;  // items dealt out as in k_select_far
    for (int b = 0; b < lanes; ++b) {
        const SeriesDev& s = S[b];
        Ctrl* c = s.ctrl;
        if (!c->active) continue;
        SweepArgs<double> A = args_of<double>(s, c);
        A.rho = prof + (int64_t)c->li * s.Npad;
        const int32_t m = A.m;
        const int64_t N = A.N;
        const int64_t Nold = std::max<int64_t>(0, n_old - m + 1);
        if (Nold >= N) continue;
        const int64_t a0 = (Nold / R) * R;
        const int64_t tA = (N - a0 + R - 1) / R;
        const int64_t cA = (N + chunk - 1) / chunk;
        const int64_t itemsA = tA * 2 * cA;
        const int64_t tB = (Nold + R - 1) / R;
        const int64_t cB = (N - Nold + chunk - 1) / chunk;
        const int64_t total = itemsA + tB * cB;
        unsigned long long ev = 0;
        const int64_t first = (int64_t)first_item(cum);
        cum += (unsigned long long)total;
        for (int64_t it = first; it < total; it += gridDim.x) {
            int64_t i0, jbeg, jend;
            bool left;
            if (it < itemsA) {
                const int64_t t = it % tA, r = it / tA;
                const int64_t cc = r >> 1;
                left = (r & 1) != 0;
                i0 = a0 + t * R;
                if (left) {
                    jend = std::min<int64_t>(N, i0 + R - m) - cc * chunk;
                    jbeg = std::max<int64_t>(0, jend - chunk);
                } else {
                    jbeg = i0 + m + cc * chunk;
                    jend = std::min<int64_t>(N, jbeg + chunk);
                }
            } else {
                const int64_t x = it - itemsA;
                const int64_t t = x % tB, cc = x / tB;
                i0 = t * R;
                left = false;
                jbeg = std::max<int64_t>(Nold, i0 + m) + cc * chunk;
                jend = std::min<int64_t>(N, jbeg + chunk);
            }
            if (jbeg >= jend) continue;
            ref_item<Q, HK_TILE>(A, i0, jbeg, jend, left, 2.0, 0, lds, ev);
        }
        if (threadIdx.x == 0 && ev)
            atomicAdd(&s.evc[EV_REF * EV_SLOTS + (blockIdx.x & (EV_SLOTS - 1))], ev);
    }
}

// A query's candidates at every lane's length (a block each): the k + KP_EXTRA
// rows of the smallest profile values, ties to the smaller index.  Each lane
// of a wave holds its own smallest row, so a round of the wave's minimum costs
// only the winner a rescan of its N / 1024 rows (a thread per bitmap word and
// a rescan by every lane: 121 us at 30,000 points); wave 0 merges the waves'
// lists.  The exact pass and k_round_end then write the length's rows, as in a
// round without pruning.
__global__ __launch_bounds__(TOPK_BLOCK) void k_stream_pick(SeriesDev* S,
                                                            const unsigned long long* __restrict__ prof)
{
    constexpr int NW = TOPK_BLOCK / 64;
    __shared__ unsigned long long pu[NW * KP_MAX];
    __shared__ long long pi[NW * KP_MAX];
    const SeriesDev& s = S[blockIdx.x];
    Ctrl* c = s.ctrl;
    if (!c->active) return;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int64_t N = s.n - c->m + 1;
    const unsigned long long* __restrict__ p = prof + (int64_t)c->li * s.Npad;
    const int kp = (int)std::min<int64_t>(N, s.k + KP_EXTRA);
    // the smallest row of [tid, N) in steps of the block past `last`
    auto next_of = [&](const Key& last) {
        constexpr int U = 8;
        Key best = {~0ull, KEY_NONE};
        for (int64_t i0 = tid; i0 < N; i0 += U * TOPK_BLOCK) {
            unsigned long long v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t i = i0 + (int64_t)u * TOPK_BLOCK;
                v[u] = i < N ? p[i] : ~0ull;
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t i = i0 + (int64_t)u * TOPK_BLOCK;
                const Key x = {v[u], i};
                if (i < N && key_less(last, x) && key_less(x, best)) best = x;
            }
        }
        return best;
    };
    Key mine = next_of(Key{0ull, -1});
    for (int r = 0; r < kp; ++r) {
        const Key v = wave_min_key(mine);
        if (lane == 0) {
            pu[w * KP_MAX + r] = v.u;
            pi[w * KP_MAX + r] = v.i;
        }
        if (mine.i == v.i && v.i != KEY_NONE && r + 1 < kp) mine = next_of(v);
    }
    __syncthreads();
    if (w != 0) return;
    Key last = {0ull, -1};
    for (int r = 0; r < kp; ++r) {
        Key best = {~0ull, KEY_NONE};
        for (int e = lane; e < NW * kp; e += 64) {
            const int ww = e / kp, at = ww * KP_MAX + (e - ww * kp);
            const Key x = {pu[at], pi[at]};
            if (x.i != KEY_NONE && key_less(last, x) && key_less(x, best)) best = x;
        }
        best = wave_min_key(best);
        if (lane == 0) s.cand[r] = best.i;
        last = best;
    }
    if (lane == 0) {
        c->nsurv = (uint32_t)N;
        c->ncand = (uint32_t)kp;
    }
}

// The exact profile of the current length as distances (Eq. (6)):
// nn[i] = sqrt(2m (1 - rho_i)) for i < N.
__global__ void k_stream_profile(SeriesDev* S, const unsigned long long* __restrict__ prof,
                                 double* nn)
{
    const SeriesDev& s = S[0];
    const Ctrl* c = s.ctrl;
    const int32_t m = c->m;
    const int64_t N = s.n - m + 1;
    const unsigned long long* p = prof + (int64_t)c->li * s.Npad;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < N;
         i += (int64_t)gridDim.x * blockDim.x) {
        const double rh = dbl_of(p[i]);
        nn[i] = sqrt(fmin(4.0 * (double)m, fmax(0.0, 2.0 * (double)m * (1.0 - rh))));
    }
}

__global__ void k_fill_u64(unsigned long long* p, int64_t count, unsigned long long v)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
template <typename F, int Q, bool WIT>
static void launch_near(const Batch& bt, const SweepCfg& cfg, const int64_t* total, hipStream_t st)
{
    const size_t lds = sizeof(double) * sweep_lds_doubles(bt.maxL_all, 64 * Q, (int)sizeof(F), false);
    if (total[PFX_NEAR] == 0) return;
    cfg.timer->begin(0, st);
    hipLaunchKernelGGL((k_select_near<F, Q, WIT ? WIT_INLINE : WIT_OFF>), dim3((unsigned int)total[PFX_NEAR]), dim3(64), lds,
                       st, bt.s, bt.B, bt.pfx[PFX_NEAR], cfg.near_cols, cfg.near_chunk);
    cfg.timer->end(0, st);
}

template <typename F, int Q, bool WIT>
static void launch_far(const Batch& bt, const SweepCfg& cfg, const int64_t* total, hipStream_t st)
{
    const size_t lds = sizeof(double) * sweep_lds_doubles(bt.maxL_all, 64 * Q, (int)sizeof(F), false);
    hipLaunchKernelGGL(k_tiles, dim3((unsigned int)total[PFX_TSEL]), dim3(TILES_BLOCK), 0, st, bt.s, bt.B,
                       bt.pfx[PFX_TSEL], 64 * Q, 0, cfg.near_cols, cfg.chunk_cols, 64 * cfg.q_near);
    cfg.timer->begin(1, st);
    hipLaunchKernelGGL((k_select_far<F, Q, WIT ? WIT_REPLAY : WIT_OFF>), dim3(cfg.far_grid), dim3(64), lds, st, bt.s, bt.B,
                       cfg.near_cols, cfg.chunk_cols, 64 * cfg.q_near);
    cfg.timer->end(1, st);
}

template <int Q, bool WIT>
static void launch_refine(const Batch& bt, const SweepCfg& cfg, const int64_t* total, hipStream_t st)
{
    hipLaunchKernelGGL(k_tiles, dim3((unsigned int)total[PFX_TREF]), dim3(TILES_BLOCK), 0, st, bt.s, bt.B,
                       bt.pfx[PFX_TREF], 64 * Q, 1, 0, cfg.chunk_cols, 64 * cfg.q_near);
    const size_t lds = sizeof(double) * sweep_lds_doubles(bt.maxL_all, 64 * Q, (int)sizeof(double), true);
    cfg.timer->begin(2, st);
    hipLaunchKernelGGL((k_refine<Q, WIT>), dim3(cfg.far_grid), dim3(64), lds, st, bt.s, bt.B,
                       cfg.chunk_cols);
    cfg.timer->end(2, st);
}

template <typename F, bool WIT>
static void launch_select(const Batch& bt, const SweepCfg& cfg, const int64_t* total,
                          hipStream_t st)
{
    if (cfg.band && total[PFX_BAND] > 0) {
        cfg.timer->begin(5, st);
        hipLaunchKernelGGL((k_select_band<F>), dim3((unsigned int)total[PFX_BAND]), dim3(64),
                           band_lds_bytes(bt.maxL_all, (int)sizeof(F)), st, bt.s, bt.B, bt.pfx[PFX_BAND],
                           WIT ? 1 : 0);
        cfg.timer->end(5, st);
    }
    switch (cfg.q_near) {
    case 2: launch_near<F, 2, WIT>(bt, cfg, total, st); break;
    case 4: launch_near<F, 4, WIT>(bt, cfg, total, st); break;
    default: launch_near<F, 8, WIT>(bt, cfg, total, st); break;
    }
    if ((int64_t)cfg.near_cols >= bt.Nmax_all) {
        // the first pass already covers every column of every series
        return;
    }
    switch (cfg.q_far) {
    case 2: launch_far<F, 2, WIT>(bt, cfg, total, st); break;
    case 4: launch_far<F, 4, WIT>(bt, cfg, total, st); break;
    default: launch_far<F, 8, WIT>(bt, cfg, total, st); break;
    }
}

template <bool WIT>
static void launch_refine_q(const Batch& bt, const SweepCfg& cfg, const int64_t* total, hipStream_t st)
{
    switch (cfg.q_ref) {
    case 4: launch_refine<4, WIT>(bt, cfg, total, st); break;
    case 8: launch_refine<8, WIT>(bt, cfg, total, st); break;
    default: launch_refine<2, WIT>(bt, cfg, total, st); break;
    }
}

// The exact pass over the rounds' candidates.  Up to SCREEN_MIN subsequences
// a launch of the screening costs more than the blocks it saves.
static void launch_exact(const Batch& bt, int full, hipStream_t st)
{
    if (bt.B > 1)
        hipLaunchKernelGGL(k_items, dim3(1), dim3(ITEMS_BLOCK), 0, st, bt.s, bt.B, bt.large, full, bt.ipfx,
                           bt.ipfx + bt.B + 1);
    const bool screened = bt.Nmax_all > SCREEN_MIN;
    if (screened) {
        const size_t wins = sizeof(_Float16) * (size_t)PM_G * SC_GS *
                            (size_t)dense_stride(std::min<int32_t>(bt.maxL_all, PM_KC));
        hipLaunchKernelGGL(k_screen, dim3(SCREEN_GRID), dim3(64 * SC_WAVES), wins, st, bt.s, bt.B, bt.large,
                           full, bt.ipfx);
        if (bt.maxL_all > PM_KC)
            hipLaunchKernelGGL(k_screen_long, dim3(SCREEN_GRID), dim3(64 * SC_WAVES), 0, st, bt.s, bt.B,
                               bt.large, full, bt.ipfx);
    }
    const size_t lds = sizeof(double) * (size_t)(PM_G * PM_XS + EX_COLS + bt.maxL_all + 4 * EX_STEPS);
    hipLaunchKernelGGL(k_exact, dim3(exact_grid(bt.large)), dim3(64 * EX_WAVES), lds, st, bt.s, bt.B,
                       bt.large, full, screened ? 1 : 0, SCREEN_GRID, bt.ipfx,
                       bt.ipfx + bt.B + 1);
}

hipError_t launch_start(const Batch& bt, const SweepCfg& cfg, hipStream_t st)
{
    hipLaunchKernelGGL(k_start, dim3(1), dim3(256), 0, st, bt.s, bt.B, cfg.guard, cfg.max_attempts,
                       bt.remaining);
    return hipGetLastError();
}

// One round: every series with work does one range search at its current
// length (a fixed launch sequence; all parameters come from the device).
// Without `full` the sweeps are left out: a series that needs them waits for
// the next full round.  more = 0: a bare range search.  wit: the sweeps keep
// the witnesses of what they prune.
hipError_t launch_round(const Batch& bt, const SweepCfg& cfg, const int64_t* total, bool full,
                        bool dense, bool more, bool wit, hipStream_t st)
{
    const unsigned int elem = (unsigned int)total[PFX_ELEM];
    cfg.timer->begin(4, st);
    hipLaunchKernelGGL(k_advance, dim3(elem), dim3(ADV_BLOCK),
                       sizeof(double) * (size_t)(ADV_BLOCK + bt.maxL_all), st, bt.s, bt.B,
                       bt.pfx[PFX_ELEM], bt.remaining);
    if (more) {
        const bool shared = bt.B > 1 && bt.B <= FAIL_ITEMS_MAXB;
        if (shared)
            hipLaunchKernelGGL(k_fail_items, dim3(1), dim3(FAIL_ITEMS_MAXB), 0, st, bt.s, bt.B,
                               (int64_t)RESCUE_GRID * (RESCUE_BLOCK / 64), bt.ipfx);
        hipLaunchKernelGGL(k_rescue, dim3(RESCUE_GRID), dim3(RESCUE_BLOCK), 0, st, bt.s, bt.B,
                           shared ? bt.ipfx : nullptr);
    }
    if (full)
        hipLaunchKernelGGL(k_helpers, dim3(elem), dim3(ADV_BLOCK), 0, st, bt.s, bt.B,
                           bt.pfx[PFX_ELEM]);
    cfg.timer->end(4, st);
    if (full) {
        hipLaunchKernelGGL(k_guard, dim3(bt.B), dim3(GUARD_BLOCK), 0, st, bt.s, cfg.guard);
        if (wit) {
            if (cfg.dist_bits == 64) launch_select<double, true>(bt, cfg, total, st);
            else launch_select<float, true>(bt, cfg, total, st);
            launch_refine_q<true>(bt, cfg, total, st);
        } else {
            // (the table of selection tiles is built for the lower tiles, which are more)
            SweepCfg tall = cfg;
            if (more && cfg.far_open && bt.Nmax_all >= FAR_TALL_MIN) tall.q_far = 8;
            if (cfg.dist_bits == 64) launch_select<double, false>(bt, cfg, total, st);
            else launch_select<float, false>(bt, tall, total, st);
            launch_refine_q<false>(bt, cfg, total, st);
        }
        hipLaunchKernelGGL(k_select_top, dim3(bt.B), dim3(TOPK_BLOCK), 0, st, bt.s);
    }
    cfg.timer->begin(3, st);
    if (dense) {
        hipLaunchKernelGGL(k_dense_list, dim3(bt.B), dim3(TOPK_BLOCK), 0, st, bt.s, full ? 1 : 0);
        if (bt.B > 1)
            hipLaunchKernelGGL(k_dense_items, dim3(1), dim3(ITEMS_BLOCK), 0, st, bt.s, bt.B, bt.ipfx);
        hipLaunchKernelGGL(k_dense, dim3(DENSE_GRID), dim3(64 * SC_WAVES),
                           sizeof(_Float16) * DN_ROWS * dense_stride(std::min(bt.maxL_all, DENSE_MAXM)),
                           st, bt.s, bt.B, bt.ipfx);
        hipLaunchKernelGGL(k_pairs, dim3(RESCUE_GRID), dim3(RESCUE_BLOCK), 0, st, bt.s, bt.B,
                           bt.ipfx);
        hipLaunchKernelGGL(k_dense_top, dim3(bt.B), dim3(TOPK_BLOCK), 0, st, bt.s);
    }
    launch_exact(bt, full ? 1 : 0, st);
    cfg.timer->end(3, st);
    hipLaunchKernelGGL(k_round_end, dim3(bt.B), dim3(END_BLOCK), 0, st, bt.s, bt.remaining,
                       64 * cfg.q_near, full ? 1 : 0, more ? 1 : 0, cfg.guard, cfg.max_attempts, bt.B,
                       bt.large, bt.ipfx + bt.B + 1);
    if (full && bt.heat)
        hipLaunchKernelGGL(k_heat, dim3(elem), dim3(ADV_BLOCK), 0, st, bt.s, bt.B, bt.pfx[PFX_ELEM]);
    return hipGetLastError();
}

__global__ void k_set_len(SeriesDev* S, int32_t m, int32_t new_len);

hipError_t launch_drift(const Batch& bt, const int64_t* total, int32_t minL, int32_t m,
                        int64_t nitems, int chunk, float guard, double* out, hipStream_t st)
{
    const hipError_t e = launch_stats_to(bt, minL, m, total, st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_guard, dim3(1), dim3(GUARD_BLOCK), 0, st, bt.s, guard);
    hipLaunchKernelGGL(k_fill_u64, dim3(1), dim3(64), 0, st, (unsigned long long*)out, (int64_t)1,
                       0ull);
    constexpr int NC = batch_cols<double>();
    const size_t lds = sizeof(double) * (sweep_hs_offset(bt.maxL_all, 512, NC) + sweep_hs_doubles(512, 8, NC) +
                                         sweep_hs_doubles(0, 4, NC));
    hipLaunchKernelGGL(k_drift, dim3(1024), dim3(64), lds, st, bt.s, nitems, chunk,
                       (unsigned long long*)out);
    hipLaunchKernelGGL(k_drift_band, dim3(1), dim3(1), 0, st, bt.s, guard, out);
    return hipGetLastError();
}

// Streaming: one append's profile updates at every length (statistics,
// helpers, band sweeps), a query's top-k rows at every length, the profile
// of one length, and the reset of every profile.
static void launch_stream_group(const Batch& bt, const int64_t* total, int32_t m0, int32_t maxL,
                                hipStream_t st)
{
    hipLaunchKernelGGL(k_stream_group, dim3(1), dim3(64), 0, st, bt.s, bt.B, m0, maxL);
    hipLaunchKernelGGL(k_stream_stats, dim3((unsigned int)(total[PFX_ELEM] / bt.B)), dim3(256), 0, st,
                       bt.s, bt.B, m0, maxL);
}

template <int Q>
static void launch_band(const Batch& bt, unsigned long long* prof, int64_t n_old, int chunk,
                        hipStream_t st)
{
    const size_t lds = sizeof(double) * sweep_lds_doubles(bt.maxL_all, 64 * Q, (int)sizeof(double), true, HK_TILE);
    hipLaunchKernelGGL((k_stream_band<Q>), dim3(STREAM_GRID), dim3(64), lds, st, bt.s, bt.B, prof, n_old,
                       chunk);
}

hipError_t launch_stream_update(const Batch& bt, const SweepCfg& cfg, const int64_t* total,
                                int32_t minL, int32_t maxL, unsigned long long* prof,
                                int64_t n_old, int64_t n, hipStream_t st)
{
    // shorter chunks until the items fill the machine (an item is a serial
    // chain of its columns)
    const int64_t R = 64 * (int64_t)cfg.q_ref, N = n - minL + 1;
    const int64_t tiles = (n - n_old + R - 1) / R, old = (n_old + R - 1) / R;
    int chunk = STREAM_CHUNK;
    while (chunk > HK_TILE &&
           bt.B * (tiles * ((N + chunk - 1) / chunk) + old * ((n - n_old + chunk - 1) / chunk)) <
               STREAM_ITEMS)
        chunk /= 2;
    for (int32_t m = minL; m <= maxL; m += bt.B) {
        launch_stream_group(bt, total, m, maxL, st);
        switch (cfg.q_ref) {
        case 4: launch_band<4>(bt, prof, n_old, chunk, st); break;
        case 8: launch_band<8>(bt, prof, n_old, chunk, st); break;
        default: launch_band<2>(bt, prof, n_old, chunk, st); break;
        }
    }
    return hipGetLastError();
}

hipError_t launch_stream_query(const Batch& bt, const SweepCfg& cfg, const int64_t* total,
                               int32_t minL, int32_t maxL, const unsigned long long* prof,
                               hipStream_t st)
{
    for (int32_t m = minL; m <= maxL; m += bt.B) {
        launch_stream_group(bt, total, m, maxL, st);
        hipLaunchKernelGGL(k_stream_pick, dim3(bt.B), dim3(TOPK_BLOCK), 0, st, bt.s, prof);
        launch_exact(bt, 0, st);
        hipLaunchKernelGGL(k_round_end, dim3(bt.B), dim3(END_BLOCK), 0, st, bt.s, bt.remaining,
                           64 * cfg.q_near, 0, 0, 0.0f, 0, bt.B, bt.large, bt.ipfx + bt.B + 1);
    }
    return hipGetLastError();
}

hipError_t launch_stream_profile(const Batch& bt, int32_t m, const unsigned long long* prof,
                                 double* nn, hipStream_t st)
{
    hipLaunchKernelGGL(k_set_len, dim3(1), dim3(1), 0, st, bt.s, m, 0);
    hipLaunchKernelGGL(k_stream_profile, dim3(256), dim3(256), 0, st, bt.s, prof, nn);
    return hipGetLastError();
}

hipError_t launch_fill_u64(unsigned long long* p, int64_t count, unsigned long long v, hipStream_t st)
{
    hipLaunchKernelGGL(k_fill_u64, dim3(1024), dim3(256), 0, st, p, count, v);
    return hipGetLastError();
}

__global__ void k_set_fixed_r(SeriesDev* S, double r)
{
    Ctrl* c = S[0].ctrl;
    c->mode = 3;
    c->r = r;
}

hipError_t launch_set_fixed_r(const Batch& bt, double r, hipStream_t st)
{
    hipLaunchKernelGGL(k_set_fixed_r, dim3(1), dim3(1), 0, st, bt.s, r);
    return hipGetLastError();
}

__global__ void k_set_len(SeriesDev* S, int32_t m, int32_t new_len)
{
    const SeriesDev& s = S[0];
    Ctrl* c = s.ctrl;
    c->m = m;
    c->li = m - s.minL;
    c->new_len = new_len;
    c->active = 1;
    c->nlive = 0x7fffffffu;
    if (new_len) {
        c->flat_min = 0x7fffffffffffffffll;
        c->flat_max = -1;
    }
}

hipError_t launch_set_len(const Batch& bt, int32_t m, hipStream_t st)
{
    hipLaunchKernelGGL(k_set_len, dim3(1), dim3(1), 0, st, bt.s, m, 0);
    return hipGetLastError();
}

// Statistics of S[0] at lengths minL..m only (no search).
hipError_t launch_stats_to(const Batch& bt, int32_t minL, int32_t m, const int64_t* total,
                           hipStream_t st)
{
    for (int32_t mm = minL; mm <= m; ++mm) {
        hipLaunchKernelGGL(k_set_len, dim3(1), dim3(1), 0, st, bt.s, mm, mm == minL ? 2 : 1);
        hipLaunchKernelGGL(k_length, dim3((unsigned int)total[PFX_ELEM]), dim3(256), 0, st, bt.s, 1,
                           bt.pfx[PFX_ELEM]);
    }
    return hipGetLastError();
}

// Sum of the per-series counters of a call (one block, a wave per series):
// out = {evals_sel, evals_ref, evals_pol, rounds, survivors, evals_near, evals_far,
//        rows_near, rows_far, evals_band}.
__global__ __launch_bounds__(1024) void k_sum_stats(SeriesDev* S, int B, unsigned long long* out)
{
    static_assert(EV_SLOTS == 64, "one slot per lane");
    __shared__ unsigned long long acc[10];
    if (threadIdx.x < 10) acc[threadIdx.x] = 0ull;
    __syncthreads();
    const int lane = threadIdx.x & 63;
    for (int b = threadIdx.x >> 6; b < B; b += 16) {
        const SeriesDev& s = S[b];
        unsigned long long v[EV_CLASSES];
#pragma unroll
        for (int e = 0; e < EV_CLASSES; ++e) v[e] = s.evc[e * EV_SLOTS + lane];
#pragma unroll
        for (int e = 0; e < EV_CLASSES; ++e)
#pragma unroll
            for (int o = 32; o >= 1; o >>= 1) v[e] += __shfl_xor(v[e], o);
        if (lane == 0) {
            const Ctrl* c = s.ctrl;
            atomicAdd(&acc[0], v[EV_NEAR] + v[EV_FAR] + v[EV_BAND] + v[EV_DENSE]);
            atomicAdd(&acc[1], v[EV_REF]);
            atomicAdd(&acc[2], v[EV_POL]);
            atomicAdd(&acc[3], c->rounds);
            atomicAdd(&acc[4], c->survivors);
            atomicAdd(&acc[5], v[EV_NEAR]);
            atomicAdd(&acc[6], v[EV_FAR]);
            atomicAdd(&acc[7], c->rows_near);
            atomicAdd(&acc[8], c->rows_far);
            atomicAdd(&acc[9], v[EV_BAND]);
        }
    }
    __syncthreads();
    if (threadIdx.x < 10) out[threadIdx.x] = acc[threadIdx.x];
}

hipError_t launch_sum_stats(const Batch& bt, unsigned long long* out, hipStream_t st)
{
    hipLaunchKernelGGL(k_sum_stats, dim3(1), dim3(1024), 0, st, bt.s, bt.B, out);
    return hipGetLastError();
}

__global__ void k_range_out(SeriesDev* S, int64_t N, unsigned long long* alive_out, double* nn_out)
{
    const SeriesDev& s = S[0];
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N || !s.ctrl->started) return;
    const int32_t m = s.ctrl->m;
    const bool on = (s.alive[i >> 6] >> (i & 63)) & 1ull;
    if ((i & 63) == 0) alive_out[i >> 6] = s.alive[i >> 6];
    double d = 0.0;
    if (on) {
        const double r = dbl_of(s.rho[i]);
        d = sqrt(fmin(4.0 * (double)m, fmax(0.0, 2.0 * (double)m * (1.0 - r))));
    }
    nn_out[i] = d;
}

hipError_t launch_range_out(const Batch& bt, int64_t N, unsigned long long* alive_out,
                            double* nn_out, hipStream_t st)
{
    hipLaunchKernelGGL(k_range_out, dim3((unsigned int)((N + 255) / 256)), dim3(256), 0, st, bt.s,
                       N, alive_out, nn_out);
    return hipGetLastError();
}

// Statistics of every window at length m by the recurrences from minL on: one
// thread walks its window through all the lengths in registers, the series'
// stretch and the lengths' constants in LDS.  (A launch per length, which
// wrote every helper of a search as well, moved 100 bytes per window and
// length: 1.66 ms at 10^6 points, m = 128 -> 192.)  Nothing is written when
// the series holds NaN or Inf (*bad).
constexpr int STATS_LENGTHS = 256;  // constants staged at a time
__global__ __launch_bounds__(ADV_BLOCK) void k_window_stats(const double* __restrict__ T, int64_t n,
                                                            int32_t minL, int32_t m,
                                                            const int32_t* bad, double* mu,
                                                            double* sigma)
{
    extern __shared__ double ts[];  // ADV_BLOCK + m values
    __shared__ double rm[STATS_LENGTHS], fm[STATS_LENGTHS];
    if (*bad) return;
    const int64_t i0 = (int64_t)blockIdx.x * ADV_BLOCK;
    const int tid = threadIdx.x;
    const int e = (int)std::min<int64_t>(n - i0, ADV_BLOCK + m);
    for (int t = tid; t < e; t += ADV_BLOCK) ts[t] = T[i0 + t];
    __syncthreads();
    const bool in = i0 + tid < n - m + 1;
    double mean = 0.0, var = 0.0;
    if (in) direct_stats(ts, tid, minL, mean, var);
    for (int32_t l0 = minL + 1; l0 <= m; l0 += STATS_LENGTHS) {
        const int cnt = std::min(STATS_LENGTHS, m - l0 + 1);
        __syncthreads();
        for (int q = tid; q < cnt; q += ADV_BLOCK) {
            const GrowBy g = grow_by(l0 + q);
            rm[q] = g.rm;
            fm[q] = g.fm;
        }
        __syncthreads();
        if (in)
            for (int q = 0; q < cnt; ++q) {
                const GrowBy g = {(double)(l0 + q), rm[q], fm[q]};
                grow_stats(ts[tid + l0 + q - 1], g, mean, var, mean, var);
            }
    }
    if (in) {
        mu[i0 + tid] = mean;
        sigma[i0 + tid] = sqrt(var);
    }
}

hipError_t launch_window_stats(const double* T, int64_t n, int32_t minL, int32_t m,
                               const int32_t* bad, double* mu, double* sigma, hipStream_t st)
{
    hipLaunchKernelGGL(k_window_stats, dim3((unsigned int)((n - m + 1 + ADV_BLOCK - 1) / ADV_BLOCK)),
                       dim3(ADV_BLOCK), sizeof(double) * (size_t)(ADV_BLOCK + m), st, T, n, minL, m, bad,
                       mu, sigma);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// per-series workspace layout and work geometry
// ---------------------------------------------------------------------------
// ---------------------------------------------------------------------------
// discord interest (Eq. (12)): per heatmap column the largest value over the
// lengths (ties: the shorter length), then the k columns with the largest
// values (ties: the smaller index)
// ---------------------------------------------------------------------------
__global__ void k_interest_cols(const double* __restrict__ heat, int32_t L, int64_t ld,
                                int64_t ncols, int32_t minL, double* score, int32_t* blen)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= ncols) return;
    // eight rows' loads are issued before they are compared
    double best = -1.0;
    int32_t bm = 0;
    for (int32_t l0 = 0; l0 < L; l0 += 8) {
        double v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = l0 + u < L ? heat[(int64_t)(l0 + u) * ld + i] : -1.0;
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (v[u] > best) {
                best = v[u];
                bm = l0 + u;
            }
    }
    score[i] = best;
    blen[i] = minL + bm;
}

constexpr int INTEREST_BLOCK = 1024;
__global__ __launch_bounds__(INTEREST_BLOCK) void k_interest_top(const double* __restrict__ score,
                                                                const int32_t* __restrict__ blen,
                                                                int64_t ncols, int32_t k,
                                                                int64_t* top_idx, int32_t* top_len,
                                                                double* top_score)
{
    __shared__ double bv_s[INTEREST_BLOCK / 64];
    __shared__ long long bi_s[INTEREST_BLOCK / 64];
    __shared__ double lastv_s;
    __shared__ long long lasti_s;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    // order: larger score first, then smaller index; round r takes the best
    // column strictly after round r - 1's in that order
    for (int r = 0; r < k; ++r) {
        const double lv = r ? lastv_s : 0.0;
        const long long li = r ? lasti_s : -1;
        double bv = -1.0;
        long long bi = -1;
        for (int64_t i0 = tid; i0 < ncols; i0 += 16 * INTEREST_BLOCK) {
            double vs[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                const int64_t i = i0 + (int64_t)u * INTEREST_BLOCK;
                vs[u] = i < ncols ? score[i] : -1.0;
            }
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                const int64_t i = i0 + (int64_t)u * INTEREST_BLOCK;
                const double v = vs[u];
                const bool after = r == 0 || v < lv || (v == lv && i > li);
                if (i < ncols && after && (v > bv || (v == bv && (bi < 0 || i < bi)))) {
                    bv = v;
                    bi = i;
                }
            }
        }
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) {
            const double v = __shfl_xor(bv, o);
            const long long j = __shfl_xor(bi, o);
            if (j >= 0 && (bi < 0 || v > bv || (v == bv && j < bi))) {
                bv = v;
                bi = j;
            }
        }
        if (lane == 0) {
            bv_s[w] = bv;
            bi_s[w] = bi;
        }
        __syncthreads();
        if (tid == 0) {
            double v = bv_s[0];
            long long j = bi_s[0];
            for (int q = 1; q < INTEREST_BLOCK / 64; ++q)
                if (bi_s[q] >= 0 && (j < 0 || bv_s[q] > v || (bv_s[q] == v && bi_s[q] < j))) {
                    v = bv_s[q];
                    j = bi_s[q];
                }
            top_idx[r] = j;
            top_len[r] = j >= 0 ? blen[j] : 0;
            top_score[r] = j >= 0 ? v : 0.0;
            lastv_s = v;
            lasti_s = j;
        }
        __syncthreads();
    }
}

hipError_t launch_interest(const double* heat, int32_t L, int64_t ld, int64_t ncols, int32_t minL,
                           int32_t k, double* col_score, int32_t* col_len, int64_t* top_idx,
                           int32_t* top_len, double* top_score, hipStream_t st)
{
    hipLaunchKernelGGL(k_interest_cols, dim3((unsigned int)((ncols + 255) / 256)), dim3(256), 0, st,
                       heat, L, ld, ncols, minL, col_score, col_len);
    hipLaunchKernelGGL(k_interest_top, dim3(1), dim3(INTEREST_BLOCK), 0, st, col_score, col_len,
                       ncols, k, top_idx, top_len, top_score);
    return hipGetLastError();
}

static size_t al256(size_t x) { return (x + 255) & ~(size_t)255; }

bool make_layout(int64_t n, int32_t minL, int32_t maxL, int32_t k, Layout* out)
{
    Layout l = {};
    l.n = n;
    l.minL = minL;
    l.maxL = maxL;
    l.k = k;
    l.L = maxL - minL + 1;
    l.kp = k + KP_EXTRA;
    l.Nmax = n - minL + 1;
    l.Npad = ((l.Nmax + 1 + R_MAX - 1) / R_MAX) * R_MAX + R_MAX;
    l.Tlen = l.Npad + maxL + 256;
    l.nwords = l.Npad / 64 + 1;
    const int64_t nblk = (l.Nmax + EXACT_COLS - 1) / EXACT_COLS;
    const int64_t nch = (l.Nmax + SCREEN_COLS - 1) / SCREEN_COLS;
    l.pcap = std::min<int64_t>(EXACT_GRID_BATCH, CAND_GROUPS * nblk) + 2 * CAND_GROUPS;
    // groups go SCREEN_GROUPS at a time where windows are short
    constexpr int SG = CAND_GROUPS / SCREEN_GROUPS;
    l.lbcap = std::max<int64_t>(std::min<int64_t>(SCREEN_GRID, CAND_GROUPS * nch) + 2 * CAND_GROUPS,
                                SCREEN_GROUPS * (std::min<int64_t>(SCREEN_GRID, SG * nch) + 2 * SG));
    const size_t hl = (size_t)(l.Npad + 64);
    size_t o = 0;
    l.off_T = o;     o = al256(o + sizeof(double) * (size_t)l.Tlen);
    l.off_mu = o;    o = al256(o + sizeof(double) * hl);
    l.off_var = o;   o = al256(o + sizeof(double) * hl);
    l.off_mu2 = o;   o = al256(o + sizeof(double) * hl);
    l.off_var2 = o;  o = al256(o + sizeof(double) * hl);
    l.off_h32 = o;   o = al256(o + 3 * al256(sizeof(float) * hl));
    // inv64, df64, dg64, rho, rhs: the last four, contiguous, hold at least
    // 32 Npad bytes and serve the screening's bounds outside a sweep (64 bytes
    // per group and exact block: CAND_GROUPS / 2 bytes per row)
    static_assert(CAND_GROUPS * CAND_GROUP * sizeof(float) <= 32 * EXACT_COLS, "bounds fit");
    l.off_h64 = o;   o = al256(o + 3 * al256(sizeof(double) * hl));
    l.off_rho = o;   o = al256(o + sizeof(unsigned long long) * (size_t)l.Npad);
    l.off_rhs = o;   o = al256(o + sizeof(unsigned long long) * (size_t)l.Npad);
    l.off_alive = o; o = al256(o + sizeof(unsigned long long) * (size_t)l.nwords);
    l.off_unc = o;   o = al256(o + sizeof(unsigned long long) * (size_t)l.nwords);
    l.off_tsel = o;  o = al256(o + sizeof(int32_t) * (size_t)(l.Npad / 64 + 1));
    l.off_tref = o;  o = al256(o + sizeof(int32_t) * (size_t)(l.Npad / 64 + 1));
    l.off_hot = o;   o = al256(o + sizeof(int32_t) * (size_t)HOT_MAX);
    l.off_twork = o; o = al256(o + sizeof(uint32_t) * (size_t)l.nwords);
    l.off_cand = o;  o = al256(o + sizeof(int64_t) * (size_t)CAND_MAX);
    l.off_part = o;  o = al256(o + sizeof(double) * (size_t)(2 * CAND_GROUP) * (size_t)l.pcap);
    l.off_lbp = o;   o = al256(o + sizeof(float) * (size_t)(CAND_GROUP * l.lbcap));
    l.off_half = o;  o = al256(o + sizeof(uint16_t) * (size_t)HALF_STRIDE * (size_t)nch);
    l.off_scale = o; o = al256(o + sizeof(double) * 2 * (size_t)nch);
    l.off_wit = o;   o = al256(o + sizeof(int32_t) * hl);
    l.off_wc = o;    o = al256(o + sizeof(double) * hl);
    l.off_hist = o;  o = al256(o + sizeof(double) * (size_t)(l.L > 0 ? l.L : 1));
    l.off_evc = o;   o = al256(o + sizeof(unsigned long long) * EV_CLASSES * EV_SLOTS);
    l.off_ctrl = o;  o = al256(o + sizeof(Ctrl));
    l.off_red = o;   o = al256(o + sizeof(double) * 2 * RED_BLOCKS);
    l.off_sgm = o;   o = al256(o + sizeof(double) * 2 * (size_t)((l.Npad + 64 + 255) / 256));
    l.total = o;
    *out = l;
    return true;
}

SeriesDev carve(void* base, const Layout& l)
{
    char* p = (char*)base;
    const size_t hl = (size_t)(l.Npad + 64);
    SeriesDev s = {};
    s.n = l.n;
    s.Nmax = l.Nmax;
    s.Npad = l.Npad;
    s.Tlen = l.Tlen;
    s.nwords = l.nwords;
    s.pcap = l.pcap;
    s.minL = l.minL;
    s.maxL = l.maxL;
    s.k = l.k;
    s.kp = l.kp;
    s.L = l.L;
    s.T = (double*)(p + l.off_T);
    s.mu = (double*)(p + l.off_mu);
    s.var = (double*)(p + l.off_var);
    s.mu2 = (double*)(p + l.off_mu2);
    s.var2 = (double*)(p + l.off_var2);
    s.df32 = (float*)(p + l.off_h32);
    s.dg32 = (float*)(p + l.off_h32 + al256(sizeof(float) * hl));
    s.inv32 = (float*)(p + l.off_h32 + 2 * al256(sizeof(float) * hl));
    s.inv64 = (double*)(p + l.off_h64);
    s.df64 = (double*)(p + l.off_h64 + al256(sizeof(double) * hl));
    s.dg64 = (double*)(p + l.off_h64 + 2 * al256(sizeof(double) * hl));
    s.alive = (unsigned long long*)(p + l.off_alive);
    s.rho = (unsigned long long*)(p + l.off_rho);
    s.rhs = (unsigned long long*)(p + l.off_rhs);
    s.unc = (unsigned long long*)(p + l.off_unc);
    s.tsel = (int32_t*)(p + l.off_tsel);
    s.tref = (int32_t*)(p + l.off_tref);
    s.hot = (int32_t*)(p + l.off_hot);
    s.twork = (uint32_t*)(p + l.off_twork);
    s.cand = (int64_t*)(p + l.off_cand);
    s.part = (double*)(p + l.off_part);
    s.lbp = (float*)(p + l.off_lbp);
    s.ub = (float*)s.df64;         // free outside a round's sweeps (see make_layout)
    s.fail = (int32_t*)s.df32;     // likewise
    s.pairs = (int2*)s.df64;       // likewise (df64, dg64)
    s.half = (uint16_t*)(p + l.off_half);
    s.chunk_scale = (double*)(p + l.off_scale);
    s.wit = (int32_t*)(p + l.off_wit);
    s.wc = (double*)(p + l.off_wc);
    s.hist = (double*)(p + l.off_hist);
    s.evc = (unsigned long long*)(p + l.off_evc);
    s.ctrl = (Ctrl*)(p + l.off_ctrl);
    s.red = (double*)(p + l.off_red);
    s.sgm = (double*)(p + l.off_sgm);
    return s;
}

void series_blocks(const Layout& l, const SweepCfg& cfg, int64_t out[PFX_KINDS])
{
    const int rn = 64 * cfg.q_near, rf = 64 * cfg.q_far, rr = 64 * cfg.q_ref;
    // chunks of the first pass: near_cols, at most every column; a dense round's
    // as far as the cap allows (its bounds cover every column in any case)
    const int64_t tiles = (l.Nmax + rn - 1) / rn;
    const auto chunks = [&](int64_t cols) {
        return (std::min(cols, l.Nmax) + cfg.near_chunk - 1) / cfg.near_chunk;
    };
    int64_t nsub = chunks(cfg.near_cols);
    if (cfg.may_dense && l.Nmax <= DENSE_NEAR_MAXN && l.minL <= DENSE_MAXM)
        nsub = std::max(nsub, std::min(chunks(DENSE_NEAR), NEAR_ITEMS / tiles));
    out[PFX_ELEM] = (l.Npad + 64 + 255) / 256;
    out[PFX_NEAR] = tiles * nsub;
    out[PFX_TSEL] = ((l.Nmax + rf - 1) / rf + 255) / 256;
    out[PFX_TREF] = ((l.Nmax + rr - 1) / rr + 255) / 256;
    out[PFX_BAND] = (l.Nmax + BAND_S - 1) / BAND_S;
}

}  // namespace palmad
