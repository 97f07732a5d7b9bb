// Adjoint of the reported nearest-neighbour distances (backward pass).
//
// For a reported discord i of length m, nnDist = min over non-self matches j
// of ED(x^, y^), the z-normalised distance of Eq. (4)-(5).  Almost
// everywhere the minimiser j* is locally constant, so
//   d nnDist / d t_{i+k} = (rho * x^_k - y^_k) / (sigma_i * d)
//   d nnDist / d t_{j*+k} = (rho * y^_k - x^_k) / (sigma_j* * d)
// with d = nnDist and rho the Pearson correlation of the two windows
// (d^2 = 2m(1 - rho), Eq. (6)).  The minimiser is not stored by the forward
// pass: each row is recomputed here with direct FP64 dot products against
// every column (ties -> smallest j), then the gradient is scattered into
// grad_T with FP64 atomics.  A zero distance or a flat window contributes
// nothing (the distance is not differentiable there).
#include "engine.h"

#include <math.h>

#include <algorithm>

namespace palmad {

constexpr int ADJ_BLOCK = 256;

__device__ __forceinline__ double adj_wave_sum(double v)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// Block-wide sum, result broadcast to every thread.
__device__ double adj_block_sum(double v, double* sh)
{
    v = adj_wave_sum(v);
    const int w = threadIdx.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh[w] = v;
    __syncthreads();
    double t = 0.0;
    for (int i = 0; i < (int)(blockDim.x >> 6); ++i) t += sh[i];
    return t;
}

// Mean and population sigma of window [p, p+m) (two passes, block-wide).
__device__ void adj_window_stats(const double* T, int64_t p, int32_t m, double* sh, double& mu,
                                 double& sg)
{
    double s = 0.0;
    for (int k = threadIdx.x; k < m; k += blockDim.x) s += T[p + k];
    mu = adj_block_sum(s, sh) / (double)m;
    double q = 0.0;
    for (int k = threadIdx.x; k < m; k += blockDim.x) {
        const double d = T[p + k] - mu;
        q += d * d;
    }
    sg = sqrt(adj_block_sum(q, sh) / (double)m);
}

// Partial nearest neighbours of up to `rows` reported rows against `span`
// blocks of 256 columns (launch_adjoint): (max rho, smallest argmax j) per row and
// block.  Consecutive rows of one length (a search reports k of each) share a
// column's mean and deviation and the reads of its window, R at a time; every
// value is the same as for a row alone.  Bound by the LDS reads, of a row's
// value for two columns, and the FP64 operations, 3 + R per offset and column.
// Held to 128 registers, four waves per SIMD: with a row's state and results in
// registers it took 204, and rows that share nothing ran slower than one at a
// time.  (Whole call, a row and 256 columns per workgroup, with 204 registers,
// so: 325 rows, five per length of 96 to 160, 200,000 columns 3.40, 2.00, 1.55 ms;
// 129 rows of different lengths 1.80, 2.37, 1.75.)
constexpr int ADJ_ROWS = 16;  // most rows per workgroup
constexpr int ADJ_RUN = 8;    // most rows sharing a column
constexpr int ADJ_SPAN = 4;   // most blocks of columns
constexpr int64_t ADJ_FILL = 2048;  // workgroups wanted: eight per CU

// The C column windows t + 256 e, less their means, against R centred rows xs
// (stride doubles apart): sums of squares and products, then each row's largest
// correlation over the wave's columns and the first column that has it.
template <int R, int C>
__device__ __forceinline__ void adj_columns(const double* t, const double* xs, int stride, int32_t m,
                                            const double (&mu)[C], int64_t N, int64_t j0, double feps,
                                            unsigned int ok, const double* sgi, const long long* ii,
                                            double (*rv)[ADJ_RUN][ADJ_BLOCK / 64],
                                            long long (*rj)[ADJ_RUN][ADJ_BLOCK / 64])
{
    double c0[C][R], c1[C][R], vv[C];
#pragma unroll
    for (int e = 0; e < C; ++e) {
        vv[e] = 0.0;
#pragma unroll
        for (int r = 0; r < R; ++r) c0[e][r] = c1[e][r] = 0.0;
    }
    int k = 0;
    for (; k + 1 < m; k += 2) {
        double d0[C], d1[C];
#pragma unroll
        for (int e = 0; e < C; ++e) {
            d0[e] = t[ADJ_BLOCK * e + k] - mu[e];
            d1[e] = t[ADJ_BLOCK * e + k + 1] - mu[e];
            vv[e] = fma(d0[e], d0[e], vv[e]);
            vv[e] = fma(d1[e], d1[e], vv[e]);
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const double x0 = xs[r * stride + k], x1 = xs[r * stride + k + 1];
#pragma unroll
            for (int e = 0; e < C; ++e) {
                c0[e][r] = fma(x0, d0[e], c0[e][r]);
                c1[e][r] = fma(x1, d1[e], c1[e][r]);
            }
        }
    }
    if (k < m) {
#pragma unroll
        for (int e = 0; e < C; ++e) {
            const double d0 = t[ADJ_BLOCK * e + k] - mu[e];
            vv[e] = fma(d0, d0, vv[e]);
#pragma unroll
            for (int r = 0; r < R; ++r) c0[e][r] = fma(xs[r * stride + k], d0, c0[e][r]);
        }
    }
    const int tid = threadIdx.x;
#pragma unroll
    for (int e = 0; e < C; ++e) {
        const int64_t j = j0 + ADJ_BLOCK * e + tid;
        const double sgj = sqrt(vv[e] / (double)m);
        const bool flat_j = sgj <= feps;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const long long i = ii[r];
            const double si = sgi[r];
            const bool flat_i = si <= feps;
            double b = -1e300;
            if (((ok >> r) & 1u) && j < N && (j <= i - m || j >= i + m))
                b = flat_i || flat_j ? (flat_i && flat_j ? 1.0 : 0.0)
                                     : fmin(1.0, fmax(-1.0, (c0[e][r] + c1[e][r]) / ((double)m * si * sgj)));
            // (columns ascend with the lane: the first lane that has the maximum)
            double top = b;
#pragma unroll
            for (int o = 32; o >= 1; o >>= 1) top = fmax(top, __shfl_xor(top, o));
            const int first = __ffsll((long long)__ballot(b == top)) - 1;
            if ((tid & 63) == 0) {
                rv[e][r][tid >> 6] = top;
                rj[e][r][tid >> 6] = top > -1e299 ? (long long)(j + first) : 0x7fffffffffffffffll;
            }
        }
    }
}

template <int C>
__global__ __launch_bounds__(ADJ_BLOCK, 4) void k_adj_rows(const double* __restrict__ T, int64_t n,
                                                        int64_t K, const int64_t* __restrict__ idx,
                                                        const int32_t* __restrict__ len,
                                                        const Ctrl* ctrl, double* part, int64_t nblk,
                                                        int rows, int span, int max_run, int stride)
{
    extern __shared__ double lds[];
    __shared__ double sh[8];
    __shared__ double rv[C][ADJ_RUN][ADJ_BLOCK / 64];
    __shared__ long long rj[C][ADJ_RUN][ADJ_BLOCK / 64];
    __shared__ double sgi[ADJ_RUN];
    __shared__ long long ii[ADJ_RUN];
    const int tid = threadIdx.x;
    const int64_t q0 = (int64_t)blockIdx.y * rows, q1 = std::min<int64_t>(K, q0 + rows);
    const int64_t x0 = (int64_t)blockIdx.x * span, x1 = std::min<int64_t>(nblk, x0 + span);
    const double feps = ctrl->flat_eps;
    double* ts = lds;                          // T[j0 .. j0 + 256 C + m)
    double* xs = lds + (ADJ_BLOCK * C + stride);  // centred windows, stride apart
    for (int64_t q = q0; q < q1;) {
        const int32_t m = len[q];
        int run = 1;
        while (run < max_run && q + run < q1 && len[q + run] == m) ++run;
        const int64_t N = n - m + 1;
        const bool len_ok = m >= 3 && m <= ctrl->m;  // ctrl->m holds max length
        unsigned int ok = 0u;
        for (int r = 0; r < run && len_ok; ++r) {
            const int64_t i = idx[q + r];
            if (i < 0 || i >= N) continue;
            ok |= 1u << r;
            double mui, sg;
            adj_window_stats(T, i, m, sh, mui, sg);
            for (int k = tid; k < m; k += ADJ_BLOCK) xs[r * stride + k] = T[i + k] - mui;
            if (tid == 0) {
                ii[r] = i;
                sgi[r] = sg;
            }
        }
        for (int64_t x = x0; x < x1; x += C) {
            const int64_t j0 = x * ADJ_BLOCK;
            __syncthreads();  // the previous blocks and run are consumed
            if (ok && j0 < N) {
                for (int t = tid; t < ADJ_BLOCK * C + m; t += ADJ_BLOCK) ts[t] = j0 + t < n ? T[j0 + t] : 0.0;
                __syncthreads();
                const double* t = ts + tid;
                double mu[C];
#pragma unroll
                for (int e = 0; e < C; ++e) mu[e] = 0.0;
                for (int k = 0; k < m; ++k)
#pragma unroll
                    for (int e = 0; e < C; ++e) mu[e] += t[ADJ_BLOCK * e + k];
#pragma unroll
                for (int e = 0; e < C; ++e) mu[e] /= (double)m;
#define ADJ_COLUMNS(R) adj_columns<R, C>(t, xs, stride, m, mu, N, j0, feps, ok, sgi, ii, rv, rj)
                switch (run) {
                case 1: ADJ_COLUMNS(1); break;
                case 2: ADJ_COLUMNS(2); break;
                case 3: ADJ_COLUMNS(3); break;
                case 4: ADJ_COLUMNS(4); break;
                case 5: ADJ_COLUMNS(5); break;
                case 6: ADJ_COLUMNS(6); break;
                case 7: ADJ_COLUMNS(7); break;
                default: ADJ_COLUMNS(8); break;
                }
#undef ADJ_COLUMNS
            } else if (tid < C * ADJ_RUN * (ADJ_BLOCK / 64)) {
                (&rv[0][0][0])[tid] = -1e300;
                (&rj[0][0][0])[tid] = 0x7fffffffffffffffll;
            }
            __syncthreads();
            const int r = tid & (ADJ_RUN - 1), e = tid / ADJ_RUN;
            if (e < C && r < run && x + e < x1) {
                double b = rv[e][r][0];
                long long bj = rj[e][r][0];
                for (int w = 1; w < ADJ_BLOCK / 64; ++w)
                    if (rv[e][r][w] > b || (rv[e][r][w] == b && rj[e][r][w] < bj)) {
                        b = rv[e][r][w];
                        bj = rj[e][r][w];
                    }
                const int64_t slot = ((q + r) * nblk + x + e) * 2;
                part[slot] = b;
                part[slot + 1] = bj == 0x7fffffffffffffffll ? 1e300 : (double)bj;  // 1e300: none
            }
        }
        __syncthreads();  // (the next run's windows take this one's place)
        q += run;
    }
}

// Per reported row: reduce the partials to j*, then scatter
// g * d nnDist / dT over both windows.
__global__ __launch_bounds__(ADJ_BLOCK) void k_adj_scatter(const double* __restrict__ T,
                                                           const int64_t* __restrict__ idx,
                                                           const int32_t* __restrict__ len,
                                                           const double* __restrict__ gin,
                                                           const Ctrl* ctrl, const double* part,
                                                           int64_t nblk, double* grad,
                                                           int64_t* jstar_out)
{
    __shared__ double sh[8];
    __shared__ double rv[ADJ_BLOCK / 64];
    __shared__ double rj[ADJ_BLOCK / 64];
    __shared__ double bcast[2];
    const int q = blockIdx.x;
    const int tid = threadIdx.x;
    double best = -1e300, bj = 1e300;
    for (int64_t p = tid; p < nblk; p += ADJ_BLOCK) {
        const double v = part[((int64_t)q * nblk + p) * 2];
        const double jj = part[((int64_t)q * nblk + p) * 2 + 1];
        if (v > best || (v == best && jj < bj)) {
            best = v;
            bj = jj;
        }
    }
    for (int o = 32; o >= 1; o >>= 1) {
        const double v = __shfl_xor(best, o);
        const double jj = __shfl_xor(bj, o);
        if (v > best || (v == best && jj < bj)) {
            best = v;
            bj = jj;
        }
    }
    if ((tid & 63) == 0) {
        rv[tid >> 6] = best;
        rj[tid >> 6] = bj;
    }
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < ADJ_BLOCK / 64; ++w)
            if (rv[w] > best || (rv[w] == best && rj[w] < bj)) {
                best = rv[w];
                bj = rj[w];
            }
        bcast[0] = best;
        bcast[1] = bj;
    }
    __syncthreads();
    const double rho = bcast[0];
    const bool found = bcast[1] < 1e299;
    const int64_t js = found ? (int64_t)bcast[1] : -1;
    const int64_t i = idx[q];
    const int32_t m = len[q];
    if (tid == 0 && jstar_out) jstar_out[q] = js;
    if (!found) return;
    const double g = gin[q];
    double mui, sgi, muj, sgj;
    adj_window_stats(T, i, m, sh, mui, sgi);
    adj_window_stats(T, js, m, sh, muj, sgj);
    const double feps = ctrl->flat_eps;
    const double d = sqrt(fmax(0.0, 2.0 * (double)m * (1.0 - rho)));
    if (!(d > 0.0) || sgi <= feps || sgj <= feps || g == 0.0) return;
    for (int k = tid; k < m; k += ADJ_BLOCK) {
        const double xh = (T[i + k] - mui) / sgi;
        const double yh = (T[js + k] - muj) / sgj;
        atomicAdd(&grad[i + k], g * (rho * xh - yh) / (sgi * d));
        atomicAdd(&grad[js + k], g * (rho * yh - xh) / (sgj * d));
    }
}

hipError_t launch_adjoint(const double* Tpad, int64_t n, int64_t K, int32_t maxm,
                          const int64_t* idx, const int32_t* len, const double* gin,
                          const Ctrl* ctrl, double* part, int64_t nblk, double* grad,
                          int64_t* jstar, hipStream_t st)
{
    if (K <= 0) return hipSuccess;
    // two columns per thread, which share the rows' reads, while those fit
    const int stride = maxm + 1;
    int cols = maxm <= 2048 ? 2 : 1, rows = ADJ_ROWS, span = ADJ_SPAN;
    // Rows and columns that share a workgroup save reads and operations, but a
    // small problem then leaves the device idle behind a few serial workgroups:
    // the shares are cut until there are ADJ_FILL of them, the columns' first
    // (that costs the least).  (Whole call, full shares and these: 8,000 points
    // and 33 rows of different lengths 0.64 and 0.24 ms; 50,000 points and 33
    // rows 0.66 and 0.29; 12,000 points and 99 rows, three per length, 0.44 and
    // 0.27.  4096 workgroups are too many: 50,000 points and 325 rows 0.71 ms
    // with 2048, 0.86.)
    const auto groups = [&] { return ((nblk + span - 1) / span) * ((K + rows - 1) / rows); };
    while (groups() < ADJ_FILL) {
        if (span > cols) span /= 2;
        else if (rows > 1) rows /= 2;
        else if (cols > 1) cols = span = 1;
        else break;
    }
    // as many rows of one length as fit 64 KB beside the columns' values
    const int max_run = std::max(
        1, std::min({ADJ_RUN, rows, (8000 - ADJ_BLOCK * cols - stride) / stride}));
    const size_t lds = sizeof(double) * (size_t)(ADJ_BLOCK * cols + (max_run + 1) * stride);
    hipLaunchKernelGGL(cols == 2 ? k_adj_rows<2> : k_adj_rows<1>,
                       dim3((unsigned int)((nblk + span - 1) / span),
                            (unsigned int)((K + rows - 1) / rows)),
                       dim3(ADJ_BLOCK), lds, st, Tpad, n, K, idx, len, ctrl, part, nblk, rows, span,
                       max_run, stride);
    hipLaunchKernelGGL(k_adj_scatter, dim3((unsigned int)K), dim3(ADJ_BLOCK), 0, st, Tpad, idx, len,
                       gin, ctrl, part, nblk, grad, jstar);
    return hipGetLastError();
}

}  // namespace palmad
