// Small kernels of the leading-eigenvector iteration (svdp_eigtop_run.h): everything else in it is k_dgemm, the blocked
// Cholesky factorisation and block Jacobi on the projected matrix.  Vectors are rows, X [k][n].  Each kernel is one
// pass over at most k x n doubles (10 MB at k = 320, n = 4096) and bound by its launch (5 to 8 us).
#pragma once

#include "svdp_whiten.h"

namespace svdp {

// Sum over the block's 256 threads, in a fixed order; every thread gets it.
__device__ __forceinline__ double block_sum_256(double v, double *sm)
{
    sm[threadIdx.x] = v;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) sm[threadIdx.x] += sm[threadIdx.x + w];
        __syncthreads();
    }
    const double s = sm[0];
    __syncthreads();
    return s;
}

// X[row0 + i][j] = a fixed pseudo-random number in (-1, 1) of its place (integer hash, splitmix64): the same start on
// every call, so that results are deterministic
__global__ __launch_bounds__(256) void k_random_rows(double *__restrict__ X, int row0, int rows, int n)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= (size_t)rows * n) return;
    const size_t at = (size_t)row0 * n + i;
    unsigned long long z = (at + 1) * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    z ^= z >> 31;
    X[at] = (double)(long long)z * (1.0 / 9223372036854775808.0);
}

// every row of X gets unit length (one block per row); a row of zeros stays one
__global__ __launch_bounds__(256) void k_normalize_rows(double *__restrict__ X, int n)
{
    __shared__ double sm[256];
    double *x = X + (size_t)blockIdx.x * n;
    double s = 0.0;
    for (int j = threadIdx.x; j < n; j += 256) s += x[j] * x[j];
    s = block_sum_256(s, sm);
    const double f = s > 0.0 ? 1.0 / sqrt(s) : 0.0;
    for (int j = threadIdx.x; j < n; j += 256) x[j] *= f;
}

__global__ __launch_bounds__(256) void k_add_diagonal(double *__restrict__ A, int n, double v)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) A[(size_t)i * n + i] += v;
}

// sel[p] = place of the p-th largest of lam [k], ties by place; theta[p] = its value.  NaN: sel is some order of the
// places all the same (the caller sees the NaN in theta).
__global__ __launch_bounds__(256) void k_rank_descending(const double *__restrict__ lam, int k, int32_t *__restrict__ sel,
                                                         double *__restrict__ theta)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= k) return;
    const double v = lam[i];
    const bool nan = !(v == v);
    int p = 0;
    for (int j = 0; j < k; ++j) {
        const double u = lam[j];
        const bool unan = !(u == u);
        p += (unan && (!nan || j < i)) || (!unan && !nan && (u > v || (u == v && j < i)));
    }
    sel[p] = i;
    theta[p] = v;
}

// res[i] = || Y[i] - theta[i] X[i] ||^2 (one block per row)
__global__ __launch_bounds__(256) void k_ritz_residual(const double *__restrict__ X, const double *__restrict__ Y,
                                                       const double *__restrict__ theta, int n, double *__restrict__ res)
{
    __shared__ double sm[256];
    const size_t at = (size_t)blockIdx.x * n;
    const double t = theta[blockIdx.x];
    double s = 0.0;
    for (int j = threadIdx.x; j < n; j += 256) {
        const double v = Y[at + j] - t * X[at + j];
        s += v * v;
    }
    s = block_sum_256(s, sm);
    if (threadIdx.x == 0) res[blockIdx.x] = s;
}

// out[i] = X[i] . Y[i] / X[i] . X[i] (one block per row)
__global__ __launch_bounds__(256) void k_rayleigh(const double *__restrict__ X, const double *__restrict__ Y, int n,
                                                  double *__restrict__ out)
{
    __shared__ double sm[256];
    const size_t at = (size_t)blockIdx.x * n;
    double xy = 0.0, xx = 0.0;
    for (int j = threadIdx.x; j < n; j += 256) {
        const double x = X[at + j];
        xy += x * Y[at + j];
        xx += x * x;
    }
    xy = block_sum_256(xy, sm);
    xx = block_sum_256(xx, sm);
    if (threadIdx.x == 0) out[blockIdx.x] = xy / xx;
}

// y = alpha y + beta x
__global__ __launch_bounds__(256) void k_combine(double *__restrict__ y, const double *__restrict__ x, double alpha, double beta,
                                                 size_t n)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) y[i] = alpha * y[i] + beta * x[i];
}

}   // namespace svdp
