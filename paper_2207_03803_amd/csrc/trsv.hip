// Back-substitution R c = (Q^T b)[0:M] (Sec. Theory: c = R^-1 Q^T b, solved as
// a series of back substitutions) and small vector utilities.
#include "trsv.h"

namespace gap {

template <class TR, bool TRANS>
__global__ __launch_bounds__(256, 1) void trsv_fused_kernel(const TR *__restrict__ R, TrsvArgs a)
{
    __shared__ TrsvLds L;
    if (threadIdx.x == 0)
        L.dead = 0;
    for (int64_t q = take_item(a, L); q < a.nb; q = take_item(a, L))
        if (!trsv_item<TR, TRANS>(R, a, L, q, a.rhs, nullptr, a.xbuf, a.x))
            break;
    trsv_finish(a, L, a.n);
}

template <class TR, bool TRANS>
static hipError_t trsv_fused(const TR *R, int64_t ld, int64_t n, const double *rhs, double *x, const TrsvSync &sync,
                             hipStream_t s)
{
    const TrsvArgs a = trsv_args(ld, n, rhs, x, sync);
    const unsigned g = (unsigned)(a.nb < TS_GRID ? a.nb : TS_GRID);
    hipLaunchKernelGGL((trsv_fused_kernel<TR, TRANS>), dim3(g), dim3(256), 0, s, R, a);
    return hipGetLastError();
}

__global__ __launch_bounds__(256) void trsv_clear_kernel(TrsvSync sync, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < 2 * n)
        sync.xbuf[i] = X_EMPTY;
    if (i < 2)
        sync.flags[i] = 0;
}

hipError_t launch_trsv_clear(const TrsvSync &sync, int64_t n, hipStream_t s)
{
    hipLaunchKernelGGL(trsv_clear_kernel, dim3((unsigned)((2 * n + 255) / 256)), dim3(256), 0, s, sync, n);
    return hipGetLastError();
}

hipError_t launch_trsv_upper(const double *R, int64_t ld, int64_t n, const double *rhs, double *x,
                             const TrsvSync &sync, hipStream_t s)
{
    return trsv_fused<double, false>(R, ld, n, rhs, x, sync, s);
}

hipError_t launch_trsv_upper_t(const double *R, int64_t ld, int64_t n, const double *rhs, double *x,
                               const TrsvSync &sync, hipStream_t s)
{
    return trsv_fused<double, true>(R, ld, n, rhs, x, sync, s);
}

hipError_t launch_trsv_upper_f32(const float *R, int64_t ld, int64_t n, const double *rhs, double *x,
                                 const TrsvSync &sync, hipStream_t s)
{
    return trsv_fused<float, false>(R, ld, n, rhs, x, sync, s);
}

hipError_t launch_trsv_upper_t_f32(const float *R, int64_t ld, int64_t n, const double *rhs, double *x,
                                   const TrsvSync &sync, hipStream_t s)
{
    return trsv_fused<float, true>(R, ld, n, rhs, x, sync, s);
}

__global__ __launch_bounds__(256) void sumsq_kernel(const double *x, int64_t n, double *out, double *part,
                                                    unsigned *counter)
{
    __shared__ double red[4];
    __shared__ int flag;
    double v = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
        v += x[i] * x[i];
    v = wave_sum(v);
    if ((threadIdx.x & 63) == 0)
        red[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0)
        part[blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
    if (!arrive_last(counter, gridDim.x, &flag))
        return;
    if (threadIdx.x == 0) {
        double s = 0.0;
        for (unsigned b = 0; b < gridDim.x; ++b)
            s += part[b];
        *out = s;
    }
}

hipError_t launch_sumsq(const double *x, int64_t n, double *out, double *part, unsigned *counter,
                        hipStream_t s)
{
    int64_t g = (n + 255) / 256;
    if (g > 256)
        g = 256;
    if (g < 1)
        g = 1;
    hipLaunchKernelGGL(sumsq_kernel, dim3((unsigned)g), dim3(256), 0, s, x, n, out, part, counter);
    return hipGetLastError();
}

__global__ void assemble_b_kernel(const double *y, const double *sigma, int64_t N, double *bcol,
                                  int64_t lda)
{
    const int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (r < N)
        bcol[r] = y[r] / sigma[r];
    else if (r < lda)
        bcol[r] = 0.0;
}

hipError_t launch_assemble_b(const double *y, const double *sigma, int64_t N, double *bcol,
                             int64_t lda, hipStream_t s)
{
    hipLaunchKernelGGL(assemble_b_kernel, dim3((unsigned)((lda + 255) / 256)), dim3(256), 0, s, y, sigma,
                       N, bcol, lda);
    return hipGetLastError();
}

__global__ void copy_f32_f64_kernel(const float *src, double *dst, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n)
        dst[i] = (double)src[i];
}

hipError_t launch_copy_f32_f64(const float *src, double *dst, int64_t n, hipStream_t s)
{
    if (n <= 0)
        return hipSuccess;
    hipLaunchKernelGGL(copy_f32_f64_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, src, dst, n);
    return hipGetLastError();
}

}  // namespace gap
