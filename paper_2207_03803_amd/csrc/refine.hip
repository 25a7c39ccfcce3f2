// Mixed precision: iterative refinement of the least-squares solution in FP64
// against the FP64 stacked matrix [A | b] kept from the build, preconditioned
// by R, the upper triangle of the FP32 Householder factorisation (triangular
// solves with R take FP64 arithmetic).
//
// Stage 1, corrected semi-normal equations (Bjorck 1987):
//   r = b - A c,  s = A^T r,  solve R^T R dc = s,  c += dc.
// Each step scales the error by roughly u_32 kappa(A), which nears or passes 1
// once kappa(A) nears 1/u_32.  When a correction, from the second on, fails to
// halve and is not yet small, the loop keeps c (without that correction when it
// grew) and moves to stage 2.
//
// Stage 2, CGLS on the right-preconditioned problem min ||A R^-1 v - b||,
// c = R^-1 v, carried out in c's coordinates (preconditioned CGLS, Bjorck,
// Numerical Methods for Least Squares Problems, 1996):
//   start  r = b - A c,  z = R^-T A^T r,  p = R^-1 z,  gamma = ||z||^2
//   step   q = A p,  alpha = gamma / ||q||^2,  c += alpha p,  r -= alpha q,
//          z = R^-T A^T r,  gamma' = ||z||^2,  p = R^-1 z + (gamma' / gamma) p.
// Its rate is set by the spread of the singular values of A R^-1, so it needs
// no bound on u_32 kappa(A).
//
// Both stages run the same three kernels per iteration, steered by a mode
// word on the device: the product with A, the product with A^T, and the two triangular solves
// with the end of the step.  A CGLS step's r -= alpha q is taken where r is next read: on the
// way in the product with A^T, and by the rows' own workgroups when they form the next q.
// Iterations stop on the device once the step is
// <= tol ||c|| (or once it stops halving at a level <= 1e-9 ||c||, the FP64
// rounding floor): later iterations' kernels see the flag and return at once,
// so the loop needs no host synchronisation.  (With seven launches per
// iteration, four of them for vectors, an iteration after the last cost 20 us instead of 10, and
// one at 2,500 x 500 71 us instead of 53.)
#include "trsv.h"

namespace gap {

constexpr int RB = 64;    // rows per workgroup in the residual
constexpr int RCH = 16;   // its column chunks, one per wave
constexpr double STALL_OK = 1e-9;  // a stalled correction this small counts as converged
constexpr int MODE_CSNE = 0, MODE_CG_START = 1, MODE_CG = 2;

__global__ void convert_f64_f32_kernel(const double *__restrict__ a, float *__restrict__ b, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
        b[i] = (float)a[i];
}

hipError_t launch_convert_f64_f32(const double *a, float *b, int64_t n, hipStream_t s)
{
    int64_t g = (n + 255) / 256;
    if (g > 65536)
        g = 65536;
    hipLaunchKernelGGL(convert_f64_f32_kernel, dim3((unsigned)g), dim3(256), 0, s, a, b, n);
    return hipGetLastError();
}

// b[r, c] = a[r, c] for rows [r0, r1) of columns [c0, c1) (column-major, ld).
__global__ void convert_block_f64_f32_kernel(const double *__restrict__ a, float *__restrict__ b, int64_t ld,
                                             int64_t r0, int64_t r1, int64_t c0, int64_t c1)
{
    const int64_t nr = r1 - r0, total = nr * (c1 - c0);
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (int64_t)gridDim.x * 256) {
        const int64_t c = c0 + i / nr, r = r0 + i % nr;
        b[c * ld + r] = (float)a[c * ld + r];
    }
}

hipError_t launch_convert_block_f64_f32(const double *a, float *b, int64_t ld, int64_t r0, int64_t r1, int64_t c0,
                                        int64_t c1, hipStream_t s)
{
    const int64_t total = (r1 - r0) * (c1 - c0);
    if (total <= 0)
        return hipSuccess;
    int64_t g = (total + 255) / 256;
    if (g > 65536)
        g = 65536;
    hipLaunchKernelGGL(convert_block_f64_f32_kernel, dim3((unsigned)g), dim3(256), 0, s, a, b, ld, r0, r1, c0, c1);
    return hipGetLastError();
}

// Fixed-order sum of a 256-thread workgroup (identical in every workgroup for
// identical inputs).
__device__ __forceinline__ double block_sum(double v, double *red)
{
    v = wave_sum(v);
    if ((threadIdx.x & 63) == 0)
        red[threadIdx.x >> 6] = v;
    __syncthreads();
    return (red[0] + red[1]) + (red[2] + red[3]);
}

// r = b - A c, or q = A p in the CGLS steps (after the last step's r -= alpha q), for rows
// [64 blockIdx.x, +64): one column chunk per wave, added in order; partial ||r||^2 (||q||^2) per
// workgroup.  FINAL: after the loop, the residual at the returned c; whether the loop converged
// (status ENOCONV otherwise).  Bound by the read of A (18,250 x 2,250: 70 us, 4.7 TB/s;
// 82 us in two launches).
template <bool FINAL>
__global__ __launch_bounds__(RCH * 64) void resid_kernel(RefineWork w)
{
    __shared__ double red[RCH][RB];
    const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    if (FINAL) {
        if (blockIdx.x == 0 && t == 0 && !*w.done)
            set_status(w.status, DST_ENOCONV);
    } else if (*w.done) {
        return;
    }
    const bool cg = !FINAL && *w.mode == MODE_CG;
    const double *v = cg ? w.p : w.c;
    const int64_t r = (int64_t)blockIdx.x * RB + lane;
    const int64_t per = (w.n + RCH - 1) / RCH;
    const int64_t j0 = wave * per;
    const int64_t j1 = (j0 + per) < w.n ? (j0 + per) : w.n;
    const double *col = w.A + (r < w.m ? r : w.m - 1);
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    int64_t j = j0;
    for (; j + 8 <= j1; j += 8) {
        double x[8];
#pragma unroll
        for (int k = 0; k < 8; ++k)
            x[k] = col[(j + k) * w.lda];
#pragma unroll
        for (int k = 0; k < 8; ++k)
            acc[k & 3] += x[k] * v[j + k];
    }
    for (; j < j1; ++j)
        acc[0] += col[j * w.lda] * v[j];
    red[wave][lane] = (acc[0] + acc[1]) + (acc[2] + acc[3]);
    __syncthreads();
    if (wave != 0)
        return;
    double ac = 0.0;
#pragma unroll
    for (int ch = 0; ch < RCH; ++ch)
        ac += red[ch][lane];
    double o = 0.0;
    if (r < w.m) {
        if (cg) {
            o = ac;
            const double alpha = w.stats[2];
            if (alpha != 0.0)  // zero: no step yet, and no q
                w.r[r] = fma(-alpha, w.q[r], w.r[r]);
            w.q[r] = o;
        } else {
            o = w.A[w.n * w.lda + r] - ac;  // b is column n of [A | b]
            w.r[r] = o;
        }
    }
    const double sq = wave_sum(o * o);
    if (lane == 0)
        w.rnorm_part[blockIdx.x] = sq;
}

// s_j = sum_i A[i][j] r[i], one column per workgroup (fixed-order reduction); in the CGLS steps
// r is r - alpha q, alpha = gamma / ||q||^2 (every workgroup sums the same partials in the same
// order).  Otherwise the first workgroup keeps ||r||^2.
template <bool FINAL>
__global__ __launch_bounds__(256) void atr_kernel(RefineWork w, int64_t nparts)
{
    __shared__ double red[4], red2[4];
    if (!FINAL && *w.done)
        return;
    const bool cg = !FINAL && *w.mode == MODE_CG;
    const int64_t j = blockIdx.x;
    double alpha = 0.0;
    if (cg || j == 0) {
        double a = 0.0;
        for (int64_t b = threadIdx.x; b < nparts; b += 256)
            a += w.rnorm_part[b];
        const double qq = block_sum(a, red2);
        if (cg)
            alpha = qq > 0.0 ? w.stats[3] / qq : 0.0;
        if (j == 0 && threadIdx.x == 0)
            w.stats[cg ? 2 : 0] = cg ? alpha : qq;
    }
    const double *col = w.A + j * w.lda;
    auto at = [&](int64_t i) { return cg ? fma(-alpha, w.q[i], w.r[i]) : w.r[i]; };
    double a0 = 0.0, a1 = 0.0;
    int64_t i = threadIdx.x;
    for (; i + 256 < w.m; i += 512) {
        a0 += col[i] * at(i);
        a1 += col[i + 256] * at(i + 256);
    }
    if (i < w.m)
        a0 += col[i] * at(i);
    const double v = block_sum(a0 + a1, red);
    if (threadIdx.x == 0)
        w.s[j] = v;
}

// End of an iteration (one workgroup).  After the triangular solves z holds
// R^-T A^T r and dc holds R^-1 z.
//   CSNE:       c += dc unless the switch to CGLS drops a grown correction;
//               convergence test on ||dc|| / ||c + dc||.
//   CGLS start: p = dc, gamma = ||z||^2.
//   CGLS step:  c += alpha p (alpha from atr_kernel), convergence test on
//               ||alpha p|| / ||c||, then p = dc + (||z||^2 / gamma) p.
DEV void refine_update(const RefineWork &w)
{
    __shared__ double red[3][4];
    __shared__ int act;
    __shared__ double beta;
    const int mode = *w.mode;
    const double alpha = w.stats[2];
    double a0 = 0.0, a1 = 0.0, a2 = 0.0;
    for (int64_t j = threadIdx.x; j < w.n; j += 256) {
        if (mode == MODE_CSNE) {
            const double d = w.dc[j];
            const double c = w.c[j] + d;
            a0 += d * d;
            a1 += c * c;
        } else if (mode == MODE_CG_START) {
            const double z = w.z[j];
            a2 += z * z;
        } else {
            const double st = alpha * w.p[j];
            const double c = w.c[j] + st;
            w.c[j] = c;
            a0 += st * st;
            a1 += c * c;
            const double z = w.z[j];
            a2 += z * z;
        }
    }
    a0 = wave_sum(a0);
    a1 = wave_sum(a1);
    a2 = wave_sum(a2);
    if ((threadIdx.x & 63) == 0) {
        red[0][threadIdx.x >> 6] = a0;
        red[1][threadIdx.x >> 6] = a1;
        red[2][threadIdx.x >> 6] = a2;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        const double d2 = (red[0][0] + red[0][1]) + (red[0][2] + red[0][3]);
        const double c2 = (red[1][0] + red[1][1]) + (red[1][2] + red[1][3]);
        const double g2 = (red[2][0] + red[2][1]) + (red[2][2] + red[2][3]);
        const double ratio = (c2 > 0.0) ? sqrt(d2 / c2) : 0.0;
        const double prev = w.stats[1];
        const bool small = d2 <= w.tol * w.tol * c2;
        w.iters[0] += 1;
        int a = 0;  // 0: nothing, 1: c += dc, 2: p = dc, 3: p = dc + beta p
        if (mode == MODE_CSNE) {
            const bool halving = ratio <= 0.5 * prev;
            // converged: the correction is below tol; or it has reached the FP64
            // rounding floor (stopped halving) at a level already below STALL_OK
            const bool stalled = w.iters[0] > 1 && !halving && ratio <= STALL_OK;
            const bool slow = w.iters[0] > 1 && !halving && !small && !stalled;
            a = (!slow || ratio < prev) ? 1 : 0;
            if (slow)
                *w.mode = MODE_CG_START;
            if (small || stalled)
                *w.done = 1;
            w.stats[1] = ratio;
        } else if (mode == MODE_CG_START) {
            w.stats[2] = 0.0;  // no step of r outstanding
            w.stats[3] = g2;
            *w.mode = MODE_CG;
            a = 2;
        } else {
            w.iters[1] += 1;
            const bool stalled = w.iters[1] > 1 && !(ratio <= 0.5 * prev) && ratio <= STALL_OK;
            if (small || stalled)
                *w.done = 1;
            const double g = w.stats[3];
            beta = g > 0.0 ? g2 / g : 0.0;
            w.stats[3] = g2;
            w.stats[1] = ratio;
            a = 3;
        }
        act = a;
    }
    __syncthreads();
    const int a = act;
    if (a == 1) {
        for (int64_t j = threadIdx.x; j < w.n; j += 256)
            w.c[j] += w.dc[j];
    } else if (a == 2) {
        for (int64_t j = threadIdx.x; j < w.n; j += 256)
            w.p[j] = w.dc[j];
    } else if (a == 3) {
        const double b = beta;
        for (int64_t j = threadIdx.x; j < w.n; j += 256)
            w.p[j] = w.dc[j] + b * w.p[j];
    }
}

// z = R^-T s and dc = R^-1 z (R from the FP32 factorisation, FP64 arithmetic) in one launch, the
// second solve's block rows behind the first's in ticket order; then the end of the iteration
// on the last workgroup.
__global__ __launch_bounds__(256, 1) void refine_step_kernel(RefineWork w, TrsvArgs a)
{
    __shared__ TrsvLds L;
    if (*w.done)
        return;
    if (threadIdx.x == 0)
        L.dead = 0;
    unsigned long long *xbuf2 = a.xbuf + a.n;
    for (int64_t q = take_item(a, L); q < 2 * a.nb; q = take_item(a, L)) {
        const bool ok = q < a.nb
                            ? trsv_item<float, true>(w.R32, a, L, q, w.s, nullptr, a.xbuf, w.z)
                            : trsv_item<float, false>(w.R32, a, L, q - a.nb, nullptr, a.xbuf, xbuf2, w.dc);
        if (!ok)
            break;
    }
    if (trsv_finish(a, L, 2 * a.n))
        refine_update(w);
}

__global__ void refine_reset_kernel(RefineWork w)
{
    if (threadIdx.x == 0) {
        *w.done = 0;
        *w.mode = MODE_CSNE;
        w.iters[0] = 0;
        w.iters[1] = 0;
        for (int k = 0; k < 4; ++k)
            w.stats[k] = 0.0;
    }
}

hipError_t launch_refine(const RefineWork &w, int max_iters, hipStream_t s)
{
    hipLaunchKernelGGL(refine_reset_kernel, dim3(1), dim3(64), 0, s, w);
    const int64_t nparts = (w.m + RB - 1) / RB;
    const TrsvArgs a = trsv_args(w.lda, w.n, nullptr, nullptr, w.sync);
    const unsigned g = (unsigned)(2 * a.nb < TS_GRID ? 2 * a.nb : TS_GRID);
    for (int it = 0; it < max_iters; ++it) {
        hipLaunchKernelGGL(resid_kernel<false>, dim3((unsigned)nparts), dim3(RCH * 64), 0, s, w);
        hipLaunchKernelGGL(atr_kernel<false>, dim3((unsigned)w.n), dim3(256), 0, s, w, nparts);
        hipLaunchKernelGGL(refine_step_kernel, dim3(g), dim3(256), 0, s, w, a);
    }
    // final residual r = b - A c at the returned c, ||r||^2, and s = A^T r
    hipLaunchKernelGGL(resid_kernel<true>, dim3((unsigned)nparts), dim3(RCH * 64), 0, s, w);
    hipLaunchKernelGGL(atr_kernel<true>, dim3((unsigned)w.n), dim3(256), 0, s, w, nparts);
    return hipGetLastError();
}

}  // namespace gap
