// Back-substitution R c = (Q^T b)[0:M] (Sec. Theory: c = R^-1 Q^T b, solved as
// a series of back substitutions) and small vector utilities.
#include "kernels.h"

namespace gap {

constexpr int TB = 64;          // rows per block row
constexpr int TS_GRID = 256;    // workgroups of one solve (all co-resident)
// A workgroup waiting for a block row gives up after this many 100 MHz ticks
// (10 s) and reports DST_EDEVICE, so that every wave always exits.
constexpr uint64_t TS_WAIT_TICKS = 1000000000ull;

// Triangular solves with the n x n upper triangle of R (column-major, ld):
// R x = rhs (back substitution, Sec. Theory: c = R^-1 Q^T b) and R^T x = rhs
// (forward substitution, used by the refinement).  R may be stored in FP32
// (TR = float); the arithmetic is FP64.
//
// One launch solves the whole system.  The block rows (64 rows each) are
// numbered in dependency order q = 0 .. nb-1 (the last block row first for
// R x = rhs, the first one first for R^T x = rhs).  A workgroup takes its next
// item from an atomic ticket when it starts it, so items are handed out in
// order to workgroups that are already running: every item a workgroup waits
// on (a smaller q) belongs to a running workgroup, whatever the dispatch order
// of the launch or the other work on the GPU, and the lowest unfinished q can
// always proceed.
//
// The solve is bound by the chain through the diagonal blocks.  A block row adds up the
// products with the earlier block rows in order, wave w taking 16 of each one's 64 values; the
// values are exchanged through xbuf, where a value that is not there yet reads as a
// signalling NaN (no arithmetic result is one), so that one round trip brings both the news
// and the value.  The diagonal block sits in the first wave's registers by then, its rows
// scaled by the reciprocal of their pivots, and takes 64 dependent multiply-adds.
// About 0.5 us per block row: 7 us at n = 500, 17 at n = 2,000 (27 and 80 with flags, a
// workgroup barrier per dependency and cross-lane shuffles in the diagonal block).
// The last workgroup to finish clears xbuf and the ticket for the next solve (the build sets
// them before the first one).  When skip is non-null and *skip != 0 the kernel returns at once.

constexpr unsigned long long X_EMPTY = 0x7FF4DEAD0BADF00Dull;  // a signalling NaN

struct TrsvArgs {
    int64_t ld, n, nb;
    const double *rhs;
    double *x;
    unsigned long long *xbuf;  // [n]
    int32_t *flags;     // [0] = abort; [1] = ticket
    unsigned *counter;  // arrival counter (zero between solves)
    const int32_t *skip;
    int32_t *status;
};

DEV double lane_value(double v, int lane)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffll), lane);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// Lanes 0 .. cnt-1 of a wave wait for p[lane]; false when the wait was abandoned (uniform).
DEV bool wait_values(const TrsvArgs &a, const unsigned long long *p, int cnt, int lane, double *out)
{
    const uint64_t t0 = __builtin_amdgcn_s_memrealtime();
    unsigned long long v = 0;
    for (;;) {
        if (lane < cnt)
            v = __hip_atomic_load(p + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (!__any(lane < cnt && v == X_EMPTY))
            break;
        if (__hip_atomic_load(&a.flags[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0)
            return false;
        if (__builtin_amdgcn_s_memrealtime() - t0 > TS_WAIT_TICKS) {
            if (lane == 0) {
                set_status(a.status, DST_EDEVICE);
                __hip_atomic_store(&a.flags[0], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            return false;
        }
    }
    *out = lane < cnt ? __longlong_as_double((long long)v) : 0.0;
    return true;
}

template <class TR, bool TRANS>
__global__ __launch_bounds__(256, 1) void trsv_fused_kernel(const TR *__restrict__ R, TrsvArgs a)
{
    __shared__ double red[4][TB];
    __shared__ int last_lds, dead;
    __shared__ int32_t ticket_lds;
    if (a.skip && *a.skip)
        return;
    const int t = threadIdx.x, lane = t & 63, grp = t >> 6;
    const int64_t ld = a.ld, n = a.n, nb = a.nb;
    if (t == 0)
        dead = 0;
    auto take = [&]() -> int64_t {
        __syncthreads();  // every thread is done with the previous item's shared state
        if (t == 0)
            ticket_lds = __hip_atomic_fetch_add(&a.flags[1], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        return ticket_lds;
    };
    for (int64_t q = take(); q < nb; q = take()) {
        const int64_t i = TRANS ? q : nb - 1 - q;
        const int64_t b0 = i * TB;
        const int bw = (int)((n - b0) < TB ? (n - b0) : TB);
        const bool in = lane < bw;
        const int64_t row = b0 + (in ? lane : 0);
        // wave grp's 16 columns of dependency qq: (row, j0 + 16 grp + e), or its transpose
        auto load = [&](int64_t qq, double (&v)[16]) {
            const int64_t j0 = (TRANS ? qq : nb - 1 - qq) * TB + 16 * grp;
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int64_t j = j0 + e < n ? j0 + e : n - 1;
                v[e] = (double)(TRANS ? R[row * ld + j] : R[j * ld + row]);
            }
        };
        double rv[16], nx[16];
        if (q > 0)
            load(0, nx);
        // the diagonal block's row of this lane, scaled by 1 / pivot
        double dg[TB], inv = 0.0, rhs = 0.0;
        if (grp == 0) {
            inv = in ? 1.0 / (double)R[row * ld + row] : 0.0;
            rhs = in ? a.rhs[row] : 0.0;
            const int lim = in ? lane : (TRANS ? -1 : TB);
#pragma unroll
            for (int c = 0; c < TB; ++c) {
                const int cc = c < bw ? c : bw - 1;
                const double v = (double)(TRANS ? R[row * ld + b0 + cc] : R[(b0 + cc) * ld + row]);
                dg[c] = (TRANS ? c < lim : c > lim) && c < bw ? v * inv : 0.0;
            }
        }
        double acc = 0.0;
        bool alive = true;
        for (int64_t qq = 0; qq < q; ++qq) {
#pragma unroll
            for (int e = 0; e < 16; ++e)
                rv[e] = nx[e];
            if (qq + 1 < q)
                load(qq + 1, nx);
            const int64_t j0 = (TRANS ? qq : nb - 1 - qq) * TB + 16 * grp;
            const int cnt = (int)(n - j0 < 16 ? (n - j0 > 0 ? n - j0 : 0) : 16);
            double xv;
            alive = wait_values(a, a.xbuf + j0, cnt, lane, &xv);
            if (!alive)
                break;
#pragma unroll
            for (int e = 0; e < 16; ++e)
                acc += rv[e] * lane_value(xv, e);
        }
        if (!alive)
            dead = 1;
        red[grp][lane] = acc;
        __syncthreads();
        if (dead)
            break;
        if (grp == 0) {
            double r = in ? (rhs - ((red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]))) * inv : 0.0;
#pragma unroll
            for (int k = 0; k < TB; ++k) {
                const int c = TRANS ? k : TB - 1 - k;
                r -= dg[c] * lane_value(r, c);
            }
            if (in) {
                __hip_atomic_store(a.xbuf + row, (unsigned long long)__double_as_longlong(r), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
                a.x[row] = r;
            }
        }
    }
    // the last workgroup to finish clears the exchange for the next solve
    if (!arrive_last(a.counter, gridDim.x, &last_lds))
        return;
    for (int64_t k = t; k < n; k += 256)
        a.xbuf[k] = X_EMPTY;
    if (t < 2)
        a.flags[t] = 0;
}

template <class TR, bool TRANS>
static hipError_t trsv_fused(const TR *R, int64_t ld, int64_t n, const double *rhs, double *x, const TrsvSync &sync,
                             const int32_t *skip, hipStream_t s)
{
    TrsvArgs a{};
    a.ld = ld;
    a.n = n;
    a.nb = (n + TB - 1) / TB;
    a.rhs = rhs;
    a.x = x;
    a.flags = sync.flags;
    a.xbuf = sync.xbuf;
    a.counter = sync.counter;
    a.skip = skip;
    a.status = sync.status;
    const unsigned g = (unsigned)(a.nb < TS_GRID ? a.nb : TS_GRID);
    hipLaunchKernelGGL((trsv_fused_kernel<TR, TRANS>), dim3(g), dim3(256), 0, s, R, a);
    return hipGetLastError();
}

__global__ __launch_bounds__(256) void trsv_clear_kernel(TrsvSync sync, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n)
        sync.xbuf[i] = X_EMPTY;
    if (i < 2)
        sync.flags[i] = 0;
}

hipError_t launch_trsv_clear(const TrsvSync &sync, int64_t n, hipStream_t s)
{
    hipLaunchKernelGGL(trsv_clear_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, sync, n);
    return hipGetLastError();
}

hipError_t launch_trsv_upper(const double *R, int64_t ld, int64_t n, const double *rhs, double *c,
                             const TrsvSync &sync, hipStream_t s)
{
    hipError_t e = trsv_fused<double, false>(R, ld, n, rhs, c, sync, nullptr, s);
    if (e != hipSuccess)
        return e;
    return launch_check_finite(c, n, sync.status, s);
}

hipError_t launch_trsv_upper_nc(const double *R, int64_t ld, int64_t n, const double *rhs, double *x,
                                const TrsvSync &sync, hipStream_t s)
{
    return trsv_fused<double, false>(R, ld, n, rhs, x, sync, nullptr, s);
}

hipError_t launch_trsv_upper_t(const double *R, int64_t ld, int64_t n, const double *rhs, double *x,
                               const TrsvSync &sync, hipStream_t s)
{
    return trsv_fused<double, true>(R, ld, n, rhs, x, sync, nullptr, s);
}

hipError_t launch_trsv_upper_f32(const float *R, int64_t ld, int64_t n, const double *rhs, double *x,
                                 const TrsvSync &sync, const int32_t *skip, hipStream_t s)
{
    return trsv_fused<float, false>(R, ld, n, rhs, x, sync, skip, s);
}

hipError_t launch_trsv_upper_t_f32(const float *R, int64_t ld, int64_t n, const double *rhs, double *x,
                                   const TrsvSync &sync, const int32_t *skip, hipStream_t s)
{
    return trsv_fused<float, true>(R, ld, n, rhs, x, sync, skip, s);
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
    release_writes();
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

__global__ void fill_kernel(double *p, int64_t n, double v)
{
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
        p[i] = v;
}

hipError_t launch_fill(double *p, int64_t n, double v, hipStream_t s)
{
    if (n <= 0)
        return hipSuccess;
    int64_t g = (n + 255) / 256;
    if (g > 65536)
        g = 65536;
    hipLaunchKernelGGL(fill_kernel, dim3((unsigned)g), dim3(256), 0, s, p, n, v);
    return hipGetLastError();
}

__global__ void zero_block_kernel(double *A, int64_t lda, int64_t r0, int64_t r1, int64_t c0, int64_t c1)
{
    const int64_t rows = r1 - r0;
    const int64_t total = rows * (c1 - c0);
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (int64_t)gridDim.x * 256) {
        const int64_t c = c0 + i / rows, r = r0 + i % rows;
        A[c * lda + r] = 0.0;
    }
}

hipError_t launch_zero_block(double *A, int64_t lda, int64_t r0, int64_t r1, int64_t c0, int64_t c1,
                             hipStream_t s)
{
    if (r1 <= r0 || c1 <= c0)
        return hipSuccess;
    int64_t g = ((r1 - r0) * (c1 - c0) + 255) / 256;
    if (g > 65536)
        g = 65536;
    hipLaunchKernelGGL(zero_block_kernel, dim3((unsigned)g), dim3(256), 0, s, A, lda, r0, r1, c0, c1);
    return hipGetLastError();
}

__global__ void check_finite_kernel(const double *x, int64_t n, int32_t *status)
{
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
        if (!isfinite(x[i])) {
            set_status(status, DST_ENONFINITE);
            return;
        }
}

hipError_t launch_check_finite(const double *x, int64_t n, int32_t *status, hipStream_t s)
{
    int64_t g = (n + 255) / 256;
    if (g > 1024)
        g = 1024;
    if (g < 1)
        g = 1;
    hipLaunchKernelGGL(check_finite_kernel, dim3((unsigned)g), dim3(256), 0, s, x, n, status);
    return hipGetLastError();
}

}  // namespace gap
