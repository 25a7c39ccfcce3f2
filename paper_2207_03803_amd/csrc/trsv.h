// Triangular solves for one launch of 256-thread workgroups: R x = rhs and R^T x = rhs.
#pragma once

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
// About 2 us per block row: 21 us at n = 500, 68 at n = 2,250 (80 and 340 with flags, a
// workgroup barrier per dependency and cross-lane shuffles in the diagonal block).  R^T x = rhs
// reads a column per lane, 16 bytes at a time (both solves of a refinement step at n = 2,250:
// 178 us with a value at a time, 153).  R starts 16-byte aligned and ld is a multiple of 64.
// The last workgroup to finish clears xbuf and the ticket for the next solve (the build sets
// them before the first one).

constexpr unsigned long long X_EMPTY = 0x7FF4DEAD0BADF00Dull;  // a signalling NaN

struct TrsvArgs {
    int64_t ld, n, nb;
    const double *rhs;
    double *x;
    unsigned long long *xbuf;  // [2 n]: a solve's exchange, and that of a second solve behind it
    int32_t *flags;     // [0] = abort; [1] = ticket
    unsigned *counter;  // arrival counter (zero between solves)
    int32_t *status;
};

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

struct TrsvLds {
    double red[4][TB];
    int last, dead;
    int32_t ticket;
};

// The workgroup's next item, in ticket order.
DEV int64_t take_item(const TrsvArgs &a, TrsvLds &L)
{
    __syncthreads();  // every thread is done with the previous item's shared state
    if (threadIdx.x == 0)
        L.ticket = __hip_atomic_fetch_add(&a.flags[1], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    return L.ticket;
}

// N consecutive entries of a column from a 16-byte aligned one on.
template <int N, class TR>
DEV void load_run(const TR *__restrict__ p, double (&v)[N])
{
    constexpr int W = 16 / sizeof(TR);
    typedef TR VR __attribute__((ext_vector_type(W)));
#pragma unroll
    for (int e = 0; e < N; e += W) {
        const VR x = *reinterpret_cast<const VR *>(p + e);
#pragma unroll
        for (int k = 0; k < W; ++k)
            v[e + k] = (double)x[k];
    }
}

// Item q of a solve: block row q in dependency order.  The right-hand side is rhs, or (null) the
// values that an earlier solve in the same launch leaves in rhs_buf.  The solution goes to xbuf
// and x.  False when a wait was abandoned.
template <class TR, bool TRANS>
DEV bool trsv_item(const TR *__restrict__ R, const TrsvArgs &a, TrsvLds &L, int64_t q, const double *rhs_ptr,
                   const unsigned long long *rhs_buf, unsigned long long *xbuf, double *x)
{
    const int t = threadIdx.x, lane = t & 63, grp = t >> 6;
    const int64_t ld = a.ld, n = a.n, nb = a.nb;
    const int64_t i = TRANS ? q : nb - 1 - q;
    const int64_t b0 = i * TB;
    const int bw = (int)((n - b0) < TB ? (n - b0) : TB);
    const bool in = lane < bw;
    const int64_t row = b0 + (in ? lane : 0);
    // wave grp's 16 columns of dependency qq: (row, j0 + 16 grp + e), or its transpose
    auto load = [&](int64_t qq, double (&v)[16]) {
        const int64_t j0 = (TRANS ? qq : nb - 1 - qq) * TB + 16 * grp;
        if constexpr (TRANS) {
            load_run(R + row * ld + j0, v);  // an earlier block row: all below n
        } else {
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int64_t j = j0 + e < n ? j0 + e : n - 1;
                v[e] = (double)R[j * ld + row];
            }
        }
    };
    double rv[16], nx[16];
    if (q > 0)
        load(0, nx);
    // the diagonal block's row of this lane, scaled by 1 / pivot
    double dg[TB], inv = 0.0, rhs = 0.0;
    if (grp == 0) {
        inv = in ? 1.0 / (double)R[row * ld + row] : 0.0;
        if (rhs_ptr)
            rhs = in ? rhs_ptr[row] : 0.0;
        const int lim = in ? lane : (TRANS ? -1 : TB);
        if constexpr (TRANS)
            load_run(R + row * ld + b0, dg);  // (rows past n are part of the column)
#pragma unroll
        for (int c = 0; c < TB; ++c) {
            if constexpr (!TRANS)
                dg[c] = (double)R[(b0 + (c < bw ? c : bw - 1)) * ld + row];
            dg[c] = (TRANS ? c < lim : c > lim) && c < bw ? dg[c] * inv : 0.0;
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
        alive = wait_values(a, xbuf + j0, cnt, lane, &xv);
        if (!alive)
            break;
#pragma unroll
        for (int e = 0; e < 16; ++e)
            acc += rv[e] * readlane_d(xv, e);
    }
    if (alive && !rhs_ptr && grp == 0)
        alive = wait_values(a, rhs_buf + b0, bw, lane, &rhs);
    if (!alive)
        L.dead = 1;
    L.red[grp][lane] = acc;
    __syncthreads();
    if (L.dead)
        return false;
    if (grp == 0) {
        double r = in ? (rhs - ((L.red[0][lane] + L.red[1][lane]) + (L.red[2][lane] + L.red[3][lane]))) * inv : 0.0;
#pragma unroll
        for (int k = 0; k < TB; ++k) {
            const int c = TRANS ? k : TB - 1 - k;
            r -= dg[c] * readlane_d(r, c);
        }
        if (in) {
            __hip_atomic_store(xbuf + row, (unsigned long long)__double_as_longlong(r), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
            x[row] = r;
        }
    }
    return true;
}

// The last workgroup to finish (true there) clears the exchange for the next launch.
DEV bool trsv_finish(const TrsvArgs &a, TrsvLds &L, int64_t used)
{
    if (!arrive_last(a.counter, gridDim.x, &L.last))
        return false;
    for (int64_t k = threadIdx.x; k < used; k += 256)
        a.xbuf[k] = X_EMPTY;
    if (threadIdx.x < 2)
        a.flags[threadIdx.x] = 0;
    return true;
}

inline TrsvArgs trsv_args(int64_t ld, int64_t n, const double *rhs, double *x, const TrsvSync &sync)
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
    a.status = sync.status;
    return a;
}

}  // namespace gap
