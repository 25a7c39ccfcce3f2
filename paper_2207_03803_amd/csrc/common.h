// Shared device helpers of the GAP fit library (gfx950 / CDNA4 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#define DEV __device__ __forceinline__

typedef double d4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));

// Device status word values (same numbering as gap_status).
enum : int32_t {
    DST_OK = 0,
    DST_EINVAL = 1,
    DST_ENOTPD = 3,
    DST_ENONFINITE = 4,
    DST_ENOCONV = 5,
    DST_EDEVICE = 6,  // a device-side wait was abandoned
    DST_ERANK = 8,    // a QR panel's Gram matrix lost positive definiteness
};

// Record the first failure seen on the device; later ones do not overwrite it.
DEV void set_status(int32_t *status, int32_t code)
{
    atomicCAS(reinterpret_cast<int *>(status), 0, code);
}

// ---------------------------------------------------------------------------
// "Last workgroup" completion pattern: every workgroup stores its partial results, then one
// arrival counter tells the last one that all partials are visible.  The counter is reset by
// that last workgroup, ready for the next launch that uses it.  Returns true in every thread of
// the last workgroup.  Callers need no fence of their own, on either side:
//   * each wave first waits until its own stores have reached the L2 (a barrier alone does not
//     wait for them, and thread 0's wait counts the stores of its own wave only);
//   * thread 0's release then writes the XCD's L2 back before the counter is raised, for the
//     workgroups of other XCDs;
//   * each wave of the last workgroup drops what its caches may hold of the partials.
// ---------------------------------------------------------------------------
DEV bool arrive_last(unsigned *counter, unsigned nblocks, int *flag_lds)
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned prev = __hip_atomic_fetch_add(counter, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
        int last = (prev == nblocks - 1);
        if (last)
            __hip_atomic_store(counter, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        *flag_lds = last;
    }
    __syncthreads();
    const bool last = *flag_lds != 0;
    if (last)
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    return last;
}

// Value of v in lane `lane` (uniform) of the wave.
DEV double readlane_d(double v, int lane)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffll), lane);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// Wave-wide sum with a fixed butterfly order (deterministic).
DEV double wave_sum(double v)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1)
        v += __shfl_xor(v, o, 64);
    return v;
}

// Row / column (within the workgroup tile) of element e of block (i, j) of a KTile's FP64
// accumulators.
template <class S>
DEV int acc_row(int wm, int i, int lane, int e)
{
    return wm * S::TM + i * 16 + (lane >> 4) + 4 * e;
}
template <class S>
DEV int acc_col(int wn, int j, int lane, int e)
{
    return wn * S::TN + j * 16 + (lane & 15);
}

// ---------------------------------------------------------------------------
// Tile products staged in 16-byte units, FP64 (v_mfma_f64_16x16x4_f64) or FP32
// (v_mfma_f32_16x16x4_f32).  A unit is V consecutive elements (two doubles or four floats);
// lane l = 16 g + r of a fragment read takes one unit, which serves V MFMAs.
//
// Rows contiguous along k (KTile):  acc(m, n) += sum_k A[m][k] B[n][k].  LDS holds a stage
// row by row, A's BM rows then B's BN; unit u of a row sits at slot u ^ swz(row), so that the
// eight lanes of a read that share u take eight different bank groups.  Lane group g takes
// unit g of each four: its V elements are one k of each of V MFMAs (A and B permute k alike).
//
// Stages are filled by direct global-to-LDS loads: no VGPRs, no LDS stores, and the loads of
// the next stage run during the MFMAs of the current one.  Measured in FP64 (262144 x 8192 x
// 400, the loop alone): 68.9 TFLOP/s with 256 x 64 tiles of 4 waves, 71.7 with 128 x 128 of 8
// waves, 68.9 with 64 x 64 of 4; K-major stages filled through registers, 55.
// ---------------------------------------------------------------------------
typedef double d2 __attribute__((ext_vector_type(2)));

template <class T>
struct Unit;
template <>
struct Unit<double> {
    typedef d2 type;
    typedef d4 acc;
    static constexpr int V = 2;
    DEV static acc mfma(double a, double b, acc c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
    DEV static int acc_m(int g, int e) { return g + 4 * e; }  // row of accumulator element e (column: r)
};
template <>
struct Unit<float> {
    typedef f4 type;
    typedef f4 acc;
    static constexpr int V = 4;
    DEV static acc mfma(float a, float b, acc c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
    DEV static int acc_m(int g, int e) { return 4 * g + e; }
};

template <class T, int BM_, int BN_, int U_, int WM_, int WN_>
struct KTile {
    typedef T elem;
    typedef typename Unit<T>::type unit;
    typedef typename Unit<T>::acc acc4;
    static constexpr int V = Unit<T>::V;
    static constexpr int BM = BM_, BN = BN_, U = U_, BK = U * V, WM = WM_, WN = WN_;
    static constexpr int NT = WM * WN * 64;
    static constexpr int TM = BM / WM, TN = BN / WN, FM = TM / 16, FN = TN / 16;
    static constexpr int UNITS = (BM + BN) * U;         // units of a stage
    static constexpr int LPT = (UNITS + NT - 1) / NT;   // units per thread (the last round may be partial)
    static_assert(U == 4 || U == 8, "4 or 8 units per row");
    static_assert(TM % 16 == 0 && TN % 16 == 0 && UNITS % 64 == 0, "whole 16x16 blocks and wave loads");
    // rows r and r + 2 (U = 4) or r + 1 (U = 8) start in the same bank group
    DEV static int swz(int row) { return U == 8 ? (row & 7) : ((row >> 1) & 3); }
    // does this thread's wave load a unit in round i?
    DEV static bool has(int i) { return UNITS % NT == 0 || i * NT + wave0() < UNITS; }
    DEV static int wave0() { return __builtin_amdgcn_readfirstlane((int)(threadIdx.x & ~63u)); }
    DEV static int unit_row(int i) { return (i * NT + (int)threadIdx.x) / U; }
    DEV static int unit_k(int i) { return V * (((i * NT + (int)threadIdx.x) % U) ^ swz(unit_row(i))); }
};

template <class T>
DEV void load_lds16(const T *g, typename Unit<T>::type *l)
{
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)g,
                                     (__attribute__((address_space(3))) void *)l, 16, 0, 0);
}

// A full stage (k0 + BK <= d) at src[i] + k0, 16-byte aligned (src[i] points at the
// thread's unit of round i).  Waits are the caller's (ktile_wait).
template <class S>
DEV void ktile_issue(const typename S::elem *const (&src)[S::LPT], int64_t k0, typename S::unit *stage)
{
#pragma unroll
    for (int i = 0; i < S::LPT; ++i)
        if (S::has(i))
            load_lds16(src[i] + k0, stage + i * S::NT + S::wave0());
}

// The same stage through registers (rows that are not 16-byte aligned).
template <class S>
DEV void ktile_load_full(const typename S::elem *const (&src)[S::LPT], int64_t k0, typename S::unit (&r)[S::LPT])
{
#pragma unroll
    for (int i = 0; i < S::LPT; ++i)
        if (S::has(i))
            __builtin_memcpy(&r[i], src[i] + k0, 16);
}

// A ragged last stage through registers, k checked against d.
template <class S>
DEV void ktile_load(const typename S::elem *const (&src)[S::LPT], int64_t k0, int64_t d,
                    typename S::unit (&r)[S::LPT])
{
#pragma unroll
    for (int i = 0; i < S::LPT; ++i)
        if (S::has(i)) {
            const int64_t k = k0 + S::unit_k(i);
            const typename S::elem *p = src[i] + k0;
#pragma unroll
            for (int v = 0; v < S::V; ++v)
                r[i][v] = k + v < d ? p[v] : typename S::elem(0);
        }
}
template <class S>
DEV void ktile_store(const typename S::unit (&r)[S::LPT], typename S::unit *stage)
{
#pragma unroll
    for (int i = 0; i < S::LPT; ++i)
        if (S::has(i))
            stage[i * S::NT + threadIdx.x] = r[i];
}

// This wave's part of the stage is in LDS, and after the barrier everyone's.
DEV void ktile_wait()
{
    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
    __syncthreads();
}

// The wave's fragments of a whole stage.  They are read before the next stage's direct
// loads are issued: the compiler takes any LDS read after one to depend on it and would
// wait for the load there.
template <class S>
struct KFrag {
    typename S::unit a[S::U / 4][S::FM], b[S::U / 4][S::FN];
};

template <class S>
DEV void ktile_read(const typename S::unit *stage, KFrag<S> &f, int wm, int wn, int lane)
{
    const int rl = lane & 15, g = lane >> 4;
    const typename S::unit *Sa = stage + (wm * S::TM + rl) * S::U, *Sb = stage + (S::BM + wn * S::TN + rl) * S::U;
#pragma unroll
    for (int q = 0; q < S::U / 4; ++q) {
        const int u = (4 * q + g) ^ S::swz(rl);
#pragma unroll
        for (int i = 0; i < S::FM; ++i)
            f.a[q][i] = Sa[i * 16 * S::U + u];
#pragma unroll
        for (int j = 0; j < S::FN; ++j)
            f.b[q][j] = Sb[j * 16 * S::U + u];
    }
}

template <class S>
DEV void ktile_mma(const KFrag<S> &f, typename S::acc4 (&acc)[S::FM][S::FN])
{
#pragma unroll
    for (int q = 0; q < S::U / 4; ++q)
#pragma unroll
        for (int h = 0; h < S::V; ++h)
#pragma unroll
            for (int i = 0; i < S::FM; ++i)
#pragma unroll
                for (int j = 0; j < S::FN; ++j)
                    acc[i][j] = Unit<typename S::elem>::mfma(f.a[q][i][h], f.b[q][j][h], acc[i][j]);
}

template <class S>
DEV void ktile_zero(typename S::acc4 (&acc)[S::FM][S::FN])
{
#pragma unroll
    for (int i = 0; i < S::FM; ++i)
#pragma unroll
        for (int j = 0; j < S::FN; ++j)
            acc[i][j] = typename S::acc4{0, 0, 0, 0};
}

// acc += the product over k = 0 .. d-1; lds: two stages (2 * S::UNITS units).  direct:
// every src[i] is 16-byte aligned.  Starts with a barrier (LDS may still be in use) and
// ends with one.
template <class S>
DEV void ktile_product(typename S::acc4 (&acc)[S::FM][S::FN], typename S::unit *lds,
                       const typename S::elem *const (&src)[S::LPT], int d, bool direct)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = wave / S::WN, wn = wave % S::WN;
    const int nk = (d + S::BK - 1) / S::BK, nkf = direct ? d / S::BK : 0;
    typename S::unit r[S::LPT];
    __syncthreads();
    if (nkf > 0) {
        ktile_issue<S>(src, 0, lds);
    } else {
        ktile_load<S>(src, 0, d, r);
        ktile_store<S>(r, lds);
    }
    int kt = 0;
    KFrag<S> f;
    for (; kt + 1 < nkf; ++kt) {
        ktile_wait();
        ktile_read<S>(lds + (kt & 1) * S::UNITS, f, wm, wn, lane);
        ktile_issue<S>(src, (kt + 1) * S::BK, lds + ((kt + 1) & 1) * S::UNITS);
        ktile_mma<S>(f, acc);
    }
    for (; kt + 1 < d / S::BK; ++kt) {  // full stages through registers
        ktile_wait();
        ktile_load_full<S>(src, (kt + 1) * S::BK, r);
        ktile_read<S>(lds + (kt & 1) * S::UNITS, f, wm, wn, lane);
        ktile_mma<S>(f, acc);
        ktile_store<S>(r, lds + ((kt + 1) & 1) * S::UNITS);
    }
    for (; kt < nk; ++kt) {  // the last full stage and a ragged one
        ktile_wait();
        const bool more = kt + 1 < nk;
        if (more)
            ktile_load<S>(src, (kt + 1) * S::BK, d, r);
        ktile_read<S>(lds + (kt & 1) * S::UNITS, f, wm, wn, lane);
        ktile_mma<S>(f, acc);
        if (more)
            ktile_store<S>(r, lds + ((kt + 1) & 1) * S::UNITS);
    }
    __syncthreads();
}

// The same product where some stages need work on the way (masks): stages [km, nfull) are
// copied as they are, load(kt, i) gives this thread's unit of round i of the others.
template <class S, class LOAD>
DEV void ktile_product_masked(typename S::acc4 (&acc)[S::FM][S::FN], typename S::unit *lds,
                              const typename S::elem *const (&src)[S::LPT], int nk, int km, int nfull, LOAD load)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = wave / S::WN, wn = wave % S::WN;
    typename S::unit r[S::LPT];
    KFrag<S> f;
    auto fetch = [&](int kt) {
#pragma unroll
        for (int i = 0; i < S::LPT; ++i)
            if (S::has(i))
                r[i] = load(kt, i);
    };
    auto step = [&](int kt) {
        ktile_wait();
        ktile_read<S>(lds + (kt & 1) * S::UNITS, f, wm, wn, lane);
    };
    int kt = 0;
    if (km <= 0 && nfull > 0) {
        ktile_issue<S>(src, 0, lds);
    } else {
        fetch(0);
        ktile_store<S>(r, lds);
    }
    for (; kt + 1 < km && kt + 1 < nk; ++kt) {
        step(kt);
        fetch(kt + 1);
        ktile_mma<S>(f, acc);
        ktile_store<S>(r, lds + ((kt + 1) & 1) * S::UNITS);
    }
    for (; kt + 1 < nfull; ++kt) {
        step(kt);
        ktile_issue<S>(src, (int64_t)(kt + 1) * S::BK, lds + ((kt + 1) & 1) * S::UNITS);
        ktile_mma<S>(f, acc);
    }
    for (; kt < nk; ++kt) {
        step(kt);
        if (kt + 1 < nk)
            fetch(kt + 1);
        ktile_mma<S>(f, acc);
        if (kt + 1 < nk)
            ktile_store<S>(r, lds + ((kt + 1) & 1) * S::UNITS);
    }
}

// ---------------------------------------------------------------------------
// Operands contiguous along their own index (MTile):  acc(m, n) += sum_p A[p][m] B[p][n].
// LDS holds BK rows p of BM + BN elements; a lane's unit is V consecutive m (or n) at p =
// 4 kk + g, one of each of V 16-wide blocks: block V ii + h of the wave's tile holds the
// indices 16 V ii + V r + h.  (So a lane's accumulators of V neighbouring column blocks are V
// consecutive n.)
// ---------------------------------------------------------------------------
template <class T, int BM_, int BN_, int BK_, int WM_, int WN_>
struct MTile {
    typedef T elem;
    typedef typename Unit<T>::type unit;
    typedef typename Unit<T>::acc acc4;
    static constexpr int V = Unit<T>::V;
    static constexpr int BM = BM_, BN = BN_, BK = BK_, WM = WM_, WN = WN_;
    static constexpr int NT = WM * WN * 64;
    static constexpr int TM = BM / WM, TN = BN / WN, FM = TM / 16, FN = TN / 16;
    static constexpr int UA = BM / V, UR = (BM + BN) / V;  // units of A, and of a whole row
    static constexpr int UNITS = BK * UR;
    static constexpr int LPT = (UNITS + NT - 1) / NT;
    static_assert(TM % (16 * V) == 0 && TN % (16 * V) == 0 && BK % 4 == 0 && UNITS % NT == 0, "whole units");
    DEV static int unit_p(int i) { return (i * NT + (int)threadIdx.x) / UR; }
    DEV static int unit_x(int i) { return (i * NT + (int)threadIdx.x) % UR; }  // < UA: A's unit, else B's
    DEV static int wave0() { return __builtin_amdgcn_readfirstlane((int)(threadIdx.x & ~63u)); }
    // index within the workgroup's tile of accumulator row (i, e) and of column block j
    DEV static int row(int wm, int i, int g, int e) { return wm * TM + 16 * V * (i / V) + V * Unit<T>::acc_m(g, e) + i % V; }
    DEV static int col(int wn, int j, int r) { return wn * TN + 16 * V * (j / V) + V * r + j % V; }
};

template <class S>
DEV void mtile_mma(typename S::acc4 (&acc)[S::FM][S::FN], typename S::unit (&fa)[S::BK / 4][S::FM / S::V],
                   typename S::unit (&fb)[S::BK / 4][S::FN / S::V])
{
#pragma unroll
    for (int k = 0; k < S::BK / 4; ++k)
#pragma unroll
        for (int i = 0; i < S::FM; ++i)
#pragma unroll
            for (int j = 0; j < S::FN; ++j)
                acc[i][j] = Unit<typename S::elem>::mfma(fa[k][i / S::V][i % S::V], fb[k][j / S::V][j % S::V], acc[i][j]);
}

// acc += the product over nk stages: [0, nfull) are copied as they are from src[i] (this
// thread's unit of round i) + kt * step[i], load(kt, i) gives the units of the others.
template <class S, class LOAD>
DEV void mtile_product(typename S::acc4 (&acc)[S::FM][S::FN], typename S::unit *lds, int nk, int nfull,
                       const typename S::elem *(&src)[S::LPT], const int64_t (&step)[S::LPT], LOAD load)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, rl = lane & 15, g = lane >> 4;
    const int wm = wave / S::WN, wn = wave % S::WN;
    typename S::unit r[S::LPT];
    typename S::unit fa[S::BK / 4][S::FM / S::V], fb[S::BK / 4][S::FN / S::V];
    auto fetch = [&](int kt) {
#pragma unroll
        for (int i = 0; i < S::LPT; ++i)
            r[i] = load(kt, i);
    };
    auto put = [&](int kt) {
#pragma unroll
        for (int i = 0; i < S::LPT; ++i)
            lds[(kt & 1) * S::UNITS + i * S::NT + threadIdx.x] = r[i];
    };
    auto issue = [&](int kt) {  // in order: src moves along
#pragma unroll
        for (int i = 0; i < S::LPT; ++i) {
            load_lds16(src[i], lds + (kt & 1) * S::UNITS + i * S::NT + S::wave0());
            src[i] += step[i];
        }
    };
    auto read = [&](int kt) {
        ktile_wait();
        const typename S::unit *st = lds + (kt & 1) * S::UNITS;
#pragma unroll
        for (int k = 0; k < S::BK / 4; ++k) {
#pragma unroll
            for (int i = 0; i < S::FM / S::V; ++i)
                fa[k][i] = st[(4 * k + g) * S::UR + wm * S::TM / S::V + 16 * i + rl];
#pragma unroll
            for (int j = 0; j < S::FN / S::V; ++j)
                fb[k][j] = st[(4 * k + g) * S::UR + S::UA + wn * S::TN / S::V + 16 * j + rl];
        }
    };
    int kt = 0;
    if (nfull > 0) {
        issue(0);
    } else {
        fetch(0);
        put(0);
    }
    for (; kt + 1 < nfull; ++kt) {
        read(kt);
        issue(kt + 1);
        mtile_mma<S>(acc, fa, fb);
    }
    for (; kt < nk; ++kt) {
        read(kt);
        if (kt + 1 < nk)
            fetch(kt + 1);
        mtile_mma<S>(acc, fa, fb);
        if (kt + 1 < nk)
            put(kt + 1);
    }
}

// 16-byte alignment of rows of d doubles at p.
DEV bool rows_aligned16(const double *p, int64_t d)
{
    return (reinterpret_cast<uintptr_t>(p) & 15) == 0 && (d & 1) == 0;
}

// Integer power by repeated multiplication, p = g^zeta (zeta >= 1).
DEV double ipow(double g, int zeta)
{
    double p = g;
    for (int z = 1; z < zeta; ++z)
        p *= g;
    return p;
}

// Map a hardware workgroup id to a logical id so that consecutive logical ids
// run on the same XCD (workgroups are dispatched to the 8 XCDs round-robin).
// total_pad must be a multiple of 8.
DEV int64_t xcd_remap(int64_t w, int64_t total_pad)
{
    const int64_t per = total_pad >> 3;
    return (w & 7) * per + (w >> 3);
}
