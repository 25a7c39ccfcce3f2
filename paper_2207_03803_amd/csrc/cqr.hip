// Panel factorisation of the blocked Householder QR by shifted CholeskyQR3
// (Fukaya, Kannan, Nakatsukasa, Yamamoto, Yanagisawa 2020), followed by the
// same Householder reconstruction as the TSQR panel (Ballard et al. 2015):
//
//   P = Q1 R1   from the Gram matrix P^T P + s I (shift s = 11 (mk pw + pw (pw+1)) u ||P||_F^2)
//   Q1 = Q2 R2, Q2 = Q R3  (two unshifted Cholesky QR passes)
//   R = S R3 R2 R1 with S and the unit lower Y1 from the LU of Q[0:pw] - S
//   Y (rows below the top block) = Q2 (U R3)^-1,  T = -U S Y1^-T,  tau = diag(T)
//
// so the panel leaves the LAPACK-form representation H = I - Y T Y^T, R above
// the diagonal, exactly as the TSQR panel does.  The intermediate Q's are kept in an FP64
// scratch panel; the factored matrix may be stored in FP32 (arithmetic stays FP64).
//
// The rows are solved with explicit inverses of the factors' 16 x 16 diagonal blocks (solve_rows). Such a
// solve loses the block's condition number times u. The blocks of R1 may be as ill-conditioned as P,
// and those of R2 up to about u^-1/2 (beyond, its Cholesky fails and the panel is refused), so there
// each block's solution is refined once. R3 is the identity up to what R2's pass leaves, the
// pivots of U lie between 1 and 2, and Y1 is unit lower with entries of at most 1. Orthogonality and
// backward error of panels of condition 1 to 1e13, Kahan's matrices among them, are those of row
// substitution (464 x 64: 31 to 43 u and 3 to 5 u; with R2's solves unrefined up to 8 u).
//
// Four launches per panel, each one pass over its rows: the Gram matrix of P; then twice
// a triangular solve of the rows together with the Gram matrix of the result; then the
// last solve, with R, T and tau formed on a workgroup beside it.  The Gram partials of the
// workgroups are summed by the last one of them to arrive (in a fixed order, in two levels
// above 16 workgroups), which then factors the 64 x 64 matrix that the next launch needs.
// Bound by the latency of this chain: at 456 rows 20 + 24 + 44 + 12 us (of the first three, 9
// us each for the Cholesky factorisation, 13 for the LU, 4 for an arrival and the sum), 387
// us with twelve launches and chains of 64 steps on one wave; at 16,000 rows in FP32 storage 37 + 44 +
// 62 + 13 (8 us more for the rows' loads, 10 for the second level of sums).  Workgroups of 256
// threads and 64-row steps took 41 + 47 + 70 + 12 there, without the second pass's refinement (4 us).
#include "kernels.h"
#include "small64.h"

namespace gap {

constexpr int CB = QR_NB;        // panel width bound (64)
static_assert(CB == S64, "panel blocks");
constexpr int CQ_NT = 512;       // threads of a workgroup; the 64 x 64 factorisations take the first 256
constexpr int CQ_ROWS = CQ_NT / 4;  // rows per workgroup and step (16 per wave)
constexpr int DT = CQ_ROWS + 2;  // LDS row stride of the transposed tile (its reads are free of bank conflicts)
constexpr int CQ_GRP = 16;       // workgroups of one first-level sum
constexpr int NENT = NBLK * BLK / CQ_NT;  // entries of a partial Gram matrix per thread
static_assert(CQ_WGS * NBLK * BLK == CQ_PART && CQ_WGS / CQ_GRP < CQ_COUNTERS, "partials and counters");
static_assert(NENT * CQ_NT == NBLK * BLK, "whole entries");

enum CqStep { CQ_GRAM, CQ_PASS1, CQ_PASS2, CQ_PASS3 };

struct CqArgs {
    QrWork w;
    int64_t j0, rows, chunk;  // panel column, its rows, rows per workgroup (64, or a multiple of CQ_ROWS)
    int pw;
    double shift;
    double *Tout;
};

struct CqLds {
    double tile[S64 * DT];  // the rows' transposed tile; then the 64 x 64 matrix being factored
    double B[S64][DL];      // the packed triangle; then Q_top and its LU
    double T[4][16][17];
    double sg[S64];
    int flag, ok;
    DEV double (*A())[DL] { return reinterpret_cast<double (*)[DL]>(tile); }
};
static_assert(PACK <= S64 * DL, "a packed triangle fits a matrix buffer");

// Rows r0 + 16 wave + r of the panel, columns 16 c + 4 e + g (zero outside).
template <class T>
DEV void load_rows(d4 (&y)[4], const T *src, int64_t ld, int64_t row, int64_t rows, int pw)
{
    const int g = (threadIdx.x & 63) >> 4;
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int col = 16 * c + 4 * e + g;
            y[c][e] = (col < pw && row < rows) ? (double)src[col * ld + row] : 0.0;
        }
}

template <class T>
DEV void store_rows(const d4 (&y)[4], T *dst, int64_t ld, int64_t row, int64_t r0, int64_t rows, int pw)
{
    const int g = (threadIdx.x & 63) >> 4;
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int col = 16 * c + 4 * e + g;
            if (col < pw && row >= r0 && row < rows)
                dst[col * ld + row] = (T)y[c][e];
        }
}

// Sum of the workgroups' partial Gram blocks in the last workgroup to arrive: entry
// t + CQ_NT q in v[q].  True there.  All loads of a group are in flight together.
DEV bool sum_partials(double *part, unsigned *counters, double (&v)[NENT], int *flag)
{
    const int t = threadIdx.x, n = (int)gridDim.x, ch = (int)blockIdx.x;
    auto add = [&](int first, int count, int step) {
        double x[CQ_GRP][NENT];
#pragma unroll
        for (int q = 0; q < CQ_GRP; ++q)
#pragma unroll
            for (int i = 0; i < NENT; ++i)
                x[q][i] = q < count ? part[(int64_t)(first + q * step) * (NBLK * BLK) + i * CQ_NT + t] : 0.0;
#pragma unroll
        for (int i = 0; i < NENT; ++i) {
            v[i] = 0.0;
#pragma unroll
            for (int q = 0; q < CQ_GRP; ++q)
                v[i] += x[q][i];
        }
    };
    if (n <= CQ_GRP) {
        if (!arrive_last(counters, n, flag))
            return false;
        add(0, n, 1);
        return true;
    }
    const int grp = ch / CQ_GRP, ngrp = (n + CQ_GRP - 1) / CQ_GRP;
    const int g0 = grp * CQ_GRP, gn = (n - g0) < CQ_GRP ? n - g0 : CQ_GRP;
    if (!arrive_last(counters + 1 + grp, gn, flag))
        return false;
    add(g0, gn, 1);
#pragma unroll
    for (int i = 0; i < NENT; ++i)
        part[(int64_t)g0 * (NBLK * BLK) + i * CQ_NT + t] = v[i];
    if (!arrive_last(counters, ngrp, flag))
        return false;
    add(0, ngrp, CQ_GRP);
    return true;
}
static_assert(CQ_WGS / CQ_GRP <= CQ_GRP, "second level");

// The summed Gram matrix into L.A() (upper blocks; identity beyond pw, shift_coef * trace on
// the diagonal); 256 threads carry on, the others have returned false.
DEV bool place_gram(const double (&v)[NENT], int pw, double shift_coef, CqLds &L)
{
    const int t = threadIdx.x;
    double(*A)[DL] = L.A();
#pragma unroll
    for (int q = 0; q < NENT; ++q) {
        const int idx = (q * CQ_NT + t) >> 8, c = blk_col(idx), b = idx - c * (c + 1) / 2;
        const int i = 16 * b + ((t >> 4) & 15), l = 16 * c + (t & 15);
        A[i][l] = (i < pw && l < pw) ? v[q] : (i == l ? 1.0 : 0.0);
    }
    if (t == 0)
        L.ok = 1;
    __syncthreads();
    if (t >= 256)
        return false;
    if (shift_coef != 0.0) {
        if (t < 64) {
            const double d = (t < pw) ? A[t][t] : 0.0;
            const double tr = wave_sum(d);
            if (t < pw)
                A[t][t] = d + shift_coef * tr;
        }
        __syncthreads();
    }
    return true;
}

DEV void copy_pack(double *dst, const double *src)
{
    static_assert(PACK % CQ_NT == 0, "whole rounds");
    double v[PACK / CQ_NT];
#pragma unroll
    for (int q = 0; q < PACK / CQ_NT; ++q)
        v[q] = src[q * CQ_NT + threadIdx.x];
#pragma unroll
    for (int q = 0; q < PACK / CQ_NT; ++q)
        dst[q * CQ_NT + threadIdx.x] = v[q];
    __syncthreads();
}

// Once R3 = chol(G) is in L.A() and packed in L.B, with this wave's rows of Q2 in y: Q_top =
// Q2[0:pw] R3^-1, the LU of Q_top - S, and U R3 for the last pass.  LU, R3 and S go to cq_G
// for panel_rest.
DEV void panel_top(const CqArgs &a, CqLds &L, d4 (&y)[4])
{
    const QrWork &w = a.w;
    const int pw = a.pw, t = threadIdx.x, lane = t & 63, wave = t >> 6, g = lane >> 4, r = lane & 15;
    double(*A)[DL] = L.A();
    solve_rows<false>(y, &L.B[0][0]);
    __syncthreads();
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e)
            L.B[16 * wave + r][16 * c + 4 * e + g] = y[c][e];
    __syncthreads();
    lu64_signs(L.B, L.sg, pw);
#pragma unroll
    for (int q = 0; q < CB * CB / 256; ++q) {
        const int e = q * 256 + t;
        w.cq_G[CB * CB + e] = L.B[e >> 6][e & 63];
        w.cq_G[2 * CB * CB + e] = A[e >> 6][e & 63];
    }
    if (t < CB)
        w.cq_G[3 * CB * CB + t] = L.sg[t];
    d4 ur[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        const int idx = wave + 4 * q;
        if (idx >= NBLK)
            break;
        const int c = blk_col(idx), b = idx - c * (c + 1) / 2;
        ur[q] = upper_product_block(
            b, c, [&](int i, int k) { return i <= k ? L.B[i][k] : 0.0; }, [&](int k, int j) { return A[k][j]; });
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        const int idx = wave + 4 * q;
        if (idx >= NBLK)
            break;
        const int c = blk_col(idx), b = idx - c * (c + 1) / 2;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int i = 16 * b + g + 4 * e, j = 16 * c + r;
            A[i][j] = (i < pw && j < pw) ? ur[q][e] : (i == j ? 1.0 : 0.0);
        }
    }
    __syncthreads();
    pack_upper([&](int i, int j) { return A[i][j]; }, w.cq_R + 3 * CB * CB, L.T);
}

// What the last pass does not wait for, on a workgroup of its own beside it: R = S R3 (R2 R1)
// and Y1 into the panel's top block, the compact-WY T = -U S Y1^-T, and tau.
template <class T>
DEV void panel_rest(const CqArgs &a, CqLds &L)
{
    const QrWork &w = a.w;
    const int pw = a.pw, t = threadIdx.x, lane = t & 63, wave = t >> 6, g = lane >> 4, r = lane & 15;
    double(*A)[DL] = L.A();
    const double *R21 = w.cq_R + 2 * CB * CB;
    double lu[CB * CB / CQ_NT], r3[CB * CB / CQ_NT];
#pragma unroll
    for (int q = 0; q < CB * CB / CQ_NT; ++q) {
        lu[q] = w.cq_G[CB * CB + q * CQ_NT + t];
        r3[q] = w.cq_G[2 * CB * CB + q * CQ_NT + t];
    }
    d4 r21[3][4];  // the blocks of R2 R1 that this wave's products take
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        const int idx = wave + 4 * q;
        if (wave < 4 && idx < NBLK) {
            const int c = blk_col(idx), b = idx - c * (c + 1) / 2;
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    r21[q][k][e] = (k >= b && k <= c) ? R21[blk_at(k, c) * BLK + (4 * e + g) * 16 + r] : 0.0;
        }
    }
    if (t < CB)
        L.sg[t] = w.cq_G[3 * CB * CB + t];
#pragma unroll
    for (int q = 0; q < CB * CB / CQ_NT; ++q) {
        const int e = q * CQ_NT + t;
        L.B[e >> 6][e & 63] = lu[q];
        A[e >> 6][e & 63] = r3[q];
    }
    __syncthreads();
    if (t >= 256)
        return;
    T *Ap = ((sizeof(T) == 8) ? reinterpret_cast<T *>(w.A) : reinterpret_cast<T *>(w.A32)) + a.j0 * w.lda + a.j0;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        const int idx = wave + 4 * q;
        if (idx >= NBLK)
            break;
        const int c = blk_col(idx), b = idx - c * (c + 1) / 2;
        d4 rc = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (k >= b && k <= c)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    rc = mfma16(A[16 * b + r][16 * k + 4 * e + g], r21[q][k][e], rc);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int i = 16 * b + g + 4 * e, j = 16 * c + r;
            if (i <= j && j < pw)
                Ap[j * w.lda + i] = (T)(L.sg[i] * rc[e]);
        }
    }
    // Y1 below the diagonal
#pragma unroll
    for (int q = 0; q < CB * CB / 256; ++q) {
        const int e = q * 256 + t, i = e & 63, j = e >> 6;
        if (i > j && i < pw)
            Ap[j * w.lda + i] = (T)L.B[i][j];
    }
    __syncthreads();
    // T = -U S Y1^-T: rows of -U S times the inverse of Y1^T (unit upper)
    double *P1 = L.tile;
    pack_upper([&](int i, int j) { return i == j ? 1.0 : ((j < pw) ? L.B[j][i] : 0.0); }, P1, L.T);
    d4 y[4];
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int i = 16 * wave + r, j = 16 * c + 4 * e + g;
            y[c][e] = (i <= j && j < pw) ? -L.B[i][j] * L.sg[j] : 0.0;
        }
    solve_rows<false>(y, P1);
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int i = 16 * wave + r, j = 16 * c + 4 * e + g;
            const double tv = (i <= j && j < pw) ? y[c][e] : 0.0;
            a.Tout[i * CB + j] = tv;
            if (i == j && i < pw)
                w.tau[a.j0 + i] = tv;
        }
}

// One pass over the panel's rows (see CqStep).  TS: what it reads, TD: what it writes, T: the
// factored matrix's storage.
template <int STEP, class TS, class TD, class T>
__global__ __launch_bounds__(CQ_NT) void cqr_step_kernel(CqArgs a, const TS *src, int64_t lds_, TD *dst, int64_t ldd)
{
    __shared__ CqLds L;
    const QrWork &w = a.w;
    const int pw = a.pw;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, g = lane >> 4, r = lane & 15;
    int64_t wg = blockIdx.x;
    if constexpr (STEP == CQ_PASS3) {
        if (wg == 0) {
            panel_rest<T>(a, L);
            return;
        }
        --wg;
    }
    const int64_t lo = wg * a.chunk;
    const int64_t hi = (lo + a.chunk) < a.rows ? (lo + a.chunk) : a.rows;
    double *P = &L.B[0][0];
    double *pack_in = w.cq_R + (STEP == CQ_PASS1 ? 0 : (STEP == CQ_PASS2 ? 1 : 3)) * CB * CB;
    d4 y[4], nxt[4];
    load_rows(nxt, src, lds_, lo + 16 * wave + r, hi, pw);
    if constexpr (STEP != CQ_GRAM)
        copy_pack(P, pack_in);
    d4 acc[2] = {d4{0.0, 0.0, 0.0, 0.0}, d4{0.0, 0.0, 0.0, 0.0}};  // Gram blocks wave, wave + 8
    for (int64_t r0 = lo; r0 < hi; r0 += CQ_ROWS) {
        const int64_t row = r0 + 16 * wave + r;
#pragma unroll
        for (int c = 0; c < 4; ++c)
            y[c] = nxt[c];
        if (r0 + CQ_ROWS < hi)
            load_rows(nxt, src, lds_, row + CQ_ROWS, hi, pw);
        const int nr = (int)((hi - r0) < CQ_ROWS ? (hi - r0) : CQ_ROWS);
        if (STEP != CQ_GRAM && 16 * wave < nr) {
            solve_rows<STEP != CQ_PASS3>(y, P);
            // the last pass leaves the top block (rows below pw) to the reconstruction
            store_rows(y, dst, ldd, row, STEP == CQ_PASS3 ? (int64_t)pw : (int64_t)0, hi, pw);
        }
        if constexpr (STEP != CQ_PASS3) {
            __syncthreads();  // the previous step's reads of the tile are done
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    L.tile[(16 * c + 4 * e + g) * DT + 16 * wave + r] = y[c][e];
            __syncthreads();
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int idx = wave + 8 * q;
                if (idx < NBLK) {
                    const int c = blk_col(idx), b = idx - c * (c + 1) / 2;
                    const double *Ta = L.tile + (16 * b + r) * DT + g, *Tb = L.tile + (16 * c + r) * DT + g;
                    for (int k = 0; k < nr; k += 64)  // rows past nr are zero
#pragma unroll
                        for (int kk = 0; kk < 64; kk += 4)
                            acc[q] = mfma16(Ta[k + kk], Tb[k + kk], acc[q]);
                }
            }
        }
    }
    if constexpr (STEP != CQ_PASS3) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int idx = wave + 8 * q;
            if (idx < NBLK)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    w.cq_part[(int64_t)blockIdx.x * (NBLK * BLK) + idx * BLK + (g + 4 * e) * 16 + r] = acc[q][e];
        }
        double v[NENT];
        if (!sum_partials(w.cq_part, w.cq_counters, v, &L.flag))
            return;
        if (!place_gram(v, pw, STEP == CQ_GRAM ? a.shift : 0.0, L))
            return;
        if constexpr (STEP == CQ_PASS2)  // the top rows, on their way during the factorisation
            load_rows(y, (const double *)w.cq_S, w.cq_ld, 16 * wave + r, (int64_t)pw, pw);
        double(*A)[DL] = L.A();
        chol64(A, STEP == CQ_PASS2 ? P : w.cq_R + (STEP == CQ_GRAM ? 0 : CB * CB), &L.ok);
        if (t == 0 && !L.ok)
            set_status(w.status, DST_ERANK);
        if constexpr (STEP == CQ_PASS1) {
            // R2 R1 (R1 is the pack this pass solved with, still in P)
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                const int idx = wave + 4 * q;
                if (idx < NBLK) {
                    const int c = blk_col(idx), b = idx - c * (c + 1) / 2;
                    const d4 p = upper_product_block(
                        b, c, [&](int i, int k) { return A[i][k]; },
                        [&](int k, int j) { return P[blk_at(k >> 4, c) * BLK + (k & 15) * 16 + (j & 15)]; });
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        w.cq_R[2 * CB * CB + idx * BLK + (g + 4 * e) * 16 + r] = p[e];
                }
            }
        } else if constexpr (STEP == CQ_PASS2) {
            panel_top(a, L, y);
        }
    }
}

template <class T>
static void cqr_panel(const QrWork &w, int64_t j0, int pw, double *Tout, hipStream_t s)
{
    T *base = ((sizeof(T) == 8) ? reinterpret_cast<T *>(w.A) : reinterpret_cast<T *>(w.A32)) + j0 * w.lda + j0;
    const int64_t mk = w.m - j0;
    CqArgs a{};
    a.w = w;
    a.j0 = j0;
    a.rows = mk;
    a.pw = pw;
    a.chunk = (mk + CQ_WGS - 1) / CQ_WGS;
    // 64 rows per workgroup while one level of sums is enough, else whole steps
    a.chunk = mk <= CQ_GRP * 64 ? 64 : (a.chunk + CQ_ROWS - 1) / CQ_ROWS * CQ_ROWS;
    const double u = 0x1p-53;
    a.shift = 11.0 * ((double)mk * pw + (double)pw * (pw + 1)) * u;
    a.Tout = Tout;
    const dim3 grid((unsigned)((mk + a.chunk - 1) / a.chunk));
    double *S = w.cq_S;
    hipLaunchKernelGGL((cqr_step_kernel<CQ_GRAM, T, T, T>), grid, dim3(CQ_NT), 0, s, a, (const T *)base, w.lda, base,
                       w.lda);
    hipLaunchKernelGGL((cqr_step_kernel<CQ_PASS1, T, double, T>), grid, dim3(CQ_NT), 0, s, a, (const T *)base, w.lda, S,
                       w.cq_ld);
    hipLaunchKernelGGL((cqr_step_kernel<CQ_PASS2, double, double, T>), grid, dim3(CQ_NT), 0, s, a, (const double *)S,
                       w.cq_ld, S, w.cq_ld);
    hipLaunchKernelGGL((cqr_step_kernel<CQ_PASS3, double, T, T>), dim3(grid.x + 1), dim3(CQ_NT), 0, s, a,
                       (const double *)S, w.cq_ld, base, w.lda);
}

void cqr_panel_f64(const QrWork &w, int64_t j0, int pw, double *Tout, hipStream_t s)
{
    cqr_panel<double>(w, j0, pw, Tout, s);
}

void cqr_panel_f32(const QrWork &w, int64_t j0, int pw, double *Tout, hipStream_t s)
{
    cqr_panel<float>(w, j0, pw, Tout, s);
}

}  // namespace gap
