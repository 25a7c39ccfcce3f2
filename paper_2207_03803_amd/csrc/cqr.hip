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
// Four launches per panel, each one pass over its rows: the Gram matrix of P; then twice
// a triangular solve of the rows together with the Gram matrix of the result; then the
// last solve.  The Gram partials of the workgroups are summed by the last one of them to
// arrive (in a fixed order, in two levels above 16 workgroups), which then factors the
// 64 x 64 matrix that the next launch needs.  A panel of a few hundred to a few thousand
// rows is bound by the latency of this chain: 456 rows take 23 + 30 + 59 + 8 us (387 us with
// twelve launches, each 64 x 64 factorisation a chain of 64 steps on one wave), 7,000 rows
// 156 us (400).
#include "kernels.h"
#include "small64.h"

namespace gap {

constexpr int CB = QR_NB;        // panel width bound (64)
static_assert(CB == S64, "panel blocks");
constexpr int CQ_ROWS = 64;      // rows per workgroup and step (16 per wave)
constexpr int CQ_GRP = 16;       // workgroups of one first-level sum
static_assert(CQ_WGS * NBLK * BLK == CQ_PART && CQ_WGS / CQ_GRP < CQ_COUNTERS, "partials and counters");

enum CqStep { CQ_GRAM, CQ_PASS1, CQ_PASS2, CQ_PASS3 };

struct CqArgs {
    QrWork w;
    int64_t j0, rows, chunk;  // panel column, its rows, rows per workgroup (a multiple of CQ_ROWS)
    int pw;
    double shift;
    double *Tout;
};

struct CqLds {
    double A[S64][DL];   // the rows' transposed tile; then the 64 x 64 matrix being factored
    double B[S64][DL];   // the packed triangle; then Q_top and its LU
    double T[4][16][17];
    double sg[S64];
    int flag, ok;
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

// Sum of the workgroups' partial Gram blocks in the last workgroup to arrive: entry t of
// block idx in v[idx].  True there.
DEV bool sum_partials(double *part, unsigned *counters, double (&v)[NBLK], int *flag)
{
    const int t = threadIdx.x, n = (int)gridDim.x, ch = (int)blockIdx.x;
    auto add = [&](int first, int count, int step) {
#pragma unroll
        for (int idx = 0; idx < NBLK; ++idx)
            v[idx] = 0.0;
#pragma unroll 4
        for (int q = 0; q < count; ++q) {
            const double *p = part + (int64_t)(first + q * step) * (NBLK * BLK) + t;
#pragma unroll
            for (int idx = 0; idx < NBLK; ++idx)
                v[idx] += p[idx * BLK];
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
    for (int idx = 0; idx < NBLK; ++idx)
        part[(int64_t)g0 * (NBLK * BLK) + idx * BLK + t] = v[idx];
    if (!arrive_last(counters, ngrp, flag))
        return false;
    add(0, ngrp, CQ_GRP);
    return true;
}

// The summed Gram matrix into S (upper blocks; identity beyond pw, shift_coef * trace on the
// diagonal) and its Cholesky factor in place.
DEV void factor_gram(const double (&v)[NBLK], int pw, double shift_coef, CqLds &L, int32_t *status)
{
    const int t = threadIdx.x, i0 = t >> 4, j0 = t & 15;
#pragma unroll
    for (int idx = 0; idx < NBLK; ++idx) {
        const int c = blk_col(idx), b = idx - c * (c + 1) / 2;
        const int i = 16 * b + i0, l = 16 * c + j0;
        L.A[i][l] = (i < pw && l < pw) ? v[idx] : (i == l ? 1.0 : 0.0);
    }
    if (t == 0)
        L.ok = 1;
    __syncthreads();
    if (shift_coef != 0.0 && t < 64) {
        const double d = (t < pw) ? L.A[t][t] : 0.0;
        const double tr = wave_sum(d);
        if (t < pw)
            L.A[t][t] = d + shift_coef * tr;
    }
    __syncthreads();
    chol64(L.A, &L.ok);
    if (t == 0 && !L.ok)
        set_status(status, DST_ERANK);
}

DEV void copy_pack(double *dst, const double *src)
{
    for (int e = threadIdx.x; e < PACK; e += 256)
        dst[e] = src[e];
    __syncthreads();
}

// After the second pass: R3 = chol(G), Q_top = Q2[0:pw] R3^-1, LU of Q_top - S, the compact-WY
// T, R = S R3 R2 R1 and Y1 into the panel's top block, tau, and U R3 for the last pass.
template <class T>
DEV void panel_top(const CqArgs &a, CqLds &L)
{
    const QrWork &w = a.w;
    const int pw = a.pw, t = threadIdx.x, lane = t & 63, wave = t >> 6, g = lane >> 4, r = lane & 15;
    double *P = &L.B[0][0], *R21 = w.cq_R + 2 * CB * CB;
    pack_upper([&](int i, int j) { return L.A[i][j]; }, P, L.T);
    d4 y[4];
    load_rows(y, (const double *)w.cq_S, w.cq_ld, 16 * wave + r, (int64_t)pw, pw);
    solve_rows<false>(y, P);
    __syncthreads();
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e)
            L.B[16 * wave + r][16 * c + 4 * e + g] = y[c][e];
    __syncthreads();
    lu64_signs(L.B, L.sg, pw);
    // R = S R3 (R2 R1) and U R3: blocks wave, wave + 4, wave + 8 of their upper triangles
    T *Ap = ((sizeof(T) == 8) ? reinterpret_cast<T *>(w.A) : reinterpret_cast<T *>(w.A32)) + a.j0 * w.lda + a.j0;
    d4 ur[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        const int idx = wave + 4 * q;
        if (idx >= NBLK)
            break;
        const int c = blk_col(idx), b = idx - c * (c + 1) / 2;
        const d4 rc = upper_product_block(
            b, c, [&](int i, int k) { return L.A[i][k]; },
            [&](int k, int j) { return R21[blk_at(k >> 4, c) * BLK + (k & 15) * 16 + (j & 15)]; });
        ur[q] = upper_product_block(
            b, c, [&](int i, int k) { return i <= k ? L.B[i][k] : 0.0; }, [&](int k, int j) { return L.A[k][j]; });
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int i = 16 * b + g + 4 * e, j = 16 * c + r;
            if (i <= j && j < pw)
                Ap[j * w.lda + i] = (T)(L.sg[i] * rc[e]);
        }
    }
    // Y1 below the diagonal
    for (int e = t; e < CB * CB; e += 256) {
        const int i = e & 63, j = e >> 6;
        if (i > j && i < pw)
            Ap[j * w.lda + i] = (T)L.B[i][j];
    }
    __syncthreads();
    // T = -U S Y1^-T: rows of -U S times the inverse of Y1^T (unit upper)
    double *P1 = &L.A[0][0];
    pack_upper([&](int i, int j) { return i == j ? 1.0 : ((j < pw) ? L.B[j][i] : 0.0); }, P1, L.T);
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
            L.A[i][j] = (i < pw && j < pw) ? ur[q][e] : (i == j ? 1.0 : 0.0);
        }
    }
    __syncthreads();
    pack_upper([&](int i, int j) { return L.A[i][j]; }, w.cq_R + 3 * CB * CB, L.T);
}

// One pass over the panel's rows (see CqStep).  TS: what it reads, TD: what it writes, T: the
// factored matrix's storage.
template <int STEP, class TS, class TD, class T>
__global__ __launch_bounds__(256, 2) void cqr_step_kernel(CqArgs a, const TS *src, int64_t lds_, TD *dst,
                                                          int64_t ldd)
{
    __shared__ CqLds L;
    const QrWork &w = a.w;
    const int pw = a.pw;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, g = lane >> 4, r = lane & 15;
    const int64_t lo = (int64_t)blockIdx.x * a.chunk;
    const int64_t hi = (lo + a.chunk) < a.rows ? (lo + a.chunk) : a.rows;
    double *P = &L.B[0][0];
    double *pack_in = w.cq_R + (STEP == CQ_PASS1 ? 0 : (STEP == CQ_PASS2 ? 1 : 3)) * CB * CB;
    d4 y[4], nxt[4];
    load_rows(nxt, src, lds_, lo + 16 * wave + r, hi, pw);
    if constexpr (STEP != CQ_GRAM)
        copy_pack(P, pack_in);
    d4 acc[3];
#pragma unroll
    for (int q = 0; q < 3; ++q)
        acc[q] = d4{0.0, 0.0, 0.0, 0.0};
    for (int64_t r0 = lo; r0 < hi; r0 += CQ_ROWS) {
        const int64_t row = r0 + 16 * wave + r;
#pragma unroll
        for (int c = 0; c < 4; ++c)
            y[c] = nxt[c];
        if (r0 + CQ_ROWS < hi)
            load_rows(nxt, src, lds_, row + CQ_ROWS, hi, pw);
        if constexpr (STEP != CQ_GRAM) {
            solve_rows<STEP == CQ_PASS1>(y, P);
            // the last pass leaves the top block (rows below pw) to the reconstruction
            store_rows(y, dst, ldd, row, STEP == CQ_PASS3 ? (int64_t)pw : (int64_t)0, hi, pw);
        }
        if constexpr (STEP != CQ_PASS3) {
            __syncthreads();  // the previous step's reads of the tile are done
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    L.A[16 * c + 4 * e + g][16 * wave + r] = y[c][e];
            __syncthreads();
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                const int idx = wave + 4 * q;
                if (idx < NBLK) {
                    const int c = blk_col(idx), b = idx - c * (c + 1) / 2;
#pragma unroll
                    for (int k = 0; k < CQ_ROWS / 4; ++k)
                        acc[q] = mfma16(L.A[16 * b + r][4 * k + g], L.A[16 * c + r][4 * k + g], acc[q]);
                }
            }
        }
    }
    if constexpr (STEP != CQ_PASS3) {
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const int idx = wave + 4 * q;
            if (idx < NBLK)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    w.cq_part[(int64_t)blockIdx.x * (NBLK * BLK) + idx * BLK + (g + 4 * e) * 16 + r] = acc[q][e];
        }
        double v[NBLK];
        if (!sum_partials(w.cq_part, w.cq_counters, v, &L.flag))
            return;
        factor_gram(v, pw, STEP == CQ_GRAM ? a.shift : 0.0, L, w.status);
        if constexpr (STEP == CQ_GRAM) {
            pack_upper([&](int i, int j) { return L.A[i][j]; }, w.cq_R, L.T);
        } else if constexpr (STEP == CQ_PASS1) {
            pack_upper([&](int i, int j) { return L.A[i][j]; }, w.cq_R + CB * CB, L.T);
            // R2 R1 (R1 is the pack this pass solved with, still in P)
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                const int idx = wave + 4 * q;
                if (idx < NBLK) {
                    const int c = blk_col(idx), b = idx - c * (c + 1) / 2;
                    const d4 p = upper_product_block(
                        b, c, [&](int i, int k) { return L.A[i][k]; },
                        [&](int k, int j) { return P[blk_at(k >> 4, c) * BLK + (k & 15) * 16 + (j & 15)]; });
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        w.cq_R[2 * CB * CB + idx * BLK + (g + 4 * e) * 16 + r] = p[e];
                }
            }
        } else {
            panel_top<T>(a, L);
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
    a.chunk = (a.chunk + CQ_ROWS - 1) / CQ_ROWS * CQ_ROWS;
    const double u = 0x1p-53;
    a.shift = 11.0 * ((double)mk * pw + (double)pw * (pw + 1)) * u;
    a.Tout = Tout;
    const dim3 grid((unsigned)((mk + a.chunk - 1) / a.chunk));
    double *S = w.cq_S;
    hipLaunchKernelGGL((cqr_step_kernel<CQ_GRAM, T, T, T>), grid, dim3(256), 0, s, a, (const T *)base, w.lda, base,
                       w.lda);
    hipLaunchKernelGGL((cqr_step_kernel<CQ_PASS1, T, double, T>), grid, dim3(256), 0, s, a, (const T *)base, w.lda, S,
                       w.cq_ld);
    hipLaunchKernelGGL((cqr_step_kernel<CQ_PASS2, double, double, T>), grid, dim3(256), 0, s, a, (const double *)S,
                       w.cq_ld, S, w.cq_ld);
    if (mk > pw)
        hipLaunchKernelGGL((cqr_step_kernel<CQ_PASS3, double, T, T>), grid, dim3(256), 0, s, a, (const double *)S,
                           w.cq_ld, base, w.lda);
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
