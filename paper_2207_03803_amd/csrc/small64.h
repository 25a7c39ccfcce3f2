// 64 x 64 building blocks of the QR panels and their compact-WY factors, for one workgroup
// of 256 threads (four waves).  Matrices sit in LDS with a row stride of DL doubles, which
// keeps a fragment read along a column free of bank conflicts.  Everything but the chains of
// 16 dependent steps inside a diagonal block runs on v_mfma_f64_16x16x4_f64; with lane
// l = 16 g + r that instruction takes A(m = r, k = g) and B(k = g, n = r) and its element e
// is C(m = g + 4 e, n = r).
#pragma once

#include <utility>

#include "common.h"

namespace gap {

constexpr int S64 = 64;
constexpr int DL = 66;          // LDS row stride
constexpr int NBLK = 10;        // 16 x 16 blocks of an upper triangle, (b, c) at c (c + 1) / 2 + b
constexpr int BLK = 256;
constexpr int PACK = NBLK * BLK + 4 * BLK;  // a triangle's blocks, then the inverses of its diagonal blocks

DEV int blk_col(int idx) { return idx >= 6 ? 3 : (idx >= 3 ? 2 : (idx >= 1 ? 1 : 0)); }
DEV int blk_at(int b, int c) { return c * (c + 1) / 2 + b; }

DEV d4 mfma16(double a, double b, d4 c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }

// Lane N of each row of 16 lanes, to the whole row: one instruction, and no scalar register
// for the next one to wait on.
template <int N>
DEV double row_bcast(double v)
{
    const long long b = __double_as_longlong(v);
    return __longlong_as_double(__builtin_amdgcn_mov_dpp(b, 0x150 + N, 0xf, 0xf, true));
}

// f(integral_constant<int, A>) ... f(integral_constant<int, B - 1>)
template <int A, int B, class F>
DEV void static_for(F f)
{
    if constexpr (A < B) {
        f(std::integral_constant<int, A>{});
        static_for<A + 1, B>(f);
    }
}

// 1 / d to about one ulp: the hardware's estimate (error e below 2^-20) and one step of third
// order, x + x (e + e^2) (a third of a division's latency, which the chains below would wait for
// at each step).  For d and 1 / d well inside the normal range (2^-1000 .. 2^1000): a subnormal d
// gives NaN.  chol64 sees to that; lu64_signs divides by pivots between 1 and 2.
DEV double fast_rcp(double d)
{
    const double x = __builtin_amdgcn_rcp(d);
    const double e = fma(-d, x, 1.0);
    return fma(x, fma(e, e, e), x);
}

// The four rows 4 e .. 4 e + 3 that element e of a 16 x 16 block holds (row 4 e + g in lanes
// 16 g + r), each in every row of 16 lanes.
DEV void rows_of(double v, double (&y)[4])
{
    const long long b = __double_as_longlong(v);
    const unsigned w[2] = {(unsigned)b, (unsigned)(b >> 32)};
    unsigned o[4][2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const auto p = __builtin_amdgcn_permlane32_swap(w[h], w[h], false, false);
        const auto lo = __builtin_amdgcn_permlane16_swap(p[0], p[0], false, false);
        const auto hi = __builtin_amdgcn_permlane16_swap(p[1], p[1], false, false);
        o[0][h] = lo[0];
        o[1][h] = lo[1];
        o[2][h] = hi[0];
        o[3][h] = hi[1];
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
        y[j] = __longlong_as_double(((long long)o[j][1] << 32) | o[j][0]);
}

// y[g]: the four rows back in one element.
DEV double row_pick(const double (&y)[4], int g)
{
    const double a = (g & 1) ? y[1] : y[0], b = (g & 1) ? y[3] : y[2];
    return (g & 2) ? b : a;
}

// The inverse of a 16 x 16 upper triangle (zeros below; row i, column c at U[i * ld + c], LDS),
// one wave, to inv[16 i + c].  Four rows at a time, the products on MFMA.
DEV void invert_upper16(const double *U, int ld, double *inv)
{
    const int lane = threadIdx.x & 63, g = lane >> 4, r = lane & 15;
    const double dinv = 1.0 / U[r * ld + r];
    d4 acc;
#pragma unroll
    for (int e = 0; e < 4; ++e)
        acc[e] = g + 4 * e == r ? 1.0 : 0.0;
    static_for<0, 4>([&](auto bc) {
        constexpr int b = 3 - bc;
        double y[4], x[4], row[4];
#pragma unroll
        for (int j = 0; j < 4; ++j)
            row[j] = U[(4 * b + j) * ld + r];
        const double below = -U[r * ld + 4 * b + g];
        rows_of(acc[b], y);
        static_for<0, 4>([&](auto jc) {
            constexpr int j = 3 - jc;
            x[j] = y[j] * row_bcast<4 * b + j>(dinv);
            static_for<0, j>([&](auto ic) { y[ic] -= row_bcast<4 * b + j>(row[ic]) * x[j]; });
        });
        const double xg = row_pick(x, g);
        inv[(4 * b + g) * 16 + r] = xg;
        if constexpr (b > 0)
            acc = mfma16(below, xg, acc);
    });
}

// The ten blocks of the upper triangle read through f(row, col) (row <= col; zeros below) to P
// (LDS or global).
template <class F>
DEV void pack_blocks(F f, double *P)
{
    const int t = threadIdx.x, i0 = t >> 4, j0 = t & 15;
#pragma unroll
    for (int idx = 0; idx < NBLK; ++idx) {
        const int c = blk_col(idx), b = idx - c * (c + 1) / 2;
        const int row = 16 * b + i0, col = 16 * c + j0;
        P[idx * BLK + t] = row <= col ? f(row, col) : 0.0;
    }
}

// A PACK: the ten blocks, then the inverses of the four diagonal blocks (wave w inverts block
// w).  T: 16 x 17 scratch per wave.  No barrier at the start; f's data must be visible.  Ends
// with a barrier.
template <class F>
DEV void pack_upper(F f, double *P, double (*T)[16][17])
{
    const int t = threadIdx.x, i0 = t >> 4, j0 = t & 15;
    pack_blocks(f, P);
#pragma unroll
    for (int b = 0; b < 4; ++b)
        T[b][i0][j0] = i0 <= j0 ? f(16 * b + i0, 16 * b + j0) : 0.0;
    __syncthreads();
    const int wave = t >> 6;
    invert_upper16(&T[wave][0][0], 17, P + (NBLK + wave) * BLK);
    __syncthreads();
}

// The same as chol64 below, a row at a time with a square root and divisions, for any finite
// pivots.
DEV void chol64_plain(double (*S)[DL], double *P, int *ok)
{
    const int t = threadIdx.x, wave = t >> 6;
#pragma unroll 1
    for (int k = 0; k < S64; ++k) {
        const double d = S[k][k];
        const bool good = d > 0.0 && d < INFINITY;
        const double u = sqrt(good ? d : 1.0);
        __syncthreads();
        if (t < S64)
            S[k][t] = t > k ? S[k][t] / u : (t == k ? u : 0.0);
        if (t == k && !good)
            *ok = 0;
        __syncthreads();
#pragma unroll 1
        for (int e = t; e < S64 * S64; e += 256) {
            const int i = e >> 6, j = e & 63;
            if (i > k && j >= i)
                S[i][j] -= S[k][i] * S[k][j];
        }
        __syncthreads();
    }
    invert_upper16(&S[16 * wave][16 * wave], DL, P + (NBLK + wave) * BLK);
    pack_blocks([&](int i, int j) { return S[i][j]; }, P);
    __syncthreads();
}

// Cholesky S = U^T U of the 64 x 64 matrix in LDS (upper triangle read), in place: U above,
// zeros below, and U as a PACK in P (LDS or global).  A pivot that is not positive and finite
// counts as 1 and clears *ok (LDS, set to 1 by the caller).
//
// Block row by block row: wave c eliminates the block row's column block c together with a copy
// of the diagonal block, four rows at a time: those four replicated in every row of 16 lanes,
// so that a step is a reciprocal (its pivot formed ahead, in every lane), row broadcasts and a
// few updates; then one MFMA for the rows below.  Square roots and row scaling come
// after the chain.  The wave whose columns are done inverts the diagonal block before.
// 9.3 us where one wave with all 64 columns and scalar broadcasts took 13, and 2 us more for the
// pack.
//
// A pivot is a diagonal entry less what the rows above take off it: at least 2^-53 of the entry,
// unless it is none at all.  With all entries in 2^-900 .. 2^900 fast_rcp can take every pivot; other
// blocks (descriptors or sigma_w of extreme size) go row by row.
DEV void chol64(double (*S)[DL], double *P, int *ok)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, g = lane >> 4, r = lane & 15;
    const double sd = S[lane][lane];
    if (__builtin_expect(__any((sd > 0.0 && sd < 0x1p-900) || (sd > 0x1p900 && sd < INFINITY)), 0)) {
        chol64_plain(S, P, ok);
        return;
    }
#pragma unroll 1
    for (int kb = 0; kb < 4; ++kb) {
        const int k0 = 16 * kb, c0 = 16 * wave;
        d4 u, p, out;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            u[e] = S[k0 + g + 4 * e][k0 + r];
            p[e] = S[k0 + g + 4 * e][c0 + r];
        }
        __syncthreads();
        if (wave >= kb) {
            double dv = 1.0;
            bool bad = false;
            static_for<0, 4>([&](auto bc) {
                constexpr int b = bc;
                double y[4], q[4], w[4];
                rows_of(u[b], y);
                rows_of(p[b], q);
                double d = row_bcast<4 * b>(y[0]);
                static_for<0, 4>([&](auto jc) {
                    constexpr int j = jc, k = 4 * b + j;
                    const bool good = d > 0.0 && d < INFINITY;
                    const double rc = good ? fast_rcp(d) : 1.0;
                    bad |= !good;
                    if (r == k)
                        dv = y[j];
                    w[j] = y[j] * rc;
                    if constexpr (j < 3) {
                        const double f = row_bcast<k + 1>(y[j]);
                        d = row_bcast<k + 1>(y[j + 1]) - (f * rc) * f;
                    }
                    static_for<j + 1, 4>([&](auto ic) {
                        constexpr int i = ic;
                        const double m = row_bcast<4 * b + i>(w[j]);
                        y[i] -= m * y[j];
                        q[i] -= m * q[j];
                    });
                });
                out[b] = row_pick(q, g);
                if constexpr (b < 3) {
                    const double wg = -row_pick(w, g);
                    u = mfma16(wg, row_pick(y, g), u);
                    p = mfma16(wg, out[b], p);
                }
            });
            const double sq = sqrt(dv > 0.0 && dv < INFINITY ? dv : 1.0), rs = 1.0 / sq;
            static_for<0, 4>([&](auto bc) {
                constexpr int b = bc;
                const double f[4] = {row_bcast<4 * b>(rs), row_bcast<4 * b + 1>(rs), row_bcast<4 * b + 2>(rs),
                                     row_bcast<4 * b + 3>(rs)};
                const int row = k0 + 4 * b + g, col = c0 + r;
                const double v = out[b] * row_pick(f, g);
                S[row][col] = col > row ? v : (col == row ? sq : 0.0);
            });
            if (bad && lane == 0 && wave == kb)
                *ok = 0;
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                S[k0 + g + 4 * e][c0 + r] = 0.0;
            if (wave == kb - 1)
                invert_upper16(&S[c0][c0], DL, P + (NBLK + wave) * BLK);
        }
        __syncthreads();
        const int nb = 3 - kb;
        for (int idx = wave; idx < nb * (nb + 1) / 2; idx += 4) {
            const int c = blk_col(idx), b = idx - c * (c + 1) / 2;
            const int rb = 16 * (kb + 1 + b), cb = 16 * (kb + 1 + c);
            d4 acc;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                acc[e] = S[rb + g + 4 * e][cb + r];
#pragma unroll
            for (int e = 0; e < 4; ++e)
                acc = mfma16(-S[k0 + 4 * e + g][rb + r], S[k0 + 4 * e + g][cb + r], acc);
#pragma unroll
            for (int e = 0; e < 4; ++e)
                S[rb + g + 4 * e][cb + r] = acc[e];
        }
        if (nb > 0)
            __syncthreads();
    }
    pack_blocks([&](int i, int j) { return S[i][j]; }, P);
    if (wave == 3)
        invert_upper16(&S[48][48], DL, P + (NBLK + 3) * BLK);
    __syncthreads();
}

// A wave's 16 rows y (16 x 64) as four 4-vectors: lane (g, r) holds y[row r][col 16 c + 4 e + g]
// at y[c][e].  y := y R^-1 for the packed upper triangle P (LDS), block column by block
// column: earlier blocks' products are subtracted on MFMA, then the diagonal block's inverse
// is applied; element e of a block is the k = 4 e + g operand of the next product, so the
// rows never leave the registers.  REFINE adds a step of residual correction per diagonal
// block, which makes each solve backward stable whatever the block's condition.
template <bool REFINE>
DEV void solve_rows(d4 (&y)[4], const double *P)
{
    const int lane = threadIdx.x & 63, g = lane >> 4, r = lane & 15;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        d4 v = y[c];
#pragma unroll
        for (int b = 0; b < c; ++b)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                v = mfma16(-P[blk_at(b, c) * BLK + (4 * e + g) * 16 + r], y[b][e], v);
        const double *inv = P + (NBLK + c) * BLK;
        d4 s = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int e = 0; e < 4; ++e)
            s = mfma16(inv[(4 * e + g) * 16 + r], v[e], s);
        if constexpr (REFINE) {
            const double *D = P + blk_at(c, c) * BLK;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                v = mfma16(-D[(4 * e + g) * 16 + r], s[e], v);
#pragma unroll
            for (int e = 0; e < 4; ++e)
                s = mfma16(inv[(4 * e + g) * 16 + r], v[e], s);
        }
        y[c] = s;
    }
}

// One 16 x 16 block (bi, bj) of the product of two upper triangles, fa and fb read by (row, col).
template <class FA, class FB>
DEV d4 upper_product_block(int bi, int bj, FA fa, FB fb)
{
    const int lane = threadIdx.x & 63, g = lane >> 4, r = lane & 15;
    d4 acc = d4{0.0, 0.0, 0.0, 0.0};
    for (int bk = bi; bk <= bj; ++bk)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int k = 16 * bk + 4 * e + g;
            acc = mfma16(fa(16 * bi + r, k), fb(k, 16 * bj + r), acc);
        }
    return acc;
}

// LU of B - diag(sg) (64 x 64 in LDS, order pw) without pivoting, sg_k = -sign of the pivot
// (sign(0) = +1), so that every pivot is at least 1 in magnitude.  In place: U on and above the
// diagonal, the unit lower factor's entries below.  Blocked like chol64; wave c takes column
// block c of the block row and row block c of the block column (as rows of the transpose),
// with copies of the diagonal block and its transpose.
DEV void lu64_signs(double (*B)[DL], double *sg, int pw)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, g = lane >> 4, r = lane & 15;
#pragma unroll 1
    for (int kb = 0; kb < 4; ++kb) {
        const int k0 = 16 * kb, c0 = 16 * wave;
        d4 u, l, pu, pl;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            u[e] = B[k0 + g + 4 * e][k0 + r];
            l[e] = B[k0 + r][k0 + g + 4 * e];
            pu[e] = B[k0 + g + 4 * e][c0 + r];
            pl[e] = B[c0 + r][k0 + g + 4 * e];
        }
        __syncthreads();
        if (wave >= kb) {
            double sv = 1.0, pv = 0.0;
            static_for<0, 4>([&](auto bc) {
                constexpr int b = bc;
                double y[4], z[4], qu[4], ql[4];
                rows_of(u[b], y);
                rows_of(l[b], z);
                rows_of(pu[b], qu);
                rows_of(pl[b], ql);
                double d = row_bcast<4 * b>(y[0]);
                static_for<0, 4>([&](auto jc) {
                    constexpr int j = jc, k = 4 * b + j;
                    const double s = (d >= 0.0) ? -1.0 : 1.0, piv = d - s;
                    const double rp = k0 + k < pw ? fast_rcp(piv) : 0.0;
                    if (r == k) {
                        sv = k0 + k < pw ? s : 1.0;
                        pv = piv;
                    }
                    // columns k of the lower factor: zero on and above the diagonal, and past pw
                    const double zj = z[j];
                    z[j] = (r > k && k0 + r < pw) ? zj * rp : 0.0;
                    ql[j] = (c0 + r > k0 + k && c0 + r < pw) ? ql[j] * rp : 0.0;
                    if constexpr (j < 3)
                        d = row_bcast<k + 1>(y[j + 1]) - (row_bcast<k + 1>(zj) * rp) * row_bcast<k + 1>(y[j]);
                    static_for<j + 1, 4>([&](auto ic) {
                        constexpr int i = ic;
                        const double m = row_bcast<4 * b + i>(z[j]);
                        y[i] -= m * y[j];
                        qu[i] -= m * qu[j];
                        const double n = row_bcast<4 * b + i>(y[j]);
                        z[i] -= n * z[j];
                        ql[i] -= n * ql[j];
                    });
                });
                const double ug = row_pick(qu, g), lg = row_pick(ql, g);
                if constexpr (b < 3) {
                    const double zg = row_pick(z, g), yg = row_pick(y, g);
                    u = mfma16(-zg, yg, u);
                    pu = mfma16(-zg, ug, pu);
                    l = mfma16(-yg, zg, l);
                    pl = mfma16(-yg, lg, pl);
                }
                const int k = k0 + 4 * b + g, x = c0 + r;  // row or column k against column or row x
                if (x > k) {
                    B[k][x] = ug;
                    B[x][k] = lg;
                }
            });
            if (wave == kb && lane < 16) {
                sg[k0 + lane] = sv;
                if (k0 + lane < pw)
                    B[k0 + lane][k0 + lane] = pv;
            }
        }
        __syncthreads();
        const int nb = 3 - kb;
        for (int idx = wave; idx < nb * nb; idx += 4) {
            const int rb = 16 * (kb + 1 + idx / nb), cb = 16 * (kb + 1 + idx % nb);
            d4 acc;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                acc[e] = B[rb + g + 4 * e][cb + r];
#pragma unroll
            for (int e = 0; e < 4; ++e)
                acc = mfma16(-B[rb + r][k0 + 4 * e + g], B[k0 + 4 * e + g][cb + r], acc);
#pragma unroll
            for (int e = 0; e < 4; ++e)
                B[rb + g + 4 * e][cb + r] = acc[e];
        }
        __syncthreads();
    }
}

}  // namespace gap
