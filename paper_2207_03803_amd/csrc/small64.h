// 64 x 64 building blocks of the QR panels and their compact-WY factors, for one workgroup
// of 256 threads (four waves).  Matrices sit in LDS with a row stride of DL doubles, which
// keeps a fragment read along a column free of bank conflicts.  Everything but the chains of
// 16 dependent steps inside a diagonal block runs on v_mfma_f64_16x16x4_f64; with lane
// l = 16 g + r that instruction takes A(m = r, k = g) and B(k = g, n = r) and its element e
// is C(m = g + 4 e, n = r).
#pragma once

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

// Value of v in lane `lane` (uniform) of the wave.
DEV double readlane_d(double v, int lane)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffll), lane);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// 1 / d for a normal d, to about one ulp: the hardware's estimate and two Newton steps (a
// third of a division's latency, which the chains below would wait for at each step).
DEV double fast_rcp(double d)
{
    double x = __builtin_amdgcn_rcp(d);
    x = fma(x, fma(-d, x, 1.0), x);
    return fma(x, fma(-d, x, 1.0), x);
}

// Cholesky S = U^T U of the 64 x 64 matrix in LDS (upper triangle read), in place: U above,
// zeros below.  Per 16 rows: one wave eliminates them over all 64 columns (lane = column, the
// 16 rows in registers, square roots and row scaling afterwards, off the chain), then the
// trailing blocks take the rank-16 update on all four waves.  A pivot that is not positive
// and finite counts as 1 and clears *ok (LDS, set to 1 by the caller).  13 us where a chain of
// 64 steps on one wave took about 40.
DEV void chol64(double (*S)[DL], int *ok)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, g = lane >> 4, r = lane & 15;
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
        if (wave == 0) {
            double x[16], dv = 1.0;
            bool bad = false;
#pragma unroll
            for (int i = 0; i < 16; ++i)
                x[i] = S[16 * kb + i][lane];
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                double d = readlane_d(x[k], 16 * kb + k);
                if (!(d > 0.0) || !(d < INFINITY)) {
                    bad = true;
                    d = 1.0;
                }
                if (lane == k)
                    dv = d;
                const double wv = x[k] * fast_rcp(d);
#pragma unroll
                for (int i = k + 1; i < 16; ++i)
                    x[i] -= readlane_d(wv, 16 * kb + i) * x[k];
            }
            const double sq = sqrt(dv), rs = 1.0 / sq;
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                const int row = 16 * kb + k;
                const double v = lane == row ? readlane_d(sq, k) : x[k] * readlane_d(rs, k);
                S[row][lane] = lane >= row ? v : 0.0;
            }
            if (bad && lane == 0)
                *ok = 0;
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
                acc = mfma16(-S[16 * kb + 4 * e + g][rb + r], S[16 * kb + 4 * e + g][cb + r], acc);
#pragma unroll
            for (int e = 0; e < 4; ++e)
                S[rb + g + 4 * e][cb + r] = acc[e];
        }
        __syncthreads();
    }
}

// The upper triangle read through f(row, col) (row <= col) as a PACK in P (LDS or global):
// its ten blocks (zeros below the diagonal), then the inverses of the four diagonal blocks
// (wave w inverts block w, one column per lane).  T: 16 x 17 scratch per wave.  No barrier at
// the start; f's data must be visible.  Ends with a barrier.
template <class F>
DEV void pack_upper(F f, double *P, double (*T)[16][17])
{
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int i0 = t >> 4, j0 = t & 15;
#pragma unroll
    for (int idx = 0; idx < NBLK; ++idx) {
        const int c = blk_col(idx), b = idx - c * (c + 1) / 2;
        const int row = 16 * b + i0, col = 16 * c + j0;
        const double v = row <= col ? f(row, col) : 0.0;
        P[idx * BLK + t] = v;
        if (b == c)
            T[b][i0][j0] = v;
    }
    __syncthreads();
    if (lane < 16) {
        double x[16];
        const double dinv = 1.0 / T[wave][lane][lane];
#pragma unroll
        for (int i = 15; i >= 0; --i) {
            double v = i == lane ? 1.0 : 0.0;
#pragma unroll
            for (int p = i + 1; p < 16; ++p)
                v -= T[wave][i][p] * x[p];
            x[i] = v * readlane_d(dinv, i);
        }
#pragma unroll
        for (int i = 0; i < 16; ++i)
            P[NBLK * BLK + wave * BLK + i * 16 + lane] = x[i];
    }
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
// diagonal, the unit lower factor's entries below.  Blocked by 16 like chol64.
DEV void lu64_signs(double (*B)[DL], double *sg, int pw)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, g = lane >> 4, r = lane & 15;
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
        const int k0 = 16 * kb;
        if (wave == 0) {
            double q[16], sv = 1.0;
#pragma unroll
            for (int c = 0; c < 16; ++c)
                q[c] = B[lane][k0 + c];
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                if (k0 + k < pw) {
                    const double d = readlane_d(q[k], k0 + k);
                    const double s = (d >= 0.0) ? -1.0 : 1.0, piv = d - s;
                    const bool below = lane > k0 + k && lane < pw;
                    const double li = below ? q[k] * fast_rcp(piv) : 0.0;
#pragma unroll
                    for (int c = k + 1; c < 16; ++c)
                        q[c] -= li * readlane_d(q[c], k0 + k);
                    if (below)
                        q[k] = li;
                    if (lane == k0 + k)
                        q[k] = piv;
                    if (lane == k)
                        sv = s;
                }
            }
            if (lane >= k0)
#pragma unroll
                for (int c = 0; c < 16; ++c)
                    B[lane][k0 + c] = q[c];
            if (lane < 16)
                sg[k0 + lane] = sv;
        }
        __syncthreads();
        // the block row: one column per lane, L11 x = b
        if (wave == 0 && lane >= k0 + 16) {
            double x[16];
#pragma unroll
            for (int i = 0; i < 16; ++i)
                x[i] = B[k0 + i][lane];
#pragma unroll
            for (int k = 0; k < 16; ++k)
#pragma unroll
                for (int i = k + 1; i < 16; ++i)
                    x[i] -= B[k0 + i][k0 + k] * x[k];
#pragma unroll
            for (int i = 0; i < 16; ++i)
                B[k0 + i][lane] = x[i];
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
