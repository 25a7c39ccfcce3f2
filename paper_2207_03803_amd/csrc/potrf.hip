// Blocked right-looking Cholesky factorisation K = U^T U (U = L^T, upper
// triangular), in place, FP64 (Sec. Theory: the lower block of A is L_MM^T).
// Steps of 64 columns go in pairs.  One launch factors a step's diagonal block and solves its
// block row; the second step of a pair first brings its own tiles up to date with the first
// one's rows.  One product of depth 128 then applies both to everything below.
#include "kernels.h"
#include "small64.h"

namespace gap {

constexpr int CNB = CHOL_NB;
static_assert(CNB == S64, "block rows of the 64 x 64 helpers");

// Two matrices only: with 68 KB a workgroup fits beside a K_NM one on a CU.  With three it waited
// for both of a CU's to end at once, so the steps on the side stream starved until
// the K_NM was over.
struct CholLds {
    double D[S64][DL];  // the diagonal block, [row][column]; then the block row's tile, [column][row]
    double E[S64][DL];  // the previous step's rows above the block, [column][p]; then U_kk packed
    int ok;
};
static_assert(PACK <= S64 * DL, "a packed triangle fits a matrix buffer");

// Columns x .. x + 63 (those below n) of the 64 rows from k0 on (rows past kb zero), as
// M[column - x][row - k0]; 256 threads, consecutive lanes on consecutive rows.
DEV void chol_load_cols(const double *U, int64_t ld, int64_t k0, int kb, int64_t x, int64_t n, double (*M)[DL])
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    double v[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const int c = wave + 4 * q;
        v[q] = (x + c < n && lane < kb) ? U[(x + c) * ld + k0 + lane] : 0.0;
    }
#pragma unroll
    for (int q = 0; q < 16; ++q)
        M[wave + 4 * q][lane] = v[q];
}

// Column x (below n) of the 64 rows from k0 on (rows past kb zero): rows 16 c + 4 e + g at y[c][e].
DEV void chol_load_frag(const double *U, int64_t ld, int64_t k0, int kb, int64_t x, int64_t n, d4 (&y)[4])
{
    const int g = (threadIdx.x & 63) >> 4;
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int row = 16 * c + 4 * e + g;
            y[c][e] = (x < n && row < kb) ? U[x * ld + k0 + row] : 0.0;
        }
}

// Step k0 (kb <= 64 columns): every workgroup factors the diagonal block for itself, then
// solves U_kk^T X = B for its 64 columns right of it (one refinement per 16-row block keeps
// each solve backward stable).  PREV: the 64 rows above (the pair's first step) are first
// subtracted from the diagonal block and the tile.  Workgroup 0 leaves U_kk in diag
// ([column][row], 64 x 64): the others still read the block in place, so the pair's
// trailing update (chol_syrk_kernel) stores it; with no columns to the right it is
// stored here.  Latency-bound: 18 us, 25 with PREV (65 and 85 beside a K_NM), where the diagonal block, the block row
// and the strip update of each step took 35 + 35 + 30 us.
template <bool PREV>
__global__ __launch_bounds__(256) void chol_step_kernel(double *U, int64_t ld, int64_t k0, int kb, int64_t n,
                                                        double *__restrict__ diag, int32_t *status)
{
    __shared__ CholLds L;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, g = lane >> 4, r = lane & 15;
    const int64_t c0 = k0 + kb + (int64_t)blockIdx.x * CNB;  // this workgroup's columns (none: >= n)
    const bool right = c0 < n;
    // the diagonal block's upper 16 x 16 blocks wave, wave + 4, wave + 8
    d4 acc[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        const int idx = wave + 4 * q, c = blk_col(idx), b = idx - c * (c + 1) / 2;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int i = 16 * b + g + 4 * e, l = 16 * c + r;
            acc[q][e] = (idx < NBLK && i < kb && l < kb) ? U[(k0 + l) * ld + k0 + i] : (i == l ? 1.0 : 0.0);
        }
    }
    // this wave's 16 columns of the block row (one per lane r), and of the rows above
    d4 y[4], f[4];
    chol_load_frag(U, ld, k0, kb, c0 + 16 * wave + r, n, y);
    if constexpr (PREV) {
        chol_load_frag(U, ld, k0 - CNB, CNB, c0 + 16 * wave + r, n, f);
        chol_load_cols(U, ld, k0 - CNB, CNB, k0, k0 + kb, L.E);
    }
    if (t == 0)
        L.ok = 1;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        const int idx = wave + 4 * q;
        if (idx >= NBLK)
            break;
        const int c = blk_col(idx), b = idx - c * (c + 1) / 2;
        if constexpr (PREV) {
#pragma unroll
            for (int k = 0; k < CNB / 4; ++k)
                acc[q] = mfma16(-L.E[16 * b + r][4 * k + g], L.E[16 * c + r][4 * k + g], acc[q]);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
            L.D[16 * b + g + 4 * e][16 * c + r] = acc[q][e];
    }
    if constexpr (PREV) {
        if (right)
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll
                for (int k = 0; k < CNB / 4; ++k)
                    y[c] = mfma16(-L.E[16 * c + r][4 * k + g], f[k / 4][k % 4], y[c]);
    }
    __syncthreads();
    double *P = &L.E[0][0];
    chol64(L.D, P, &L.ok);
    if (blockIdx.x == 0) {
        if (t == 0 && !L.ok)
            set_status(status, DST_ENOTPD);
#pragma unroll
        for (int q = 0; q < CNB * CNB / 256; ++q) {
            const int e = q * 256 + t, i = e & 63, l = e >> 6;
            if (right)
                diag[e] = L.D[i][l];
            else if (i < kb && l < kb)
                U[(k0 + l) * ld + k0 + i] = L.D[i][l];
        }
    }
    if (!right)
        return;
    solve_rows<true>(y, P);
    __syncthreads();
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e)
            L.D[16 * wave + r][16 * c + 4 * e + g] = y[c][e];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const int c = wave + 4 * q;
        if (c0 + c < n && lane < kb)
            U[(c0 + c) * ld + k0 + lane] = L.D[c][lane];
    }
}

// Trailing update of the upper triangle: A[r][c] -= sum_{p < kb} U[k0+p][r] U[k0+p][c]
// for k1 <= r <= c < n, one tile per workgroup (enumerated column by column), both operands
// contiguous along p.  The tile is computed transposed, acc(c, r), so that
// consecutive lanes update consecutive rows of the column-major matrix; in the small tiles the
// accumulators start from -A, so that its loads run beside the first stages (the large ones would
// spill: n = 10,000 13.4 -> 17.0 ms).  The last workgroup stores the two diagonal blocks that the
// steps left in diag.  Bound by latency at a few tiles: 12 us (15 with A read at the end and
// the blocks stored by the first tile's workgroup).

// The 64 x 64 block dg ([column][row]) into U at k0, by NT threads: all loads in flight.
template <int NT>
DEV void chol_store_block(double *U, int64_t ld, int64_t k0, const double *dg)
{
    constexpr int N = CNB * CNB / NT;
    double v[N];
#pragma unroll
    for (int q = 0; q < N; ++q)
        v[q] = dg[q * NT + threadIdx.x];
#pragma unroll
    for (int q = 0; q < N; ++q) {
        const int e = q * NT + threadIdx.x;
        U[(k0 + (e >> 6)) * ld + k0 + (e & 63)] = v[q];
    }
}

template <class S>
__global__ __launch_bounds__(S::NT, S::NT == 512 ? 4 : 2) void chol_syrk_kernel(double *U, int64_t ld, int64_t k0,
                                                                                int kb, int64_t k1, int64_t n,
                                                                                const double *__restrict__ diag)
{
    __shared__ __align__(16) d2 lds[2 * S::UNITS];
    static_assert(S::BM == S::BN, "square tiles");
    const int64_t L = blockIdx.x;
    if (L == (int64_t)gridDim.x - 1) {
        chol_store_block<S::NT>(U, ld, k0, diag);
        chol_store_block<S::NT>(U, ld, k0 + CNB, diag + CNB * CNB);
        return;
    }
    int64_t tj = (int64_t)((sqrt(8.0 * (double)L + 1.0) - 1.0) * 0.5);
    while ((tj + 1) * (tj + 2) / 2 <= L)
        ++tj;
    while (tj * (tj + 1) / 2 > L)
        --tj;
    const int64_t ti = L - tj * (tj + 1) / 2;
    const int64_t r0 = k1 + ti * S::BM, c0 = k1 + tj * S::BN;
    const double *src[S::LPT];
#pragma unroll
    for (int i = 0; i < S::LPT; ++i) {
        const int x = S::unit_row(i);
        int64_t col = x < S::BM ? c0 + x : r0 + x - S::BM;
        col = col < n ? col : n - 1;  // computed, not stored
        src[i] = U + col * ld + k0 + S::unit_k(i);
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = wave / S::WN, wn = wave % S::WN;
    constexpr bool FROM_A = S::NT == 256;
    d4 acc[S::FM][S::FN];
    ktile_zero<S>(acc);
    if constexpr (FROM_A)
#pragma unroll
        for (int i = 0; i < S::FM; ++i)
#pragma unroll
            for (int j = 0; j < S::FN; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int64_t c = c0 + acc_row<S>(wm, i, lane, e);
                    const int64_t r = r0 + acc_col<S>(wn, j, lane, e);
                    if (r <= c && c < n)
                        acc[i][j][e] = -U[c * ld + r];
                }
    ktile_product<S>(acc, lds, src, kb, rows_aligned16(U + k0, ld));
#pragma unroll
    for (int i = 0; i < S::FM; ++i)
#pragma unroll
        for (int j = 0; j < S::FN; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int64_t c = c0 + acc_row<S>(wm, i, lane, e);
                const int64_t r = r0 + acc_col<S>(wn, j, lane, e);
                if (r <= c && c < n)
                    U[c * ld + r] = FROM_A ? -acc[i][j][e] : U[c * ld + r] - acc[i][j][e];
            }
}

// The diagonal block that a step with no trailing update after it left in diag.
__global__ __launch_bounds__(256) void chol_store_kernel(double *U, int64_t ld, int64_t k0, const double *diag)
{
    chol_store_block<256>(U, ld, k0, diag);
}

// diag: 2 x 64 x 64 doubles of scratch.
hipError_t launch_potrf_upper(double *U, int64_t ld, int64_t n, double *diag, int32_t *status, hipStream_t s)
{
    using SL = KTile<double, 128, 128, 4, 2, 4>;
    using SS = KTile<double, 64, 64, 8, 2, 2>;
    auto blocks = [](int64_t x, int64_t b) { return (x + b - 1) / b; };
    auto step = [&](int64_t k0, int kb, bool prev, double *dg) {
        const int64_t rest = n - k0 - kb;
        const dim3 grid((unsigned)(rest > 0 ? blocks(rest, CNB) : 1));
        if (prev)
            hipLaunchKernelGGL(chol_step_kernel<true>, grid, dim3(256), 0, s, U, ld, k0, kb, n, dg, status);
        else
            hipLaunchKernelGGL(chol_step_kernel<false>, grid, dim3(256), 0, s, U, ld, k0, kb, n, dg, status);
        return rest;
    };
    for (int64_t k0 = 0; k0 < n; k0 += 2 * CNB) {
        const int kb = (int)((n - k0) < CNB ? (n - k0) : CNB);
        if (step(k0, kb, false, diag) <= 0)
            break;
        const int64_t k1 = k0 + CNB;
        const int kb1 = (int)((n - k1) < CNB ? (n - k1) : CNB);
        const int64_t rest = step(k1, kb1, true, diag + CNB * CNB);
        if (rest <= 0) {  // no trailing update: the first step's block is still in diag
            hipLaunchKernelGGL(chol_store_kernel, dim3(1), dim3(256), 0, s, U, ld, k0, (const double *)diag);
            break;
        }
        // 64 x 64 tiles where large ones would leave CUs without one
        const int64_t nl = blocks(rest, SL::BM), ns = blocks(rest, SS::BM);
        if (nl * (nl + 1) / 2 >= 256)
            hipLaunchKernelGGL(chol_syrk_kernel<SL>, dim3((unsigned)(nl * (nl + 1) / 2 + 1)), dim3(SL::NT), 0, s, U, ld, k0,
                               2 * CNB, k1 + CNB, n, (const double *)diag);
        else
            hipLaunchKernelGGL(chol_syrk_kernel<SS>, dim3((unsigned)(ns * (ns + 1) / 2 + 1)), dim3(SS::NT), 0, s, U, ld, k0,
                               2 * CNB, k1 + CNB, n, (const double *)diag);
    }
    return hipGetLastError();
}

}  // namespace gap
