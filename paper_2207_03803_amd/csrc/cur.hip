// CUR sparse-point selection (Sec. Implementation: sparse points chosen by
// CUR-based methods, after Mahoney & Drineas 2009).  For the n x d matrix X of
// descriptor rows, the leverage of row i over the row space of X is
//   lev_i = x_i^T (X^T X)^-1 x_i = ||x_i U^-1||^2,  X^T X = U^T U,
// and M rows are taken either as the M largest leverages or, with one Exp(1)
// variate e_i per row from the caller, as a sample without replacement with
// probabilities proportional to the leverage: the M smallest keys e_i / lev_i
// (the exponential-key method of Efraimidis & Spirakis).  Equal keys are taken
// in row order; the indices come out ascending.
//
// Steps: G = X^T X on FP64 MFMA (split over row chunks, upper block pairs,
// fixed-order sum), the Cholesky factor U (the K_MM factorisation), W = U^-1
// (one workgroup per column), Y = X W on FP64 MFMA with the row sums of squares
// in the epilogue (W upper triangular: a column tile needs k up to its last
// column only), keys, then the M-th smallest key by an 8-pass radix select on
// its bits and an ordered compaction.
#include <stddef.h>

#include "kernels.h"

namespace gap {

// Gram blocks of 64 x 64 (d = 400 pads to 448 columns; 128-wide blocks would pad to 512) and
// projection tiles of 128 rows x 64 columns.
using CG = MTile<double, 64, 64, 16, 2, 2>;
using CP = KTile<double, 128, 64, 4, 2, 2>;
template <int BN>
using CPW = KTile<double, 128, BN, 4, 4, 1>;  // a last tile of 80 or 96 columns
constexpr int CUR_GB = 64;                 // block of G
constexpr int CUR_NB = 128;                // columns of Y whose squares one workgroup sums
constexpr int64_t CUR_MAX_CHUNKS = 64;     // row chunks the partials' space is sized for (128-wide blocks)
constexpr int64_t CUR_PLACES = 1024;       // Gram workgroups resident at once (four per CU)
constexpr int CUR_SEL_NT = 256;
constexpr int CUR_SEL_PER = 4096;          // keys per workgroup in the compaction
constexpr int CUR_MAX_D = 4096;

struct CurState {
    unsigned long long prefix, mask;  // radix select: bits fixed so far
    long long k;                      // rank still to find among keys matching the prefix
    int32_t status;
    int32_t pad;
};

int64_t cur_nb(int d) { return (d + CUR_NB - 1) / CUR_NB; }
int64_t cur_chunks(int64_t n, int d)
{
    const int64_t nb = cur_nb(d), pairs = nb * (nb + 1) / 2;
    int64_t nch = (2048 + pairs - 1) / pairs;
    if (nch > CUR_MAX_CHUNKS)
        nch = CUR_MAX_CHUNKS;
    if (nch > (n + 255) / 256)
        nch = (n + 255) / 256;
    return nch < 1 ? 1 : nch;
}
int64_t cur_sel_blocks(int64_t n) { return (n + CUR_SEL_PER - 1) / CUR_SEL_PER; }

// Column tiles of the projection: of 64, the last one with up to 32 columns more.
__host__ __device__ inline int64_t cur_proj_tiles(int d)
{
    const int full = d / CP::BN, rest = d % CP::BN;
    return full + (rest > 0 && (full == 0 || rest > 32) ? 1 : 0);
}

// Byte offsets of the workspace parts (each 256-aligned).
struct CurLayout {
    size_t state, G, part, W, rowpart, keys, hist, cnt, base, total;
};
CurLayout cur_layout(int64_t n, int d)
{
    CurLayout L{};
    size_t o = 0;
    auto take = [&](size_t bytes) {
        const size_t at = o;
        o = (o + bytes + 255) / 256 * 256;
        return at;
    };
    const int64_t nb = cur_nb(d), pairs = nb * (nb + 1) / 2;
    L.state = take(sizeof(CurState));
    L.G = take(sizeof(double) * (size_t)d * (size_t)d);
    L.part = take(sizeof(double) * (size_t)cur_chunks(n, d) * (size_t)pairs * CUR_NB * CUR_NB);
    L.W = take(sizeof(double) * (size_t)d * (size_t)d);
    L.rowpart = take(sizeof(double) * (size_t)nb * (size_t)n);
    L.keys = take(sizeof(double) * (size_t)n);
    L.hist = take(sizeof(unsigned) * 256);
    L.cnt = take(sizeof(long long) * 2 * (size_t)cur_sel_blocks(n));
    L.base = take(sizeof(long long) * 2 * (size_t)cur_sel_blocks(n));
    L.total = o;
    return L;
}

// Block pair index -> (bi, bj), bi <= bj, row-major over the upper triangle.
DEV void cur_pair(int64_t bp, int64_t nb, int64_t &bi, int64_t &bj)
{
    bi = 0;
    int64_t rem = bp;
    while (rem >= nb - bi) {
        rem -= nb - bi;
        ++bi;
    }
    bj = bi + rem;
}

// Row chunks of the Gram product: what the partials' space holds, rounded down to whole rounds
// of resident workgroups, at least 256 rows each.
int64_t cur_gram_chunks(int64_t n, int d)
{
    const int64_t nb = cur_nb(d), room = cur_chunks(n, d) * (nb * (nb + 1) / 2) * CUR_NB * CUR_NB;
    const int64_t gb = (d + CUR_GB - 1) / CUR_GB, pairs = gb * (gb + 1) / 2;
    int64_t nch = room / (pairs * CUR_GB * CUR_GB);
    if (nch * pairs > CUR_PLACES)
        nch = nch * pairs / CUR_PLACES * CUR_PLACES / pairs;
    if (nch > (n + 255) / 256)
        nch = (n + 255) / 256;
    return nch < 1 ? 1 : nch;
}

// Partial Gram block (bi, bj) over the rows of a chunk:
// part[ch][bp][p][q] = sum_r X[r][64 bi + p] X[r][64 bj + q].  Bound by the matrix cores; a
// chunk's blocks run on one XCD, which then reads the chunk's rows once.  1e6 x 400:
// 3.4 ms, 8.0 with 128 x 128 blocks on K-major stages filled through registers.
__global__ __launch_bounds__(CG::NT, 4) void cur_gram_kernel(const double *__restrict__ X, int64_t n, int d,
                                                             int64_t gb, int64_t nch, int64_t chunk,
                                                             double *__restrict__ part)
{
    using S = CG;
    __shared__ __align__(16) d2 lds[2 * S::UNITS];
    const int64_t pairs = gb * (gb + 1) / 2, total = pairs * nch;
    const int64_t lw = xcd_remap(blockIdx.x, (total + 7) & ~int64_t(7));
    if (lw >= total)
        return;
    const int64_t ch = lw / pairs, bp = lw % pairs;
    int64_t bi, bj;
    cur_pair(bp, gb, bi, bj);
    const int64_t rlo = ch * chunk;
    const int64_t rhi = (rlo + chunk) < n ? (rlo + chunk) : n;
    d4 acc[S::FM][S::FN];
    ktile_zero<S>(acc);
    if (rlo < rhi) {
        const int len = (int)(rhi - rlo), nk = (len + S::BK - 1) / S::BK;
        const double *src[S::LPT];
        int64_t step[S::LPT];
        int64_t col[S::LPT];
#pragma unroll
        for (int i = 0; i < S::LPT; ++i) {
            const int x = S::unit_x(i);
            const int64_t c = x < S::UA ? bi * CUR_GB + 2 * x : bj * CUR_GB + 2 * (x - S::UA);
            col[i] = c;
            // columns past d repeat column 0 of the row and are not used
            src[i] = X + (rlo + S::unit_p(i)) * (int64_t)d + (c < d ? c : 0);
            step[i] = (int64_t)S::BK * d;
        }
        mtile_product<S>(acc, lds, nk, rows_aligned16(X, d) ? len / S::BK : 0, src, step, [&](int kt, int i) {
            const int64_t r = rlo + (int64_t)kt * S::BK + S::unit_p(i);
            const double *p = X + (r < rhi ? r : rlo) * (int64_t)d + (col[i] < d ? col[i] : 0);
            d2 v;
            v.x = p[0];
            v.y = p[col[i] + 1 < d ? 1 : 0];
            if (r >= rhi)
                v = d2{0.0, 0.0};
            return v;
        });
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, g = lane >> 4, rl = lane & 15;
    const int wm = wave / S::WN, wn = wave % S::WN;
    double *P = part + (ch * pairs + bp) * (int64_t)(CUR_GB * CUR_GB);
#pragma unroll
    for (int i = 0; i < S::FM; ++i)
#pragma unroll
        for (int j = 0; j < S::FN; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                P[S::row(wm, i, g, e) * CUR_GB + S::col(wn, j, rl)] = acc[i][j][e];
}

// G (column-major, leading dimension d, both triangles) from the partials, the
// chunks summed in order.  One element of one block pair per thread.
__global__ __launch_bounds__(256) void cur_gram_sum_kernel(const double *__restrict__ part, int64_t nch,
                                                           int64_t pairs, int64_t gb, int d, double *__restrict__ G)
{
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= pairs * CUR_GB * CUR_GB)
        return;
    const int64_t bp = e / (CUR_GB * CUR_GB), pq = e % (CUR_GB * CUR_GB);
    int64_t bi, bj;
    cur_pair(bp, gb, bi, bj);
    const int64_t p = bi * CUR_GB + pq / CUR_GB, q = bj * CUR_GB + pq % CUR_GB;
    if (p >= d || q >= d)
        return;
    double s = 0.0;
#pragma unroll 8
    for (int64_t ch = 0; ch < nch; ++ch)
        s += part[(ch * pairs + bp) * (int64_t)(CUR_GB * CUR_GB) + pq];
    G[q * d + p] = s;
    G[p * d + q] = s;
}

// W = U^-1 for the upper triangular U (column-major, leading dimension d):
// workgroup j solves U w = e_j by back substitution, right-looking (w_i from
// b_i, then b_k -= U[k][i] w_i for k < i), and writes column j of W.
__global__ __launch_bounds__(256) void cur_trinv_kernel(const double *__restrict__ U, int d, double *__restrict__ W)
{
    __shared__ double b[CUR_MAX_D];
    __shared__ double wi_s;
    const int j = blockIdx.x, t = threadIdx.x;
    for (int k = t; k < d; k += 256)
        b[k] = (k == j) ? 1.0 : 0.0;
    for (int i = t + j + 1; i < d; i += 256)
        W[(int64_t)j * d + i] = 0.0;
    for (int i = j; i >= 0; --i) {
        __syncthreads();
        if (t == 0) {
            wi_s = b[i] / U[(int64_t)i * d + i];
            W[(int64_t)j * d + i] = wi_s;
        }
        __syncthreads();
        const double wi = wi_s;
        const double *Ui = U + (int64_t)i * d;
        for (int k = t; k < i; k += 256)
            b[k] -= Ui[k] * wi;
    }
}

// Y = X W for 128 rows and the columns of tile 2 ct + odd (64, up to 96 in the last one);
// rowpart[ct][r] = the sum of Y[r][q]^2 over the tile's columns (a fixed order), added to the
// even tile's by the odd one's launch.
template <class S>
DEV void cur_proj_tile(const double *__restrict__ X, int64_t n, int d, const double *__restrict__ W, int64_t r0,
                       int64_t q0, double *out, int odd, d2 *lds, double (*rsum)[CP::BM])
{
    static_assert(S::BM == CP::BM && S::NT == CP::NT && S::UNITS <= CPW<96>::UNITS && S::WN <= CP::WN, "LDS");
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, g = lane >> 4, rl = lane & 15;
    const int wm = wave / S::WN, wn = wave % S::WN;
    const int K = (int)((q0 + S::BN) < d ? (q0 + S::BN) : d);  // W[k][q] = 0 for k > q
    const double *src[S::LPT];
#pragma unroll
    for (int i = 0; i < S::LPT; ++i) {
        const int r = S::has(i) ? S::unit_row(i) : 0;
        // rows past n and columns past d repeat the last one; the columns count as zero below
        const int64_t row = r < S::BM ? (r0 + r < n ? r0 + r : n - 1) : (q0 + r - S::BM < d ? q0 + r - S::BM : d - 1);
        src[i] = (r < S::BM ? X : W) + row * (int64_t)d + S::unit_k(i);
    }
    d4 acc[S::FM][S::FN];
    ktile_zero<S>(acc);
    ktile_product<S>(acc, lds, src, K, rows_aligned16(X, d) && rows_aligned16(W, d));
#pragma unroll
    for (int i = 0; i < S::FM; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            double s = 0.0;
#pragma unroll
            for (int j = 0; j < S::FN; ++j) {
                const double y = q0 + acc_col<S>(wn, j, lane, e) < d ? acc[i][j][e] : 0.0;
                s += y * y;
            }
            s += __shfl_xor(s, 1, 64);
            s += __shfl_xor(s, 2, 64);
            s += __shfl_xor(s, 4, 64);
            s += __shfl_xor(s, 8, 64);
            if (rl == 0)
                rsum[wn][wm * S::TM + 16 * i + g + 4 * e] = s;
        }
    __syncthreads();
    if (t < S::BM && r0 + t < n) {
        double rs = rsum[0][t];
        if constexpr (S::WN == 2)
            rs += rsum[1][t];
        out[r0 + t] = odd ? out[r0 + t] + rs : rs;
    }
}

// A row tile's column tiles start together on one XCD and walk its rows of X in step,
// so that they are read from HBM once per launch; both halves in one workgroup, one after
// the other, read them at their own pace (1e6 x 400: 5.4 ms against 4.7; 6.0 on K-major
// 128 x 128 tiles).  Up to 32 columns past the last full tile go with it (cur_proj_tiles): they
// take all of K, and a tile of their own costs as much as a full one (d = 400: 4.7 ms; on a 16
// wide tile, bound by its stages' latency, 4.3; 3.3 with the last 80 columns together).
__global__ __launch_bounds__(CP::NT, 3) void cur_proj_kernel(const double *__restrict__ X, int64_t n, int d,
                                                             const double *__restrict__ W, int64_t nct, int odd,
                                                             double *__restrict__ rowpart)
{
    __shared__ __align__(16) d2 lds[2 * CPW<96>::UNITS];
    __shared__ double rsum[CP::WN][CP::BM];
    const int64_t total = (n + CP::BM - 1) / CP::BM * nct;
    const int64_t lw = xcd_remap(blockIdx.x, (total + 7) & ~int64_t(7));
    if (lw >= total)
        return;
    const int64_t r0 = lw / nct * CP::BM, ct = lw % nct, tile = 2 * ct + odd, q0 = tile * CP::BN;
    const int64_t width = tile == cur_proj_tiles(d) - 1 ? d - q0 : CP::BN;
    double *out = rowpart + ct * n;
    if (width <= CP::BN)
        cur_proj_tile<CP>(X, n, d, W, r0, q0, out, odd, lds, rsum);
    else if (width <= 80)
        cur_proj_tile<CPW<80>>(X, n, d, W, r0, q0, out, odd, lds, rsum);
    else
        cur_proj_tile<CPW<96>>(X, n, d, W, r0, q0, out, odd, lds, rsum);
}

// lev = sum of the column tiles' parts in order; key = draw / lev (1 / lev
// without draws), +inf for a zero row.
__global__ __launch_bounds__(256) void cur_keys_kernel(const double *__restrict__ rowpart, int64_t n, int64_t nct,
                                                       const double *__restrict__ draws, double *__restrict__ lev_out,
                                                       double *__restrict__ keys)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n)
        return;
    double l = 0.0;
    for (int64_t ct = 0; ct < nct; ++ct)
        l += rowpart[ct * n + i];
    if (lev_out)
        lev_out[i] = l;
    double k = (draws ? draws[i] : 1.0) / l;
    if (!(k == k))
        k = __builtin_inf();
    keys[i] = k;
}

__global__ void cur_select_init_kernel(CurState *st, unsigned *hist, long long M)
{
    const int t = threadIdx.x;
    if (t < 256)
        hist[t] = 0u;
    if (t == 0) {
        st->prefix = 0ull;
        st->mask = 0ull;
        st->k = M;
        st->status = 0;
    }
}

// Histogram of bits [shift, shift + 8) of the keys whose higher bits match the prefix.
__global__ __launch_bounds__(256) void cur_hist_kernel(const double *__restrict__ keys, int64_t n,
                                                       const CurState *__restrict__ st, int shift,
                                                       unsigned *__restrict__ hist)
{
    __shared__ unsigned h[256];
    h[threadIdx.x] = 0u;
    __syncthreads();
    const unsigned long long prefix = st->prefix, mask = st->mask;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        const unsigned long long b = (unsigned long long)__double_as_longlong(keys[i]);
        if ((b & mask) == prefix)
            atomicAdd(&h[(b >> shift) & 255ull], 1u);
    }
    __syncthreads();
    if (h[threadIdx.x])
        atomicAdd(&hist[threadIdx.x], h[threadIdx.x]);
}

// Fix the next 8 bits: the digit whose cumulative count first reaches k.
__global__ __launch_bounds__(256) void cur_pick_kernel(CurState *st, unsigned *hist, int shift)
{
    __shared__ long long c[256];
    const int t = threadIdx.x;
    c[t] = hist[t];
    __syncthreads();
    for (int off = 1; off < 256; off <<= 1) {
        const long long v = t >= off ? c[t - off] : 0;
        __syncthreads();
        c[t] += v;
        __syncthreads();
    }
    const long long k = st->k;
    const long long below = t > 0 ? c[t - 1] : 0;
    __syncthreads();
    if (below < k && c[t] >= k) {
        st->k = k - below;
        st->prefix |= (unsigned long long)t << shift;
        st->mask |= 255ull << shift;
    }
    hist[t] = 0u;
}

// Per compaction block: keys below the threshold T and keys equal to it.
__global__ __launch_bounds__(CUR_SEL_NT) void cur_count_kernel(const double *__restrict__ keys, int64_t n,
                                                               const CurState *__restrict__ st,
                                                               long long *__restrict__ cnt)
{
    __shared__ long long sl[CUR_SEL_NT], se[CUR_SEL_NT];
    const unsigned long long T = st->prefix;
    const int64_t lo = (int64_t)blockIdx.x * CUR_SEL_PER;
    const int64_t hi = (lo + CUR_SEL_PER) < n ? (lo + CUR_SEL_PER) : n;
    long long a = 0, b = 0;
    for (int64_t i = lo + threadIdx.x; i < hi; i += CUR_SEL_NT) {
        const unsigned long long x = (unsigned long long)__double_as_longlong(keys[i]);
        a += x < T;
        b += x == T;
    }
    sl[threadIdx.x] = a;
    se[threadIdx.x] = b;
    __syncthreads();
    for (int off = CUR_SEL_NT / 2; off > 0; off >>= 1) {
        if ((int)threadIdx.x < off) {
            sl[threadIdx.x] += sl[threadIdx.x + off];
            se[threadIdx.x] += se[threadIdx.x + off];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        cnt[2 * blockIdx.x] = sl[0];
        cnt[2 * blockIdx.x + 1] = se[0];
    }
}

// Exclusive prefix sums of the per-block counts (one workgroup).
__global__ __launch_bounds__(256) void cur_scan_kernel(const long long *__restrict__ cnt, int64_t nblk,
                                                       long long *__restrict__ base)
{
    __shared__ long long carry_l, carry_e;
    __shared__ long long sl[256], se[256];
    const int t = threadIdx.x;
    if (t == 0) {
        carry_l = 0;
        carry_e = 0;
    }
    __syncthreads();
    for (int64_t b0 = 0; b0 < nblk; b0 += 256) {
        const int64_t b = b0 + t;
        const long long l = b < nblk ? cnt[2 * b] : 0, e = b < nblk ? cnt[2 * b + 1] : 0;
        sl[t] = l;
        se[t] = e;
        __syncthreads();
        for (int off = 1; off < 256; off <<= 1) {
            const long long vl = t >= off ? sl[t - off] : 0, ve = t >= off ? se[t - off] : 0;
            __syncthreads();
            sl[t] += vl;
            se[t] += ve;
            __syncthreads();
        }
        if (b < nblk) {
            base[2 * b] = carry_l + sl[t] - l;
            base[2 * b + 1] = carry_e + se[t] - e;
        }
        __syncthreads();
        if (t == 255) {
            carry_l += sl[255];
            carry_e += se[255];
        }
        __syncthreads();
    }
}

// Write the selected row indices in ascending order: row i is taken when its
// key is below T, or equal to T and among the first k such rows; its place is
// (rows taken before it) = less_before + min(equal_before, k).
__global__ __launch_bounds__(CUR_SEL_NT) void cur_write_kernel(const double *__restrict__ keys, int64_t n,
                                                               const CurState *__restrict__ st,
                                                               const long long *__restrict__ base,
                                                               int64_t *__restrict__ out)
{
    __shared__ int sl[CUR_SEL_NT], se[CUR_SEL_NT];
    __shared__ long long run_l, run_e;
    const unsigned long long T = st->prefix;
    const long long kq = st->k;
    const int t = threadIdx.x;
    const int64_t lo = (int64_t)blockIdx.x * CUR_SEL_PER;
    const int64_t hi = (lo + CUR_SEL_PER) < n ? (lo + CUR_SEL_PER) : n;
    if (t == 0) {
        run_l = base[2 * blockIdx.x];
        run_e = base[2 * blockIdx.x + 1];
    }
    __syncthreads();
    for (int64_t i0 = lo; i0 < hi; i0 += CUR_SEL_NT) {
        const int64_t i = i0 + t;
        int fl = 0, fe = 0;
        if (i < hi) {
            const unsigned long long x = (unsigned long long)__double_as_longlong(keys[i]);
            fl = x < T;
            fe = x == T;
        }
        sl[t] = fl;
        se[t] = fe;
        __syncthreads();
        for (int off = 1; off < CUR_SEL_NT; off <<= 1) {
            const int vl = t >= off ? sl[t - off] : 0, ve = t >= off ? se[t - off] : 0;
            __syncthreads();
            sl[t] += vl;
            se[t] += ve;
            __syncthreads();
        }
        const long long lb = run_l + sl[t] - fl, eb = run_e + se[t] - fe;  // before row i
        if (fl || (fe && eb < kq))
            out[lb + (eb < kq ? eb : kq)] = i;
        __syncthreads();
        if (t == CUR_SEL_NT - 1) {
            run_l += sl[t];
            run_e += se[t];
        }
        __syncthreads();
    }
}

size_t cur_workspace_bytes(int64_t n, int d) { return cur_layout(n, d).total; }
size_t cur_status_offset() { return offsetof(CurState, status); }

hipError_t launch_cur_select(const CurLaunch &c, hipStream_t s)
{
    const int64_t n = c.n;
    const int d = c.d;
    const CurLayout L = cur_layout(n, d);
    char *ws = static_cast<char *>(c.workspace);
    CurState *st = reinterpret_cast<CurState *>(ws + L.state);
    double *G = reinterpret_cast<double *>(ws + L.G);
    double *part = reinterpret_cast<double *>(ws + L.part);
    double *W = reinterpret_cast<double *>(ws + L.W);
    double *rowpart = reinterpret_cast<double *>(ws + L.rowpart);
    double *keys = reinterpret_cast<double *>(ws + L.keys);
    unsigned *hist = reinterpret_cast<unsigned *>(ws + L.hist);
    long long *cnt = reinterpret_cast<long long *>(ws + L.cnt);
    long long *base = reinterpret_cast<long long *>(ws + L.base);
    const int64_t gb = (d + CUR_GB - 1) / CUR_GB, pairs = gb * (gb + 1) / 2;
    const int64_t nch = cur_gram_chunks(n, d);
    int64_t chunk = (n + nch - 1) / nch;
    chunk = (chunk + 15) / 16 * 16;
    hipLaunchKernelGGL(cur_select_init_kernel, dim3(1), dim3(256), 0, s, st, hist, (long long)c.M);
    hipLaunchKernelGGL(cur_gram_kernel, dim3((unsigned)((pairs * nch + 7) & ~int64_t(7))), dim3(CG::NT), 0, s, c.x, n, d,
                       gb, nch, chunk, part);
    hipLaunchKernelGGL(cur_gram_sum_kernel, dim3((unsigned)((pairs * CUR_GB * CUR_GB + 255) / 256)), dim3(256), 0, s,
                       part, nch, pairs, gb, d, G);
    hipError_t e = launch_potrf_upper(G, d, d, part, &st->status, s);
    if (e != hipSuccess)
        return e;
    hipLaunchKernelGGL(cur_trinv_kernel, dim3((unsigned)d), dim3(256), 0, s, G, d, W);
    for (int odd = 0; odd < 2; ++odd) {
        const int64_t nct = (cur_proj_tiles(d) + 1 - odd) / 2, ptiles = (n + CP::BM - 1) / CP::BM * nct;
        if (ptiles > 0)
            hipLaunchKernelGGL(cur_proj_kernel, dim3((unsigned)((ptiles + 7) & ~int64_t(7))), dim3(CP::NT), 0, s, c.x, n,
                               d, W, nct, odd, rowpart);
    }
    hipLaunchKernelGGL(cur_keys_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, rowpart, n,
                       (cur_proj_tiles(d) + 1) / 2, c.draws,
                       c.lev_out, keys);
    int64_t hg = (n + 255) / 256;
    if (hg > 2048)
        hg = 2048;
    for (int pass = 0; pass < 8; ++pass) {
        const int shift = 56 - 8 * pass;
        hipLaunchKernelGGL(cur_hist_kernel, dim3((unsigned)hg), dim3(256), 0, s, keys, n, st, shift, hist);
        hipLaunchKernelGGL(cur_pick_kernel, dim3(1), dim3(256), 0, s, st, hist, shift);
    }
    const int64_t nblk = cur_sel_blocks(n);
    hipLaunchKernelGGL(cur_count_kernel, dim3((unsigned)nblk), dim3(CUR_SEL_NT), 0, s, keys, n, st, cnt);
    hipLaunchKernelGGL(cur_scan_kernel, dim3(1), dim3(256), 0, s, cnt, nblk, base);
    hipLaunchKernelGGL(cur_write_kernel, dim3((unsigned)nblk), dim3(CUR_SEL_NT), 0, s, keys, n, st, base, c.out);
    return hipGetLastError();
}

int cur_max_d() { return CUR_MAX_D; }

}  // namespace gap
