// Blocked Householder QR of the augmented stacked matrix [A | b] in FP64
// (Sec. Implementation: the factorisation leaves R in the upper triangle and
// the Householder vectors below it with their weights tau; Q^T b comes from
// carrying b along as an extra column, which is what applying the stored
// reflectors to b computes).
//
// Each 64-column panel is factored by shifted CholeskyQR3 (cqr.hip) or, as
// selected per handle, as a tall-skinny QR (TSQR) over a 4-ary tree of
// 256-row tiles with its explicit Q formed top-down; in both cases the
// Householder vectors Y and the compact-WY factor T recovered from that Q by
// an LU factorisation of Q - S with the sign matrix S chosen to keep every
// pivot at least 1 in magnitude (Ballard, Demmel, Grigori, Jacquelin, Knight,
// Nguyen 2015, "Reconstructing Householder vectors from tall-skinny QR").  The
// result is the LAPACK-style representation H = I - Y T Y^T with Y unit lower
// trapezoidal, R = S R_tsqr, tau_i = T_ii.  The trailing columns (b included)
// are then updated on MFMA: P = Y^T C (split over row chunks), W = T^T P,
// C -= Y W.
//
// Reflector convention inside the tiles: H = I - tau v v^T, v(0) = 1,
// beta = -sign(alpha) ||(alpha, x)||, tau = (beta - alpha)/beta,
// v(1:) = x / (alpha - beta); tau = 0 when x is exactly zero.
#include <algorithm>

#include "kernels.h"
#include "qr_split.h"
#include "small64.h"

namespace gap {

constexpr int NB = QR_NB;
constexpr int TR = TS_ROWS;
constexpr int TILE = TR * NB;  // doubles per tile
constexpr int NPART = 8;           // threads per tile column
constexpr int TS_NT = NB * NPART;  // threads of the TSQR kernels
constexpr int SLOTS = TR / NPART;  // rows held per thread (row = NPART * slot + part)
constexpr int64_t MAX_CHUNKS = 32;     // row chunks of the split-K products into the bulk buffer
constexpr int64_t MAX_CHUNKS_S = 256;  // into the small buffer at 2 QR_NB columns (half that at 4 QR_NB)

int64_t qr_max_chunks() { return MAX_CHUNKS; }
int64_t qr_max_chunks_s() { return MAX_CHUNKS_S; }

TsqrTree tsqr_tree(int64_t m)
{
    TsqrTree t;
    int64_t n = (m + TR - 1) / TR;
    int64_t toff = 0, aoff = 0;
    for (int l = 0; l < TS_MAX_LEVELS; ++l) {
        t.nodes[l] = n;
        t.tile_off[l] = toff;
        t.tau_off[l] = aoff;
        toff += n * TILE;
        aoff += n * NB;
        t.levels = l + 1;
        if (n <= 1)
            break;
        n = (n + TS_FAN - 1) / TS_FAN;
    }
    t.tiles_doubles = toff;
    t.tau_doubles = aoff;
    return t;
}

// Node counts for a panel of mk rows (never more than the tree was sized for).
struct PanelTree {
    int levels;
    int64_t nodes[TS_MAX_LEVELS];
};

static PanelTree panel_tree(int64_t mk)
{
    PanelTree p{};
    int64_t n = (mk + TR - 1) / TR;
    for (int l = 0; l < TS_MAX_LEVELS; ++l) {
        p.nodes[l] = n;
        p.levels = l + 1;
        if (n <= 1)
            break;
        n = (n + TS_FAN - 1) / TS_FAN;
    }
    return p;
}

// Rows [lo, hi) of level-0 tile i out of n0 (balanced split of mk rows).
DEV void leaf_rows(int64_t i, int64_t n0, int64_t mk, int64_t &lo, int64_t &hi)
{
    lo = (i * mk) / n0;
    hi = ((i + 1) * mk) / n0;
}

// The matrix being factored: FP64 storage (w.A) or FP32 storage (w.A32).
template <class T>
DEV T *qmat(const QrWork &w);
template <>
DEV double *qmat<double>(const QrWork &w) { return w.A; }
template <>
DEV float *qmat<float>(const QrWork &w) { return w.A32; }

// Sum over the NPART consecutive lanes that hold one column (deterministic).
DEV double col_sum(double v)
{
    v += __shfl_xor(v, 1, 64);
    v += __shfl_xor(v, 2, 64);
    v += __shfl_xor(v, 4, 64);
    return v;
}

// ---------------------------------------------------------------------------
// Householder QR of one 256 x pw tile held in registers.  Thread t owns
// column q = t / 8 and the rows r = 8 * slot + (t % 8).  Level 0 reads rows
// of the panel; level l >= 1 stacks the R factors of up to 4 children.  The
// factored tile (R above the diagonal, v below) and tau go to the tree.
// ---------------------------------------------------------------------------
template <class T>
__global__ __launch_bounds__(TS_NT) void tsqr_factor_kernel(QrWork w, int64_t j0, int pw, int level,
                                                          int64_t n_level, int64_t n_prev, int64_t mk)
{
    __shared__ double vbuf[2][TR];
    __shared__ double taus[NB];
    const int t = threadIdx.x, q = t / NPART, part = t % NPART;
    const int64_t node = blockIdx.x;
    double x[SLOTS];
    if (level == 0) {
        int64_t lo, hi;
        leaf_rows(node, n_level, mk, lo, hi);
        const T *col = qmat<T>(w) + (j0 + q) * w.lda + j0 + lo;
        const int64_t nr = hi - lo;
#pragma unroll
        for (int i = 0; i < SLOTS; ++i) {
            const int r = NPART * i + part;
            x[i] = (q < pw && r < nr) ? (double)col[r] : 0.0;
        }
    } else {
        const double *prev = w.ts_tiles + w.tree.tile_off[level - 1];
        const int64_t c0 = node * TS_FAN;
        const int64_t nc = (n_prev - c0) < TS_FAN ? (n_prev - c0) : TS_FAN;
#pragma unroll
        for (int i = 0; i < SLOTS; ++i) {
            const int r = NPART * i + part;
            const int k = r / pw, rr = r % pw;
            x[i] = (q < pw && k < nc && rr <= q) ? prev[(c0 + k) * TILE + q * TR + rr] : 0.0;
        }
    }
    for (int j = 0; j < pw; ++j) {
        double *v = vbuf[j & 1];
        if (q == j) {
            double s = 0.0, a = 0.0;
#pragma unroll
            for (int i = 0; i < SLOTS; ++i) {
                const int r = NPART * i + part;
                if (r > j)
                    s += x[i] * x[i];
                if (r == j)
                    a = x[i];
            }
            s = col_sum(s);
            a = col_sum(a);  // one lane holds alpha, the others 0
            double tau = 0.0, scale = 0.0, beta = a;
            if (s != 0.0) {
                const double norm = sqrt(a * a + s);
                beta = (a >= 0.0) ? -norm : norm;
                tau = (beta - a) / beta;
                scale = 1.0 / (a - beta);
            }
#pragma unroll
            for (int i = 0; i < SLOTS; ++i) {
                const int r = NPART * i + part;
                if (r == j)
                    x[i] = beta;
                else if (r > j)
                    x[i] *= scale == 0.0 ? 1.0 : scale;
                v[r] = (r == j) ? 1.0 : (r > j ? x[i] : 0.0);
            }
            if (part == 0)
                taus[j] = tau;
        }
        __syncthreads();
        const double tau = taus[j];
        if (q > j && q < pw && tau != 0.0) {
            double d = 0.0;
#pragma unroll
            for (int i = 0; i < SLOTS; ++i)
                d += v[NPART * i + part] * x[i];
            d = col_sum(d) * tau;
#pragma unroll
            for (int i = 0; i < SLOTS; ++i)
                x[i] -= d * v[NPART * i + part];
        }
    }
    double *out = w.ts_tiles + w.tree.tile_off[level] + node * TILE + q * TR;
#pragma unroll
    for (int i = 0; i < SLOTS; ++i)
        out[NPART * i + part] = x[i];
    if (part == 0)
        w.ts_tau[w.tree.tau_off[level] + node * NB + q] = (q < pw) ? taus[q] : 0.0;
}

// ---------------------------------------------------------------------------
// Explicit Q, top-down: X_node = H_0 H_1 ... H_{pw-1} [S ; 0] where S is the
// node's pw x pw slice of its parent's X (the identity at the root).  Level 0
// writes its X into the panel's rows of A.
// ---------------------------------------------------------------------------
template <class T>
__global__ __launch_bounds__(TS_NT) void tsqr_formq_kernel(QrWork w, int64_t j0, int pw, int level,
                                                         int64_t n_level, int is_root, int64_t mk)
{
    __shared__ double V[NB * (TR + 1)];
    __shared__ double taus[NB];
    const int t = threadIdx.x, q = t / NPART, part = t % NPART;
    const int64_t node = blockIdx.x;
    const double *tile = w.ts_tiles + w.tree.tile_off[level] + node * TILE;
    for (int idx = t; idx < TILE; idx += TS_NT) {
        const int c = idx / TR, r = idx % TR;
        V[c * (TR + 1) + r] = tile[idx];
    }
    if (t < NB)
        taus[t] = w.ts_tau[w.tree.tau_off[level] + node * NB + t];
    double x[SLOTS];
    if (is_root) {
#pragma unroll
        for (int i = 0; i < SLOTS; ++i) {
            const int r = NPART * i + part;
            x[i] = (r == q && q < pw) ? 1.0 : 0.0;
        }
    } else {
        const int64_t parent = node / TS_FAN, pos = node % TS_FAN;
        const double *px = w.ts_X + w.tree.tile_off[level + 1] + parent * TILE + q * TR + pos * pw;
#pragma unroll
        for (int i = 0; i < SLOTS; ++i) {
            const int r = NPART * i + part;
            x[i] = (q < pw && r < pw) ? px[r] : 0.0;
        }
    }
    __syncthreads();
    if (q < pw) {
        for (int j = pw - 1; j >= 0; --j) {
            const double tau = taus[j];
            if (tau == 0.0)
                continue;
            const double *vc = V + j * (TR + 1);
            double d = 0.0;
#pragma unroll
            for (int i = 0; i < SLOTS; ++i) {
                const int r = NPART * i + part;
                const double vr = (r > j) ? vc[r] : (r == j ? 1.0 : 0.0);
                d += vr * x[i];
            }
            d = col_sum(d) * tau;
#pragma unroll
            for (int i = 0; i < SLOTS; ++i) {
                const int r = NPART * i + part;
                const double vr = (r > j) ? vc[r] : (r == j ? 1.0 : 0.0);
                x[i] -= d * vr;
            }
        }
    }
    if (level == 0) {
        int64_t lo, hi;
        leaf_rows(node, n_level, mk, lo, hi);
        if (q < pw) {
            T *col = qmat<T>(w) + (j0 + q) * w.lda + j0 + lo;
            const int64_t nr = hi - lo;
#pragma unroll
            for (int i = 0; i < SLOTS; ++i) {
                const int r = NPART * i + part;
                if (r < nr)
                    col[r] = (T)x[i];
            }
        }
    } else {
        double *out = w.ts_X + w.tree.tile_off[level] + node * TILE + q * TR;
#pragma unroll
        for (int i = 0; i < SLOTS; ++i)
            out[NPART * i + part] = x[i];
    }
}

// ---------------------------------------------------------------------------
// Reconstruction, top block (one workgroup): LU of Q1 - S with s_k =
// -sign(pivot) (sign(0) = +1), giving U and the unit lower Y1; then
// T = -U S Y1^-T, R = S R_root; writes R above and Y1 below the diagonal of
// the panel's top block, tau = diag(T), and U for the row solve below.
// ---------------------------------------------------------------------------
template <class T>
__global__ __launch_bounds__(256) void tsqr_lu_kernel(QrWork w, int64_t j0, int pw, int root_level, double *Tout)
{
    __shared__ double B[NB][NB + 1];
    __shared__ double Z[NB][NB + 1];
    __shared__ double sg[NB];
    const int t = threadIdx.x;
    for (int idx = t; idx < pw * pw; idx += 256) {
        const int r = idx % pw, c = idx / pw;
        B[r][c] = (double)qmat<T>(w)[(j0 + c) * w.lda + j0 + r];
    }
    __syncthreads();
    for (int k = 0; k < pw; ++k) {
        if (t == 0) {
            const double d = B[k][k];
            const double s = (d >= 0.0) ? -1.0 : 1.0;
            B[k][k] = d - s;
            sg[k] = s;
        }
        __syncthreads();
        const double piv = B[k][k];
        for (int i = k + 1 + t; i < pw; i += 256)
            B[i][k] /= piv;
        __syncthreads();
        const int wdt = pw - k - 1;
        for (int idx = t; idx < wdt * wdt; idx += 256) {
            const int i = k + 1 + idx % wdt, c = k + 1 + idx / wdt;
            B[i][c] -= B[i][k] * B[k][c];
        }
        __syncthreads();
    }
    // Z = Y1^-T (unit upper): column c by back-substitution, one thread per column
    if (t < pw) {
        const int c = t;
        for (int r = pw - 1; r >= 0; --r) {
            double v = (r == c) ? 1.0 : 0.0;
            if (r < c)
                for (int p = r + 1; p <= c; ++p)
                    v -= B[p][r] * Z[p][c];
            Z[r][c] = (r <= c) ? v : 0.0;
        }
    }
    __syncthreads();
    const double *root = w.ts_tiles + w.tree.tile_off[root_level];  // node 0
    for (int idx = t; idx < NB * NB; idx += 256) {
        const int r = idx / NB, c = idx % NB;
        double tv = 0.0;
        if (r < pw && c < pw && r <= c) {
            for (int p = r; p <= c; ++p)
                tv -= B[r][p] * sg[p] * Z[p][c];
        }
        Tout[idx] = tv;
        w.U[idx] = (r < pw && c < pw && r <= c) ? B[r][c] : 0.0;
        if (r < pw && c < pw) {
            double out;
            if (r <= c)
                out = sg[r] * root[c * TR + r];
            else
                out = B[r][c];
            qmat<T>(w)[(j0 + c) * w.lda + j0 + r] = (T)out;
        }
        if (r == c && r < pw)
            w.tau[j0 + r] = tv;
    }
}

// Rows below the top block: Y = Q U^-1 (one row per thread).
template <class T>
__global__ __launch_bounds__(256) void tsqr_trsm_kernel(QrWork w, int64_t j0, int pw)
{
    __shared__ double U[NB][NB + 1];
    for (int idx = threadIdx.x; idx < NB * NB; idx += 256)
        U[idx / NB][idx % NB] = w.U[idx];
    __syncthreads();
    const int64_t r = j0 + pw + (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (r >= w.m)
        return;
    double y[NB];
#pragma unroll
    for (int c = 0; c < NB; ++c)
        y[c] = (c < pw) ? (double)qmat<T>(w)[(j0 + c) * w.lda + r] : 0.0;
#pragma unroll
    for (int c = 0; c < NB; ++c) {
        if (c < pw) {
            double v = y[c];
#pragma unroll
            for (int i = 0; i < c; ++i)
                v -= y[i] * U[i][c];
            y[c] = v / U[c][c];
        }
    }
#pragma unroll
    for (int c = 0; c < NB; ++c)
        if (c < pw)
            qmat<T>(w)[(j0 + c) * w.lda + r] = (T)y[c];
}

// Tile of a trailing-update product: logical tiles are numbered row block by
// row block (the column tiles of one row block consecutive), and consecutive
// logical tiles run on the same XCD, so that the row block's Y tile stays in
// that XCD's L2 while its column tiles go by.
DEV bool update_tile(int64_t n_rb, int64_t n_cb, int64_t &rb, int64_t &cb)
{
    const int64_t total = n_rb * n_cb;
    const int64_t lw = xcd_remap(blockIdx.x, (total + 7) & ~int64_t(7));
    if (lw >= total)
        return false;
    rb = lw / n_cb;
    cb = lw % n_cb;
    return true;
}

constexpr int OB = 2 * NB;                 // a TSQR panel pair (one factor_block)
constexpr int OB2 = 2 * OB;                // outer block of the trailing update: two panel pairs

// Tiles of the two products, four waves each.  The small ones spread the narrow products of the
// panel chain (64 or 128 columns) and short matrices over more workgroups.  Bound by the matrix
// cores and, at the tiles' ends, by what the CU's other workgroups leave to do: in FP64, waves of
// 64 x 32 with two or three workgroups per CU against 128 x 128 tiles of eight waves, 70,000 x
// 10,000: Y^T C 127 -> 124 ms, C - Y W 111 -> 107 ms (60 and 62 TFLOP/s); 128 x 128 tiles of four
// waves 124 and 113, 256 x 64 124 and 109 with spills.
template <class T>
struct QrTiles;
template <>
struct QrTiles<double> {
    using WL = KTile<double, OB, 64, 8, 2, 2>;  // P = Y^T C over a row chunk
    static constexpr int WL_WAVES = 2;          // per SIMD
    using WS = KTile<double, 64, 64, 8, 2, 2>;
    using UL = MTile<double, 64, 128, 8, 2, 2>;  // C^T -= W^T Y^T (rows of C along the MFMA N axis)
    using US = MTile<double, 64, 64, 8, 2, 2>;
};
template <>
struct QrTiles<float> {
    using WL = KTile<float, OB, 128, 4, 2, 2>;
    static constexpr int WL_WAVES = 3;
    using WS = KTile<float, 64, 64, 4, 2, 2>;
    using UL = MTile<float, 128, 128, 8, 2, 2>;
    using US = MTile<float, 64, 64, 8, 1, 1>;
};

// Element of row r of a unit lower trapezoid's column whose diagonal row is diag (PLAIN: a
// column that is taken as it is).
constexpr int64_t PLAIN = INT64_MIN;
template <class T>
DEV T unit_lower(T v, int64_t r, int64_t diag)
{
    return r > diag ? v : (r == diag ? T(1) : T(0));
}

// P[ch][p][q] = sum over the chunk's rows r of Y[r][p] C[r][q].  Y is the
// block at (j0, j0) of width pw; C is either columns c0 .. c0+nt of A
// (ymode = 0) or the unit lower trapezoidal block at (c0, c0) of width nt
// (ymode = 1, used for Y_A^T Y_B with rows below Y_A's triangle).  Rows r0 .. m.  Both operands
// are contiguous along the summed rows and go straight to LDS, except in the stages that
// meet a unit triangle and a ragged last one.
template <class S, int WAVES>
__global__ __launch_bounds__(S::NT, WAVES) void qr_wpart_kernel(
    QrWork w, int64_t j0, int pw, int64_t c0, int64_t nt, int ymode, int64_t r0, int64_t chunk)
{
    using T = typename S::elem;
    __shared__ __align__(16) typename S::unit lds[2 * S::UNITS];
    // blockIdx.z: rows S::BM z .. of P
    const int prow0 = S::BM * (int)blockIdx.z;
    j0 += prow0;
    pw = (pw - prow0) < S::BM ? (pw - prow0) : S::BM;
    if (pw <= 0)
        return;
    const int64_t ch = blockIdx.y;
    const int64_t q0 = (int64_t)blockIdx.x * S::BN;
    const int64_t rlo = r0 + ch * chunk;
    int64_t rhi = rlo + chunk;
    if (rhi > w.m)
        rhi = w.m;
    if (rlo >= rhi)
        return;
    const T *A = qmat<T>(w);
    const int64_t lda = w.lda;
    // rows of P past pw and columns past nt repeat the last one and are not stored
    const T *src[S::LPT];
#pragma unroll
    for (int i = 0; i < S::LPT; ++i) {
        const int r = S::unit_row(i);
        const int64_t q = q0 + r - S::BM;
        const int64_t col = r < S::BM ? j0 + (r < pw ? r : pw - 1) : c0 + (q < nt ? q : nt - 1);
        src[i] = A + col * lda + rlo + S::unit_k(i);
    }
    const int64_t tri_end = ymode ? c0 + nt : j0 + pw;  // rows before it may meet the triangle
    const int len = (int)(rhi - rlo), nk = (len + S::BK - 1) / S::BK;
    const int km = tri_end > rlo ? (int)(tri_end - rlo) : 0;
    typename S::acc4 acc[S::FM][S::FN];
    ktile_zero<S>(acc);
    ktile_product_masked<S>(acc, lds, src, nk, (km + S::BK - 1) / S::BK, len / S::BK, [&](int kt, int i) {
        // (reads stay inside the column: rlo and BK are multiples of 16, lda of 64)
        typename S::unit v;
        __builtin_memcpy(&v, __builtin_assume_aligned(src[i] + (int64_t)kt * S::BK, 16), 16);
        const int r = S::unit_row(i);
        const int64_t row = rlo + kt * S::BK + S::unit_k(i);
        const int64_t diag = r < S::BM ? (ymode ? PLAIN : j0 + r) : (ymode ? c0 + q0 + r - S::BM : PLAIN);
#pragma unroll
        for (int e = 0; e < S::V; ++e)
            v[e] = row + e < rhi ? unit_lower<T>(v[e], row + e, diag) : T(0);
        return v;
    });
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, g = lane >> 4, rl = lane & 15;
    const int wm = wave / S::WN, wn = wave % S::WN;
    double *P = w.wpart + (ch * OB2 + prow0) * w.wp_ld;
#pragma unroll
    for (int i = 0; i < S::FM; ++i)
#pragma unroll
        for (int j = 0; j < S::FN; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int p = wm * S::TM + 16 * i + Unit<T>::acc_m(g, e);
                const int64_t q = q0 + wn * S::TN + 16 * j + rl;
                if (p < pw && q < nt)
                    P[p * w.wp_ld + q] = (double)acc[i][j][e];
            }
}

// W = T^T P of a block of one or two panel pairs a | b, from the chunk partials of P = Y^T C:
// W_a = T_a^T P_a, and with pair b W_b = T_b^T (P_b - H^T P_a) (see the note on the blocks
// below).  A workgroup takes 16 columns: it sums their chunk partials into LDS (even chunks,
// odd chunks, then the two sums), and its four waves form the products on MFMA, the factors'
// operands read straight from L2.  One launch instead of three; 64-column workgroups of
// scalar sums took 41 us for the narrow updates of the panel chain, this 11-13 us.
constexpr int W_CHUNKS = 8;  // chunk partials that qr_w_kernel sums itself (an even number)
struct WArgs {
    const double *Ta, *Tb, *H;  // row-major, T upper triangular with zeros below
    int tld, pwa, pwb;          // T_a's leading dimension (T_b and H: OB); pair widths
    int64_t nch, nt;
};
template <class TW>
__global__ __launch_bounds__(256) void qr_w_kernel(QrWork w, WArgs a, TW *__restrict__ W)
{
    __shared__ double Ps[OB2][16];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, g = lane >> 4, r = lane & 15;
    const int64_t q0 = (int64_t)blockIdx.x * 16;
    {
        const int ql = t & 15;
        const int64_t q = q0 + ql, step = (int64_t)OB2 * w.wp_ld;
        const int halves = a.pwb > 0 ? 2 : 1;
        constexpr int NU = OB / 16;
        for (int h = 0; h < halves; ++h) {
            double v[NU][W_CHUNKS];  // all loads in flight
#pragma unroll
            for (int u = 0; u < NU; ++u) {
                const int p = (t >> 4) + 16 * u;
                const bool in = q < a.nt && p < (h ? a.pwb : a.pwa);
                const double *src = w.wpart + (in ? (h * OB + p) * w.wp_ld + q : 0);
#pragma unroll
                for (int ch = 0; ch < W_CHUNKS; ++ch)
                    v[u][ch] = in && ch < a.nch ? src[ch * step] : 0.0;
            }
#pragma unroll
            for (int u = 0; u < NU; ++u) {
                double s0 = 0.0, s1 = 0.0;
#pragma unroll
                for (int ch = 0; ch < W_CHUNKS; ch += 2) {
                    s0 += v[u][ch];
                    s1 += v[u][ch + 1];
                }
                Ps[h * OB + (t >> 4) + 16 * u][ql] = s0 + s1;
            }
        }
    }
    __syncthreads();
    // rows 16 mb .. of T^T P (T upper triangular: terms s <= p), P rows from LDS row base
    auto tri = [&](const double *T, int ld, int mb, int base, int pw) {
        double av[OB / 16][4];  // all loads in flight
        const int p = 16 * mb + r;
#pragma unroll
        for (int sb = 0; sb < OB / 16; ++sb)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int sr = 16 * sb + 4 * e + g;
                av[sb][e] = (sb <= mb && sr < pw && p < pw) ? T[sr * ld + p] : 0.0;
            }
        d4 acc = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int sb = 0; sb < OB / 16; ++sb)
            if (sb <= mb)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    acc = Unit<double>::mfma(av[sb][e], Ps[base + 16 * sb + 4 * e + g][r], acc);
        return acc;
    };
    auto put = [&](int prow, int pw, int mb, const d4 &acc) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int p = 16 * mb + g + 4 * e;
            if (p < pw && q0 + r < a.nt)
                W[(prow + p) * w.ldw + q0 + r] = (TW)acc[e];
        }
    };
#pragma unroll
    for (int q = 0; q < 2; ++q) {  // block rows wave and 7 - wave: nine steps per wave
        const int mb = q ? 7 - wave : wave;
        if (16 * mb < a.pwa)
            put(0, a.pwa, mb, tri(a.Ta, a.tld, mb, 0, a.pwa));
    }
    if (a.pwb <= 0)
        return;
    // P_b -= H^T P_a
    d4 pb[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int mb = wave + 4 * q;
#pragma unroll
        for (int e = 0; e < 4; ++e)
            pb[q][e] = Ps[OB + 16 * mb + g + 4 * e][r];
        if (16 * mb < a.pwb) {
            double av[OB / 16][4];  // zeros past pwa and pwb
#pragma unroll
            for (int sb = 0; sb < OB / 16; ++sb)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    av[sb][e] = a.H[(16 * sb + 4 * e + g) * OB + 16 * mb + r];
#pragma unroll
            for (int sb = 0; sb < OB / 16; ++sb)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    pb[q] = Unit<double>::mfma(-av[sb][e], Ps[16 * sb + 4 * e + g][r], pb[q]);
        }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int e = 0; e < 4; ++e)
            Ps[OB + 16 * (wave + 4 * q) + g + 4 * e][r] = pb[q][e];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int mb = q ? 7 - wave : wave;
        if (16 * mb < a.pwb)
            put(OB, a.pwb, mb, tri(a.Tb, OB, mb, OB, a.pwb));
    }
}

// Sum of the split-K partials over the row chunks into chunk 0's slot, one
// (p, q) element per thread (even chunks, odd chunks, then the two sums), for many
// chunks: qr_w_kernel then reads a single one (its own sums run on only
// ceil(nt / 16) workgroups).
__global__ __launch_bounds__(256) void qr_psum_kernel(QrWork w, int pw, int64_t nch, int64_t nt)
{
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (e >= (int64_t)pw * nt)
        return;
    const int64_t p = e / nt, q = e % nt;
    double *src = w.wpart + p * w.wp_ld + q;
    const int64_t step = (int64_t)OB2 * w.wp_ld;
    double s0 = 0.0, s1 = 0.0;
    int64_t ch = 0;
#pragma unroll 8
    for (; ch + 1 < nch; ch += 2) {
        s0 += src[ch * step];
        s1 += src[(ch + 1) * step];
    }
    if (ch < nch)
        s0 += src[ch * step];
    src[0] = s0 + s1;
}

// G = Y_A^T Y_B from the chunk partials (one entry per thread: ld x ld
// entries, rows p < ld of the partials, columns q < pwb, G row-major with leading
// dimension ld; chunks summed in the same fixed order as qr_psum_kernel).
__global__ __launch_bounds__(256) void qr_gsum_kernel(QrWork w, int pwb, int64_t nch, double *__restrict__ G, int ld)
{
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (e >= ld * ld)
        return;
    const int p = e / ld, q = e % ld;
    double s0 = 0.0, s1 = 0.0;
    if (q < pwb) {
        const double *src = w.wpart + p * w.wp_ld + q;
        const int64_t step = (int64_t)OB2 * w.wp_ld;
        int64_t ch = 0;
#pragma unroll 8
        for (; ch + 1 < nch; ch += 2) {
            s0 += src[ch * step];
            s1 += src[(ch + 1) * step];
        }
        if (ch < nch)
            s0 += src[ch * step];
    }
    G[e] = s0 + s1;
}

// Combined compact-WY factor of two consecutive panels A | B:
// T = [[T_A, -T_A G T_B], [0, T_B]] with G = Y_A^T Y_B (summed by qr_gsum_kernel).  The two
// products run on MFMA, a wave per 16 rows; bound by the latency of its loads, all issued at
// the start (67 us; 25 with loads one after the other; 8).
__global__ __launch_bounds__(256) void qr_tcombine_kernel(QrWork w, const double *__restrict__ Gs,
                                                         double *__restrict__ Tout)
{
    __shared__ double G[NB][DL], B[NB][DL];  // G, then T_A; T_B, then X
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, g = lane >> 4, r = lane & 15;
    const double *Ta = w.Tin, *Tb = w.Tin + NB * NB;
    constexpr int NQ = NB * NB / 256;
    double gv[NQ], tav[NQ], tbv[NQ];  // all loads in flight
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        gv[q] = Gs[q * 256 + t];
        tbv[q] = Tb[q * 256 + t];
        tav[q] = Ta[q * 256 + t];
    }
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const int i = q * 4 + wave, c = lane;
        G[i][c] = gv[q];
        B[i][c] = tbv[q];
        Tout[i * OB + c] = tav[q];
        Tout[(NB + i) * OB + c] = 0.0;
        Tout[(NB + i) * OB + NB + c] = tbv[q];
    }
    __syncthreads();
    d4 acc[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {  // X = G T_B
        acc[c] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int k = 0; k < 4 * (c + 1); ++k)
            acc[c] = mfma16(G[16 * wave + r][4 * k + g], B[4 * k + g][16 * c + r], acc[c]);
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e)
            B[16 * wave + g + 4 * e][16 * c + r] = acc[c][e];
#pragma unroll
    for (int q = 0; q < NQ; ++q)
        G[q * 4 + wave][lane] = tav[q];
    __syncthreads();
#pragma unroll
    for (int c = 0; c < 4; ++c) {  // -T_A X (T_A's zeros below its diagonal included)
        acc[c] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int k = 0; k < NB / 4; ++k)
            acc[c] = mfma16(-G[16 * wave + r][4 * k + g], B[4 * k + g][16 * c + r], acc[c]);
#pragma unroll
        for (int e = 0; e < 4; ++e)
            Tout[(16 * wave + g + 4 * e) * OB + NB + 16 * c + r] = acc[c][e];
    }
}

// ---------------------------------------------------------------------------
// A trailing-update block of two panel pairs a | b (up to 256 columns).  Its
// compact-WY factor is T = [[T_a, -T_a G T_b], [0, T_b]] with G = Y_a^T Y_b, so
// W = T^T P for P = Y^T C splits into W_a = T_a^T P_a and
// W_b = T_b^T (P_b - H^T P_a) with H = T_a G: the two 128-row halves reuse the
// 128-column reduction, and the update C -= Y W runs once with depth 256.
// ---------------------------------------------------------------------------

// H = T_a G (T_a upper triangular pwa x pwa, row-major ld tld, zeros below; G and H row-major,
// leading dimension OB; zeros past pwa and pwb): one 16 x 16 block per wave, 16 workgroups.
__global__ __launch_bounds__(256) void qr_hmat_kernel(const double *__restrict__ Ta, int tld, int pwa,
                                                      const double *__restrict__ G, int pwb, double *__restrict__ H)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, g = lane >> 4, r = lane & 15;
    const int bi = blockIdx.x >> 1, bj = 4 * (blockIdx.x & 1) + wave;
    d4 acc = d4{0.0, 0.0, 0.0, 0.0};
    const int i = 16 * bi + r, j = 16 * bj + r;
    double av[OB / 16][4], bv[OB / 16][4];  // all loads in flight
#pragma unroll
    for (int kb = 0; kb < OB / 16; ++kb)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int k = 16 * kb + 4 * e + g;
            const bool in = kb >= bi && k < pwa;
            av[kb][e] = in && i < pwa ? Ta[i * tld + k] : 0.0;
            bv[kb][e] = in && j < pwb ? G[k * OB + j] : 0.0;
        }
#pragma unroll
    for (int kb = 0; kb < OB / 16; ++kb)
        if (kb >= bi)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                acc = mfma16(av[kb][e], bv[kb][e], acc);
#pragma unroll
    for (int e = 0; e < 4; ++e)
        H[(16 * bi + g + 4 * e) * OB + j] = acc[e];
}

// C[r][q] -= sum_p Y[r][p] W[p][q] for rows j0.. and columns c0 .. c0+nt; the
// tile is computed transposed so that consecutive lanes own consecutive rows.
// The accumulators start from -C (its loads in flight with the first
// operand slices), so the epilogue is a plain store.  Y and W go straight to LDS, except
// where a row block meets Y's unit triangle and in a ragged last slice.
template <class S>
__global__ __launch_bounds__(S::NT, 3) void qr_update_kernel(
    QrWork w, int64_t j0, int pw, int64_t c0, int64_t nt)
{
    using T = typename S::elem;
    __shared__ __align__(16) typename S::unit lds[2 * S::UNITS];
    int64_t rb, cb;
    if (!update_tile((w.m - j0 + S::BN - 1) / S::BN, (nt + S::BM - 1) / S::BM, rb, cb))
        return;
    const int64_t q0 = cb * S::BM, r0 = j0 + rb * S::BN;
    const T *A = qmat<T>(w);
    T *C = qmat<T>(w) + c0 * w.lda;
    const T *W = sizeof(T) == 8 ? reinterpret_cast<const T *>(w.W) : reinterpret_cast<const T *>(w.W32);
    const int64_t lda = w.lda, m = w.m, ldW = w.ldw;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, g = lane >> 4, rl = lane & 15;
    const int wm = wave / S::WN, wn = wave % S::WN;
    const bool inside = r0 + S::BN <= m && q0 + S::BM <= nt;  // no checks on C
    typename S::acc4 acc[S::FM][S::FN];
#pragma unroll
    for (int i = 0; i < S::FM; ++i)
#pragma unroll
        for (int j = 0; j < S::FN; j += S::V)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int64_t q = q0 + S::row(wm, i, g, e), r = r0 + S::col(wn, j, rl);
                typename S::unit v;
                if (inside) {
                    __builtin_memcpy(&v, __builtin_assume_aligned(C + q * lda + r, 16), 16);
                } else {
#pragma unroll
                    for (int h = 0; h < S::V; ++h)
                        v[h] = (q < nt && r + h < m) ? C[q * lda + r + h] : T(0);
                }
#pragma unroll
                for (int h = 0; h < S::V; ++h)
                    acc[i][j + h][e] = -v[h];
            }
    // columns past nt and rows past m (and past lda: the next column's) are computed, not stored
    const T *src[S::LPT];
    int64_t step[S::LPT];
#pragma unroll
    for (int i = 0; i < S::LPT; ++i) {
        const int x = S::unit_x(i);
        const int64_t p = S::unit_p(i);
        src[i] = x < S::UA ? W + p * ldW + q0 + S::V * x : A + (j0 + p) * lda + r0 + S::V * (x - S::UA);
        step[i] = S::BK * (x < S::UA ? ldW : lda);
    }
    const bool masked = r0 < j0 + pw;  // the row block meets Y's unit upper triangle
    mtile_product<S>(acc, lds, (pw + S::BK - 1) / S::BK, masked ? 0 : pw / S::BK, src, step, [&](int kt, int i) {
        const int x = S::unit_x(i);
        const int64_t p = kt * S::BK + S::unit_p(i);
        const T *at = x < S::UA ? W + q0 + S::V * x : A + j0 * lda + r0 + S::V * (x - S::UA);
        typename S::unit v;
        __builtin_memcpy(&v, __builtin_assume_aligned(at + (p < pw ? p : 0) * (x < S::UA ? ldW : lda), 16), 16);
        const int64_t diag = x < S::UA ? PLAIN : j0 + p;
#pragma unroll
        for (int h = 0; h < S::V; ++h)
            v[h] = p < pw ? unit_lower<T>(v[h], r0 + S::V * (x - S::UA) + h, diag) : T(0);
        return v;
    });
    // recompute the store addresses rather than keep the loads' live through the product
    int64_t q0s = q0, r0s = r0;
    asm volatile("" : "+s"(q0s), "+s"(r0s));
#pragma unroll
    for (int i = 0; i < S::FM; ++i)
#pragma unroll
        for (int j = 0; j < S::FN; j += S::V)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int64_t q = q0s + S::row(wm, i, g, e), r = r0s + S::col(wn, j, rl);
                typename S::unit v;
#pragma unroll
                for (int h = 0; h < S::V; ++h)
                    v[h] = -acc[i][j + h][e];
                if (inside) {
                    __builtin_memcpy(__builtin_assume_aligned(C + q * lda + r, 16), &v, 16);
                } else if (q < nt) {
#pragma unroll
                    for (int h = 0; h < S::V; ++h)
                        if (r + h < m)
                            C[q * lda + r + h] = v[h];
                }
            }
}

// w with its rows cut to those that can be nonzero in columns [0, j_end): below a
// trailing upper-triangular block's row tri0 + j_end, every column before j_end
// is still zero, so the reflectors of those columns are zero there and leave
// those rows unchanged.
static QrWork rows_to(const QrWork &w, int64_t j_end)
{
    QrWork r = w;
    if (w.tri0 > 0 && w.tri0 + j_end < w.m)
        r.m = w.tri0 + j_end;
    return r;
}

// TSQR + reconstruction of the panel at (j0, j0) of width pw; its T goes to Tout.
template <class T>
static void factor_panel(const QrWork &wf, int64_t j0, int pw, double *Tout, hipStream_t s)
{
    const QrWork w = rows_to(wf, j0 + pw);
    if (w.panel == 0) {
        if constexpr (sizeof(T) == 8)
            cqr_panel_f64(w, j0, pw, Tout, s);
        else
            cqr_panel_f32(w, j0, pw, Tout, s);
        return;
    }
    const int64_t mk = w.m - j0;
    const PanelTree pt = panel_tree(mk);
    for (int l = 0; l < pt.levels; ++l)
        hipLaunchKernelGGL(tsqr_factor_kernel<T>, dim3((unsigned)pt.nodes[l]), dim3(TS_NT), 0, s, w, j0, pw, l,
                           pt.nodes[l], l > 0 ? pt.nodes[l - 1] : 0, mk);
    for (int l = pt.levels - 1; l >= 0; --l)
        hipLaunchKernelGGL(tsqr_formq_kernel<T>, dim3((unsigned)pt.nodes[l]), dim3(TS_NT), 0, s, w, j0, pw, l,
                           pt.nodes[l], l == pt.levels - 1 ? 1 : 0, mk);
    hipLaunchKernelGGL(tsqr_lu_kernel<T>, dim3(1), dim3(256), 0, s, w, j0, pw, pt.levels - 1, Tout);
    if (mk > pw)
        hipLaunchKernelGGL(tsqr_trsm_kernel<T>, dim3((unsigned)((mk - pw + 255) / 256)), dim3(256), 0, s, w, j0,
                           pw);
}

// P = Y^T C for the block at (j0, j0) of width pw, split over row chunks; returns their number.
template <class T>
static int64_t launch_wpart(const QrWork &w, int64_t j0, int pw, int64_t c0, int64_t nt, int ymode, int64_t r0,
                            int64_t target, hipStream_t s)
{
    using L = typename QrTiles<T>::WL;
    using M = typename QrTiles<T>::WS;
    const QrSplit q = qr_split(w.m - r0, pw, nt, L::BM, L::BN, sizeof(T) == 4, target, w.max_chunks);
    const dim3 grid((unsigned)q.nq, (unsigned)q.nch, (unsigned)q.np);
    static_assert(M::BM == QR_SMALL_TILE && M::BN == QR_SMALL_TILE, "small tiles");
    if (q.small)
        hipLaunchKernelGGL((qr_wpart_kernel<M, 3>), grid, dim3(M::NT), 0, s, w, j0, pw, c0, nt, ymode, r0, q.chunk);
    else
        hipLaunchKernelGGL((qr_wpart_kernel<L, QrTiles<T>::WL_WAVES>), grid, dim3(L::NT), 0, s, w, j0, pw, c0, nt,
                           ymode, r0, q.chunk);
    return q.nch;
}

// The compact-WY data of a trailing-update block at column J: panel pair a
// (pwa <= OB columns, T_a) and, when present, pair b (pwb columns, T_b) with
// H = T_a Y_a^T Y_b.  Storage: four OB x OB row-major matrices (Ta, Tb, G, H).
struct BlockT {
    double *store;
    int pwa = 0, pwb = 0;
    const double *ta = nullptr;  // T_a as apply_block reads it (row-major, ld tld); null: Ta()
    int tld = OB;
    double *Ta() const { return store; }
    double *Tb() const { return store + OB * OB; }
    double *G() const { return store + 2 * OB * OB; }
    double *H() const { return store + 3 * OB * OB; }
    int pw() const { return pwa + pwb; }
};

// C := (I - Y T Y^T)^T C for the columns c0 .. c0+nt, Y the block at (J, J).
template <class T>
static void apply_block(const QrWork &wf, int64_t J, const BlockT &bt, int64_t c0, int64_t nt, hipStream_t s)
{
    if (nt <= 0)
        return;
    const int pw = bt.pw();
    const QrWork w = rows_to(wf, J + pw);
    const int64_t rows = w.m - J;
    WArgs a{};
    a.nch = launch_wpart<T>(w, J, pw, c0, nt, 0, J, w.split_wgs, s);
    if (a.nch > W_CHUNKS) {
        hipLaunchKernelGGL(qr_psum_kernel, dim3((unsigned)(((int64_t)pw * nt + 255) / 256)), dim3(256), 0, s, w, pw,
                           a.nch, nt);
        a.nch = 1;
    }
    a.Ta = bt.ta ? bt.ta : bt.Ta();
    a.tld = bt.ta ? bt.tld : OB;
    a.Tb = bt.pwb > 0 ? bt.Tb() : nullptr;
    a.H = bt.pwb > 0 ? bt.H() : nullptr;
    a.pwa = bt.pwa;
    a.pwb = bt.pwb;
    a.nt = nt;
    if constexpr (sizeof(T) == 8)
        hipLaunchKernelGGL(qr_w_kernel<double>, dim3((unsigned)((nt + 15) / 16)), dim3(256), 0, s, w, a, w.W);
    else
        hipLaunchKernelGGL(qr_w_kernel<float>, dim3((unsigned)((nt + 15) / 16)), dim3(256), 0, s, w, a, w.W32);
    // the large tiles from two per CU on (from 256, 1,024 or 2,048 tiles on: within 1 %)
    using L = typename QrTiles<T>::UL;
    using M = typename QrTiles<T>::US;
    auto tiles = [](int64_t x, int64_t b) { return (x + b - 1) / b; };
    auto grid = [](int64_t n) { return dim3((unsigned)((n + 7) & ~int64_t(7))); };
    const int64_t nl = tiles(rows, L::BN) * tiles(nt, L::BM), nm = tiles(rows, M::BN) * tiles(nt, M::BM);
    if (nl >= 512)
        hipLaunchKernelGGL(qr_update_kernel<L>, grid(nl), dim3(L::NT), 0, s, w, J, pw, c0, nt);
    else
        hipLaunchKernelGGL(qr_update_kernel<M>, grid(nm), dim3(M::NT), 0, s, w, J, pw, c0, nt);
}

// The small-scratch view w for products with up to OB2 columns (the same buffers).
static QrWork wide_view(const QrWork &w)
{
    QrWork r = w;
    r.wp_ld = OB2;
    r.ldw = OB2;
    r.max_chunks = MAX_CHUNKS_S / 2;
    return r;
}

// Factor the panel pair at column J (main-stream scratch in w): panel A, its
// update of panel B, panel B, and the pair's compact-WY T (row-major, copied
// to Tdst with leading dimension OB).  Returns the pair's width.
//
// With the matrix's last column in the pair, only the right-hand side is left: each panel is
// applied to it directly (it lies beside panel B's columns) and no T is combined.  64 x 200
// configurations, M = 256: 126 us less than combining the last block's T for one column.
template <class T>
static int factor_pair(const QrWork &w, int64_t J, double *Tdst, hipStream_t s)
{
    double *Ta = w.Tin, *Tb = w.Tin + NB * NB;
    const int pwa = (int)((w.n - J) < NB ? (w.n - J) : NB);
    const int64_t jb = J + pwa, nrhs = w.ncols - w.n;
    const int pwb = (int)((w.n - jb) < NB ? (w.n - jb) : NB);
    const bool last = jb + pwb == w.n;
    factor_panel<T>(w, J, pwa, Ta, s);
    const BlockT pa{nullptr, pwa, 0, Ta, NB};  // panel A alone
    apply_block<T>(w, J, pa, jb, pwb + (last ? nrhs : 0), s);
    if (pwb == 0)
        return pwa;
    factor_panel<T>(w, jb, pwb, Tb, s);
    if (last) {
        const BlockT pb{nullptr, pwb, 0, Tb, NB};
        apply_block<T>(w, jb, pb, w.n, nrhs, s);
        return pwa + pwb;
    }
    const QrWork wg = rows_to(w, jb + pwb);  // G = Y_a^T Y_b
    const int64_t nch = launch_wpart<T>(wg, J, pwa, jb, (int64_t)pwb, 1, jb, 2048, s);
    hipLaunchKernelGGL(qr_gsum_kernel, dim3(NB * NB / 256), dim3(256), 0, s, wg, pwb, nch, wg.cq_G, NB);
    hipLaunchKernelGGL(qr_tcombine_kernel, dim3(1), dim3(256), 0, s, w, (const double *)w.cq_G, Tdst);
    return pwa + pwb;
}

// Factor the trailing-update block at column J: panel pair a, its update of
// pair b's columns, pair b, then G = Y_a^T Y_b and H = T_a G.  bt.store holds the
// results; returns the block's width (up to OB2).  The last block also updates the
// right-hand side, and leaves no T.
template <class T>
static int factor_block(const QrWork &w, int64_t J, BlockT &bt, hipStream_t s)
{
    bt.pwa = factor_pair<T>(w, J, bt.Ta(), s);
    bt.pwb = 0;
    const int64_t jb = J + bt.pwa;
    const int pwb_max = (int)((w.n - jb) < OB ? (w.n - jb) : OB);
    if (pwb_max <= 0)
        return bt.pwa;
    const bool last = jb + pwb_max == w.n;
    BlockT a{bt.store, bt.pwa, 0};
    if (last)
        apply_block<T>(wide_view(w), J, a, jb, w.ncols - jb, s);
    else
        apply_block<T>(w, J, a, jb, pwb_max, s);
    bt.pwb = factor_pair<T>(w, jb, bt.Tb(), s);
    if (last)
        return bt.pw();
    const QrWork wg = rows_to(w, jb + bt.pwb);  // G = Y_a^T Y_b
    const int64_t nch = launch_wpart<T>(wg, J, bt.pwa, jb, (int64_t)bt.pwb, 1, jb, 2048, s);
    hipLaunchKernelGGL(qr_gsum_kernel, dim3(OB * OB / 256), dim3(256), 0, s, wg, bt.pwb, nch, bt.G(), OB);
    hipLaunchKernelGGL(qr_hmat_kernel, dim3(16), dim3(256), 0, s, (const double *)bt.Ta(), OB, bt.pwa,
                       (const double *)bt.G(), bt.pwb, bt.H());
    return bt.pw();
}

template <class T>
static void geqrf(const QrWork &w, hipStream_t s, const QrAsync *la)
{
    // small-scratch views: wn for the products inside a block (at most OB rows
    // and columns of P), its wide view for the main stream's update of the next block (OB2)
    QrWork wn = w;
    wn.wpart = w.wpart_s;
    wn.wp_ld = OB;
    wn.W = w.W_s;
    wn.W32 = w.W32_s;
    wn.ldw = OB;
    wn.max_chunks = MAX_CHUNKS_S;  // more row chunks keep the panel chain's GEMMs wide
    const QrWork wm = wide_view(wn);
    if (!la) {
        BlockT bt{w.T};
        for (int64_t J = 0; J < w.n; J += bt.pw()) {
            factor_block<T>(wn, J, bt, s);
            if (J + bt.pw() < w.n)
                apply_block<T>(w, J, bt, J + bt.pw(), w.ncols - (J + bt.pw()), s);
        }
        return;
    }
    BlockT bt[2] = {BlockT{w.T}, BlockT{w.T2}};
    (void)hipEventRecord(la->fork, s);
    (void)hipStreamWaitEvent(la->side, la->fork, 0);
    factor_block<T>(wn, 0, bt[0], s);
    (void)hipEventRecord(la->t_ready, s);
    int64_t k = 0;
    for (int64_t J = 0; J < w.n; ++k) {
        const BlockT &cur = bt[k & 1];
        const int64_t cn = J + cur.pw();                          // first column of block k+1
        const int64_t nn = (w.n - cn) < OB2 ? (w.n - cn) : OB2;   // its width
        if (nn <= 0)
            break;
        // side: block k's update of everything right of block k+1 (b included)
        (void)hipStreamWaitEvent(la->side, la->t_ready, 0);
        apply_block<T>(w, J, cur, cn + nn, w.ncols - (cn + nn), la->side);
        (void)hipEventRecord(la->bulk[k & 1], la->side);
        // main: block k+1's columns need every earlier block's update first; its
        // T buffer is the one block k-1's side update read
        if (k > 0)
            (void)hipStreamWaitEvent(s, la->bulk[(k - 1) & 1], 0);
        apply_block<T>(wm, J, cur, cn, nn, s);
        if (cn + nn == w.n)  // the last block updates the right-hand side itself
            (void)hipStreamWaitEvent(s, la->bulk[k & 1], 0);
        factor_block<T>(wn, cn, bt[(k + 1) & 1], s);
        (void)hipEventRecord(la->t_ready, s);
        J = cn;
    }
    (void)hipEventRecord(la->join, la->side);
    (void)hipStreamWaitEvent(s, la->join, 0);
}

hipError_t launch_geqrf(const QrWork &w, hipStream_t s, const QrAsync *la)
{
    if (w.A32)
        geqrf<float>(w, s, la);
    else
        geqrf<double>(w, s, la);
    return hipGetLastError();
}

}  // namespace gap
