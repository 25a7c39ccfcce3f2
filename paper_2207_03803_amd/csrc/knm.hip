// K_NM / K_MM builder: descriptor GEMM on FP64 MFMA with the dot-product
// covariance, the per-configuration segment-sum and the Sigma^-1/2 row scale
// fused into the epilogue (Sec. Theory: definition of K_MN; the upper block of
// A; Eqs. 1-2).  The n_atoms x M matrix of atom-level covariances is never
// written to HBM.
#include "knm.h"
#include "small64.h"

#include <atomic>
#include <type_traits>

namespace gap {

// ---------------------------------------------------------------------------
// Tile plan.  The rows of K_NM are independent per configuration, so a tile
// may hold any set of whole configurations.  The configurations are split, in
// order, into chunks of at most PLAN_C; each chunk is sorted by atom count (largest
// first, then by index) and packed: a configuration of more than
// KNM_CAP atoms gets a tile of its own (processed in atom chunks); the others
// fill tiles of at most KNM_CAP atoms and KNM_MAX_SEG configurations, each
// tile taking the largest remaining configuration that still fits until none
// does.  Output: cfg_list (the configurations, tile by tile) and tile_start[t]
// (the first position of tile t in cfg_list).  The offsets are validated too.
//
// One wave packs a chunk; each step takes as many configurations of one size as fit, so a
// chunk of 512 is about 200 dependent steps: 82 us (50 with 256, 33 with 128), where one
// thread per chunk of 2048 took 743 us (143 us for 200 configurations).  The tiles of U[8, 64]-atom
// configurations are 99.1 % full with chunks of 512, about 3.5 / chunk short of full.
// ---------------------------------------------------------------------------
constexpr int PLAN_C = 512;                // configurations per chunk, at most (a power of two)
constexpr int PLAN_C_LEAST = 128;          // and at least

// Configurations per chunk: a chunk costs 0.15 us per configuration, and a K_NM of T us loses
// 3.5 T / chunk to its chunks' last tiles; 128 up to 1.3 ms, 256 up to 4.5 ms (at 63 TFLOP/s).
int knm_plan_chunk(int64_t n_atoms, int64_t M, int64_t d)
{
    const double flops = 2.0 * (double)n_atoms * (double)M * (double)d;
    return flops < 8.2e10 ? PLAN_C_LEAST : (flops < 2.8e11 ? 256 : PLAN_C);
}
constexpr int PLAN_LARGE = KNM_CAP + 1;    // bucket of the configurations above KNM_CAP atoms
constexpr int PLAN_WORDS = (KNM_CAP + 64) / 64;

static int64_t plan_chunks(int64_t N, int chunk) { return (N + chunk - 1) / chunk; }
// cfg_list [N] and, per chunk, its tile count and first positions (16 bits each)
int64_t knm_plan_ints(int64_t N, int chunk) { return N + plan_chunks(N, chunk) * (chunk / 2); }
int64_t knm_plan_room(int64_t N) { return knm_plan_ints(N, PLAN_C); }

// lists: chunk c's tile starts at [c * chunk]; entry 0, always position 0, holds the tile
// count instead.
__global__ __launch_bounds__(256) void plan_chunk_kernel(const int64_t *__restrict__ offsets, int64_t N,
                                                         int64_t n_atoms, int chunk, int32_t *__restrict__ cfg_list,
                                                         uint16_t *__restrict__ lists, int32_t *status)
{
    __shared__ int32_t key[PLAN_C];
    __shared__ int32_t bfirst[64 * PLAN_WORDS], blast[64 * PLAN_WORDS];
    __shared__ uint32_t bucket[64 * PLAN_WORDS];  // bfirst | items left << 16
    __shared__ uint16_t order[PLAN_C];
    __shared__ int bad_s, nlarge_s;
    const int t = threadIdx.x;
    const int64_t c0 = (int64_t)blockIdx.x * chunk;
    const int cnt = (int)((N - c0) < chunk ? (N - c0) : chunk);
    uint16_t *ls = lists + blockIdx.x * (int64_t)chunk;
    if (t == 0) {
        bad_s = 0;
        nlarge_s = 0;
        if (blockIdx.x == 0 && offsets[0] != 0)
            bad_s = 1;
        if (c0 + cnt == N && offsets[N] != n_atoms)
            bad_s = 1;
    }
    for (int b = t; b < 64 * PLAN_WORDS; b += 256)
        bfirst[b] = blast[b] = 0;
    __syncthreads();
    // key = (PLAN_LARGE - bucket) << 16 | local index: ascending = largest first
    for (int i = t; i < chunk; i += 256) {
        int32_t k = INT32_MAX;
        if (i < cnt) {
            const int64_t sz = offsets[c0 + i + 1] - offsets[c0 + i];
            if (sz < 0)
                bad_s = 1;
            const int b = sz > KNM_CAP ? PLAN_LARGE : (sz < 0 ? 0 : (int)sz);
            k = ((PLAN_LARGE - b) << 16) | i;
        }
        key[i] = k;
    }
    __syncthreads();
    for (int kk = 2; kk <= chunk; kk <<= 1)
        for (int jj = kk >> 1; jj > 0; jj >>= 1) {
            // pair p: its lower element i has bit jj clear
            const int i = 2 * t - (t & (jj - 1)), l = i | jj;
            if (l < chunk) {
                const int32_t x = key[i], y = key[l];
                if ((x > y) == ((i & kk) == 0)) {
                    key[i] = y;
                    key[l] = x;
                }
            }
            __syncthreads();
        }
    // bucket b occupies sorted positions [bfirst[b], blast[b]); the large ones come first
    for (int i = t; i < cnt; i += 256) {
        const int b = PLAN_LARGE - (key[i] >> 16);
        const bool head = i == 0 || (key[i - 1] >> 16) != (key[i] >> 16);
        const bool tail = i == cnt - 1 || (key[i + 1] >> 16) != (key[i] >> 16);
        if (b == PLAN_LARGE) {
            if (tail)
                nlarge_s = i + 1;
        } else {
            if (head)
                bfirst[b] = i;
            if (tail)
                blast[b] = i + 1;
        }
    }
    __syncthreads();
    if (bad_s) {
        if (t == 0) {
            set_status(status, DST_EINVAL);
            ls[0] = 0;
        }
        return;
    }
    if (t < 64) {
        const int nlarge = __builtin_amdgcn_readfirstlane(nlarge_s);
        for (int i = t; i < nlarge; i += 64) {  // one tile each
            order[i] = (uint16_t)i;
            if (i > 0)
                ls[i] = (uint16_t)i;
        }
        // non-empty buckets 0..KNM_CAP as a bit set, word w in lane w; some: its non-empty words
        uint64_t word = 0;
        uint32_t some = 0;
#pragma unroll
        for (int w = 0; w < PLAN_WORDS; ++w) {
            const int b = 64 * w + t, left = blast[b] - bfirst[b];
            bucket[b] = (uint32_t)bfirst[b] | (uint32_t)left << 16;
            const uint64_t m = __ballot(left > 0);
            if (t == w)
                word = m;
            some |= m ? 1u << w : 0u;
        }
        auto word_of = [&](int w) -> uint64_t {
            return (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(word >> 32), w) << 32 |
                   (uint32_t)__builtin_amdgcn_readlane((int)word, w);
        };
        int pos = nlarge, ntile = nlarge;
        while (pos < cnt) {
            if (t == 0 && ntile > 0)
                ls[ntile] = (uint16_t)pos;
            ++ntile;
            int r = KNM_CAP, nseg = 0;
            while (nseg < KNM_MAX_SEG) {
                // largest non-empty bucket b <= r
                int w = r >> 6;
                uint64_t m = word_of(w) & ((2ull << (r & 63)) - 1);
                if (m == 0) {
                    const uint32_t lower = some & ((1u << w) - 1);
                    if (lower == 0)
                        break;
                    w = 31 - __clz(lower);
                    m = word_of(w);
                }
                const int found = w * 64 + 63 - __clzll(m);
                // as many of its items as fit (r / found: the half keeps the quotient of these
                // small integers away from a whole number)
                const uint32_t bk = __builtin_amdgcn_readfirstlane(bucket[found]);
                const int i0 = bk & 0xffff, left = bk >> 16;
                int take = found > 0 ? (int)(((float)r + 0.5f) * __builtin_amdgcn_rcpf((float)found)) : left;
                take = __builtin_amdgcn_readfirstlane(take);
                take = take < left ? take : left;
                take = take < KNM_MAX_SEG - nseg ? take : KNM_MAX_SEG - nseg;
                for (int q = t; q < take; q += 64)
                    order[pos + q] = (uint16_t)(i0 + q);
                if (t == 0)
                    bucket[found] = (uint32_t)(i0 + take) | (uint32_t)(left - take) << 16;
                if (take == left) {
                    if (t == w)
                        word &= ~(1ull << (found & 63));
                    if (word_of(w) == 0)
                        some &= ~(1u << w);
                }
                pos += take;
                nseg += take;
                r -= take * found;
            }
        }
        if (t == 0)
            ls[0] = (uint16_t)ntile;
    }
    __syncthreads();
    for (int i = t; i < cnt; i += 256)
        cfg_list[c0 + i] = (int32_t)(c0 + (key[order[i]] & 0xffff));
}

// Global tile table: tile_start[base_c + j] = chunk c's j-th tile, n_tiles.
__global__ __launch_bounds__(256) void plan_publish_kernel(const uint16_t *__restrict__ lists, int64_t n_chunks,
                                                           int chunk, int64_t N, int32_t *__restrict__ tile_start,
                                                           int32_t *__restrict__ n_tiles, int64_t max_tiles,
                                                           int32_t *status)
{
    __shared__ int64_t sum_s[4];
    const int64_t c = blockIdx.x;
    int64_t before = 0;
    for (int64_t q = threadIdx.x; q < c; q += 256)
        before += lists[q * chunk];
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1)
        before += __shfl_xor(before, o, 64);
    if ((threadIdx.x & 63) == 0)
        sum_s[threadIdx.x >> 6] = before;
    __syncthreads();
    const int64_t base = (sum_s[0] + sum_s[1]) + (sum_s[2] + sum_s[3]), nt = lists[c * chunk];
    const bool bad = (*status != 0) || base + nt > max_tiles;
    if (!bad)
        for (int64_t j = threadIdx.x; j < nt; j += 256)
            tile_start[base + j] = (int32_t)(c * chunk + (j > 0 ? lists[c * chunk + j] : 0));
    if (c == n_chunks - 1 && threadIdx.x == 0) {
        if (bad) {
            if (base + nt > max_tiles)
                set_status(status, DST_EINVAL);
            *n_tiles = 0;
        } else {
            tile_start[base + nt] = (int32_t)N;
            *n_tiles = (int32_t)(base + nt);
        }
    }
}

int64_t knm_max_tiles(int64_t N, int64_t n_atoms, int chunk)
{
    // Within a chunk, a tile closes only when the largest remaining
    // configuration does not fit, so two consecutive tiles hold more than
    // KNM_CAP atoms unless the first was closed by the configuration cap; each
    // chunk may end with one more partial tile.
    int64_t bound = 2 * ((n_atoms + KNM_CAP - 1) / KNM_CAP) + (N + KNM_MAX_SEG - 1) / KNM_MAX_SEG +
                    plan_chunks(N, chunk) + 1;
    return bound < N ? bound : N;
}
int64_t knm_tiles_room(int64_t N, int64_t n_atoms) { return knm_max_tiles(N, n_atoms, PLAN_C_LEAST); }

// 256 threads, 4 waves of 64 x BN (BN = 64 by default, 32 as a tuning choice), BK = 8.
// Bound by the FP64 matrix cores; two workgroups share a CU and one's tile set-up and
// epilogue run beside the other's MFMAs.  901,000 atoms x 10,000 x 400: 134 ms (53.7
// TFLOP/s) with K-major stages filled through registers and 4x4x4 MFMAs, 114 ms (63.0)
// now.  8 waves of 64 x 32 need 128 VGPRs for the same occupancy and spill: 118 ms.
template <int BN>
using KSB = KTile<double, KNM_BM, BN, 4, 4, 1>;
using KS = KSB<KNM_BN>;
constexpr int KNM_NT = 256;
static_assert(KS::NT == KNM_NT && KSB<32>::NT == KNM_NT, "K_NM kernels assume 256 threads");

constexpr int EPC = 32;           // epilogue columns per pass
constexpr int EPLD = EPC + 1;     // padded LDS row of the epilogue buffer

template <int BN>
constexpr int knm_lds_units()
{
    return (2 * KSB<BN>::UNITS > KNM_BM * EPLD / 2) ? 2 * KSB<BN>::UNITS : KNM_BM * EPLD / 2;
}

// A derivative position whose gradient row and atom are in range.
DEV bool kdm_valid(const KnmArgs &a, int64_t pos)
{
    const int64_t g = a.pos_grad[pos];
    return g >= 0 && g < a.n_grad && a.grad_atom[g] >= 0 && a.grad_atom[g] < a.n_src;
}

// What a segment's rows are: a configuration's atoms, one point (K_MM), or an observation's
// positions.
enum KnmRows { CONFIGS, POINTS, POSITIONS };

// One workgroup's tile; bid = the workgroup's index within this K_NM's own grid
// (a multiple-of-8 offset into a grouped grid keeps bid's XCD the hardware's).
template <int BN, KnmRows ROWS = CONFIGS>
DEV void knm_body(const KnmArgs &a, int64_t bid)
{
    constexpr bool DERIV = ROWS == POSITIONS, unit = ROWS == POINTS;
    using KS = KSB<BN>;
    constexpr int KNM_BN = BN;
    static_assert(BN == 32 || BN == 64, "column tile of 32 or 64 sparse points");
    __shared__ __align__(16) d2 lds[knm_lds_units<BN>()];
    __shared__ int32_t sstart[KNM_MAX_SEG + 1];  // atom offset of each segment within the tile
    __shared__ int32_t scan_tot[KNM_MAX_SEG / 64];
    __shared__ int64_t rowpos[KNM_BM];           // row of X of each tile row (-1: none)
    __shared__ int64_t sbase[KNM_MAX_SEG];       // first atom (row of X) of each segment
    __shared__ int32_t srow[KNM_MAX_SEG];        // output row of each segment
    __shared__ double carry[KNM_BN];
    __shared__ double rowf[DERIV ? KNM_BM : 1];      // derivative rows: zeta sw2 w of tile row r
    __shared__ int64_t rowatom[DERIV ? KNM_BM : 1];  // and its gradient's atom (-1 past the tile)

    // The grid is sized for the largest possible tile count; the remap uses
    // the actual count so that all eight XCDs get an equal share of the tiles.
    const int64_t n_tiles = unit ? (a.n_rows_unit + KNM_BM - 1) / KNM_BM : (int64_t)*a.n_tiles_dev;
    int64_t t, ct;
    if constexpr (DERIV) {
        // tiles dealt to the XCDs in turn (tile t to XCD t mod 8), each tile's column
        // tiles on its XCD in order: observations of very different sizes (multi-chunk
        // virials beside small force components) spread evenly over the XCDs
        const int64_t tiles8 = (n_tiles + 7) / 8;
        if (bid >= tiles8 * 8 * a.n_ct)
            return;
        const int64_t x = bid & 7, q = bid >> 3;
        t = 8 * (q / a.n_ct) + x;
        ct = q % a.n_ct;
        if (t >= n_tiles)
            return;
    } else {
        const int64_t total = n_tiles * a.n_ct;
        const int64_t total_pad = (total + 7) & ~int64_t(7);
        if (bid >= total_pad)
            return;
        const int64_t lw = xcd_remap(bid, total_pad);
        if (lw >= total)
            return;
        t = lw / a.n_ct;
        ct = lw % a.n_ct;
    }
    const int64_t col0 = ct * KNM_BN;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave / KS::WN, wn = wave % KS::WN;

    // K_MM, upper triangle only: a tile wholly below the diagonal is zero (no product)
    if (unit && a.upper_only && t * KNM_BM > col0 + KNM_BN - 1) {
        const int64_t r0 = t * KNM_BM;
        const int nr = (int)((a.n_rows_unit - r0) < KNM_BM ? (a.n_rows_unit - r0) : KNM_BM);
        for (int item = tid; item < nr * KNM_BN; item += KS::NT) {
            const int r = item % nr, c = item / nr;
            const int64_t colg = col0 + c;
            if (colg < a.M)
                a.out[colg * a.ldo + a.row_off + r0 + r] = 0.0;
        }
        return;
    }

    // The tile's segments: rows of the unit block, or configurations from the plan.
    int n_seg;
    int64_t n_at;  // atoms in the tile
    if (unit) {
        const int64_t r0 = t * KNM_BM;
        n_seg = (int)((a.n_rows_unit - r0) < KNM_BM ? (a.n_rows_unit - r0) : KNM_BM);
        if (tid == 0)
            sstart[0] = 0;
        if (tid < n_seg) {
            sstart[tid + 1] = tid + 1;
            sbase[tid] = r0 + tid;
            srow[tid] = (int32_t)(r0 + tid);
        }
        n_at = n_seg;
    } else {
        const int64_t p0 = a.tile_start[t];
        n_seg = (int)(a.tile_start[t + 1] - p0);
        int64_t sz = 0;
        if (tid < n_seg) {
            const int32_t cfg = a.cfg_list[p0 + tid];
            const int64_t lo = a.offsets[cfg];
            sz = a.offsets[cfg + 1] - lo;
            sbase[tid] = lo;
            srow[tid] = cfg;
        }
        // inclusive scan of the segment sizes (one per thread of the first four waves)
        int32_t incl = (int32_t)sz;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int32_t x = __shfl_up(incl, off, 64);
            if (lane >= off)
                incl += x;
        }
        if (tid < KNM_MAX_SEG && lane == 63)
            scan_tot[wave] = incl;
        __syncthreads();
        if (tid < KNM_MAX_SEG) {
            for (int q = 0; q < wave; ++q)
                incl += scan_tot[q];
            sstart[tid + 1] = incl;
        }
        if (tid == 0)
            sstart[0] = 0;
        __syncthreads();
        n_at = sstart[n_seg];
    }
    __syncthreads();

    // Row scale of segment s (loaded where its latency can overlap other work).
    auto sig = [&](int s) { return a.sigma ? a.sigma[srow[s]] : 1.0; };
    auto emit = [&](int s, int64_t colg, double sum, double sg) {
        const int64_t row = srow[s];
        double v = sum;
        if (unit) {
            if (row == colg)
                v += a.jitter;
            if (a.upper_only && row > colg)
                v = 0.0;
        }
        if (a.sigma)
            v = v / sg;
        a.out[colg * a.ldo + a.row_off + row] = v;
    };

    if (n_at == 0) {  // only empty configurations: their sums are zero
        for (int item = tid; item < n_seg * KNM_BN; item += KS::NT) {
            const int s = item % n_seg, c = item / n_seg;
            const int64_t colg = col0 + c;
            if (colg < a.M)
                emit(s, colg, 0.0, sig(s));
        }
        return;
    }

    const bool multi = n_at > KNM_BM;  // then n_seg == 1: a configuration in several atom chunks
    const bool direct = rows_aligned16(a.X, a.d) && rows_aligned16(a.XM, a.d);
    d4 acc[KS::FM][KS::FN];
    for (int64_t cs = 0; cs < n_at; cs += KNM_BM) {
        const bool first = (cs == 0), last = (cs + KNM_BM >= n_at);
        // the tile rows' positions: segment by binary search (the first one when multi)
        if (tid < KNM_BM) {
            int64_t pos = -1;
            if (cs + tid < n_at) {
                int lo = 0, hi = multi ? 0 : n_seg - 1;
                while (lo < hi) {
                    const int mid = (lo + hi + 1) >> 1;
                    if (sstart[mid] <= tid)
                        lo = mid;
                    else
                        hi = mid - 1;
                }
                pos = sbase[lo] + (cs + tid - sstart[lo]);
            }
            if constexpr (DERIV) {
                // this tile row's weight and its gradient's atom
                if (pos >= 0 && !kdm_valid(a, pos)) {
                    pos = -1;  // the row counts as zero
                    set_status(a.status, DST_EINVAL);
                }
                rowf[tid] = pos >= 0 ? a.zeta * a.sw2 * a.pos_weight[pos] : 0.0;
                rowatom[tid] = pos >= 0 ? a.grad_atom[a.pos_grad[pos]] : -1;
                if (pos >= 0)
                    pos = a.pos_grad[pos];
            }
            rowpos[tid] = pos;
        }
        __syncthreads();
        // this thread's units; a missing atom row or sparse row reads the first sparse row
        // (its products are never used)
        const double *src[KS::LPT];
#pragma unroll
        for (int i = 0; i < KS::LPT; ++i) {
            const int r = KS::unit_row(i);
            const double *p = a.XM;
            if (r < KNM_BM) {
                const int64_t pos = rowpos[r];
                if (pos >= 0)
                    p = a.X + pos * (int64_t)a.d;
            } else if (col0 + r - KNM_BM < a.M) {
                p = a.XM + (col0 + r - KNM_BM) * (int64_t)a.d;
            }
            src[i] = p + KS::unit_k(i);
        }
#pragma unroll
        for (int i = 0; i < KS::FM; ++i)
#pragma unroll
            for (int j = 0; j < KS::FN; ++j)
                acc[i][j] = d4{0.0, 0.0, 0.0, 0.0};
        ktile_product<KS>(acc, lds, src, a.d, direct);

        if constexpr (DERIV) {
            // d k / dr = zeta sigma_w^2 (x_i . x_j)^(zeta - 1) (x' . x_j), times the
            // position's weight: applied below as the values are parked
        } else {
            // k = sigma_w^2 g^zeta, in registers.
#pragma unroll
            for (int i = 0; i < KS::FM; ++i)
#pragma unroll
                for (int j = 0; j < KS::FN; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        acc[i][j][e] = a.sw2 * ipow(acc[i][j][e], a.zeta);
        }

        double *E = reinterpret_cast<double *>(lds);  // [256][EPLD], reused after the GEMM
        for (int p = 0; p < (KNM_BN + EPC - 1) / EPC; ++p) {
            // waves owning columns of the pass park their values in LDS
            if (wn * KS::TN < (p + 1) * EPC && (wn + 1) * KS::TN > p * EPC) {
#pragma unroll
                for (int i = 0; i < KS::FM; ++i)
#pragma unroll
                    for (int j = 0; j < KS::FN; ++j)
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const int cl = acc_col<KS>(wn, j, lane, e) - p * EPC;
                            if (cl >= 0 && cl < EPC) {
                                const int r = acc_row<KS>(wm, i, lane, e);
                                double v = acc[i][j][e];
                                if constexpr (DERIV) {
                                    // (rowf / rowatom were written before the GEMM's barriers)
                                    const int64_t at = rowatom[r], colg = col0 + p * EPC + cl;
                                    const double dv = (a.D && at >= 0 && colg < a.M) ? a.D[at * a.ldd + colg] : 1.0;
                                    v = at >= 0 ? v * (rowf[r] * dv) : 0.0;
                                }
                                E[r * EPLD + cl] = v;
                            }
                        }
            }
            __syncthreads();
            if (unit) {  // one row per thread
                if (tid < n_seg) {
                    const double sg = sig(tid);
#pragma unroll 8
                    for (int c = 0; c < EPC; ++c) {
                        const int64_t colg = col0 + p * EPC + c;
                        if (colg < a.M)
                            emit(tid, colg, E[tid * EPLD + c], sg);
                    }
                }
            } else if (!multi) {
                for (int item = tid; item < n_seg * EPC; item += KS::NT) {
                    const int s = item % n_seg, c = item / n_seg;
                    const int64_t colg = col0 + p * EPC + c;
                    if (colg >= a.M)
                        continue;
                    // in atom order; the loads of 8 (then 4) rows are issued together
                    const double sg = sig(s);
                    const int a1 = sstart[s + 1];
                    int r = sstart[s];
                    double sum = 0.0;
                    for (; r + 8 <= a1; r += 8) {
                        double v[8];
#pragma unroll
                        for (int k = 0; k < 8; ++k)
                            v[k] = E[(r + k) * EPLD + c];
#pragma unroll
                        for (int k = 0; k < 8; ++k)
                            sum += v[k];
                    }
                    if (r + 4 <= a1) {
                        double v[4];
#pragma unroll
                        for (int k = 0; k < 4; ++k)
                            v[k] = E[(r + k) * EPLD + c];
#pragma unroll
                        for (int k = 0; k < 4; ++k)
                            sum += v[k];
                        r += 4;
                    }
                    for (; r < a1; ++r)
                        sum += E[r * EPLD + c];
                    emit(s, colg, sum, sg);
                }
            } else if (tid < EPC) {
                const int c = tid;
                const int64_t colg = col0 + p * EPC + c;
                const int nr = (int)((n_at - cs) < KNM_BM ? (n_at - cs) : KNM_BM);
                double sum = 0.0;
                for (int r = 0; r < nr; ++r)
                    sum += E[r * EPLD + c];
                const double tot = first ? sum : carry[p * EPC + c] + sum;
                carry[p * EPC + c] = tot;
                if (last && colg < a.M)
                    emit(0, colg, tot, sig(0));
            }
            __syncthreads();
        }
    }
}

template <int BN, KnmRows ROWS>
__global__ __launch_bounds__(KNM_NT, 2) void knm_kernel(KnmArgs a)
{
    knm_body<BN, ROWS>(a, blockIdx.x);
}

// Derivative observation rows: the K_NM tile loop over the observations' positions.
__global__ __launch_bounds__(KNM_NT, 2) void kdm_kernel(KnmArgs a) { knm_body<64, POSITIONS>(a, blockIdx.x); }

// ---------------------------------------------------------------------------
// Derivative rows in two steps, where gradient rows serve several positions (a force
// component and the virials of its configuration): for a block of w columns, first
// H[g][j] = zeta sw2 D(i(g), j) (x'_g . x_j) of every gradient row g, once, into scratch (bound
// by the matrix cores), then each observation's weighted sum of rows of H (bound by the cache
// that holds H).  The tile loop over positions (kdm_kernel) multiplies a row once per position:
// 150 configurations (234,000 rows, 702,000 positions, M = 1,500, d = 400) take 8.1 ms here,
// 20.0 there.  64-row tiles: 96-column blocks are 3.6 rounds of 128-row ones, 400 us against 364.
// ---------------------------------------------------------------------------
template <int BN>
using GradTile = KTile<double, 64, BN, 8, 2, 2>;

template <class S>
__global__ __launch_bounds__(S::NT, 3) void grad_rows_kernel(KnmArgs a, int64_t col0, int w, double *__restrict__ H)
{
    __shared__ __align__(16) d2 lds[2 * S::UNITS];
    const int64_t n_ct = (w + S::BN - 1) / S::BN, total = (a.n_grad + S::BM - 1) / S::BM * n_ct;
    const int64_t lw = xcd_remap(blockIdx.x, (total + 7) & ~int64_t(7));
    if (lw >= total)
        return;
    const int64_t r0 = lw / n_ct * S::BM, c0 = lw % n_ct * S::BN;  // rows, columns of the block
    const int64_t cols = a.M - col0 < w ? a.M - col0 : w;
    const double *src[S::LPT];
#pragma unroll
    for (int i = 0; i < S::LPT; ++i) {
        const int r = S::unit_row(i);
        const double *p;
        if (r < S::BM)  // rows and columns past the end repeat the last one, unused
            p = a.X + (r0 + r < a.n_grad ? r0 + r : a.n_grad - 1) * (int64_t)a.d;
        else
            p = a.XM + (col0 + (c0 + r - S::BM < cols ? c0 + r - S::BM : cols - 1)) * (int64_t)a.d;
        src[i] = p + S::unit_k(i);
    }
    d4 acc[S::FM][S::FN];
    ktile_zero<S>(acc);
    ktile_product<S>(acc, lds, src, a.d, rows_aligned16(a.X, a.d) && rows_aligned16(a.XM, a.d));
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = wave / S::WN, wn = wave % S::WN;
    const double f = a.zeta * a.sw2;
#pragma unroll
    for (int i = 0; i < S::FM; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int64_t g = r0 + acc_row<S>(wm, i, lane, e);
            if (g >= a.n_grad)
                continue;
            const int64_t at = a.grad_atom[g];
            const bool ok = at >= 0 && at < a.n_src;  // (reported where a position uses the row)
#pragma unroll
            for (int j = 0; j < S::FN; ++j) {
                const int64_t c = c0 + acc_col<S>(wn, j, lane, e);
                if (c < cols)
                    H[g * w + c] = ok ? acc[i][j][e] * (f * (a.D ? a.D[at * a.ldd + col0 + c] : 1.0)) : 0.0;
            }
        }
}

// Rows of A for the columns col0 .. of the block: observation o's sum over its positions p of
// w_p H[pos_grad[p]], in position order, one wave per observation and 64 columns (one column per
// lane); an observation of more than LONG_OBS positions is cut into four runs, one per wave,
// added in order.
constexpr int LONG_OBS = 64;
__global__ __launch_bounds__(256) void obs_sum_kernel(KnmArgs a, int64_t n_obs, int64_t n_pos, int64_t col0, int w,
                                                      const double *__restrict__ H)
{
    __shared__ double part[4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t o0 = 4 * (int64_t)blockIdx.x;
    const int64_t c = 64 * (int64_t)blockIdx.y + lane;
    const bool in = c < w && col0 + c < a.M;
    const double *Hc = H + (in ? c : 0);
    auto run = [&](int64_t lo, int64_t hi) {
        double s = 0.0;
        for (int64_t p0 = lo; p0 < hi; p0 += 64) {
            // 64 positions' rows and weights at once, one per lane; then rows of H in flight 16 (8, 4) at a time
            const int cnt = (int)(hi - p0 < 64 ? hi - p0 : 64);
            int64_t g = lane < cnt ? a.pos_grad[p0 + lane] : 0;
            const bool ok = g >= 0 && g < a.n_grad;
            const double wt = lane < cnt && ok ? a.pos_weight[p0 + lane] : 0.0;
            const int row = ok ? (int)g : 0;
            auto rows = [&](int p, auto n) {
                double v[decltype(n)::value];
#pragma unroll
                for (int k = 0; k < decltype(n)::value; ++k)
                    v[k] = Hc[(int64_t)__builtin_amdgcn_readlane(row, p + k) * w];
#pragma unroll
                for (int k = 0; k < decltype(n)::value; ++k)
                    s += readlane_d(wt, p + k) * v[k];
            };
            int p = 0;
            for (; p + 16 <= cnt; p += 16)
                rows(p, std::integral_constant<int, 16>());
            if (p + 8 <= cnt) {
                rows(p, std::integral_constant<int, 8>());
                p += 8;
            }
            if (p + 4 <= cnt) {
                rows(p, std::integral_constant<int, 4>());
                p += 4;
            }
            for (; p < cnt; ++p)
                rows(p, std::integral_constant<int, 1>());
        }
        return s;
    };
    auto emit = [&](int64_t o, double s) {
        if (in)
            a.out[(col0 + c) * a.ldo + a.row_off + o] = s / a.sigma[o];
    };
    if (blockIdx.x == 0 && threadIdx.x == 0 && (a.offsets[0] != 0 || a.offsets[n_obs] != n_pos))
        set_status(a.status, DST_EINVAL);
    for (int k = 0; k < 4; ++k) {
        const int64_t o = o0 + k;
        if (o >= n_obs)
            break;
        const int64_t lo = a.offsets[o], hi = a.offsets[o + 1];
        if (lo < 0 || hi < lo || hi > n_pos) {
            if (threadIdx.x == 0)
                set_status(a.status, DST_EINVAL);
            continue;
        }
        if (col0 == 0 && blockIdx.y == 0)  // the positions' indices, checked once
            for (int64_t p = lo + threadIdx.x; p < hi; p += 256)
                if (!kdm_valid(a, p))
                    set_status(a.status, DST_EINVAL);
        if (hi - lo <= LONG_OBS) {
            if (wave == k)
                emit(o, run(lo, hi));
        } else {
            const int64_t q = (hi - lo + 3) / 4;
            const int64_t l = lo + wave * q < hi ? lo + wave * q : hi, h = l + q < hi ? l + q : hi;
            part[wave][lane] = run(l, h);
            __syncthreads();
            if (wave == 0)
                emit(o, (part[0][lane] + part[1][lane]) + (part[2][lane] + part[3][lane]));
            __syncthreads();
        }
    }
}

// The K_NM of several fits in one grid: fit i owns workgroups [base[i], base[i+1]).
template <int BN>
__global__ __launch_bounds__(KNM_NT, 2) void knm_group_kernel(KnmGroup g)
{
    const int64_t b = blockIdx.x;
    int i = 0;
    while (i + 1 < g.n && b >= g.base[i + 1])
        ++i;
    knm_body<BN>(g.f[i], b - g.base[i]);
}

// ---------------------------------------------------------------------------
// Prediction (Eqs. 1-2): y_A = sum_{i in A} sum_j c_j sigma_w^2 (x_i . x_j)^zeta.
//
// The order of the sums is the same whatever the request: within a column tile of KNM_BN
// sparse points as the wave adds them up, the tiles of a group of PRED_G in order, the groups in
// order, then the configuration's atoms in order.  So a configuration's energy does not depend,
// to the bit, on the configurations beside it or on how the work is split.
//
// The atoms are cut into tiles of consecutive rows, the sparse points into runs of one column
// tile or of a whole group; workgroup (tile, run) forms its atoms' energies over its run (the
// atom-by-sparse covariances stay in registers).  A second kernel adds up an atom's runs and a
// configuration's atoms.  One request's column runs thus spread over the chip: with one
// workgroup per few configurations and all columns, a single configuration against 4,000
// points took 4.2 ms on one CU, and 4,096 configurations 21 ms with the
// CUs a third idle in the last round.  A request whose energies exceed what a call may claim is
// taken in ranges of atoms, one after the other.
//
// The atoms' energies lie in a static pool of PRED_CHUNKS chunks of 1 MiB per GPU (a predict
// call has no workspace).  Every call has a number of its own; its first kernel claims the
// consecutive chunks it needs by writing that number into their owner words, the other kernels look
// for it there, and the last workgroup of the last one frees them.  Nothing of a call's state lies in
// memory that another call may write, the caller's output included.  Claiming on the device works for any
// streams, threads and captured graphs (whose replays, one after the other, keep their number),
// and never waits: with no room free, the
// second kernel computes its groups' atoms itself, with the same sums in the same order.
//
// Bound by the matrix cores from a few hundred configurations on (d = 400, M = 4,000:
// 4,096 configurations 21.5 -> 7.3 ms, 64 TFLOP/s; d = 256, M = 2,250: 333
// configurations 3.2 -> 0.26 ms; d = 128, M = 1,000: 150,000 configurations in nine ranges 39.8 ->
// 25.4 ms), by the latency of the column tile's k loop below (one configuration 4,230 -> 30 us,
// three launches).  Without room in the pool a request takes about the time on the left.
// ---------------------------------------------------------------------------
constexpr int PRED_G = 4;               // column tiles of a group
constexpr int PRED_CHUNKS = 128;
constexpr int64_t PRED_CHUNK = 131072;  // doubles of a chunk
constexpr int PRED_MAX = 20;            // chunks of one call, at most
static __device__ double g_pred_pool[PRED_CHUNKS * PRED_CHUNK];
static __device__ unsigned long long g_pred_owner[PRED_CHUNKS];  // the call's number; 0: free
static __device__ unsigned g_pred_done[PRED_CHUNKS];             // arrivals, at the call's first chunk
static_assert(PRED_CHUNKS == 128 && PRED_MAX <= 64, "two owner words per lane; one lane per claimed chunk");

// Both tile heights give waves of 64 columns and the same order of every sum.
using PSL = KTile<double, KNM_BM, KNM_BN, 4, 4, 1>;  // 256 atoms
using PSS = KTile<double, 64, KNM_BN, 8, 4, 1>;     // 64 atoms
static_assert(PSL::TN == PSS::TN && PSL::WN == 1 && PSS::WN == 1 && PSL::NT == KNM_NT, "one summation order");
static_assert(PSS::NT == KNM_NT && PSL::BM == KNM_NT, "a thread per atom");

struct PredArgs {
    const double *X;
    const int64_t *offsets;
    int64_t N, n_atoms;
    const double *XM;
    int64_t M;
    int d, zeta;
    double sw2;
    const double *c;
    double *y;
    int32_t *status;
    int64_t C;              // configurations per group (checked together; a bad one makes the group NaN)
    int64_t n_ct;           // column tiles
    int run;                // column tiles per run: 1 or PRED_G (0: the atoms' energies are not kept)
    int64_t n_runs;
    int64_t a0, a1;         // the atoms of this range
    int64_t tiles, ld;      // atom tiles, and atoms they cover: a run's energies lie ld apart
    int chunks;             // claimed
    unsigned long long id;  // the call's number (positive)
};

// Energy of atom row0 + threadIdx.x (the first S::BM threads) over column tiles [ct0, ct1).
template <class S>
DEV double predict_tile_energy(const PredArgs &a, int64_t row0, int64_t ct0, int64_t ct1, d2 *lds, double *part)
{
    const int tid = threadIdx.x, lane = tid & 63, wm = tid >> 6;
    const bool direct = rows_aligned16(a.X, a.d) && rows_aligned16(a.XM, a.d);
    double e_sum = 0.0;
    for (int64_t ct = ct0; ct < ct1; ++ct) {
        const int64_t col0 = ct * S::BN;
        const double *src[S::LPT];
#pragma unroll
        for (int i = 0; i < S::LPT; ++i) {
            const int r = S::unit_row(i);
            const double *p = a.XM;  // a missing row reads the first sparse row, unused below
            if (r < S::BM) {
                if (row0 + r < a.n_atoms)
                    p = a.X + (row0 + r) * (int64_t)a.d;
            } else if (col0 + r - S::BM < a.M) {
                p = a.XM + (col0 + r - S::BM) * (int64_t)a.d;
            }
            src[i] = p + S::unit_k(i);
        }
        d4 acc[S::FM][S::FN];
        ktile_zero<S>(acc);
        ktile_product<S>(acc, lds, src, a.d, direct);
        double cw[S::FN];
        bool in[S::FN];
#pragma unroll
        for (int j = 0; j < S::FN; ++j) {
            const int64_t col = col0 + acc_col<S>(0, j, lane, 0);
            in[j] = col < a.M;
            cw[j] = in[j] ? a.c[col] : 0.0;
        }
#pragma unroll
        for (int i = 0; i < S::FM; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                double s = 0.0;
#pragma unroll
                for (int j = 0; j < S::FN; ++j)
                    s += in[j] ? cw[j] * (a.sw2 * ipow(acc[i][j][e], a.zeta)) : 0.0;
                // the 16 lanes that share l / 16 share this row
                s += __shfl_xor(s, 1, 64);
                s += __shfl_xor(s, 2, 64);
                s += __shfl_xor(s, 4, 64);
                s += __shfl_xor(s, 8, 64);
                if ((lane & 15) == 0)
                    part[acc_row<S>(wm, i, lane, e)] = s;
            }
        __syncthreads();
        if (tid < S::BM)
            e_sum += part[tid];
    }
    return e_sum;
}

// Where the call's part of the pool starts (-1: it has none), the same in every lane.
DEV int64_t pred_base(unsigned long long id)
{
    const int lane = threadIdx.x & 63;
    const auto owner = [](int k) {
        return __hip_atomic_load(&g_pred_owner[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    const uint64_t lo = __ballot(owner(lane) == id), hi = __ballot(owner(64 + lane) == id);
    const int k = lo ? __builtin_ctzll(lo) : (hi ? 64 + __builtin_ctzll(hi) : -1);
    return k < 0 ? -1 : k * PRED_CHUNK;
}

// Gives back what a call holds whose last kernel could not be launched.
__global__ __launch_bounds__(PRED_CHUNKS) void predict_release_kernel(unsigned long long id)
{
    if (atomicCAS(&g_pred_owner[threadIdx.x], id, 0ull) == id)
        g_pred_done[threadIdx.x] = 0u;
}

// One wave claims a.chunks consecutive free chunks, each lane one of them; if another call took one
// of them meanwhile, it gives the others back and looks again.
constexpr int CLAIM_TRIES = 16;
__global__ __launch_bounds__(64) void predict_claim_kernel(PredArgs a)
{
    const int lane = threadIdx.x;
    const auto owner = [](int k) {
        return __hip_atomic_load(&g_pred_owner[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    for (int t = 0; t < CLAIM_TRIES; ++t) {
        const uint64_t lo = __ballot(owner(lane) == 0ull), hi = __ballot(owner(64 + lane) == 0ull);
        int at = -1;
        for (int k = 0, run = 0; k < PRED_CHUNKS && at < 0; ++k) {
            run = ((k < 64 ? lo >> k : hi >> (k - 64)) & 1) ? run + 1 : 0;
            if (run == a.chunks)
                at = k + 1 - run;
        }
        if (at < 0)
            return;
        const bool mine = lane < a.chunks && atomicCAS(&g_pred_owner[at + lane], 0ull, a.id) == 0ull;
        if (__popcll(__ballot(mine)) == a.chunks)
            return;
        if (mine)
            __hip_atomic_store(&g_pred_owner[at + lane], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

template <class S>
__global__ __launch_bounds__(S::NT, S::BM == 64 ? 3 : 2) void predict_tile_kernel(PredArgs a)
{
    __shared__ __align__(16) d2 lds[2 * S::UNITS];
    __shared__ double part[S::BM];
    const int64_t total = a.tiles * a.n_runs;
    const int64_t lw = xcd_remap(blockIdx.x, (total + 7) & ~int64_t(7));
    if (lw >= total)
        return;
    const int64_t base = pred_base(a.id);
    if (base < 0)
        return;
    const int64_t t = lw / a.n_runs, s = lw % a.n_runs;
    const int64_t ct0 = s * a.run, ct1 = ct0 + a.run < a.n_ct ? ct0 + a.run : a.n_ct;
    const double e = predict_tile_energy<S>(a, a.a0 + t * S::BM, ct0, ct1, lds, part);
    if (threadIdx.x < S::BM)
        g_pred_pool[base + s * a.ld + t * S::BM + threadIdx.x] = e;
}

// Adds up to B of an atom's run energies, at p, p + ld, ... (p the same in every lane, t the atom; n of
// them) to e: groups of PRED_G column tiles in order, as a workgroup that takes a whole group adds
// them. All loads in flight, those past the last run repeated (a branch around each costs more).
template <int B>
DEV void pred_add_runs(const PredArgs &a, const double *&p, int n, int t, double &e)
{
    static_assert(B % PRED_G == 0, "whole groups");
    double v[B];
#pragma unroll
    for (int k = 0; k < B; ++k) {
        v[k] = p[t];
        p += k + 1 < n || k + 1 == B ? a.ld : 0;
    }
#pragma unroll
    for (int k = 0; k < B; ++k)
        v[k] = k < n ? v[k] : 0.0;
    if (a.run == 1) {
#pragma unroll
        for (int k = 0; k < B; k += PRED_G) {
            double g = 0.0;
#pragma unroll
            for (int q = 0; q < PRED_G; ++q)
                g += v[k + q];
            e += g;
        }
    } else {
#pragma unroll
        for (int k = 0; k < B; ++k)
            e += v[k];
    }
}

// v, known to be the same in every lane.
DEV int64_t uniform(int64_t v)
{
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)v), hi = __builtin_amdgcn_readfirstlane((unsigned)(v >> 32));
    return (int64_t)((uint64_t)hi << 32 | lo);
}

// One group of configurations: checks their offsets, then adds up their atoms' energies, 256 atoms at a
// time, for the atoms of the range.  LAST: the last range; the group's result if its offsets are bad, and all
// of its atoms if the call has no part of the pool.  (The ranges before pass most groups by at
// once; without the code and the LDS of the tiles more of them do so at a time.)
template <bool LAST>
__global__ __launch_bounds__(KNM_NT, LAST ? 2 : 4) void predict_sum_kernel(PredArgs a)
{
    using S = PSL;
    __shared__ __align__(16) d2 lds[LAST ? 2 * S::UNITS : 1];
    __shared__ double part[LAST ? S::BM : 1];
    __shared__ double eps[S::BM];
    __shared__ int bad_s, last_s;
    const int tid = threadIdx.x;
    const int64_t cfg_lo = (int64_t)blockIdx.x * a.C;
    const int64_t cfg_hi = (cfg_lo + a.C < a.N) ? cfg_lo + a.C : a.N;
    const int ncfg = (int)(cfg_hi - cfg_lo);
    const int64_t g0 = a.offsets[cfg_lo], g1 = a.offsets[cfg_hi];
    if (!LAST && (g1 < a.a0 || g0 >= a.a1))
        return;
    const int64_t base = a.run > 0 ? pred_base(a.id) : -1;
    if (!LAST && base < 0)
        return;
    // Every configuration must be a range inside [0, n_atoms); offsets[0] = 0 and offsets[N] =
    // n_atoms are checked by the first and last group.  A violation gives NaN energies for the
    // group and GAP_EINVAL in the status word (when there is one).
    if (tid == 0)
        bad_s = 0;
    const int64_t my_lo = tid < ncfg ? a.offsets[cfg_lo + tid] : 0, my_hi = tid < ncfg ? a.offsets[cfg_lo + tid + 1] : 0;
    __syncthreads();
    if (my_lo < 0 || my_hi < my_lo || my_hi > a.n_atoms)
        bad_s = 1;
    if (tid == 0 && ((cfg_lo == 0 && g0 != 0) || (cfg_hi == a.N && g1 != a.n_atoms)))
        bad_s = 1;
    __syncthreads();
    double ysum = 0.0;
    bool out = tid < ncfg;
    if (bad_s != 0) {
        out = out && LAST;
        ysum = __builtin_nan("");
        if (LAST && tid == 0 && a.status)
            set_status(a.status, DST_EINVAL);
    } else {
        // a configuration starts in the range of its first atom (an empty one at the very end in the
        // last), and is carried on from one range to the next in y
        const int64_t a0 = base >= 0 ? a.a0 : 0;
        const bool begun = my_lo < a0;
        out = out && (begun ? my_hi > a0 : (LAST || my_lo < a.a1));
        if (out && begun)
            ysum = a.y[cfg_lo + tid];
        const int64_t lo = g0 > a0 ? g0 : a0, hi = g1 < a.a1 ? g1 : a.a1;
        for (int64_t cs = lo; cs < hi; cs += S::BM) {
            double e = 0.0;
            if (base >= 0) {
                const double *p = g_pred_pool + uniform(base + (cs - a0));
                const int t = cs + tid < hi ? tid : (int)(hi - cs) - 1;  // past the end: the last atom, unused
                for (int n = (int)a.n_runs; n > 0;) {
                    if (n <= 8) {
                        pred_add_runs<8>(a, p, n, t, e);
                        n -= 8;
                    } else if (n <= 16) {
                        pred_add_runs<16>(a, p, n, t, e);
                        n -= 16;
                    } else {
                        pred_add_runs<32>(a, p, n, t, e);
                        n -= 32;
                    }
                }
            } else if constexpr (LAST) {
                for (int64_t ct = 0; ct < a.n_ct; ct += PRED_G)
                    e += predict_tile_energy<S>(a, cs, ct, ct + PRED_G < a.n_ct ? ct + PRED_G : a.n_ct, lds, part);
            }
            __syncthreads();  // the previous atoms' sums have read eps
            eps[tid] = e;
            __syncthreads();
            const int64_t r0 = my_lo > cs ? my_lo : cs;
            int64_t r1 = my_hi < cs + S::BM ? my_hi : cs + S::BM;
            r1 = r1 < hi ? r1 : hi;
            if (tid < ncfg)
#pragma unroll 8
                for (int64_t r = r0; r < r1; ++r)
                    ysum += eps[r - cs];
        }
    }
    // the last workgroup to have read the energies (before the barriers above) frees them
    if (LAST && base >= 0 && (gridDim.x == 1 || arrive_last(&g_pred_done[base / PRED_CHUNK], gridDim.x, &last_s)) &&
        tid < a.chunks)
        __hip_atomic_store(&g_pred_owner[base / PRED_CHUNK + tid], 0ull, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
    if (out)
        a.y[cfg_lo + tid] = ysum;
}

hipError_t launch_predict(const double *X, int64_t n_atoms, const int64_t *offsets, int64_t N,
                          const double *XM, int64_t M, int d, int zeta, double sw2, const double *c,
                          double *y, int32_t *status, hipStream_t s)
{
    if (N <= 0)
        return hipSuccess;
    PredArgs a{};
    a.X = X;
    a.offsets = offsets;
    a.N = N;
    a.n_atoms = n_atoms;
    a.XM = XM;
    a.M = M;
    a.d = d;
    a.zeta = zeta;
    a.sw2 = sw2;
    a.c = c;
    a.y = y;
    a.status = status;
    static std::atomic<unsigned long long> calls{0};
    a.id = ++calls;
    a.C = n_atoms > 0 ? (224 * N) / n_atoms : N;
    a.C = a.C < 1 ? 1 : (a.C > 256 ? 256 : a.C);
    const int64_t groups = (N + a.C - 1) / a.C;
    a.n_ct = (M + KNM_BN - 1) / KNM_BN;
    auto tiles = [](int64_t n, int64_t b) { return (n + b - 1) / b; };
    // runs of one column tile where their energies fit what a call may claim, else whole groups
    constexpr int64_t ROOM = PRED_MAX * PRED_CHUNK;
    a.run = tiles(n_atoms, PSS::BM) * PSS::BM * a.n_ct <= ROOM ? 1 : PRED_G;
    a.n_runs = tiles(a.n_ct, a.run);
    // as many atoms at a time as the claim holds, in ranges of equal length
    const int64_t most = ROOM / a.n_runs / PSL::BM * PSL::BM;
    const int64_t n_ranges = n_atoms > 0 && most > 0 ? tiles(n_atoms, most) : 1;
    const int64_t range = tiles(tiles(n_atoms, n_ranges), PSL::BM) * PSL::BM;
    // The tile height whose whole rounds of workgroups take less: 512 places of 256 atoms, or 768 of 64,
    // 3.5 % slower per atom (9,009 runs of large tiles, 18 rounds: 1,829 us, 1,873 on small ones, 47 rounds;
    // 1,692, 4 rounds: 275 us, 254 in 9 rounds of small ones; 3,336, 7 rounds: 1,053 us, 1,016 in 18)
    auto rounds = [&](int64_t rows, int64_t places) { return tiles(tiles(range, rows) * a.n_runs, places); };
    const bool small = 1.035 * (double)(rounds(PSS::BM, 768) * 768 * PSS::BM) < (double)(rounds(PSL::BM, 512) * 512 * PSL::BM);
    const int64_t bm = small ? PSS::BM : PSL::BM;
    const int64_t ld = tiles(range < n_atoms ? range : n_atoms, bm) * bm;
    a.chunks = (int)tiles(ld * a.n_runs, PRED_CHUNK);
    if (n_atoms == 0 || most == 0)  // (then one range)
        a.run = a.chunks = 0;
    if (a.run > 0)
        hipLaunchKernelGGL(predict_claim_kernel, dim3(1), dim3(64), 0, s, a);
    for (int64_t r = 0; r < n_ranges; ++r) {
        a.a0 = r * range;
        a.a1 = a.a0 + range < n_atoms ? a.a0 + range : n_atoms;
        if (a.run > 0) {
            a.tiles = tiles(a.a1 - a.a0, bm);
            a.ld = a.tiles * bm;
            const unsigned grid = (unsigned)((a.tiles * a.n_runs + 7) & ~int64_t(7));
            if (small)
                hipLaunchKernelGGL(predict_tile_kernel<PSS>, dim3(grid), dim3(PSS::NT), 0, s, a);
            else
                hipLaunchKernelGGL(predict_tile_kernel<PSL>, dim3(grid), dim3(PSL::NT), 0, s, a);
        }
        if (r == n_ranges - 1)
            hipLaunchKernelGGL(predict_sum_kernel<true>, dim3((unsigned)groups), dim3(KNM_NT), 0, s, a);
        else
            hipLaunchKernelGGL(predict_sum_kernel<false>, dim3((unsigned)groups), dim3(KNM_NT), 0, s, a);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess && a.chunks > 0) {
        hipLaunchKernelGGL(predict_release_kernel, dim3(1), dim3(PRED_CHUNKS), 0, s, a.id);
        (void)hipGetLastError();
    }
    return e;
}

hipError_t launch_plan_tiles(const int64_t *offsets, int64_t N, int64_t n_atoms, int chunk, const KnmPlan &p,
                             int64_t max_tiles, int32_t *status, hipStream_t s)
{
    const int64_t nc = plan_chunks(N, chunk);
    hipLaunchKernelGGL(plan_chunk_kernel, dim3((unsigned)nc), dim3(256), 0, s, offsets, N, n_atoms, chunk, p.cfg_list,
                       p.lists, status);
    hipLaunchKernelGGL(plan_publish_kernel, dim3((unsigned)nc), dim3(256), 0, s, (const uint16_t *)p.lists,
                       nc, chunk, N, p.tile_start, p.n_tiles, max_tiles, status);
    return hipGetLastError();
}

static int bn_of(const KnmArgs &a) { return a.bn == 32 ? 32 : 64; }

hipError_t launch_knm_group(const KnmArgs *fits, const int64_t *max_tiles, int n, hipStream_t s)
{
    for (int bn : {64, 32}) {  // one grid per column-tile width
        KnmGroup g{};
        auto flush = [&]() {
            if (g.n > 0 && g.base[g.n] > 0) {
                if (bn == 64)
                    hipLaunchKernelGGL(knm_group_kernel<64>, dim3((unsigned)g.base[g.n]), dim3(KNM_NT), 0, s, g);
                else
                    hipLaunchKernelGGL(knm_group_kernel<32>, dim3((unsigned)g.base[g.n]), dim3(KNM_NT), 0, s, g);
            }
            g = KnmGroup{};
        };
        for (int i = 0; i < n; ++i) {
            if (bn_of(fits[i]) != bn)
                continue;
            KnmArgs a = fits[i];
            a.n_ct = (a.M + bn - 1) / bn;
            const int64_t total = max_tiles[i] * a.n_ct;
            a.total_pad = (total + 7) & ~int64_t(7);
            g.f[g.n] = a;
            g.base[g.n + 1] = g.base[g.n] + a.total_pad;
            if (++g.n == KNM_GROUP)
                flush();
        }
        flush();
    }
    return hipGetLastError();
}

// Columns per block of the two-step derivative rows with `room` doubles of scratch; 0: use the
// position tiles (too little room for 32 columns, or more gradient rows than positions).
int kdm_block_cols(int64_t n_grad, int64_t n_pos, int64_t M, int64_t room)
{
    if (n_grad > n_pos || n_grad > INT32_MAX)
        return 0;
    for (int w : {256, 128, 96, 64, 32})
        if (n_grad * w <= room && (w == 32 || w < 2 * M))
            return w;
    return 0;
}

hipError_t launch_kdm_blocks(const KnmArgs &a, int64_t n_obs, int64_t n_pos, int w, double *H, hipStream_t s)
{
    auto rows = [&](auto tile, int64_t col0) {
        using S = decltype(tile);
        const int64_t tiles = (a.n_grad + S::BM - 1) / S::BM * ((w + S::BN - 1) / S::BN);
        hipLaunchKernelGGL(grad_rows_kernel<S>, dim3((unsigned)((tiles + 7) & ~int64_t(7))), dim3(S::NT), 0, s, a, col0,
                           w, H);
    };
    for (int64_t col0 = 0; col0 < a.M; col0 += w) {
        if (w == 96)
            rows(GradTile<96>(), col0);
        else
            rows(GradTile<64>(), col0);
        hipLaunchKernelGGL(obs_sum_kernel, dim3((unsigned)((n_obs + 3) / 4), (unsigned)((w + 63) / 64)), dim3(256), 0, s,
                           a, n_obs, n_pos, col0, w, (const double *)H);
    }
    return hipGetLastError();
}

hipError_t launch_kdm(KnmArgs a, int64_t max_tiles, hipStream_t s)
{
    a.n_ct = (a.M + 63) / 64;
    a.total_pad = (max_tiles + 7) / 8 * 8 * a.n_ct;  // whole rounds of 8 tiles (see knm_body)
    if (a.total_pad == 0)
        return hipSuccess;
    hipLaunchKernelGGL(kdm_kernel, dim3((unsigned)a.total_pad), dim3(KNM_NT), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_knm(KnmArgs a, int64_t max_tiles, hipStream_t s)
{
    const int bn = bn_of(a);
    a.n_ct = (a.M + bn - 1) / bn;
    const int64_t total = max_tiles * a.n_ct;
    a.total_pad = (total + 7) & ~int64_t(7);
    if (a.total_pad == 0)
        return hipSuccess;
    const auto kernel = a.offsets ? (bn == 64 ? knm_kernel<64, CONFIGS> : knm_kernel<32, CONFIGS>)
                                  : (bn == 64 ? knm_kernel<64, POINTS> : knm_kernel<32, POINTS>);
    hipLaunchKernelGGL(kernel, dim3((unsigned)a.total_pad), dim3(KNM_NT), 0, s, a);
    return hipGetLastError();
}

}  // namespace gap
