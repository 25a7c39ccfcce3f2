// How the QR's products P = Y^T C are split: tiles, and chunks of the summed rows (host rule).
#pragma once

#include <stdint.h>

#include <algorithm>

namespace gap {

constexpr int QR_SMALL_TILE = 64;

struct QrSplit {
    bool small;         // 64 x 64 tiles
    int64_t nq, np;     // tiles across C's columns and Y's
    int64_t chunk, nch; // rows of a chunk, chunks
};

// pw columns of Y, nt of C, over `rows` rows; bm x bn the large tiles; at most cap chunks.
//
// The 64 x 64 tiles where either side is at most 64 wide, and where the large tiles would be
// fewer than one per CU even with chunks of 512 rows.
//
// Chunks, target <= 0, FP64: chunks of 1,024 rows, but at least 512 workgroups (two per CU) and at
// most 2,048. More chunks write and read more partial sums, fewer leave the last round of
// workgroups half empty (110,000 x 10,000, 512 workgroups: 45 ms more than 2,048).
// FP32: always about 2,048 workgroups, counted in 128 x 128 tiles. A chunk's rows are summed in FP32
// and the chunks in FP64, so longer chunks would cost accuracy (chunks of 1,024 rows at 18,250 x
// 2,250 took 9.26 ms for the QR against 9.45).
// A positive target: about that many workgroups.
//
// Chunks are multiples of 64 rows, the longer FP32 ones of 16 (a stage's rows). At least 64: 2,500
// x 500 in FP32 2 % of the fit, 7,100 x 1,111 0.5 % slower than 128.
inline QrSplit qr_split(int64_t rows, int64_t pw, int64_t nt, int64_t bm, int64_t bn, bool fp32, int64_t target,
                        int64_t cap)
{
    auto tiles = [](int64_t x, int64_t b) { return (x + b - 1) / b; };
    QrSplit q;
    q.small = pw <= 64 || nt <= 64 || tiles(nt, bn) * tiles(pw, bm) * tiles(rows, 512) < 256;
    q.nq = tiles(nt, q.small ? QR_SMALL_TILE : bn);
    q.np = tiles(pw, q.small ? QR_SMALL_TILE : bm);
    const int64_t n = fp32 ? tiles(nt, 128) * tiles(pw, 128) : q.nq * q.np;
    auto count = [&](int64_t wgs) { return tiles(wgs, n); };
    if (target > 0)
        q.nch = count(target);
    else if (fp32)
        q.nch = count(2048);
    else
        q.nch = std::max(count(512), std::min(count(2048), rows / 1024));
    q.nch = std::min(q.nch, cap);
    q.chunk = tiles(rows, q.nch);
    const int64_t unit = fp32 && q.chunk > 256 ? 16 : 64;
    q.chunk = tiles(q.chunk, unit) * unit;
    q.chunk = std::max(q.chunk, rows <= 4096 ? int64_t(64) : int64_t(128));
    q.nch = tiles(rows, q.chunk);
    return q;
}

}  // namespace gap
