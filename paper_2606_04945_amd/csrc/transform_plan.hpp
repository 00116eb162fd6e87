// Which tile or kernel a transform takes: host code with no HIP in it, so that it is also
// compiled and checked without a GPU compiler.
#pragma once
#include <stddef.h>

namespace sq {
namespace {

// Tiles of the matrix-core transform (transform_fast.hip).  x2, x3, x4: four waves,
// without k groups, that many workgroups per CU; the others take most of a CU's LDS.
enum class FastTile { k32x32, k32x64, k64x64, k64x64x4, k64x64x3, k128x64, k128x128, k128x128x2, k256x128, k256x192 };

// A tile that fills most of a CU's LDS runs in rounds of 256 workgroups.
// Up to 128 x 128, the smallest tile that needs one round (waves of 64 x 64 where the
// tile holds them: 250 x 4096 25.4 us on 64 x 64 tiles of one such wave in four k
// groups, 29.9 with four waves of 32 x 32; 512 x 4096 37.9 on 128 x 64, 40.9 with
// waves of 64 x 32): 64 x 4096 15.0 us on 32 x 32 against 19.0 on 32 x 64, 128 x 4096
// 19.6 on 32 x 64 against 23.5 on 64 x 64, 64 x 12288 135 on 64 x 64 against 148 on
// 128 x 64, 128 x 12288 166 on 128 x 64 against 214 on 128 x 128.  Up to 32 rows 32 x
// 32 whatever the grid (reading Ps bounds it, and a taller tile is padding: 16 x 4096
// 14.4, 20.1 on 64 x 64; 32 x 18944 283, 322); at 64 rows its second round reads X
// and fills half the chip again (64 x 12288 163, 64 x 18944 384 against 298 on 128 x
// 128).
// Past one round, the least of rounds x time of a round, in the ratio 57 : 100 : 140
// of 128 x 128, 256 x 128 (eight waves of 64 x 64) and 256 x 192 (64 x 96): 1024 x
// 12288 570 us in 3 rounds, 650 in 2, 505 in 1; 4096 x 12288 2076 in 12, 1939 in 6,
// 1832 in 4; 4096 x 4096 254 in 4, 209 in 2, 270 in 2; 16384 x 3584 790, 684, 667.
// A shallow K (steps of 32) leaves a workgroup that has its CU to itself waiting for
// its first stages and its stores; several small ones cover for each other, and their
// one accumulator per output sums in plain k order.  Measured against the tile taken
// otherwise: up to 128 whatever the grid (192 up to 32 rows; 16 x 64 4.4 -> 3.4 us); one
// round of 64 x 64, K <= 1152: 1119 x 640 9.2 -> 7.7 (but 543 x 1024, whose rows lie a
// power of two apart, 10.8 -> 12.1); of 128 x 64, K < 1024: 1665 x 640 11.2 -> 9.7, from
// 340 tiles of 64 x 64 on K <= 896 with three per CU: 3213 x 512 11.1 -> 9.7; of
// 128 x 128: 4113 x 512 17.2 -> 12.0, 1585 x 1280 27.0 -> 20.4 (deeper the fewer tiles
// there are: 1450 x 3072 0.8 of the time), up to 1024 tiles at K = 512.  Past one round,
// where 128 x 128 tiles are the choice, up to K = 2048: two per CU (9344 x 896 47.9 ->
// 38.7, 9371 x 1216 79.7 -> 65.9).
inline FastTile fast_tile(int M, int K) {
    auto tiles = [&](int bm, int bn) { return (size_t)((M + bm - 1) / bm) * (size_t)((K + bn - 1) / bn); };
    auto rounds = [&](int bm, int bn) { return (tiles(bm, bn) + 255) / 256; };
    if (K <= 128 || (K <= 192 && M <= 32)) return FastTile::k64x64x4;
    if (M <= 32 || rounds(32, 32) == 1) return FastTile::k32x32;
    if (rounds(32, 64) == 1) return FastTile::k32x64;
    const size_t t = tiles(64, 64);
    if (t <= 256) return K <= 1152 && K != 1024 ? FastTile::k64x64x4 : FastTile::k64x64;
    if (rounds(128, 64) == 1) {
        if (t <= 340 && K < 1024) return FastTile::k64x64x4;
        return t > 340 && K <= 896 ? FastTile::k64x64x3 : FastTile::k128x64;
    }
    if (rounds(128, 128) == 1)
        return K <= (t <= 512 ? 3072 : t <= 768 ? 1536 : t <= 1024 ? 512 : 0) ? FastTile::k64x64x3 : FastTile::k128x128;
    const size_t t0 = 57 * rounds(128, 128), t1 = 100 * rounds(256, 128), t2 = 140 * rounds(256, 192);
    if (t0 <= t1 && t0 <= t2) return K <= 2048 ? FastTile::k128x128x2 : FastTile::k128x128;
    return t1 < t2 ? FastTile::k256x128 : FastTile::k256x192;
}

// Fixed-order transform with its chunks of 256 k split over the waves of a workgroup
// (transform_split.hip): blocks of 16 x 16 outputs per workgroup, and its waves.
struct SplitShape {
    int rb, cb, waves;
    long cost;
};
constexpr int kSplitChunk = 256;
constexpr long kCus = 256;

// Most waves a workgroup of RB x CB blocks holds: 16 waves leave 128 registers
// each, which the larger tiles exceed.
constexpr int split_waves(int blocks) { return blocks <= 4 ? 16 : 8; }

// Time of a tile shape, in 16 x 16 x 256 block chunks of the fp32 matrix cores
// per SIMD (64 MFMAs, 0.85 us at 2.4 GHz; measured 0.8-1.2 us each), the largest of
//  - the matrix cores: the busiest CU's workgroups, as many side by side as their
//    waves fit, times their rounds of chunks; twice that for 4 x 4 and 2 x 4 blocks with
//    up to four waves, whose registers leave a SIMD one or two (3612 x 512: 39.6 us on
//    4 x 4, the smaller shapes 22.7 - 30.3; 6877 x 256 with the quantiser behind it, so
//    that x comes from memory again: 31.2 on 2 x 4, 23.6 on 1 x 4, 26.3 tiled);
//  - P's bytes at 4.9 TB/s, more where fewer than 192 workgroups read them (16 x
//    8192: 57 us on 256 workgroups, 66 on 128; 16 x 12288: 127 us on 192);
//  - P read again by every row tile: 64-, 128- and 256-byte runs (CB = 1, 2, 4) came
//    back at 5.0, 6.9 and 11.5 TB/s (100 x 12288 in 7 row tiles: 849, 613, 367 us).
inline SplitShape split_cost(int rb, int cb, int M, int K) {
    const long nch = (K + kSplitChunk - 1) / kSplitChunk;
    const int cap = split_waves(rb * cb), W = (int)(nch < cap ? nch : cap);
    const long rows = (M + 16 * rb - 1) / (16 * rb);
    const long wgs = rows * (K / (16 * cb));
    const long n = (wgs + kCus - 1) / kCus, side = cap / W;
    const long passes = (n + side - 1) / side, at_once = n < side ? n : side;
    long cost = passes * ((at_once * W + 3) / 4) * ((nch + W - 1) / W) * rb * cb;
    if (rb * cb >= 8 && W <= 4) cost *= 2;
    const long p_read = (long)K * K;                 // x 1400000; divided last, small K count too
    const long mem = p_read * 192 / (1400000 * (wgs < 192 ? wgs : 192));
    const long again = p_read * rows * (cb == 1 ? 16 : cb == 2 ? 10 : 7) / (16 * 1400000);
    if (cost < mem) cost = mem;
    if (cost < again) cost = again;
    return {rb, cb, W, cost};
}

inline SplitShape split_shape(int M, int K) {
    // largest tile first: among equals it reads P and X least often
    constexpr int shapes[][2] = {{4, 4}, {2, 4}, {1, 4}, {1, 2}, {1, 1}};
    SplitShape best{0, 0, 0, 0};
    for (const auto& s : shapes) {
        if (K % (16 * s[1]) || (s[0] > 1 && M <= 8 * s[0])) continue;   // no row block of padding only
        const SplitShape c = split_cost(s[0], s[1], M, K);
        if (!best.rb || c.cost < best.cost) best = c;
    }
    return best;
}

// The tiled kernels take 64 x 128 tiles (32 blocks on four SIMDs: 8 per chunk)
// or, from 512 tiles on, 128 x 128.  One tile per CU costs them a fifth more per
// block than two.  Measured at K = 4096: 512 rows 145 us split, 169 tiled (equal
// costs, one tile per CU); 1024 rows 288 and 273 (equal, two); K = 4160: 256
// rows 118 and 171 (cost 144 against 136, one tile per CU); K = 12288: 256 rows
// 641 and 793, 512 rows 1271 and 1250 (equal, three); K = 1536: 4608 rows 222 and
// 210 (cost 182 against 192, four), so several tiles need a sixteenth less.  From
// five to eight chunks, which one round of the waves holds, three thirty-seconds
// less: 2705 x 1344 112.6 us split and 95.3 tiled, 4029 x 1280 152.8 and 139.5; up
// to three chunks the tiles' own ends cost as much: 3612 x 512 22.7 and 27.7.
// Up to 32 rows the split is always taken.
// With a state per row the tiled kernel groups the rows by it and skips the column
// tiles that lie wholly in a row's zeroed band, here taken as half of the rows on
// either side; the split kernel reads all of K.  384 x 12288 with two bands of 6016
// 785 us tiled and 979 split, 901 x 6784 with two of 3328 448 and 783, 1703 x 4032
// with one of 3870 203 and 509.  At up to two tiles per CU the gain goes into waiting
// for the fullest CU: those calls are judged without it (384 x 12288 with two bands
// of 384 fills three, of which 34 tiles in 576 are skipped: 978 split, 1242 tiled).
inline bool split_faster(int M, int K, int dm, int du, bool gated) {
    if ((size_t)M * K * 2 > 0x7fffffff) return false;   // X is addressed with 32-bit buffer offsets
    if (M <= 32) return true;
    const long cols = (K + 127) / 128;
    if ((long)((M + 127) / 128) * cols >= 512) return false;
    const long rows = (M + 63) / 64;
    long n = (rows * cols + kCus - 1) / kCus;
    if (gated && n > 2) {
        const long u0 = K - du, m0 = u0 - dm;
        const long skip_u = cols - (u0 + 127) / 128, skip_m = u0 / 128 - (m0 + 127) / 128;
        const long skip = (skip_u > 0 ? skip_u : 0) + (skip_m > 0 ? skip_m : 0);   // for half of the rows
        // half a tile per CU more, for the uneven rest
        const long left = (rows * (2 * cols - skip) + kCus + 2 * kCus - 1) / (2 * kCus);
        n = left < 2 ? 2 : left < n ? left : n;
    }
    const long nch = (K + kSplitChunk - 1) / kSplitChunk, tiled = n * 8 * nch;
    const long less = nch <= 3 ? 0 : nch >= 5 && nch <= 8 ? 3 : 2;
    return split_shape(M, K).cost < (n == 1 ? tiled + tiled / 8 + 1 : tiled - tiled * less / 32);
}

}  // namespace
}  // namespace sq
