// Which tile a transform takes: host code with no HIP in it, so that it is also
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

}  // namespace
}  // namespace sq
