// How many rows a workgroup of the fused calibration + quantisation kernel streams:
// host code with no HIP in it, so that it is also compiled and checked without a GPU
// compiler.
#pragma once

namespace sq {
namespace {

constexpr int kTqMaxRows = 64;               // rows per workgroup (their states live in LDS)

// About two workgroups per CU; one where a CU holds only one (g = 16 at K > 3584: nine
// waves of 124 registers), and at g = 16 and seven waves up to 768 rows, where reading
// the block rows (16 g K bits per workgroup) weighs most: 1024 x 4096 14.1 -> 11.0 us,
// 2000 x 4096 20.6 -> 17.3, 700 x 3584 10.6 -> 9.4 (900 x 3584 10.8 against 11.0, 2000 x
// 3584 15.4 against 16.4).  513 rows are 257 workgroups of two rows, the last with one,
// or 171 of three: 8.7 us against 9.2.
inline int tac_quant_rows(int M, int K, int g) {
    const int cw = (K / 8 + 63) / 64;                // waves that hold a row
    const int wgs = g == 16 && (cw == 8 || (cw == 7 && M <= 768 && M != 513)) ? 256 : 512;
    const int rows = (M + wgs - 1) / wgs;
    return rows < 1 ? 1 : rows > kTqMaxRows ? kTqMaxRows : rows;
}

}  // namespace
}  // namespace sq
