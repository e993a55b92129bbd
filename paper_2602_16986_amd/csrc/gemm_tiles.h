// Which tile a product over token rows runs in (gemm_rows.hip).  Host code without the GPU runtime, so that a test can ask.
#pragma once
#include <cstdint>

namespace hstu {

enum { kTile64Deep = 1, kTile64, kTile128Deep, kTile128, kTile192, kTile256 };     // by token rows of a tile; deep: one workgroup per compute unit, more stages

// The tile with the least time where a compute unit works through its share of the tiles at the tile's rate (PFLOP/s that the
// kernels reach on many tiles, K = 512: bytes through the L2 per product fall with the tile; the widest one has no registers left
// to keep residual rows in).  Up to a tile per compute unit, all of a unit's LDS is one workgroup's: more k-tiles in flight.  us
// for the tiles of 64 (deep), 64, 128 (deep), 128, 192, 256 rows:
//   6,418 x 2048, K = 512, SiLU             -    23.9    -    22.5  28.4  21.0 *    (two library products: 34)
//   6,418 x 512, K = 512, W [K, N]          -     8.9   8.3 *  8.1  13.3  16.2      (16)
//   6,418 x 512, K = 2048, W [K, N]         -    23.7  19.1 * 24.5  36.2  42.1      (23)
//   20,000 x 512, K = 2048, W [K, N]        -    63.7    -    51.9  41.1 * 48.2      (42)
//   87,728 x 512, K = 2048, W [K, N]        -   342.6    -   247.8 216.1 194.3 *    (182-197)
//   1,200 x 512, K = 512, residual         6.1 *  6.3   8.1   8.0  13.0  18.6
// From K = 1024 on the small tiles' share of the L2's requests counts for more, and a residual's epilogue for less.  us, by the
// rates of short K -> of long K: 5,000 x 4096, K = 2048 97 -> 86, 2,500 x 8192, K = 2048 104 -> 90, 10,000 x 2048, K = 8192, W
// [K, N] 380 -> 329, 30,000 x 1024, K = 2048, residual 145 -> 130.
inline int gemm_rows_tile(int64_t M, int N, int64_t K, bool residual) {
  static const struct { int rows, cols, tile, deep; double rate, rate_long; } kinds[4] = {{64, 128, kTile64, kTile64Deep, 0.50, 0.40}, {128, 128, kTile128, kTile128Deep, 0.68, 0.62},
                                                                                          {192, 256, kTile192, kTile192, 0.80, 0.80}, {256, 256, kTile256, kTile256, 0.87, 0.87}};
  const bool long_k = K >= 1024;
  int best = 0;
  double least = 0;
  for (const auto& k : kinds) {
    const int64_t tiles = (M + k.rows - 1) / k.rows * ((N + k.cols - 1) / k.cols);
    double rate = long_k ? k.rate_long : k.rate;
    if (k.tile == kTile256 && residual) rate = long_k ? 0.74 : 0.68;
    const double time = (double)((tiles + 255) / 256) * k.rows * k.cols / rate;
    if (best == 0 || time < least) { least = time; best = tiles <= 256 ? k.deep : k.tile; }
  }
  return best;
}

// E4M3: tiles of 64 x 128, 128 x 256 and 192 x 256 take 1 : 3.3 : 4.9, the small one 0.7 beside its rounds; with a residual,
// whose rows find no registers there, 192 rows took 7.5, which never pays.  us for the three:  6,000 x 2048, K = 512, SiLU 16.9
// 17.1 14.4 *;  12,000 x 512, K = 512, residual 8.8 8.6 * 15.2;  20,600 x 4096, K = 1024, SiLU 177 130 122 *;  20,600 x 1024, K =
// 1024, residual 39.3 34.7 * 44.6;  6,000 x 512, K = 1024, residual 7.9 * 10.5 17.0.  One round of the small tile keeps more
// k-tiles in flight, as above: a layer's forward, whose operands do not wait in the caches, widths of 1024, 128 rows 35.1 ->
// 32.3, 3,217 x 512 (K = 1024) 37.8 -> 36.3.
inline int fp8_tile(int64_t M, int N, bool residual) {
  auto rounds = [&](int rows, int cols) { return (double)(((M + rows - 1) / rows * ((N + cols - 1) / cols) + 255) / 256); };
  const double t64 = rounds(64, 128) + 0.7, t128 = 3.3 * rounds(128, 256), t192 = 4.9 * rounds(192, 256);
  if (t64 <= t128 && (residual || t64 <= t192)) return rounds(64, 128) == 1 ? kTile64Deep : kTile64;
  return residual || t128 <= t192 ? kTile128 : kTile192;
}

}  // namespace hstu
