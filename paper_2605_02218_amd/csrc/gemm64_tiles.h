// Which tiles a plain fp64 product is computed in (gemm64.hip); on the host only.
#pragma once

namespace covspec {

constexpr int kUnits = 256;      // compute units

enum Gemm64Tile { TILE_16x16, TILE_32x32, TILE_64x32, TILE_64x48, TILE_64x64, TILE_64x80, TILE_64x96 };

// M x N x K, `batch` of them; triangle: M = N, only the tiles on and below the diagonal; f64: both operands fp64, else bf16.
//
// 16 x 16 while a compute unit gets one.  us, the tiles below / 16 x 16, back to back: 144 (192 x 192 x 192) 5.5 / 4.6, 240 (192 x 320 x 320) 7.4 / 6.3, 256
// (128 x 256 x 256, batch 2) 6.8 / 5.7, 78 (192 x 192 x 1664, the triangle) 20.7 / 14.7; 312 (the same, batch 4) 22.0 / 25.9, 320 18.3 / 21.9, 480 (192 x
// 320 x 320, batch 2) 7.6 / 8.8.  With long k in between, us of covspec_select, triangles as below / on 16 x 16: 1638 rows, 156 tiles 1508 / 1467, 234 1769 /
// 1734, 252 (blocks of 128, batch 7) 2538 / 2519.
//
// Else the tile whose fullest compute unit has the least to do: rounds of tiles over the compute units, times the tile's area, times what a
// unit of area costs more or less in such tiles (operand reads per MFMA).  us, 64 x 96 / 80 / 64 / 48 / 32 and 32 x 32:
//   192 x 1664 x 1664, batch 4 83 / 72 / 109 / 83 / 86 and 83     192 x 1280 x 1280, batch 4 65 / 56 / 50 / 64 / 49 and 49
//   384 x 1152 x 1152, batch 8 162 / 140 / 151 / 144 / 139, 149   256 x 640 x 640, batch 64 218 / 213 / 218 / 235 / 229 and 247
//   320 x 1024 x 1024, batch 4 54 / 82 / 69 / 53 / 55 and 52      192 x 960 x 960, batch 7 51 / 44 / 67 / 50 / 53 and 49
//   384 x 1280 x 1280, batch 12 238 / 253 / 249 / 252 / 260, 269  128 x 512 x 512, batch 10 29 / 25 / 22 / 18 / 22 and 18
// (64 x 112, 64 x 128, 128 x 64, 128 x 96, 128 x 128 and a second group of waves on 64 x 80 or 64 x 64: never the best by more than 1 %.)
// Symmetric products and bf16 on 64 x 64 and 32 x 32 only: 192 x 192 x 1664, batch 4 59 and 24; 256 x 256 x 640, batch 64 88 and 77.
inline Gemm64Tile plain_tile(long M, long N, long K, long batch, bool triangle, bool f64) {
  const auto tiles = [&](int h, int w) {
    const long m = (M + h - 1) / h, n = (N + w - 1) / w;
    return (triangle ? m * (m + 1) / 2 : m * n) * batch;
  };
  if (f64 && tiles(16, 16) >= 1 && tiles(16, 16) <= kUnits && K % 64 == 0) return TILE_16x16;
  const auto fullest = [](long t) { return (double)((t + kUnits - 1) / kUnits); };
  double least = 1.18 * fullest(tiles(32, 32));
  Gemm64Tile tile = TILE_32x32;
  if (triangle) return 4.0 * fullest(tiles(64, 64)) <= least ? TILE_64x64 : tile;
  const auto consider = [&](Gemm64Tile t, int w, double per_area) {
    const double cost = w / 16 * per_area * fullest(tiles(64, w));
    if (cost < least) { least = cost; tile = t; }
  };
  consider(TILE_64x64, 64, 1.0);
  if (f64) {
    consider(TILE_64x96, 96, 0.99);
    consider(TILE_64x80, 80, 1.0);
    consider(TILE_64x48, 48, 1.02);
  }
  consider(TILE_64x32, 32, 1.06);
  return tile;
}

}  // namespace covspec
