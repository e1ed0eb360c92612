// Tiles of a Hermitian 2^n x 2^n matrix stored row-major (index (r << n) | c): 32 x 32 elements, four
// per thread of a 256-thread workgroup.  Kernels that need one triangle run over the tiles (R, C)
// with R <= C.
#pragma once

#include "device_common.h"

namespace rsv {

constexpr int kTileSide = 32, kTileRows = 8, kTileElems = 4;  // thread: rows row0 + 8 q, one column

struct HermTile {
  uint32_t R, C;
  size_t base;  // of the tile's first element
};

// Tile number t in row-major order of the tiles (upper: of those with R <= C), nt tiles a side.
__device__ __forceinline__ HermTile herm_tile(uint32_t t, int n, bool upper) {
  const uint32_t nt = 1u << (n - 5);
  HermTile h;
  if (upper) {
    // row R starts at R nt - R (R - 1) / 2
    const double b = (double)nt + 0.5;
    int32_t R = (int32_t)(b - sqrt(b * b - 2.0 * (double)t));
    auto start = [&](int32_t r) { return (int64_t)r * nt - (int64_t)r * (r - 1) / 2; };
    while (R > 0 && start(R) > (int64_t)t) --R;
    while (start(R + 1) <= (int64_t)t) ++R;
    h.R = (uint32_t)R;
    h.C = h.R + (uint32_t)(t - start(R));
  } else {
    h.R = t >> (n - 5);
    h.C = t & (nt - 1);
  }
  h.base = ((size_t)h.R * kTileSide << n) + (size_t)h.C * kTileSide;
  return h;
}
inline uint32_t herm_tiles(int n, bool upper) {
  const uint32_t nt = 1u << (n - 5);
  return upper ? nt * (nt + 1) / 2 : nt * nt;
}

// How often element (row, col) of the tile counts in a sum over the whole matrix.
__device__ __forceinline__ double herm_weight(const HermTile& h, uint32_t row, uint32_t col) {
  if (h.R != h.C) return 2.0;
  return col > row ? 2.0 : col == row ? 1.0 : 0.0;
}

}  // namespace rsv
