// Tiles of a view: the shape a split leaves of a 64-ray tile, and how a
// tile's place in the view's grid is held (shared by host and device, without
// either's headers).
#pragma once
#include <cstdint>

namespace rgx {

// Tiles of 64 / split rays: the tile shape loses its longer side's half per
// factor of two.
inline void split_tile(int split, int &tile_w, int &tile_h) {
  for (int k = split; k > 1; k >>= 1) {
    if (tile_h >= tile_w) tile_h >>= 1;
    else tile_w >>= 1;
  }
}

// A tile's column and row in one word of a tile-order table, 16 bits each.  A
// view with more tiles than that on a side has no table and is marched row by
// row.  (Rows are unsigned: a sign bit would send rows past 32767 to pixels
// before the image.)
constexpr int kTileCodeMax = 1 << 16;
constexpr bool tile_codes_hold(int64_t columns, int64_t rows) {
  return columns <= kTileCodeMax && rows <= kTileCodeMax;
}
constexpr uint32_t tile_code(uint32_t column, uint32_t row) { return column | row << 16; }
constexpr int tile_column(uint32_t code) { return (int)(code & 0xffffu); }
constexpr int tile_row(uint32_t code) { return (int)(code >> 16); }

}  // namespace rgx
