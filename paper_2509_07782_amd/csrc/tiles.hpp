// Tiles of a view: how many lanes share a ray, the shape that leaves of a
// 64-ray tile, and how a tile's place in the view's grid is held (shared by
// host and device, without either's headers).
#pragma once
#include <cstdint>

namespace rgx {

// Lanes per ray of the views whose camera is outside / inside the means' bounds.
struct Split {
  int outside = 1, inside = 1;
};

// How many lanes share a ray in a call of `tiles` 64-ray tiles over n
// Gaussians on a chip of `cu` CUs.  A 64-ray tile is one wave's serial march,
// and a few tiles at a scene's silhouette take many times the mean, so a launch
// too small to keep the chip busy beside them lasts as long as they do; tiles
// of 16 or 32 rays shorten every march, at 2.5 or 1.5 times the total work.  The
// lines lie where both sides were measured (ms forward, 1 / 2 / 4 lanes a
// ray): 100k Gaussians, cluster, 512 tiles 5.4 / 3.4 / 1.7, 1536 tiles 3.9 /
// 2.6 / 2.0, 2048 tiles 3.0 / 2.4 / 2.6, 4096 tiles 2.8 / 2.7 / 3.9, 6144 tiles
// 2.8 / 3.5 / 5.3; 1M, 8192 tiles 11.8 / 10.7 / 12.3, 12288 tiles 11.7 / 11.9 /
// 14.9; with the record and a backward, 2600 tiles, 210k 8.7 / 6.3 / 6.2, 1M 23.8
// / 17.2 / 14.8; 3000 tiles, 2 and 4 lanes, 210k 6.2 / 6.4, 400k 9.4 / 8.8, 700k
// 13.0 / 11.8; 3300 tiles, 210k 8.5 / 6.8 / 7.1, 400k 11.6 / 9.1 / 9.3 (a fixed step
// 11.1 / 8.8 / 10.0), 1M 24.1 / 18.0 / 17.1; 4090 tiles, 210k 7.8 / 6.4 / 7.6, 400k
// 11.9 / 9.2 / 11.0 (10.5 / 9.6 / 10.8), 700k 16.3 / 13.0 / 13.6 (17.2 / 14.4 /
// 14.0), 1M 25.0 / 17.4 / 16.9; 5k large ones, 512 tiles 2.3 / 1.4 /
// 1.3, 1024 tiles 1.9 / 1.8 / 2.3, 1536 tiles 1.8 / 2.2 / 3.0.  Where the
// camera stands inside a dense scene every ray starts in the medium and the
// tiles are alike, so those views have lines of their own (outdoor layout,
// forward + backward): 192 tiles, 30k 10.7 / 7.3 / 5.1, 300k 1.65 / 1.39 /
// 1.29, 3M 6.54 / 5.64 / 5.27; 256 tiles, 30k 11.2 / 8.0 / 6.0, 100k 1.78 / 1.58
// / 1.42, 200k 1.45 / 1.32 / 1.34, 300k 1.63 / 1.45 / 1.50, 1M 2.04 / 1.77 /
// 2.00, 3M 6.60 / 5.64 / 6.64; 512 tiles, 2.5k 4.9 / 3.8 / 4.2, 100k 1.65 / 1.59 /
// 1.79, 300k 1.45 / 1.52 / 1.69, 3M 5.2 / 5.9 / 6.8; 1024 tiles, 2.5k 4.6 / 4.8 /
// 6.2, 300k 1.7 / 1.9 / 2.6.  It is the backward that four lanes slow down there
// (3M, 208 tiles: 3.5 / 3.0 / 3.8, forward 3.04 / 2.66 / 2.39): a forward
// without a state, which none follows, takes them up to a tile a CU.
inline Split choose_split(int64_t cu, int64_t n, int64_t tiles, bool backward) {
  Split s;
  if (tiles <= 2 * cu || (tiles <= 12 * cu && n >= 50 * tiles) || (tiles <= 16 * cu && n >= 160 * tiles))
    s.outside = 4;
  else if (tiles <= 4 * cu || (tiles <= 32 * cu && n >= 24 * tiles)) s.outside = 2;
  if (tiles <= cu) s.inside = !backward || 4 * tiles <= 3 * cu || n <= 400 * tiles ? 4 : 2;
  else if (tiles <= 2 * cu && n <= 400 * tiles) s.inside = 2;
  return s;
}

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
