"""Tile shapes and tile-order words at the limits of accepted image sizes, and
the rule for lanes sharing a ray: the host-and-device header the library uses,
compiled here for the host."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2509_07782_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <initializer_list>
#include "tiles.hpp"
using namespace rgx;
#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)
int main() {
  // every shape of 64 rays keeps 64 / split of them
  for (int w = 1; w <= 64; w *= 2)
    for (int split = 1; split <= 4; split *= 2) {
      int tw = w, th = 64 / w;
      split_tile(split, tw, th);
      CHECK(tw >= 1 && th >= 1 && tw * th == 64 / split && (tw & (tw - 1)) == 0);
    }
  // every tile of the tallest and widest accepted images (65535 * 8 pixels a
  // side) is found again, or the image has no table
  const int sizes[] = {1, 8, 63, 65535, 65536, 65537, 131071, 131072, 131073, 140000, 200000,
                       262144, 262145, 524279, 524280};
  for (int w = 1; w <= 64; w *= 2)
    for (int split = 1; split <= 4; split *= 2) {
      int tw = w, th = 64 / w;
      split_tile(split, tw, th);
      for (int size : sizes) {
        const int64_t columns = (size + tw - 1) / tw, rows = (size + th - 1) / th;
        CHECK(tile_codes_hold(columns, 1) == (columns <= 65536));
        CHECK(tile_codes_hold(1, rows) == (rows <= 65536));
        for (int64_t x : {(int64_t)0, columns / 2, columns - 1}) {
          const uint32_t c = tile_code((uint32_t)x, 7);
          CHECK(!tile_codes_hold(columns, 1) || (tile_column(c) == x && tile_row(c) == 7));
        }
        for (int64_t y : {(int64_t)0, rows / 2, rows - 1}) {
          const uint32_t c = tile_code(5, (uint32_t)y);
          CHECK(!tile_codes_hold(1, rows) || (tile_column(c) == 5 && tile_row(c) == y && tile_row(c) * th < size));
        }
      }
    }
  return 0;
}
"""

LANES = r"""
#include <cstdio>
#include <initializer_list>
#include "tiles.hpp"
using namespace rgx;
#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)
int main() {
  // (CUs, Gaussians, 64-ray tiles): the fastest of 1, 2 and 4 lanes at the
  // measured sizes on both sides of every line
  for (bool back : {false, true}) {
    CHECK(choose_split(256, 1000, 512, back).outside == 4 && choose_split(256, 1000, 1024, back).outside == 2);
    CHECK(choose_split(256, 1000, 2048, back).outside == 1);
    for (int64_t n : {210000, 400000, 700000}) CHECK(choose_split(256, n, 3000, back).outside == 4);
    CHECK(choose_split(256, 700000, 4090, back).outside == 4);
    for (int64_t n : {210000, 400000})
      for (int64_t tiles : {3300, 4090}) CHECK(choose_split(256, n, tiles, back).outside == 2);
    CHECK(choose_split(256, 1000000, 3300, back).outside == 4 && choose_split(256, 1000000, 4096, back).outside == 4);
    CHECK(choose_split(256, 1000000, 8192, back).outside == 2);
    CHECK(choose_split(256, 1000000, 12288, back).outside == 1);
    for (int64_t n : {30000, 300000, 3000000}) CHECK(choose_split(256, n, 192, back).inside == 4);
    for (int64_t n : {30000, 100000}) CHECK(choose_split(256, n, 256, back).inside == 4);
    for (int64_t n : {200000, 300000, 1000000, 3000000})
      for (int64_t tiles : {208, 240, 256})
        CHECK(choose_split(256, n, tiles, back).inside == (back ? 2 : 4));
    CHECK(choose_split(256, 2500, 512, back).inside == 2 && choose_split(256, 300000, 512, back).inside == 1);
    CHECK(choose_split(256, 2500, 1024, back).inside == 1);
  }
  return 0;
}
"""


@pytest.mark.parametrize("program", [PROGRAM, LANES], ids=["tiles", "lanes"])
def test_tile_words_and_lane_rule(tmp_path, program):
    if shutil.which("g++") is None:
        pytest.skip("no host C++ compiler")
    src, exe = tmp_path / "tiles.cpp", tmp_path / "tiles"
    src.write_text(program)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(src), "-o", str(exe)],
                   check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
