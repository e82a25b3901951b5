"""Growth of the device buffers whose addresses a captured graph may hold: the
host-only header the library uses, compiled here with a counting allocator."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2509_07782_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include <set>
#include "buffers.hpp"
using namespace rgx;
#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)
int main() {
  std::set<void *> live;
  size_t room = 1000;                       // what the device still has
  int calls = 0;
  auto alloc = [&](size_t n) -> void * {
    calls++;
    if (n > room) return nullptr;
    room -= n;
    void *p = std::malloc(n);
    live.insert(p);
    return p;
  };
  DevBuf b;
  std::vector<void *> retired;
  // one view, then a capture holds its address, then three views
  CHECK(grow_items(b, 10, 1, true, 240, retired, alloc) == 1);
  void *captured = b.p;
  CHECK(grow_items(b, 10, 3, true, 240, retired, alloc) == 3);
  CHECK(b.p != captured && b.bytes >= 30);
  CHECK(live.count(captured) && retired.size() == 1 && retired[0] == captured);
  // a call of fewer views changes nothing; a capture never grows
  void *held = b.p;
  calls = 0;
  CHECK(grow_items(b, 10, 2, true, 240, retired, alloc) == 2 && b.p == held && calls == 0);
  CHECK(grow_items(b, 10, 24, false, 240, retired, alloc) == 3 && b.p == held && calls == 0);
  // out of memory: fewer at a time, and the held block stays where even
  // that is more than there is
  room = 130;
  CHECK(grow_items(b, 10, 24, true, 240, retired, alloc) == 12 && live.count(held));
  held = b.p;
  room = 0;
  CHECK(grow_items(b, 10, 24, true, 240, retired, alloc) == 12 && b.p == held && live.count(held));
  DevBuf none;
  CHECK(grow_items(none, 10, 24, true, 240, retired, alloc) == 0 && none.p == nullptr);
  // however a buffer grows, what is retired stays below twice the limit
  for (size_t item : {1, 7, 10}) {
    DevBuf g;
    std::vector<void *> old;
    std::vector<size_t> sizes;
    room = 1u << 20;
    auto sized = [&](size_t n) { sizes.push_back(n); return std::malloc(n); };
    const int most = 240 / (int)item;
    for (int n = 1; n <= most; n++) CHECK(grow_items(g, item, n, true, 240, old, sized) == n);
    size_t sum = 0;
    for (size_t i = 0; i + 1 < sizes.size(); i++) sum += sizes[i];
    CHECK(old.size() + 1 == sizes.size() && sum <= 2 * 240);
  }
  return 0;
}
"""


def test_outgrown_buffers_stay(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("no host C++ compiler")
    src, exe = tmp_path / "buffers.cpp", tmp_path / "buffers"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(src), "-o", str(exe)],
                   check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
