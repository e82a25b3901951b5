// Growth of device buffers that a captured graph may address (host only; the
// allocator is a parameter, so that this is testable without a device).
#pragma once
#include <algorithm>
#include <cstddef>
#include <vector>

namespace rgx {

struct DevBuf {
  void *p = nullptr;
  size_t bytes = 0;
};

// Grows b to at least `need` bytes with alloc(bytes) (nullptr: it failed).  A
// captured graph may hold the old block's address: it moves to `retired`, to
// be freed with b's owner, and stays b's where the new block cannot be made.
// The block doubles up to `most` bytes, so the retired ones never hold more
// than twice the larger of `most` and the largest need.
template <class Alloc>
bool grow_kept(DevBuf &b, size_t need, size_t most, std::vector<void *> &retired, Alloc &&alloc) {
  if (b.p && b.bytes >= need) return true;
  retired.reserve(retired.size() + 1);   // (nothing to undo if this throws)
  size_t bytes = std::max(need, std::min(2 * b.bytes, most));
  void *p = alloc(bytes);
  if (!p && bytes > need) p = alloc(bytes = need);
  if (!p) return false;
  if (b.p) retired.push_back(b.p);
  b.p = p;
  b.bytes = bytes;
  return true;
}

// Makes b hold as many items of `item` bytes as it can, `want` at most, and
// returns how many it holds (0: not even one).  Where b should not grow (a
// stream capture) or cannot, those it holds already, if any.
template <class Alloc>
int grow_items(DevBuf &b, size_t item, int want, bool may_grow, size_t most,
               std::vector<void *> &retired, Alloc &&alloc) {
  const int held = b.p ? (int)std::min<size_t>(b.bytes / item, (size_t)want) : 0;
  if (held > 0 && !may_grow) return held;
  for (int n = want; n > held; n /= 2)
    if (grow_kept(b, (size_t)n * item, most, retired, alloc)) return n;
  return held;
}

}  // namespace rgx
