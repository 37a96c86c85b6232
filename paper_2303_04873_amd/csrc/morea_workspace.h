// Device workspace kept by an object between calls (host code only).
#pragma once
#include <stddef.h>

#include <algorithm>

namespace morea {

struct Workspace {
  void* data = nullptr;
  size_t bytes = 0;
  bool refused = false;   // the last growth got less than it asked for
};

// Room for `fixed` bytes and `per_item` for each item of a slab: `largest`
// items a slab where memory allows, else `smallest`.  Returns the items a slab
// may have, 0 without memory for the smallest (the workspace is empty then).
// Growth frees first, so that the old and the new need not fit together.  After
// a refused growth, calls that the workspace has room for take the slab it
// holds: asking again on each would free, wait and fail each time.
// alloc(bytes) returns null on failure.
template <typename Alloc, typename Free>
size_t reserve_slab(Workspace& w, size_t fixed, size_t per_item, size_t smallest, size_t largest, Alloc alloc,
                    Free release) {
  smallest = std::min(smallest, largest);
  if (fixed + per_item * largest <= w.bytes) return largest;
  if (w.refused && fixed + per_item * smallest <= w.bytes)
    return std::max(smallest, (w.bytes - fixed) / per_item / smallest * smallest);
  if (w.data) release(w.data);
  w = Workspace{};
  for (const size_t n : {largest, smallest}) {
    const size_t bytes = fixed + per_item * n;
    w.data = alloc(bytes);
    if (w.data) {
      w.bytes = bytes;
      w.refused = n < largest;
      return n;
    }
    if (n == smallest) break;
  }
  return 0;
}

}  // namespace morea
