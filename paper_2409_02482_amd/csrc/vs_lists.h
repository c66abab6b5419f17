// How the groups of triangles share the raster's list.  For the device and for
// the host, where a test replays it.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace vs {

constexpr uint32_t kGroupNoRun = 0xffffffffu;
constexpr int kParts = 8;   // parts of a view's list, one for the groups of each XCD

// Room for a run of `need` words: its first word in the view's kParts parts of part_words each, or
// kGroupNoRun.  Part p's counter holds the words taken from it: load(p) reads it, add(p, n) adds n modulo
// 2^32 and returns what it held before.  The own part's counter is added to at once (one round trip to
// memory); another part's is looked at first, as it is only tried when the own one is full.  What found no
// room is taken off again, so that later and smaller runs find what is left and a counter never passes
// part_words by more than one run for each block that is running (2,048 of at most 332 k words, with parts
// of at most 2^29): it cannot wrap and hand out words that are taken.
template <class Load, class Add>
__host__ __device__ inline uint32_t reserve_run(uint32_t need, uint32_t part_words, uint32_t own, Load load, Add add) {
  if (need > part_words) return kGroupNoRun;
  for (uint32_t q = 0; q < (uint32_t)kParts; ++q) {
    const uint32_t p = (own + q) % kParts;
    if (q > 0 && load(p) > part_words - need) continue;
    const uint32_t from = add(p, need);
    if (from <= part_words - need) return p * part_words + from;
    add(p, 0u - need);
  }
  return kGroupNoRun;
}

}  // namespace vs
