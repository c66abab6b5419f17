// How the groups of triangles share the raster's list.  For the device and for
// the host, where a test replays it.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace vs {

constexpr uint32_t kGroupNoRun = 0xffffffffu;
constexpr uint32_t kListWords = 0xe0000000u;   // most words of the list
constexpr int kParts = 8;                      // parts of the list, one for the groups of each XCD
constexpr int kPartApart = 8;                  // 64-bit words from one part's counter to the next one's

// Most tiles that the table of a group of 256 R triangles counts.  Record, table and total of a full group take
// four words per triangle then, what the workspace holds per triangle beside its entries; 1,024 triangles may have
// five words more, which the five words per bin beside them cover for up to kWideGroups such groups of a layer in a
// view (4 x 4,092 words beyond those of the layer's last group), so that a view of 1,024 x 1,024 pixels is counted in
// its bins of 16.
constexpr int kWideGroups = 3270;
__host__ __device__ constexpr int group_tiles(int R) { return R == 4 ? 4096 : 4 * 256 * R - 5; }

// Most entries of a side (front-facing or not) that a table's 16-bit sums count.  A group with more, hundreds
// of triangles over many tiles each, is counted in larger macro tiles: at last in four, four entries a triangle.
constexpr uint32_t kSideEntries = 0xffffu;

// Smallest shift, from s on, at which a rectangle of tiles has at most `most` macro tiles of 2^shift x 2^shift.
__host__ __device__ inline int macro_shift(int x0, int y0, int x1, int y1, int most, int s) {
  while (((x1 >> s) - (x0 >> s) + 1) * ((y1 >> s) - (y0 >> s) + 1) > most) ++s;
  return s;
}

// The list's parts: `words` each, and `entries` (triangles in tiles) that their runs may have.
struct ListRoom {
  uint32_t words, entries;
  int32_t parts;
};

// Room for a run of `need` words with `entries` entries: its first word in the list, or kGroupNoRun.  A
// part's counter holds the words taken from it and, << 32, their entries: load(p) reads it, add(p, n) adds n
// modulo 2^64 and returns what it held before.  The own part's counter is added to at once (one round trip to
// memory); another part's is looked at first, as it is only tried when the own one is full.  What found no
// room is taken off again, so that later and smaller runs find what is left and a counter never passes its
// part by more than one run for each block that is running (2,048 of at most 135 k words: below 2^32 - kListWords):
// it cannot wrap and hand out words that are taken.
template <class Load, class Add>
__host__ __device__ inline uint32_t reserve_run(uint32_t need, uint32_t entries, ListRoom room, uint32_t own, Load load, Add add) {
  if (need > room.words || entries > room.entries) return kGroupNoRun;
  const uint64_t mine = ((uint64_t)entries << 32) | need;
  const auto fits = [&](uint64_t taken) {
    return (uint32_t)taken <= room.words - need && (uint32_t)(taken >> 32) <= room.entries - entries;
  };
  for (uint32_t q = 0; q < (uint32_t)room.parts; ++q) {
    const uint32_t p = (own + q) % (uint32_t)room.parts;
    if (q > 0 && !fits(load(p))) continue;
    const uint64_t taken = add(p, mine);
    if (fits(taken)) return p * room.words + (uint32_t)taken;
    add(p, 0ull - mine);
  }
  return kGroupNoRun;
}

}  // namespace vs
