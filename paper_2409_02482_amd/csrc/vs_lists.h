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

// The list's parts: `words` each.  A caller's capacity bounds the entries (triangles in tiles) of all runs, in one
// part; ~0: no bound.
struct ListRoom {
  uint32_t words, entries;
  int32_t parts;
};

// Room for a run of `need` words with `entries` entries: its first word in the list, or kGroupNoRun.  A
// part's counter holds the words asked of it: load(p) reads it, add(p, n) adds n and returns what it held
// before; count(n) does so with the entries.  Counters only grow, and in 64 bits: what found no room stays
// added (taken off again, it would be handed out twice, for what other groups got in the meantime lies above
// it), and no counter can wrap.  The own part's counter is added to at once.  A look before that costs as much
// again, as all groups' come to eight lines of memory (metric scene 365 -> 979 us); so a run that
// finds no room there also uses up what is left of that part, less than itself.  Another part's is looked at first, so
// that its room stays for runs that fit.
template <class Load, class Add, class Count>
__host__ __device__ inline uint32_t reserve_run(uint32_t need, uint32_t entries, ListRoom room, uint32_t own, Load load, Add add,
                                                Count count) {
  if (need > room.words) return kGroupNoRun;
  if (room.entries != ~0u && count(entries) + entries > (uint64_t)room.entries) return kGroupNoRun;
  for (uint32_t q = 0; q < (uint32_t)room.parts; ++q) {
    const uint32_t p = (own + q) % (uint32_t)room.parts;
    if (q > 0 && load(p) > room.words - need) continue;
    const uint64_t from = add(p, need);
    if (from <= room.words - need) return p * room.words + (uint32_t)from;
  }
  return kGroupNoRun;
}

}  // namespace vs
