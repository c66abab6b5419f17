// Visibility kernels (steps 1-3): vertex projection and per-layer
// rasterisation into 64-bit (depth, triangle id) keys.
//
// Binned pipeline (one call of vs_raster_layers), three launches:
//   k_setup        snapped screen positions and w = 1/z for every (view, layer, vertex);
//                  view tables of the tiles; counters cleared
//   k_bin          per group of 256 to 1,024 consecutive triangles of a layer: set-up, cull,
//                  bounding boxes -> screen tiles of B x bin_rows(B) pixels; the group's
//                  triangle ids sorted by tile (front faces first), with a table of the
//                  tiles' starts, written as one run of the list
//   k_raster_bins  one block per bin = (view, tile, layer): finds the groups that reach its
//                  tile from their records; an LDS tile of keys starts EMPTY, the
//                  bin's triangles take 64-bit LDS minima, and the finished
//                  tile is stored once, coalesced (so no clear pass is needed);
//                  a fragment whose depth lower bound already loses to the
//                  tile's key skips the exact FP64 depth, and a back-facing
//                  triangle whose bound loses everywhere in its bounding box
//                  is skipped whole
#pragma once

#include <type_traits>

#include "vs_common.h"

namespace vs {

constexpr int kRasterThreads = 256;

// Bins are B pixels wide and bin_rows(B) high (a whole number of 8-row
// sub-tiles): 64-pixel bins are 56 rows high, so that a block's 64-bit key
// tile (28 KiB) and back-face queue leave room for five blocks per CU (a
// 64 x 64 tile alone, 32 KiB, fits only four).  Metric scene / k = 9 scene,
// raster phase: 56 rows 5.31 / 8.78 ms; 48 rows (still five blocks) 5.67 /
// 8.78 ms; 40 rows (six blocks) 5.63 / 8.47 ms.
__host__ __device__ constexpr int bin_rows(int B) { return B == 64 ? 56 : B; }
constexpr int kSmallSpan = 16384;   // small-triangle path: bbox extents <= 64 px, so edge values fit int32
// ... and at most this many candidate pixels in the tile.  A lane tests one candidate in about 50
// cycles and draws one in about 350; the wavefront path spends about 350 instructions on a triangle
// of a few 8 x 8 blocks.  Raster kernel at 256 / 512 / 1024 candidates: coarse shells (k = 7, 25,280
// triangles a layer, 16 views at 1000^2) 0.84 / 0.71 / 0.66 ms, a 256^2 view of 1,292-triangle shells
// 39 / 42 / 44 us, the metric scene 2.35 / 2.36 / 2.36 ms.
constexpr int kSmallArea = 512;
constexpr uint32_t kBigQueue = 16;   // larger back-facing triangles of a bin that its block queues, and
// groups whose entries it draws at once: 31.2 KiB of LDS with 56, so five blocks a CU, for bins of 64 pixels; smaller bins
// have LDS left, and in a mesh whose triangles come in no order many groups have an entry or two in each of them.
__host__ __device__ constexpr int bin_segs(int B) { return B == 64 ? 56 : 224; }
static_assert(kBigQueue <= (uint32_t)kRasterThreads && bin_segs(8) <= kRasterThreads, "one round deals the whole queue, or looks at all groups");

// Fill n u64 words with a value (grid-stride).
__global__ void __launch_bounds__(256) k_fill_u64(uint64_t* __restrict__ p, int64_t n, uint64_t val) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = val;
}

// The list is shared out in kParts equal parts, one for the groups of each XCD, in which runs are reserved by
// atomics on the parts' own counters: requests to one word are served one after the other (about 6 ns each;
// on a single word 168k groups would take 1 ms).  A run that its part has no room for goes to the next one
// that has: the views share the whole list, whatever their sizes.

// Everything that binning, drawing and shading find ready, one launch with the view in grid.y (views times
// vertices may pass what one grid dimension holds): a view's first proj_blocks blocks take step 1 for every
// (layer, vertex); the other blocks of all views, dealt round, take tile_view[g] = view owning
// 16-pixel tile g, and then bin_view[g] likewise for the bins' tiles (n_tiles_bin = 0: none).
struct SetupArgs {
  const vs_view* views;
  ProjVert* proj;
  int64_t vpv;
  int32_t* tile_view;
  int32_t* bin_view;
  int64_t n_tiles16, n_tiles_bin;
  unsigned long long* status;
  unsigned long long* parts;
  int32_t n_views, slot;
  uint32_t proj_blocks, tile_blocks;
};

__global__ void __launch_bounds__(256) k_setup(SetupArgs A, LayerTable L) {
  const int v = (int)blockIdx.y;
  if (blockIdx.x < A.proj_blocks) {
    const int64_t g = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (v == 0 && blockIdx.x == 0) {
      if (threadIdx.x < VS_STAT_COUNT) A.status[threadIdx.x] = 0ull;
      if (threadIdx.x < kParts) A.parts[threadIdx.x * kPartApart] = 0ull;
    }
    if (g >= A.vpv) return;
    int l = 0;
    while (l + 1 < L.k && L.vert_off[l + 1] <= g) ++l;
    A.proj[(int64_t)v * A.vpv + g] = project_vertex(L.xyz[l] + 3 * (g - L.vert_off[l]), A.views[v].cam);
    return;
  }
  const int64_t b = (int64_t)(blockIdx.x - A.proj_blocks) * gridDim.y + v;
  const bool bins = b >= A.tile_blocks;   // uniform
  const int64_t g = (bins ? b - A.tile_blocks : b) * 256 + threadIdx.x;
  if (bins) {
    if (g < A.n_tiles_bin) A.bin_view[g] = find_view_tile(A.views, A.n_views, g, A.slot);
  } else if (g < A.n_tiles16) {
    A.tile_view[g] = find_view_tile(A.views, A.n_views, g, 1);
  }
}

// Pixel-centre range covered by the triangle's fixed-point bounding box, clipped to the view.
struct PixRange { int i0, i1, j0, j1; };

__device__ inline PixRange pixel_range(const TriSetup& T, int W, int H) {
  const double mnx = fmin(T.X[0], fmin(T.X[1], T.X[2])), mxx = fmax(T.X[0], fmax(T.X[1], T.X[2]));
  const double mny = fmin(T.Y[0], fmin(T.Y[1], T.Y[2])), mxy = fmax(T.Y[0], fmax(T.Y[1], T.Y[2]));
  PixRange r;
  r.i0 = max((int)ceil((mnx - 128.0) * (1.0 / 256.0)), 0);
  r.i1 = min((int)floor((mxx - 128.0) * (1.0 / 256.0)), W - 1);
  r.j0 = max((int)ceil((mny - 128.0) * (1.0 / 256.0)), 0);
  r.j1 = min((int)floor((mxy - 128.0) * (1.0 / 256.0)), H - 1);
  return r;
}

__device__ inline int cull_slot(int r) {
  return r == kTriInvalid ? VS_STAT_CULLED_INVALID : r == kTriDegenerate ? VS_STAT_CULLED_DEGENERATE
                                                                        : VS_STAT_BAD_INDEX;
}

// A triangle's pixel bounding box clipped to the view, packed in 52 bits: i0 | i1 << 13 | j0 << 26 | j1 << 39.
__device__ inline uint64_t pack_box(int i0, int i1, int j0, int j1) {
  return (uint64_t)i0 | ((uint64_t)i1 << 13) | ((uint64_t)j0 << 26) | ((uint64_t)j1 << 39);
}

__device__ inline void unpack_box(uint64_t b, int& i0, int& i1, int& j0, int& j1) {
  i0 = (int)(b & 8191); i1 = (int)((b >> 13) & 8191); j0 = (int)((b >> 26) & 8191); j1 = (int)((b >> 39) & 8191);
}

// Groups of 256 R consecutive triangles of one layer, numbered over the layers of a view.
struct BinGroups {
  int32_t off[kMaxLayers + 1];
};

// Record of one group in one view.  Its tiles' rectangle is counted in macro tiles of
// 2^shift x 2^shift bins (shift 0 unless the rectangle has more of them than a table, or the group more
// entries than its sums).  The
// group's run of the list, from word `base`: per macro tile of the rectangle, row
// by row, how many front-facing entries and, << 16, how many others come before its own, then both
// totals in the same form; the front-facing entries (triangle ids); the others.
// "Front" marks a negative screen area before orientation normalisation, which is the front side of
// an outward, counter-clockwise wound closed mesh under this camera convention (y down).  Front
// faces are drawn first; an entry of another triangle says where it lies in the macro tile and how
// near it can be, so that the raster can skip one that cannot lower any key without loading its
// vertices:
//   index in the group | box << 10 | depth << 22,
// the box in units of unit_log(B, shift) pixels from the macro tile's corner (first column, first
// row, last column, last row, three bits each), the depth as (z - near) >> near_shift in 10 bits, z the
// high word of the triangle's depth_lower_key and near the group's smallest one, its low 19 bits
// cleared: no larger than z when taken apart, and as fine as a thousandth of the group's range.
struct alignas(16) GroupRec {
  uint16_t tx0, ty0, tw, th;   // tw = 0: reaches no bin
  uint32_t base;               // kGroupNoRun: no room in the list, its bins go through all of its triangles
  uint32_t form;               // shift | near_shift << 4 | near >> 19 << 9
};
constexpr uint32_t kSegAll = 0xf0000000u;   // a raster segment of all triangles from id base - kSegAll on; the list ends before it
static_assert(kListWords <= kSegAll, "words of the list and triangle ids of a segment are told apart");
__host__ __device__ constexpr int bin_log(int B) { return B == 64 ? 6 : B == 32 ? 5 : B == 16 ? 4 : 3; }
__host__ __device__ inline int unit_log(int B, int shift) { return max(3, bin_log(B) + shift - 3); }

// Triangles per thread of a group's block: larger groups cost a bin fewer runs to go through, smaller
// ones fill the chip.  One 1024^2 view of seven layers (696 groups of 1,024), binning and raster kernel
// with one, two or four: 15.8 + 87, 15.4 + 74, 16.3 + 75 us; with eight, the metric scene takes 414 + 2639
// us against 388 + 2660 with four, the k = 9 scene 1423 + 3261 against 1336 + 3452 (all with back faces of
// four words; now 14.6 + 76 us, 365 + 2540, 1285 + 3180).
// A view of more tiles than their table counts takes larger ones from 500 groups of 1,024 on: triangles that come in
// no order reach all tiles, and a table of macro tiles gives every bin the entries of its neighbours as well.
inline int bin_reps(int64_t n_tri, int n_views, int64_t tiles) {
  const int64_t groups = (n_tri + 1023) / 1024 * n_views;
  const int reps = groups >= 2048 ? 4 : groups >= 300 ? 2 : 1;
  return reps == 2 && groups >= 500 && tiles > group_tiles(2) ? 4 : reps;
}

// One block per group.  Its triangles' tiles are counted in LDS, so that only the group's one
// reservation of list space leaves the compute unit, and the counts' prefix sums give both the table
// and every entry's place.  It replaces a count with atomics per triangle, three scan launches and a
// scatter that read the records back: metric scene 1.49 -> 0.37 ms, k = 9 scene 3.61 -> 1.29 ms, one
// 1024^2 view 99 -> 15 us (the raster kernel, which now looks the runs up, 2.36 -> 2.54 ms, 2.87 -> 3.18 ms and
// 70 -> 76 us).  Bound by VALU issue: set-up in FP64, 1,294 instructions a wavefront, 0.98 of the cycles.
// One word an entry, front-facing or not, and one list for all views: 64 views at 800^2 of three shells of
// 1,292 triangles take 0.77 ms in all and every group has a run; records of four words and a list shared out to
// the views in equal parts left more than half of the groups without one (1.82 ms; 2.79 with lists per bin).
template <int B, int R>
__global__ void __launch_bounds__(256) k_bin(const vs_view* __restrict__ views, LayerTable L, BinGroups Q,
                                             const ProjVert* __restrict__ proj, int64_t vpv,
                                             GroupRec* __restrict__ recs, uint32_t* __restrict__ list, ListRoom room, int most,
                                             unsigned long long* __restrict__ parts,
                                             unsigned long long* __restrict__ status) {
  constexpr int BH = bin_rows(B);
  __shared__ uint32_t hist[group_tiles(R)];   // per macro tile: front entries, other entries << 16; then their next places
  __shared__ int32_t ext[4][6];
  __shared__ uint32_t sums[4][2];
  __shared__ uint32_t run_base;
  const int k = L.k, tid = threadIdx.x, wv = tid >> 6, lane = tid & 63;
  // XCD-contiguous remap: blocks are dealt round-robin to the 8 XCDs and gridDim.x is a multiple of 8,
  // so that triangles that share vertices share that XCD's L2
  const int grp = (int)((blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3));
  if (grp >= Q.off[k]) return;
  const int v = blockIdx.y;
  int l = 0;
  while (l + 1 < k && Q.off[l + 1] <= grp) ++l;
  const vs_view& V = views[v];
  const int W = V.cam.width, H = V.cam.height;
  const ProjVert* P = proj + (int64_t)v * vpv + L.vert_off[l];
  const int32_t* tri = L.tri[l];
  const int32_t n_vert = L.n_vert[l], n_tri = L.n_tri[l];
  const int32_t t0 = (grp - Q.off[l]) * (256 * R) + tid;
  GroupRec* rec = recs + (int64_t)v * Q.off[k] + grp;
  // ids of every repetition first (small); vertex records two at a time, the
  // next record's loads issued as soon as a record slot is free
  int3 ids[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    ids[r] = make_int3(0, 0, 0);
    if (t0 + 256 * r < n_tri) ids[r] = load_ids(tri, (uint32_t)(t0 + 256 * r));
  }
  auto fetch = [&](int r, TriLoad& q) {
    // defined on every lane: left undefined, the records stay live across the
    // divergent loads and cost about 16 more registers
    q.a = q.b = q.c = make_int4(0, 0, 0, 0);
    q.id[0] = q.id[1] = q.id[2] = 0;
    q.bad = false;
    if (t0 + 256 * r < n_tri) load_vertices(ids[r], n_vert, P, q);
  };
  TriLoad qa, qb;
  fetch(0, qa);
  if (R > 1) fetch(1, qb);
  uint64_t box[R];
  int32_t zlo[R];
  uint32_t live = 0, front = 0;
  int32_t ex0 = INT32_MAX, ey0 = INT32_MAX, ex1 = -1, ey1 = -1, near = INT32_MAX, far = 0;   // tiles, depth bounds
#pragma unroll
  for (int r = 0; r < R; ++r) {
    TriLoad& qr = (r & 1) ? qb : qa;
    box[r] = 0;
    zlo[r] = 0;
    const int32_t t = t0 + 256 * r;
    if (t < n_tri) {
      TriSetup T;
      const int st = setup_loaded(qr, T);
      if (st != kTriOk) {
        atomicAdd(status + cull_slot(st), 1ull);
      } else {
        const PixRange pr = pixel_range(T, W, H);
        if (pr.i0 <= pr.i1 && pr.j0 <= pr.j1) {
          const int tx0 = pr.i0 / B, tx1 = pr.i1 / B, ty0 = pr.j0 / BH, ty1 = pr.j1 / BH;
          box[r] = pack_box(pr.i0, pr.i1, pr.j0, pr.j1);
          ex0 = min(ex0, tx0); ey0 = min(ey0, ty0); ex1 = max(ex1, tx1); ey1 = max(ey1, ty1);
          live |= 1u << r;
          if (T.orig_sign < 0) {
            front |= 1u << r;
          } else {
            zlo[r] = (int32_t)(depth_lower_key(T, (uint32_t)t) >> 32);   // a positive float's bits: in order as integers
            near = min(near, zlo[r]); far = max(far, zlo[r]);
          }
        }
      }
    }
    if (r + 2 < R) fetch(r + 2, qr);   // this record slot is free now
  }
  // the group's rectangle of tiles, and the depth bounds of its triangles that are not front-facing
  ex0 = wave_min(ex0); ey0 = wave_min(ey0); ex1 = wave_max(ex1); ey1 = wave_max(ey1);
  near = wave_min(near); far = wave_max(far);
  if (lane == 0) {
    ext[wv][0] = ex0; ext[wv][1] = ey0; ext[wv][2] = ex1; ext[wv][3] = ey1; ext[wv][4] = near; ext[wv][5] = far;
  }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    ex0 = min(ex0, ext[w][0]); ey0 = min(ey0, ext[w][1]); ex1 = max(ex1, ext[w][2]); ey1 = max(ey1, ext[w][3]);
    near = min(near, ext[w][4]); far = max(far, ext[w][5]);
  }
  ex0 = __builtin_amdgcn_readfirstlane(ex0); ey0 = __builtin_amdgcn_readfirstlane(ey0);
  ex1 = __builtin_amdgcn_readfirstlane(ex1); ey1 = __builtin_amdgcn_readfirstlane(ey1);
  GroupRec out;
  out.tx0 = out.ty0 = out.tw = out.th = 0;
  out.base = kGroupNoRun;
  out.form = 0;
  if (ex1 < ex0) {   // uniform
    if (tid == 0) *rec = out;
    return;
  }
  int s = macro_shift(ex0, ey0, ex1, ey1, most, 0), rx, ry, tw, th, n, e0, e1;
  // each (triangle, macro tile): use(repetition, tile's column and row, its histogram word, front-facing)
  auto each = [&](auto use) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if (!((live >> r) & 1u)) continue;
      int i0, i1, j0, j1;
      unpack_box(box[r], i0, i1, j0, j1);
      const int x0 = (i0 / B) >> s, y0 = (j0 / BH) >> s, x1 = (i1 / B) >> s, y1 = (j1 / BH) >> s;
      const bool f = (front >> r) & 1u;
      for (int y = y0; y <= y1; ++y)
        for (int x = x0; x <= x1; ++x) use(r, x, y, &hist[(y - ry) * tw + (x - rx)], f);
    }
  };
  uint32_t f, o, total_f, total_o;
  for (;; s = macro_shift(ex0, ey0, ex1, ey1, most, s + 1)) {   // uniform; once unless a side has too many entries
    rx = ex0 >> s; ry = ey0 >> s; tw = (ex1 >> s) - rx + 1; th = (ey1 >> s) - ry + 1; n = tw * th;
    for (int e = tid; e < n; e += 256) hist[e] = 0;
    __syncthreads();
    each([&](int, int, int, uint32_t* h, bool is_front) { atomicAdd(h, is_front ? 1u : 0x10000u); });
    __syncthreads();
    // exclusive prefix sums over the tiles, `per` consecutive ones per thread
    const int per = (n + 255) / 256;
    e0 = min(tid * per, n); e1 = min(e0 + per, n);
    uint32_t mine_f = 0, mine_o = 0;
    for (int e = e0; e < e1; ++e) {
      mine_f += hist[e] & 0xffffu;
      mine_o += hist[e] >> 16;
    }
    f = mine_f; o = mine_o;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const uint32_t fb = __shfl_up(f, off), ob = __shfl_up(o, off);
      if (lane >= off) {
        f += fb;
        o += ob;
      }
    }
    if (lane == 63) {
      sums[wv][0] = f;
      sums[wv][1] = o;
    }
    __syncthreads();
    f -= mine_f;
    o -= mine_o;
    total_f = total_o = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      f += w < wv ? sums[w][0] : 0u;
      o += w < wv ? sums[w][1] : 0u;
      total_f += sums[w][0];
      total_o += sums[w][1];
    }
    if (max(total_f, total_o) <= kSideEntries) break;
    __syncthreads();   // the counts and sums are written anew
  }
  const uint32_t entries = total_f + total_o, need = (uint32_t)n + 1u + entries;   // words
  near = __builtin_amdgcn_readfirstlane(total_o ? near & ~0x7ffff : 0);
  far = __builtin_amdgcn_readfirstlane(total_o ? far : 0);
  const int near_shift = max(0, 22 - __clz(far - near));   // the range in 10 bits
  if (tid == 0) {
    const uint32_t base = reserve_run(
        need, entries, room, blockIdx.x,
        [&](uint32_t p) { return __hip_atomic_load(parts + p * kPartApart, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); },
        [&](uint32_t p, uint64_t words) { return atomicAdd(parts + p * kPartApart, (unsigned long long)words); },
        [&](uint64_t more) { return atomicAdd(parts + kPartApart, (unsigned long long)more); });   // one part then: the second counter
    run_base = base;
    out.tx0 = (uint16_t)rx; out.ty0 = (uint16_t)ry; out.tw = (uint16_t)tw; out.th = (uint16_t)th;
    out.base = base;
    out.form = (uint32_t)s | (uint32_t)near_shift << 4 | (uint32_t)near >> 19 << 9;
    *rec = out;
  }
  __syncthreads();
  const uint32_t base = run_base;
  if (base == kGroupNoRun) return;   // uniform
  for (int e = e0; e < e1; ++e) {
    const uint32_t c = hist[e], places = f | (o << 16);
    list[base + e] = places;
    hist[e] = places;
    f += c & 0xffffu;
    o += c >> 16;
  }
  if (tid == 0) list[base + n] = total_f | (total_o << 16);
  __syncthreads();
  uint32_t* fronts = list + base + n + 1;
  uint32_t* rest = fronts + total_f;
  const int ul = unit_log(B, s);
  each([&](int r, int x, int y, uint32_t* h, bool is_front) {
    const uint32_t old = atomicAdd(h, is_front ? 1u : 0x10000u);
    if (is_front) {
      fronts[old & 0xffffu] = (uint32_t)(t0 + 256 * r);
    } else {
      int i0, i1, j0, j1;
      unpack_box(box[r], i0, i1, j0, j1);
      const int ax = x * (B << s), ay = y * (BH << s);
      const uint32_t c0 = (uint32_t)(max(i0 - ax, 0) >> ul), c1 = (uint32_t)(min(i1 - ax, (B << s) - 1) >> ul);
      const uint32_t r0 = (uint32_t)(max(j0 - ay, 0) >> ul), r1 = (uint32_t)(min(j1 - ay, (BH << s) - 1) >> ul);
      rest[old >> 16] = (uint32_t)(256 * r + tid) | c0 << 10 | r0 << 13 | c1 << 16 | r1 << 19 |
                        (uint32_t)(zlo[r] - near) >> near_shift << 22;
    }
  });
}

__device__ inline int4 readlane4(int4 v, int lane) {
  return make_int4(__builtin_amdgcn_readlane(v.x, lane), __builtin_amdgcn_readlane(v.y, lane),
                   __builtin_amdgcn_readlane(v.z, lane), __builtin_amdgcn_readlane(v.w, lane));
}

// One block per bin.  Small triangles (bounding box <= 64 px on each side and
// few candidate pixels) are walked with exact int32 edge values by one lane, or
// by 2 to 16 lanes that take their rows in turn where the chunk of (at most
// 256) triangles being drawn is smaller than the block: the walk is a serial
// chain of LDS reads, FP64 depths and LDS minima, so idle lanes beside it are
// time lost, while a repeated set-up costs little.  Larger triangles are queued
// for the whole block, dealt round its wavefronts after the chunks, and drawn
// one 8 x 8 pixel block of the tile at a time with exact FP64 edge values.
// Wavefronts work independently on the LDS tile (64-bit atomic minimum).
// Against one lane per triangle and larger ones tested over the whole tile by
// the wavefront that met them: metric scene 3.11 -> 2.36 ms, k = 9 scene 2.95 ->
// 2.87 ms (before the bins' lists became runs of groups), a single 1024^2 view 92 -> 70 us, coarse shells (k = 7, 25,280
// triangles a layer, 16 views at 1000^2) 3.50 -> 0.71 ms, a 256^2 view of
// 1,292-triangle shells 234 -> 42 us.  Sharing only chunks of at most 64 or 32
// triangles: metric 2.75 and 3.07 ms; two or four lanes per triangle in full
// chunks too: metric 2.39 and 2.58 ms, k = 9 scene 3.26 and 4.19 ms.
//
// The bin's list holds its front-facing triangles first.  They are drawn
// first; then the tile's largest key per 8 x 8 sub-tile is taken, and a
// back-facing triangle whose depth lower bound (a key no larger than any key it
// can produce) is at least every sub-tile maximum under its bounding box is
// skipped: every pixel it could reach already holds a key no larger than any
// of its own, so the minimum cannot change (keys only decrease).  On a closed
// shell seen from outside, the back faces lie behind the front faces covering
// the same pixels, so most of them are skipped without a pixel walk.  An empty
// pixel keeps its sub-tile maximum at EMPTY, so nothing is skipped there.  With
// fragment counting on, nothing is skipped (the count covers every covered
// pixel of every triangle).
template <int B>
__global__ void __launch_bounds__(kRasterThreads, 5) k_raster_bins(
    const vs_view* __restrict__ views, const int32_t* __restrict__ bin_view, int64_t n_tiles, LayerTable L, BinGroups Q,
    int group_log, const ProjVert* __restrict__ proj, int64_t vpv, int slot, const GroupRec* __restrict__ recs,
    const uint32_t* __restrict__ list, unsigned long long* __restrict__ vis,
    unsigned long long* __restrict__ status, int count_frags) {
  constexpr int BH = bin_rows(B);              // bin rows
  constexpr int kSub = 8;                      // sub-tile edge of the depth bound
  constexpr int kNs = B / kSub;                // sub-tiles per row
  constexpr int kNsY = BH / kSub;              // sub-tile rows
  constexpr int kSegs = bin_segs(B);
  // entries before a group, front-facing ones and others << kHalf; a group has at most 1,024 in a tile
  using Start = std::conditional_t<kSegs <= 63, uint32_t, uint64_t>;
  constexpr int kHalf = 4 * sizeof(Start);
  constexpr Start kLow = ((Start)1 << kHalf) - 1;
  static_assert(B % kSub == 0 && BH % kSub == 0, "bins must be whole sub-tiles");
  __shared__ __align__(16) unsigned long long tile[B * BH];
  __shared__ uint32_t smax[kNs * kNsY];   // per sub-tile, the depth word of its largest key
  __shared__ int32_t queue[2 * kRasterThreads];   // back-facing triangles that may lower a key
  __shared__ int32_t late_bigs[kBigQueue];        // large triangles among those (large front-facing ones: in the queue)
  __shared__ uint32_t qadd[3], bign;              // entries queued by a chunk, for three chunks in turn
  __shared__ uint32_t seg_base[kSegs];            // groups that reach the tile: list word of their first front-facing entry here
  __shared__ uint32_t seg_rest[kSegs];            // ... from there to their first other entry | shift << 18 | near_shift << 22
  __shared__ uint32_t seg_group[kSegs];           // ... the group's number in the layer << 12 | near >> 19
  __shared__ Start seg_start[kSegs];              // ... and the entries before it
  __shared__ uint32_t seg_n[3];                   // groups, front-facing entries, other entries
  __shared__ int32_t seg_next;                    // first group that found no place
  __shared__ uint32_t wave_n[2][kRasterThreads / 64];   // groups found by each wavefront, for two batches in turn
  __shared__ uint32_t no_run;                     // a group without a run reaches this tile
  const int k = L.k;
  const int64_t n_bins = n_tiles * k;
  // XCD-contiguous remap of the block index
  const int64_t chunk = (n_bins + 7) / 8;
  const int64_t bid = ((int64_t)blockIdx.x % 8) * chunk + (int64_t)blockIdx.x / 8;
  if (bid >= n_bins) return;
  const int64_t g = bid / k;
  const int l = (int)(bid - g * k);
  const int v = bin_view[g];
  const vs_view& V = views[v];
  const int W = V.cam.width, H = V.cam.height;
  const int ntx = (W + B - 1) / B;
  const int64_t tl = g - V.tile_offset[slot];
  const int ty = (int)(tl / ntx), tx = (int)(tl - (int64_t)ty * ntx);
  const int x0 = tx * B, y0 = ty * BH;
  const int x1 = min(x0 + B, W) - 1, y1 = min(y0 + BH, H) - 1;
  const int tid = threadIdx.x, lane = tid & 63;
  if (tid == 0) qadd[0] = qadd[1] = qadd[2] = bign = no_run = 0;
  for (int p = tid; p < B * BH / 2; p += kRasterThreads)   // 16-byte stores
    reinterpret_cast<ulonglong2*>(tile)[p] = make_ulonglong2(kEmpty, kEmpty);
  const ProjVert* P = proj + (int64_t)v * vpv + L.vert_off[l];
  const int32_t* tri = L.tri[l];
  const int32_t nvert = L.n_vert[l];
  const GroupRec* grec = recs + (int64_t)v * Q.off[k] + Q.off[l];
  const int n_groups = Q.off[l + 1] - Q.off[l], n_tri = L.n_tri[l];
  unsigned long long frags = 0;
  // Loads the groups from g0 on that reach this tile, as many as kSegs holds, and returns the group to go
  // on from.  All triangles of a group without a run are taken for front-facing: nothing is skipped then.
  // Called by the whole block.
  auto load_segs = [&](int g0) -> int {
    int have = 0, turn = 0;
    bool full = false;
    int me = tid;
    asm volatile("" : "+v"(me));   // nothing derived from it is held in registers across the drawing
    const int tid = me, lane = me & 63;
    while (g0 < n_groups && !full) {   // uniform: 256 groups at a time
      uint32_t base = 0, rest = 0, near = 0, nf = 0, nb = 0;
      if (g0 + tid < n_groups) {
        const uint4 raw = *reinterpret_cast<const uint4*>(grec + g0 + tid);
        const int s = (int)(raw.w & 15u);
        const int mx = (tx >> s) - (int)(raw.x & 0xffffu), my = (ty >> s) - (int)(raw.x >> 16);
        const int tw = (int)(raw.y & 0xffffu), th = (int)(raw.y >> 16);
        if (mx >= 0 && mx < tw && my >= 0 && my < th) {
          if (raw.z == kGroupNoRun) {
            base = kSegAll + ((uint32_t)(g0 + tid) << group_log);
            nf = (uint32_t)min(1 << group_log, n_tri - ((g0 + tid) << group_log));
          } else {
            const uint32_t* starts = list + raw.z + my * tw + mx;
            const uint32_t at = starts[0], next = starts[1];
            const uint32_t ids = raw.z + (uint32_t)(tw * th) + 1u, total_f = list[ids - 1u] & 0xffffu;
            base = ids + (at & 0xffffu);
            nf = (next & 0xffffu) - (at & 0xffffu);
            rest = (total_f - (at & 0xffffu) + (at >> 16)) | (raw.w & 15u) << 18 | (raw.w >> 4 & 31u) << 22;
            near = raw.w >> 9;
            nb = (next >> 16) - (at >> 16);
          }
        }
      }
      const bool hit = nf + nb > 0;
      const uint64_t hits = __ballot(hit);
      if (lane == 0) wave_n[turn][tid >> 6] = (uint32_t)__popcll(hits);
      __syncthreads();
      int at = have + (int)__popcll(hits & __lanemask_lt());
#pragma unroll
      for (int w = 0; w < kRasterThreads / 64; ++w) {
        const int n = __builtin_amdgcn_readfirstlane((int)wave_n[turn][w]);
        at += w < (tid >> 6) ? n : 0;
        have += n;
      }
      if (hit && at < kSegs) {
        seg_base[at] = base;
        seg_rest[at] = rest;
        seg_group[at] = (uint32_t)(g0 + tid) << 12 | near;
        seg_start[at] = (Start)nf | ((Start)nb << kHalf);
      }
      if (hit && at == kSegs) seg_next = g0 + tid;
      full = have > kSegs;
      g0 += kRasterThreads;
      turn ^= 1;
    }
    have = min(have, kSegs);
    __syncthreads();
    if (full) g0 = __builtin_amdgcn_readfirstlane(seg_next);
    if (tid < 64) {   // one wavefront sums the entries up
      uint32_t sum_f = 0, sum_o = 0;
#pragma unroll 1
      for (int c0 = 0; c0 < (kSegs <= 64 ? 1 : have); c0 += 64) {   // uniform
        const int e = c0 + lane;
        const Start c = e < have ? seg_start[e] : 0;
        const uint32_t nf = (uint32_t)(c & kLow), nb = (uint32_t)(c >> kHalf);
        uint32_t f = nf, o = nb;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
          const uint32_t fb = __shfl_up(f, off), ob = __shfl_up(o, off);
          if (lane >= off) {
            f += fb;
            o += ob;
          }
        }
        if (e < have) seg_start[e] = (Start)(sum_f + f - nf) | ((Start)(sum_o + o - nb) << kHalf);
        sum_f += __builtin_amdgcn_readlane(f, 63);
        sum_o += __builtin_amdgcn_readlane(o, 63);
      }
      if (lane == 0) {
        seg_n[0] = (uint32_t)have;
        seg_n[1] = sum_f;
        seg_n[2] = sum_o;
      }
    }
    __syncthreads();
    return g0;
  };
  // The loaded group that holds front-facing (shift 0) or other (shift kHalf) entry c: the last one that
  // starts at or before c (one without such entries starts where the next does).
  auto find_seg = [&](uint32_t c, int shift) {
    uint32_t a = 0, b = seg_n[0] - 1;
    while (a < b) {
      const uint32_t mid = (a + b + 1) / 2;
      if ((uint32_t)((seg_start[mid] >> shift) & kLow) <= c) a = mid; else b = mid - 1;
    }
    return a;
  };
  auto front_entry = [&](uint32_t c) -> int32_t {
    const uint32_t a = find_seg(c, 0), at = seg_base[a] + c - (uint32_t)(seg_start[a] & kLow);
    return at >= kSegAll ? (int32_t)(at - kSegAll) : (int32_t)list[at];
  };
  // Other entry c of the loaded groups: its triangle; the columns and rows of 8 x 8 sub-tiles of this bin that its box
  // may reach, none if first > last; and a bound that no depth word of its keys is below.
  struct Other {
    int32_t t, c0, c1, r0, r1;
    uint32_t z;
  };
  auto other_entry = [&](uint32_t c) -> Other {
    const uint32_t a = find_seg(c, kHalf), rest = seg_rest[a], group = seg_group[a];
    const uint32_t e = list[seg_base[a] + (rest & 0x3ffffu) + c - (uint32_t)(seg_start[a] >> kHalf)];
    const int s = (int)(rest >> 18 & 15u), ul = unit_log(B, s), in = (1 << s) - 1;
    const int dx = (tx & in) * B, dy = (ty & in) * BH;   // this bin's corner in the macro tile
    Other o;
    o.t = (int32_t)((group >> 12 << group_log) + (e & 1023u));
    o.c0 = max(((int)(e >> 10 & 7u) << ul) - dx, 0) >> 3;
    o.r0 = max(((int)(e >> 13 & 7u) << ul) - dy, 0) >> 3;
    o.c1 = min((((int)(e >> 16 & 7u) + 1) << ul) - 1 - dx, B - 1) >> 3;
    o.r1 = min((((int)(e >> 19 & 7u) + 1) << ul) - 1 - dy, BH - 1) >> 3;
    o.z = ((group & 0xfffu) << 19) + (e >> 22 << (rest >> 22));
    return o;
  };
  __syncthreads();
  // Triangles drawn by the whole wavefront, one after the other: every lane's triangle (big < 0:
  // none) is loaded at once, so that the wavefront waits for memory once, and handed round.  For
  // each, the lanes first test one 8 x 8 pixel block each (an edge function is linear, so its
  // largest value over a block sits at a corner), then the wavefront visits the surviving blocks,
  // one pixel a lane.
  auto draw_bigs = [&](int32_t big) {
    TriLoad q;
    q.a = q.b = q.c = make_int4(0, 0, 0, 0);
    if (big >= 0) load_vertices<true>(load_ids(tri, (uint32_t)big), nvert, P, q);
    for (uint64_t bm = __ballot(big >= 0); bm; bm &= bm - 1) {
      const int from = (int)__builtin_ctzll(bm);
      const int32_t t = __builtin_amdgcn_readlane(big, from);
      TriLoad u;
      u.a = readlane4(q.a, from); u.b = readlane4(q.b, from); u.c = readlane4(q.c, from);
      u.id[0] = u.id[1] = u.id[2] = 0;
      u.bad = false;
      TriSetup T;
      setup_loaded(u, T);   // a valid triangle: its first setup said so
      const unsigned long long lbkey = depth_lower_key(T, (uint32_t)t);
      const PixRange pr = pixel_range(T, W, H);
      const int lx = lane & 7, ly = lane >> 3;
      double E[3], ax[3], ay[3];   // edge values at this lane's pixel of the bin's first block; steps per pixel
      edge_values(T, 256.0 * (x0 + lx) + 128.0, 256.0 * (y0 + ly) + 128.0, E);
      ax[0] = (T.Y[1] - T.Y[2]) * 256.0; ay[0] = (T.X[2] - T.X[1]) * 256.0;
      ax[1] = (T.Y[2] - T.Y[0]) * 256.0; ay[1] = (T.X[0] - T.X[2]) * 256.0;
      ax[2] = (T.Y[0] - T.Y[1]) * 256.0; ay[2] = (T.X[1] - T.X[0]) * 256.0;
      // this lane's block (lx, ly): its first pixel is 7 lx right of and 7 ly below this lane's own pixel
      bool may = x0 + 8 * lx <= min(pr.i1, x1) && x0 + 8 * lx + 7 >= pr.i0 && y0 + 8 * ly <= min(pr.j1, y1) &&
                 y0 + 8 * ly + 7 >= pr.j0 && lx < kNs && ly < kNsY;
#pragma unroll
      for (int e = 0; e < 3; ++e) {
        const double at = E[e] + 7.0 * (lx * ax[e] + ly * ay[e]);
        may = may && at + 7.0 * (fmax(ax[e], 0.0) + fmax(ay[e], 0.0)) >= T.th[e];
      }
      for (uint64_t m = __ballot(may); m; m &= m - 1) {
        const int b = (int)__builtin_ctzll(m), bx = b & 7, by = b >> 3;
        const double e0 = E[0] + 8.0 * (bx * ax[0] + by * ay[0]);
        const double e1 = E[1] + 8.0 * (bx * ax[1] + by * ay[1]);
        const double e2 = E[2] + 8.0 * (bx * ax[2] + by * ay[2]);
        if (x0 + 8 * bx + lx > x1 || y0 + 8 * by + ly > y1) continue;
        if (e0 >= T.th[0] && e1 >= T.th[1] && e2 >= T.th[2]) {
          unsigned long long* slotp = &tile[(8 * by + ly) * B + 8 * bx + lx];
          if (__hip_atomic_load(slotp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) > lbkey)
            atomicMin(slotp, (unsigned long long)depth_key(T, e0, e1, e2, (uint32_t)t));
          ++frags;
        }
      }
    }
  };
  // where large triangles wait: front-facing ones in the queue, which is free until the others come
  int32_t* bigs = queue;
  uint32_t big_cap = kRasterThreads;
  // A triangle for the whole wavefront rather than one lane (its box clipped to the bin is i0..i1 x j0..j1).
  auto is_big = [&](const TriSetup& T, int i0, int i1, int j0, int j1) {
    const double spanx = fmax(T.X[0], fmax(T.X[1], T.X[2])) - fmin(T.X[0], fmin(T.X[1], T.X[2]));
    const double spany = fmax(T.Y[0], fmax(T.Y[1], T.Y[2])) - fmin(T.Y[0], fmin(T.Y[1], T.Y[2]));
    return !(spanx <= kSmallSpan && spany <= kSmallSpan && (i1 - i0 + 1) * (j1 - j0 + 1) <= kSmallArea);
  };
  // Lanes that share one triangle of a chunk of m, as a power of two: a chunk that leaves lanes idle
  // gives each triangle several of them, which take its rows in turn.
  auto share = [](uint32_t m) { return m > 128 ? 0 : m > 64 ? 1 : m > 32 ? 2 : m > 16 ? 3 : 4; };
  // Draw every parts-th row from row part of triangle tq of this layer (tq < 0: nothing); large ones are
  // queued for flush_bigs.
  auto draw = [&](int32_t tq, int part, int parts) {
    TriSetup T;
    if (tq >= 0 && setup_triangle<true>(tri, (uint32_t)tq, nvert, P, T) == kTriOk) {
      const int32_t t = tq;
      PixRange pr = pixel_range(T, W, H);
      const int ci0 = max(pr.i0, x0), ci1 = min(pr.i1, x1), cj0 = max(pr.j0, y0), cj1 = min(pr.j1, y1);
      if (ci0 <= ci1 && cj0 <= cj1) {
        const unsigned long long lbkey = depth_lower_key(T, (uint32_t)t);
        if (!is_big(T, ci0, ci1, cj0, cj1)) {
          // exact int32 edge walk: every edge value inside the bbox is below 2^30 in magnitude
          double E[3];
          edge_values(T, 256.0 * ci0 + 128.0, 256.0 * (cj0 + part) + 128.0, E);
          int32_t er0 = (int32_t)E[0] - (int32_t)T.th[0];
          int32_t er1 = (int32_t)E[1] - (int32_t)T.th[1];
          int32_t er2 = (int32_t)E[2] - (int32_t)T.th[2];
          const int32_t ax0 = (int32_t)(-(T.Y[2] - T.Y[1]) * 256.0), ay0 = (int32_t)((T.X[2] - T.X[1]) * 256.0);
          const int32_t ax1 = (int32_t)(-(T.Y[0] - T.Y[2]) * 256.0), ay1 = (int32_t)((T.X[0] - T.X[2]) * 256.0);
          const int32_t ax2 = (int32_t)(-(T.Y[1] - T.Y[0]) * 256.0), ay2 = (int32_t)((T.X[1] - T.X[0]) * 256.0);
          for (int j = cj0 + part; j <= cj1; j += parts) {
            int32_t e0 = er0, e1 = er1, e2 = er2;
            for (int i = ci0; i <= ci1; ++i) {
              if ((e0 | e1 | e2) >= 0) {
                unsigned long long* slotp = &tile[(j - y0) * B + (i - x0)];
                // keys only decrease, so a single-copy-atomic read at or below the bound proves a loss
                if (__hip_atomic_load(slotp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) > lbkey) {
                  const double E0 = (double)e0 + T.th[0], E1 = (double)e1 + T.th[1], E2 = (double)e2 + T.th[2];
                  atomicMin(slotp, (unsigned long long)depth_key(T, E0, E1, E2, (uint32_t)t));
                }
                ++frags;
              }
              e0 += ax0; e1 += ax1; e2 += ax2;
            }
            er0 += ay0 * parts; er1 += ay1 * parts; er2 += ay2 * parts;
          }
        } else if (part == 0) {
          const uint32_t at = atomicAdd(&bign, 1u);
          if (at < big_cap) bigs[at] = t;
        }
      }
    }
  };
  // Draw the large triangles that draw() met among the loaded groups' entries of one side, dealt round the
  // wavefronts; if they were more than the queue holds, the entries are gone through again.  Called by the
  // whole block.
  auto flush_bigs = [&](bool fronts) {
    __syncthreads();
    const uint32_t nb = bign;
    if (nb == 0) return;   // uniform
    const uint32_t dealt = lane * (kRasterThreads / 64) + (tid >> 6);
    if (nb <= big_cap) {
      draw_bigs(dealt < nb ? bigs[dealt] : -1);
    } else {
      const uint32_t n = fronts ? seg_n[1] : seg_n[2];
      for (uint32_t c = 0; c < n; c += kRasterThreads) {
        int32_t t = -1;
        if (c + dealt < n) {
          const int32_t tc = fronts ? front_entry(c + dealt) : other_entry(c + dealt).t;
          TriSetup T;
          if (setup_triangle<true>(tri, (uint32_t)tc, nvert, P, T) == kTriOk) {
            const PixRange pr = pixel_range(T, W, H);
            const int ci0 = max(pr.i0, x0), ci1 = min(pr.i1, x1), cj0 = max(pr.j0, y0), cj1 = min(pr.j1, y1);
            if (ci0 <= ci1 && cj0 <= cj1 && is_big(T, ci0, ci1, cj0, cj1)) t = tc;
          }
        }
        draw_bigs(t);
      }
    }
    __syncthreads();
    if (tid == 0) bign = 0;
  };
  // phase 1: front-facing entries
  bool one_load = false, any_back = false;   // uniform
  for (int g0 = 0; g0 < n_groups;) {
    const int next = load_segs(g0);
    one_load = g0 == 0 && next >= n_groups;
    g0 = next;
    const uint32_t n_front = seg_n[1], n_back = seg_n[2];
    any_back = any_back || n_back > 0;
    if (tid < (int)seg_n[0] && seg_base[tid] >= kSegAll) no_run = 1;
    for (uint32_t c0 = 0; c0 < n_front; c0 += kRasterThreads) {
      const int sh = share(n_front - c0);
      const uint32_t c = c0 + (tid >> sh);
      draw(c < n_front ? front_entry(c) : -1, tid & ((1 << sh) - 1), 1 << sh);
    }
    flush_bigs(true);
    if (!one_load) __syncthreads();   // the groups are loaded anew
  }
  if (any_back) {   // uniform: back-facing entries follow
    bigs = late_bigs;
    big_cap = kBigQueue;
    __syncthreads();
    {
      // sub-tile maxima without LDS atomics: the kThr consecutive lanes of a sub-tile
      // each take kPer of its keys (whole row pieces) and combine by lane exchange
      constexpr int kSubs = kNs * kNsY;
      constexpr int kThr = kSubs * 64 <= kRasterThreads ? 64 : kSubs * 16 <= kRasterThreads ? 16 : 4;   // per sub-tile
      constexpr int kPer = kSub * kSub / kThr;                                                          // keys per thread
      static_assert(kSubs * kThr <= kRasterThreads && kSub * kSub % kThr == 0, "sub-tile reduction shape");
      if (tid < kSubs * kThr) {   // whole wavefronts
        const int sub = tid / kThr, u = tid % kThr;
        const int sx = sub % kNs, sy = sub / kNs;
        unsigned long long m = 0ull;
#pragma unroll
        for (int e = 0; e < kPer; ++e) {
          const int kk = u * kPer + e;
          m = max(m, tile[(sy * kSub + kk / kSub) * B + sx * kSub + kk % kSub]);
        }
#pragma unroll
        for (int off = kThr / 2; off > 0; off >>= 1) m = max(m, (unsigned long long)__shfl_xor(m, off));
        if (u == 0) smax[sub] = (uint32_t)(m >> 32);
      }
    }
    __syncthreads();
    // phase 2: each back-facing entry is tested from its word (box and depth bound) alone;
    // the ones that may lower a key are queued in LDS and drawn 256 at a time, so that the
    // skipped majority costs no vertex loads and leaves no idle lanes behind.  A wavefront may be at the
    // next chunk while another still reads what this one queued: each chunk counts in a word of its own,
    // cleared between the barrier after its last reader and the one before its next use.
    uint32_t q = 0;   // queue entries, uniform
    int turn = 0;
    for (int g0 = 0; g0 < n_groups;) {
      g0 = one_load ? n_groups : load_segs(g0);
      const uint32_t n = seg_n[2];
      for (uint32_t c0 = 0; c0 < n; c0 += kRasterThreads) {
        const uint32_t c = c0 + tid;
        bool keep = false;
        int32_t t = 0;
        if (c < n) {
          const Other o = other_entry(c);
          t = o.t;
          keep = count_frags != 0;   // every covered pixel is counted then: nothing is skipped
          for (int sj = o.r0; sj <= o.r1; ++sj)
            for (int si = o.c0; si <= o.c1; ++si) keep = keep || smax[sj * kNs + si] >= o.z;
        }
        const uint64_t kb = __ballot(keep);
        uint32_t base = 0;
        if (lane == 0 && kb) base = atomicAdd(&qadd[turn], (uint32_t)__popcll(kb));
        base = q + __builtin_amdgcn_readfirstlane(base);
        if (keep) queue[base + (uint32_t)__popcll(kb & __lanemask_lt())] = t;
        __syncthreads();
        q += qadd[turn];
        if (tid == 0) qadd[turn == 0 ? 2 : turn - 1] = 0;
        turn = turn == 2 ? 0 : turn + 1;
        const bool last = c0 + kRasterThreads >= n;
        while (q >= kRasterThreads || (last && q > 0)) {   // uniform
          const int sh = share(q), e = tid >> sh;
          draw(e < (int)q ? queue[e] : -1, tid & ((1 << sh) - 1), 1 << sh);
          const uint32_t rest = q > kRasterThreads ? q - kRasterThreads : 0;
          const int32_t moved = tid < (int)rest ? queue[kRasterThreads + tid] : 0;
          __syncthreads();
          if (tid < (int)rest) queue[tid] = moved;
          __syncthreads();
          q = rest;
        }
      }
      flush_bigs(false);
      if (!one_load) __syncthreads();   // the groups are loaded anew
    }
  }
  __syncthreads();
  // coalesced store of the finished tile: pairs of keys as 16-byte stores when
  // every row of the bin starts 16-byte aligned (even view width and plane
  // start; x0 is even), single keys otherwise
  unsigned long long* plane = vis + (int64_t)k * V.pix_offset + (int64_t)l * W * H;
  if (B >= 2 && (W & 1) == 0 && (reinterpret_cast<uintptr_t>(plane) & 15) == 0) {   // uniform
    const ulonglong2* tile2 = reinterpret_cast<const ulonglong2*>(tile);
    for (int p = tid; p < B * BH / 2; p += kRasterThreads) {
      const int i = x0 + (2 * p) % B, j = y0 + (2 * p) / B;
      if (j > y1) continue;
      const ulonglong2 kv = tile2[p];
      unsigned long long* dst = plane + (int64_t)j * W + i;
      if (i + 1 <= x1) *reinterpret_cast<ulonglong2*>(dst) = kv;   // x1 - x0 + 1 is even unless W ends the row
      else if (i <= x1) dst[0] = kv.x;
    }
  } else {
    for (int p = tid; p < B * BH; p += kRasterThreads) {
      const int i = x0 + (p % B), j = y0 + (p / B);
      if (i <= x1 && j <= y1) plane[(int64_t)j * W + i] = tile[p];
    }
  }
  if (count_frags) {
    for (int off = 32; off > 0; off >>= 1) frags += __shfl_xor(frags, off);
    if ((tid & 63) == 0 && frags) atomicAdd(status + VS_STAT_FRAGMENTS, frags);
  }
  if (tid == 0 && no_run) atomicAdd(status + VS_STAT_BIN_OVERFLOW, 1ull);
}

// Steps 2-3, direct form (reference path for tests): one thread per (view,
// layer, triangle) walks its bounding box and takes 64-bit atomic minima in
// the visibility plane, which must hold EMPTY before.
__global__ void __launch_bounds__(256) k_raster_direct(const vs_view* __restrict__ views, LayerTable L,
                                                       const ProjVert* __restrict__ proj, int64_t vpv,
                                                       unsigned long long* __restrict__ vis,
                                                       unsigned long long* __restrict__ status, int count_frags) {
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int v = blockIdx.y;
  const int k = L.k;
  if (g >= L.tri_off[k]) return;
  int l = 0;
  while (l + 1 < k && L.tri_off[l + 1] <= g) ++l;
  const int32_t t = (int32_t)(g - L.tri_off[l]);
  const vs_view& V = views[v];
  const int W = V.cam.width, H = V.cam.height;
  const ProjVert* P = proj + (int64_t)v * vpv + L.vert_off[l];
  TriSetup T;
  const int r = setup_triangle(L.tri[l], (uint32_t)t, L.n_vert[l], P, T);
  if (r != kTriOk) {
    atomicAdd(status + cull_slot(r), 1ull);
    return;
  }
  const PixRange pr = pixel_range(T, W, H);
  if (pr.i0 > pr.i1 || pr.j0 > pr.j1) return;
  unsigned long long* plane = vis + (int64_t)k * V.pix_offset + (int64_t)l * W * H;
  const double dx0 = -(T.Y[2] - T.Y[1]) * 256.0, dy0 = (T.X[2] - T.X[1]) * 256.0;
  const double dx1 = -(T.Y[0] - T.Y[2]) * 256.0, dy1 = (T.X[0] - T.X[2]) * 256.0;
  const double dx2 = -(T.Y[1] - T.Y[0]) * 256.0, dy2 = (T.X[1] - T.X[0]) * 256.0;
  double Er[3];
  edge_values(T, 256.0 * pr.i0 + 128.0, 256.0 * pr.j0 + 128.0, Er);
  unsigned long long frags = 0;
  for (int j = pr.j0; j <= pr.j1; ++j) {
    double E0 = Er[0], E1 = Er[1], E2 = Er[2];
    for (int i = pr.i0; i <= pr.i1; ++i) {
      if (E0 >= T.th[0] && E1 >= T.th[1] && E2 >= T.th[2]) {
        atomicMin(plane + (int64_t)j * W + i, (unsigned long long)depth_key(T, E0, E1, E2, (uint32_t)t));
        ++frags;
      }
      E0 += dx0; E1 += dx1; E2 += dx2;
    }
    Er[0] += dy0; Er[1] += dy1; Er[2] += dy2;
  }
  if (count_frags && frags) atomicAdd(status + VS_STAT_FRAGMENTS, frags);
}

}  // namespace vs
