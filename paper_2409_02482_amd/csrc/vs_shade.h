// Shading kernels (steps 4-5): perspective-correct UV, bilinear texture
// fetch, fixed-order front-to-back blending, and the texture adjoint.
//
// Barycentrics, UVs and texel coordinates are computed in FP64 (an FP32 texel
// coordinate near 1024 has an ulp of 6e-5 texel); the fractional offsets,
// the bilinear blend and the compositing run in FP32.
//
// Work decomposition: one 256-thread block per 16 x 16 pixel tile of one
// view, one thread per pixel, layers walked front to back.  Tiles of all
// views are numbered consecutively; the block -> tile mapping gives each XCD
// (blocks are dealt round-robin to the 8 XCDs) a contiguous run of tiles so
// that neighbouring tiles, which read neighbouring texels, share an L2.
#pragma once

#include "vs_common.h"

namespace vs {

constexpr int kShadeTile = 16;      // 16 x 16 pixel tiles, one 256-thread block each
constexpr int kShadeTileSlot = 1;   // vs_view::tile_offset slot of 16-pixel tiles
constexpr int kNumXcd = 8;

struct Foot {
  int32_t i0, i1, j0, j1;  // wrapped texel indices of the 2x2 footprint
  float fx, fy;            // offsets from texel centre (i0, j0)
};

// Split a texel-centre coordinate into the two neighbouring texel indices and
// the offset from the first, wrapping (repeat) or clamping to [0, n-1].
__device__ inline void split_coord(double x, int32_t n, double inv_n, int wrap, int32_t& i0, int32_t& i1,
                                   float& fr) {
  x = fmin(fmax(x, -1.0e9), 1.0e9);  // also maps NaN to a finite value
  if (wrap == kWrapClamp) {
    x = fmin(fmax(x, 0.0), (double)(n - 1));
    const double f = floor(x);
    i0 = (int32_t)f;
    fr = (float)(x - f);
    i1 = i0 + 1 < n ? i0 + 1 : n - 1;
    return;
  }
  const double f = floor(x);
  fr = (float)(x - f);
  double m = f - (double)n * floor(f * inv_n);  // f mod n, exact for |f| < 2^52
  int32_t i = (int32_t)m;
  if (i < 0) i += n;
  if (i >= n) i -= n;
  i0 = i;
  i1 = i + 1 == n ? 0 : i + 1;
}

// The second texel index of a footprint from the first (as split_coord pairs them).
__device__ inline int32_t next_index(int32_t i0, int32_t n, int wrap) {
  return wrap == kWrapClamp ? (i0 + 1 < n ? i0 + 1 : n - 1) : (i0 + 1 == n ? 0 : i0 + 1);
}

// Texel idx of a texture and float idx of a gradient plane, addressed as 32-bit
// byte offsets from the (uniform) plane base, so that the loads and atomics use
// a scalar base register and no per-lane 64-bit address arithmetic: a texture
// has at most 16384^2 texels, whose 16-byte texels and 4-byte gradient floats
// both stay below 2^32 bytes.
__device__ inline float4 texel_at(const float4* __restrict__ tex, uint32_t idx) {
  return *reinterpret_cast<const float4*>(reinterpret_cast<const char*>(tex) + (size_t)(idx << 4));
}

__device__ inline void grad_add(float* G, uint32_t fidx, float val) {
  unsafeAtomicAdd(reinterpret_cast<float*>(reinterpret_cast<char*>(G) + (size_t)(fidx << 2)), val);
}

__device__ inline float4 bilinear(const float4* __restrict__ tex, int32_t W, const Foot& f) {
#pragma clang fp contract(fast)
  const uint32_t w = (uint32_t)W, r0 = (uint32_t)f.j0 * w, r1 = (uint32_t)f.j1 * w;
  const float4 t00 = texel_at(tex, r0 + (uint32_t)f.i0);
  const float4 t01 = texel_at(tex, r0 + (uint32_t)f.i1);
  const float4 t10 = texel_at(tex, r1 + (uint32_t)f.i0);
  const float4 t11 = texel_at(tex, r1 + (uint32_t)f.i1);
  const float gx = 1.0f - f.fx, gy = 1.0f - f.fy;
  const float w00 = gx * gy, w01 = f.fx * gy, w10 = gx * f.fy, w11 = f.fx * f.fy;
  float4 r;
  r.x = w00 * t00.x + w01 * t01.x + w10 * t10.x + w11 * t11.x;
  r.y = w00 * t00.y + w01 * t01.y + w10 * t10.y + w11 * t11.y;
  r.z = w00 * t00.z + w01 * t01.z + w10 * t10.z + w11 * t11.z;
  r.w = w00 * t00.w + w01 * t01.w + w10 * t10.w + w11 * t11.w;
  return r;
}

struct Tri3 { int32_t a, b, c; };

// Rebuild the triangle a key names and interpolate its UV at the pixel centre
// (px, py) (1/256 px units).  Barycentrics are perspective-correct:
// lambda_q = E_q w_q / sum_r E_r w_r, which does not depend on the winding,
// so no orientation normalisation is needed here.  Returns false (and counts
// a bad key) if the key names no valid triangle.
__device__ inline bool slot_uv(const int32_t* __restrict__ tri, int32_t n_tri, int32_t n_vert,
                               const ProjVert* __restrict__ P, const float2* __restrict__ uv, uint64_t key,
                               int32_t px, int32_t py, double& u, double& v, unsigned long long* status) {
#pragma clang fp contract(fast)
  const uint32_t t = (uint32_t)(key & 0xffffffffu);
  if (t >= (uint32_t)n_tri) {
    atomicAdd(status + VS_STAT_BAD_KEY, 1ull);
    return false;
  }
  const Tri3 id = elem_at<Tri3>(tri, t);
  if ((uint32_t)id.a >= (uint32_t)n_vert || (uint32_t)id.b >= (uint32_t)n_vert ||
      (uint32_t)id.c >= (uint32_t)n_vert) {
    atomicAdd(status + VS_STAT_BAD_KEY, 1ull);
    return false;
  }
  const ProjVert a = elem_at<ProjVert>(P, (uint32_t)id.a), b = elem_at<ProjVert>(P, (uint32_t)id.b),
                 c = elem_at<ProjVert>(P, (uint32_t)id.c);
  const float2 ua = elem_at<float2>(uv, (uint32_t)id.a), ub = elem_at<float2>(uv, (uint32_t)id.b),
               uc = elem_at<float2>(uv, (uint32_t)id.c);
  // relative to the pixel the corners are integers below 2^25, so that the products (below 2^50) and the
  // edge values are exact, as they are from the edges' differences, in fewer steps
  const double ax = a.X - px, ay = a.Y - py, bx = b.X - px, by = b.Y - py, cx = c.X - px, cy = c.Y - py;
  const double E0 = bx * cy - by * cx, E1 = cx * ay - cy * ax, E2 = ax * by - ay * bx;
  const double q0 = E0 * a.w, q1 = E1 * b.w, q2 = E2 * c.w;
  const double s = q0 + q1 + q2;
  // 1/s: hardware reciprocal refined by two Newton steps (relative error ~1e-16)
  double r = __builtin_amdgcn_rcp(s);
  r = r * (2.0 - s * r);
  r = r * (2.0 - s * r);
  const double la = q0 * r, lb = q1 * r, lc = q2 * r;
  u = la * (double)ua.x + lb * (double)ub.x + lc * (double)uc.x;
  v = la * (double)ua.y + lb * (double)ub.y + lc * (double)uc.y;
  return true;
}

// The slot's bilinear footprint in a W x H texture.
__device__ inline bool slot_footprint(const int32_t* __restrict__ tri, int32_t n_tri, int32_t n_vert,
                                      const ProjVert* __restrict__ P, const float2* __restrict__ uv, uint64_t key,
                                      int32_t px, int32_t py, int32_t W, int32_t H, double invW, double invH, int wrap,
                                      Foot& f, unsigned long long* status) {
  double u, v;
  if (!slot_uv(tri, n_tri, n_vert, P, uv, key, px, py, u, v, status)) return false;
  split_coord(u * (double)W - 0.5, W, invW, wrap, f.i0, f.i1, f.fx);
  split_coord(v * (double)H - 0.5, H, invH, wrap, f.j0, f.j1, f.fy);
  return true;
}

struct TileCoord {
  int v, x, y;
  bool valid;
  bool live;   // false for padding blocks of the XCD remap
};

// Block -> (view, tile) with an XCD-contiguous remap; tile_view[g] is the view of tile g.
// A tile whose table entry is out of range (a workspace not filled by
// vs_raster_layers for these views) is skipped rather than trusted.
// A block takes TILES consecutive tiles, 256 threads each.
template <int TILES = 1>
__device__ inline TileCoord shade_tile_coord(const vs_view* __restrict__ views, int n_views,
                                             const int32_t* __restrict__ tile_view, int64_t n_tiles) {
  TileCoord c;
  const int64_t chunk = (n_tiles + kNumXcd - 1) / kNumXcd;
  const int64_t b = blockIdx.x;
  const int64_t in = TILES == 1 ? b / kNumXcd : b / kNumXcd * TILES + __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);
  const int64_t g = (b % kNumXcd) * chunk + in;
  c.v = 0; c.x = c.y = 0; c.valid = false;
  c.live = in < chunk && g < n_tiles;
  if (!c.live) return c;
  c.v = tile_view[g];
  if ((unsigned)c.v >= (unsigned)n_views) { c.v = 0; c.live = false; return c; }
  const vs_view& V = views[c.v];
  const int64_t local = g - V.tile_offset[kShadeTileSlot];
  const int tiles_x = (V.cam.width + kShadeTile - 1) / kShadeTile;
  const int64_t ty = local / tiles_x, tx = local - ty * tiles_x;
  if (local < 0 || ty * kShadeTile >= V.cam.height) { c.live = false; return c; }
  // row-major: wave w covers rows 4w..4w+3 of the tile, and each DPP row of 16 lanes is a pixel row
  const int t = threadIdx.x & 255;
  c.x = (int)tx * kShadeTile + (t & 15);
  c.y = (int)ty * kShadeTile + (t >> 4);
  c.valid = c.x < V.cam.width && c.y < V.cam.height;
  return c;
}

__host__ __device__ inline int64_t shade_grid_blocks(int64_t n_tiles, int tiles = 1) {
  return ((n_tiles + kNumXcd - 1) / kNumXcd + tiles - 1) / tiles * kNumXcd;
}

// Forward: one thread per pixel, layers front to back.
__global__ void __launch_bounds__(256) k_shade_fwd(const vs_view* __restrict__ views, int n_views,
                                                   const int32_t* __restrict__ tile_view,
                                                   int64_t n_tiles, LayerTable L, TexTable X,
                                                   const ProjVert* __restrict__ proj, int64_t vpv,
                                                   const uint64_t* __restrict__ vis, float4* __restrict__ out,
                                                   float eps_T, int wrap, unsigned long long* __restrict__ status) {
#pragma clang fp contract(fast)
  const TileCoord c = shade_tile_coord(views, n_views, tile_view, n_tiles);
  if (!c.live) return;
  const vs_view& V = views[c.v];
  const int W = V.cam.width, H = V.cam.height;
  const int64_t P = (int64_t)W * H;
  const int k = L.k;
  const int64_t pix = (int64_t)c.y * W + c.x;
  const uint64_t* vrow = vis + (int64_t)k * V.pix_offset + pix;
  const ProjVert* pview = proj + (int64_t)c.v * vpv;
  const int32_t px = 256 * c.x + 128, py = 256 * c.y + 128;
  float Cr = 0.f, Cg = 0.f, Cb = 0.f, T = c.valid ? 1.0f : 0.0f;
  // keys of the first layers are requested together (several loads in flight)
  constexpr int kPre = 4;
  uint64_t pre[kPre];
#pragma unroll
  for (int l = 0; l < kPre; ++l) pre[l] = (l < k && c.valid) ? vrow[l * P] : kEmpty;
  for (int l = 0; l < k; ++l) {
    uint64_t key;
    if (l < kPre) {
      key = pre[0];
#pragma unroll
      for (int q = 1; q < kPre; ++q) key = (l == q) ? pre[q] : key;
    } else {
      key = c.valid ? vrow[l * P] : kEmpty;
    }
    if (key != kEmpty) {
      Foot f;
      const int32_t Wt = X.w[l], Ht = X.h[l];
      if (slot_footprint(L.tri[l], L.n_tri[l], L.n_vert[l], pview + L.vert_off[l],
                         reinterpret_cast<const float2*>(L.uv[l]), key, px, py, Wt, Ht, X.inv_w[l], X.inv_h[l],
                         wrap, f, status)) {
        const float4 s = bilinear(X.tex[l], Wt, f);
        const float ta = T * s.w;
        Cr += ta * s.x; Cg += ta * s.y; Cb += ta * s.z;
        T *= (1.0f - s.w);
      }
    }
    if (eps_T > 0.f && __all(T < eps_T)) break;
  }
  if (c.valid) out[V.pix_offset + pix] = make_float4(Cr, Cg, Cb, 1.0f - T);
}

// Orders this wavefront's LDS accesses (a wave's LDS instructions execute in order).
__device__ inline void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Relative texel offset of index i from reference r in [-n/2, n/2) (repeat) or plain difference (clamp).
__device__ inline int32_t rel_index(int32_t i, int32_t r, int32_t n, int wrap) {
  int32_t d = i - r;
  if (wrap == kWrapClamp) return d;
  if (d >= (n >> 1)) d -= n;
  else if (d < -(n >> 1)) d += n;
  return d;
}

__device__ inline int32_t abs_index(int32_t r, int32_t d, int32_t n, int wrap) {
  int32_t i = r + d;
  if (wrap == kWrapClamp) return i;
  if (i >= n) i -= n;
  else if (i < 0) i += n;
  return i;
}

// Texels in each wavefront's LDS gradient window, and wavefronts per SIMD, by the
// largest layer count of the instantiation and its 16 x 16 pixel tiles per block.
// Up to 9 layers seven blocks of 272-texel windows (21 KiB) share a CU at 72
// registers (8 and 9 layers spill 5 and 14).  Windows of 320, 272 and 240 texels
// at six, seven and eight blocks: metric scene 6.73 / 6.36 / 6.61 ms, 128 views at
// 800^2 9.35 / 8.90 / 9.03 (fastest launches; with 272 texels they average 9.7 in a fitting
// loop), k = 9 scene 6.72 / 6.66 / 6.90, 384 texels at five blocks 7.25 / 9.77 / 6.91.  Up to 16 layers, five blocks of 288 (384 texels at two, four blocks of
// 320): 12 layers, six views of 700 x 600, 550 us (690, 611); 16 layers 771 us (931, 842).
// Two tiles per block (kShadeLossTiles) halve the atomics into the one double of
// the loss sum, which the memory side takes one after the other (5.8 ns each,
// beside all others): up to 4 layers they take longer than the pixels.  Three
// layers, six views of 801 x 603: 168 us with one tile per block, 120 with two, 105
// without a sum; without a sum two tiles cost 3 % (four layers), and from 5 layers
// on they cost more than they save (metric 6.36 -> 6.93 ms).
template <int KMAX, int TILES> struct BwdShape {
  static constexpr int win = KMAX > 9 ? 288 : TILES == 1 ? 272 : 252;
  static constexpr int waves = KMAX > 9 ? 5 : TILES == 1 ? 7 : 8;
};
constexpr int kShadeLossTiles = 2;
constexpr int kShadeLossLayers = 4;   // ... up to this many layers

// v + (v of lane + N) within a DPP row of 16 lanes (row_shl:N).
template <int N>
__device__ inline float add_next(float v) {
  return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x100 + N, 0xf, 0xf, false));
}

// One step of summing runs: the lanes of src add their values into the lanes N below.  Only
// these lanes are active, so that the lane exchange folds into the adds (16 v_add_f32_dpp per
// step) and no value of another run is touched; what a src lane computes is discarded.
template <int N>
__device__ inline void run_step(uint64_t src, float (&v)[16]) {
  if (src == 0) return;   // uniform
  if (__builtin_amdgcn_inverse_ballot_w64(src | (src >> N))) {
#pragma unroll
    for (int q = 0; q < 16; ++q) v[q] = add_next<N>(v[q]);
  }
}

// Sums the contributions of each run of neighbouring pixels of a row that share a base texel
// (key >= 0) into the run's first lane, by halves of the distance from it; the other lanes of a
// run drop out (key = -1).  Runs start anywhere, where aligned pairs (x +- 1, y +- 1, x +- 2) left
// 3.2 rounds of adding per window: metric adjoint 7.38 -> 7.06 ms, four magnified layers 405 -> 390 us.
__device__ inline void merge_runs(int32_t& key, float (&v)[16], int lane) {
  const int32_t prev = __builtin_amdgcn_update_dpp(-2, key, 0x111, 0xf, 0xf, false);   // lane - 1; -2 at a row's start
  const bool cont = key >= 0 && prev == key;
  if (!__any(cont)) return;   // uniform
  // distance from the run's first lane: the nearest lane at or below this one, in its row, that continues nothing
  const uint64_t first = ~__ballot(cont);
  const uint32_t word = lane < 32 ? (uint32_t)first : (uint32_t)(first >> 32);
  const uint32_t upto = word & ((2u << (lane & 31)) - 1u) & (0xffffu << (lane & 16));
  const int o = (lane & 31) - 31 + __clz((int)upto);
  run_step<1>(__ballot(cont && (o & 1) == 1), v);
  run_step<2>(__ballot(cont && (o & 3) == 2), v);
  run_step<4>(__ballot(cont && (o & 7) == 4), v);
  run_step<8>(__ballot(cont && o == 8), v);
  if (cont) key = -1;
}

// The adjoint's arguments, passed by value.
struct BwdArgs {
  LayerTable L;
  TexTable X;
  const vs_view* views;
  const int32_t* tile_view;
  int64_t n_tiles;
  const ProjVert* proj;
  int64_t vpv;
  const uint64_t* vis;
  const float4* grad_out;
  const float4* target;
  float4* out;
  double* sse;
  unsigned long long* status;
  int32_t n_views, loss, wrap, count_paths;
  float loss_scale, eps_T;
};
// Backward: recompute the layers front to back (keeping T in front of each hit layer and
// its bilinear footprint), form dL/d(RGB, A), then walk back to front:
//   dL/dc_l = g_rgb a_l T_l,  dL/da_l = T_l <g_rgb, c_l - S_l> + g_A T_l prod_{m>l}(1 - a_m),
// S_l the colour blended behind layer l.  Division-free (a = 1 is fine).
// Each of the 4 corner texels receives its bilinear weight times these.
//
// Scatter, per wavefront (16 x 4 pixels) and layer: neighbouring pixels
// mostly share their base texel (a texel spans several pixels when
// magnified), so the lanes of each run along a pixel row that share a base
// texel first sum their 16 contributions in registers (merge_runs).  The
// survivors add into an LDS texel window (wrap-aware, relative to the first
// surviving lane's base texel) with plain read-modify-writes, one lane per base
// texel and round (an owner word per cell elects it); the window is then
// flushed with global float atomics whose lanes cover consecutive floats, and
// zeroed by the same pass, so it starts every use empty.  A window covers the
// base texels' bounding box plus one column and one row: the second corner of a
// footprint is always the next cell (wrapping happens when the window is mapped
// back to texels; a corner that coincides with the base texel at a clamped edge
// was folded onto it and adds zero).  A footprint larger than the window is
// retried per half wavefront, then per quarter (8 x 2 pixels); what still does
// not fit is added pixel by pixel, 16 consecutive lanes per pixel.
//
// What bounds it (timing variants that skip work, metric scene / 128 views at
// 800^2): the layers' recompute 3.0 / 3.5 ms, forming and merging the
// contributions 0.7 / 0.8, window boxes and flush loops 0.8 / 1.4, electing and
// adding 0.5 / 0.3, the flush's atomics at the memory side 1.35 / 2.6 and those
// of pixels that fit no window 0.55 / 1.55 before they were grouped.
template <int KMAX, int TILES>
__global__ void __launch_bounds__(256 * TILES, (BwdShape<KMAX, TILES>::waves)) k_shade_bwd(BwdArgs args) {
#pragma clang fp contract(fast)
  constexpr int kWaveWin = BwdShape<KMAX, TILES>::win;
  constexpr int kWaves = 4 * TILES;
  __shared__ __align__(16) float win_all[kWaves][kWaveWin * 5];   // per wave: RGBA sums, then the owner words
  __shared__ double sred[kWaves];                                 // per wave: the loss sum
  // the window is zero before its first use; every flush leaves it zero again
  for (int e = threadIdx.x & 63; e < kWaveWin; e += 64)
    reinterpret_cast<float4*>(win_all[threadIdx.x >> 6])[e] = make_float4(0.f, 0.f, 0.f, 0.f);
  const LayerTable& L = args.L;
  const TexTable& X = args.X;
  const TileCoord c = shade_tile_coord<TILES>(args.views, args.n_views, args.tile_view, args.n_tiles);
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  // one atomic per block into the loss
  auto add_loss = [&](double mine) {
    for (int off = 32; off > 0; off >>= 1) mine += __shfl_xor(mine, off);
    if (lane == 0) sred[tid >> 6] = mine;
    __syncthreads();
    if (tid == 0) {
      double sum = sred[0];
#pragma unroll
      for (int q = 1; q < kWaves; ++q) sum += sred[q];
      unsafeAtomicAdd(args.sse, sum);
    }
  };
  if (!c.live) {   // uniform per tile
    if (args.sse && TILES > 1) add_loss(0.0);
    return;
  }
  float* win = win_all[tid >> 6];
  float4* wg = reinterpret_cast<float4*>(win);                     // [cell] RGBA sums
  int32_t* owner = reinterpret_cast<int32_t*>(win + kWaveWin * 4);  // [cell]
  const vs_view& V = args.views[c.v];
  const int W = V.cam.width, H = V.cam.height;
  const int64_t P = (int64_t)W * H;
  const int k = L.k, wrap = args.wrap;
  const float eps_T = args.eps_T;
  const int64_t pix = (int64_t)c.y * W + c.x;
  const uint64_t* vrow = args.vis + (int64_t)k * V.pix_offset + pix;
  const ProjVert* pview = args.proj + (int64_t)c.v * args.vpv;
  const int32_t px = 256 * c.x + 128, py = 256 * c.y + 128;
  // every layer's key is requested before any is used (k loads in flight)
  uint64_t keys[KMAX];
#pragma unroll
  for (int l = 0; l < KMAX; ++l) keys[l] = (l < k && c.valid) ? vrow[l * P] : kEmpty;
  // Kept per hit layer for the backward walk: T in front of it and the footprint; the
  // sample itself is re-read there (four texels, still cache resident), which keeps the
  // register count, and so the number of resident wavefronts, up: keeping the samples
  // instead costs either spills (at five blocks per CU) or a block per CU.
  float Tl[KMAX], fxs[KMAX], fys[KMAX];
  int32_t ij[KMAX];   // packed (j0 << 16 | i0); i1, j1 follow from them
  uint32_t hitmask = 0;
  // T starts at 0 on padding lanes, as in k_shade_fwd, so that both kernels take the same early exit
  float Cr = 0.f, Cg = 0.f, Cb = 0.f, T = c.valid ? 1.0f : 0.0f;
  bool walk = true;
#pragma unroll
  for (int l = 0; l < KMAX; ++l) {
    Foot f;
    if (walk && keys[l] != kEmpty &&
        slot_footprint(L.tri[l], L.n_tri[l], L.n_vert[l], pview + L.vert_off[l],
                       reinterpret_cast<const float2*>(L.uv[l]), keys[l], px, py, X.w[l], X.h[l], X.inv_w[l],
                       X.inv_h[l], wrap, f, args.status)) {
      const float4 s = bilinear(X.tex[l], X.w[l], f);
      hitmask |= 1u << l;
      Tl[l] = T;
      fxs[l] = f.fx; fys[l] = f.fy;
      ij[l] = (f.j0 << 16) | f.i0;
      const float ta = T * s.w;
      Cr += ta * s.x; Cg += ta * s.y; Cb += ta * s.z;
      T *= (1.0f - s.w);
    }
    // the forward kernel's early exit: the layers behind it are neither blended nor differentiated
    if (l < k && eps_T > 0.f && __all(T < eps_T)) walk = false;
  }
  float gr = 0.f, gg = 0.f, gb = 0.f, gA = 0.f;
  double my_sse = 0.0;
  if (c.valid) {
    const int64_t gp = V.pix_offset + pix;
    const float loss_scale = args.loss_scale;
    if (args.target) {
      const float4 tg = args.target[gp];
      const float dr = Cr - tg.x, dg = Cg - tg.y, db = Cb - tg.z;
      if (args.loss == VS_LOSS_L1) {
        // d|x|/dx = sign(x), 0 at a tie
        auto sgn = [](float x) { return (float)((x > 0.0f) - (x < 0.0f)); };
        gr = loss_scale * sgn(dr); gg = loss_scale * sgn(dg); gb = loss_scale * sgn(db);
        my_sse = (double)fabsf(dr) + (double)fabsf(dg) + (double)fabsf(db);
      } else {
        const float s2 = 2.0f * loss_scale;
        gr = s2 * dr; gg = s2 * dg; gb = s2 * db;
        my_sse = (double)dr * dr + (double)dg * dg + (double)db * db;
      }
    } else {
      const float4 go = args.grad_out[gp];
      gr = go.x; gg = go.y; gb = go.z; gA = go.w;
    }
    if (args.out) args.out[gp] = make_float4(Cr, Cg, Cb, 1.0f - T);
  }
  if (args.sse) add_loss(my_sse);   // before the scatter: a barrier after it would wait for every gradient atomic
  float Sr = 0.f, Sg = 0.f, Sb = 0.f, Pm = 1.0f;
  const int quarter = (lane >> 5) * 2 + ((lane >> 3) & 1);   // 8 x 2 pixel block of the wavefront's 16 x 4
  uint32_t n_path[4] = {0u, 0u, 0u, 0u};   // wavefront-uniform: window per wave / half / quarter, direct
#pragma unroll
  for (int l = KMAX - 1; l >= 0; --l) {
    if (l >= k) continue;  // uniform
    const bool hit = (hitmask >> l) & 1u;
    if (!__any(hit)) continue;  // uniform per wavefront
    const int32_t Wt = X.w[l], Ht = X.h[l];
    float v[16];
    int32_t key = -1, i0 = 0, j0 = 0;
#pragma unroll
    for (int q = 0; q < 16; ++q) v[q] = 0.0f;
    if (hit) {
      i0 = ij[l] & 0xffff; j0 = ij[l] >> 16;
      Foot f;
      f.i0 = i0; f.j0 = j0; f.i1 = next_index(i0, Wt, wrap); f.j1 = next_index(j0, Ht, wrap);
      f.fx = fxs[l]; f.fy = fys[l];
      const float4 smp = bilinear(X.tex[l], Wt, f);   // the same sample as the forward walk
      const float a = smp.w, Tv = Tl[l];
      const float aT = a * Tv;
      float d[4];
      d[0] = gr * aT; d[1] = gg * aT; d[2] = gb * aT;
      d[3] = Tv * (gr * (smp.x - Sr) + gg * (smp.y - Sg) + gb * (smp.z - Sb)) + gA * Tv * Pm;
      Sr = a * smp.x + (1.0f - a) * Sr;
      Sg = a * smp.y + (1.0f - a) * Sg;
      Sb = a * smp.z + (1.0f - a) * Sb;
      Pm *= (1.0f - a);
      const float fx = fxs[l], fy = fys[l], gx = 1.0f - fx, gy = 1.0f - fy;
      const float wq[4] = {gx * gy, fx * gy, gx * fy, fx * fy};
#pragma unroll
      for (int n = 0; n < 4; ++n) {
#pragma unroll
        for (int ch = 0; ch < 4; ++ch) v[n * 4 + ch] = wq[n] * d[ch];
      }
      key = j0 * Wt + i0;
    }
    // Clamped at the last column or row (or a texture one texel wide or high), corners
    // coincide: fold them onto the base texel's row or column, so that the corner
    // after it receives zero.  Uniform test: never taken for repeat-wrapped textures
    // wider and higher than one texel.
    if (wrap == kWrapClamp || Wt == 1 || Ht == 1) {
      if (hit && next_index(i0, Wt, wrap) == i0) {
#pragma unroll
        for (int ch = 0; ch < 4; ++ch) { v[ch] += v[4 + ch]; v[4 + ch] = 0.f; v[8 + ch] += v[12 + ch]; v[12 + ch] = 0.f; }
      }
      if (hit && next_index(j0, Ht, wrap) == j0) {
#pragma unroll
        for (int ch = 0; ch < 4; ++ch) { v[ch] += v[8 + ch]; v[8 + ch] = 0.f; v[4 + ch] += v[12 + ch]; v[12 + ch] = 0.f; }
      }
    }
    merge_runs(key, v, lane);
    const bool live_all = key >= 0;
    bool direct = false;   // a quarter wavefront whose footprint did not fit: direct atomics below
    float* G = X.grad[l];
    // A footprint larger than the window is retried per half wavefront (lanes
    // 0-31, then 32-63), a half that does not fit per quarter (16 lanes: an
    // 8 x 2 pixel block); a quarter that still does not fit uses direct atomics.
    for (int pass = 0, npass = 1; pass < npass; ++pass) {   // uniform control flow
      const bool live = live_all && (npass == 1 || (npass == 2 ? lane >> 5 : quarter) == pass);
      const uint64_t live_bits = __ballot(live);
      if (live_bits == 0) continue;
      // window relative to the base texel of the first surviving lane, wrap-aware
      const int first = __builtin_ctzll(live_bits);
      const int32_t ri = __builtin_amdgcn_readlane(i0, first), rj = __builtin_amdgcn_readlane(j0, first);
      const int32_t di = live ? rel_index(i0, ri, Wt, wrap) : 0;
      const int32_t dj = live ? rel_index(j0, rj, Ht, wrap) : 0;
      const int32_t dmin_i = wave_min(live ? di : INT32_MAX);
      const int32_t dmax_i = wave_max(live ? di : INT32_MIN) + 1;
      const int32_t dmin_j = wave_min(live ? dj : INT32_MAX);
      const int32_t dmax_j = wave_max(live ? dj : INT32_MIN) + 1;
      const int32_t ww = dmax_i - dmin_i + 1, wh = dmax_j - dmin_j + 1;
      if (ww * wh <= kWaveWin) {
        ++n_path[npass == 1 ? 0 : npass == 2 ? 1 : 2];
        const int32_t c00 = (dj - dmin_j) * ww + (di - dmin_i);
        const int32_t cells[4] = {c00, c00 + 1, c00 + ww, c00 + ww + 1};
        // For each corner, distinct base texels give distinct cells.  One owner word per
        // base cell elects one lane per base texel and round; the winners then apply the four
        // corners' read-modify-writes one corner at a time.  A wave's LDS instructions complete
        // in order, so no atomics are needed; lanes that lost (equal base texel) retry.
        bool pend = live;
        while (__any(pend)) {
          if (pend) owner[c00] = lane;
          wave_lds_sync();
          const bool mine = pend && owner[c00] == lane;
#pragma unroll
          for (int n = 0; n < 4; ++n) {
            if (mine) {
              float4 acc = wg[cells[n]];
              acc.x += v[n * 4 + 0]; acc.y += v[n * 4 + 1]; acc.z += v[n * 4 + 2]; acc.w += v[n * 4 + 3];
              wg[cells[n]] = acc;
            }
            __asm__ volatile("" ::: "memory");   // keep the corners' LDS accesses in program order
          }
          pend = pend && !mine;
        }
        wave_lds_sync();
        // flush and zero: the window's wh rows of row = 4 ww floats are taken 64 consecutive
        // floats per step (flat index p = y row + cc, so an atomic instruction covers one or
        // two pieces of texture rows, and no lane idles at a row's end); y = floor(p / row) is
        // the high word of p m with m = ceil(2^32 / row), exact since p (m row - 2^32) < 2^32
        // for p < 4 kWaveWin and row <= 4 kWaveWin.
        const int32_t row = ww * 4;
        const int32_t nf = wh * row;                                // floats in the window
        const uint32_t m = 0xffffffffu / (uint32_t)row + 1u;       // uniform (scalar)
        const int32_t bi = ri + dmin_i, bj = rj + dmin_j;   // texel of window cell (0, 0), unwrapped
        const bool flat = bi >= 0 && bi + ww <= Wt && bj >= 0 && bj + wh <= Ht;
        if (flat) {   // the window does not wrap: plain strided addresses
          const uint32_t gbase = ((uint32_t)bj * (uint32_t)Wt + (uint32_t)bi) * 4u;
          const uint32_t gstride = (uint32_t)Wt * 4u;
          for (int32_t p = lane; p < nf; p += 64) {
            const uint32_t y = __umulhi((uint32_t)p, m);
            const uint32_t cc = (uint32_t)p - y * (uint32_t)row;
            const float val = win[p];
            win[p] = 0.0f;
            if (val != 0.0f) grad_add(G, gbase + y * gstride + cc, val);
          }
        } else {
          // wrapped (repeat) or outside the texture (clamp: only zeros land there)
          for (int32_t p = lane; p < nf; p += 64) {
            const int32_t y = (int32_t)__umulhi((uint32_t)p, m);
            const int32_t cc = p - y * row;
            const float val = win[p];
            win[p] = 0.0f;
            if (val != 0.0f) {
              const int32_t tj = abs_index(rj, dmin_j + y, Ht, wrap);
              const int32_t ti = abs_index(ri, dmin_i + (cc >> 2), Wt, wrap);
              grad_add(G, ((uint32_t)tj * (uint32_t)Wt + (uint32_t)ti) * 4u + (uint32_t)(cc & 3), val);
            }
          }
        }
        wave_lds_sync();   // the window is reused by the next pass or layer
      } else if (npass == 1) {
        npass = 2;      // retry by halves
        pass = -1;
      } else if (npass == 2) {
        npass = 4;      // this half again as two quarters, and the halves after it as quarters
        pass = 2 * pass - 1;
      } else {
        direct = direct || live;
        ++n_path[3];
      }
    }
    // What fitted no window (minified texels, pole fans) goes through the window's space as 16
    // floats per lane, so that consecutive lanes of an atomic instruction take the four channels
    // of a texel and of the next one: an atomic request costs the memory side the same for one
    // float as for the 64 bytes around it (with one channel of 64 texels per instruction four
    // layers of 1500^2 textures over six 300^2 views took 304 us instead of 170, and 128 views at
    // 800^2 10.4 ms instead of 9.35).
    constexpr int kParts = kWaveWin * 4 >= 64 * 16 ? 1 : 2;   // lanes' floats that the window's space holds at once
    static_assert(64 / kParts * 16 <= kWaveWin * 4 && 64 / kParts <= kWaveWin, "16 floats and an owner word per lane");
    if (__any(direct)) {
#pragma unroll 1
      for (int part = 0; part < kParts; ++part) {   // uniform
        const bool now = direct && (kParts == 1 || lane >> 5 == part);
        const uint64_t bits = __ballot(now);
        if (now) {
          const uint32_t at = (uint32_t)__popcll(bits & __lanemask_lt());
#pragma unroll
          for (int n = 0; n < 4; ++n) wg[4 * at + n] = make_float4(v[4 * n], v[4 * n + 1], v[4 * n + 2], v[4 * n + 3]);
          owner[at] = (j0 << 16) | i0;
        }
        wave_lds_sync();
        const int32_t nf = 16 * (int32_t)__popcll(bits);
        for (int32_t p = lane; p < nf; p += 64) {
          const float val = win[p];
          win[p] = 0.0f;
          if (val != 0.0f) {
            const int32_t at = owner[p >> 4];
            int32_t ti = at & 0xffff, tj = at >> 16;
            if (p & 4) ti = next_index(ti, Wt, wrap);
            if (p & 8) tj = next_index(tj, Ht, wrap);
            grad_add(G, ((uint32_t)tj * (uint32_t)Wt + (uint32_t)ti) * 4u + (uint32_t)(p & 3), val);
          }
        }
        wave_lds_sync();
      }
    }
  }
  if (args.count_paths && lane == 0) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (n_path[q]) atomicAdd(args.status + VS_STAT_SCATTER_WAVE + q, (unsigned long long)n_path[q]);
  }
}

}  // namespace vs
