// k-SDF volume rendering (Sec. 4.1 "k-SDF", Sec. 4.2 "Surfaces Blending",
// Sec. 4.4 "Occupancy Grid" and "Importance Sampling").
//
// Fields live on vertex grids over the cube [lo, hi]^3 ([z][y][x] order) and
// are read trilinearly.  The occupancy grid is one thread per voxel, decided in
// FP64 and packed to bits with a wavefront ballot.  Rendering is one pixel ray
// per half wavefront (32 lanes): the ray's march steps are spread over the
// lanes (a ballot is 32 steps' bits; occupied-length ranks are a prefix sum of
// words' counts), and so are its samples, up to four a lane.  Transmittance and
// the importance CDF are scans across lanes, inversion a search over the CDF in
// the wave's LDS, and the merge of new samples (existing samples first on ties)
// a gather through a bit map of the places that they take.
// Ray set-up, marching, sample positions and SDF values are FP64 (the
// occupancy decisions and march steps match a plain FP64 evaluation exactly);
// weights, appearance and blending are FP32.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "vs_common.h"

namespace vs {

constexpr int kKsdfWaves = 1;      // wavefronts per block
constexpr int kKsdfBatch = 16;     // most rays a wavefront renders, two at a time

struct KsdfParams {
  const float* sdf;
  const float4* rgba;
  int32_t sdf_res, rgba_res, occ_res;
  double lo, hi, h_occ;
  double inv_sdf, inv_rgba, inv_occ;       // R / (hi - lo) of each grid
  int32_t occ_frac;                        // fraction bits f of the march's fixed point: (occ_res + 1) 2^f <= 2^32
  float cinv[2][VS_KSDF_MAX_SURFACES];     // exp(-beta_r o_j) for beta_r = beta / 2 (round 0) and beta
  float cexp[VS_KSDF_MAX_SURFACES];        // exp(beta o_j)
  int32_t factor;                          // 1: every |beta o_j| <= 60, so exp(-beta_r (d + o_j)) = E cinv
  int32_t k;
  double off[VS_KSDF_MAX_SURFACES];
  double beta, occ_threshold, half_diag;
  double deep;                             // no surface's Phi is 0 in FP64 above this distance
  int32_t n, m, steps;
  float pdf_floor;
};

// The parameters where the launch put them: the first argument of each kernel
// here.  A kernel that loops over rays asks for them anew in each phase, so
// that nothing derived from them is held in registers across the loop (which
// cost 45 spilled registers).
typedef const __attribute__((address_space(4))) KsdfParams& KsdfArgs;
__device__ inline KsdfArgs ksdf_args() {
  uint64_t p = (uint64_t)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return *(const __attribute__((address_space(4))) KsdfParams*)p;
}

// Grid element at a 32-bit element index (grids are limited to 2^32 bytes, so
// the byte offset is a 32-bit unsigned value added to a scalar base address).
__device__ inline float ksdf_at(const float* __restrict__ g, uint32_t i) {
  return *(const float*)((const char*)g + (i << 2));
}
__device__ inline float4 ksdf_at4(const float4* __restrict__ g, uint32_t i) {
  return *(const float4*)((const char*)g + (i << 4));
}

// Cell of a grid coordinate along one axis: base vertex and weight (FP64).
__device__ inline void ksdf_cell(double g, int R, uint32_t& b, double& f) {
  const double c = fmin(fmax(g, 0.0), (double)R);
  b = min((uint32_t)c, (uint32_t)(R - 1));
  f = c - (double)b;
}

// Trilinear lookup of the SDF grid in FP64 at grid coordinates (the
// accumulation order of a plain evaluation: corners z-major, then y, then x).
__device__ inline double ksdf_sdf(KsdfArgs P, double cx, double cy, double cz) {
  const int R = P.sdf_res;
  uint32_t ix, iy, iz;
  double fx, fy, fz;
  ksdf_cell(cx, R, ix, fx);
  ksdf_cell(cy, R, iy, fy);
  ksdf_cell(cz, R, iz, fz);
  const uint32_t R1 = R + 1;
  double acc = 0.0;
#pragma unroll
  for (int dz = 0; dz < 2; ++dz)
#pragma unroll
    for (int dy = 0; dy < 2; ++dy)
#pragma unroll
      for (int dx = 0; dx < 2; ++dx) {
        const double w = ((dx ? fx : 1.0 - fx) * (dy ? fy : 1.0 - fy)) * (dz ? fz : 1.0 - fz);
        const uint32_t idx = ((iz + dz) * R1 + (iy + dy)) * R1 + (ix + dx);
        acc += w * (double)ksdf_at(P.sdf, idx);
      }
  return acc;
}

// The cell's eight SDF values at grid coordinates, and the weights along each axis.
__device__ inline void ksdf_corners(KsdfArgs P, double cx, double cy, double cz, double (&g)[2][2][2], double& fx,
                                    double& fy, double& fz) {
  const int R = P.sdf_res;
  uint32_t ix, iy, iz;
  ksdf_cell(cx, R, ix, fx);
  ksdf_cell(cy, R, iy, fy);
  ksdf_cell(cz, R, iz, fz);
  const uint32_t R1 = R + 1, base = (iz * R1 + iy) * R1 + ix;
#pragma unroll
  for (int dz = 0; dz < 2; ++dz)
#pragma unroll
    for (int dy = 0; dy < 2; ++dy)
#pragma unroll
      for (int dx = 0; dx < 2; ++dx) g[dz][dy][dx] = (double)ksdf_at(P.sdf, base + (dz * R1 + dy) * R1 + dx);
}
// Trilinear lookup of the RGBA grid: FP64 grid coordinates, FP32 weights and sum.
__device__ inline float4 ksdf_rgba(KsdfArgs P, double cx, double cy, double cz) {
#pragma clang fp contract(fast)
  const int R = P.rgba_res;
  uint32_t ix, iy, iz;
  double dfx, dfy, dfz;
  ksdf_cell(cx, R, ix, dfx);
  ksdf_cell(cy, R, iy, dfy);
  ksdf_cell(cz, R, iz, dfz);
  const float fx = (float)dfx, fy = (float)dfy, fz = (float)dfz;
  const uint32_t R1 = R + 1;
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
  for (int dz = 0; dz < 2; ++dz)
#pragma unroll
    for (int dy = 0; dy < 2; ++dy)
#pragma unroll
      for (int dx = 0; dx < 2; ++dx) {
        const float w = ((dx ? fx : 1.f - fx) * (dy ? fy : 1.f - fy)) * (dz ? fz : 1.f - fz);
        const float4 g = ksdf_at4(P.rgba, ((iz + dz) * R1 + (iy + dy)) * R1 + (ix + dx));
        acc.x += w * g.x;
        acc.y += w * g.y;
        acc.z += w * g.z;
        acc.w += w * g.w;
      }
  return acc;
}

// ---------------------------------------------------------------------------
// occupancy grid
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_ksdf_occupancy(KsdfParams, uint32_t* __restrict__ occ, int64_t n_vox,
                                                        int64_t n_words) {
  KsdfArgs P = ksdf_args();
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  bool bit = false;
  if (i < n_vox) {
    const int64_t R = P.occ_res;
    const int64_t x = i % R, y = (i / R) % R, z = i / (R * R);
    const double cx = P.lo + ((double)x + 0.5) * P.h_occ;
    const double cy = P.lo + ((double)y + 0.5) * P.h_occ;
    const double cz = P.lo + ((double)z + 0.5) * P.h_occ;
    const double dc = ksdf_sdf(P, (cx - P.lo) * P.inv_sdf, (cy - P.lo) * P.inv_sdf, (cz - P.lo) * P.inv_sdf);
    for (int j = 0; j < P.k; ++j) {
      const double delta = fmax(fabs(dc + P.off[j]) - P.half_diag, 0.0);
      const double e = exp(-P.beta * fabs(delta));
      const double phi = P.beta * e / ((1.0 + e) * (1.0 + e));
      bit = bit || phi > P.occ_threshold;
    }
  }
  const uint64_t b = __ballot(bit);
  const int lane = threadIdx.x & 63;
  const int64_t word = i >> 5;
  if ((lane & 31) == 0 && word < n_words) occ[word] = (uint32_t)(lane ? b >> 32 : b);
}

// ---------------------------------------------------------------------------
// half-wavefront helpers: a wavefront renders two rays, one per 32-lane half
// (DPP row shifts within 16-lane rows, a row broadcast from row 0 to row 1 and
// from row 2 to row 3, whole-wave shifts by one lane with the half edges
// patched)
// ---------------------------------------------------------------------------
template <int CTRL, int ROW_MASK = 0xf>
__device__ inline float ksdf_dpp(float old, float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(old), __float_as_int(x), CTRL, ROW_MASK, 0xf, false));
}
// A permutation within rows: every lane has a source.
template <int CTRL>
__device__ inline float ksdf_dpp_full(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, true));
}
template <int CTRL, int ROW_MASK = 0xf>
__device__ inline int ksdf_dpp_i(int old, int x) {
  return __builtin_amdgcn_update_dpp(old, x, CTRL, ROW_MASK, 0xf, false);
}

// Inclusive prefix sum / product within each half.  The float ones are written
// as instructions that leave lanes without a source alone (s_nop: a DPP source must have been
// written two wait states before).
__device__ inline int ksdf_hscan_add_i(int x) {
  x += ksdf_dpp_i<0x111>(0, x);
  x += ksdf_dpp_i<0x112>(0, x);
  x += ksdf_dpp_i<0x114>(0, x);
  x += ksdf_dpp_i<0x118>(0, x);
  x += ksdf_dpp_i<0x142, 0xa>(0, x);
  return x;
}
__device__ inline float ksdf_hscan_add(float x) {
  asm("s_nop 1\n\tv_add_f32_dpp %0, %0, %0 row_shr:1 row_mask:0xf bank_mask:0xf\n\t"
      "s_nop 1\n\tv_add_f32_dpp %0, %0, %0 row_shr:2 row_mask:0xf bank_mask:0xf\n\t"
      "s_nop 1\n\tv_add_f32_dpp %0, %0, %0 row_shr:4 row_mask:0xf bank_mask:0xf\n\t"
      "s_nop 1\n\tv_add_f32_dpp %0, %0, %0 row_shr:8 row_mask:0xf bank_mask:0xf\n\t"
      "s_nop 1\n\tv_add_f32_dpp %0, %0, %0 row_bcast:15 row_mask:0xa bank_mask:0xf\n\ts_nop 1"
      : "+v"(x));
  return x;
}
__device__ inline float ksdf_hscan_mul(float x) {
  asm("s_nop 1\n\tv_mul_f32_dpp %0, %0, %0 row_shr:1 row_mask:0xf bank_mask:0xf\n\t"
      "s_nop 1\n\tv_mul_f32_dpp %0, %0, %0 row_shr:2 row_mask:0xf bank_mask:0xf\n\t"
      "s_nop 1\n\tv_mul_f32_dpp %0, %0, %0 row_shr:4 row_mask:0xf bank_mask:0xf\n\t"
      "s_nop 1\n\tv_mul_f32_dpp %0, %0, %0 row_shr:8 row_mask:0xf bank_mask:0xf\n\t"
      "s_nop 1\n\tv_mul_f32_dpp %0, %0, %0 row_bcast:15 row_mask:0xa bank_mask:0xf\n\ts_nop 1"
      : "+v"(x));
  return x;
}

// Value of lane l of this lane's half.
__device__ inline float ksdf_hlane(float x, int l, int h) {
  const float a = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), l));
  const float b = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 32 + l));
  return h ? b : a;
}
__device__ inline int ksdf_hlane_i(int x, int l, int h) {
  const int a = __builtin_amdgcn_readlane(x, l), b = __builtin_amdgcn_readlane(x, 32 + l);
  return h ? b : a;
}

// Sums of four values over this lane's half: x's in lanes 0..7, z's in 8..15,
// y's in 16..23, w's in 24..31.  A row swap adds two values' rows at once, a
// select two values' half rows, and the last three steps serve all four.
__device__ inline float ksdf_hsum4(float x, float y, float z, float w, int l) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
  const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(z), __float_as_uint(w), false, false);
  float p = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  float q = __uint_as_float(b[0]) + __uint_as_float(b[1]);
  p += ksdf_dpp_full<0x128>(p);       // row_ror:8
  q += ksdf_dpp_full<0x128>(q);
  float r = l & 8 ? q : p;
  r += ksdf_dpp_full<0x141>(r);       // row_half_mirror
  r += ksdf_dpp_full<0xb1>(r);        // quad_perm 1, 0, 3, 2
  r += ksdf_dpp_full<0x4e>(r);        // quad_perm 2, 3, 0, 1
  return r;
}

// Value of lane - 1 of the half (old at the half's first lane).
__device__ inline float ksdf_hbelow(float old, float x, int l) {
  const float y = ksdf_dpp<0x138>(old, x);
  return l == 0 ? old : y;
}

__device__ inline void ksdf_wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// LDS of one ray (half a wavefront).  A place p < 32 NSL of t and d is a sorted
// sample, place 32 NSL + q a new one of the current importance round, so that
// the merge reads either by one index.  The march's lists are done with before
// the first round.
template <int NSL>
struct KsdfLds {
  double t[32 * NSL + 64];  // sample parameters
  double d[32 * NSL + 64];  // their SDF values
  union {
    float cdf[128];         // importance CDF c_0..c_{N-1}, then infinite
    uint32_t odd[128];      // blend: ksdf_odd_surfaces of each interval, if any
    struct {
      uint64_t mask[32];    // march: occupied-step bits per lane
      int32_t pre[32];      // march: exclusive prefix of occupied steps per lane
    };
  };
  uint32_t place[4];        // bit p: a new sample goes to place p
};

// LDS of one wavefront's rays, each set up by one lane.
struct KsdfRays {
  double o[3][kKsdfBatch], v[3][kKsdfBatch];   // origin and unit direction
  double t_in[kKsdfBatch], D[kKsdfBatch];      // interval start and march step
  int32_t flags[kKsdfBatch];
};
enum { kKsdfReal = 1, kKsdfHit = 2, kKsdfFixed = 4 };

// A ray's position at parameter t, relative to the cube's corner, along one
// axis, with the steps of a plain evaluation: a ray may run along a cell face,
// and the cell decides about its normals.
__device__ inline double ksdf_from_lo(KsdfArgs P, const KsdfRays& S, int axis, int slot, double t) {
  return (S.o[axis][slot] + t * S.v[axis][slot]) - P.lo;
}
__device__ inline double ksdf_sample(KsdfArgs P, const KsdfRays& S, int slot, double t) {
  return ksdf_sdf(P, ksdf_from_lo(P, S, 0, slot, t) * P.inv_sdf, ksdf_from_lo(P, S, 1, slot, t) * P.inv_sdf,
                  ksdf_from_lo(P, S, 2, slot, t) * P.inv_sdf);
}

// |cos| of the angle between the ray and the gradient of the trilinear SDF
// inside the cell at grid coordinates c (along each axis, the corner
// differences of the cell's 4 grid lines weighted by the other two axes'
// weights); 0 where the gradient is.  Its scale does not matter.
__device__ inline double ksdf_abs_cos(KsdfArgs P, const KsdfRays& S, int slot, const double (&c)[3]) {
  double g[2][2][2], fx, fy, fz;
  ksdf_corners(P, c[0], c[1], c[2], g, fx, fy, fz);
  const double wx[2] = {1.0 - fx, fx}, wy[2] = {1.0 - fy, fy}, wz[2] = {1.0 - fz, fz};
  double gx = 0.0, gy = 0.0, gz = 0.0;
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      gx = __builtin_fma(wy[a] * wz[b], g[b][a][1] - g[b][a][0], gx);
      gy = __builtin_fma(wx[a] * wz[b], g[b][1][a] - g[b][0][a], gy);
      gz = __builtin_fma(wx[a] * wy[b], g[1][b][a] - g[0][b][a], gz);
    }
  const double n2 = (gx * gx + gy * gy) + gz * gz;
  const double gv = (gx * S.v[0][slot] + gy * S.v[1][slot]) + gz * S.v[2][slot];
  return n2 > 0.0 ? fabs(gv) / sqrt(n2) : 0.0;
}

// Camera ray of pixel `ray`, its interval in the cube and its march step.
__device__ inline void ksdf_setup(const vs_view* __restrict__ views, int n_views, int64_t total, KsdfArgs P,
                                  int64_t ray, KsdfRays& S, int slot) {
  const bool real = ray < total;
  const int64_t rr = real ? ray : total - 1;
  int lo_v = 0, hi_v = n_views - 1;
  while (lo_v < hi_v) {
    const int mid = (lo_v + hi_v + 1) / 2;
    if (views[mid].pix_offset <= rr) lo_v = mid; else hi_v = mid - 1;
  }
  const vs_camera& C = views[lo_v].cam;
  const int64_t pix = rr - views[lo_v].pix_offset;
  const int64_t pi = pix % C.width, pj = pix / C.width;
  double o[3], v[3];
#pragma unroll
  for (int q = 0; q < 3; ++q) o[q] = -((C.R[q] * C.t[0] + C.R[3 + q] * C.t[1]) + C.R[6 + q] * C.t[2]);
  const double xc = (((double)pi + 0.5) - C.cx) / C.fx, yc = (((double)pj + 0.5) - C.cy) / C.fy;
#pragma unroll
  for (int q = 0; q < 3; ++q) v[q] = (C.R[q] * xc + C.R[3 + q] * yc) + C.R[6 + q];
  const double vn = sqrt((v[0] * v[0] + v[1] * v[1]) + v[2] * v[2]);
#pragma unroll
  for (int q = 0; q < 3; ++q) v[q] = v[q] / vn;

  // slab interval in the cube, t >= 0
  double t_in = 0.0, t_out = INFINITY;
  bool hit = real;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    if (v[a] != 0.0) {
      const double t1 = (P.lo - o[a]) / v[a], t2 = (P.hi - o[a]) / v[a];
      t_in = fmax(t_in, fmin(t1, t2));
      t_out = fmin(t_out, fmax(t1, t2));
    } else {
      hit = hit && o[a] >= P.lo && o[a] <= P.hi;
    }
  }
  hit = hit && t_out > t_in;
  // The fixed-point march allows for FP64 rounding of less than one unit: 2^-49 of the largest term, the
  // origin's voxel coordinate (false for NaN).
  const double far = (double)((uint64_t)1 << (48 - P.occ_frac));
  bool fixed = (v[0] * v[0] + v[1] * v[1]) + v[2] * v[2] < 2.0;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    fixed = fixed && fabs((o[a] - P.lo) * P.inv_occ) < far;
    S.o[a][slot] = o[a];
    S.v[a][slot] = v[a];
  }
  S.t_in[slot] = t_in;
  S.D[slot] = hit ? (t_out - t_in) / (double)P.steps : 0.0;
  S.flags[slot] = (real ? kKsdfReal : 0) | (hit ? kKsdfHit : 0) | (fixed ? kKsdfFixed : 0);
}

// Occupancy bits of the march steps of two rays, one per half: lane l of a half
// gets those of steps 64 l .. 64 l + 63 of its ray, the voxel of step s's
// midpoint being floor(A + tm B), tm = t_in + (s + 1/2) D, in FP64, clamped to
// the grid.  Without `hit` a lane's steps count as empty.
//
// Most rays of a view cross the cube without meeting an occupied voxel and cost
// nothing else, so this is the larger part of the render.  Lane l looks at
// steps l, l + 32, ..: the lanes of a half read neighbouring voxels, a few
// cache lines at a time (runs of consecutive steps per lane read 32), and a
// ballot is a word of the bits.  The steps are taken in fixed point, one 32-bit
// addition per axis: with f fraction bits the first coordinate and the
// increment are each off by at most half a unit, and the FP64 evaluation by
// less than one (kKsdfFixed), so the n-th of a lane's steps lies within
// n / 2 + 2 units of its sum.  Where no sum comes that close to a voxel face,
// every voxel is the FP64 evaluation's; otherwise (1 wavefront in 45 at 256^3
// voxels and 1,024 steps) the steps are taken again in FP64.  The first and
// last step of a lane are checked to lie in the grid, and so do those between
// them.  8 x 512^2 rays, 1,024 steps, set-up and march alone: 2.9 -> 2.1 ms.
__device__ inline uint64_t ksdf_march(KsdfArgs P, const uint32_t* __restrict__ occ, const KsdfRays& S, int slot, bool hit,
                                      bool fixed, int l, int lane) {
  const int Ro = P.occ_res, n = P.steps / 64;
  const double t_in = S.t_in[slot], D = S.D[slot];
  double A[3], B[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    A[a] = (S.o[a][slot] - P.lo) * P.inv_occ;
    B[a] = S.v[a][slot] * P.inv_occ;
  }
  uint32_t bits[2] = {0, 0};
  // the ballots of steps 64 i + l and 64 i + 32 + l go to lane i of their half
  const auto keep = [&](int i, uint64_t w0, uint64_t w1) {
    asm("s_nop 1\n\ts_mov_b32 m0, %6\n\ts_nop 1\n\tv_writelane_b32 %0, %2, m0\n\tv_writelane_b32 %1, %4, m0\n\t"
        "s_mov_b32 m0, %7\n\ts_nop 1\n\tv_writelane_b32 %0, %3, m0\n\tv_writelane_b32 %1, %5, m0"
        : "+v"(bits[0]), "+v"(bits[1])
        : "s"((uint32_t)w0), "s"((uint32_t)(w0 >> 32)), "s"((uint32_t)w1), "s"((uint32_t)(w1 >> 32)), "s"(i), "s"(32 + i)
        : "m0");
  };
  const auto word_of = [&](uint32_t idx) { return *(const uint32_t*)((const char*)occ + ((idx >> 5) << 2)); };
  const auto test = [&](uint32_t word, uint32_t idx) { return __ballot((int32_t)(word << (~idx & 31)) < 0); };
  bool ok = fixed || !hit;
  if (__all(ok)) {
    const int f = P.occ_frac;
    const uint32_t frac = ((uint32_t)1 << f) - 1, e = (uint32_t)n + 2, end = (uint32_t)Ro << f;
    const double F = (double)((uint32_t)1 << f), tm = t_in + ((double)l + 0.5) * D;
    uint32_t X[3], dX[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      X[a] = (uint32_t)fmin(fmax(rint((A[a] + tm * B[a]) * F), 0.0), 4294967295.0) + e;
      dX[a] = (uint32_t)(int32_t)rint(32.0 * D * B[a] * F);
      ok = ok && X[a] < end && X[a] + (uint32_t)(2 * n - 1) * dX[a] < end;
    }
    uint32_t near = frac;
    if (!(hit && ok)) {     // these lanes stay at the grid's first voxel
#pragma unroll
      for (int a = 0; a < 3; ++a) X[a] = dX[a] = 0;
    }
    const auto walk = [&](auto groups, int i) {
      constexpr int G = 2 * decltype(groups)::value;
      uint32_t idx[G], word[G];
#pragma unroll
      for (int q = 0; q < G; ++q) {
        near = min(near, min(X[0] & frac, min(X[1] & frac, X[2] & frac)));
        idx[q] = mad24(mad24(X[2] >> f, Ro, X[1] >> f), Ro, X[0] >> f);
        word[q] = word_of(idx[q]);
#pragma unroll
        for (int a = 0; a < 3; ++a) X[a] += dX[a];
      }
#pragma unroll
      for (int q = 0; q < G; q += 2) keep(i + q / 2, test(word[q], idx[q]), test(word[q + 1], idx[q + 1]));
    };
    int i = 0;
    for (; i + 4 <= n; i += 4) walk(std::integral_constant<int, 4>{}, i);
    for (; i < n; ++i) walk(std::integral_constant<int, 1>{}, i);
    ok = !hit || (ok && near > 2 * e);
  }
  if (!__all(ok)) {
    for (int i = 0; i < n; ++i) {
      uint64_t w[2];
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const double tm = t_in + ((double)(64 * i + 32 * q + l) + 0.5) * D;
        uint32_t vox[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          // floor, then clamp to [0, Ro - 1] (the coordinate stays within a rounding of [0, Ro])
          vox[a] = (uint32_t)min(max((int)floor(A[a] + tm * B[a]), 0), Ro - 1);
        }
        const uint32_t idx = mad24(mad24(vox[2], Ro, vox[1]), Ro, vox[0]);
        w[q] = test(word_of(idx), idx);
      }
      keep(i, w[0], w[1]);
    }
  }
  return hit ? (uint64_t)bits[1] << 32 | bits[0] : 0;
}

// Place of the r-th (from 0) set bit of a mask that has it.
__device__ inline int ksdf_select(uint64_t mask, int r) {
  uint32_t w = (uint32_t)mask;
  int at = 0, c = __popc(w);
  if (r >= c) {
    r -= c;
    at = 32;
    w = (uint32_t)(mask >> 32);
  }
#pragma unroll
  for (int s = 16; s > 0; s >>= 1) {
    c = __popc(w & ((1u << s) - 1));
    const bool up = r >= c;
    r -= up ? c : 0;
    w >>= up ? s : 0;
    at += up ? s : 0;
  }
  return at;
}

// exp(x), the part of x that a float leaves out included: its rounding alone
// would cost 60 units in the last place at x = 60.
__device__ inline float ksdf_exp(double x) {
  const float xh = (float)x;
  const float e = expf(xh);
  return e > 0.f && e < INFINITY ? e + e * (float)(x - (double)xh) : e;
}

// What the surfaces share of the opacity of the interval from a sample with SDF
// value d to one with dn: 1 - Phi_{i+1} / Phi_i with Phi = 1 / (1 + exp(-beta x))
// is (1 - r) / (1 + g_j), r = exp(-beta (d - dn)), g_j = exp(beta (dn + o_j)),
// and not below 0.  q is 1 - r held to that (0 next to a NaN), G is g without o_j.
// Far inside all surfaces g is 0, far outside infinite, with opacity 0.
__device__ inline void ksdf_interval(double beta, double d, double dn, float& q, float& G) {
  q = fmaxf(-expm1f(-(float)(beta * (d - dn))), 0.f);
  G = q > 0.f ? ksdf_exp(beta * dn) : 1.f;
}

// Surfaces whose opacity over the interval that form does not give: bit j, it is 0 for surface j, because Phi_i is
// 0 in FP64 (exp(-beta x) overflows); bit 16 + j, it is 1, because only Phi_{i+1} is, or because d is a NaN and
// Phi_{i+1} 0 in FP32, formed as in the importance weights (ksdf_cdf).
constexpr double kKsdfDeep = 709.782712893384;   // log of the largest double
static_assert(VS_KSDF_MAX_SURFACES <= 16, "bits of a word");
__device__ inline uint32_t ksdf_odd_surfaces(KsdfArgs P, double d, double dn) {
  uint32_t bits = 0;
  for (int j = 0; j < P.k; ++j) {
    const double x = -P.beta * (d + P.off[j]), xn = -P.beta * (dn + P.off[j]);
    const float en = P.factor ? expf(-(float)(P.beta * dn)) * P.cinv[1][j] : expf((float)xn);
    if (x > kKsdfDeep) bits |= 1u << j;
    else if (xn > kKsdfDeep || (isnan(d) && isinf(en))) bits |= 0x10000u << j;
  }
  return bits;
}

// NeuS interval weights of one surface, w_i = a_i prod_{l<i} (1 - a_l), for lane
// l's samples [NS l, NS l + NS) of this half's ray.  g_j is G cexp_j, or an
// exponential of its own where the offsets are too large for the factor to
// stay a normal float.
template <int NS>
__device__ inline void ksdf_weights(KsdfArgs P, int j, const double (&dn)[NS],
                                    const float (&q)[NS], const float (&G)[NS], const uint32_t* odd,
                                    float (&w)[NS], int l) {
#pragma clang fp contract(fast)
  float a[NS], pass = 1.f;
  const float c = P.cexp[j];
#pragma unroll
  for (int sl = 0; sl < NS; ++sl) a[sl] = 1.f + G[sl] * c;
  if (!P.factor) {
#pragma unroll
    for (int sl = 0; sl < NS; ++sl) a[sl] = q[sl] > 0.f ? 1.f + ksdf_exp(P.beta * (dn[sl] + P.off[j])) : 1.f;
  }
#pragma unroll
  for (int sl = 0; sl < NS; ++sl) a[sl] = q[sl] * __builtin_amdgcn_rcpf(a[sl]);
  if (odd) {   // uniform
#pragma unroll
    for (int sl = 0; sl < NS; ++sl) {
      const uint32_t bits = odd[NS * l + sl] >> j;
      a[sl] = bits & 1u ? 0.f : bits & 0x10000u ? 1.f : a[sl];
    }
  }
#pragma unroll
  for (int sl = 0; sl < NS; ++sl) pass *= 1.f - a[sl];
  float T = ksdf_hbelow(1.f, ksdf_hscan_mul(pass), l);
#pragma unroll
  for (int sl = 0; sl < NS; ++sl) {
    w[sl] = T * a[sl];
    T *= 1.f - a[sl];
  }
}

// Importance CDF of one round over Ncur samples: the surfaces' weights summed,
// plus the floor.  Sample 32 sl + l lies in lane l's slot sl.  The new samples'
// positions follow from the CDF's last bits, and a normal jumps where a sample
// crosses a cell face: so the weights keep this form, e_j = E cexp_j at both
// ends of an interval, opacity (e_{i+1} - e_i) / (1 + e_{i+1}), one scan per 32
// samples, none of it contracted; 0 where Phi_i = 0 (e_i infinite), 1 where only
// Phi_{i+1} = 0.  Samples past the last repeat it: intervals of weight 0.
template <int NS, int NSL>
__device__ inline void ksdf_cdf(KsdfArgs P, KsdfLds<NSL>& L, int round, double beta_r, int Ncur, int l, int h) {
  float E[NS], En[NS], W[NS];
  double d[NS], dn[NS];
#pragma unroll
  for (int sl = 0; sl < NS; ++sl) {
    const int i = 32 * sl + l;
    d[sl] = L.d[min(i, Ncur - 1)];
    dn[sl] = L.d[min(i + 1, Ncur - 1)];
    E[sl] = expf(-(float)(beta_r * d[sl]));
    En[sl] = expf(-(float)(beta_r * dn[sl]));
    W[sl] = 0.f;
  }
  for (int j = 0; j < P.k; ++j) {
    const float c = P.cinv[round][j];
    float carry = 1.f;
#pragma unroll
    for (int sl = 0; sl < NS; ++sl) {
      float e = E[sl] * c, en = En[sl] * c;
      if (!P.factor) {
        e = expf(-(float)(beta_r * (d[sl] + P.off[j])));
        en = expf(-(float)(beta_r * (dn[sl] + P.off[j])));
      }
      float a = fmaxf((en - e) * __builtin_amdgcn_rcpf(1.f + en), 0.f);
      a = en == INFINITY ? 1.f : a;
      a = e == INFINITY ? 0.f : a;
      const float t = ksdf_hscan_mul(1.f - a) * carry;
      W[sl] += ksdf_hbelow(carry, t, l) * a;
      if (sl + 1 < NS) carry = ksdf_hlane(t, 31, h);
    }
  }
  float sum = 0.f;
#pragma unroll
  for (int sl = 0; sl < NS; ++sl) {
    W[sl] = 32 * sl + l < Ncur - 1 ? W[sl] + P.pdf_floor : 0.f;
    sum += W[sl];
  }
  const float rS = 1.f / ksdf_hlane(ksdf_hscan_add(sum), 31, h);
  float carry = 0.f;
#pragma unroll
  for (int sl = 0; sl < 4; ++sl) {
    const int i = 32 * sl + l;
    float c = INFINITY;                    // places past the last sample's, which the search may read
    if (sl < NS) {
      const float part = ksdf_hscan_add(W[sl < NS ? sl : 0] * rS) + carry;
      carry = ksdf_hlane(part, 31, h);
      if (i < Ncur - 1) c = part;
    }
    if (i < 127) L.cdf[i + 1] = c;
  }
  if (l == 0) L.cdf[0] = 0.f;
}

// Appearance of the ray's samples, per-surface quadrature and fixed-order
// blend; lanes 0, 16, 8, 24 hold r, g, b and alpha.
template <int NS, int NSL>
__device__ inline float ksdf_blend(KsdfArgs P, KsdfLds<NSL>& L, const KsdfRays& S, int slot, int N, int l,
                                   int h, int comp, int64_t ray, int64_t total, bool live, float* __restrict__ layers) {
  bool odd = false;
#pragma unroll
  for (int sl = 0; sl < NS; ++sl) odd = odd || !(L.d[min(32 * sl + l, N - 1)] > P.deep);   // true for NaN
  odd = __any(odd);
  if (odd) {
    for (int i = l; i < 32 * NS; i += 32) L.odd[i] = ksdf_odd_surfaces(ksdf_args(), L.d[min(i, N - 1)], L.d[min(i + 1, N - 1)]);
    ksdf_wave_sync();
  }
  float4 app[NS];
  float q[NS], G[NS], aw[NS];
  double d[NS];
  // at each interval start: colour, and opacity attenuated by the view direction
#pragma unroll
  for (int sl = 0; sl < NS; ++sl) {
    const int i = NS * l + sl;
    app[sl] = make_float4(0.f, 0.f, 0.f, 0.f);
    aw[sl] = 0.f;
    d[sl] = L.d[min(i + 1, N - 1)];
    ksdf_interval(P.beta, L.d[min(i, N - 1)], d[sl], q[sl], G[sl]);
    if (i < N - 1) {
      const double t = L.t[i];
      const double x = ksdf_from_lo(P, S, 0, slot, t), y = ksdf_from_lo(P, S, 1, slot, t), z = ksdf_from_lo(P, S, 2, slot, t);
      app[sl] = ksdf_rgba(ksdf_args(), x * P.inv_rgba, y * P.inv_rgba, z * P.inv_rgba);
      const double c[3] = {x * P.inv_sdf, y * P.inv_sdf, z * P.inv_sdf};
      const double vdn = ksdf_abs_cos(ksdf_args(), S, slot, c);
      aw[sl] = (2.f / (1.f + expf(-10.f * (float)vdn)) - 1.f) * app[sl].w;
    }
  }
  float acc = 0.f, T = 1.f;
  for (int j = 0; j < P.k; ++j) {
#pragma clang fp contract(fast)
    float w[NS];
    ksdf_weights<NS>(P, j, d, q, G, odd ? L.odd : nullptr, w, l);
    float pr = 0.f, pg = 0.f, pb = 0.f, pa = 0.f;
#pragma unroll
    for (int sl = 0; sl < NS; ++sl) {
      pr += w[sl] * app[sl].x;
      pg += w[sl] * app[sl].y;
      pb += w[sl] * app[sl].z;
      pa += w[sl] * aw[sl];
    }
    const float c = ksdf_hsum4(pr, pg, pb, pa, l);
    const float ca = ksdf_hlane(c, 24, h);
    acc += (T * ca) * c;
    T *= 1.f - ca;
    if (layers && comp >= 0) layers[((int64_t)j * total + ray) * 4 + comp] = live ? c : 0.f;
  }
  return l == 24 ? 1.f - T : acc;
}

// Block b -> a contiguous run of rays per XCD (blocks are dealt round-robin to the 8 XCDs).
__device__ inline int64_t ksdf_block() {
  const int64_t chunk = (int64_t)gridDim.x / 8;
  return ((int64_t)blockIdx.x % 8) * chunk + (int64_t)blockIdx.x / 8;
}

// per_wave rays per wavefront, set up by one lane each and rendered two at a
// time, 32 lanes each: the 96 samples of the paper's 64 + 32 fill three slots
// of 32 exactly (NSL = slots per lane, from the sample count).
//
// Bound by VALU issue: 8 x 512^2 rays, k = 7, 64 + 32 samples, 1,024 steps took
// 8.6 ms at 6.1e9 wavefront instructions and take 5.9 ms at 3.6e9, nine tenths
// of the cycles the SIMDs have.  What went: each of a wavefront's 64 lanes setting
// up its own ray (one lane does now), the FP64 march, exchanges between lanes
// for the next sample's terms, in the blend one transmittance scan per 32
// samples and surface (one per 96 now), four half-wave sums per surface (one
// now) and opacities from each surface's own exponentials, rank searches in the
// merge.  A block is one wavefront, for its rays may all miss while another's
// all hit (four a block: 0.6 ms more); registers allow 16 a CU.  Samples lie in
// LDS between the phases and parameters are asked for anew, so that nothing
// spills.
template <int NSL>
__global__ void __launch_bounds__(64 * kKsdfWaves, 4) k_ksdf_render(KsdfParams, const vs_view* __restrict__ views,
                                                     int n_views, int64_t total, int per_wave,
                                                     const uint32_t* __restrict__ occ,
                                                     float* __restrict__ out, float* __restrict__ layers,
                                                     double* __restrict__ samples) {
  __shared__ KsdfLds<NSL> lds_all[2 * kKsdfWaves];
  __shared__ KsdfRays rays_all[kKsdfWaves];
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), first_lane = threadIdx.x & 63;
  KsdfRays& S = rays_all[wv];
  const int64_t first = (ksdf_block() * kKsdfWaves + wv) * per_wave;
  if (first >= total) return;
  if (first_lane < per_wave) ksdf_setup(views, n_views, total, ksdf_args(), first + first_lane, S, first_lane);
  ksdf_wave_sync();

  for (int r0 = 0; r0 < per_wave && first + r0 < total; r0 += 2) {
    KsdfArgs P = ksdf_args();
    int lane = first_lane;
    asm volatile("" : "+v"(lane));            // likewise: nothing derived from the lane is held across the loop
    const int h = lane >> 5, l = lane & 31;
    const int comp = l & 7 ? -1 : l == 0 ? 0 : l == 16 ? 1 : l == 8 ? 2 : 3;   // the channel this lane holds at the end
    KsdfLds<NSL>& L = lds_all[2 * wv + h];
    const int N = P.n + P.m, m2 = P.m / 2;
    const int slot = r0 + h;
    const int64_t ray = first + slot;
    const int flags = S.flags[slot];
    const bool real = flags & kKsdfReal;

    // march: lane l of the half gets the bits of steps [64 l, 64 l + 64)
    const uint64_t mask =
        ksdf_march(ksdf_args(), occ, S, slot, flags & kKsdfHit, flags & kKsdfFixed, l, lane);
    const int cnt = __popcll(mask);
    const int incl = ksdf_hscan_add_i(cnt);
    const int M = ksdf_hlane_i(incl, 31, h);
    const bool live = M > 0;
    if (__builtin_amdgcn_readlane((int)live, 0) == 0 && __builtin_amdgcn_readlane((int)live, 32) == 0) {
      if (real && comp >= 0) {
        out[ray * 4 + comp] = 0.f;
        if (layers)
          for (int j = 0; j < P.k; ++j) layers[((int64_t)j * total + ray) * 4 + comp] = 0.f;
      }
      if (real && samples)
        for (int i = l; i < N; i += 32) samples[ray * N + i] = -1.0;
      continue;
    }
    L.pre[l] = incl - cnt;
    L.mask[l] = mask;
    if (l < 4) L.place[l] = 0;
    ksdf_wave_sync();

    // uniform samples in occupied length (a ray without any: parameter 0 and a far-outside SDF, no weight)
    for (int i = l; i < P.n; i += 32) {
      double t = 0.0, d = 1e30;
      if (live) {
        const double rho = (((double)i + 0.5) * (double)M) / (double)P.n;
        const double qf = floor(rho);
        const int qi = (int)qf;
        int a = 0;                          // largest lane with pre <= qi
#pragma unroll
        for (int st = 16; st > 0; st >>= 1) a += L.pre[a + st] <= qi ? st : 0;
        const int s = 64 * a + ksdf_select(L.mask[a], qi - L.pre[a]);
        t = S.t_in[slot] + ((double)s + (rho - qf)) * S.D[slot];
        d = ksdf_sample(ksdf_args(), S, slot, t);
      }
      L.t[i] = t;
      L.d[i] = d;
    }
    ksdf_wave_sync();

    // two importance rounds
    int Ncur = P.n;
#pragma unroll 1
    for (int round = 0; round < 2 && m2 > 0; ++round) {
      const double beta_r = round == 0 ? P.beta / 2.0 : P.beta;
      if (Ncur <= 32) ksdf_cdf<1, NSL>(ksdf_args(), L, round, beta_r, Ncur, l, h);
      else if (NSL == 2 || Ncur <= 64) ksdf_cdf<2, NSL>(ksdf_args(), L, round, beta_r, Ncur, l, h);
      else if (NSL == 3 || Ncur <= 96) ksdf_cdf<(NSL > 2 ? 3 : 2), NSL>(ksdf_args(), L, round, beta_r, Ncur, l, h);
      else ksdf_cdf<NSL, NSL>(ksdf_args(), L, round, beta_r, Ncur, l, h);
      ksdf_wave_sync();
      for (int qn = l; qn < m2; qn += 32) {
        const double u = ((double)qn + 0.5) / (double)m2;
        float uf = (float)u;                  // the largest float that is not above u
        if ((double)uf > u) uf = __uint_as_float(__float_as_uint(uf) - 1);
        int a = 0;                            // largest i with cdf[i] <= u
#pragma unroll
        for (int st = 64; st > 0; st >>= 1) a += L.cdf[a + st] <= uf ? st : 0;
        a = min(a, Ncur - 2);
        const double ca = (double)L.cdf[a], cb = (double)L.cdf[a + 1];
        const double fr = cb > ca ? (u - ca) / (cb - ca) : 0.0;
        const double t = L.t[a] + fr * (L.t[a + 1] - L.t[a]);
        int below = a + 1;                    // existing samples <= t, which go first
        while (below < Ncur && L.t[below] <= t) ++below;
        const int p = below + qn;
        atomicOr(&L.place[p >> 5], 1u << (p & 31));
        L.t[32 * NSL + qn] = t;
        L.d[32 * NSL + qn] = live ? ksdf_sample(ksdf_args(), S, slot, t) : 1e30;
      }
      ksdf_wave_sync();
      // the merged order: place p is the next new sample if its bit is set, else the next existing one
      Ncur += m2;
      double tm[NSL], dm[NSL];
      int before = 0;
#pragma unroll
      for (int sl = 0; sl < NSL; ++sl) {
        const uint32_t w = L.place[sl];
        const int p = 32 * sl + l, nb = before + __popc(w & ((1u << l) - 1));
        const int from = (w >> l) & 1 ? 32 * NSL + nb : p - nb;
        tm[sl] = L.t[from];
        dm[sl] = L.d[from];
        before += __popc(w);
      }
      ksdf_wave_sync();
#pragma unroll
      for (int sl = 0; sl < NSL; ++sl) {
        const int p = 32 * sl + l;
        if (p < Ncur) {
          L.t[p] = tm[sl];
          L.d[p] = dm[sl];
        }
      }
      if (l < 4) L.place[l] = 0;
      ksdf_wave_sync();
    }

    float* lay = real ? layers : nullptr;
    float c;
    if (NSL == 2) {
      c = N <= 32 ? ksdf_blend<1, NSL>(ksdf_args(), L, S, slot, N, l, h, comp, ray, total, live, lay)
                  : ksdf_blend<2, NSL>(ksdf_args(), L, S, slot, N, l, h, comp, ray, total, live, lay);
    } else {
      c = ksdf_blend<NSL, NSL>(ksdf_args(), L, S, slot, N, l, h, comp, ray, total, live, lay);
    }
    if (real && comp >= 0) out[ray * 4 + comp] = live ? c : 0.f;
    if (real && samples)
      for (int i = l; i < N; i += 32) samples[ray * N + i] = live ? L.t[i] : -1.0;
    ksdf_wave_sync();
  }
}

}  // namespace vs
