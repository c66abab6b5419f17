// Neural textures (Sec. 4.3 "Texturing Meshes"): a 2-D multiresolution hash
// grid and a small MLP, grounded to the texture resolution by evaluating them
// at the texel centres only (Fig. 5), so that the renderer samples an ordinary
// RGBA texture.  Per texel (i, j) at u = (i + 1/2)/W, v = (j + 1/2)/H:
//   level l: x = u N_l, y = v N_l (FP64, as the texel coordinates elsewhere),
//            bilinear over the 4 surrounding vertices of 2 features each;
//            vertex index y (N_l + 1) + x when (N_l + 1)^2 <= T, else
//            (x XOR y * 2654435761) mod 2^32 masked to T - 1;
//   e = concat_l features (2L), z1 = W1 e + b1, h1 = relu(z1) (64),
//   z2 = W2 h1 + b2, h2 = relu(z2) (64), o = W3 h2 + b3 (4), texel = sigmoid(o).
// Parameters per layer, flat f32:
//   tables [L][T][2] | W1 [64][2L] | b1 [64] | W2 [64][64] | b2 [64] | W3 [4][64] | b3 [4].
// All products run on the matrix cores (see k_ngp_bake and k_ngp_backward);
// the backward evaluates the layers again from the staged encodings, and a
// second kernel scatters dL/de into the tables (k_ngp_scatter).
#pragma once

#include "vs_common.h"

namespace vs {

constexpr int kNgpHidden = 64;
constexpr int kNgpOut = 4;
constexpr int kNgpMaxLevels = 16;
constexpr uint32_t kNgpPrimeY = 2654435761u;
constexpr int kNgpTile = 16;   // texels per tile side; a block of 256 threads covers one tile
constexpr int kNgpSlots = 576; // vertices of a level's LDS window in the table scatter (24 x 24)

struct NgpShape {
  int32_t levels, log2_table;
  int32_t res[kNgpMaxLevels];
  int32_t dense[kNgpMaxLevels];
  int64_t o_w1, o_b1, o_w2, o_b2, o_w3, o_b3, total;   // o_tab = 0
};

// Per layer buffers and sizes; block_off is the prefix sum of 256-texel tiles
// over layers, and row block_off * 256 + thread is a texel's staging row.
struct NgpTable {
  const float* params[kMaxLayers];
  float* tex[kMaxLayers];
  const float* gtex[kMaxLayers];
  float* gparams[kMaxLayers];
  int32_t w[kMaxLayers], h[kMaxLayers];
  int64_t block_off[kMaxLayers + 1];
  int32_t k;
};

// Staging for the backward, feature-major [feature][R] over R = 256 * tiles
// rows (every access of a wavefront is then consecutive).  Rows of texels
// outside the texture hold zeros.
struct NgpStage {
  float* a1;   // [2L][R] encodings e, from the bake
  float* de;   // [2L][R] dL/de, between the backward's two kernels
  int64_t R;
};

__device__ inline uint32_t ngp_index(uint32_t x, uint32_t y, int32_t N, int32_t dense, uint32_t mask) {
  return dense ? y * (uint32_t)(N + 1) + x : ((x ^ (y * kNgpPrimeY)) & mask);
}

// Encoding of one texel centre.
template <int LMAX>
__device__ inline void ngp_encode(const float* __restrict__ tables, const NgpShape& S, double u, double v, float (&e)[2 * LMAX]) {
  const uint32_t T = 1u << S.log2_table, mask = T - 1u;
#pragma unroll
  for (int lv = 0; lv < LMAX; ++lv) {
    e[2 * lv] = 0.f;
    e[2 * lv + 1] = 0.f;
    if (lv >= S.levels) continue;
    const int32_t N = S.res[lv];
    const double x = u * (double)N, y = v * (double)N;
    const double x0 = floor(x), y0 = floor(y);
    const float fx = (float)(x - x0), fy = (float)(y - y0);
    const uint32_t xi = (uint32_t)x0, yi = (uint32_t)y0;
    const float2* tab = reinterpret_cast<const float2*>(tables) + (int64_t)lv * T;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const uint32_t dx = c & 1, dy = c >> 1;
      const uint32_t q = ngp_index(xi + dx, yi + dy, N, S.dense[lv], mask);
      const float w = (dx ? fx : 1.0f - fx) * (dy ? fy : 1.0f - fy);
      const float2 f = tab[q];
      e[2 * lv] += w * f.x;
      e[2 * lv + 1] += w * f.y;
    }
  }
}

// Orders this wavefront's LDS accesses (a wavefront's LDS instructions execute in order).
__device__ inline void ngp_wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ inline float ngp_sigmoid(float x) { return 1.0f / (1.0f + expf(-x)); }

// texture = sigmoid(MLP(encoding)) at every texel centre of every layer; with
// STAGE the encodings e are kept for the backward, which evaluates the layers
// again.  Seven 1024^2 textures of 8 levels: 1.08 ms, of which the matrix cores
// need 0.57 (459k texel rows of 96 MFMAs at 32 cycles) and the encodings alone
// take 0.24; 2.03 ms with h1 and h2 staged as well (0.5 KB per texel) and the
// weights laid out by every tile's block.  One, two or four texel rows per weight
// fragment: 1.11, 1.11 and 1.08 ms; three blocks a CU spill (1.06 - 1.36 ms).
//
// The three layers are dense products over the block's 256 texels and run on
// the matrix cores (v_mfma_f32_16x16x4_f32, FP32 in and out) in transposed
// form, Z^T = W X^T + b: the hidden units are the 16-row M tiles, 16 texels
// (one texel row of the tile) the N tile.  An MFMA leaves lane l with
// D[4 (l / 16) + r][l % 16], r = 0..3, and takes its B operand as
// B[k = l / 16][n = l % 16]; issuing the r-th of four MFMAs with the r-th
// register of the previous layer's output therefore feeds that output straight
// back as the next B operand, with the K index permuted to 4 (l / 16) + r; the
// weights (A operands) are laid out in LDS in that permuted order, one 64-lane
// fragment per MFMA.  Encodings go through LDS to become layer 1's B operand.
// Blocks of the bake and the backward: layer l's tiles are shared by blocks off[l] .. off[l + 1] - 1, each of
// which takes a contiguous run of them, so that a block lays out its layer's weights once.
struct NgpBlocks {
  int32_t off[kMaxLayers + 1];
};

typedef float ngp_f4 __attribute__((ext_vector_type(4)));

template <int LMAX, bool STAGE>
__global__ void __launch_bounds__(256, 2) k_ngp_bake(NgpTable T, NgpShape S, NgpStage G, NgpBlocks Q) {
  constexpr int KIN = 2 * LMAX, KS1 = KIN / 4, EST = KIN + 1;
  constexpr int NT = 4;                   // a wavefront's texel rows (N tiles), taken together
  __shared__ float w1f[4 * KS1 * 64];     // [mt][ks][lane]: W1[16 mt + lane % 16][4 ks + lane / 16]
  __shared__ float w2f[64 * 64];          // [mt][it][r][lane]: W2[16 mt + lane % 16][16 it + 4 (lane / 16) + r]
  __shared__ float w3f[16 * 64];          // [it][r][lane]: W3[lane % 16][16 it + 4 (lane / 16) + r] (rows >= 4: 0)
  __shared__ float es[4][64 * EST];       // per wave: the encodings of its 64 texels
  const int tid = threadIdx.x, wv = tid >> 6, lane = tid & 63;
  int l = 0;
  while (l + 1 < T.k && Q.off[l + 1] <= (int)blockIdx.x) ++l;
  const int part = (int)blockIdx.x - Q.off[l], parts = Q.off[l + 1] - Q.off[l];
  const int64_t tiles = T.block_off[l + 1] - T.block_off[l];
  const float* P = T.params[l];
  const int nin = 2 * S.levels;
  for (int f = tid; f < 4 * KS1 * 64; f += 256) {
    const int ln = f & 63, fr = f >> 6, mt = fr / KS1, ks = fr - mt * KS1;
    const int m = 16 * mt + (ln & 15), kk = 4 * ks + (ln >> 4);
    w1f[f] = kk < nin ? P[S.o_w1 + m * nin + kk] : 0.f;
  }
  for (int f = tid; f < 64 * 64; f += 256) {
    const int ln = f & 63, fr = f >> 6, mt = fr >> 4, it = (fr >> 2) & 3, r = fr & 3;
    w2f[f] = P[S.o_w2 + (16 * mt + (ln & 15)) * kNgpHidden + 16 * it + 4 * (ln >> 4) + r];
  }
  for (int f = tid; f < 16 * 64; f += 256) {
    const int ln = f & 63, fr = f >> 6, it = fr >> 2, r = fr & 3, m = ln & 15;
    w3f[f] = m < kNgpOut ? P[S.o_w3 + m * kNgpHidden + 16 * it + 4 * (ln >> 4) + r] : 0.f;
  }
  __syncthreads();
  const int g = lane >> 4, n = lane & 15;
  ngp_f4 b1[4], b2[4], b3;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
      b1[mt][r] = P[S.o_b1 + 16 * mt + 4 * g + r];
      b2[mt][r] = P[S.o_b2 + 16 * mt + 4 * g + r];
    }
    b3[r] = g == 0 ? P[S.o_b3 + r] : 0.f;
  }
  const int W = T.w[l], H = T.h[l], tiles_x = (W + kNgpTile - 1) / kNgpTile;
  float* ew = es[wv];
  const int64_t t0 = tiles * part / parts, t1 = tiles * (part + 1) / parts;
#pragma unroll 1
  for (int64_t tile = t0; tile < t1; ++tile) {
    const int ty = (int)(tile / tiles_x), tx = (int)(tile - (int64_t)ty * tiles_x);
    const int i = tx * kNgpTile + n, j = ty * kNgpTile + (tid >> 4);
    // this thread's encoding (zeros outside the texture)
    float e[KIN];
#pragma unroll
    for (int q = 0; q < KIN; ++q) e[q] = 0.f;
    if (i < W && j < H) {
      const double u = ((double)i + 0.5) / (double)W, v = ((double)j + 0.5) / (double)H;
      ngp_encode<LMAX>(P, S, u, v, e);
    }
#pragma unroll
    for (int q = 0; q < KIN; ++q) ew[lane * EST + q] = e[q];
    if (STAGE) {
      // 32-bit element offsets (the workspace holds < 2^31 floats per array)
      const uint32_t row = (uint32_t)((T.block_off[l] + tile) * 256 + tid), R = (uint32_t)G.R;
#pragma unroll
      for (int q = 0; q < KIN; ++q)
        if (q < nin) G.a1[q * R + row] = e[q];
    }
    ngp_wave_sync();
    // N tile c: texels 16 c + n of this wave = texel row 4 wv + c of the tile
    ngp_f4 h[NT][4], z[NT][4], o[NT];
#pragma unroll
    for (int c = 0; c < NT; ++c) {
#pragma unroll
      for (int mt = 0; mt < 4; ++mt) {
        h[c][mt] = b1[mt];
        z[c][mt] = b2[mt];
      }
      o[c] = b3;
    }
#pragma unroll
    for (int ks = 0; ks < KS1; ++ks) {
      float bop[NT];
#pragma unroll
      for (int c = 0; c < NT; ++c) bop[c] = ew[(16 * c + n) * EST + 4 * ks + g];
#pragma unroll
      for (int mt = 0; mt < 4; ++mt) {
        const float aop = w1f[(mt * KS1 + ks) * 64 + lane];
#pragma unroll
        for (int c = 0; c < NT; ++c) h[c][mt] = __builtin_amdgcn_mfma_f32_16x16x4f32(aop, bop[c], h[c][mt], 0, 0, 0);
      }
    }
#pragma unroll
    for (int c = 0; c < NT; ++c)
#pragma unroll
      for (int mt = 0; mt < 4; ++mt)
#pragma unroll
        for (int r = 0; r < 4; ++r) h[c][mt][r] = fmaxf(h[c][mt][r], 0.f);
#pragma unroll
    for (int it = 0; it < 4; ++it)
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) {
          const float aop = w2f[((mt * 4 + it) * 4 + r) * 64 + lane];
#pragma unroll
          for (int c = 0; c < NT; ++c)
            z[c][mt] = __builtin_amdgcn_mfma_f32_16x16x4f32(aop, h[c][it][r], z[c][mt], 0, 0, 0);
        }
#pragma unroll
    for (int c = 0; c < NT; ++c) {
#pragma unroll
      for (int mt = 0; mt < 4; ++mt)
#pragma unroll
        for (int r = 0; r < 4; ++r) z[c][mt][r] = fmaxf(z[c][mt][r], 0.f);
    }
#pragma unroll
    for (int it = 0; it < 4; ++it)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float aop = w3f[(it * 4 + r) * 64 + lane];
#pragma unroll
        for (int c = 0; c < NT; ++c) o[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(aop, z[c][it][r], o[c], 0, 0, 0);
      }
#pragma unroll
    for (int c = 0; c < NT; ++c) {
      const int tj = ty * kNgpTile + 4 * wv + c;
      if (g == 0 && i < W && tj < H)
        reinterpret_cast<float4*>(T.tex[l])[(int64_t)tj * W + i] =
            make_float4(ngp_sigmoid(o[c][0]), ngp_sigmoid(o[c][1]), ngp_sigmoid(o[c][2]), ngp_sigmoid(o[c][3]));
    }
    ngp_wave_sync();   // the encodings are written again for the next tile
  }
}

// Backward of the network, for every layer, from dL/dtex of a texture baked with
// the same parameters: weight and bias gradients, and dL/de (staged).
//
// Every product of one texel row (16 texels, the N tile) runs on the matrix
// cores (v_mfma_f32_16x16x4_f32) as in the bake, one wavefront per row:
//   forward again: h1 = relu(W1 e + b1), h2 = relu(W2 h1 + b2)
//   d0 = dL/dtex t (1 - t) from the baked texel t
//   d2 = (W3^T d0) [h2 > 0], d1 = (W2^T d2) [h1 > 0], de = W1^T d1
//   dW3 += d0 h2^T, dW2 += d2 h1^T, dW1 += d1 e^T over the row's texels
// An output D[4 (l / 16) + r][l % 16] is chained into the next product as its B
// operand with the K index permuted (as in the bake); the weight gradients
// contract over texels instead, so both factors pass through the wavefront's LDS
// (row stride kNgpRow) and come back unit-per-lane.  260 MFMAs per row.  The
// weight gradients stay in registers (96 accumulators per lane) over all the
// tiles of a block, are summed over its wavefronts in LDS and added to the
// gradient once per block; two blocks share a CU (LDS).  What bounds it is the
// FP32 matrix rate: 459k rows of 260 MFMAs at 32 cycles are 1.6 ms of the 1,024
// SIMDs at 2.4 GHz (seven 1024^2 textures).  It replaces a chain of kernels that
// staged h1, h2, d1 and d2 (1.1 KB per texel written, 1.9 KB read) and formed the
// weight gradients on the VALU: 11.4 ms -> 2.2 ms and 0.27 ms for the scatter below.
constexpr int kNgpRow = 76;

template <int LMAX>
__global__ void __launch_bounds__(256, LMAX <= 8 ? 2 : 1) k_ngp_backward(NgpTable T, NgpShape S, NgpStage G, NgpBlocks Q) {
  constexpr int KIN = 2 * LMAX, KS1 = KIN / 4, MT1 = (KIN + 15) / 16;
  constexpr int W1F = 4 * KS1 * 64, W2N = 64 * 64, W1T = MT1 * 16 * 64;
  __shared__ float wts[W1F + 2 * W2N + W1T + 4 * 64];           // the weights' fragments, and at the end the block's sums
  __shared__ __align__(16) float buf_all[4][2][16 * kNgpRow];   // per wavefront: two [texel][unit] factors
  static_assert(64 * KIN + 64 + 64 * 64 + 64 + 4 * 64 + 4 <= W1F + 2 * W2N + W1T + 4 * 64, "the sums fit the weights' space");
  float* w1f = wts;          // [mt][ks][lane]: W1[16 mt + lane % 16][4 ks + lane / 16]
  float* w2f = w1f + W1F;    // [mt][it][r][lane]: W2[16 mt + lane % 16][16 it + 4 (lane / 16) + r]
  float* w2t = w2f + W2N;    // [mt][it][r][lane]: W2[16 it + 4 (lane / 16) + r][16 mt + lane % 16]
  float* w1t = w2t + W2N;    // [mt][it][r][lane]: W1[16 it + 4 (lane / 16) + r][16 mt + lane % 16]
  float* w3t = w1t + W1T;    // [mt][lane]: W3[lane / 16][16 mt + lane % 16]
  const int tid = threadIdx.x, wv = tid >> 6, lane = tid & 63, g = lane >> 4, n = lane & 15;
  int l = 0;
  while (l + 1 < T.k && Q.off[l + 1] <= (int)blockIdx.x) ++l;
  const int part = (int)blockIdx.x - Q.off[l], parts = Q.off[l + 1] - Q.off[l];
  const int64_t tiles = T.block_off[l + 1] - T.block_off[l];
  const int W = T.w[l], H = T.h[l], tiles_x = (W + kNgpTile - 1) / kNgpTile;
  const float* P = T.params[l];
  const int nin = 2 * S.levels;
  const uint32_t R = (uint32_t)G.R;
  for (int f = tid; f < 4 * KS1 * 64; f += 256) {
    const int ln = f & 63, fr = f >> 6, mt = fr / KS1, ks = fr - mt * KS1;
    const int m = 16 * mt + (ln & 15), kk = 4 * ks + (ln >> 4);
    w1f[f] = kk < nin ? P[S.o_w1 + m * nin + kk] : 0.f;
  }
  for (int f = tid; f < 64 * 64; f += 256) {
    const int ln = f & 63, fr = f >> 6, mt = fr >> 4, it = (fr >> 2) & 3, r = fr & 3;
    const int a = 16 * mt + (ln & 15), b = 16 * it + 4 * (ln >> 4) + r;
    w2f[f] = P[S.o_w2 + a * kNgpHidden + b];
    w2t[f] = P[S.o_w2 + b * kNgpHidden + a];
  }
  for (int f = tid; f < MT1 * 16 * 64; f += 256) {
    const int ln = f & 63, fr = f >> 6, mt = fr >> 4, it = (fr >> 2) & 3, r = fr & 3;
    const int q = 16 * mt + (ln & 15), j = 16 * it + 4 * (ln >> 4) + r;
    w1t[f] = q < nin ? P[S.o_w1 + j * nin + q] : 0.f;
  }
  for (int f = tid; f < 4 * 64; f += 256) w3t[f] = P[S.o_w3 + ((f >> 4) & 3) * kNgpHidden + 16 * (f >> 6) + (f & 15)];
  __syncthreads();
  float* x0 = buf_all[wv][0];
  float* x1 = buf_all[wv][1];
  ngp_f4 b1[4], b2[4];
#pragma unroll
  for (int mt = 0; mt < 4; ++mt)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      b1[mt][r] = P[S.o_b1 + 16 * mt + 4 * g + r];
      b2[mt][r] = P[S.o_b2 + 16 * mt + 4 * g + r];
    }
  // accumulators: dW2[16 mt + 4 g + r][16 nt + n], dW1[16 mt + 4 g + r][16 nt + n], dW3[n][16 mt + 4 g + r] (n < 4),
  // and per lane the sums of d2 and d1 (unit 16 mt + n) and d0 (output g) over its share of the texels
  ngp_f4 c2[4][4], c1[4][MT1], c3[4];
  float s2[4], s1[4], s0 = 0.f;
#pragma unroll
  for (int a = 0; a < 4; ++a) {
#pragma unroll
    for (int b = 0; b < 4; ++b) c2[a][b] = ngp_f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int b = 0; b < MT1; ++b) c1[a][b] = ngp_f4{0.f, 0.f, 0.f, 0.f};
    c3[a] = ngp_f4{0.f, 0.f, 0.f, 0.f};
    s2[a] = s1[a] = 0.f;
  }
  const int64_t t0 = tiles * part / parts, t1 = tiles * (part + 1) / parts;
#pragma unroll 1
  for (int64_t row4 = 4 * t0; row4 < 4 * t1; ++row4) {   // this wavefront's texel rows: four of each tile
    const int64_t tile = row4 >> 2;
    const int rr = 4 * wv + (int)(row4 & 3);
    const int ty = (int)(tile / tiles_x), tx = (int)(tile - (int64_t)ty * tiles_x);
    const int ti = tx * kNgpTile + n, tj = ty * kNgpTile + rr;
    const bool valid = ti < W && tj < H;
    const uint32_t row = (uint32_t)((T.block_off[l] + tile) * 256 + 16 * rr + n);
    float e[KS1];
#pragma unroll
    for (int ks = 0; ks < KS1; ++ks) e[ks] = 4 * ks + g < nin ? G.a1[(uint32_t)(4 * ks + g) * R + row] : 0.f;
    float d0 = 0.f;
    if (valid) {
      const int64_t at = ((int64_t)tj * W + ti) * 4 + g;
      const float t = T.tex[l][at];
      d0 = T.gtex[l][at] * t * (1.0f - t);
    }
    s0 += d0;
    // forward
    ngp_f4 h1[4], h2[4];
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) h1[mt] = b1[mt];
#pragma unroll
    for (int ks = 0; ks < KS1; ++ks)
#pragma unroll
      for (int mt = 0; mt < 4; ++mt)
        h1[mt] = __builtin_amdgcn_mfma_f32_16x16x4f32(w1f[(mt * KS1 + ks) * 64 + lane], e[ks], h1[mt], 0, 0, 0);
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
#pragma unroll
      for (int r = 0; r < 4; ++r) h1[mt][r] = fmaxf(h1[mt][r], 0.f);
      h2[mt] = b2[mt];
    }
#pragma unroll
    for (int it = 0; it < 4; ++it)
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int mt = 0; mt < 4; ++mt)
          h2[mt] = __builtin_amdgcn_mfma_f32_16x16x4f32(w2f[((mt * 4 + it) * 4 + r) * 64 + lane], h1[it][r], h2[mt], 0, 0, 0);
#pragma unroll
    for (int mt = 0; mt < 4; ++mt)
#pragma unroll
      for (int r = 0; r < 4; ++r) h2[mt][r] = fmaxf(h2[mt][r], 0.f);
    if (!__all(valid)) {   // no hidden unit is on outside the texture: nothing of it meets an infinite weight or gradient
#pragma unroll
      for (int mt = 0; mt < 4; ++mt)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          h1[mt][r] = valid ? h1[mt][r] : 0.f;
          h2[mt][r] = valid ? h2[mt][r] : 0.f;
        }
    }
    // d2, and dW3 from h2 and d0
    ngp_f4 d2[4];
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
      d2[mt] = __builtin_amdgcn_mfma_f32_16x16x4f32(w3t[mt * 64 + lane], d0, ngp_f4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
#pragma unroll
      for (int r = 0; r < 4; ++r) d2[mt][r] = h2[mt][r] > 0.f ? d2[mt][r] : 0.f;
      *reinterpret_cast<ngp_f4*>(x0 + n * kNgpRow + 16 * mt + 4 * g) = h2[mt];
    }
    x1[n * kNgpRow + g] = d0;
    ngp_wave_sync();
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      const float* at = x1 + (4 * ks + g) * kNgpRow;
      const float bop = n < kNgpOut ? at[n & 3] : 0.f;
#pragma unroll
      for (int mt = 0; mt < 4; ++mt)
        c3[mt] = __builtin_amdgcn_mfma_f32_16x16x4f32(x0[(4 * ks + g) * kNgpRow + 16 * mt + n], bop, c3[mt], 0, 0, 0);
    }
    ngp_wave_sync();
    // dW2 from d2 and h1
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
      *reinterpret_cast<ngp_f4*>(x0 + n * kNgpRow + 16 * mt + 4 * g) = h1[mt];
      *reinterpret_cast<ngp_f4*>(x1 + n * kNgpRow + 16 * mt + 4 * g) = d2[mt];
    }
    ngp_wave_sync();
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      float aop[4], bop[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        aop[q] = x1[(4 * ks + g) * kNgpRow + 16 * q + n];
        bop[q] = x0[(4 * ks + g) * kNgpRow + 16 * q + n];
        s2[q] += aop[q];
      }
#pragma unroll
      for (int mt = 0; mt < 4; ++mt)
#pragma unroll
        for (int nt = 0; nt < 4; ++nt)
          c2[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(aop[mt], bop[nt], c2[mt][nt], 0, 0, 0);
    }
    // d1, then dW1 from d1 and e
    ngp_f4 d1[4];
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) d1[mt] = ngp_f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int it = 0; it < 4; ++it)
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int mt = 0; mt < 4; ++mt)
          d1[mt] = __builtin_amdgcn_mfma_f32_16x16x4f32(w2t[((mt * 4 + it) * 4 + r) * 64 + lane], d2[it][r], d1[mt], 0, 0, 0);
    ngp_wave_sync();
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
#pragma unroll
      for (int r = 0; r < 4; ++r) d1[mt][r] = h1[mt][r] > 0.f ? d1[mt][r] : 0.f;
      *reinterpret_cast<ngp_f4*>(x1 + n * kNgpRow + 16 * mt + 4 * g) = d1[mt];
    }
#pragma unroll
    for (int ks = 0; ks < KS1; ++ks) x0[n * kNgpRow + 4 * ks + g] = e[ks];
    ngp_wave_sync();
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      float bop[MT1];
#pragma unroll
      for (int nt = 0; nt < MT1; ++nt) bop[nt] = x0[(4 * ks + g) * kNgpRow + 16 * nt + n];
#pragma unroll
      for (int mt = 0; mt < 4; ++mt) {
        const float aop = x1[(4 * ks + g) * kNgpRow + 16 * mt + n];
        s1[mt] += aop;
#pragma unroll
        for (int nt = 0; nt < MT1; ++nt) c1[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(aop, bop[nt], c1[mt][nt], 0, 0, 0);
      }
    }
    ngp_wave_sync();
    // de
#pragma unroll
    for (int mt = 0; mt < MT1; ++mt) {
      ngp_f4 de = ngp_f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int it = 0; it < 4; ++it)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          de = __builtin_amdgcn_mfma_f32_16x16x4f32(w1t[((mt * 4 + it) * 4 + r) * 64 + lane], d1[it][r], de, 0, 0, 0);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const uint32_t q = 16 * mt + 4 * g + r;
        if (q < (uint32_t)nin) G.de[q * R + row] = de[r];
      }
    }
  }
  // sum over the wavefronts in LDS (the weights' space), then into the gradient, one atomic per parameter
  __syncthreads();
  float* sum = wts;   // W1 | b1 | W2 | b2 | W3 | b3, as the parameters lie
  const int m1 = 64 * nin, q2 = m1 + 64, q3 = q2 + 64 * 64 + 64, total = q3 + 4 * 64 + 4;
  for (int f = tid; f < total; f += 256) sum[f] = 0.f;
  for (int w = 0; w < 4; ++w) {
    __syncthreads();
    if (wv != w) continue;
#pragma unroll
    for (int mt = 0; mt < 4; ++mt)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = 16 * mt + 4 * g + r;
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) sum[q2 + m * 64 + 16 * nt + n] += c2[mt][nt][r];
#pragma unroll
        for (int nt = 0; nt < MT1; ++nt)
          if (16 * nt + n < nin) sum[m * nin + 16 * nt + n] += c1[mt][nt][r];
        if (n < kNgpOut) sum[q3 + n * 64 + m] += c3[mt][r];
      }
#pragma unroll
    for (int q = 0; q < 4; ++q) {   // a lane's sums cover every fourth texel: add the four lanes of a unit
      float v2 = s2[q], v1 = s1[q];
      v2 += __shfl_xor(v2, 16); v2 += __shfl_xor(v2, 32);
      v1 += __shfl_xor(v1, 16); v1 += __shfl_xor(v1, 32);
      if (g == 0) {
        sum[q2 + 64 * 64 + 16 * q + n] += v2;
        sum[m1 + 16 * q + n] += v1;
      }
    }
    float v0 = s0;
#pragma unroll
    for (int off = 1; off < 16; off <<= 1) v0 += __shfl_xor(v0, off);
    if (n == 0) sum[q3 + 4 * 64 + g] += v0;
  }
  __syncthreads();
  float* gp = T.gparams[l] + S.o_w1;
  for (int f = tid; f < total; f += 256)
    if (sum[f] != 0.0f) unsafeAtomicAdd(gp + f, sum[f]);
}

// Scatter of the staged dL/de into the hash tables, one 16 x 16 texel tile per
// block, one level per wavefront at a time.
//
// A vertex of a level receives sum_j sum_i wy(j) wx(i) de[j][i] over the tile's
// texels: the bilinear weights are a product of an x and a y part, so the sums
// are two small matrix products on the matrix cores (v_mfma_f32_16x16x4_f32),
// D[j][vx] = de[j][i] Wx[i][vx] and then Wy[vy][j] D[j][vx], whose second operand
// is the first's output registers (K permuted as in the bake; de is loaded as 16
// bytes per lane in that order).  However many texels share a vertex, nothing is
// added twice to one LDS or memory word.  The window of ex x ey vertices that the
// tile touches goes through LDS, so that the global atomics, one per table float,
// run over consecutive floats.  LDS float atomics per texel and corner, 64 of
// them on one word at a coarse level, took 2.87 ms for seven 1024^2 textures of 8
// levels; this takes 0.27 ms.
// A window of more than kNgpSlots vertices (vertices finer than texels) adds each
// corner with a global atomic, and so does a level with an infinite or NaN de,
// or one so large that a sum of products might overflow, for infinity times a
// weight of zero is NaN: such a value must reach its own four vertices only.
template <int LMAX>
__global__ void __launch_bounds__(256) k_ngp_scatter(NgpTable T, NgpShape S, NgpStage G) {
  __shared__ int32_t first[LMAX][2];                       // per level: the window's first vertex (x, y)
  __shared__ __align__(16) int32_t cell[LMAX][2][16];      // per level, axis and texel column or row: vertex in the window
  __shared__ __align__(16) float frac[LMAX][2][16];        // ... and offset from it
  __shared__ float win_all[4][2 * kNgpSlots];              // per wavefront: the window's sums [vy][vx][feature]
  const int64_t b = blockIdx.x;
  int l = 0;
  while (l + 1 < T.k && T.block_off[l + 1] <= b) ++l;
  const int W = T.w[l], H = T.h[l], tiles_x = (W + kNgpTile - 1) / kNgpTile;
  const int64_t tb = b - T.block_off[l];
  const int ty = (int)(tb / tiles_x), tx = (int)(tb - (int64_t)ty * tiles_x);
  const int tid = threadIdx.x, wv = tid >> 6, lane = tid & 63, g = lane >> 4, n = lane & 15;
  for (int q = tid; q < 32 * S.levels; q += 256) {
    const int lv = q >> 5, axis = (q >> 4) & 1, c = q & 15;
    const double N = (double)S.res[lv], size = axis ? (double)H : (double)W;
    const int at0 = kNgpTile * (axis ? ty : tx);
    const double x = ((double)(at0 + c) + 0.5) / size * N, x0 = floor(x), xa = floor(((double)at0 + 0.5) / size * N);
    cell[lv][axis][c] = (int32_t)(x0 - xa);
    frac[lv][axis][c] = (float)(x - x0);
    if (c == 0) first[lv][axis] = (int32_t)xa;
  }
  __syncthreads();
  const uint32_t TT = 1u << S.log2_table, mask = TT - 1u;
  float* win = win_all[wv];
#pragma unroll 1
  for (int lv = wv; lv < S.levels; lv += 4) {
    float* gtab = T.gparams[l] + (int64_t)lv * TT * 2;
    const int32_t N = S.res[lv], dense = S.dense[lv];
    // de of texel row n, columns 4 g .. 4 g + 3
    const float* src = G.de + (uint32_t)(2 * lv) * (uint32_t)G.R + (uint32_t)(b * 256) + 16 * n + 4 * g;
    ngp_f4 de[2];
    de[0] = *reinterpret_cast<const ngp_f4*>(src);
    de[1] = *reinterpret_cast<const ngp_f4*>(src + G.R);
    const int ex = cell[lv][0][15] + 2, ey = cell[lv][1][15] + 2;   // uniform
    const uint32_t vx0 = (uint32_t)first[lv][0], vy0 = (uint32_t)first[lv][1];
    bool bounded = true;   // 256 texels' values of at most 2^112, weighted by at most 1, sum to a float (false for NaN)
#pragma unroll
    for (int q = 0; q < 8; ++q) bounded = bounded && fabsf(de[q >> 2][q & 3]) <= 0x1p112f;
    if ((int64_t)ex * ey <= kNgpSlots && __all(bounded)) {
      const int4 cx = *reinterpret_cast<const int4*>(&cell[lv][0][4 * g]), cy = *reinterpret_cast<const int4*>(&cell[lv][1][4 * g]);
      const float4 fx = *reinterpret_cast<const float4*>(&frac[lv][0][4 * g]);
      const float4 fy = *reinterpret_cast<const float4*>(&frac[lv][1][4 * g]);
      const int cxs[4] = {cx.x, cx.y, cx.z, cx.w}, cys[4] = {cy.x, cy.y, cy.z, cy.w};
      const float fxs[4] = {fx.x, fx.y, fx.z, fx.w}, fys[4] = {fy.x, fy.y, fy.z, fy.w};
      for (int nx = 0; nx < ex; nx += 16) {
        ngp_f4 d[2] = {ngp_f4{0.f, 0.f, 0.f, 0.f}, ngp_f4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int at = nx + n - cxs[q];
          const float w = at == 0 ? 1.0f - fxs[q] : at == 1 ? fxs[q] : 0.f;
#pragma unroll
          for (int f = 0; f < 2; ++f) d[f] = __builtin_amdgcn_mfma_f32_16x16x4f32(de[f][q], w, d[f], 0, 0, 0);
        }
        for (int ny = 0; ny < ey; ny += 16) {
          ngp_f4 o[2] = {ngp_f4{0.f, 0.f, 0.f, 0.f}, ngp_f4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int at = ny + n - cys[q];
            const float w = at == 0 ? 1.0f - fys[q] : at == 1 ? fys[q] : 0.f;
#pragma unroll
            for (int f = 0; f < 2; ++f) o[f] = __builtin_amdgcn_mfma_f32_16x16x4f32(w, d[f][q], o[f], 0, 0, 0);
          }
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int vy = ny + 4 * g + r, vx = nx + n;
            if (vy < ey && vx < ex) *reinterpret_cast<float2*>(win + 2 * (vy * ex + vx)) = make_float2(o[0][r], o[1][r]);
          }
        }
      }
      ngp_wave_sync();
      // vertex p / 2 of the window: its row is the high word of a product with ceil(2^32 / ex) (exact below 2^16)
      const uint32_t m = 0xffffffffu / (uint32_t)ex + 1u;
      for (int p = lane; p < 2 * ex * ey; p += 64) {
        const float v = win[p];
        if (v != 0.0f) {
          const uint32_t slot = (uint32_t)p >> 1, vy = __umulhi(slot, m), vx = slot - vy * (uint32_t)ex;
          unsafeAtomicAdd(gtab + 2 * (int64_t)ngp_index(vx0 + vx, vy0 + vy, N, dense, mask) + (p & 1), v);
        }
      }
      ngp_wave_sync();   // the window is written again by the next level
    } else {
      const int j = kNgpTile * ty + n;
      const uint32_t yi = vy0 + (uint32_t)cell[lv][1][n];
      const float fy = frac[lv][1][n];
      for (int q = 0; q < 4; ++q) {
        const int i = kNgpTile * tx + 4 * g + q;
        if (i >= W || j >= H) continue;
        const uint32_t xi = vx0 + (uint32_t)cell[lv][0][4 * g + q];
        const float fx = frac[lv][0][4 * g + q];
        const float v0 = q == 0 ? de[0][0] : q == 1 ? de[0][1] : q == 2 ? de[0][2] : de[0][3];
        const float v1 = q == 0 ? de[1][0] : q == 1 ? de[1][1] : q == 2 ? de[1][2] : de[1][3];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const uint32_t dx = c & 1, dy = c >> 1;
          const float w = (dx ? fx : 1.0f - fx) * (dy ? fy : 1.0f - fy);
          float* to = gtab + 2 * (int64_t)ngp_index(xi + dx, yi + dy, N, dense, mask);
          unsafeAtomicAdd(to, w * v0);
          unsafeAtomicAdd(to + 1, w * v1);
        }
      }
    }
  }
}

}  // namespace vs
