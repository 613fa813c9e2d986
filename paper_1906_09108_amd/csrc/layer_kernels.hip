// Kernels of the layers that only the Tiny-ImageNet networks of Table V need: the ImageNet stem of ResNet-18 (7x7
// convolution of stride 2 as row gathers + a 1x1 contraction, 3x3 max-pool of stride 2) and the depthwise 3x3 convolution of
// MobileNet-v2's inverted residual block.  All of them move each tensor once and do a handful of operations per element:
// HBM-bound.  Tensors are NHWC; a thread owns 8 consecutive channels of one pixel (one 16-byte bf16 access).
#include "fdg_internal.h"

#include <algorithm>

namespace fdg {
namespace {

__device__ __forceinline__ float lo16(uint32_t u) { return __builtin_bit_cast(float, u << 16); }
__device__ __forceinline__ float hi16(uint32_t u) { return __builtin_bit_cast(float, u & 0xffff0000u); }
__device__ __forceinline__ void unpack(const uint4& u, float (&f)[8]) {
  f[0] = lo16(u.x); f[1] = hi16(u.x); f[2] = lo16(u.y); f[3] = hi16(u.y);
  f[4] = lo16(u.z); f[5] = hi16(u.z); f[6] = lo16(u.w); f[7] = hi16(u.w);
}
__device__ __forceinline__ uint32_t pack2(float a, float b) {
  const bf16_t l = (bf16_t)a, h = (bf16_t)b;
  return (uint32_t)__builtin_bit_cast(uint16_t, l) | ((uint32_t)__builtin_bit_cast(uint16_t, h) << 16);
}
__device__ __forceinline__ uint4 pack(const float (&f)[8]) {
  return make_uint4(pack2(f[0], f[1]), pack2(f[2], f[3]), pack2(f[4], f[5]), pack2(f[6], f[7]));
}
__device__ __forceinline__ void store_f32(float* p, const float (&f)[8]) {
  *reinterpret_cast<float4*>(p) = make_float4(f[0], f[1], f[2], f[3]);
  *reinterpret_cast<float4*>(p + 4) = make_float4(f[4], f[5], f[6], f[7]);
}
__device__ __forceinline__ void load_f32(const float* p, float (&f)[8]) {
  const float4 a = *reinterpret_cast<const float4*>(p), b = *reinterpret_cast<const float4*>(p + 4);
  f[0] = a.x; f[1] = a.y; f[2] = a.z; f[3] = a.w; f[4] = b.x; f[5] = b.y; f[6] = b.z; f[7] = b.w;
}
int grid_for(size_t threads) {
  const size_t b = (threads + 255) / 256;
  return (int)(b < 1 ? 1 : b);
}

// ---- 7x7 convolution of stride 2, padding 3, over an input of 8 stored channels --------------------------------
// col[m, kh, kw, c] = x[n, 2 oh - 3 + kh, 2 ow - 3 + kw, c] (m = (n, oh, ow); kh < 7; kw < 8, the column kw = 7 is zero, as is
// everything outside the image).  Row m of col is the 448-element operand of output pixel m: the convolution is
// col [M, 448] times w [Co, 448] and its weight gradient dy^T col, which the 1x1 kernels compute.
__global__ __launch_bounds__(256) void im2col7_kernel(const uint4* __restrict__ x, uint4* __restrict__ col, int N, int H, int W,
                                                      int Ho, int Wo) {
  const size_t total = (size_t)N * Ho * Wo * 56;
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= total) return;
  const int kw = (int)(i % 8), kh = (int)((i / 8) % 7);
  const size_t m = i / 56;
  const int ow = (int)(m % Wo), oh = (int)((m / Wo) % Ho), n = (int)(m / ((size_t)Wo * Ho));
  const int h = 2 * oh - 3 + kh, w = 2 * ow - 3 + kw;
  uint4 v = make_uint4(0u, 0u, 0u, 0u);
  if (kw < 7 && h >= 0 && h < H && w >= 0 && w < W) v = x[((size_t)n * H + h) * W + w];
  col[i] = v;
}

// ---- 3x3 max-pool of stride 2, padding 1 --------------------------------------------------------------------------
__global__ __launch_bounds__(256) void maxpool3s2_kernel(const bf16_t* __restrict__ x, float* __restrict__ y_f32,
                                                         bf16_t* __restrict__ y_b16, int N, int H, int W, int C, int Ho, int Wo) {
  const int CG = C / 8;
  const size_t total = (size_t)N * Ho * Wo * CG;
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= total) return;
  const int cg = (int)(i % CG);
  const size_t m = i / CG;
  const int wo = (int)(m % Wo), ho = (int)((m / Wo) % Ho), n = (int)(m / ((size_t)Wo * Ho));
  float best[8];
  bool have = false;
#pragma unroll
  for (int r = 0; r < 3; ++r)
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const int h = 2 * ho - 1 + r, w = 2 * wo - 1 + q;
      if (h < 0 || h >= H || w < 0 || w >= W) continue;
      float f[8];
      unpack(*reinterpret_cast<const uint4*>(x + (((size_t)n * H + h) * W + w) * C + cg * 8), f);
#pragma unroll
      for (int k = 0; k < 8; ++k) best[k] = (!have || f[k] > best[k]) ? f[k] : best[k];
      have = true;
    }
  const size_t o = m * C + cg * 8;
  if (y_f32) store_f32(y_f32 + o, best);
  if (y_b16) *reinterpret_cast<uint4*>(y_b16 + o) = pack(best);   // exact: a maximum of bf16 values
}

// dx[n, h, w, c] = sum of dy over the windows whose FIRST maximum (rows, then columns) is the cell (h, w).  One thread per
// input cell and 8 channels; it looks at the (at most four) windows that contain the cell.
__global__ __launch_bounds__(256) void maxpool3s2_bwd_kernel(const bf16_t* __restrict__ x, const float* __restrict__ dy,
                                                             float* __restrict__ dx, int N, int H, int W, int C, int Ho, int Wo) {
  const int CG = C / 8;
  const size_t total = (size_t)N * H * W * CG;
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= total) return;
  const int cg = (int)(i % CG);
  const size_t pix = i / CG;
  const int w0 = (int)(pix % W), h0 = (int)((pix / W) % H), n = (int)(pix / ((size_t)W * H));
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  // windows ho with 2 ho - 1 <= h0 <= 2 ho + 1
  const int ho_lo = h0 / 2, ho_hi = (h0 + 1) / 2, wo_lo = w0 / 2, wo_hi = (w0 + 1) / 2;
  for (int ho = ho_lo; ho <= ho_hi; ++ho) {
    if (ho >= Ho) continue;
    for (int wo = wo_lo; wo <= wo_hi; ++wo) {
      if (wo >= Wo) continue;
      float best[8];
      bool mine[8] = {false, false, false, false, false, false, false, false};
      bool have = false;
#pragma unroll
      for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int q = 0; q < 3; ++q) {
          const int h = 2 * ho - 1 + r, w = 2 * wo - 1 + q;
          if (h < 0 || h >= H || w < 0 || w >= W) continue;
          float f[8];
          unpack(*reinterpret_cast<const uint4*>(x + (((size_t)n * H + h) * W + w) * C + cg * 8), f);
          const bool me = h == h0 && w == w0;
#pragma unroll
          for (int k = 0; k < 8; ++k)
            if (!have || f[k] > best[k]) { best[k] = f[k]; mine[k] = me; }
          have = true;
        }
      float g[8];
      load_f32(dy + (((size_t)n * Ho + ho) * Wo + wo) * C + cg * 8, g);
#pragma unroll
      for (int k = 0; k < 8; ++k)
        if (mine[k]) acc[k] += g[k];
    }
  }
  store_f32(dx + pix * C + cg * 8, acc);
}

// ---- depthwise 3x3 convolution, padding 1, stride 1 or 2; wt = [9][C] bf16 (tap-major) ------------------------------
// Memory sets the floor (each tensor moved once), but a thread that made one output cell spent its time on the vector ALU:
// four 64-bit divisions, and nine taps each unpacked for one use.  Here a thread makes 2 x 2 output cells of 8 channels from a
// patch of (S + 3)^2 cells whose loads are all issued first; a cell is unpacked once for up to four outputs, the filter once
// for the thread, and the image index comes from the block index.  128 x 16 x 16 x 384, stride 1: forward 26.5 -> 17.3 us
// (50 MB, 2.9 TB/s), data gradient 40.5 -> 17.4 us.
// FLIP: the data gradient at unit stride, dx[h, w] = sum of dy[h + 1 - r, w + 1 - q] * w[r][q]: the same patch, its cells taken
// from the last to the first.  Sums run over (r, q) in order either way.  A cell outside the image is left out, not multiplied as
// a zero: an infinite weight or cell reaches the outputs it reaches in the definition and no others.
template <int S, bool FLIP>
__device__ __forceinline__ void dw_cells(const bf16_t* img, const float (&k)[9][8], int h0, int w0, int H, int W, int C, float (&acc)[2][2][8]) {
  constexpr int P = S + 3;
  uint4 raw[P][P];
#pragma unroll
  for (int r = 0; r < P; ++r)
#pragma unroll
    for (int q = 0; q < P; ++q) {
      const int h = h0 + r, w = w0 + q;
      raw[r][q] = make_uint4(0u, 0u, 0u, 0u);
      if (h >= 0 && h < H && w >= 0 && w < W) raw[r][q] = *reinterpret_cast<const uint4*>(img + ((size_t)h * W + w) * C);
    }
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int j = 0; j < 8; ++j) acc[a][b][j] = 0.f;
#pragma unroll
  for (int rr = 0; rr < P; ++rr)
#pragma unroll
    for (int qq = 0; qq < P; ++qq) {
      const int pr = FLIP ? P - 1 - rr : rr, pq = FLIP ? P - 1 - qq : qq;
      const int h = h0 + pr, w = w0 + pq;
      if (h < 0 || h >= H || w < 0 || w >= W) continue;
      float f[8];
      unpack(raw[pr][pq], f);
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          const int tr = pr - a * S, tq = pq - b * S;
          if (tr < 0 || tr > 2 || tq < 0 || tq > 2) continue;
          const int t = FLIP ? (2 - tr) * 3 + 2 - tq : tr * 3 + tq;
#pragma unroll
          for (int j = 0; j < 8; ++j) acc[a][b][j] += f[j] * k[t][j];
        }
    }
}
__device__ __forceinline__ void dw_filter(const bf16_t* wt, int C, int cg, float (&k)[9][8]) {
#pragma unroll
  for (int t = 0; t < 9; ++t) unpack(*reinterpret_cast<const uint4*>(wt + (size_t)t * C + cg * 8), k[t]);
}
template <int S, bool FLIP>
__global__ __launch_bounds__(256) void dwconv3_kernel(const bf16_t* __restrict__ x, const bf16_t* __restrict__ wt,
                                                      bf16_t* __restrict__ y, int H, int W, int C, int Ho, int Wo,
                                                      int blocks_per_image) {
  static_assert(!FLIP || S == 1, "a stride-2 data gradient has a kernel of its own");
  const int CG = C / 8, WB = (Wo + 1) / 2, HB = (Ho + 1) / 2;
  const int n = blockIdx.x / blocks_per_image;
  const unsigned i = (unsigned)(blockIdx.x % blocks_per_image) * 256u + threadIdx.x;
  if (i >= (unsigned)HB * WB * CG) return;
  const int cg = i % CG, p = i / CG, wb = p % WB, hb = p / WB;
  float k[9][8], acc[2][2][8];
  dw_filter(wt, C, cg, k);
  dw_cells<S, FLIP>(x + (size_t)n * H * W * C + cg * 8, k, 2 * S * hb - 1, 2 * S * wb - 1, H, W, C, acc);
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const int ho = 2 * hb + a, wo = 2 * wb + b;
      if (ho >= Ho || wo >= Wo) continue;
      const size_t o = (((size_t)n * Ho + ho) * Wo + wo) * C + cg * 8;
      *reinterpret_cast<uint4*>(y + o) = pack(acc[a][b]);
    }
}

// Data gradient at stride 2: dx[h, w] = sum over taps with h + 1 - r = 2 ho, w + 1 - q = 2 wo of dy[ho, wo] * w[r][q].  A thread
// makes the cells (2a, 2b) .. (2a + 1, 2b + 1), which together take each of the nine taps once, from dy[a .. a + 1][b .. b + 1].
// 128 x 32 x 32 x 192 from 16 x 16: 52.2 -> 13.9 us (63 MB, 4.5 TB/s).
__device__ __forceinline__ void dw_dgrad2_cells(const bf16_t* img, const float (&k)[9][8], int hb, int wb, int Ho, int Wo, int C,
                                                float (&acc)[2][2][8]) {
  float g[2][2][8];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      uint4 u = make_uint4(0u, 0u, 0u, 0u);
      if (hb + a < Ho && wb + b < Wo) u = *reinterpret_cast<const uint4*>(img + ((size_t)(hb + a) * Wo + wb + b) * C);
      unpack(u, g[a][b]);
    }
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int j = 0; j < 8; ++j) acc[a][b][j] = 0.f;
  // dy cell by dy cell, the last first: every sum then runs over (r, q) in order.  r = 1 reaches the even row from dy row a, r = 0
  // and 2 the odd row from dy rows a + 1 and a; columns alike.  A cell outside dy is left out, not multiplied as a zero.
#pragma unroll
  for (int cell = 3; cell >= 0; --cell) {
    const int ga = cell >> 1, gb = cell & 1;
    if (hb + ga >= Ho || wb + gb >= Wo) continue;
#pragma unroll
    for (int t = 0; t < 9; ++t) {
      const int r = t / 3, q = t % 3;
      if ((r == 0 ? 1 : 0) != ga || (q == 0 ? 1 : 0) != gb) continue;
#pragma unroll
      for (int j = 0; j < 8; ++j) acc[r == 1 ? 0 : 1][q == 1 ? 0 : 1][j] += g[ga][gb][j] * k[t][j];
    }
  }
}
__global__ __launch_bounds__(256) void dwconv3_dgrad2_kernel(const bf16_t* __restrict__ dy, const bf16_t* __restrict__ wt,
                                                             bf16_t* __restrict__ dx, int H, int W, int C, int Ho, int Wo,
                                                             int blocks_per_image) {
  const int CG = C / 8, WB = (W + 1) / 2, HB = (H + 1) / 2;   // Ho = HB, Wo = WB
  const int n = blockIdx.x / blocks_per_image;
  const unsigned i = (unsigned)(blockIdx.x % blocks_per_image) * 256u + threadIdx.x;
  if (i >= (unsigned)HB * WB * CG) return;
  const int cg = i % CG, p = i / CG, wb = p % WB, hb = p / WB;
  float k[9][8], acc[2][2][8];
  dw_filter(wt, C, cg, k);
  dw_dgrad2_cells(dy + (size_t)n * Ho * Wo * C + cg * 8, k, hb, wb, Ho, Wo, C, acc);
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const int h = 2 * hb + a, w = 2 * wb + b;
      if (h >= H || w >= W) continue;
      const size_t o = (((size_t)n * H + h) * W + w) * C + cg * 8;
      *reinterpret_cast<uint4*>(dx + o) = pack(acc[a][b]);
    }
}

// The same cells with the per-channel sums of the batch norm beside them, which saves that batch norm a pass over the result: of the
// forward (bf16) the sum and the sum of squares; of a data gradient (fp32, zeroed where the gate is not strictly between 0 and
// gate_hi) the sum and the sum of its products with bnx, taken around the mean of bnx.  A workgroup owns 64 channels, eight to a
// thread, and takes 32 blocks of 2 x 2 cells a round, so that its sums stay in registers and end in one exact add per channel and
// value (2 x 2 cells of all channels, as above, would add for every block).  Orders are fixed.  128 x 16 x 16 x 384, the passes it
// replaces -> here: forward 17.4 + 8.7 -> 20.7 us, data gradient 21.9 + 19.4 (and 3.4 of the pass that follows, which reads no gate)
// -> 34.7 us (126 MB).  At every size: what is saved on the smallest tensors is the launches (two blocks over one 8 x 8 image, 1 x 8 x
// 8 x 192, 317 .. 322 -> 311 us a step; 2 x 16 x 16 441 -> 406; seven blocks, 128 x 32 x 32 2340 -> 2186).
struct DwSums {
  const bf16_t* src;    // [N, Hs, Ws, C]
  const bf16_t* wt;
  bf16_t* y;            // forward
  float* dx;            // data gradient
  const bf16_t* gate;
  const bf16_t* bnx;
  const stat_t* bnx_sums;   // forward sums of bnx's batch norm: the second sum is taken around its mean (StatMean); nullptr: around 0
  float gate_hi;
  stat_t* sums;
  int rep_stride;
  int N, Hs, Ws, C, Hd, Wd;   // Hd, Wd: the result's
  int rounds;                 // of 32 blocks a workgroup
};
template <int S, bool DGRAD>
__global__ __launch_bounds__(256) void dwconv3_sums_kernel(DwSums a) {
  __shared__ float red[2][32][64];
  __shared__ float centre[64];
  const int C = a.C, CG = C / 8, WB = (a.Wd + 1) / 2, HB = (a.Hd + 1) / 2;
  const int cgl = threadIdx.x & 7, rl = threadIdx.x >> 3, cg = blockIdx.x * 8 + cgl;
  const int own = blockIdx.x * 64 + threadIdx.x;
  const bool centres = DGRAD && threadIdx.x < 64 && a.bnx_sums && own < C;
  StatMean sm;
  if (centres) sm.load(a.bnx_sums, C, own, a.rep_stride);
  float k[9][8], mu[8];
  if (cg < CG) dw_filter(a.wt, C, cg, k);
  if (DGRAD) {
    if (threadIdx.x < 64) centre[threadIdx.x] = centres ? sm.mean(1.0 / ((double)a.N * a.Hd * a.Wd)) : 0.f;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 8; ++j) mu[j] = centre[cgl * 8 + j];
  }
  float s1[8], s2[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) s1[j] = s2[j] = 0.f;
  if (cg < CG) {
    const unsigned per_image = (unsigned)HB * WB, units = (unsigned)a.N * per_image;
    for (int round = 0; round < a.rounds; ++round) {
      const unsigned u = (blockIdx.y * (unsigned)a.rounds + round) * 32u + rl;
      if (u >= units) break;
      const unsigned n = u / per_image, p = u - n * per_image;
      const int hb = p / WB, wb = p - hb * WB;
      const size_t out0 = (size_t)n * a.Hd * a.Wd * C + cg * 8;
      uint4 gt[2][2], bx[2][2];
      if (DGRAD) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int h = 2 * hb + (i >> 1), w = 2 * wb + (i & 1);
          const size_t o = out0 + ((size_t)(h < a.Hd ? h : 0) * a.Wd + (w < a.Wd ? w : 0)) * C;
          gt[i >> 1][i & 1] = *reinterpret_cast<const uint4*>(a.gate + o);
          bx[i >> 1][i & 1] = *reinterpret_cast<const uint4*>(a.bnx + o);
        }
      }
      float acc[2][2][8];
      const bf16_t* img = a.src + (size_t)n * a.Hs * a.Ws * C + cg * 8;
      if constexpr (DGRAD && S == 2) dw_dgrad2_cells(img, k, hb, wb, a.Hs, a.Ws, C, acc);
      else dw_cells<S, DGRAD>(img, k, 2 * S * hb - 1, 2 * S * wb - 1, a.Hs, a.Ws, C, acc);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int h = 2 * hb + (i >> 1), w = 2 * wb + (i & 1);
        if (h >= a.Hd || w >= a.Wd) continue;
        const size_t o = out0 + ((size_t)h * a.Wd + w) * C;
        float (&f)[8] = acc[i >> 1][i & 1];
        if (DGRAD) {
          float g[8], x[8];
          unpack(gt[i >> 1][i & 1], g);
          unpack(bx[i >> 1][i & 1], x);
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            if (!(g[j] > 0.f) || g[j] >= a.gate_hi) f[j] = 0.f;
            s1[j] += f[j];
            s2[j] += f[j] * (x[j] - mu[j]);
          }
          store_f32(a.dx + o, f);
        } else {
          const uint4 packed = pack(f);
          *reinterpret_cast<uint4*>(a.y + o) = packed;
          unpack(packed, f);
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            s1[j] += f[j];
            s2[j] += f[j] * f[j];
          }
        }
      }
    }
  }
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    red[0][rl][cgl * 8 + j] = s1[j];
    red[1][rl][cgl * 8 + j] = s2[j];
  }
  __syncthreads();
  const int which = threadIdx.x >> 6, c = blockIdx.x * 64 + (threadIdx.x & 63);
  if (which < 2 && c < C) {
    auto total = [&](int w) {
      float t = 0.f;
#pragma unroll
      for (int r = 0; r < 32; ++r) t += red[w][r][threadIdx.x & 63];
      return t;
    };
    double t = total(which);
    if (DGRAD && which == 1 && a.bnx_sums) t += (double)centre[threadIdx.x & 63] * total(0);
    stat_add(a.sums + (size_t)((blockIdx.x + blockIdx.y) % kStatReplicas) * a.rep_stride, C, which, c, t);
  }
}

// Weight gradient, first pass: workgroup (channel block bx of 8 groups of 8 channels, chunk by) adds dy * x for all nine taps
// over its share of the output rows, cut into segments of kDwSegment cells.  One of 32 lanes per channel group walks a segment
// with the three columns of x in registers, so that a step loads and unpacks one new column (two at stride 2) and one cell of
// dy.  The 72 sums of a lane are added over the eight lanes of a wave that share its channels by halves (lanes exchange the
// half they do not keep: 63 shuffles instead of 216, or of 9 rounds through LDS), over the four waves through LDS, and go to
// part[by][tap][c]; second pass: dw[c][tap] = sum over chunks.  All orders are fixed.  Products with cells outside the image or
// past the end of a row are left out, not added as zeros (an infinity on the other side would make them NaN).
// 128 x 16 x 16 x 384, stride 1, both passes: 67.0 -> 17.1 us (50 MB); 128 x 32 x 32 x 192, stride 2: 69.1 -> 17.8 us.
constexpr int kDwSegment = 8;
template <int S>
__global__ __launch_bounds__(256) void dwconv3_wgrad_kernel(const bf16_t* __restrict__ x, const bf16_t* __restrict__ dy,
                                                            float* __restrict__ part, int N, int H, int W, int C, int Ho, int Wo,
                                                            int units_per_chunk) {
  __shared__ float red[4][9 * 64];
  const int CG = C / 8;
  const int cgl = threadIdx.x & 7, pl = threadIdx.x >> 3, lane = threadIdx.x & 63;
  const int cg = blockIdx.x * 8 + cgl;
  const int segs = (Wo + kDwSegment - 1) / kDwSegment;
  const size_t units = (size_t)N * Ho * segs;
  const size_t u_lo = (size_t)blockIdx.y * units_per_chunk;
  const size_t u_hi = u_lo + units_per_chunk < units ? u_lo + units_per_chunk : units;
  float acc[72];
#pragma unroll
  for (int t = 0; t < 72; ++t) acc[t] = 0.f;
  if (cg < CG) {
    for (size_t u = u_lo + pl; u < u_hi; u += 32) {
      const unsigned row = (unsigned)(u / segs), seg = (unsigned)(u % segs), n = row / Ho, ho = row % Ho;
      const int w_lo = (int)seg * kDwSegment, h0 = (int)ho * S - 1;
      const bf16_t* img = x + (size_t)n * H * W * C + cg * 8;
      const bf16_t* out = dy + ((size_t)row * Wo + w_lo) * C + cg * 8;
      auto cell = [&](int r, int w) {
        const int h = h0 + r;
        uint4 v = make_uint4(0u, 0u, 0u, 0u);
        if (h >= 0 && h < H && w >= 0 && w < W) v = *reinterpret_cast<const uint4*>(img + ((size_t)h * W + w) * C);
        return v;
      };
      float f[3][3][8];   // [column][row]
      uint4 first_columns[3 - S][3];
#pragma unroll
      for (int q = 0; q < 3 - S; ++q)
#pragma unroll
        for (int r = 0; r < 3; ++r) first_columns[q][r] = cell(r, w_lo * S - 1 + q);
      // the loads of AHEAD steps before their sums: across the branches below the compiler moves none.  At unit stride a second
      // step ahead costs the third wave of a SIMD (128 x 16 x 16 x 384: 17.1 -> 22.7 us)
      constexpr int AHEAD = S;
      uint4 gv[AHEAD], nv[AHEAD][S][3];
#pragma unroll
      for (int i = 0; i < kDwSegment; ++i) {
        const int wo = w_lo + i, slot = i % AHEAD;
        if (slot == 0) {
          if (wo >= Wo) break;
#pragma unroll
          for (int k = 0; k < AHEAD; ++k) {
            gv[k] = make_uint4(0u, 0u, 0u, 0u);
            if (wo + k < Wo) gv[k] = *reinterpret_cast<const uint4*>(out + (size_t)(i + k) * C);
#pragma unroll
            for (int q = 0; q < S; ++q)
#pragma unroll
              for (int r = 0; r < 3; ++r) nv[k][q][r] = cell(r, (wo + k) * S + 2 - S + q);
          }
        }
        if (i == 0) {
#pragma unroll
          for (int q = 0; q < 3 - S; ++q)
#pragma unroll
            for (int r = 0; r < 3; ++r) unpack(first_columns[q][r], f[q][r]);
        }
        float g[8];
        unpack(gv[slot], g);
#pragma unroll
        for (int q = 0; q < S; ++q)
#pragma unroll
          for (int r = 0; r < 3; ++r) unpack(nv[slot][q][r], f[3 - S + q][r]);
#pragma unroll
        for (int q = 0; q < 3; ++q) {
          const int w = wo * S - 1 + q;
          if (wo >= Wo || w < 0 || w >= W) continue;
#pragma unroll
          for (int r = 0; r < 3; ++r) {
            if (h0 + r < 0 || h0 + r >= H) continue;
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[(r * 3 + q) * 8 + j] += g[j] * f[q][r][j];
          }
        }
#pragma unroll
        for (int q = 0; q < 3 - S; ++q)
#pragma unroll
          for (int r = 0; r < 3; ++r)
#pragma unroll
            for (int j = 0; j < 8; ++j) f[q][r][j] = f[q + S][r][j];
      }
    }
  }
  // halves: after the three steps a lane holds sums first .. first + 8 of its channel group, over the wave
  int first = 0;
#pragma unroll
  for (int step = 0; step < 3; ++step) {
    const int half = 36 >> step, bit = 32 >> step;
    const bool upper = (lane & bit) != 0;
#pragma unroll
    for (int t = 0; t < 36; ++t) {
      if (t >= half) break;
      const float keep = upper ? acc[half + t] : acc[t], give = upper ? acc[t] : acc[half + t];
      acc[t] = keep + __shfl_xor(give, bit, 64);
    }
    if (upper) first += half;
  }
#pragma unroll
  for (int t = 0; t < 9; ++t) {
    const int e = first + t;   // tap * 8 + channel of the group
    red[threadIdx.x >> 6][(e >> 3) * 64 + cgl * 8 + (e & 7)] = acc[t];
  }
  __syncthreads();
  for (int e = threadIdx.x; e < 9 * 64; e += 256) {
    const int c = blockIdx.x * 64 + (e & 63);
    if (c < C) part[((size_t)blockIdx.y * 9 + (e >> 6)) * C + c] = (red[0][e] + red[1][e]) + (red[2][e] + red[3][e]);
  }
}
// 32 (tap, channel) sums per workgroup, the chunks dealt to 8 thread groups with independent loads (one thread per sum walked
// up to 1024 chunks one after the other)
__global__ __launch_bounds__(256) void dwconv3_wgrad_reduce_kernel(const float* __restrict__ part, float* __restrict__ dw, int C,
                                                                   int chunks) {
  __shared__ float red[8][32];
  const int l = threadIdx.x & 31, ph = threadIdx.x >> 5;
  const int i = blockIdx.x * 32 + l;   // (tap, c)
  float s = 0.f;
  if (i < 9 * C) {
#pragma unroll 8
    for (int k = ph; k < chunks; k += 8) s += part[(size_t)k * 9 * C + i];
  }
  red[ph][l] = s;
  __syncthreads();
  if (ph != 0 || i >= 9 * C) return;
  s = ((red[0][l] + red[1][l]) + (red[2][l] + red[3][l])) + ((red[4][l] + red[5][l]) + (red[6][l] + red[7][l]));
  dw[(size_t)(i % C) * 9 + i / C] = s;
}

// Segments of the weight gradient's rows, and the chunks they are dealt to: one segment to a lane (32 to a workgroup) up to about
// 1024 workgroups.  With less scratch the chunks are longer: any scratch for a chunk per 256 cells does.
size_t dw_units(int N, int Ho, int Wo) { return (size_t)N * Ho * ((Wo + kDwSegment - 1) / kDwSegment); }
size_t dw_most_chunks(int C) { const size_t cblocks = (C / 8 + 7) / 8; return (1024 + cblocks - 1) / cblocks; }
size_t dw_chunks(int N, int Ho, int Wo, int C) { return std::min((dw_units(N, Ho, Wo) + 31) / 32, dw_most_chunks(C)); }
size_t dw_least_chunks(int N, int Ho, int Wo, int C) { return std::min(((size_t)N * Ho * Wo + 255) / 256, dw_most_chunks(C)); }

}  // namespace

hipError_t launch_im2col7(const bf16_t* x8, bf16_t* col, int N, int H, int W, hipStream_t s) {
  if (N <= 0 || H <= 0 || W <= 0) return hipErrorInvalidValue;
  const int Ho = (H - 1) / 2 + 1, Wo = (W - 1) / 2 + 1;
  const size_t total = (size_t)N * Ho * Wo * 56;
  if (total >= ((size_t)1 << 31) * 256) return hipErrorInvalidValue;
  hipLaunchKernelGGL(im2col7_kernel, dim3(grid_for(total)), dim3(256), 0, s, reinterpret_cast<const uint4*>(x8),
                     reinterpret_cast<uint4*>(col), N, H, W, Ho, Wo);
  return hipGetLastError();
}

hipError_t launch_maxpool3s2(const bf16_t* x, float* y_f32, bf16_t* y_b16, int N, int H, int W, int C, hipStream_t s) {
  if (N <= 0 || H <= 0 || W <= 0 || C <= 0 || C % 8 != 0 || (!y_f32 && !y_b16)) return hipErrorInvalidValue;
  const int Ho = (H - 1) / 2 + 1, Wo = (W - 1) / 2 + 1;
  hipLaunchKernelGGL(maxpool3s2_kernel, dim3(grid_for((size_t)N * Ho * Wo * (C / 8))), dim3(256), 0, s, x, y_f32, y_b16, N, H, W, C, Ho, Wo);
  return hipGetLastError();
}

hipError_t launch_maxpool3s2_bwd(const bf16_t* x, const float* dy, float* dx, int N, int H, int W, int C, hipStream_t s) {
  if (N <= 0 || H <= 0 || W <= 0 || C <= 0 || C % 8 != 0) return hipErrorInvalidValue;
  const int Ho = (H - 1) / 2 + 1, Wo = (W - 1) / 2 + 1;
  hipLaunchKernelGGL(maxpool3s2_bwd_kernel, dim3(grid_for((size_t)N * H * W * (C / 8))), dim3(256), 0, s, x, dy, dx, N, H, W, C, Ho, Wo);
  return hipGetLastError();
}

// workgroups of the kernels that make 2 x 2 cells of 8 channels a thread; 0 where they do not fit a grid
static unsigned dw_blocks_per_image(int N, int Ho, int Wo, int C) {
  const size_t b = ((size_t)((Ho + 1) / 2) * ((Wo + 1) / 2) * (C / 8) + 255) / 256;
  return b * N < ((size_t)1 << 31) && b < ((size_t)1 << 23) ? (unsigned)b : 0;
}

hipError_t launch_dwconv3_fwd(const bf16_t* x, const bf16_t* wt, bf16_t* y, int N, int H, int W, int C, int stride, hipStream_t s) {
  if (N <= 0 || H <= 0 || W <= 0 || C <= 0 || C % 8 != 0 || (stride != 1 && stride != 2)) return hipErrorInvalidValue;
  const int Ho = (H - 1) / stride + 1, Wo = (W - 1) / stride + 1;
  const unsigned bpi = dw_blocks_per_image(N, Ho, Wo, C);
  if (!bpi) return hipErrorInvalidValue;
  if (stride == 1)
    hipLaunchKernelGGL((dwconv3_kernel<1, false>), dim3(bpi * N), dim3(256), 0, s, x, wt, y, H, W, C, Ho, Wo, (int)bpi);
  else
    hipLaunchKernelGGL((dwconv3_kernel<2, false>), dim3(bpi * N), dim3(256), 0, s, x, wt, y, H, W, C, Ho, Wo, (int)bpi);
  return hipGetLastError();
}

hipError_t launch_dwconv3_dgrad(const bf16_t* dy, const bf16_t* wt, bf16_t* dx, int N, int H, int W, int C, int stride, hipStream_t s) {
  if (N <= 0 || H <= 0 || W <= 0 || C <= 0 || C % 8 != 0 || (stride != 1 && stride != 2) || !dx) return hipErrorInvalidValue;
  const int Ho = (H - 1) / stride + 1, Wo = (W - 1) / stride + 1;
  const unsigned bpi = dw_blocks_per_image(N, H, W, C);
  if (!bpi) return hipErrorInvalidValue;
  if (stride == 1)
    hipLaunchKernelGGL((dwconv3_kernel<1, true>), dim3(bpi * N), dim3(256), 0, s, dy, wt, dx, Ho, Wo, C, H, W, (int)bpi);
  else
    hipLaunchKernelGGL(dwconv3_dgrad2_kernel, dim3(bpi * N), dim3(256), 0, s, dy, wt, dx, H, W, C, Ho, Wo, (int)bpi);
  return hipGetLastError();
}

// rounds so that about 1024 workgroups are left, and the sums of a channel get at most as many partials as one array holds
static hipError_t launch_dw_sums(DwSums a, int stride, bool dgrad, hipStream_t s) {
  const size_t units = (size_t)a.N * ((a.Hd + 1) / 2) * ((a.Wd + 1) / 2), cblocks = (a.C / 8 + 7) / 8, blocks = (units + 31) / 32;
  if (units >= ((size_t)1 << 31)) return hipErrorInvalidValue;
  a.rounds = (int)std::max<size_t>(1, (blocks * cblocks + 512) / 1024);
  const dim3 grid((unsigned)cblocks, (unsigned)((blocks + a.rounds - 1) / a.rounds));
  if (dgrad) {
    if (stride == 1) hipLaunchKernelGGL((dwconv3_sums_kernel<1, true>), grid, dim3(256), 0, s, a);
    else hipLaunchKernelGGL((dwconv3_sums_kernel<2, true>), grid, dim3(256), 0, s, a);
  } else {
    if (stride == 1) hipLaunchKernelGGL((dwconv3_sums_kernel<1, false>), grid, dim3(256), 0, s, a);
    else hipLaunchKernelGGL((dwconv3_sums_kernel<2, false>), grid, dim3(256), 0, s, a);
  }
  return hipGetLastError();
}

hipError_t launch_dwconv3_fwd_sums(const bf16_t* x, const bf16_t* wt, bf16_t* y, stat_t* sums, int rep_stride, int N, int H, int W, int C,
                                   int stride, hipStream_t s) {
  if (N <= 0 || H <= 0 || W <= 0 || C <= 0 || C % 8 != 0 || (stride != 1 && stride != 2) || !x || !wt || !y || !sums) return hipErrorInvalidValue;
  DwSums a{};
  a.src = x; a.wt = wt; a.y = y; a.sums = sums; a.rep_stride = rep_stride;
  a.N = N; a.Hs = H; a.Ws = W; a.C = C; a.Hd = (H - 1) / stride + 1; a.Wd = (W - 1) / stride + 1;
  return launch_dw_sums(a, stride, false, s);
}

hipError_t launch_dwconv3_dgrad_sums(const bf16_t* dy, const bf16_t* wt, const bf16_t* gate, float gate_hi, const bf16_t* bnx,
                                     const stat_t* bnx_sums, float* dx, stat_t* sums, int rep_stride, int N, int H, int W, int C, int stride, hipStream_t s) {
  if (N <= 0 || H <= 0 || W <= 0 || C <= 0 || C % 8 != 0 || (stride != 1 && stride != 2) || !dy || !wt || !gate || !bnx || !dx || !sums)
    return hipErrorInvalidValue;
  DwSums a{};
  a.src = dy; a.wt = wt; a.dx = dx; a.gate = gate; a.gate_hi = gate_hi; a.bnx = bnx; a.bnx_sums = bnx_sums; a.sums = sums; a.rep_stride = rep_stride;
  a.N = N; a.Hs = (H - 1) / stride + 1; a.Ws = (W - 1) / stride + 1; a.C = C; a.Hd = H; a.Wd = W;
  return launch_dw_sums(a, stride, true, s);
}

size_t dwconv3_wgrad_scratch_bytes(int N, int H, int W, int C, int stride) {
  if (N <= 0 || H <= 0 || W <= 0 || C <= 0 || C % 8 != 0 || (stride != 1 && stride != 2)) return 0;
  const int Ho = (H - 1) / stride + 1, Wo = (W - 1) / stride + 1;
  return dw_chunks(N, Ho, Wo, C) * 9 * C * sizeof(float);
}

hipError_t launch_dwconv3_wgrad(const bf16_t* x, const bf16_t* dy, float* dw, float* scratch, size_t scratch_bytes, int N, int H, int W,
                                int C, int stride, hipStream_t s) {
  if (!dwconv3_wgrad_scratch_bytes(N, H, W, C, stride) || !scratch) return hipErrorInvalidValue;
  const int Ho = (H - 1) / stride + 1, Wo = (W - 1) / stride + 1;
  const size_t room = scratch_bytes / ((size_t)9 * C * sizeof(float));
  if (room < dw_least_chunks(N, Ho, Wo, C)) return hipErrorInvalidValue;
  const size_t units = dw_units(N, Ho, Wo);
  if (units >= ((size_t)1 << 32)) return hipErrorInvalidValue;
  int chunks = (int)std::min(dw_chunks(N, Ho, Wo, C), room);
  const int per = (int)((units + chunks - 1) / chunks);
  chunks = (int)((units + per - 1) / per);
  const dim3 grid((C / 8 + 7) / 8, chunks);
  if (stride == 1) hipLaunchKernelGGL(dwconv3_wgrad_kernel<1>, grid, dim3(256), 0, s, x, dy, scratch, N, H, W, C, Ho, Wo, per);
  else hipLaunchKernelGGL(dwconv3_wgrad_kernel<2>, grid, dim3(256), 0, s, x, dy, scratch, N, H, W, C, Ho, Wo, per);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(dwconv3_wgrad_reduce_kernel, dim3((9 * C + 31) / 32), dim3(256), 0, s, scratch, dw, C, chunks);
  return hipGetLastError();
}

}  // namespace fdg
