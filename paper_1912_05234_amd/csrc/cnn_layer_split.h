// Convolution calls for the shape of the network's second convolution (six input and twelve output maps, 5 x 5 kernel,
// 12 x 12 input) on many images: one wave per image, as products of bfloat16 pieces (cnn_split.h), eight waves and
// one workgroup per compute unit.  Definitions: arXiv 1912.05234, Section 3 (conv / mconv, backweights, backbias, backin).
// The fp32 forms (cnn_conv_wave.h, cnn_col2im.h) issue 152, 160 and 120 instructions of 32 clocks per image, 2.1, 2.2
// and 1.6 us of a SIMD.  Measured, in us for 10000 (60000) images: forward 32 (148) before, 22.5 (105) now; weight gradient
// 32 (163), 26 (124); input gradient 32 (167), 27 (137).  About 5 us of each are the start (launch, weights, first loads); then
// an image costs twice the time of its matrix instructions, whose issue and the vector instructions' exclude each other in
// part.  Three waves per SIMD gained 3 (forward) and 10 us (input gradient) of 60000 images and lost as much at 10000.
#pragma once

#include "cnn_conv_wave.h"
#include "cnn_split.h"

namespace cnn {
namespace conv2_split {

constexpr int WAVES = 8, THREADS = 64 * WAVES, NK2 = 1800;

// The wave's image as S1 of the fused step: pieces, channels last, both copies.  Lane l < 36 has four pixels of all six
// channels, 48 bytes of a plane: written in items of 16 bytes, and of 4 and 16 in the second copy, which lies an odd number
// of words further.
struct Planes {
  f4 v[6];
  __device__ __forceinline__ void load(const float* __restrict__ in, size_t n) {
    const int l = threadIdx.x & 63;
    if (l < 36)
#pragma unroll
      for (int c = 0; c < 6; ++c) v[c] = reinterpret_cast<const f4*>(in + n * NS1)[36 * c + l];
  }
};
__device__ __forceinline__ void store_planes(unsigned* s1, const Planes& x) {
  const int l = threadIdx.x & 63;
  if (l >= 36) return;
  unsigned w[3][12];  // pixel 0: channels 01, 23, 45, then pixel 1, ..
#pragma unroll
  for (int i = 0; i < 12; ++i) {
    const Split2 a = split2(x.v[2 * (i % 3)][i / 3], x.v[2 * (i % 3) + 1][i / 3]);
    w[0][i] = a.h, w[1][i] = a.m, w[2][i] = a.l;
  }
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    unsigned* to = s1 + j * SPLIT_S1_PLANE + 12 * l;
#pragma unroll
    for (int i = 0; i < 3; ++i) reinterpret_cast<u4v*>(to)[i] = u4v{w[j][4 * i], w[j][4 * i + 1], w[j][4 * i + 2], w[j][4 * i + 3]};
    to += SPLIT_S1B;
    constexpr int HEAD = (4 - SPLIT_S1B % 4) % 4;
#pragma unroll
    for (int i = 0; i < HEAD; ++i) to[i] = w[j][i];
#pragma unroll
    for (int i = HEAD; i + 4 <= 12; i += 4) *reinterpret_cast<u4v*>(to + i) = u4v{w[j][i], w[j][i + 1], w[j][i + 2], w[j][i + 3]};
#pragma unroll
    for (int i = 12 - (12 - HEAD) % 4; i < 12; ++i) to[i] = w[j][i];
  }
}
// The words behind the planes are read by the last items and meet zero weights.
__device__ __forceinline__ void pad_planes(unsigned* s1) {
  const int l = threadIdx.x & 63;
  if (l < 4) s1[3 * SPLIT_S1_PLANE + l] = s1[SPLIT_S1B + 3 * SPLIT_S1_PLANE + l] = 0;
}

// ---- forward ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(THREADS) void forward_kernel(const float* __restrict__ in, const float* __restrict__ k,
                                                          const float* __restrict__ bias, float* __restrict__ out, int B) {
  __shared__ u4v items[SPLIT_C2_ITEMS];
  __shared__ __align__(16) unsigned planes[WAVES][SPLIT_S1_WORDS];
  const Share<WAVES, 1> mine;
  const int t = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(t >> 6), l = t & 63, q = l >> 4, n16 = l & 15;
  StagedLoad<THREADS, NK2> weights;
  weights.fetch(k);
  Planes cur;
  if (mine.first < (size_t)B) cur.load(in, mine.first);
  weights.commit(reinterpret_cast<float*>(planes));
  __syncthreads();
  if (t < C2_TASKS) make_c2_items(items - SPLIT_C1_ITEMS, t, reinterpret_cast<const float*>(planes), 1.0f);
  __syncthreads();
  pad_planes(planes[wave]);
  const C2SLane ln = c2s_lane(planes[wave], items - SPLIT_C1_ITEMS, l);
  const float b = bias ? bias[n16 < 12 ? n16 : 0] : 0.0f;
  for (size_t n = mine.first; n < (size_t)B; n += mine.step) {
    store_planes(planes[wave], cur);
    wave_sync();
    if (n + mine.step < (size_t)B) cur.load(in, n + mine.step);  // in flight during this image
    f4 acc[4];
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) acc[mt] = f4{b, b, b, b};
    c2s_gemm(acc, ln);
    wave_sync();
    // register r of tile mt is pixel (y, x) = (2 mt + r / 2, 2 q + r % 2) of map n16: two 8-byte stores per tile
    if (n16 < 12) {
      float* dst = out + n * NC2 + n16 * 64 + 2 * q;
#pragma unroll
      for (int mt = 0; mt < 4; ++mt) {
        *reinterpret_cast<float2*>(dst + 16 * mt) = float2{acc[mt][0], acc[mt][1]};
        *reinterpret_cast<float2*>(dst + 16 * mt + 8) = float2{acc[mt][2], acc[mt][3]};
      }
    }
  }
}

// d_out of image n in the result layout: lane (q, n16) holds map n16's window 4 q of the four tiles (padding lanes: map 11's).
__device__ __forceinline__ void load_error(const float* __restrict__ d_out, size_t n, f4 (&d)[4]) {
  const int l = threadIdx.x & 63, q = l >> 4, n16 = l & 15;
  const float* src = d_out + n * NC2 + (n16 < 12 ? n16 : 11) * 64 + 2 * q;
#pragma unroll
  for (int mt = 0; mt < 4; ++mt) {
    const float2 lo = *reinterpret_cast<const float2*>(src + 16 * mt), hi = *reinterpret_cast<const float2*>(src + 16 * mt + 8);
    d[mt] = f4{lo.x, lo.y, hi.x, hi.y};
  }
}
__device__ __forceinline__ void cut_error(const f4 (&d)[4], float sign, u4v (&d2)[2][3]) {
#pragma unroll
  for (int mt = 0; mt < 4; ++mt)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const Split2 p = split2(sign * d[mt][2 * h], sign * d[mt][2 * h + 1]);
      d2[mt >> 1][0][2 * (mt & 1) + h] = p.h;
      d2[mt >> 1][1][2 * (mt & 1) + h] = p.m;
      d2[mt >> 1][2][2 * (mt & 1) + h] = p.l;
    }
}

// ---- weight and bias gradient -------------------------------------------------------------------------------
// part: [gridDim.x][10 tiles][16 rows j][16 taps] then the bias rows [gridDim.x][16], as igemm::wgrad_reduce_kernel reads them.
constexpr int ACC_FLOATS = 10 * 4 * 64;  // a wave's sums
static_assert(4 * ACC_FLOATS <= WAVES * SPLIT_S1_WORDS, "the waves' sums meet over the planes");
__global__ __launch_bounds__(THREADS) void bwd_weight_kernel(
    const float* __restrict__ in, const float* __restrict__ d_out, float* __restrict__ part, int B) {
  __shared__ __align__(16) unsigned planes[WAVES][SPLIT_S1_WORDS];
  __shared__ float bsum[WAVES][64];
  const Share<WAVES, 1> mine;
  const int t = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(t >> 6), l = t & 63, q = l >> 4, n16 = l & 15;
  const float sign = wave & 1 ? -1.0f : 1.0f;  // (cnn_train.h, wave_image)
  f4 acc[10];
#pragma unroll
  for (int i = 0; i < 10; ++i) acc[i] = f4{0.0f, 0.0f, 0.0f, 0.0f};
  float g_b = 0.0f, g_eight = 0.0f;  // the bias's sum, eight images at a time: a chain over all of a wave's was less exact than before
  int images = 0;
  Planes cur;
  f4 d[4];
  if (mine.first < (size_t)B) {
    cur.load(in, mine.first);
    load_error(d_out, mine.first, d);
  }
  pad_planes(planes[wave]);
  for (size_t n = mine.first; n < (size_t)B; n += mine.step) {
    store_planes(planes[wave], cur);
    u4v d2[2][3];
    cut_error(d, sign, d2);
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) g_eight += (d[mt][0] + d[mt][1]) + (d[mt][2] + d[mt][3]);
    if ((++images & 7) == 0) {
      g_b += g_eight;
      g_eight = 0.0f;
    }
    wave_sync();
    if (n + mine.step < (size_t)B) {  // in flight during this image
      cur.load(in, n + mine.step);
      load_error(d_out, n + mine.step, d);
    }
    k2_gradient(acc, d2, planes[wave], l);
    wave_sync();
  }
#pragma unroll
  for (int i = 0; i < 10; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[i][r] *= sign;
  // the waves' sums in a fixed order, the upper half to the lower: (w, w + 4), then (w, w + 2), then (0, 1)
  bsum[wave][l] = g_b + g_eight;
  float* comb = reinterpret_cast<float*>(planes);
#pragma unroll
  for (int half = WAVES / 2; half >= 1; half >>= 1) {
    __syncthreads();
    if (wave >= half && wave < 2 * half) {
      float* dst = comb + (wave - half) * ACC_FLOATS;
#pragma unroll
      for (int i = 0; i < 10; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) dst[(4 * i + r) * 64 + l] = acc[i][r];
    }
    __syncthreads();
    if (wave < half) {
      const float* src = comb + wave * ACC_FLOATS;
#pragma unroll
      for (int i = 0; i < 10; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[i][r] += src[(4 * i + r) * 64 + l];
    }
  }
  if (wave == 0) {
    // tile 2 u + t, column n16 is element kk = 16 t + n16 = 6 v + c of kernel row u: tap 25 c + 5 u + v; row j = 4 q + r
    float* tile = part + (size_t)blockIdx.x * 10 * 256 + 64 * q;
#pragma unroll
    for (int tt = 0; tt < 2; ++tt) {
      const int kk = 16 * tt + n16;
      if (kk < 30) {
#pragma unroll
        for (int u = 0; u < 5; ++u) {
          const int tap = 25 * (kk % 6) + 5 * u + kk / 6;
#pragma unroll
          for (int r = 0; r < 4; ++r) tile[(tap >> 4) * 256 + 16 * r + (tap & 15)] = acc[2 * u + tt][r];
        }
      }
    }
  } else if (wave == 1 && l < 16) {
    float s = 0.0f;
    if (l < 12)
      for (int w = 0; w < WAVES; ++w) s += (bsum[w][l] + bsum[w][l + 16]) + (bsum[w][l + 32] + bsum[w][l + 48]);
    part[(size_t)gridDim.x * 10 * 256 + (size_t)blockIdx.x * 16 + l] = s;
  }
}

// ---- input gradient ---------------------------------------------------------------------------------------------
constexpr int REC_WORDS = 64 * BWD_REC / 2;
static_assert(6 * DS1_MAP <= REC_WORDS && DS1_MAP % 4 == 0, "the result lies over the records");
__global__ __launch_bounds__(THREADS) void bwd_input_kernel(const float* __restrict__ d_out, const float* __restrict__ k,
                                                            float* __restrict__ d_in, int B) {
  __shared__ __align__(16) unsigned short rows[BWD_TILES * 16 * BWD_REC];
  __shared__ __align__(16) float lds[WAVES][REC_WORDS];
  const Share<WAVES, 1> mine;
  const int t = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(t >> 6), l = t & 63;
  StagedLoad<THREADS, NK2> weights;
  weights.fetch(k);
  f4 d[4];
  if (mine.first < (size_t)B) load_error(d_out, mine.first, d);
  weights.commit(&lds[0][0]);
  __syncthreads();
  if (t < BWD_TASKS) make_bwd_record(rows, t, &lds[0][0], 1.0f);
  __syncthreads();
  float* acc = lds[wave];
  // the 216 fours of an image: where they lie in d_in [6][12][DS1_ROW]
  int at[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int e = i < 3 || l < 24 ? l + 64 * i : l, row = e / 3, c = row / 12;
    at[i] = c * DS1_MAP + (row - 12 * c) * DS1_ROW + 4 * (e - 3 * row);
  }
  for (size_t n = mine.first; n < (size_t)B; n += mine.step) {
    u4v d2[2][3];
    cut_error(d, 1.0f, d2);
    store_records(reinterpret_cast<unsigned short*>(acc), d2, l);
    wave_sync();
    if (n + mine.step < (size_t)B) load_error(d_out, n + mine.step, d);  // in flight during this image
    col2im_split(rows, reinterpret_cast<const unsigned short*>(acc), acc, 1.0f, l);
    wave_sync();
    f4* dst = reinterpret_cast<f4*>(d_in + n * NS1);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const f4 v = *reinterpret_cast<const f4*>(acc + at[i]);
      if (i < 3 || l < 24) dst[l + 64 * i] = v;
    }
    wave_sync();
  }
}

}  // namespace conv2_split
}  // namespace cnn
