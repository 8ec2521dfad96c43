// What the implicit-GEMM convolution kernels share: matrix instruction, index arithmetic, LDS barrier, and the
// second kernel of the weight gradients that leave partial 16 x 16 tiles (cnn_conv_wave.h, cnn_fc_wave.h).  Definitions: arXiv 1912.05234, Section 3 -- listings conv / mconv (forward), backin (input
// gradient), backweights and backbias (weight and bias gradients).
//
// Every operation is an implicit GEMM D[M x N] = A[M x K] * B[K x N] in 16 x 16 tiles; with
// v_mfma_f32_16x16x4_f32 lane l = 16 q + j of a wave supplies A[i = j][k = q] and B[k = q][j] and
// receives D[i = 4 q + r][j] in result register r.
//
// Column packing (layers with few output channels): P horizontally adjacent output
// pixels x = P X + sh share one GEMM column (y, X) and take P rows (m, sh) instead.  With v' = v + sh
// the gathered operand staged[c][y+u][P X + v'] does not depend on sh, so
//   D[(m,sh)][(y,X)] = sum_{c,u,v' < KW+P-1} W[(m,sh)][(c,u,v')] * staged[c][y+u][P X + v'],
//   W[(m,sh)][(c,u,v')] = k[m][c][u][v'-sh]  (zero where v'-sh is outside 0..KW-1):
// a 16-row tile is filled by M*P rows and the number of matrix instructions falls by
// P*KW / (KW+P-1).  P = 1 is the plain form.
#pragma once

#include "cnn_common.h"

namespace cnn {
namespace igemm {

using f4 = float __attribute__((ext_vector_type(4)));
using f2 = float __attribute__((ext_vector_type(2)));
using i4 = int __attribute__((ext_vector_type(4)));
__device__ __forceinline__ f4 mfma16(float a, float b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

constexpr int THREADS = 256;  // four waves per workgroup
constexpr int WAVES = THREADS / 64;

// Workgroup barrier that orders LDS accesses only: global loads and stores stay in flight across it.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// e / d and e % d for 0 <= e < 2^22, d >= 1, inv = 1.0f / d: the float estimate is off by at most
// one and is corrected.
__device__ __forceinline__ void divmod(int e, int d, float inv, int& quo, int& rem) {
  int qv = (int)((float)e * inv);
  int rv = e - qv * d;
  if (rv < 0) {
    --qv;
    rv += d;
  } else if (rv >= d) {
    ++qv;
    rv -= d;
  }
  quo = qv;
  rem = rv;
}
__host__ __device__ inline int round4(int v) { return (v + 3) & ~3; }
// Row stride (floats) of a table read 16 bytes per lane with one row per lane: a multiple of 4 that
// is not a multiple of 8, so that eight consecutive rows start in eight different groups of four banks.
__host__ __device__ inline int row_stride(int blocks) { return 4 * blocks + ((blocks & 1) ? 0 : 4); }

// d_k[co][ci][u][v] = sum over the GP partial tiles and the P shifts of T[(co,sh)][(ci,u,v+sh)], at most sixteen rows (co,sh);
// d_bias[co] = sum over the GP partial bias rows and the P shifts.  A workgroup takes EPW outputs (few outputs are spread
// over more workgroups); THREADS / EPW interleaved strands walk the partials in ascending order, sixteen loads in
// flight (the walk is bound by load latency), and are combined by a fixed tree, those of a wave between its lanes (a barrier per
// level and the P shifts one after the other: first two layers of 100 images 3.9, now 3.3 us, of 10000 images 5.6, now 5.3).
template <int EPW, int P>
__global__ __launch_bounds__(THREADS) void wgrad_reduce_kernel(const float* __restrict__ part, int GP, int NT, int Cout, int Cin,
                                                               int KH, int KW, float* __restrict__ d_k,
                                                               float* __restrict__ d_bias) {
  constexpr int STRANDS = THREADS / EPW, DEEP = 16 / P;
  __shared__ float red[WAVES][EPW];
  const int t = threadIdx.x, strand = t / EPW, el = blockIdx.x * EPW + t % EPW;
  const int KWP = KW + P - 1, nk = Cout * Cin * KH * KW, total = nk + (d_bias ? Cout : 0);
  float sum = 0.0f;
  if (el < total) {
    const float* p[P];
    size_t stride;
#pragma unroll
    for (int sh = 0; sh < P; ++sh) {
      if (el < nk) {
        const int v = el % KW, cu = (el / KW) % (Cin * KH), co = el / (KW * Cin * KH);
        const int row = co * P + sh, col = cu * KWP + v + sh;
        p[sh] = part + (size_t)(col >> 4) * 256 + row * 16 + (col & 15);
        stride = (size_t)NT * 256;
      } else {
        p[sh] = part + (size_t)GP * NT * 256 + (size_t)(el - nk) * P + sh;
        stride = 16;
      }
    }
    for (int g = strand; g < GP; g += DEEP * STRANDS) {
      float v[DEEP][P];
#pragma unroll
      for (int k = 0; k < DEEP; ++k)
#pragma unroll
        for (int sh = 0; sh < P; ++sh) v[k][sh] = g + k * STRANDS < GP ? p[sh][(g + k * STRANDS) * stride] : 0.0f;
#pragma unroll
      for (int k = 0; k < DEEP; ++k)
#pragma unroll
        for (int sh = 0; sh < P; ++sh) sum += v[k][sh];
    }
  }
#pragma unroll
  for (int s = EPW; s < 64; s *= 2) sum += __shfl_xor(sum, s);
  if ((t & 63) < EPW) red[t >> 6][t & 63] = sum;
  __syncthreads();
  if (t < EPW && el < total) {
    static_assert(WAVES == 4, "pairs of pairs");
    (el < nk ? d_k[el] : d_bias[el - nk]) = (red[0][t] + red[1][t]) + (red[2][t] + red[3][t]);
  }
}

}  // namespace igemm
}  // namespace cnn
