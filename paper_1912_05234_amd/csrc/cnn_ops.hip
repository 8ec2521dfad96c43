// Stateless per-operation kernels (general shapes) and their C entry points.
// Definitions: arXiv 1912.05234, Section 3 -- listings conv, mconv, sigmoid,
// avgpool, backweights, backbias, backin, backavgpool.  Convolutions and fully
// connected layers run as implicit GEMMs on the matrix cores (cnn_tile.h; the network's
// own layers in kernels of their own); the plain one-thread-per-output kernels below serve
// the `*_valu` calls, weight gradients without a workspace, and images beyond the 32-bit offsets
// of the others.  The fused training step lives in cnn_fused.hip.
#include <algorithm>
#include <cmath>
#include <mutex>

#include "cnn_common.h"
#include "cnn_igemm.h"
#include "cnn_tile.h"
#include "cnn_tile_bf16.h"
#include "cnn_col2im.h"
#include "cnn_conv_wave.h"
#include "cnn_fc_wave.h"

namespace {

using namespace cnn;

constexpr int TPB = 256;

inline unsigned grid_for(size_t n) {
  size_t g = (n + TPB - 1) / TPB;
  const size_t cap = 256 * 32;  // grid-stride beyond this
  return (unsigned)(g < cap ? (g ? g : 1) : cap);
}

// Streaming kernels: one item per thread (neighbouring workgroups then touch neighbouring memory,
// which the memory system likes better than a few workgroups striding far: 6.2 against 5.0 TB/s for
// a 566 MB copy), and outputs written with the non-temporal hint (+ 4 to 20 %): nothing here reads
// its own output again.
inline unsigned grid_stream(size_t n) {
  size_t g = (n + TPB - 1) / TPB;
  const size_t cap = 0x7fffffff;
  return (unsigned)(g < cap ? (g ? g : 1) : cap);
}
typedef float vec2 __attribute__((ext_vector_type(2)));
typedef float vec4 __attribute__((ext_vector_type(4)));

// out[b,co,y,x] = bias[co] + sum_{ci,u,v} in[b,ci,y+u,x+v] * k[co,ci,u,v]
template <bool BF16>
__global__ __launch_bounds__(TPB) void conv_fwd_kernel(const float* __restrict__ in,
                                                       const float* __restrict__ k,
                                                       const float* __restrict__ bias,
                                                       float* __restrict__ out, size_t total, int Cin,
                                                       int H, int W, int Cout, int KH, int KW) {
  const int Ho = H - KH + 1, Wo = W - KW + 1;
  for (size_t o = blockIdx.x * (size_t)TPB + threadIdx.x; o < total; o += (size_t)gridDim.x * TPB) {
    const int x = (int)(o % Wo);
    const int y = (int)((o / Wo) % Ho);
    const int co = (int)((o / ((size_t)Wo * Ho)) % Cout);
    const size_t b = o / ((size_t)Wo * Ho * Cout);
    float acc = bias ? bias[co] : 0.0f;
    for (int ci = 0; ci < Cin; ++ci) {
      const float* ip = in + ((b * Cin + ci) * H + y) * (size_t)W + x;
      const float* kp = k + ((size_t)co * Cin + ci) * KH * KW;
      for (int u = 0; u < KH; ++u)
        for (int v = 0; v < KW; ++v) acc = fmaf(operand<BF16>(ip[u * W + v]), operand<BF16>(kp[u * KW + v]), acc);
    }
    out[o] = acc;
  }
}

// d_in[b,ci,p,q] = sum_co sum_{u,v valid} k[co,ci,u,v] * d_out[b,co,p-u,q-v]
template <bool BF16>
__global__ __launch_bounds__(TPB) void conv_bwd_input_kernel(const float* __restrict__ d_out,
                                                             const float* __restrict__ k,
                                                             float* __restrict__ d_in, size_t total,
                                                             int Cin, int H, int W, int Cout, int KH,
                                                             int KW) {
  const int Ho = H - KH + 1, Wo = W - KW + 1;
  for (size_t o = blockIdx.x * (size_t)TPB + threadIdx.x; o < total; o += (size_t)gridDim.x * TPB) {
    const int q = (int)(o % W);
    const int p = (int)((o / W) % H);
    const int ci = (int)((o / ((size_t)W * H)) % Cin);
    const size_t b = o / ((size_t)W * H * Cin);
    const int u_lo = max(0, p - Ho + 1), u_hi = min(KH - 1, p);
    const int v_lo = max(0, q - Wo + 1), v_hi = min(KW - 1, q);
    float acc = 0.0f;
    for (int co = 0; co < Cout; ++co) {
      const float* dp = d_out + (b * Cout + co) * (size_t)Ho * Wo;
      const float* kp = k + ((size_t)co * Cin + ci) * KH * KW;
      for (int u = u_lo; u <= u_hi; ++u)
        for (int v = v_lo; v <= v_hi; ++v)
          acc = fmaf(operand<BF16>(kp[u * KW + v]), operand<BF16>(dp[(p - u) * Wo + (q - v)]), acc);
    }
    d_in[o] = acc;
  }
}

// Fixed-order reduction of one value per thread over the workgroup.
__device__ __forceinline__ float block_sum(float v, float* red) {
  red[threadIdx.x] = v;
  __syncthreads();
  for (int s = TPB / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  const float r = red[0];
  __syncthreads();
  return r;
}

// One workgroup per weight (blocks [0, Cout*Cin*KH*KW)) or per bias (the next Cout
// blocks): d_k[co,ci,u,v] = sum_{b,y,x} in[b,ci,y+u,x+v] * d_out[b,co,y,x].
template <bool BF16>
__global__ __launch_bounds__(TPB) void conv_bwd_weight_kernel(const float* __restrict__ in,
                                                              const float* __restrict__ d_out,
                                                              float* __restrict__ d_k,
                                                              float* __restrict__ d_bias, int B, int Cin,
                                                              int H, int W, int Cout, int KH, int KW) {
  __shared__ float red[TPB];
  const int Ho = H - KH + 1, Wo = W - KW + 1;
  const int nk = Cout * Cin * KH * KW;
  const size_t dom = (size_t)B * Ho * Wo;
  const int id = blockIdx.x;
  float acc = 0.0f;
  if (id < nk) {
    const int v = id % KW, u = (id / KW) % KH, ci = (id / (KW * KH)) % Cin, co = id / (KW * KH * Cin);
    for (size_t e = threadIdx.x; e < dom; e += TPB) {
      const int x = (int)(e % Wo), y = (int)((e / Wo) % Ho);
      const size_t b = e / ((size_t)Wo * Ho);
      acc = fmaf(operand<BF16>(in[((b * Cin + ci) * H + y + u) * (size_t)W + x + v]),
                 operand<BF16>(d_out[((b * Cout + co) * Ho + y) * (size_t)Wo + x]), acc);
    }
    acc = block_sum(acc, red);
    if (threadIdx.x == 0) d_k[id] = acc;
  } else {
    const int co = id - nk;
    for (size_t e = threadIdx.x; e < dom; e += TPB) {
      const size_t b = e / ((size_t)Wo * Ho), r = e % ((size_t)Wo * Ho);
      acc += operand<BF16>(d_out[(b * Cout + co) * (size_t)Ho * Wo + r]);
    }
    acc = block_sum(acc, red);
    if (threadIdx.x == 0) d_bias[co] = acc;
  }
}

// V neighbouring outputs per thread.  With rows counted over all maps (r = map * Ho + p) the 2x2
// window of output (r, q) is rows 2 r, 2 r + 1 and columns 2 q, 2 q + 1 of the input, so one division
// per item suffices (ITEM: the type that counts them).  Where a row has an even number of outputs, two of them are one 8-byte item and
// their columns 16-byte ones.  Us, one output per thread and divisions of 64 bits -> this: 10000 images of 6 x 24 x 24 forward 27.9 -> 24.3,
// 40000 forward 123.6 -> 118.4, backward 149.6 -> 124.7; of 12 x 8 x 8, 10000 forward 6.4 -> 4.8.
template <typename ITEM>
__device__ __forceinline__ ITEM row_of(ITEM e, ITEM per_row, tile::FastDiv by, ITEM& rest) {
  if constexpr (sizeof(ITEM) == 4) return tile::divide(e, by, rest);
  const ITEM r = e / per_row;
  rest = e - r * per_row;
  return r;
}
template <int V, typename ITEM>
__global__ __launch_bounds__(TPB) void avgpool_fwd_kernel(const float* __restrict__ in, float* __restrict__ out,
                                                          ITEM items, size_t W, tile::FastDiv by) {
  typedef float wide __attribute__((ext_vector_type(2 * V)));
  typedef float item __attribute__((ext_vector_type(V)));
  for (ITEM e = blockIdx.x * (ITEM)TPB + threadIdx.x; e < items; e += (ITEM)gridDim.x * TPB) {
    ITEM q;
    const size_t r = row_of<ITEM>(e, (ITEM)(W / (2 * V)), by, q);
    const float* ip = in + 2 * r * W + 2 * V * (size_t)q;
    const wide a = *reinterpret_cast<const wide*>(ip), b = *reinterpret_cast<const wide*>(ip + W);
    item o;
#pragma unroll
    for (int i = 0; i < V; ++i) o[i] = (a[2 * i] + a[2 * i + 1] + b[2 * i] + b[2 * i + 1]) * 0.25f;
    reinterpret_cast<item*>(out)[e] = o;
  }
}

// V neighbouring elements of d_out per thread: it writes the 2x2 blocks that it spreads into (same row arithmetic).
template <int V, typename ITEM>
__global__ __launch_bounds__(TPB) void avgpool_bwd_kernel(const float* __restrict__ d_out, float* __restrict__ d_in,
                                                          ITEM items, size_t W, tile::FastDiv by) {
  typedef float wide __attribute__((ext_vector_type(2 * V)));
  typedef float item __attribute__((ext_vector_type(V)));
  for (ITEM e = blockIdx.x * (ITEM)TPB + threadIdx.x; e < items; e += (ITEM)gridDim.x * TPB) {
    ITEM q;
    const size_t r = row_of<ITEM>(e, (ITEM)(W / (2 * V)), by, q);
    const item d = reinterpret_cast<const item*>(d_out)[e];
    wide w;
#pragma unroll
    for (int i = 0; i < V; ++i) w[2 * i] = w[2 * i + 1] = d[i] * 0.25f;
    float* op = d_in + 2 * r * W + 2 * V * (size_t)q;
    *reinterpret_cast<wide*>(op) = w;
    *reinterpret_cast<wide*>(op + W) = w;
  }
}

// `total` pooled elements in rows of W / 2.
template <bool FORWARD, int V, typename ITEM>
int pool_as(const float* src, float* dst, size_t total, size_t W, hipStream_t st) {
  const ITEM items = (ITEM)(total / V);
  const tile::FastDiv by = sizeof(ITEM) == 4 ? tile::fast_div((long long)(W / (2 * V))) : tile::FastDiv{1, 0};
  if (FORWARD)
    avgpool_fwd_kernel<V, ITEM><<<grid_stream(items), TPB, 0, st>>>(src, dst, items, W, by);
  else
    avgpool_bwd_kernel<V, ITEM><<<grid_stream(items), TPB, 0, st>>>(src, dst, items, W, by);
  return hipGetLastError() == hipSuccess ? CNN_OK : CNN_EHIP;
}
template <bool FORWARD>
int pool(const float* src, float* dst, size_t total, size_t W, hipStream_t st) {
  const bool even = W % 4 == 0, few = total < (1u << 31);  // (a division of 32 bits takes a fifth of the instructions)
  return even ? few ? pool_as<FORWARD, 2, unsigned>(src, dst, total, W, st) : pool_as<FORWARD, 2, size_t>(src, dst, total, W, st)
              : few ? pool_as<FORWARD, 1, unsigned>(src, dst, total, W, st) : pool_as<FORWARD, 1, size_t>(src, dst, total, W, st);
}

__global__ __launch_bounds__(TPB) void fc_fwd_kernel(const float* __restrict__ in,
                                                     const float* __restrict__ w,
                                                     const float* __restrict__ bias,
                                                     float* __restrict__ out, size_t total, int I, int O) {
  for (size_t e = blockIdx.x * (size_t)TPB + threadIdx.x; e < total; e += (size_t)gridDim.x * TPB) {
    const int o = (int)(e % O);
    const size_t b = e / O;
    float acc = bias ? bias[o] : 0.0f;
    for (int i = 0; i < I; ++i) acc = fmaf(in[b * I + i], w[(size_t)o * I + i], acc);
    out[e] = acc;
  }
}

__global__ __launch_bounds__(TPB) void fc_bwd_input_kernel(const float* __restrict__ d_out,
                                                           const float* __restrict__ w,
                                                           float* __restrict__ d_in, size_t total, int I,
                                                           int O) {
  for (size_t e = blockIdx.x * (size_t)TPB + threadIdx.x; e < total; e += (size_t)gridDim.x * TPB) {
    const int i = (int)(e % I);
    const size_t b = e / I;
    float acc = 0.0f;
    for (int o = 0; o < O; ++o) acc = fmaf(w[(size_t)o * I + i], d_out[b * O + o], acc);
    d_in[e] = acc;
  }
}

// One workgroup per weight (blocks [0, O*I)) or per bias (next O blocks).
__global__ __launch_bounds__(TPB) void fc_bwd_weight_kernel(const float* __restrict__ in,
                                                            const float* __restrict__ d_out,
                                                            float* __restrict__ d_w,
                                                            float* __restrict__ d_bias, int B, int I,
                                                            int O) {
  __shared__ float red[TPB];
  const int id = blockIdx.x;
  float acc = 0.0f;
  if (id < O * I) {
    const int i = id % I, o = id / I;
    for (size_t b = threadIdx.x; b < (size_t)B; b += TPB) acc = fmaf(d_out[b * O + o], in[b * I + i], acc);
    acc = block_sum(acc, red);
    if (threadIdx.x == 0) d_w[id] = acc;
  } else {
    const int o = id - O * I;
    for (size_t b = threadIdx.x; b < (size_t)B; b += TPB) acc += d_out[b * O + o];
    acc = block_sum(acc, red);
    if (threadIdx.x == 0) d_bias[o] = acc;
  }
}

// Four elements per thread as one 16-byte item; the last n % 4 elements one by one.
__global__ __launch_bounds__(TPB) void logistic_fwd_kernel(const float* __restrict__ x,
                                                           float* __restrict__ y, size_t n) {
  const size_t n4 = n / 4, stride = (size_t)gridDim.x * TPB, first = blockIdx.x * (size_t)TPB + threadIdx.x;
  for (size_t e = first; e < n4; e += stride) {
    const float4 v = reinterpret_cast<const float4*>(x)[e];
    __builtin_nontemporal_store(vec4{logistic(v.x), logistic(v.y), logistic(v.z), logistic(v.w)},
                                reinterpret_cast<vec4*>(y) + e);
  }
  for (size_t e = 4 * n4 + first; e < n; e += stride) y[e] = logistic(x[e]);
}

__global__ __launch_bounds__(TPB) void logistic_bwd_kernel(const float* __restrict__ y,
                                                           const float* __restrict__ d_y,
                                                           float* __restrict__ d_x, size_t n) {
  const size_t n4 = n / 4, stride = (size_t)gridDim.x * TPB, first = blockIdx.x * (size_t)TPB + threadIdx.x;
  for (size_t e = first; e < n4; e += stride) {
    const float4 v = reinterpret_cast<const float4*>(y)[e], d = reinterpret_cast<const float4*>(d_y)[e];
    __builtin_nontemporal_store(vec4{d.x * v.x * (1.0f - v.x), d.y * v.y * (1.0f - v.y),
                                     d.z * v.z * (1.0f - v.z), d.w * v.w * (1.0f - v.w)},
                                reinterpret_cast<vec4*>(d_x) + e);
  }
  for (size_t e = 4 * n4 + first; e < n; e += stride) {
    const float v = y[e];
    d_x[e] = d_y[e] * v * (1.0f - v);
  }
}

inline int launched() { return hipGetLastError() == hipSuccess ? CNN_OK : CNN_EHIP; }

// ---- launch plans of the matrix-core kernels ----------------------------------------------------
constexpr int CU_LDS = 160 * 1024;
constexpr int TILE_LDS_LIMIT = 79 * 1024;   // of an image-tiled kernel: two workgroups per compute unit
constexpr int NUM_CU = 256;

// ---- image-tiled kernels (cnn_tile.h) ------------------------------------------------------------------
// Plans made before, by shape, so that a call does not choose one twice.  Choosing takes 2 to 3 us of host time in the
// median over 1500 layers, 6 for the fp32 weight gradient, and 40 to 100 at most (every candidate evaluated, instead of
// only those whose least cost is below the best one's: 6 to 8, 22, and 70 to 170).  A plan is a pure function of its key
// (it holds no caller's pointer).  WAYS entries for each of SETS hash values, the oldest of a set is given up: a program
// that goes round 40 batch sizes of a layer keeps them all.
template <typename PLAN, int KEYS>
class PlanMemo {
  struct Entry {
    int key[KEYS];
    PLAN plan;
  };
  static constexpr int SETS = 64, WAYS = 4;
  Entry entry[SETS][WAYS];
  unsigned char used[SETS] = {}, next[SETS] = {};
  std::mutex guard;

  static unsigned set_of(const int (&key)[KEYS]) {
    unsigned h = 0;
    for (int k : key) h = (h ^ (unsigned)k) * 0x9e3779b1u, h ^= h >> 15;
    return h % SETS;
  }

 public:
  template <typename MAKE>
  PLAN get(const int (&key)[KEYS], MAKE make) {
    const unsigned set = set_of(key);
    {
      std::lock_guard<std::mutex> lock(guard);
      for (int i = 0; i < used[set]; ++i)
        if (std::equal(key, key + KEYS, entry[set][i].key)) return entry[set][i].plan;
    }
    const PLAN plan = make();
    std::lock_guard<std::mutex> lock(guard);
    Entry& slot = entry[set][next[set]];
    next[set] = (next[set] + 1) % WAYS;
    if (used[set] < WAYS) ++used[set];
    std::copy(key, key + KEYS, slot.key);
    slot.plan = plan;
    return plan;
  }
};

struct TileConvPlan {
  tile::ConvArgs a;
  int nt = 0, mt = 0;  // column and row tiles per wave; nt = 0: no unit fits in LDS
  int run = 1;         // staged floats that a lane reads at once
  dim3 grid;
  size_t lds_bytes = 0;
  double cost = 0.0;
};

inline long long ceil_div(long long a, long long b) { return (a + b - 1) / b; }
inline int up(int a, int b) { return (a + b - 1) / b; }  // (for the planner's inner loops: a 64-bit division takes three times as long)

// The unit's geometry in `a`; false when it cannot be.
bool tile_unit(tile::ConvArgs& a, int P, int mt, int NB, int TH, int TXC) {
  a.P = P, a.MR = a.M * P, a.KWP = a.KW + P - 1;
  const long long OWP = ceil_div(a.OW, P);
  a.NB = NB, a.TH = TH, a.TXC = TXC;
  a.groups = (int)ceil_div(a.B, NB), a.bands = (int)ceil_div(a.OH, TH), a.strips = (int)ceil_div(OWP, TXC);
  if ((long long)a.groups * a.bands * a.strips > 0x3fffffff || (long long)NB * a.M * a.OH * a.OW >= tile::FAR_SIZE / 4) return false;
  a.units = a.groups * a.bands * a.strips;
  a.by_unit = tile::fast_div((long long)a.bands * a.strips), a.by_strip = tile::fast_div(a.strips), a.by_cc = tile::fast_div(a.SC);
  a.RH = TH + a.KH - 1;
  const bool border = a.pady || a.padx || a.strips > 1;
  a.LW = border ? TXC * P + a.KW - 1 : a.SW;
  if ((long long)a.RH * a.LW > TILE_LDS_LIMIT / 4) return false;
  a.RPI = a.LW <= 64 ? 64 / a.LW : 1;
  // (by rows, the last instruction of a plane may bring rows past RH)
  a.LP = border ? (int)ceil_div(a.RH, a.RPI) * a.RPI * a.LW : a.bands == 1 ? a.SH * a.SW : a.RH * a.LW;
  a.R = a.MR < 16 * mt ? a.MR : 16 * mt;
  return true;
}
// Bytes per lane of the staging loads of borderless planes, 0 for staging by rows.
int tile_linear(const tile::ConvArgs& a, bool border) {
  if (border) return 0;
  const long long plane = (long long)a.SH * a.SW;
  return (a.bands == 1 ? a.SC * plane % 4 == 0 && a.CC * plane % 4 == 0 && a.LI % 4 == 0
                       : plane % 4 == 0 && a.LP % 4 == 0 && a.TH * a.SW % 4 == 0) ? 16 : 4;
}
// Workgroups in x for `res` per compute unit and `gy` in y (res = 0: one).
int tile_columns(int units, int gy, int res) {
  if (gy >= NUM_CU * res) return 1;
  const int gx = gy == 1 ? NUM_CU * res : NUM_CU * res / gy;
  return gx < units ? gx : units;
}
void tile_constants(tile::ConvArgs& a) {
  a.inv_p = 1.0f / a.P, a.inv_khkwp = 1.0f / (float)(a.KH * a.KWP), a.inv_kwp = 1.0f / (float)a.KWP;
  a.inv_cols = 1.0f / (float)(a.TH * a.TXC), a.inv_txc = 1.0f / (float)a.TXC, a.inv_lw = 1.0f / (float)a.LW;
  a.inv_khkw = 1.0f / (float)(a.KH * a.KW), a.inv_kw = 1.0f / (float)a.KW, a.inv_cc = 1.0f / (float)a.CC;
}

// Clocks per block of a column tile beside the matrix instructions, by the floats a lane reads at once: 12 and 23 fewer
// for 2 and 4 in 61 and 7 pairs of timed plans that differ in nothing else (1.04x and 1.08x in time).
constexpr double RUN_CLOCKS[5] = {0.0, 80.0, 68.0, 0.0, 57.0};

// Keeps the best of one unit's candidates: runs, weights resident or not, 1 .. 4 workgroups per compute unit.  The cost is
// an estimate of the kernel's clocks, linear in what a compute unit has to do: matrix instructions (32 clocks each, partly
// hidden under the vector instructions of other waves), blocks of operand reads, staging and store instructions,
// a fixed share per unit, and a memory round trip per unit that a workgroup takes.  The coefficients are a least
// squares fit to 5000 timed plans of 40 shapes (7 % rms); the plan it picks was on average 1.4 % slower than the
// fastest one of a shape.  The weights' share `wt` is a memory round trip and P writes per item of eight maps that a thread
// takes (estimated; plans picked with it were 2 % faster over 60 shapes than with the share of the way before).
void tile_conv_candidates(TileConvPlan& best, TileConvPlan& p, int P, int mt, int nt, int NB, int TH, int TXC) {
  tile::ConvArgs& a = p.a;
  if (!tile_unit(a, P, mt, NB, TH, TXC)) return;
  const bool border = a.pady || a.padx || a.strips > 1;
  const int MB = up(a.MR, 16 * mt), by_regs = tile::conv_residency(nt, mt);
  const int wide = P % 4 == 0 && a.OW % 4 == 0 ? 4 : P % 2 == 0 && a.OW % 2 == 0 ? 2 : 1;
  const long long total = (long long)a.units * MB, taps = (long long)a.KH * a.KWP;
  const double per_cu = (double)ceil_div(total, NUM_CU), stores = 16.5 * nt * mt * 4 / wide + 83.0 * nt;
  // what every candidate of the unit costs at least
  const double read = RUN_CLOCKS[mt > 1 || P % 2 ? 1 : P % 4 ? 2 : 4] * nt + 23.0;
  if (best.nt && 9800.0 + per_cu * ((double)ceil_div(a.SC * taps, 16) * (64.0 * nt * mt + read) + 430.0 + stores) +
                     1630.0 * up(a.units, tile_columns(a.units, MB, 4)) >= best.cost)
    return;
  for (int run = 1; run <= (mt == 1 ? 4 : 1) && P % run == 0; run <<= 1) {
    if (run > 1) {
      // whole runs of taps in a row (filled up with zero taps they cost more than the runs give: 362 images 22 -> 6, 19 x 36,
      // 4 x 4, forward with 5 taps as 6 31.4 -> 39.0 us), staged rows and planes in whole runs
      if (border) {
        a.LW = up(a.LW, run) * run;
        a.RPI = a.LW <= 64 ? 64 / a.LW : 1;
        a.LP = up(a.RH, a.RPI) * a.RPI * a.LW;
      }
      if (a.KWP % run || a.LW % run || a.LP % run) continue;
    }
    // channels per chunk: the fewest equal shares that fit, with all the weights in LDS or with each chunk's own
    for (int resident = 1; resident >= 0; --resident) {
      // (floats: `fixed` and `each` per channel at least)
      const long long fixed = resident ? a.SC * taps * (a.R + 1) : 0, each = (resident ? taps : (a.R + 2) * taps) + 2LL * NB * a.LP;
      const long long most = (TILE_LDS_LIMIT / 4 - fixed) / each;
      if (fixed > TILE_LDS_LIMIT / 4 || most < 1) continue;
      const int fewest = (int)ceil_div(a.SC, most);
      for (int chunks = std::max(fewest, resident ? 1 : 2); chunks <= a.SC && (chunks == 1 || NB == 1 || !border); ++chunks) {
        a.CC = up(a.SC, chunks);
        if (up(a.SC, a.CC) != chunks) continue;
        const long long K = a.CC * taps;
        if (K > (1 << 16) || (long long)a.CC * a.LP * NB > TILE_LDS_LIMIT / 4) continue;
        a.chunks = chunks, a.resident = resident, a.K = (int)K, a.NBK = up((int)K, 16), a.LI = a.CC * a.LP;
        // the sixteen columns of a tile are the same pixel of sixteen images when there are few pixels: images start in different banks
        if (NB > 1 && a.TH * a.TXC < 16 && !border && a.LI % 8 == 0) a.LI += 4;
        a.SP = igemm::row_stride(resident ? a.NBK * chunks : a.NBK), a.SK = igemm::row_stride(a.NBK);
        const long long lds = (long long)tile::conv_lds(a).total * 4;
        if (lds > TILE_LDS_LIMIT) continue;
        a.linear = tile_linear(a, border);
        const int by_lds = CU_LDS / ((int)lds + 512);
        const double stage = 0.25 * NB * (!border && a.bands == 1 ? up(a.CC * a.LP, 16 * a.linear) : a.CC * 1.0 * (!border ? up(a.LP, 16 * a.linear) : a.LW <= 64 ? up(a.RH, a.RPI) : a.RH * up(a.LW, 64)));
        const double mfma = 128.0 * a.NBK * nt * mt, reads = a.NBK * (RUN_CLOCKS[run] * nt + 23.0) + stage * (border ? 50.0 : 82.0) + 430.0;
        const double wt = chunks * (double)up(a.CC * a.KH * a.KW * up(a.R, 8 * P), tile::THREADS) * (450.0 + 90.0 * P);
        for (int res = 1; res <= 4 && res <= by_lds && res <= by_regs && (res == 1 || total > NUM_CU * (res - 1)); ++res) {
          // workgroups of a compute unit, units it works off, units one workgroup takes in turn
          const int gx = tile_columns(a.units, MB, res), wgs = total < NUM_CU * res ? (int)ceil_div(total, NUM_CU) : res;
          const double turns = (double)up(a.units, gx) * chunks, unit = chunks * (mfma * (wgs == 1 ? 1.1 : wgs == 2 ? 0.6 : 0.5) + reads) + stores;
          const double cost = 9300.0 + 500.0 * wgs + wt * (resident ? wgs : per_cu) + per_cu * unit + turns * (wgs == 1 ? 1970.0 : wgs == 2 ? 1820.0 : 1630.0);
          if (best.nt && cost >= best.cost) continue;
          p.cost = cost, p.nt = nt, p.mt = mt, p.run = run, p.lds_bytes = (size_t)lds;
          p.grid = dim3((unsigned)gx, (unsigned)MB);
          best = p;
        }
        break;
      }
    }
  }
}

// The problem in `a`; false where the kernels' 32-bit offsets end.
bool tile_args(tile::ConvArgs& a, int B, int M, int SC, int SH, int SW, int KH, int KW, int OH, int OW, int pady, int padx, int flip) {
  if ((long long)SC * SH * SW > (1ll << 29) || (long long)SH * SW >= tile::FAR_SIZE / 4 || OH > (1 << 24) ||
      (long long)M * SC * KH * KW >= tile::FAR_SIZE / 8 || ceil_div(M, 16) > 60000)
    return false;
  a.src = a.w = a.bias = nullptr, a.dst = nullptr;
  a.B = B, a.M = M, a.SC = SC, a.SH = SH, a.SW = SW, a.KH = KH, a.KW = KW, a.OH = OH, a.OW = OW;
  a.pady = pady, a.padx = padx, a.flip = flip;
  return true;
}
// Hands every unit worth considering to `consider`: packing, row and column tiles, images, rows and columns.  Six
// column tiles per wave only for whole images of 257 to 384 columns without a border, which four would cut into bands: 2000
// images 2 -> 16, 20 x 20, 3 x 3 25.4 -> 20.6 us, bf16 22.2 -> 16.6; 700 images 12 -> 7, 19 x 33, one tap 17.1 -> 14.3 and 18.9 -> 14.6.
// With a border, or elsewhere, they were 5 to 20 % slower as often as faster (two or three workgroups per compute unit).
// (Layers of one tap are packed too: as many matrix instructions, but P times fewer columns to address, and stores P times as
// wide.  3000 images 2 -> 2, 24 x 24: forward 34.6 -> 10.7 us, input gradient 34.6 -> 10.5, bf16 36.2 -> 15.3; 500 images
// 8 -> 8, 20 x 20: 9.5 -> 8.4.  In the weight gradient packing multiplies rows and taps alike: 22 -> 28 us at 700 images
// 12 -> 7, 19 x 33.)
template <typename CONSIDER>
void tile_units(const tile::ConvArgs& a, CONSIDER consider) {
  const int M = a.M, OH = a.OH, OW = a.OW, B = a.B;
  for (int P = 1; P <= OW && (P == 1 || P * M <= 16); ++P) {
    if ((P & (P - 1)) && P != 16 / M && OW % P) continue;  // powers of two (wide stores), divisors of the row, the one that fills the tile best
    for (int mt = 1; mt <= (M > 16 ? 2 : 1); ++mt)
      for (int nt = 1; nt <= 4; nt <<= 1) {
        auto sizes = [&](int NB, long long TH, long long TXC) {
          consider(P, mt, nt, NB, (int)TH, (int)TXC);
        };
        const long long OWP = ceil_div(OW, P), most = 64 * nt;
        if (OWP > most) {
          sizes(1, 1, ceil_div(OWP, ceil_div(OWP, most)));
          continue;
        }
        const long long TH = most / OWP;
        if (TH >= OH) {
          const long long NB = most / (OH * OWP);
          sizes((int)(NB < B ? NB : B), OH, OWP);
          if (NB > 1) sizes((int)(NB / 2 < B ? NB / 2 : B), OH, OWP);
        }
        if (OH > 1) {
          const long long bands = ceil_div(OH, TH < OH ? TH : OH - 1);
          for (int f = 1; f <= 4; f <<= 1) sizes(1, ceil_div(OH, bands * f), OWP);
        }
      }
    const long long image = OH * ceil_div(OW, P);
    if (!a.pady && !a.padx && B >= 2 * NUM_CU && image > 256 && image <= 384) consider(P, 1, 6, 1, OH, (int)ceil_div(OW, P));
  }
}

TileConvPlan plan_tile_conv(const float* src, const float* w, const float* bias, float* dst, int B, int M, int SC,
                            int SH, int SW, int KH, int KW, int OH, int OW, int pady, int padx, int flip) {
  static PlanMemo<TileConvPlan, 12> memo;
  TileConvPlan p = memo.get({B, M, SC, SH, SW, KH, KW, OH, OW, pady, padx, flip}, [&] {
    TileConvPlan best, c;
    if (!tile_args(c.a, B, M, SC, SH, SW, KH, KW, OH, OW, pady, padx, flip)) return best;
    tile_units(c.a, [&](int P, int mt, int nt, int NB, int TH, int TXC) { tile_conv_candidates(best, c, P, mt, nt, NB, TH, TXC); });
    if (best.nt) tile_constants(best.a);
    return best;
  });
  p.a.src = src, p.a.w = w, p.a.bias = bias, p.a.dst = dst;
  return p;
}

// More than 64 KB of dynamic LDS has to be asked for.
template <typename ARGS>
void launch_tiled(void (*kernel)(const ARGS), dim3 grid, size_t lds_bytes, hipStream_t stream, const ARGS& args) {
  if (lds_bytes > 64 * 1024)
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
  kernel<<<grid, tile::THREADS, lds_bytes, stream>>>(args);
}

template <bool BORDER, int RUN, bool ROUND>
void launch_tile_conv_as(const TileConvPlan& p, hipStream_t stream) {
  switch (p.nt) {
    case 1: launch_tiled(tile::conv_kernel<1, 1, BORDER, RUN, ROUND>, p.grid, p.lds_bytes, stream, p.a); break;
    case 2: launch_tiled(tile::conv_kernel<2, 1, BORDER, RUN, ROUND>, p.grid, p.lds_bytes, stream, p.a); break;
    case 4: launch_tiled(tile::conv_kernel<4, 1, BORDER, RUN, ROUND>, p.grid, p.lds_bytes, stream, p.a); break;
    default:
      if constexpr (!BORDER) launch_tiled(tile::conv_kernel<6, 1, false, RUN, ROUND>, p.grid, p.lds_bytes, stream, p.a);
  }
}

template <bool BORDER, bool ROUND>
void launch_tile_conv_as(const TileConvPlan& p, hipStream_t stream) {
  switch (p.run) {
    case 2: return launch_tile_conv_as<BORDER, 2, ROUND>(p, stream);
    case 4: return launch_tile_conv_as<BORDER, 4, ROUND>(p, stream);
    default: return launch_tile_conv_as<BORDER, 1, ROUND>(p, stream);
  }
}

template <bool BORDER>
void launch_two_row_tiles(const TileConvPlan& p, hipStream_t stream) {
  switch (p.nt) {
    case 1: launch_tiled(tile::conv_kernel<1, 2, BORDER, 1, false>, p.grid, p.lds_bytes, stream, p.a); break;
    case 2: launch_tiled(tile::conv_kernel<2, 2, BORDER, 1, false>, p.grid, p.lds_bytes, stream, p.a); break;
    default: launch_tiled(tile::conv_kernel<4, 2, BORDER, 1, false>, p.grid, p.lds_bytes, stream, p.a); break;
  }
}

int launch_tile_conv(const TileConvPlan& p, hipStream_t stream) {
  if (p.mt == 2)
    p.a.linear ? launch_two_row_tiles<false>(p, stream) : launch_two_row_tiles<true>(p, stream);
  else
    p.a.linear ? launch_tile_conv_as<false, false>(p, stream) : launch_tile_conv_as<true, false>(p, stream);
  return launched();
}

// With operands rounded to bfloat16 (one row tile).
int launch_tile_conv_rounded(const TileConvPlan& p, hipStream_t stream) {
  p.a.linear ? launch_tile_conv_as<false, true>(p, stream) : launch_tile_conv_as<true, true>(p, stream);
  return launched();
}

struct TileWgradPlan {
  tile::WgradArgs a;
  int nt = 0, mt = 0;
  bool rounded = false;  // with operands rounded to bfloat16
  dim3 grid;
  size_t lds_bytes = 0, workspace_bytes = 0, interface_bytes = 0;
  double cost = 0.0;
};

// Clocks of the weight gradient's parts beside its matrix instructions: per tap tile of a block and per block, per load of
// x and of d_out with 16 and with 4 bytes per lane, per unit that a workgroup takes.  Unpacked plans: fit to 1924 timed plans of
// 122 layers, 10 % rms; packed ones, whose loads of d_out are scattered: 12600 plans of the kernels before, and a factor that
// brings the two together.  The plan picked is 4.3 % slower on average than the fastest of the sixteen or so that were timed
// of a layer, 15 % in the worst twentieth.
struct WgradClocks {
  double tile, block, x16, x4, d16, d4, turn, scale;
};
inline WgradClocks wgrad_clocks(int P) {
  return P == 1 ? WgradClocks{45.0, 135.0, 55.0, 25.0, 32.0, 17.5, 900.0, 1.0} : WgradClocks{5.0, 320.0, 19.0, 19.0, 33.0, 33.0, 2000.0, 1.05};
}

// As above for the weight gradient.  A form is its packing and the row and tap tiles of a workgroup; false when there is no
// such form, or none of its units can be better than `best`.
bool tile_wgrad_form(TileWgradPlan& p, const TileWgradPlan& best, int P, int mt, int nt) {
  tile::WgradArgs& a = p.a;
  a.P = P, a.MR = a.Cout * P, a.KWP = a.KW + P - 1, a.WOP = up(a.Wo, P);
  a.K = a.Cin * a.KH * a.KWP, a.MT = up(a.MR, 16), a.NT = up(a.K, 16);
  // taps of a workgroup: all of its tiles, or (packed) whole groups of KWP
  a.TG = P == 1 ? 16 * nt : 16 * nt / a.KWP * a.KWP;
  if (a.TG < 1) return false;
  if (a.TG > a.K) a.TG = a.K;
  a.NTG = up(a.K, a.TG);
  a.R = a.MR < 16 * mt ? a.MR : 16 * mt;
  a.RS = a.Cout * a.Cin * a.KH * a.KW + a.Cout;
  // channels a group of 16 nt consecutive taps can touch
  const long long KHKWP = (long long)a.KH * a.KWP, cg = a.NTG == 1 ? a.Cin : (16LL * nt + KHKWP - 2) / KHKWP + 1;
  a.CG = (int)(cg < a.Cin ? cg : a.Cin);
  p.nt = nt, p.mt = mt;
  p.grid.y = (unsigned)(up(a.MT, mt) * a.NTG);
  if (!best.nt) return true;
  const double rounds = (double)a.B * a.Ho * a.WOP / 64.0 * p.grid.y / NUM_CU;
  const WgradClocks k = wgrad_clocks(P);
  return k.scale * (9500.0 + 256.0 * nt * mt + rounds * (64.0 * nt * mt + k.tile * nt + k.block + (P == 1 ? k.d16 / 4.0 : k.d4) * a.R)) < best.cost;
}

// Five tap tiles of a workgroup: where it takes a unit after the other, at most two of them per compute unit.  The fit counts the matrix
// instructions that six tiles waste and not what more of them cost before a first unit.  Against plans without them, over random
// layers that would take them: one unit per workgroup 0.94 to 1.03 times as fast (403 images 3 -> 20, 18 x 15, 7 x 7 15.0 -> 19.2 us),
// from one and three quarters on 1.06 to 1.10 (worst 0.96) with two workgroups per compute unit, 1.03 to 1.05 (worst 0.88) with more.
inline bool five_tiles_pay(int units, int gx, int gy) { return 4ll * units >= 7ll * gx && (long long)gx * gy <= 2 * NUM_CU; }

// Keeps the best of one unit of p's form, `few` .. `most` workgroups per compute unit; 0: one workgroup column, which needs
// no second kernel.
void tile_wgrad_candidates(TileWgradPlan& best, TileWgradPlan& p, int NB, int TH, int few, int most) {
  tile::WgradArgs& a = p.a;
  const int plane = a.H * a.W, gy = (int)p.grid.y, nt = p.nt, mt = p.mt;
  const WgradClocks k = wgrad_clocks(a.P);
  const long long groups = NB == 1 ? a.B : ceil_div(a.B, NB), units = TH == a.Ho ? groups : groups * up(a.Ho, TH);
  if (units > 0x3fffffff || (long long)NB * a.Cout * a.Ho * a.Wo >= tile::FAR_SIZE / 4 || (long long)NB * TH * a.WOP > 4096) return;
  a.NB = NB, a.TH = TH, a.groups = (int)groups, a.bands = TH == a.Ho ? 1 : up(a.Ho, TH), a.units = (int)units;
  a.N = NB * TH * a.WOP, a.NBK = up(a.N, 16), a.NPS = 16 * a.NBK + 4;
  a.vec_d = a.P == 1 && a.Ho * a.Wo % 4 == 0 && TH * a.Wo % 4 == 0 ? 16 : 4;
  const double blocks = up(a.NBK, tile::WAVES), mfma = 128.0 * blocks * nt * mt, d_loads = a.R * (a.vec_d == 16 ? k.d16 * up(a.NBK, 16) : k.d4 * up(a.NBK, 4));
  const double per_unit = blocks * (k.tile * nt + k.block) + d_loads, work = (double)units * gy / NUM_CU;
  auto second_kernel = [&](int gx) { return gx > 1 ? 6650.0 + 0.0097 * gx * a.RS + 2.4 * gx : 0.0; };
  // what every candidate of the unit costs at least
  if (best.nt && k.scale * (9500.0 + 256.0 * nt * mt + (work > 1.0 ? work : 1.0) * (mfma * 0.5 + per_unit) + k.turn * up(a.units, tile_columns(a.units, gy, 4)) +
                            second_kernel(tile_columns(a.units, gy, few))) >= best.cost)
    return;
  a.RH = a.bands == 1 ? a.H : TH + a.KH - 1;
  if ((long long)NB * a.CG * a.RH * a.W > TILE_LDS_LIMIT / 4) return;
  a.LP = a.RH * a.W, a.LI = a.CG * a.LP;
  a.vec_x = plane % 4 == 0 && a.LP % 4 == 0 && (a.bands == 1 || TH * a.W % 4 == 0) ? 16 : 4;
  if (a.bands == 1 && a.NTG == 1 && (long long)a.Cin * plane % 4 == 0) a.vec_x = 16;  // (runs of whole images)
  const long long end = tile::wgrad_end_floats(nt, mt), all = tile::wgrad_lds(a).total, lds = 4 * (all > end ? all : end);
  if (lds > TILE_LDS_LIMIT) return;
  const int resident = std::min(CU_LDS / ((int)lds + 512), tile::wgrad_residency(nt, mt, p.rounded));
  auto loads = [&](int floats) { return a.vec_x == 16 ? k.x16 * up(floats, 256) : k.x4 * up(floats, 64); };
  const double around = per_unit + NB * (a.bands == 1 ? loads(a.LI) : a.CG * loads(a.LP));
  for (int res = few; res <= most && res <= resident && (res <= 1 || (long long)a.units * gy > NUM_CU * (res - 1)); ++res) {
    const int gx = tile_columns(a.units, gy, res);
    if (nt == 5 && !five_tiles_pay(a.units, gx, gy)) continue;
    const long long total = (long long)gx * gy, wgs = total > NUM_CU ? ceil_div(total, NUM_CU) : 1;
    const double share = total > NUM_CU ? (double)total / NUM_CU : 1.0, turns = up(a.units, gx);
    const double cost = k.scale * (9500.0 + 256.0 * wgs * nt * mt + turns * (share * (mfma * (wgs == 1 ? 2.0 : wgs == 2 ? 0.9 : 0.5) + around) + k.turn) + second_kernel(gx));
    if (best.nt && cost >= best.cost) continue;
    p.cost = cost, p.lds_bytes = (size_t)lds;
    p.grid.x = (unsigned)gx;
    p.workspace_bytes = gx > 1 ? (size_t)gx * a.RS * sizeof(float) : 0;
    best = p;
  }
}

// The workspace that callers have been asked for, and the shapes that the built-in scratch has been documented to
// accept or to refuse, are part of the interface: a layout of one 16 x 16 tile per workgroup column, row tile and tap
// tile, with as many columns as workgroups of whole images are resident.  0 for shapes whose images do not fit in
// LDS.  The tiled kernels need less.
size_t tile_layout_bytes(int B, int Cin, int H, int W, int Cout, int KH, int KW) {
  constexpr int LDS_LIMIT = 64 * 1024 - 512, LDS_TARGET = 36 * 1024, MAX_GROUP = 64, MAX_COLUMNS = 1024;
  const long long Ho = H - KH + 1, Wo = W - KW + 1, per_image = (long long)Cin * H * W;
  auto bytes_for = [&](int P) -> size_t {
    const long long K = (long long)Cin * KH * (KW + P - 1), SPI = Ho * (Wo / P), MT = ceil_div((long long)Cout * P, 16), NT = ceil_div(K, 16);
    const long long R = Cout * P < 16 ? Cout * P : 16, cx = per_image % 4 == 0 ? 256 : 64, cd = P == 1 && Ho * Wo % 4 == 0 ? 256 : 64;
    if (2 * (per_image + 2 * SPI) > LDS_LIMIT / 4 || K > (1 << 20)) return 0;
    auto lds = [&](long long nb) {
      const long long blocks = ceil_div(nb * SPI, 16), total = 16 * blocks + 2 * ((R + 1) * (16 * blocks + 4) + ceil_div(nb * per_image, cx) * cx);
      const long long handover = 16 * blocks + igemm::WAVES * 272;
      return 4 * (total > handover ? total : handover);
    };
    if (SPI > 16 * cd || lds(1) > LDS_LIMIT) return 0;
    long long nb = 1;
    for (long long c = 2; c <= MAX_GROUP && c <= B && c <= ceil_div(B, MAX_COLUMNS) && lds(c) <= LDS_TARGET && c * SPI <= 16 * cd; ++c) nb = c;
    long long per_cu = CU_LDS / (lds(nb) + 512);
    per_cu = per_cu > 8 ? 8 : per_cu < 1 ? 1 : per_cu;
    long long gx = NUM_CU * per_cu / (MT * ceil_div(NT, 16));
    gx = gx < 1 ? 1 : gx > MAX_COLUMNS ? MAX_COLUMNS : gx;
    if (gx > ceil_div(B, nb)) gx = ceil_div(B, nb);
    return (size_t)(gx * MT * (NT * 256 + 16)) * sizeof(float);
  };
  int best = 1;
  long long best_cost = -1;
  for (int P = 1; KW > 1 && P * Cout <= 16; ++P) {
    if (Wo % P) continue;
    const long long cost = ceil_div((long long)Cin * KH * (KW + P - 1), 16) * ceil_div(Ho * (Wo / P), 16);
    if (best_cost < 0 || cost < best_cost) best_cost = cost, best = P;
  }
  for (int P = best; P >= 1; --P)
    if (Wo % P == 0)
      if (const size_t bytes = bytes_for(P)) return bytes;
  return 0;
}

// Five tap tiles of a workgroup: only for unpacked fp32 plans (five_tiles_pay).  With rounded operands they are slower than the fit
// says (305 images 21 -> 12, 33 x 23, 4 x 4 43.6 -> 46.6 us), packed ones too (850 images 24 -> 1, 19 x 11, 5 x 5 19.7 -> 25.1).  Nine
// were no gain: 1.02 times as fast as without where a workgroup takes several units, 0.93 where it takes one (509 images
// 16 -> 12, 13 x 33, 5 x 5 37.4 -> 47.4 us).
TileWgradPlan search_tile_wgrad(int B, int Cin, int H, int W, int Cout, int KH, int KW, bool rounded) {
  TileWgradPlan best, p;
  p.rounded = rounded;
  tile::WgradArgs& a = p.a;
  a.in = a.d_out = nullptr, a.out_k = a.out_b = nullptr;
  a.B = B, a.Cin = Cin, a.H = H, a.W = W, a.Cout = Cout, a.KH = KH, a.KW = KW, a.Ho = H - KH + 1, a.Wo = W - KW + 1;
  const long long K = (long long)Cin * KH * KW;
  if ((long long)Cin * H * W > (1ll << 29) || (long long)H * W >= tile::FAR_SIZE / 4 || 16 * K > (1 << 22)) return best;
  if (ceil_div(Cout, 16) * ceil_div(K, 16) > 60000) return best;
  // Few images beyond the LDS, for which the size query has always been zero: without a workspace only one workgroup
  // column is possible, and where that reads for longer than the plain kernel takes (one workgroup per weight: about
  // 4.4 clocks a pixel) the plain kernel stays.  From 30 us of the plain kernel on, partial sums pay in any case: 30
  // images of 22 x 24 x 23, one tap, took it 33 us, one workgroup column would take 172, many columns take 13.
  const double plain = 9600.0 + 4.4 * B * a.Ho * a.Wo * ceil_div(Cout * K, 8 * NUM_CU);
  const bool tiny = B <= 64 && plain <= 72000.0 && (double)B * Cout * a.Ho * a.Wo * K <= 2097152.0 &&
                    tile_layout_bytes(B, Cin, H, W, Cout, KH, KW) == 0;
  for (int P = 1; P <= a.Wo && (P == 1 || (KW > 1 && P * Cout <= 16)); ++P) {
    if ((P & (P - 1)) && P != 16 / Cout && a.Wo % P) continue;
    for (int mt = 1; mt <= (Cout > 16 ? 2 : 1); ++mt) {
      const int NT = up(Cin * KH * (KW + P - 1), 16);
      for (int nt : {1, 2, 3, 4, 5, 6, 8, 12}) {
        if (nt == 5 && (P > 1 || rounded)) continue;
        if (nt * mt > 16 || (nt > 1 && nt / 2 >= NT) || 16 * nt < KW + P - 1 || !tile_wgrad_form(p, best, P, mt, nt)) continue;
        auto consider = [&](int NB, int TH) { tile_wgrad_candidates(best, p, NB, TH, B > 64 ? 1 : 0, tiny ? 0 : 4); };
        for (long long NB = 1; NB <= B && NB * a.Ho * a.WOP <= 1536; NB = NB < 4 ? NB + 1 : 2 * NB) consider((int)NB, a.Ho);
        for (int TH = 1; TH < a.Ho && (long long)TH * a.WOP <= 1536; ++TH)
          if (TH <= 4 || up(a.Ho, TH) != up(a.Ho, TH - 1)) consider(1, TH);
      }
    }
  }
  if (best.nt) {
    tile::WgradArgs& b = best.a;
    b.inv_khkwp = 1.0f / (float)(KH * b.KWP), b.inv_kwp = 1.0f / (float)b.KWP, b.inv_slots = 1.0f / (float)(b.TH * b.WOP), b.inv_wop = 1.0f / (float)b.WOP;
    b.by_band = tile::fast_div(b.bands), b.by_p = tile::fast_div(b.P);
  }
  if (tiny && best.cost > plain) best.nt = 0, best.cost = plain;
  return best;
}

TileWgradPlan plan_tile_wgrad(int B, int Cin, int H, int W, int Cout, int KH, int KW, bool rounded) {
  static PlanMemo<TileWgradPlan, 8> memo;
  return memo.get({B, Cin, H, W, Cout, KH, KW, rounded}, [&] {
    TileWgradPlan p = search_tile_wgrad(B, Cin, H, W, Cout, KH, KW, rounded);
    p.interface_bytes = tile_layout_bytes(B, Cin, H, W, Cout, KH, KW);
    return p;
  });
}

// The second kernel of a weight gradient with more than one workgroup column.
int launch_reduce_rows(const float* part, int G, int RS, int nk, float* d_k, float* d_bias, hipStream_t st) {
  if (G > 1 && RS > 8192)
    tile::reduce_rows_kernel<64><<<(unsigned)ceil_div(RS, 64), tile::REDUCE_THREADS, 0, st>>>(part, G, RS, nk, d_k, d_bias);
  else if (G > 1)
    tile::reduce_rows_kernel<16><<<(unsigned)ceil_div(RS, 16), tile::REDUCE_THREADS, 0, st>>>(part, G, RS, nk, d_k, d_bias);
  return launched();
}

template <bool ROUND>
int launch_tile_wgrad(TileWgradPlan& p, const float* in, const float* d_out, float* d_k, float* d_bias, float* part,
                      hipStream_t st) {
  const int nk = p.a.RS - p.a.Cout, G = (int)p.grid.x;
  p.a.in = in, p.a.d_out = d_out, p.a.out_k = G > 1 ? part : d_k, p.a.out_b = G > 1 ? part + nk : d_bias;
#define CNN_TILE_WGRAD(KIND, NT, MT, PACKED) \
  case 1000 * KIND + NT: launch_tiled(tile::wgrad_kernel<NT, MT, ROUND, PACKED>, p.grid, p.lds_bytes, st, p.a); break
  switch (1000 * (p.mt == 2 ? 2 : p.a.P > 1 ? 1 : 0) + p.nt) {  // (two row tiles are never packed)
    CNN_TILE_WGRAD(0, 1, 1, false);
    CNN_TILE_WGRAD(0, 2, 1, false);
    CNN_TILE_WGRAD(0, 3, 1, false);
    CNN_TILE_WGRAD(0, 4, 1, false);
    CNN_TILE_WGRAD(0, 6, 1, false);
    CNN_TILE_WGRAD(0, 8, 1, false);
    CNN_TILE_WGRAD(0, 12, 1, false);
    CNN_TILE_WGRAD(1, 1, 1, true);
    CNN_TILE_WGRAD(1, 2, 1, true);
    CNN_TILE_WGRAD(1, 3, 1, true);
    CNN_TILE_WGRAD(1, 4, 1, true);
    CNN_TILE_WGRAD(1, 6, 1, true);
    CNN_TILE_WGRAD(1, 8, 1, true);
    CNN_TILE_WGRAD(1, 12, 1, true);
    CNN_TILE_WGRAD(2, 1, 2, false);
    CNN_TILE_WGRAD(2, 2, 2, false);
    CNN_TILE_WGRAD(2, 3, 2, false);
    CNN_TILE_WGRAD(2, 4, 2, false);
    CNN_TILE_WGRAD(2, 6, 2, false);
    CNN_TILE_WGRAD(2, 8, 2, false);
#undef CNN_TILE_WGRAD
    default:
      if constexpr (ROUND) {
        return CNN_EINVAL;
      } else {
        if (p.a.P > 1 || p.nt != 5) return CNN_EINVAL;
        launch_tiled(p.mt == 1 ? tile::wgrad_kernel<5, 1, false, false> : tile::wgrad_kernel<5, 2, false, false>, p.grid, p.lds_bytes, st, p.a);
      }
  }
  return launch_reduce_rows(part, G, p.a.RS, nk, d_k, d_bias, st);
}

// ---- the network's own layers: how many waves share an image (cnn_conv_wave.h, cnn_col2im.h) -----------------
// One wave per image leaves the machine idle while there are fewer images than SIMDs (1024): a call then takes as long as
// one image does in one wave, next to seven others of its workgroup.  Up to SPLIT_IMAGES the image's pixels (input
// gradient: its maps) are shared out among waves, in workgroups of fewer images, as long as all of them are
// resident at once; beyond, the copies of the image and of the operand tables cost more than the shorter chain gives.
// Kernel times, us, one wave per image -> as below (weight gradients: + 0 .. 2 us of the second kernel, which adds more rows):
//   images            10              100             250             500             800             2000 (split, not taken)
//   C1 forward        7.5 -> 3.9      8.5 -> 4.0      8.8 -> 4.2      8.9 -> 5.4      9.3 -> 7.0      10.2 -> 11.1
//   C2 forward        7.4 -> 4.6      8.1 -> 4.7      8.3 -> 4.9      8.7 -> 5.4      8.9 -> 7.0      10.3 -> 10.6
//   C2 input gr.      8.1 -> 6.4      8.4 -> 6.5      8.6 -> 6.6      8.8 -> 6.9      9.0 -> 8.0       9.7 -> 12.6
//   C1 weight gr.     6.9 -> 3.7      8.0 -> 3.7      8.2 -> 3.8      9.1 -> 5.8      9.3 -> 6.4      10.2 + 5.8 -> 9.7 + 7.6
//   C2 weight gr.     8.7 -> 4.9     10.6 -> 5.1     10.6 -> 5.4     11.0 -> 7.1     10.5 -> 8.2      11.6 + 5.8 -> 11.8 + 7.6
// FEW_IMAGES: one workgroup per compute unit at one image each; above, the finest split of C1 forward has two (5.7 us
// at 500 images where two waves per image take 5.4), and the second kernel of the weight gradients has as many
// rows to add as there are workgroups (C2 at 500 images: 6.4 + 5.4 us with two waves per image, 7.1 + 3.9 with one).
constexpr int FEW_IMAGES = NUM_CU, SPLIT_IMAGES = 4 * NUM_CU;

// The grid of a kernel whose workgroups take `images` images per round: at most two workgroups per compute unit.
inline unsigned image_groups(int B, int images) {
  const long long g = ceil_div(B, images);
  return (unsigned)(g < 2 * NUM_CU ? g : 2 * NUM_CU);
}

template <bool ROUND>
int launch_conv1_fwd(const float* in, const float* k, const float* bias, float* out, int B, hipStream_t st) {
  if (B <= FEW_IMAGES)
    conv1::forward_kernel<6, 6, ROUND><<<image_groups(B, 1), 64 * 6, 0, st>>>(in, k, bias, out, B);
  else if (B <= SPLIT_IMAGES)
    conv1::forward_kernel<4, 2, ROUND><<<image_groups(B, 2), 64 * 4, 0, st>>>(in, k, bias, out, B);
  else
    conv1::forward_kernel<8, 1, ROUND><<<image_groups(B, 8), 64 * 8, 0, st>>>(in, k, bias, out, B);
  return launched();
}

// One output map: nothing for a matrix tile to share.
template <bool ROUND>
int launch_conv1_bwd_input(const float* d_out, const float* k, float* d_in, int B, hipStream_t st) {
  const int groups = (B + conv1::WAVES_PER_GROUP - 1) / conv1::WAVES_PER_GROUP;
  conv1::bwd_input_kernel<ROUND><<<groups < NUM_CU ? groups : NUM_CU, conv1::THREADS, 0, st>>>(d_out, k, d_in, B);  // 128 KB of LDS: one workgroup per compute unit
  return launched();
}

void launch_conv2_fwd(const float* in, const float* k, const float* bias, float* out, int B, hipStream_t st) {
  // (beyond: two workgroups per compute unit; one, three or four measured the same, the kernel is bound by its matrix instructions)
  if (B <= SPLIT_IMAGES)
    conv2::forward_kernel<8, 4><<<image_groups(B, 2), 64 * 8, 0, st>>>(in, k, bias, out, B);
  else
    conv2::forward_kernel<8, 1><<<image_groups(B, 8), 64 * 8, 0, st>>>(in, k, bias, out, B);
}

void launch_conv2_bwd_input(const float* d_out, const float* k, float* d_in, int B, hipStream_t st) {
  // col2im form, 120 instead of 414 matrix instructions per image; beyond: 112 registers per lane, four waves per SIMD
  if (B <= SPLIT_IMAGES)
    col2im::conv_bwd_input_kernel<4, 2><<<image_groups(B, 2), 64 * 4, 0, st>>>(d_out, k, d_in, B);
  else
    col2im::conv_bwd_input_kernel<8, 1><<<image_groups(B, 8), 64 * 8, 0, st>>>(d_out, k, d_in, B);
}

// Images per round of a workgroup of the weight gradients launched below.
inline int conv1_wgrad_images(int B) { return B <= FEW_IMAGES ? 1 : B <= SPLIT_IMAGES ? 4 : 8; }
inline int conv2_wgrad_images(int B) { return B <= FEW_IMAGES ? 2 : B <= SPLIT_IMAGES ? 4 : 8; }

void launch_conv1_wgrad(const float* in, const float* d_out, float* part, int B, unsigned gx, hipStream_t st) {
  switch (conv1_wgrad_images(B)) {
    case 1: conv1::bwd_weight_kernel<3, 3><<<gx, 64 * 3, 0, st>>>(in, d_out, part, B); break;
    case 4: conv1::bwd_weight_kernel<4, 1><<<gx, 64 * 4, 0, st>>>(in, d_out, part, B); break;
    default: conv1::bwd_weight_kernel<8, 1><<<gx, 64 * 8, 0, st>>>(in, d_out, part, B); break;
  }
}

void launch_conv2_wgrad(const float* in, const float* d_out, float* part, int B, unsigned gx, hipStream_t st) {
  switch (conv2_wgrad_images(B)) {
    case 2: conv2::bwd_weight_kernel<4, 2><<<gx, 64 * 4, 0, st>>>(in, d_out, part, B); break;
    case 4: conv2::bwd_weight_kernel<4, 1><<<gx, 64 * 4, 0, st>>>(in, d_out, part, B); break;
    default: conv2::bwd_weight_kernel<8, 1><<<gx, 64 * 8, 0, st>>>(in, d_out, part, B); break;
  }
}

// A plan of one workgroup column leaves no partial sums, but asks for a workspace all the same: a call without one is the
// plain kernel, which multiplies nothing by padding zeros and so keeps a NaN or an infinity to the weights that meet it.
constexpr size_t NO_PARTIAL_SUMS_BYTES = 16;

struct WgradPlan {
  // which kernel: cnn_tile.h by the plan in `tile`, or one of the network's own layers (gx workgroups that leave partial
  // 16 x 16 tiles, NT of them, for igemm::wgrad_reduce_kernel)
  enum { PLAIN, TILED, CONV1, CONV2, FC } kernel = PLAIN;
  TileWgradPlan tile;
  int NT = 0;
  unsigned gx = 0;
  size_t workspace_bytes = 0;  // what the plan uses
  size_t least_bytes = 0;      // what it can run with
};

WgradPlan plan_wgrad(int B, int Cin, int H, int W, int Cout, int KH, int KW) {
  WgradPlan p;
  if (conv1::shape_fits(Cin, H, W, Cout, KH, KW)) {
    p.kernel = WgradPlan::CONV1;
    p.NT = 2;  // rows (map, x parity), columns the shifted taps: what the second kernel joins
    p.gx = image_groups(B, conv1_wgrad_images(B));
    p.workspace_bytes = conv1::bwd_weight_workspace_bytes(p.gx);
    p.least_bytes = conv1::bwd_weight_workspace_bytes(image_groups(B, 8));
  } else if (H == 1 && W == 1 && KH == 1 && KW == 1 && fc::shape_fits(Cin, Cout)) {
    p.kernel = WgradPlan::FC;
    p.NT = fc::NT;
    p.gx = image_groups(B, 4 * fc::AHEAD * fc::WGRAD_WAVES);  // a wave takes fc::AHEAD steps of four images per memory round trip
    // (up to fc::DIRECT_MAX_ROWS nothing is left there, but a call with less of it is the plain kernel, as for any shape)
    p.workspace_bytes = p.least_bytes = fc::bwd_weight_workspace_bytes(p.gx);
  } else if (conv2::shape_fits(Cin, H, W, Cout, KH, KW)) {
    p.kernel = WgradPlan::CONV2;
    p.NT = 10;
    p.gx = image_groups(B, conv2_wgrad_images(B));
    p.workspace_bytes = conv2::bwd_weight_workspace_bytes(p.gx);
    p.least_bytes = conv2::bwd_weight_workspace_bytes(image_groups(B, 8));
  } else {
    p.tile = plan_tile_wgrad(B, Cin, H, W, Cout, KH, KW, false);
    if (p.tile.nt) p.kernel = WgradPlan::TILED;
    if (p.tile.nt) p.workspace_bytes = std::max({p.tile.workspace_bytes, p.tile.interface_bytes, NO_PARTIAL_SUMS_BYTES});
    p.least_bytes = p.workspace_bytes;
  }
  return p;
}

// Fits the plan to the caller's workspace; false: it cannot run in it.  (The network's own layers have asked for the
// rows of workgroups of eight images before they were split; with a workspace of that size they run in as many workgroups
// as it has rows for.)
bool fit_wgrad(WgradPlan& p, size_t bytes) {
  if (p.kernel == WgradPlan::PLAIN || bytes < p.least_bytes) return false;
  if (bytes < p.workspace_bytes) p.gx = (unsigned)(bytes / (p.workspace_bytes / p.gx));
  return true;
}

// ---- reduced precision: the image-tiled kernels with bf16 operands (cnn_tile_bf16.h) -----------------------
struct Tile16ConvPlan {
  tile16::ConvArgs a;
  int nt = 0, mt = 0;
  dim3 grid;
  size_t lds_bytes = 0;
  double cost = 0.0;
};

void tile16_conv_candidates(Tile16ConvPlan& best, Tile16ConvPlan& p, int P, int mt, int nt, int NB, int TH, int TXC) {
  tile::ConvArgs& a = p.a.t;
  if (!tile_unit(a, P, mt, NB, TH, TXC)) return;
  const bool border = a.pady || a.padx || a.strips > 1;
  const int MB = up(a.MR, 16 * mt), eights = up(a.SC, 8), plane = a.SH * a.SW, by_regs = tile16::conv_residency(nt, mt);
  const long long total = (long long)a.units * MB, taps = (long long)a.KH * a.KWP;
  const int wide = P % 4 == 0 && a.OW % 4 == 0 ? 4 : P % 2 == 0 && a.OW % 2 == 0 ? 2 : 1;
  const double per_cu = (double)ceil_div(total, NUM_CU), stores = 16.0 * nt * mt * 4 / wide + 76.0 * nt, block = 15.0 * nt + 1.5 * nt * mt + 18.0;
  // what every candidate of the unit costs at least
  if (best.nt && 12115.0 + per_cu * (block * (double)ceil_div(taps * eights, 4) + stores) + 3600.0 * up(a.units, tile_columns(a.units, MB, 4)) >= best.cost) return;
  // planes are staged without their border, which lies around them in the items
  // (rows an odd number of items apart when the columns of a tile are an even number apart: they start in different banks)
  if (border && P % 2 == 0) a.LW |= 1;
  a.LP = a.bands == 1 ? plane : (a.RH < a.SH ? a.RH : a.SH) * a.SW;
  p.a.LPIX = a.RH * a.LW;
  p.a.RI = a.bands == 1 ? a.SH : a.RH, p.a.r0 = a.bands == 1 ? a.pady : 0;
  p.a.CI = a.strips == 1 ? a.SW : TXC * P + a.KW - 1, p.a.c0 = a.strips == 1 ? a.padx : 0;
  p.a.edges = (a.bands > 1 && a.pady) || a.strips > 1 || (a.bands > 1 && a.OH % TH) ? 1 : 0;
  for (int resident = 1; resident >= 0; --resident) {
    // the fewest chunks whose weights and items can fit (bytes: `fixed`, and `each` per eight channels at least)
    const long long fixed = resident ? 16 * taps * eights * (a.R + 1) : 0, each = (resident ? 0 : 16 * taps * (a.R + 1)) + 16LL * NB * p.a.LPIX;
    const long long most = (TILE_LDS_LIMIT - fixed) / each;
    if (fixed > TILE_LDS_LIMIT || most < 1) continue;
    for (int chunks = std::max((int)ceil_div(eights, most), resident ? 1 : 2); chunks <= eights; ++chunks) {
      p.a.C8 = up(eights, chunks);
      if (up(eights, p.a.C8) != chunks) continue;
      a.CC = chunks == 1 ? a.SC : 8 * p.a.C8;
      const long long K8 = taps * p.a.C8;
      if (K8 > (1 << 14) || (long long)a.CC * a.LP * NB > TILE_LDS_LIMIT / 4) continue;
      a.chunks = chunks, a.resident = resident, a.K = (int)(8 * K8), a.NBK = up((int)K8, 4), a.LI = a.CC * a.LP;
      p.a.RS = 64 * a.NBK * (resident ? chunks : 1) + 16;
      const long long lds = tile16::conv_lds(p.a).total;
      if (lds > TILE_LDS_LIMIT) continue;
      a.linear = (a.bands == 1 ? (long long)a.SC * plane % 4 == 0 && (long long)a.CC * plane % 4 == 0
                               : plane % 4 == 0 && (a.SW % 4 == 0 || (!a.pady && a.LP % 4 == 0 && TH * a.SW % 4 == 0))) ? 16 : 4;
      const int by_lds = CU_LDS / ((int)lds + 512);
      const double stage = 0.25 * (a.bands == 1 ? (double)NB * up(a.CC * a.LP, 16 * a.linear) : (double)a.CC * up(a.LP, 16 * a.linear));
      const double turned = up(NB * p.a.C8 * p.a.RI * p.a.CI, tile::THREADS), wt = (a.R + 1.0) * a.NBK * 4 * chunks / tile::THREADS;
      const double unit = chunks * (a.NBK * block + turned * 340.0 + stage * 40.0) + stores;
      for (int res = 1; res <= 4 && res <= by_lds && res <= by_regs && (res == 1 || total > NUM_CU * (res - 1)); ++res) {
        const int gx = tile_columns(a.units, MB, res), wgs = total < NUM_CU * res ? (int)ceil_div(total, NUM_CU) : res;
        const double turns = (double)up(a.units, gx) * chunks;
        const double cost = 11600.0 + 515.0 * wt * (resident ? wgs : per_cu) + per_cu * unit + turns * (wgs == 1 ? 4900.0 : wgs == 2 ? 4200.0 : 3600.0);
        if (best.nt && cost >= best.cost) continue;
        p.cost = cost, p.nt = nt, p.mt = mt, p.lds_bytes = (size_t)lds;
        p.grid = dim3((unsigned)gx, (unsigned)MB);
        best = p;
      }
      break;
    }
  }
}

Tile16ConvPlan plan_tile16_conv(const float* src, const float* w, const float* bias, float* dst, int B, int M, int SC,
                                int SH, int SW, int KH, int KW, int OH, int OW, int pady, int padx, int flip) {
  static PlanMemo<Tile16ConvPlan, 12> memo;
  Tile16ConvPlan p = memo.get({B, M, SC, SH, SW, KH, KW, OH, OW, pady, padx, flip}, [&] {
    Tile16ConvPlan best, c;
    if (!tile_args(c.a.t, B, M, SC, SH, SW, KH, KW, OH, OW, pady, padx, flip)) return best;
    tile_units(c.a.t, [&](int P, int mt, int nt, int NB, int TH, int TXC) { tile16_conv_candidates(best, c, P, mt, nt, NB, TH, TXC); });
    if (best.nt) {
      tile16::ConvArgs& a = best.a;
      tile_constants(a.t);
      a.inv_places = 1.0f / (float)(a.C8 * (a.t.resident ? a.t.chunks : 1) * KH * KW);
      a.inv_c8 = 1.0f / (float)a.C8, a.by_c8 = tile::fast_div(a.C8);
      a.inv_plane = 1.0f / (float)(a.RI * a.CI), a.inv_ci = 1.0f / (float)a.CI;
    }
    return best;
  });
  p.a.t.src = src, p.a.t.w = w, p.a.t.bias = bias, p.a.t.dst = dst;
  return p;
}

template <bool BORDER>
int launch_tile16_conv_as(const Tile16ConvPlan& p, hipStream_t stream) {
  switch (10 * p.mt + p.nt) {
    case 11: launch_tiled(tile16::conv_kernel<1, 1, BORDER>, p.grid, p.lds_bytes, stream, p.a); break;
    case 12: launch_tiled(tile16::conv_kernel<2, 1, BORDER>, p.grid, p.lds_bytes, stream, p.a); break;
    case 14: launch_tiled(tile16::conv_kernel<4, 1, BORDER>, p.grid, p.lds_bytes, stream, p.a); break;
    case 16:
      if constexpr (!BORDER) launch_tiled(tile16::conv_kernel<6, 1, false>, p.grid, p.lds_bytes, stream, p.a);
      break;
    case 21: launch_tiled(tile16::conv_kernel<1, 2, BORDER>, p.grid, p.lds_bytes, stream, p.a); break;
    case 22: launch_tiled(tile16::conv_kernel<2, 2, BORDER>, p.grid, p.lds_bytes, stream, p.a); break;
    default: launch_tiled(tile16::conv_kernel<4, 2, BORDER>, p.grid, p.lds_bytes, stream, p.a); break;
  }
  return launched();
}

int launch_tile16_conv(const Tile16ConvPlan& p, hipStream_t stream) {
  const bool border = p.a.t.pady || p.a.t.padx || p.a.t.strips > 1;
  return border ? launch_tile16_conv_as<true>(p, stream) : launch_tile16_conv_as<false>(p, stream);
}

// Forward and input gradient in reduced precision: items of eight channels on the bf16 matrix cores, or the fp32 kernel
// with its operands rounded in LDS, whichever the two fits say is faster.  With few channels most of an item is zeros, and a
// small call is over before its items are made.  ROUND_CLOCKS per 1024 floats of a unit's staged planes and ROUND_UNIT_CLOCKS for
// the barrier behind them were fitted to 224 timed calls; the margin keeps calls where the fits err with the items (4 of the 85
// calls that change are more than 3 % slower, 5 % at most).  Measured, us, items / rounded: 680 images 2 -> 2 of 29 x 22, 3 x 3
// 12.4 / 8.2; 1000 images 1 -> 1 of 40 x 40, 7 x 7 20.6 / 15.0; 3 images 6 -> 5 of 6 x 18, one tap 5.3 / 4.8; 1500 images 7 -> 9 of
// 20 x 20, 3 x 3 17.8 / 26.2.
struct Conv16Plan {
  Tile16ConvPlan items;
  TileConvPlan rounded;
  bool use_rounded() const {
    constexpr double ROUND_CLOCKS = 190.0, ROUND_UNIT_CLOCKS = 140.0, MARGIN = 1.1;
    if (rounded.mt != 1) return false;
    if (!items.nt) return true;
    const double per_cu = (double)ceil_div((long long)rounded.a.units * rounded.grid.y, NUM_CU) * rounded.a.chunks;
    const double rounding = per_cu * (ROUND_CLOCKS * up(tile::conv_lds(rounded.a).buf, 1024) + ROUND_UNIT_CLOCKS);
    return MARGIN * (rounded.cost + rounding) < items.cost;
  }
};

Conv16Plan plan_conv16(const float* src, const float* w, const float* bias, float* dst, int B, int M, int SC,
                       int SH, int SW, int KH, int KW, int OH, int OW, int pady, int padx, int flip) {
  Conv16Plan p;
  p.items = plan_tile16_conv(src, w, bias, dst, B, M, SC, SH, SW, KH, KW, OH, OW, pady, padx, flip);
  p.rounded = plan_tile_conv(src, w, bias, dst, B, M, SC, SH, SW, KH, KW, OH, OW, pady, padx, flip);
  return p;
}

int launch_conv16(const Conv16Plan& p, hipStream_t stream) {
  return p.use_rounded() ? launch_tile_conv_rounded(p.rounded, stream) : launch_tile16_conv(p.items, stream);
}

struct Tile16WgradPlan {
  tile16::WgradArgs a;
  int nt = 0, mt = 0;
  dim3 grid;
  size_t lds_bytes = 0, workspace_bytes = 0;
  double cost = 0.0;
};

bool tile16_wgrad_form(Tile16WgradPlan& p, const Tile16WgradPlan& best, int P, int mt, int nt) {
  tile16::WgradArgs& a = p.a;
  a.P = P, a.MR = a.Cout * P, a.KWP = a.KW + P - 1, a.WOP = a.Wo / P;
  a.K = a.Cin * a.KH * a.KWP, a.MT = up(a.MR, 16), a.NT = up(a.K, 16);
  a.TG = P == 1 ? 16 * nt : 16 * nt / a.KWP * a.KWP;
  if (a.TG < 1) return false;
  if (a.TG > a.K) a.TG = a.K;
  a.NTG = up(a.K, a.TG);
  a.groups = (int)ceil_div(a.B, 8);
  p.nt = nt, p.mt = mt;
  const double rounds = (double)a.groups * a.Ho * a.WOP / 16.0 * up(a.MT, mt) * a.NTG / NUM_CU;
  return !best.nt || 450.0 * nt * mt + rounds * 49.0 * nt * mt + 12000.0 < best.cost;
}

void tile16_wgrad_candidates(Tile16WgradPlan& best, Tile16WgradPlan& p, int TH, int few) {
  tile16::WgradArgs& a = p.a;
  const int plane = a.H * a.W, KHKWP = a.KH * a.KWP, MB = up(a.MT, p.mt), nt = p.nt, mt = p.mt;
  a.TH = TH, a.bands = up(a.Ho, TH);
  const long long units = (long long)a.groups * a.bands;
  if (units > 0x3fffffff) return;
  a.units = (int)units;
  const double blocks = (double)ceil_div((long long)TH * a.WOP, 4 * tile::WAVES), work = (double)units * MB * a.NTG / NUM_CU;
  if (best.nt && 450.0 * nt * mt + (work > 1.0 ? work : 1.0) * (blocks * 49.0 * nt * mt + 207.0) + 12000.0 * up(a.units, tile_columns(a.units, MB * a.NTG, 4)) >= best.cost)
    return;
  a.RS = a.Cout * a.Cin * a.KH * a.KW + a.Cout;
  const long long cg = a.NTG == 1 ? a.Cin : (a.TG + KHKWP - 2LL) / KHKWP + 1;
  a.CG = (int)(cg < a.Cin ? cg : a.Cin);
  const int R = a.MR < 16 * mt ? a.MR : 16 * mt;
  a.CO = R / a.P;
  a.RH = a.bands == 1 ? a.H : TH + a.KH - 1;
  if ((long long)a.CG * a.RH * a.W > TILE_LDS_LIMIT / 32 || (long long)a.CO * TH * a.Wo > TILE_LDS_LIMIT / 32) return;
  a.LP = a.RH * a.W, a.LI = a.CG * a.LP;
  a.DL = TH * a.Wo, a.DI = a.CO * a.DL, a.DP = a.DL | 1;
  a.N = TH * a.WOP, a.NBK = up(a.N, 4);
  a.vec_x = plane % 4 == 0 && a.LP % 4 == 0 && (a.bands == 1 || TH * a.W % 4 == 0) ? 16 : 4;
  if (a.bands == 1 && a.NTG == 1 && (long long)a.Cin * plane % 4 == 0) a.vec_x = 16;  // (runs of whole images)
  const int HoWo = a.Ho * a.Wo;
  a.vec_d = a.bands == 1 ? ((long long)a.Cout * HoWo % 4 == 0 && a.CO * HoWo % 4 == 0 && 16 * mt / a.P * HoWo % 4 == 0 ? 16 : 4) : (HoWo % 4 == 0 && a.DL % 4 == 0 ? 16 : 4);
  if (a.MT > mt && a.bands == 1 && a.Cout % a.CO * HoWo % 4) a.vec_d = 4;
  const long long end = 4ll * tile::wgrad_end_floats(nt, mt), all = tile16::wgrad_lds(a).total, lds = all > end ? all : end;
  if (lds > TILE_LDS_LIMIT) return;
  const int regs = 4 * nt * mt + 9 * nt + 8 * mt + 50;
  const int resident = std::min(CU_LDS / ((int)lds + 512), 512 / regs);
  const double x_instr = 8.0 * (a.bands == 1 ? up(a.CG * a.LP, 16 * a.vec_x) : a.CG * up(a.LP, 16 * a.vec_x));
  const double d_instr = 8.0 * (a.bands == 1 ? up(a.CO * HoWo, 16 * a.vec_d) : a.CO * up(a.DL, 16 * a.vec_d));
  for (int res = few; res <= 4 && res <= resident && (res <= 1 || (double)a.units * MB * a.NTG > NUM_CU * (res - 1.0)); ++res) {
    const int gx = tile_columns(a.units, MB * a.NTG, res);
    const long long total = (long long)gx * MB * a.NTG, wgs = total > NUM_CU ? ceil_div(total, NUM_CU) : 1;
    const double share = total > NUM_CU ? (double)total / NUM_CU : 1.0, turns = up(a.units, gx);
    const double cost = 450.0 * wgs * nt * mt + turns * (share * (blocks * 49.0 * nt * mt + 10.0 * x_instr + 22.0 * d_instr + 207.0) + 12000.0) +
                        (gx > 1 ? 13400.0 + 0.0193 * gx * a.RS : 0.0);
    if (best.nt && cost >= best.cost) continue;
    p.cost = cost, p.lds_bytes = (size_t)lds;
    p.grid = dim3((unsigned)gx, (unsigned)(MB * a.NTG));
    p.workspace_bytes = gx > 1 ? (size_t)gx * a.RS * sizeof(float) : 0;
    best = p;
  }
}

Tile16WgradPlan plan_tile16_wgrad(int B, int Cin, int H, int W, int Cout, int KH, int KW) {
  static PlanMemo<Tile16WgradPlan, 7> memo;
  return memo.get({B, Cin, H, W, Cout, KH, KW}, [&] {
    Tile16WgradPlan best, p;
    tile16::WgradArgs& a = p.a;
    a.in = a.d_out = nullptr, a.out_k = a.out_b = nullptr;
    a.B = B, a.Cin = Cin, a.H = H, a.W = W, a.Cout = Cout, a.KH = KH, a.KW = KW, a.Ho = H - KH + 1, a.Wo = W - KW + 1;
    const long long K = (long long)Cin * KH * KW;
    if ((long long)Cin * H * W > (1ll << 29) || (long long)H * W >= tile::FAR_SIZE / 4 || 16 * K > (1 << 22)) return best;
    if (ceil_div(Cout, 16) * ceil_div(K, 16) > 60000) return best;
    for (int P = 1; P <= a.Wo && (P == 1 || (KW > 1 && P * Cout <= 16)); ++P) {
      if (a.Wo % P) continue;
      for (int mt = 1; mt <= (Cout > 16 ? 2 : 1); ++mt) {
        const int NT = up(Cin * KH * (KW + P - 1), 16);
        for (int nt : {1, 2, 3, 4, 6, 8, 12}) {
          if (nt * mt > 16 || (nt > 1 && nt / 2 >= NT) || 16 * nt < KW + P - 1 || !tile16_wgrad_form(p, best, P, mt, nt)) continue;
          for (int TH = 1; TH <= a.Ho; ++TH)
            if (TH <= 2 || up(a.Ho, TH) != up(a.Ho, TH - 1)) tile16_wgrad_candidates(best, p, TH, B > 64 ? 1 : 0);
        }
      }
    }
    if (best.nt) {
      tile16::WgradArgs& b = best.a;
      b.inv_khkwp = 1.0f / (float)(KH * b.KWP), b.inv_kwp = 1.0f / (float)b.KWP, b.inv_wop = 1.0f / (float)b.WOP;
      b.inv_dl = 1.0f / (float)b.DL;
      b.by_band = tile::fast_div(b.bands);
    }
    return best;
  });
}

int launch_tile16_wgrad(Tile16WgradPlan& p, const float* in, const float* d_out, float* d_k, float* d_bias, float* part,
                        hipStream_t st) {
  const int nk = p.a.RS - p.a.Cout, G = (int)p.grid.x;
  p.a.in = in, p.a.d_out = d_out, p.a.out_k = G > 1 ? part : d_k, p.a.out_b = G > 1 ? part + nk : d_bias;
#define CNN_TILE_WGRAD(NT, MT) \
  case 100 * MT + NT: launch_tiled(tile16::wgrad_kernel<NT, MT>, p.grid, p.lds_bytes, st, p.a); break
  switch (100 * p.mt + p.nt) {
    CNN_TILE_WGRAD(1, 1);
    CNN_TILE_WGRAD(2, 1);
    CNN_TILE_WGRAD(3, 1);
    CNN_TILE_WGRAD(4, 1);
    CNN_TILE_WGRAD(6, 1);
    CNN_TILE_WGRAD(8, 1);
    CNN_TILE_WGRAD(12, 1);
    CNN_TILE_WGRAD(1, 2);
    CNN_TILE_WGRAD(2, 2);
    CNN_TILE_WGRAD(3, 2);
    CNN_TILE_WGRAD(4, 2);
    CNN_TILE_WGRAD(6, 2);
    CNN_TILE_WGRAD(8, 2);
    default: return CNN_EINVAL;
  }
#undef CNN_TILE_WGRAD
  return launch_reduce_rows(part, G, p.a.RS, nk, d_k, d_bias, st);
}

// The weight gradient in reduced precision: eight images at a time on the bf16 matrix cores, or (few images, few
// operands) the fp32 kernel with rounded operands, whichever the two fits say is faster; the factor is what rounding
// costs that kernel's vector unit.  Measured (us, eight images / rounded): 10000 images 6 -> 12 of 12 x 12, 5 x 5 taps
// 28.8 / 67; 256 images 16 -> 32 of 28 x 28, 3 x 3 taps 59 / 45; 900 images 4 -> 30 of 31 x 18, 3 x 3 taps 47 / 33; 172 layers
// with this rule 1.4 % slower than with the faster of the two for each.
struct Wgrad16Plan {
  Tile16WgradPlan eight;
  TileWgradPlan rounded;
  bool use_rounded() const { return rounded.nt && (!eight.nt || 1.08 * rounded.cost < eight.cost); }
  bool use_plain() const { return !rounded.nt && (!eight.nt || (rounded.cost > 0.0 && rounded.cost < eight.cost)); }
  size_t workspace_bytes() const { return use_plain() ? 0 : std::max(use_rounded() ? rounded.workspace_bytes : eight.workspace_bytes, NO_PARTIAL_SUMS_BYTES); }
};

Wgrad16Plan plan_wgrad16(int B, int Cin, int H, int W, int Cout, int KH, int KW) {
  Wgrad16Plan p;
  p.eight = plan_tile16_wgrad(B, Cin, H, W, Cout, KH, KW);
  p.rounded = plan_tile_wgrad(B, Cin, H, W, Cout, KH, KW, true);
  return p;
}

int launch_wgrad16(Wgrad16Plan& p, const float* in, const float* d_out, float* d_k, float* d_bias, float* part, hipStream_t st) {
  return p.use_rounded() ? launch_tile_wgrad<true>(p.rounded, in, d_out, d_k, d_bias, part, st)
                         : launch_tile16_wgrad(p.eight, in, d_out, d_k, d_bias, part, st);
}

inline bool conv_args_ok(int B, int Cin, int H, int W, int Cout, int KH, int KW) {
  return B >= 1 && Cin >= 1 && Cout >= 1 && KH >= 1 && KW >= 1 && H >= KH && W >= KW &&
         (size_t)Cout * Cin * KH * KW + (size_t)Cout < (size_t)1 << 30;
}

inline bool wgrad_args_ok(const float* in, const float* d_out, const float* d_k, const float* d_bias, int B, int Cin,
                          int H, int W, int Cout, int KH, int KW) {
  return in && d_out && d_k && conv_args_ok(B, Cin, H, W, Cout, KH, KW) && aligned16(in) && aligned16(d_out) &&
         aligned16(d_k) && (!d_bias || aligned16(d_bias));
}

// The matrix-core weight gradient: partial tiles per workgroup column into `part`, then the
// fixed-order sum of the columns.
int launch_wgrad(WgradPlan& p, const float* in, const float* d_out, float* d_k, float* d_bias, int B, int Cin, int Cout,
                 int KH, int KW, float* part, hipStream_t st) {
  switch (p.kernel) {
    case WgradPlan::TILED: return launch_tile_wgrad<false>(p.tile, in, d_out, d_k, d_bias, part, st);
    case WgradPlan::FC:
      if (B <= fc::DIRECT_MAX_ROWS) {
        fc::bwd_weight_direct_kernel<<<fc::NT, fc::WGRAD_THREADS, 0, st>>>(in, d_out, d_k, d_bias, B);
        return launched();
      }
      fc::bwd_weight_kernel<<<p.gx, fc::WGRAD_THREADS, 0, st>>>(in, d_out, part, B);
      break;
    case WgradPlan::CONV1: launch_conv1_wgrad(in, d_out, part, B, p.gx, st); break;
    case WgradPlan::CONV2: launch_conv2_wgrad(in, d_out, part, B, p.gx, st); break;
    default: return CNN_EINVAL;
  }
  const size_t outputs = (size_t)Cout * Cin * KH * KW + Cout;
  const int epw = p.kernel == WgradPlan::CONV1 ? 4 : 8;  // outputs per workgroup of the second kernel: 156 of the first layer, 1812 and 1930
  const auto second = p.kernel == WgradPlan::CONV1 ? igemm::wgrad_reduce_kernel<4, 2> : igemm::wgrad_reduce_kernel<8, 1>;
  second<<<(unsigned)((outputs + epw - 1) / epw), igemm::THREADS, 0, st>>>(part, (int)p.gx, p.NT, Cout, Cin, KH, KW, d_k, d_bias);
  return launched();
}

int launch_wgrad_plain(const float* in, const float* d_out, float* d_k, float* d_bias, int B, int Cin, int H, int W,
                       int Cout, int KH, int KW, hipStream_t st) {
  const unsigned blocks = (unsigned)(Cout * Cin * KH * KW + (d_bias ? Cout : 0));
  conv_bwd_weight_kernel<false><<<blocks, TPB, 0, st>>>(in, d_out, d_k, d_bias, B, Cin, H, W, Cout, KH, KW);
  return launched();
}

// ---- built-in scratch for callers that cannot allocate ----------------------------------------------
// Device memory that belongs to the loaded code object: every GPU the library runs on holds its own
// copy at its own address until the process ends.  In host code the array's name is only a handle
// for hipGetSymbolAddress; kernels get the address that call returned for the current device.
constexpr size_t SCRATCH_FLOATS = CNN_STATIC_SCRATCH_BYTES / sizeof(float);
static __device__ __align__(256) float scratch[SCRATCH_FLOATS];
constexpr int SCRATCH_MAX_DEVICES = 64;

// The current device's copy of `scratch`, looked up once per device.
int scratch_of_current_device(float** out) {
  static float* ptr[SCRATCH_MAX_DEVICES] = {};
  static std::mutex guard;
  int dev = -1;
  CNN_HIP_TRY(hipGetDevice(&dev));
  if (dev < 0 || dev >= SCRATCH_MAX_DEVICES) return CNN_EINVAL;
  std::lock_guard<std::mutex> lock(guard);
  if (!ptr[dev]) {
    void* p = nullptr;
    CNN_HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p) return CNN_EHIP;
    ptr[dev] = static_cast<float*>(p);
  }
  *out = ptr[dev];
  return CNN_OK;
}

// Workgroups of the fully connected layer's row kernels: one tile of sixteen rows per wave while the
// machine has room, then the waves loop.
unsigned fc_groups(int B) {
  const long long tiles = ((long long)B + fc::TILE - 1) / fc::TILE;
  const long long groups = (tiles + fc::WAVES_PER_GROUP - 1) / fc::WAVES_PER_GROUP, resident = 4LL * NUM_CU;
  return (unsigned)(groups < resident ? groups : resident);
}

}  // namespace

extern "C" {

int cnn_conv_fwd(const float* in, const float* k, const float* bias, float* out, int B, int Cin, int H,
                 int W, int Cout, int KH, int KW, void* hip_stream) {
  if (!in || !k || !out || !conv_args_ok(B, Cin, H, W, Cout, KH, KW)) return CNN_EINVAL;
  if (!aligned16(in) || !aligned16(k) || !aligned16(out) || (bias && !aligned16(bias))) return CNN_EINVAL;
  if (conv1::shape_fits(Cin, H, W, Cout, KH, KW))  // the network's first convolution
    return launch_conv1_fwd<false>(in, k, bias, out, B, (hipStream_t)hip_stream);
  if (conv2::shape_fits(Cin, H, W, Cout, KH, KW)) {  // the network's second convolution
    launch_conv2_fwd(in, k, bias, out, B, (hipStream_t)hip_stream);
    return launched();
  }
  const TileConvPlan p = plan_tile_conv(in, k, bias, out, B, Cout, Cin, H, W, KH, KW, H - KH + 1, W - KW + 1, 0, 0, 0);
  if (p.nt) return launch_tile_conv(p, (hipStream_t)hip_stream);
  const size_t total = (size_t)B * Cout * (H - KH + 1) * (W - KW + 1);
  conv_fwd_kernel<false><<<grid_for(total), TPB, 0, (hipStream_t)hip_stream>>>(in, k, bias, out, total, Cin,
                                                                                H, W, Cout, KH, KW);
  return launched();
}

int cnn_conv_bwd_input(const float* d_out, const float* k, float* d_in, int B, int Cin, int H, int W,
                       int Cout, int KH, int KW, void* hip_stream) {
  if (!d_out || !k || !d_in || !conv_args_ok(B, Cin, H, W, Cout, KH, KW)) return CNN_EINVAL;
  if (!aligned16(d_out) || !aligned16(k) || !aligned16(d_in)) return CNN_EINVAL;
  if (col2im::shape_fits(Cin, H, W, Cout, KH, KW)) {  // the network's second convolution
    launch_conv2_bwd_input(d_out, k, d_in, B, (hipStream_t)hip_stream);
    return launched();
  }
  if (conv1::shape_fits(Cin, H, W, Cout, KH, KW)) return launch_conv1_bwd_input<false>(d_out, k, d_in, B, (hipStream_t)hip_stream);
  const TileConvPlan p = plan_tile_conv(d_out, k, nullptr, d_in, B, Cin, Cout, H - KH + 1, W - KW + 1, KH, KW, H, W,
                                        KH - 1, KW - 1, 1);
  if (p.nt) return launch_tile_conv(p, (hipStream_t)hip_stream);
  const size_t total = (size_t)B * Cin * H * W;
  conv_bwd_input_kernel<false><<<grid_for(total), TPB, 0, (hipStream_t)hip_stream>>>(d_out, k, d_in, total,
                                                                                      Cin, H, W, Cout, KH, KW);
  return launched();
}

int cnn_conv_fwd_valu(const float* in, const float* k, const float* bias, float* out, int B, int Cin, int H,
                      int W, int Cout, int KH, int KW, void* hip_stream) {
  if (!in || !k || !out || !conv_args_ok(B, Cin, H, W, Cout, KH, KW)) return CNN_EINVAL;
  if (!aligned16(in) || !aligned16(k) || !aligned16(out) || (bias && !aligned16(bias))) return CNN_EINVAL;
  const size_t total = (size_t)B * Cout * (H - KH + 1) * (W - KW + 1);
  conv_fwd_kernel<false><<<grid_for(total), TPB, 0, (hipStream_t)hip_stream>>>(in, k, bias, out, total, Cin,
                                                                                H, W, Cout, KH, KW);
  return launched();
}

int cnn_conv_bwd_input_valu(const float* d_out, const float* k, float* d_in, int B, int Cin, int H, int W,
                            int Cout, int KH, int KW, void* hip_stream) {
  if (!d_out || !k || !d_in || !conv_args_ok(B, Cin, H, W, Cout, KH, KW)) return CNN_EINVAL;
  if (!aligned16(d_out) || !aligned16(k) || !aligned16(d_in)) return CNN_EINVAL;
  const size_t total = (size_t)B * Cin * H * W;
  conv_bwd_input_kernel<false><<<grid_for(total), TPB, 0, (hipStream_t)hip_stream>>>(d_out, k, d_in, total,
                                                                                      Cin, H, W, Cout, KH, KW);
  return launched();
}

int cnn_conv_fwd_bf16(const float* in, const float* k, const float* bias, float* out, int B, int Cin, int H,
                      int W, int Cout, int KH, int KW, void* hip_stream) {
  if (!in || !k || !out || !conv_args_ok(B, Cin, H, W, Cout, KH, KW)) return CNN_EINVAL;
  if (!aligned16(in) || !aligned16(k) || !aligned16(out) || (bias && !aligned16(bias))) return CNN_EINVAL;
  if (conv1::shape_fits(Cin, H, W, Cout, KH, KW)) return launch_conv1_fwd<true>(in, k, bias, out, B, (hipStream_t)hip_stream);
  const Conv16Plan p = plan_conv16(in, k, bias, out, B, Cout, Cin, H, W, KH, KW, H - KH + 1, W - KW + 1, 0, 0, 0);
  if (p.use_rounded() || p.items.nt) return launch_conv16(p, (hipStream_t)hip_stream);
  const size_t total = (size_t)B * Cout * (H - KH + 1) * (W - KW + 1);
  conv_fwd_kernel<true><<<grid_for(total), TPB, 0, (hipStream_t)hip_stream>>>(in, k, bias, out, total, Cin,
                                                                               H, W, Cout, KH, KW);
  return launched();
}

int cnn_conv_bwd_input_bf16(const float* d_out, const float* k, float* d_in, int B, int Cin, int H, int W,
                            int Cout, int KH, int KW, void* hip_stream) {
  if (!d_out || !k || !d_in || !conv_args_ok(B, Cin, H, W, Cout, KH, KW)) return CNN_EINVAL;
  if (!aligned16(d_out) || !aligned16(k) || !aligned16(d_in)) return CNN_EINVAL;
  // (one wave per image: 85 -> 55 us at 10000 images, as fast as the other forms at 1000, 7.8 -> 12 us at 64)
  if (B > SPLIT_IMAGES && conv1::shape_fits(Cin, H, W, Cout, KH, KW))
    return launch_conv1_bwd_input<true>(d_out, k, d_in, B, (hipStream_t)hip_stream);
  const Conv16Plan p = plan_conv16(d_out, k, nullptr, d_in, B, Cin, Cout, H - KH + 1, W - KW + 1, KH, KW, H, W,
                                   KH - 1, KW - 1, 1);
  if (p.use_rounded() || p.items.nt) return launch_conv16(p, (hipStream_t)hip_stream);
  const size_t total = (size_t)B * Cin * H * W;
  conv_bwd_input_kernel<true><<<grid_for(total), TPB, 0, (hipStream_t)hip_stream>>>(d_out, k, d_in, total,
                                                                                     Cin, H, W, Cout, KH, KW);
  return launched();
}

size_t cnn_conv_bwd_weight_workspace_bytes(int B, int Cin, int H, int W, int Cout, int KH, int KW) {
  if (!conv_args_ok(B, Cin, H, W, Cout, KH, KW)) return 0;
  return plan_wgrad(B, Cin, H, W, Cout, KH, KW).workspace_bytes;
}

int cnn_conv_bwd_weight(const float* in, const float* d_out, float* d_k, float* d_bias, int B, int Cin,
                        int H, int W, int Cout, int KH, int KW, void* workspace, size_t workspace_bytes,
                        void* hip_stream) {
  if (!wgrad_args_ok(in, d_out, d_k, d_bias, B, Cin, H, W, Cout, KH, KW)) return CNN_EINVAL;
  if (workspace && !aligned16(workspace)) return CNN_EINVAL;
  WgradPlan p = plan_wgrad(B, Cin, H, W, Cout, KH, KW);
  if (fit_wgrad(p, workspace ? workspace_bytes : 0))
    return launch_wgrad(p, in, d_out, d_k, d_bias, B, Cin, Cout, KH, KW, static_cast<float*>(workspace), (hipStream_t)hip_stream);
  return launch_wgrad_plain(in, d_out, d_k, d_bias, B, Cin, H, W, Cout, KH, KW, (hipStream_t)hip_stream);
}

int cnn_conv_bwd_weight_static(const float* in, const float* d_out, float* d_k, float* d_bias, int B, int Cin,
                               int H, int W, int Cout, int KH, int KW, void* hip_stream) {
  if (!wgrad_args_ok(in, d_out, d_k, d_bias, B, Cin, H, W, Cout, KH, KW)) return CNN_EINVAL;
  WgradPlan p = plan_wgrad(B, Cin, H, W, Cout, KH, KW);
  if (p.kernel == WgradPlan::PLAIN)  // only the kernel without partial sums serves this shape: it needs no scratch at all
    return launch_wgrad_plain(in, d_out, d_k, d_bias, B, Cin, H, W, Cout, KH, KW, (hipStream_t)hip_stream);
  if (p.workspace_bytes > sizeof(float) * SCRATCH_FLOATS) return CNN_ESCRATCH;
  float* part = nullptr;
  const int rc = scratch_of_current_device(&part);
  if (rc != CNN_OK) return rc;
  // every partial tile and bias row the second kernel reads is written by the first one in the same
  // call, so nothing of the previous call's contents has to be cleared
  return launch_wgrad(p, in, d_out, d_k, d_bias, B, Cin, Cout, KH, KW, part, (hipStream_t)hip_stream);
}

size_t cnn_conv_bwd_weight_bf16_workspace_bytes(int B, int Cin, int H, int W, int Cout, int KH, int KW) {
  if (!conv_args_ok(B, Cin, H, W, Cout, KH, KW)) return 0;
  // in whole rows of padded 16 x 16 tiles and biases, the unit this query has always had
  const size_t rows = ceil_div(Cout, 16), row = sizeof(float) * rows * (ceil_div((long long)Cin * KH * KW, 16) * 256 + 16);
  return ceil_div(plan_wgrad16(B, Cin, H, W, Cout, KH, KW).workspace_bytes(), row) * row;
}

int cnn_conv_bwd_weight_bf16(const float* in, const float* d_out, float* d_k, float* d_bias, int B, int Cin,
                             int H, int W, int Cout, int KH, int KW, void* workspace, size_t workspace_bytes,
                             void* hip_stream) {
  if (!in || !d_out || !d_k || !conv_args_ok(B, Cin, H, W, Cout, KH, KW)) return CNN_EINVAL;
  if (!aligned16(in) || !aligned16(d_out) || !aligned16(d_k) || (d_bias && !aligned16(d_bias)))
    return CNN_EINVAL;
  if (workspace && !aligned16(workspace)) return CNN_EINVAL;
  Wgrad16Plan p = plan_wgrad16(B, Cin, H, W, Cout, KH, KW);
  if (!p.use_plain() && workspace && workspace_bytes >= p.workspace_bytes())
    return launch_wgrad16(p, in, d_out, d_k, d_bias, static_cast<float*>(workspace), (hipStream_t)hip_stream);
  const unsigned blocks = (unsigned)(Cout * Cin * KH * KW + (d_bias ? Cout : 0));
  conv_bwd_weight_kernel<true><<<blocks, TPB, 0, (hipStream_t)hip_stream>>>(in, d_out, d_k, d_bias, B, Cin, H,
                                                                            W, Cout, KH, KW);
  return launched();
}

int cnn_avgpool_fwd(const float* in, float* out, int B, int C, int H, int W, void* hip_stream) {
  if (!in || !out || B < 1 || C < 1 || H < 2 || W < 2 || (H & 1) || (W & 1)) return CNN_EINVAL;
  if (!aligned16(in) || !aligned16(out)) return CNN_EINVAL;
  return pool<true>(in, out, (size_t)B * C * (H / 2) * (W / 2), W, (hipStream_t)hip_stream);
}

int cnn_avgpool_bwd(const float* d_out, float* d_in, int B, int C, int Ho, int Wo, void* hip_stream) {
  if (!d_out || !d_in || B < 1 || C < 1 || Ho < 1 || Wo < 1) return CNN_EINVAL;
  if (!aligned16(d_out) || !aligned16(d_in)) return CNN_EINVAL;
  return pool<false>(d_out, d_in, (size_t)B * C * Ho * Wo, 2 * (size_t)Wo, (hipStream_t)hip_stream);
}

int cnn_fc_fwd(const float* in, const float* w, const float* bias, float* out, int B, int I, int O,
               void* hip_stream) {
  if (!in || !w || !out || B < 1 || I < 1 || O < 1) return CNN_EINVAL;
  if (!aligned16(in) || !aligned16(w) || !aligned16(out) || (bias && !aligned16(bias))) return CNN_EINVAL;
  if (fc::shape_fits(I, O)) {
    // the shape of the network's own layer: every wave takes tiles of sixteen rows straight from global memory
    fc::forward_kernel<<<fc_groups(B), fc::THREADS, 0, (hipStream_t)hip_stream>>>(in, w, bias, out, B);
    return launched();
  }
  const TileConvPlan p = plan_tile_conv(in, w, bias, out, B, O, I, 1, 1, 1, 1, 1, 1, 0, 0, 0);
  if (p.nt) return launch_tile_conv(p, (hipStream_t)hip_stream);
  const size_t total = (size_t)B * O;
  fc_fwd_kernel<<<grid_for(total), TPB, 0, (hipStream_t)hip_stream>>>(in, w, bias, out, total, I, O);
  return launched();
}

int cnn_fc_bwd_input(const float* d_out, const float* w, float* d_in, int B, int I, int O,
                     void* hip_stream) {
  if (!d_out || !w || !d_in || B < 1 || I < 1 || O < 1) return CNN_EINVAL;
  if (!aligned16(d_out) || !aligned16(w) || !aligned16(d_in)) return CNN_EINVAL;
  if (fc::shape_fits(I, O)) {
    fc::bwd_input_kernel<<<fc_groups(B), fc::THREADS, 0, (hipStream_t)hip_stream>>>(d_out, w, d_in, B);
    return launched();
  }
  const TileConvPlan p = plan_tile_conv(d_out, w, nullptr, d_in, B, I, O, 1, 1, 1, 1, 1, 1, 0, 0, 1);
  if (p.nt) return launch_tile_conv(p, (hipStream_t)hip_stream);
  const size_t total = (size_t)B * I;
  fc_bwd_input_kernel<<<grid_for(total), TPB, 0, (hipStream_t)hip_stream>>>(d_out, w, d_in, total, I, O);
  return launched();
}

size_t cnn_fc_bwd_weight_workspace_bytes(int B, int I, int O) {
  return cnn_conv_bwd_weight_workspace_bytes(B, I, 1, 1, O, 1, 1);
}

int cnn_fc_bwd_weight(const float* in, const float* d_out, float* d_w, float* d_bias, int B, int I, int O,
                      void* workspace, size_t workspace_bytes, void* hip_stream) {
  if (!in || !d_out || !d_w || B < 1 || I < 1 || O < 1 || (size_t)I * O + O >= (size_t)1 << 30)
    return CNN_EINVAL;
  if (!aligned16(in) || !aligned16(d_out) || !aligned16(d_w) || (d_bias && !aligned16(d_bias)))
    return CNN_EINVAL;
  if (workspace && !aligned16(workspace)) return CNN_EINVAL;
  WgradPlan p = plan_wgrad(B, I, 1, 1, O, 1, 1);
  if (fit_wgrad(p, workspace ? workspace_bytes : 0))
    return launch_wgrad(p, in, d_out, d_w, d_bias, B, I, O, 1, 1, static_cast<float*>(workspace), (hipStream_t)hip_stream);
  const unsigned blocks = (unsigned)(O * I + (d_bias ? O : 0));
  fc_bwd_weight_kernel<<<blocks, TPB, 0, (hipStream_t)hip_stream>>>(in, d_out, d_w, d_bias, B, I, O);
  return launched();
}

int cnn_logistic_fwd(const float* x, float* y, size_t n, void* hip_stream) {
  if (!x || !y || n < 1 || !aligned16(x) || !aligned16(y)) return CNN_EINVAL;
  logistic_fwd_kernel<<<grid_stream((n + 3) / 4), TPB, 0, (hipStream_t)hip_stream>>>(x, y, n);
  return launched();
}

int cnn_logistic_bwd(const float* y, const float* d_y, float* d_x, size_t n, void* hip_stream) {
  if (!y || !d_y || !d_x || n < 1 || !aligned16(y) || !aligned16(d_y) || !aligned16(d_x))
    return CNN_EINVAL;
  logistic_bwd_kernel<<<grid_stream((n + 3) / 4), TPB, 0, (hipStream_t)hip_stream>>>(y, d_y, d_x, n);
  return launched();
}

}  // extern "C"
