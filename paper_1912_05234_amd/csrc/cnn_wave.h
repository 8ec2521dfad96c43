// What the kernels of the fused step share: the expanded operand table, the fp32 matrix-instruction forms of the
// convolutions' GEMMs, wave helpers.  Definitions: arXiv 1912.05234, Section 3 (forward, conv, mconv, sigmoid, avgpool,
// backweights, backbias, backin, backavgpool).  Used by the kernels with eight waves per image (cnn_group.h), those with
// one (cnn_train.h, cnn_split.h) and the single-layer kernels (cnn_conv_wave.h, cnn_col2im.h).
//
// Pixel order of C2: pixel index p = 4 w + sub, w = 4 wy + wx over the 4x4 pooling windows; tile mt covers p in
// [16mt, 16mt+16), so that avgpool is a sum inside a lane's four MFMA result registers.
// MFMA operand layouts (64 lanes, q = lane/16, n16 = lane%16):
//   16x16x4: A[i=n16][k=q], B[k=q][j=n16], D[i=4q+r][j=n16] in result register r.
//   4x4x1  : D_r(lane) += A(4*(lane/4)+r) * B(lane).
#pragma once

#include <type_traits>

#include "cnn_common.h"

// Hook for a cycle-counter probe at phase boundaries; empty in the library build.
#ifndef CNN_GROUP_MARK
#define CNN_GROUP_MARK(k)
#endif

namespace cnn {

typedef float f4 __attribute__((ext_vector_type(4)));

constexpr int D2S = 68;   // row stride of the C2 error array in LDS (floats)

// LDS of the small-batch training step (cnn_group.h; one image per workgroup).  d_s1 comes first:
// the col2im rows of the two padding maps (c = 6, 7) add 0.0 at offsets up to 1152 floats past its
// start, which stays inside the struct.  `pool` holds, at the P_* offsets, the arrays that are dead
// by the time the C1 weight gradient runs; that phase reuses the whole pool for the staged C1 error.
constexpr int P_S1 = 0;                 // s1[6][12][12] + 288 (padded K steps of the C2 forward read them)
constexpr int P_S2 = P_S1 + NS1 + 288;  // s2[192]
constexpr int P_DS2 = P_S2 + NS2;       // d_s2[192] + 64 (rows of the padding maps of the C2 tiles)
constexpr int P_D2 = P_DS2 + NS2 + 64;  // d2[16][D2S]: error at C2's pre-activation, [map][pixel p]
constexpr int P_END = P_D2 + 16 * D2S;
// The C1 error is staged over the whole pool as d1[6][24][24] with the maps D1_MAP floats apart: the
// gradient GEMM's A operand reads all six maps in one instruction, and a map stride of 576 (a
// multiple of the 32 banks) would put them on the same four banks.
constexpr int D1_MAP = 24 * 24 + 4;
// The same in chunks of eight rows, d1c[6][8][24] (the kernels with one wave per image).
constexpr int D1C_MAP = 8 * 24 + 4;
constexpr int POOL_FLOATS = 6 * D1_MAP + 32;
static_assert(POOL_FLOATS >= P_END + 4 * NS2, "pool holds the forward/C2 arrays and the upper waves' errors at S2");
struct __align__(16) TrainLds {
  float d_s1[NS1];  // error at S1 (col2im target)
  float img[NI];
  float pool[POOL_FLOATS];
};
// Shared operand table, [entry][lane].
constexpr int TAB_BF = 0;          // 38: C2 forward B operand, k2[j = n16][tap(s, q)]
constexpr int TAB_FCW = 38;        // 30: fc[o][lane + 64 k] at entry 3 o + k
constexpr int TAB_FWD_ENTRIES = 68;
constexpr int TAB_AB = 68;         // 21: C2 input-error A operand of input maps 0..3, entry tile*3 + s
constexpr int TAB_AB1 = 89;        // 21: the same for input maps 4..7 (the small-batch kernel)
constexpr int TAB_C1A = 110;       // 8: C1 forward A operand of the small-batch kernel, W[(m,sh) = n16][tap 4 ks + q]
constexpr int TAB_TRAIN_ENTRIES = 118;  // all of them; what the small-batch kernel reads
// Last: the biases read per image, bias[0..11] = b2, bias[16..25] = b, zeros elsewhere.
constexpr int TAB_BIAS_FLOATS = 32;
constexpr int TAB_BIAS_B = 16, TAB_BIAS_B1 = 26;  // bias[16..25] = b, bias[26..31] = b1
template <int ENTRIES>
struct __align__(16) OperandTable {
  float e[ENTRIES * 64];
  float bias[TAB_BIAS_FLOATS];
};
// The table is kept expanded in global memory next to the flat parameter vector (all entries, then
// bias); a kernel copies the part it needs into LDS with 16-byte loads.
constexpr int TABG_BIAS = TAB_TRAIN_ENTRIES * 64;
constexpr int TABG_FLOATS = TABG_BIAS + TAB_BIAS_FLOATS;

__device__ __forceinline__ float quad_xor1(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0xB1, 0xF, 0xF, true));
}
__device__ __forceinline__ float quad_xor2(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x4E, 0xF, 0xF, true));
}
__device__ __forceinline__ float dpp_row_half_mirror(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x141, 0xF, 0xF, true));
}
__device__ __forceinline__ float dpp_row_mirror(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x140, 0xF, 0xF, true));
}
// Sum over the 64 lanes in a fixed order, same value in every lane: quad, 8, 16 lanes by DPP,
// then the four rows of 16 through scalar registers.
__device__ __forceinline__ float wave_sum(float v) {
  v += quad_xor1(v);
  v += quad_xor2(v);
  v += dpp_row_half_mirror(v);
  v += dpp_row_mirror(v);
  const int iv = __builtin_bit_cast(int, v);
  const float r0 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(iv, 0));
  const float r1 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(iv, 16));
  const float r2 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(iv, 32));
  const float r3 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(iv, 48));
  return (r0 + r1) + (r2 + r3);
}
__device__ __forceinline__ f4 mfma16(float a, float b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f4 mfma4(float a, float b, f4 c) {
  return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, 0, 0, 0);
}
// Ordering point inside ONE wave: LDS writes issued before it by any lane are seen by LDS reads
// issued after it by any lane of the same wave.  The LDS unit executes one wave's instructions in
// order, so nothing has to be waited for; the fences only stop the compiler from moving LDS
// accesses across this point.  No other wave is involved.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ---- K order of the C2 forward GEMM: step s < 38, lane quarter q -> tap (c,u,v) -------------
// steps 0..29: (c = s/5, v = s%5), u = q            LDS offset c*144 + v      + 12 q
// steps 30..35: c = s-30, u = 4, v = q               LDS offset c*144 + 48     + q
// steps 36,37: u = v = 4, c = 4(s-36) + q (c < 6)    LDS offset 576(s-36) + 52 + 144 q
__host__ __device__ constexpr int fwd_tap(int s, int q) {
  return s < 30 ? (s / 5) * 25 + q * 5 + (s % 5)
                : s < 36 ? (s - 30) * 25 + 20 + q : (4 * (s - 36) + q < 6 ? (4 * (s - 36) + q) * 25 + 24 : -1);
}
__host__ __device__ constexpr int fwd_imm(int s) {
  return s < 30 ? (s / 5) * 144 + (s % 5) : s < 36 ? (s - 30) * 144 + 48 : 576 * (s - 36) + 52;
}
// ---- M tiles of the C2 input-error GEMM.  Row i = 4 qi + ri of every tile belongs to input map
// c = 4 cg + qi (cg = 0, 1; maps 6, 7 are zero padding) and to the tap
//   tile V(v), v < 5 : (u = ri, v)        tile U4 : (u = 4, v = ri)        tile C : (4, 4) in ri = 0 only.
// A lane's result register r of tile (cg, .) therefore lands in d_s1[c = 4 cg + q] at row y+u, column x+v.
enum BwdTile { kTileV0 = 0, kTileU4 = 5, kTileC = 6 };  // V(v) = kTileV0 + v; tile C is used by the small-batch kernel only
__host__ __device__ constexpr int bwd_tap(int tile, int ri) {
  return tile < 5 ? 5 * ri + tile : tile == kTileU4 ? 20 + ri : (ri == 0 ? 24 : -1);
}
// Packed tiles for input maps 4 and 5 (a plain tile would leave the rows of maps 6, 7 empty): rows
// qi = 0, 1 belong to map 4 + qi and the taps of columns v = 0, 1, 2; rows qi = 2, 3 to map 4 + (qi - 2)
// again and the taps of columns v = 3, 4, whose terms are added into a second copy of the two maps
// (lanes of both halves would otherwise meet in the same cells within a round).
//   tile PV(s), s < 3 : qi < 2: (u = ri, v = s)       qi >= 2: (u = ri, v = 3 + s) for s < 2, nothing for s = 2
//   tile PU           : qi < 2: (4, v = ri), ri < 3   qi >= 2: ri = 0: (4, 3), ri = 1: (4, 4)
// so that in round s every lane finds "its" u = 4 term in result register s of PU.  Register 3 of
// PU is used by no round: its rows (qi, ri = 3) take tap (4, 4) of the maps 0..3, map qi, which puts
// the term into the very lane that owns map qi when those maps are summed (the plain tile C of
// those maps would use four rows of sixteen).
// Returns 25 c + tap, or -1 for a zero row.
enum PackedTile { kTilePV0 = 0, kTilePU = 3 };
__host__ __device__ constexpr int bwd_packed_source(int tile, int qi, int ri) {
  const int c = 4 + (qi & 1);
  if (tile < 3) return qi < 2 ? 25 * c + 5 * ri + tile : (tile < 2 ? 25 * c + 5 * ri + 3 + tile : -1);
  if (ri == 3) return 25 * qi + 24;
  if (qi < 2) return 25 * c + 20 + ri;
  return ri < 2 ? 25 * c + 23 + ri : -1;
}
// ---- C1 forward as a GEMM (16x16x4 MFMA) -----------------------------------------------------------
// Output pixels are taken in horizontal pairs x = 2X + sh (sh = 0, 1).  With v' = v + sh the image
// factor img[y+u][2X+v'] does not depend on sh:
//   pre[(m,sh)][(y,X)] = b1[m] + sum_{u < 5, v' < 6} W[(m,sh)][(u,v')] * img[y+u][2X+v'],
//   W[(m,sh)][(u,v')] = k1[m][u][v'-sh]  (zero where v'-sh is outside 0..4).
// M = 12 rows (m,sh), i = 2m + sh, in one 16-row tile; K = 30 taps t = 6u + v' in 8 steps of four
// (t = 4 ks + q); N = 288 pixel pairs in 18 tiles of 16.  Tile T = 3 ty + tx covers the 2 x 4 block of
// pooling windows wy = 2 ty + a, wx = 4 tx + bx; column j = lane%16 = 4 bx + 2 a + dy is the pair
// (y = 2 wy + dy, X = wx).  Lanes j and j^1 are the two rows of one window and a lane's result
// registers of one map (sh = 0, 1) are its two columns, so avgpool is two adds and one DPP add.
//   A[i = lane%16][k = q] = W[i][4 ks + q]      (rows 12..15 and taps 30, 31 are zero)
//   B[k = q][j = lane%16] = img[y + u][2X + v']
//   D[i = 4q + r][j]: map m = 2q + r/2, sh = r%2, in result register r (lanes q = 3 hold padding rows).
constexpr int C1F_TILES = 18, C1F_KSTEPS = 8;
__host__ __device__ constexpr int c1f_weight(int ks, int lane) {  // flat parameter index or -1
  const int q = lane >> 4, i = lane & 15, t = 4 * ks + q;
  if (t >= 30 || i >= 12) return -1;
  const int u = t / 6, v = t % 6 - (i & 1);
  return v >= 0 && v < 5 ? OFF_K1 + (i >> 1) * 25 + u * 5 + v : -1;
}
// Offsets (floats) that depend on the tile only: image, pooled [6][12][12] arrays, [6][24][24] arrays.
__host__ __device__ constexpr int c1f_tile_img(int T) { return (T / 3) * 112 + (T % 3) * 8; }
__host__ __device__ constexpr int c1f_tile_s1(int T) { return (T / 3) * 24 + (T % 3) * 4; }
__host__ __device__ constexpr int c1f_tile_c1(int T) { return (T / 3) * 96 + (T % 3) * 8; }
// Offsets that depend on the lane only.
struct C1Lane {
  int img[C1F_KSTEPS];  // B operand of K step ks
  int s1;               // map 2q of a pooled array (map 2q + 1 is 144 further)
  int c1;               // map 2q, sh = 0 of the staged d1 (map 2q + 1 is D1_MAP further)
};
__device__ __forceinline__ C1Lane c1f_lane() {
  const int l = threadIdx.x & 63, q = l >> 4, n16 = l & 15;
  const int dy = n16 & 1, a = (n16 >> 1) & 1, bx = n16 >> 2;
  C1Lane o;
#pragma unroll
  for (int ks = 0; ks < C1F_KSTEPS; ++ks) {
    const int t = 4 * ks + q, tt = t < 30 ? t : 0;
    o.img[ks] = (2 * a + dy + tt / 6) * 28 + 2 * bx + tt % 6;
  }
  o.s1 = 2 * q * 144 + a * 12 + bx;
  o.c1 = 2 * q * D1_MAP + (2 * a + dy) * 24 + 2 * bx;
  return o;
}
// Pre-activations of two tiles at once (two independent accumulation chains); img0 / img1 point at
// the tiles' origins in the image.  The B operand of step ks + 1 is read while step ks issues.
__device__ __forceinline__ void c1f_gemm_pair(const float (&wa)[C1F_KSTEPS], const C1Lane& ln, const float* img0,
                                              const float* img1, f4 binit, f4& d0, f4& d1) {
  d0 = binit;
  d1 = binit;
  float x0[3], x1[3];
  x0[0] = img0[ln.img[0]];
  x1[0] = img1[ln.img[0]];
  x0[1] = img0[ln.img[1]];
  x1[1] = img1[ln.img[1]];
#pragma unroll
  for (int ks = 0; ks < C1F_KSTEPS; ++ks) {
    if (ks + 2 < C1F_KSTEPS) {
      x0[(ks + 2) % 3] = img0[ln.img[ks + 2]];
      x1[(ks + 2) % 3] = img1[ln.img[ks + 2]];
    }
    d0 = mfma16(wa[ks], x0[ks % 3], d0);
    d1 = mfma16(wa[ks], x1[ks % 3], d1);
  }
}
// The same for a single tile (one chain).
__device__ __forceinline__ void c1f_gemm_one(const float (&wa)[C1F_KSTEPS], const C1Lane& ln, const float* img0,
                                             f4 binit, f4& d0) {
  d0 = binit;
  float x0[3];
  x0[0] = img0[ln.img[0]];
  x0[1] = img0[ln.img[1]];
#pragma unroll
  for (int ks = 0; ks < C1F_KSTEPS; ++ks) {
    if (ks + 2 < C1F_KSTEPS) x0[(ks + 2) % 3] = img0[ln.img[ks + 2]];
    d0 = mfma16(wa[ks], x0[ks % 3], d0);
  }
}
// sigmoid in place, then S1 = avgpool for the tile's windows: s1 points at the tile's origin in the
// pooled array.  Lanes j and j^1 store the same value to the same cell; the padding rows of lanes
// q = 3 land in the (finite, never used) cells behind the sixth map.
__device__ __forceinline__ void c1f_finish(f4& d, const C1Lane& ln, float* s1) {
#pragma unroll
  for (int r = 0; r < 4; ++r) d[r] = logistic(d[r]);
  float p0 = d[0] + d[1], p1 = d[2] + d[3];
  p0 += quad_xor1(p0);
  p1 += quad_xor1(p1);
  s1[ln.s1] = 0.25f * p0;
  s1[ln.s1 + 144] = 0.25f * p1;
}

// Flat parameter index whose value slot i of the expanded table holds, or -1 for a zero.
__host__ __device__ constexpr int table_source(int i) {
  if (i < TABG_BIAS) {
    const int e = i >> 6, l = i & 63, q = l >> 4, n16 = l & 15;
    if (e < TAB_FCW) {
      const int tap = fwd_tap(e, q);
      return n16 < 12 && tap >= 0 ? OFF_K2 + n16 * 150 + tap : -1;
    }
    if (e < TAB_AB) {
      const int o = (e - TAB_FCW) / 3, k = (e - TAB_FCW) % 3;
      return OFF_FC + o * NS2 + l + 64 * k;
    }
    if (e >= TAB_C1A) return c1f_weight(e - TAB_C1A, l);
    const int cg = e >= TAB_AB1 ? 1 : 0, t = e - (cg ? TAB_AB1 : TAB_AB), sidx = t % 3, tile = t / 3;
    const int c = 4 * cg + (n16 >> 2), tap = bwd_tap(tile, n16 & 3);
    return c < 6 && tap >= 0 ? OFF_K2 + (4 * sidx + q) * 150 + c * 25 + tap : -1;
  }
  const int k = i - TABG_BIAS;
  return k < 12 ? OFF_B2 + k
                : k >= TAB_BIAS_B && k < TAB_BIAS_B + NY ? OFF_B + (k - TAB_BIAS_B)
                                                         : k >= TAB_BIAS_B1 ? OFF_B1 + (k - TAB_BIAS_B1) : -1;
}
// Factor a slot holds its parameter multiplied by: the forward weights and biases of both
// convolution layers carry -log2(e) (see logistic_of_scaled); the C2 input-error operand carries the
// 1/4 of the average pooling below it (backavgpool, Section 3), which the C1 error then does not apply.
__host__ __device__ constexpr float table_scale(int i) {
  if (i < TABG_BIAS) {
    const int e = i >> 6;
    return e < TAB_FCW ? NEG_LOG2E : e >= TAB_AB && e < TAB_C1A ? 0.25f : 1.0f;
  }
  return i - TABG_BIAS < 12 ? NEG_LOG2E : 1.0f;
}
// No parameter sits in more than four slots:
// the SGD kernel refreshes the expanded table by writing every updated parameter to its recorded places.
constexpr int TABLE_MAX_DEST = 4;
constexpr int table_max_multiplicity() {
  int count[NPARAM] = {};
  int most = 0;
  for (int i = 0; i < TABG_FLOATS; ++i) {
    const int p = table_source(i);
    if (p >= 0 && ++count[p] > most) most = count[p];
  }
  return most;
}

// Copies the expanded table from global memory into the workgroup's LDS in two halves, so that a
// kernel can do other set-up work while the loads are in flight: `fetch` issues all of a thread's
// 16-byte loads, `commit` stores them to LDS.  All THREADS threads of the workgroup take part and
// the caller follows the commit with a workgroup barrier.
// COHERENT: the table was written by other compute units during this kernel (the device-side
// epoch loop): its 16-byte pieces are fetched with agent-scope loads, which do not take stale lines
// from this XCD's L2 cache.
// ENTRIES counts the entries of the LDS copy, of which the first LOADED come from global memory.
// FIRST: the entry whose pieces are fetched first; `commit_first` stores those (one round of loads)
// and the tail, `commit_rest` the others, each followed by a barrier of the caller's.
// Of the entries, SKIPPED from SKIP on (before FIRST) stay where they are.
template <int ENTRIES, int THREADS, bool COHERENT = false, int LOADED = ENTRIES, int FIRST = 0, int SKIP = 0, int SKIPPED = 0>
struct TableLoad {
  static constexpr int PIECES = (LOADED - SKIPPED) * 16, ROUNDS = (PIECES + THREADS - 1) / THREADS;
  static constexpr int TAIL = TAB_BIAS_FLOATS / 4;
  typedef OperandTable<ENTRIES> Table;
  static_assert(TAIL <= THREADS, "one thread per piece of the tail");
  static_assert(FIRST >= SKIP + SKIPPED && FIRST < LOADED, "the entry fetched first is one of the loaded ones");
  f4 v[ROUNDS], tail;
  // 16-byte piece of the table that this thread moves in round r (the same in global memory and in
  // LDS), or -1: the pieces are taken in the order FIRST * 16, .., PIECES - 1, 0, .., FIRST * 16 - 1, so
  // that round 0 brings the entries from FIRST on (what the caller needs first) and loads return in
  // the order they are issued
  static __device__ __forceinline__ int piece(int r) {
    const int i = r * THREADS + (int)threadIdx.x, at = i + (FIRST - SKIPPED) * 16, of = at < PIECES ? at : at - PIECES;
    return i < PIECES ? (of < SKIP * 16 ? of : of + SKIPPED * 16) : -1;
  }
  // Issue order: round 0, the tail (biases), the other rounds.
  __device__ __forceinline__ void fetch(const float* __restrict__ tabg) {
    const int t = threadIdx.x;
    if (COHERENT) {
      const __amdgpu_buffer_rsrc_t rs =
          __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(tabg), 0, sizeof(float) * TABG_FLOATS, 0x00020000);
      constexpr int AGENT_SCOPE = 16;  // the sc1 bit of the cache policy
      typedef unsigned u4 __attribute__((ext_vector_type(4)));
      auto load = [&](int byte) { return __builtin_bit_cast(f4, (u4)__builtin_amdgcn_raw_buffer_load_b128(rs, byte, 0, AGENT_SCOPE)); };
      { const int i = piece(0); v[0] = load(16 * (i >= 0 ? i : 0)); }
      tail = load(4 * TABG_BIAS + 16 * (t < TAIL ? t : 0));
#pragma unroll
      for (int r = 1; r < ROUNDS; ++r) {
        const int i = piece(r);
        v[r] = load(16 * (i >= 0 ? i : 0));
      }
      return;
    }
    const f4* src = reinterpret_cast<const f4*>(tabg);
    { const int i = piece(0); v[0] = src[i >= 0 ? i : 0]; }
    tail = src[TABG_BIAS / 4 + (t < TAIL ? t : 0)];
#pragma unroll
    for (int r = 1; r < ROUNDS; ++r) {
      const int i = piece(r);
      v[r] = src[i >= 0 ? i : 0];
    }
  }
  // Round 0 and the tail: the entries FIRST .. (and the first ones again, as far as a round reaches).
  __device__ __forceinline__ void commit_first(Table& tab) const {
    const int t = threadIdx.x, i = piece(0);
    if (i >= 0) reinterpret_cast<f4*>(tab.e)[i] = v[0];
    if (t < TAIL) reinterpret_cast<f4*>(tab.bias)[t] = tail;
  }
  __device__ __forceinline__ void commit_rest(Table& tab) const {
#pragma unroll
    for (int r = 1; r < ROUNDS; ++r) {
      const int i = piece(r);
      if (i >= 0) reinterpret_cast<f4*>(tab.e)[i] = v[r];
    }
  }
  __device__ __forceinline__ void commit(Table& tab) const {
    commit_first(tab);
    commit_rest(tab);
  }
};
// ---- C1 weight gradient as one GEMM per image (16x16x4 MFMA) ------------------------------------
//   g_k1[m][u][v] = sum_{y,x < 24} d1[m][y][x] * img[y+u][x+v]            (backweights, Section 3)
// Pixels are taken in horizontal pairs x = 2X + sh (sh = 0, 1).  With v' = v + sh the image factor
// img[y+u][2X+v'] no longer depends on sh, so
//   T[(m,sh)][(u,v')] = sum_{y,X} d1[m][y][2X+sh] * img[y+u][2X+v'],   g_k1[m][u][v] = T[(m,0)][(u,v)] + T[(m,1)][(u,v+1)]
// is a GEMM with M = 12 rows (m,sh) in one 16-row tile, N = 30 columns (u,v'), c = 6u + v', in two
// 16-column tiles, and K = 288 pixel pairs in 72 steps of four: step kk covers row y = kk / 3 and
// pairs X = 4 (kk % 3) + q, q = lane / 16.  d1 is staged in LDS as d1[m][24][24], maps D1_MAP apart.
//   A[i = lane%16][k = q] = d1[m = (i/2) % 6][y][2X + i%2]     (rows 12..15 repeat rows 0..3, dropped)
//   B[k = q][j = lane%16] = img[y + u][2X + v'], c = 16 nt + j  (columns 30, 31 read tap 0, dropped)
//   D[i = 4q + r][j]: register r of tile nt.
constexpr int C1G_STEPS = 72;
constexpr int C1G_PARK = 16 * 32;  // floats: T as [row i][column c]
__host__ __device__ constexpr int c1g_imm_a(int kk) { return 24 * (kk / 3) + 8 * (kk % 3); }
__host__ __device__ constexpr int c1g_imm_b(int kk) { return 28 * (kk / 3) + 8 * (kk % 3); }
// Lane parts of the operand addresses (floats): d1 (maps MAP floats apart) and the two image tiles.
template <int MAP = D1_MAP>
__device__ __forceinline__ void c1g_lane_offsets(int& a, int (&bt)[2], int l) {
  const int q = l >> 4, n16 = l & 15;
  a = ((n16 >> 1) % 6) * MAP + (n16 & 1) + 2 * q;
#pragma unroll
  for (int nt = 0; nt < 2; ++nt) {
    const int c = 16 * nt + n16;
    bt[nt] = (c < 30 ? (c / 6) * 28 + c % 6 : 0) + 2 * q;
  }
}
// STEPS steps of the GEMM from the given origins of d1 and the image: operands of step kk + 2 are
// read while the two MFMAs of step kk issue.
// With `ones` (C1G_ONES floats of 1.0): the two padding columns 30, 31 read 1.0 instead of image
// pixels, so that column 30 of the result is the sum of the A operand over all steps,
//   T[(m,sh)][30] = sum_{y,X} d1[m][y][2X+sh],   g_b1[m] = T[(m,0)][30] + T[(m,1)][30]      (backbias, Section 3)
// at no cost in instructions.
constexpr int C1G_ONES = 224;  // the reach of a lane's B operand over eight image rows: 28 * 7 + 16 + 6 + 1
template <int STEPS, int MAP = D1_MAP>
__device__ __forceinline__ void c1g_accumulate(f4 (&acc)[2], const float* d1, const float* img, int lane,
                                               const float* ones = nullptr) {
  static_assert(28 * ((STEPS - 1) / 3) + 8 * 2 + 6 < C1G_ONES || STEPS > 24, "the ones cover a padding lane's reads");
  int a, bt[2];
  c1g_lane_offsets<MAP>(a, bt, lane);
  const float* pa = d1 + a;
  const float* pb0 = img + bt[0];
  const float* pb1 = ones && (lane & 15) >= 14 ? ones + 2 * (lane >> 4) : img + bt[1];
  float oa[3], ob0[3], ob1[3];
  auto load_step = [&](int kk, int slot) {
    oa[slot] = pa[c1g_imm_a(kk)];
    ob0[slot] = pb0[c1g_imm_b(kk)];
    ob1[slot] = pb1[c1g_imm_b(kk)];
  };
  load_step(0, 0);
  if (STEPS > 1) load_step(1, 1);
#pragma unroll
  for (int kk = 0; kk < STEPS; ++kk) {
    if (kk + 2 < STEPS) load_step(kk + 2, (kk + 2) % 3);
    acc[0] = mfma16(oa[kk % 3], ob0[kk % 3], acc[0]);
    acc[1] = mfma16(oa[kk % 3], ob1[kk % 3], acc[1]);
    if (kk + 2 < STEPS) __builtin_amdgcn_sched_group_barrier(0x100, 3, 0);
    __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
  }
}
// The same GEMM restricted to the K steps of NT tiles of the C1 forward tiling (c1f_tile_*): tile T
// covers four pixel rows and one group of four pixel pairs, i.e. four K steps whose operand
// offsets are the tile's origin plus 24 (d1) or 28 (image) floats per row.  d1t[k] / imgt[k] point
// at the origins of tile k.
template <int NT>
__device__ __forceinline__ void c1g_accumulate_tiles(f4 (&acc)[2], const float* const (&d1t)[3],
                                                     const float* const (&imgt)[3]) {
  int a, bt[2];
  c1g_lane_offsets(a, bt, threadIdx.x & 63);
  float oa[3], ob0[3], ob1[3];
  auto load_step = [&](int st, int slot) {
    const int k = st >> 2, row = st & 3;
    oa[slot] = d1t[k][a + 24 * row];
    ob0[slot] = imgt[k][bt[0] + 28 * row];
    ob1[slot] = imgt[k][bt[1] + 28 * row];
  };
  load_step(0, 0);
  load_step(1, 1);
#pragma unroll
  for (int st = 0; st < 4 * NT; ++st) {
    if (st + 2 < 4 * NT) load_step(st + 2, (st + 2) % 3);
    acc[0] = mfma16(oa[st % 3], ob0[st % 3], acc[0]);
    acc[1] = mfma16(oa[st % 3], ob1[st % 3], acc[1]);
    if (st + 2 < 4 * NT) __builtin_amdgcn_sched_group_barrier(0x100, 3, 0);
    __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
  }
}
// Parks T: park[i * 32 + c] for the lane's rows i = 4q + r and columns c = 16 nt + lane%16.
__device__ __forceinline__ void c1g_park(const f4 (&acc)[2], float* park) {
  const int l = threadIdx.x & 63, q = l >> 4, n16 = l & 15;
#pragma unroll
  for (int nt = 0; nt < 2; ++nt)
#pragma unroll
    for (int r = 0; r < 4; ++r) park[(4 * q + r) * 32 + 16 * nt + n16] = acc[nt][r];
}
// g_k1 element e = m * 25 + 5 u + v from a parked T.
__device__ __forceinline__ float c1g_combine(const float* park, int e) {
  const int m = e / 25, tap = e - 25 * m, u = tap / 5, v = tap - 5 * u;
  return park[(2 * m) * 32 + 6 * u + v] + park[(2 * m + 1) * 32 + 6 * u + v + 1];
}

// Optional per-image outputs of the forward pass.
struct DumpPtrs {
  float *c1, *s1, *c2, *s2;
};

// The 196 16-byte pieces of one image as four float4 registers per lane (the fourth only in lanes
// 0..3).  Kept as separate values so that they stay in registers.
struct Pixels {
  f4 a, b, c, d;
};
__device__ __forceinline__ Pixels load_pixels(const float* __restrict__ image) {
  const f4* src = reinterpret_cast<const f4*>(image);
  const int l = threadIdx.x & 63;
  Pixels px;
  px.a = src[l];  // consecutive lanes -> consecutive 16 bytes
  px.b = src[l + 64];
  px.c = src[l + 128];
  px.d = src[l < 4 ? l + 192 : l];  // lanes >= 4 re-read a piece they already have (no divergence)
  return px;
}

__device__ __forceinline__ void store_pixels(float* img, const Pixels& px) {
  const int l = threadIdx.x & 63;
  f4* dst = reinterpret_cast<f4*>(img);
  dst[l] = px.a;
  dst[l + 64] = px.b;
  dst[l + 128] = px.c;
  if (l < 4) dst[l + 192] = px.d;
}
}  // namespace cnn
