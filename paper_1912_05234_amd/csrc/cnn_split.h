// The network's two convolutions, forward and (the second) backward, on the bfloat16 matrix instruction, in fp32 accuracy.  A float is cut into
// three bfloat16 pieces, x = h + m + l: eight significant bits each, so nothing of its twenty-four is lost, and the range of a
// bfloat16 is a float's.  A product of two floats is then nine products of pieces, each exact, summed in fp32: h h, h m,
// m h, m m, h l, l h, and of 2^-25 of the whole m l, l m (l l is 2^-34).  Why: a
// v_mfma_f32_16x16x32_bf16 takes 7.6 ns of a SIMD for 8192 multiply-adds, a v_mfma_f32_16x16x4_f32 14.6 ns for 1024, so
// six of the former replace eight of the latter in 46 instead of 117 ns, and they run beside the vector instructions of the
// SIMD's other waves, which the fp32 ones do not.
// Error against sums in 64 bits.  Left out are m l and l m, where their slots are not free, and l l: at most 2^-24 of a product.
// The instruction adds sixteen products at a time, cut at 2^-24 of the largest of them and of the sum they are added to,
// which is rounded each time.  Uniform operands: 0.7 (160 products) to 0.35 (32) times the error of the fp32 instructions.
// A single product is up to one last bit off (rms 1.3 times that of fp32), sums of four are as exact: fit for this network,
// whose sums are 25 products and a bias, 150, 12 times up to 25, and 64 per image, not for calls on operands of any kind.
//
// Layouts (64 lanes, q = lane / 16, n16 = lane % 16): A[i = n16][k = 8 q ..  8 q + 7], B[k = 8 q .. 8 q + 7][j = n16],
// D[i = 4 q + r][j = n16] in register r.  An "item" is what a lane supplies to one instruction: eight bfloat16, 16 bytes.
#pragma once

#include <type_traits>

#include "cnn_wave.h"

namespace cnn {

typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef unsigned u4v __attribute__((ext_vector_type(4)));
typedef unsigned u2v __attribute__((ext_vector_type(2)));

__device__ __forceinline__ f4 mfma_bf16(bf8 a, bf8 b, f4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }

// The pieces of x (low half of each word) and y (high half), each rounded to nearest, so that m is at most 2^-8 and l 2^-17 of
// x's power of two and both have either sign.  (With h cut off, m and l are twice as large and m has x's sign: one product was
// off by up to 2^-22, the C1 weight gradient of 40000 images by 5.8e-8 where this gives 4.5e-8 and fp32 instructions 4.6e-8.)
// Below 2^-109 (1.5e-33) the last bits of l leave bfloat16's range: an operand is then kept to 2^-134 in place of 24 bits.
struct Split2 {
  unsigned h, m, l;
};
__device__ __forceinline__ unsigned pack_bf16(float x, float y) {
  using f2v = float __attribute__((ext_vector_type(2)));
  using bf2v = __bf16 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(unsigned, __builtin_convertvector(f2v{x, y}, bf2v));
}
__device__ __forceinline__ Split2 split2_rest(float x, float y, unsigned h) {
  Split2 s;
  s.h = h;
  const float rx = x - __uint_as_float(h << 16), ry = y - __uint_as_float(h & 0xffff0000u);
  s.m = pack_bf16(rx, ry);
  s.l = pack_bf16(rx - __uint_as_float(s.m << 16), ry - __uint_as_float(s.m & 0xffff0000u));
  return s;
}
// For values below 2^127.
__device__ __forceinline__ Split2 split2_bounded(float x, float y) { return split2_rest(x, y, pack_bf16(x, y)); }
// For any finite values: h stops at the largest bfloat16, where rounding would make an infinity.
__device__ __forceinline__ Split2 split2(float x, float y) {
  const float top = __uint_as_float(0x7f7f0000u);
  return split2_rest(x, y, pack_bf16(__builtin_amdgcn_fmed3f(x, -top, top), __builtin_amdgcn_fmed3f(y, -top, top)));
}

// ---- operand items in LDS, shared by the waves of a workgroup -----------------------------------------------------
// C1: item (piece, u, m, sh) holds kernel row u of map m shifted by sh: slot v' = k1[m][u][v' - sh], zero elsewhere.
// C2: item (u, piece, q, j) holds slots kk = 8 q .. 8 q + 7 of kernel row u of map j, kk = 6 v + c, two zeros at the end.
// Both carry -log2(e), like the float operands (logistic_of_scaled); C2's also the 1/4 of the average pooling below it (S1 is
// kept as the sums of four).  A kernel cuts the flat weights itself when it starts: ready-made items, kept in step by the
// update kernel like the float operands, cost every training step 0.28 us.
constexpr int SPLIT_C1_ITEMS = 3 * 5 * 6 * 4, SPLIT_C2_ITEMS = 5 * 3 * 4 * 12;
constexpr int SPLIT_ITEMS = SPLIT_C1_ITEMS + SPLIT_C2_ITEMS;
__host__ __device__ constexpr int split_c1_item(int piece, int u, int m, int sh) { return ((piece * 5 + u) * 6 + m) * 4 + sh; }
__host__ __device__ constexpr int split_c2_item(int u, int piece, int q, int j) { return SPLIT_C1_ITEMS + ((u * 3 + piece) * 4 + q) * 12 + j; }
// Input error of C2 (training): T[row][pixel] = sum_j W[row][j] * d_c2[j][pixel] over twelve maps, rows as in cnn_wave.h (tiles
// V(0..4), U4 of the maps 0..3, then the packed PV(0..2), PU), W = k2[j] / 4.  Twelve K elements would leave most of a step
// of 32 empty, so eight products (all but l l) lie side by side: 96 slots, three steps of 32.  A row is a
// record [h 12][m 12][l 12][4 unused], and so is a pixel of d_c2; slot group g < 24 (four slots) is part g % 3 of product g / 3.
constexpr int BWD_TILES = 10, BWD_REC = 40, BWD_PV = 6, BWD_PU = 9;
__host__ __device__ constexpr int bwd_row(int c, int u, int v) {  // row of tap (c, u, v), 16 to a tile
  if (c < 4) return u < 4 ? 16 * v + 4 * c + u : v < 4 ? 16 * 5 + 4 * c + v : 16 * BWD_PU + 4 * c + 3;
  const int e = 4 * (c - 4) + (v < 3 ? 0 : 8), s = v < 3 ? v : v - 3;
  return u < 4 ? 16 * (BWD_PV + s) + e + u : 16 * BWD_PU + e + s;
}
// Every other row holds the negative of its weights, and its terms are subtracted: the instruction cuts what it aligns towards
// minus infinity (the mean of T comes out 7e-9 of its mean magnitude too low, a tenth of its rms error), which the sums of
// the C1 gradients over all pixels and images, where most of T cancels, would show (8e-7 instead of 5e-8 at 700 images).
__host__ __device__ constexpr bool bwd_negative(int c, int u, int v) { return (u + (c < 4 || v < 3 ? v : v - 3)) & 1; }
// The tap of a row; false: none (the upper eight rows of PV(2), two of PU), its record is zero.
__host__ __device__ constexpr bool bwd_tap_of_row(int row, int& c, int& u, int& v) {
  const int tile = row >> 4, r = row & 15, e = r >> 2, s = r & 3;
  const int packed = tile - BWD_PV;  // PV(packed) or, at three, PU
  if (tile < 5) c = e, u = s, v = tile;
  else if (tile == 5) c = e, u = 4, v = s;
  else if (packed == 3 && s == 3) c = e, u = 4, v = 4;
  else c = 4 + (e & 1), u = packed == 3 ? 4 : s, v = (packed == 3 ? s : packed) + (e >= 2 ? 3 : 0);
  return v < 5;
}
constexpr bool bwd_rows_ok() {
  int rows = 0;
  for (int row = 0; row < 16 * BWD_TILES; ++row) {
    int c = 0, u = 0, v = 0;
    if (!bwd_tap_of_row(row, c, u, v)) continue;
    if (bwd_row(c, u, v) != row) return false;
    ++rows;
  }
  return rows == 150;
}
static_assert(bwd_rows_ok(), "the inverse of bwd_row");
__host__ __device__ constexpr int bwd_group(int g, bool a) {  // offset of slot group g in a record, in fours
  constexpr int PA[8] = {2, 1, 2, 0, 1, 1, 0, 0}, PB[8] = {1, 2, 0, 2, 1, 0, 1, 0};
  return 3 * (a ? PA[g / 3] : PB[g / 3]) + g % 3;
}
// The group that quarter q supplies as half i of the items (steps of two halves, the small products first): quarters 0 and 1,
// and 2 and 3, differ by an odd number in both offsets, so that the sixteen records of both (an odd multiple of four
// words apart) lie on different banks.  (All but the last pair, which is left over.)
constexpr int BWD_GROUPS[6][4] = {{0, 1, 2, 3}, {4, 5, 6, 7}, {8, 12, 9, 10}, {11, 14, 15, 16}, {17, 18, 19, 20}, {13, 22, 21, 23}};
constexpr bool bwd_groups_ok() {
  int seen = 0;
  for (int i = 0; i < 6; ++i)
    for (int q = 0; q < 4; ++q) {
      seen |= 1 << BWD_GROUPS[i][q];
      for (int a = 0; a < 2; ++a)
        if (q % 2 == 0 && 4 * i + q < 22 && (bwd_group(BWD_GROUPS[i][q], a) + bwd_group(BWD_GROUPS[i][q + 1], a)) % 2 == 0) return false;
    }
  return seen == (1 << 24) - 1;
}
static_assert(bwd_groups_ok(), "every group once, neighbours on different banks");
__host__ __device__ constexpr unsigned bwd_groups(int q, bool a) {  // four bits each
  unsigned w = 0;
  for (int i = 0; i < 6; ++i) w |= (unsigned)bwd_group(BWD_GROUPS[i][q], a) << (4 * i);
  return w;
}
// A thread makes whole items, or a whole record, from the weights staged in LDS, and writes them in pieces of 16 bytes.  (A
// thread per weight, writing its pieces slot by slot: 3600 clocks of conflicting 2-byte stores and divisions, half of
// what a workgroup did before its first image.  Gradient of 1000 images 24.8 -> 24.2 us, evaluation of 1100 13.6 -> 13.1 us.)
constexpr int C2_TASKS = 5 * 4 * 12, BWD_TASKS = 16 * BWD_TILES, C1_TASKS = 5 * 6 * 2;
// C2: kernel row u, quarter q of map j (k2 staged as it is): elements kk = 8 q + i = 6 v + c, zeros at 30 and 31.
__device__ __forceinline__ void make_c2_items(u4v* items, int task, const float* k2, float scale) {
  const int u = task % 5, q = (task / 5) & 3, j = task / 20, c0 = q == 3 ? 0 : 2 * q, v0 = q == 3 ? 4 : q;
  const float* k = k2 + 150 * j + 5 * u + 25 * c0 + v0;
  u4v p[3];
#pragma unroll
  for (int h = 0; h < 4; ++h) {
    float x[2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
      x[i] = h == 3 && q == 3 ? 0.0f : scale * k[h == 3 && q == 3 ? 0 : 25 * (2 * h + i) + (c0 + 2 * h + i >= 6 ? 1 - 150 : 0)];
    const Split2 s = split2(x[0], x[1]);
    p[0][h] = s.h, p[1][h] = s.m, p[2][h] = s.l;
  }
#pragma unroll
  for (int i = 0; i < 3; ++i) items[split_c2_item(u, i, q, j)] = p[i];
}
// The record of a row of the input error.
__device__ __forceinline__ void make_bwd_record(unsigned short* bwd, int row, const float* k2, float scale) {
  int c, u, v;
  const bool tap = bwd_tap_of_row(row, c, u, v);
  const float* k = k2 + (tap ? 25 * c + 5 * u + v : 0);
  const bool negative = bwd_negative(c, u, v);
  unsigned p[20];
#pragma unroll
  for (int i = 0; i < 6; ++i) {
    const float x = scale * k[300 * i], y = scale * k[300 * i + 150];
    const Split2 s = split2(!tap ? 0.0f : negative ? -x : x, !tap ? 0.0f : negative ? -y : y);
    p[i] = s.h, p[6 + i] = s.m, p[12 + i] = s.l;
  }
  p[18] = p[19] = 0;
  u4v* to = reinterpret_cast<u4v*>(bwd + BWD_REC * row);
#pragma unroll
  for (int i = 0; i < 5; ++i) to[i] = u4v{p[4 * i], p[4 * i + 1], p[4 * i + 2], p[4 * i + 3]};
}
// C1: shifts sh and sh + 2, sh < 2, of row u of map m.
__device__ __forceinline__ void make_c1_items(u4v* items, int task, const float* k1) {
  const int sh = task & 1, row = task >> 1, u = row % 5, m = row / 5;
  float x[5];
#pragma unroll
  for (int i = 0; i < 5; ++i) x[i] = NEG_LOG2E * k1[5 * row + i];
  const Split2 a = split2(sh ? 0.0f : x[0], sh ? x[0] : x[1]), b = split2(sh ? x[1] : x[2], sh ? x[2] : x[3]),
               c = split2(sh ? x[3] : x[4], sh ? x[4] : 0.0f);
  const unsigned p[3][3] = {{a.h, b.h, c.h}, {a.m, b.m, c.m}, {a.l, b.l, c.l}};
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    items[split_c1_item(i, u, m, sh)] = u4v{p[i][0], p[i][1], p[i][2], 0};
    items[split_c1_item(i, u, m, sh + 2)] = u4v{0, p[i][0], p[i][1], p[i][2]};
  }
}
// COUNT floats from global memory, all in flight, then in LDS.
template <int THREADS, int COUNT>
struct StagedLoad {
  float v[(COUNT + THREADS - 1) / THREADS];
  __device__ __forceinline__ void fetch(const float* __restrict__ w) {
#pragma unroll
    for (int r = 0; r * THREADS < COUNT; ++r) {
      const int p = threadIdx.x + THREADS * r;
      v[r] = w[p < COUNT ? p : 0];
    }
  }
  __device__ __forceinline__ void commit(float* stage) const {
#pragma unroll
    for (int r = 0; r * THREADS < COUNT; ++r)
      if ((int)threadIdx.x + THREADS * r < COUNT) stage[threadIdx.x + THREADS * r] = v[r];
  }
};
// All operands from the flat weights.  BWD: the records of the input error too.
template <int THREADS, bool BWD>
struct SplitLoad : StagedLoad<THREADS, OFF_B2> {
  static constexpr int ROW_THREAD = 256, C1_THREAD = 448;  // one task per thread, kinds on whole waves where it fits
  static_assert(C2_TASKS <= ROW_THREAD && ROW_THREAD + BWD_TASKS <= C1_THREAD && C1_THREAD + C1_TASKS <= THREADS, "one task per thread");
  // `stage`: OFF_B2 words of LDS that nobody uses until the caller's barrier.
  __device__ __forceinline__ void commit(float* stage, u4v* items, unsigned short* bwd = nullptr) const {
    StagedLoad<THREADS, OFF_B2>::commit(stage);
    __syncthreads();
    const int t = threadIdx.x;
    if (t < C2_TASKS) make_c2_items(items, t, stage + OFF_K2, 0.25f * NEG_LOG2E);
    if (BWD && t >= ROW_THREAD && t < ROW_THREAD + BWD_TASKS) make_bwd_record(bwd, t - ROW_THREAD, stage + OFF_K2, 0.25f);
    if (t >= C1_THREAD && t < C1_THREAD + C1_TASKS) make_c1_items(items, t - C1_THREAD, stage + OFF_K1);
  }
};

// ---- the image in LDS: three planes of pieces, [28][28] each ---------------------------------------------------
constexpr int SPLIT_IMG_PLANE = NI / 2;  // words
__device__ __forceinline__ void split_store_pixels(unsigned* img, int at, f4 v) {  // four pixels from pixel 4 at on
  const Split2 a = split2(v[0], v[1]), b = split2(v[2], v[3]);
  reinterpret_cast<u2v*>(img)[at] = u2v{a.h, b.h};
  reinterpret_cast<u2v*>(img + SPLIT_IMG_PLANE)[at] = u2v{a.m, b.m};
  reinterpret_cast<u2v*>(img + 2 * SPLIT_IMG_PLANE)[at] = u2v{a.l, b.l};
}

// ---- C1 forward ---------------------------------------------------------------------------------------------------
// Output pixels are taken four at a time, x = 4 X + sh.  With v' = v + sh < 8 the image factor img[y+u][4X+v'] does not
// depend on sh, and its eight values are one item of the image:
//   pre[(sh,m)][(y,X)] = sum_{u < 5, v' < 8} W[(sh,m)][(u,v')] * img[y+u][4X+v'],  W = k1[m][u][v'-sh].
// Rows i = 4 sh + m % 4, so that lane (q, n16) of the result holds the maps of ONE pixel, x = 4 X + q: tile 0 the maps 0..3,
// tile 1 the maps 4, 5 (its other rows repeat them and are not used).  Columns: nine tiles T = 3 ty + tx of sixteen (y, X),
// y = 8 ty + 2 a + dy, X = 2 tx + bx, n16 = dy + 2 a + 8 bx.  K: an instruction takes four (u, product) pairs, one per lane
// quarter: quarter q takes row u = q in six instructions, one per product, and row u = 4's products (with m l and l m,
// whose quarters are free) are two instructions more: 16 instructions per column tile, 144 per image.
struct C1SWeights {
  bf8 row[2][3];    // pieces of row u = q
  bf8 mixed[2][2];  // row u = 4, piece by quarter
};
__device__ __forceinline__ void c1s_load_weights(C1SWeights& w, const u4v* items, int l) {
  const int q = l >> 4, n16 = l & 15, sh = n16 >> 2;
#pragma unroll
  for (int mt = 0; mt < 2; ++mt) {
    const int m = mt == 0 ? n16 & 3 : 4 + (n16 & 1);
#pragma unroll
    for (int k = 0; k < 3; ++k) w.row[mt][k] = __builtin_bit_cast(bf8, items[split_c1_item(k, q, m, sh)]);
    // image pieces l, h, m, m | h, h, l, m (c1s_lane) meet weight pieces h, l, m, h | m, h, m, l
    w.mixed[mt][0] = __builtin_bit_cast(bf8, items[split_c1_item(q == 1 ? 2 : q == 2 ? 1 : 0, 4, m, sh)]);
    w.mixed[mt][1] = __builtin_bit_cast(bf8, items[split_c1_item(q == 1 ? 0 : q == 3 ? 2 : 1, 4, m, sh)]);
  }
}
struct C1SLane {
  const unsigned *row, *mixed0, *mixed1;  // the lane's items of column tile 0
};
__device__ __forceinline__ C1SLane c1s_lane(const unsigned* img, int l) {
  const int q = l >> 4, n16 = l & 15, y = n16 & 7, bx = n16 >> 3;  // y = 2 a + dy
  const unsigned* at = img + 14 * y + 2 * bx;
  C1SLane o;
  o.row = at + 14 * q;
  o.mixed0 = at + 14 * 4 + SPLIT_IMG_PLANE * (q == 0 ? 2 : q == 1 ? 0 : 1);
  o.mixed1 = at + 14 * 4 + SPLIT_IMG_PLANE * (q < 2 ? 0 : q == 2 ? 2 : 1);
  return o;
}
__host__ __device__ constexpr int c1s_tile_img(int T) { return (T / 3) * 112 + (T % 3) * 4; }  // words
// Sixteen bytes from an 8-byte aligned LDS address, as two loads that must not become one ds_read2_b64: that takes the LDS 16
// cycles where two ds_read_b64 take 2 each.  (The compiler keeps such loads in the order they are written: what is to
// be read ahead is written ahead.)
__device__ __forceinline__ bf8 item8(const unsigned* p) {
  typedef const volatile u2v __attribute__((address_space(3)))* LdsPair;
  const u2v a = *(LdsPair)p, b = *(LdsPair)(p + 2);
  return __builtin_bit_cast(bf8, u4v{a.x, a.y, b.x, b.y});
}

struct C1SItems {
  bf8 row[3], mixed[2];
};
__device__ __forceinline__ void c1s_load(C1SItems& it, const C1SLane& ln, int T) {
  const int o = c1s_tile_img(T);
#pragma unroll
  for (int k = 0; k < 3; ++k) it.row[k] = item8(ln.row + o + k * SPLIT_IMG_PLANE);
  it.mixed[0] = item8(ln.mixed0 + o);
  it.mixed[1] = item8(ln.mixed1 + o);
}
// Both row tiles of one column tile, the small products first; d0, d1 enter with the biases.
__device__ __forceinline__ void c1s_gemm(const C1SWeights& w, const C1SItems& it, f4& d0, f4& d1) {
  constexpr int PX[6] = {2, 0, 1, 1, 0, 0}, PW[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    d0 = mfma_bf16(w.mixed[0][k], it.mixed[k], d0);
    d1 = mfma_bf16(w.mixed[1][k], it.mixed[k], d1);
  }
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    d0 = mfma_bf16(w.row[0][PW[k]], it.row[PX[k]], d0);
    d1 = mfma_bf16(w.row[1][PW[k]], it.row[PX[k]], d1);
  }
}

// ---- S1 in LDS: three planes of pieces, channels last, [12][12][6] each ------------------------------------------
// Twice: a pixel is twelve bytes, and in the second copy, SPLIT_S1B words further, the odd pixels are eight-byte aligned.
// Its place puts the four pixels of a transposing read (two rows of 36 words, odd pixels in the second copy) on different
// banks: ranges of 14 words for two quarters at 0, 36 and 14 further.
constexpr int SPLIT_S1_PLANE = NS1 / 2;                       // words
constexpr int SPLIT_S1_COPY = 3 * SPLIT_S1_PLANE + 4;         // the last items reach 4 bytes past the planes (zero weights)
constexpr int SPLIT_S1B = SPLIT_S1_COPY + 55;
constexpr int SPLIT_S1_WORDS = SPLIT_S1B + SPLIT_S1_COPY + 1;
static_assert(SPLIT_S1B % 2 == 1 && (SPLIT_S1B + 3) % 64 == 14 && SPLIT_S1_WORDS % 4 == 0, "alignment and banks");
// Lanes xor 16 of two registers at once: returns a's (even quarters) and b's (odd quarters) sum over the lane pair.
__device__ __forceinline__ float pair16_sum(float a, float b) {
  const u2v r = __builtin_bit_cast(u2v, __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false));
  return __uint_as_float(r.x) + __uint_as_float(r.y);
}
// Average pooling of one column tile: a window is the lanes (q, q ^ 1) x (n16, n16 ^ 1).  Sums of the maps 0..3, one per
// lane: map (q & 1) + 2 (n16 & 1); and of the maps 4, 5 over q alone: map 4 + (q & 1).
__device__ __forceinline__ void c1s_pool(const float (&c)[6], float& low, float& high) {
  const bool dy = threadIdx.x & 1;
  const float s01 = pair16_sum(c[0], c[1]), s23 = pair16_sum(c[2], c[3]);
  low = (dy ? s23 : s01) + quad_xor1(dy ? s01 : s23);
  high = pair16_sum(c[4], c[5]);
}
__device__ __forceinline__ float c1s_pool_rows(float ha, float hb) {  // lanes n16 even: tile a, odd: tile b
  const bool dy = threadIdx.x & 1;
  return (dy ? hb : ha) + quad_xor1(dy ? ha : hb);
}
__host__ __device__ constexpr int c1s_tile_s1(int T) { return ((T / 3) * 48 + (T % 3) * 4) * 6; }  // elements
// The lane's element of S1 for the sum `low` of tile 0 (`high`: element + 4 - 2 (n16 & 1)).
__device__ __forceinline__ int c1s_lane_s1(int l) {
  const int q = l >> 4, n16 = l & 15, a = (n16 >> 1) & 3, bx = n16 >> 3;
  return (a * 12 + 2 * bx + (q >> 1)) * 6 + (q & 1) + 2 * (n16 & 1);
}
// Pieces of two values to two elements; BOTH: of both copies.
template <bool BOTH>
__device__ __forceinline__ void split_store_s1(unsigned short* s1, int e0, float v0, int e1, float v1) {
  const Split2 s = split2_bounded(v0, v1);
  const unsigned p[3] = {s.h, s.m, s.l};
#pragma unroll
  for (int k = 0; k < 3; ++k) {
#pragma unroll
    for (int copy = 0; copy < (BOTH ? 2 : 1); ++copy) {
      s1[e0 + k * NS1 + copy * 2 * SPLIT_S1B] = (unsigned short)p[k];
      s1[e1 + k * NS1 + copy * 2 * SPLIT_S1B] = (unsigned short)(p[k] >> 16);
    }
  }
}

// The same for one value.
template <bool BOTH>
__device__ __forceinline__ void split_store_s1_one(unsigned short* s1, int e, float v) {
  const Split2 s = split2_bounded(v, 0.0f);
  const unsigned p[3] = {s.h, s.m, s.l};
#pragma unroll
  for (int k = 0; k < 3; ++k)
#pragma unroll
    for (int copy = 0; copy < (BOTH ? 2 : 1); ++copy) s1[e + k * NS1 + copy * 2 * SPLIT_S1B] = (unsigned short)p[k];
}
// S1 itself at index e of [6][12][12]: a quarter of the sum of its pieces, which is exactly the value that was cut.
__device__ __forceinline__ float split_s1_value(const unsigned short* s1, int e) {
  const int c = e / 144, at = 6 * (e - 144 * c) + c;
  float p[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) p[k] = __uint_as_float((unsigned)s1[at + k * NS1] << 16);
  return 0.25f * (p[0] + (p[1] + p[2]));
}

// ---- C2 forward ---------------------------------------------------------------------------------------------------
// M = 64 pixels in four tiles (cnn_wave.h: a result lane's registers are one pooling window), N = 12(16) maps, K = one
// kernel row u at a time: the patch row s1[y+u][x .. x+4][0..5] is thirty neighbouring elements, with two more (the next
// pixel's, zero weights) one K step of 32.  Five steps of six products, 120 instructions.
// Tile mt's row u is row u + 2 mt of the image plane: eleven rows of items, each read once.
struct C2SLane {
  const unsigned* s1;  // the lane's item of row 0
  const u4v* w;
};
__device__ __forceinline__ C2SLane c2s_lane(const unsigned* s1, const u4v* items, int l) {
  const int q = l >> 4, n16 = l & 15;
  const int pp = 12 * ((n16 & 3) >> 1) + 2 * (n16 >> 2) + (n16 & 1);
  return C2SLane{s1 + ((n16 & 1) ? SPLIT_S1B : 0) + 3 * pp + 4 * q, items + split_c2_item(0, 0, q, n16 < 12 ? n16 : n16 - 12)};
}
// One piece of the image after the other (l, m, h), so that seven rows of items are in registers and not all of them; a step's
// new row, and the next piece's first rows, are read a step ahead.
// The pixel tiles M0 .. M0 + N - 1.
template <int M0, int N>
__device__ __forceinline__ void c2s_gemm(f4 (&d)[N], const C2SLane& ln) {
  constexpr int ROWS = 2 * N + 3;  // rows 2 M0 .. of S1
  bf8 x[2][ROWS];
  auto load_row = [&](int k, int row) {
    if (row < ROWS) x[k & 1][row] = item8(ln.s1 + 36 * (2 * M0 + row) + k * SPLIT_S1_PLANE);
  };
#pragma unroll
  for (int row = 0; row < 2 * N - 1; ++row) load_row(2, row);
#pragma unroll
  for (int k = 2; k >= 0; --k)  // piece l meets h; m meets m, h; h meets l, m, h
#pragma unroll
    for (int u = 0; u < 5; ++u) {
      if (u < 4) load_row(k, u + 2 * N - 1);
      if (k > 0 && u >= 1) {
        // (what the first kernel row of the next piece needs; its other rows follow under its products)
        load_row(k - 1, 2 * u - 2 < 2 * N - 1 ? 2 * u - 2 : ROWS);
        if (u < 4) load_row(k - 1, 2 * u - 1 < 2 * N - 1 ? 2 * u - 1 : ROWS);
      }
#pragma unroll
      for (int j = 2 - k; j >= 0; --j) {
        const bf8 b = __builtin_bit_cast(bf8, ln.w[(u * 3 + j) * 48]);
#pragma unroll
        for (int mt = 0; mt < N; ++mt) d[mt] = mfma_bf16(x[k & 1][u + 2 * mt], b, d[mt]);
      }
    }
}

// ---- C2 weight gradient --------------------------------------------------------------------------------------------
// C2 backweights: G[j, (c,u,v)] += sum_p d_c2[j, p] * s1[c, y(p)+u, x(p)+v].  K is the pixels: a step takes the windows 4 q + r
// of the tiles 2 S and 2 S + 1, slots in the order of the result registers of d_c2, which so are the A operand as they
// stand.  The columns of kernel row u are the thirty elements s1[y+u][x .. x+4][0..5], two tiles; a transposing
// read brings four pixels (rows, twelve bytes apart) of sixteen columns: lane 4 r + i of a quarter gives the address of
// pixel r's columns 4 i .. 4 i + 3 and receives column n16 of all four.
// Over the pixel tiles 2 S and 2 S + 1, S0 <= S < S0 + NS.
template <int S0, int NS>
__device__ __forceinline__ void k2_gradient(f4 (&acc)[10], const u4v (&d2)[2][3], const unsigned* s1, int l) {
  typedef __bf16 bf4 __attribute__((ext_vector_type(4)));
  typedef bf4 __attribute__((address_space(3)))* LdsQuad;
  const int q = l >> 4, n16 = l & 15, r = n16 >> 2, dx = r & 1;
  LdsQuad at = (LdsQuad)(reinterpret_cast<const unsigned short*>(s1 + (dx ? SPLIT_S1B : 0)) + 6 * (12 * (r >> 1) + 2 * q + dx) + 4 * (n16 & 3));
  bf8 a[2][3];
#pragma unroll
  for (int S = S0; S < S0 + NS; ++S)
#pragma unroll
    for (int k = 0; k < 3; ++k) a[S][k] = __builtin_bit_cast(bf8, d2[S][k]);
  // Rows R = u + 4 S and R + 2 of the image plane make an operand.  Every one is read afresh (two operands may share a row, but
  // not in the same half of their registers), the next one's under an operand's products.  The image's sums are made on
  // their own and then added: steps onto the sums over all images would be rounded, and cut, at their size.
  bf8 x[2][2][3];
  auto load = [&](int n) {
    const int R = n / NS + 4 * (S0 + n % NS);
    LdsQuad from = at;
    asm volatile("" : "+v"(from));
#pragma unroll
    for (int k = 2; k >= 0; --k)
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const u2v lo = __builtin_bit_cast(u2v, __builtin_amdgcn_ds_read_tr16_b64_v4bf16(from + (R * 72 + 16 * t + k * NS1) / 4));
        const u2v hi = __builtin_bit_cast(u2v, __builtin_amdgcn_ds_read_tr16_b64_v4bf16(from + ((R + 2) * 72 + 16 * t + k * NS1) / 4));
        x[n & 1][t][k] = __builtin_bit_cast(bf8, u4v{lo.x, lo.y, hi.x, hi.y});
      }
  };
  constexpr int PX[6] = {2, 0, 1, 1, 0, 0}, PA[6] = {0, 2, 1, 0, 1, 0};
  load(0);
  f4 sum[2];
#pragma unroll
  for (int n = 0; n < 5 * NS; ++n) {  // u = n / NS, S = S0 + n % NS
    if (n < 5 * NS - 1) load(n + 1);
    if (n % NS == 0) sum[0] = sum[1] = f4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int k = 0; k < 6; ++k)
#pragma unroll
      for (int t = 0; t < 2; ++t) sum[t] = mfma_bf16(a[S0 + n % NS][PA[k]], x[n & 1][t][PX[k]], sum[t]);
    if (n % NS == NS - 1)
#pragma unroll
      for (int t = 0; t < 2; ++t) {
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[2 * (n / NS) + t][r] += sum[t][r];
        asm volatile("" : "+v"(acc[2 * (n / NS) + t]));  // now: the compiler would keep the sums and the old `acc` until the end of the image
      }
  }
}

// ---- C2 input error -------------------------------------------------------------------------------------------------
// d_in [6][12][16 of which 12], eight words more between maps: the lanes of two quarters (two maps, two rows of eight
// neighbours in each) then lie on 32 different banks.
constexpr int DS1_ROW = 16, DS1_MAP = 12 * DS1_ROW + 8;
// Records of an image's d from its pieces d2[S][piece] (result layout: register r of tile 2 S + mt % 2 is pixel
// (2 mt + r / 2, 2 q + r % 2)).  Record 16 mt + 2 x + y % 2 is pixel (y, x): the two rows of a tile alternate, see col2im_split.
template <int S0, int NS>
__device__ __forceinline__ void store_records(unsigned short* recs, const u4v (&d2)[2][3], int l) {
  const int q = l >> 4, n16 = l & 15;
  unsigned short* rec = recs + 4 * q * BWD_REC + n16;
  if (n16 < 12) {
#pragma unroll
    for (int mt = 2 * S0; mt < 2 * (S0 + NS); ++mt)
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          const unsigned p = d2[mt >> 1][k][2 * (mt & 1) + h];
          rec[(16 * mt + h) * BWD_REC + 12 * k] = (unsigned short)p;
          rec[(16 * mt + 2 + h) * BWD_REC + 12 * k] = (unsigned short)(p >> 16);
        }
  }
}
template <int CTRL>  // row_shl:n 0x100 + n, row_shr:n 0x110 + n: lanes that nothing reaches get 0
__device__ __forceinline__ float dpp(float v) {
  return __uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(v), CTRL, 15, 15, true));
}
template <int CTRL, int ROWS>  // only the quarters ROWS, the others keep old
__device__ __forceinline__ float dpp(float old, float v) {
  return __uint_as_float(__builtin_amdgcn_update_dpp(__float_as_uint(old), __float_as_uint(v), CTRL, ROWS, 15, true));
}
// A sum over tap columns v of values shifted right by v: columns 0..7 of two rows in a quarter's sixteen lanes (lane 2 x + row),
// columns 8..11 in the first lanes of a second register.
template <int V>
__device__ __forceinline__ void add_column(float& lo, float& hi, float e) {
  if constexpr (V == 0) {
    lo = e;
    hi = 0.0f;
  } else {
    const float a = dpp<0x110 + 2 * V>(e), b = dpp<0x100 + 16 - 2 * V>(e);
    lo = V & 1 ? lo - a : lo + a;  // (bwd_negative)
    hi = V & 1 ? hi - b : hi + b;
  }
}
// C2 backin summed over the twelve maps, col2im form:
//      T[(c,u,v), p] = sum_j k2[j,c,u,v] * d[j,p];   d_in[c, y(p)+u, x(p)+v] += T[(c,u,v), p].
// All in registers: with level = 2 nt + u (nt = pixel tile = row pair of p), terms of equal level and v are the same cells of
// the same lanes, and an odd level shares its rows half and half with the two even ones beside it.  What is added over levels
// is shifted by v within the quarter (one map) and added over v.  With the sums in
// LDS, in sixteen dependent rounds of reads, additions and writes (its clearing, a second copy of the maps 4 and 5), an image
// kept the LDS busy for 1000 clocks, eight waves 8000 of 13000; training on 60000 images took 588 us instead of 572.
// The input maps 0..3 and 4, 5 are taken one after the other: half the registers.
// d_in may lie over the records; its columns 12..15 get zeros.  `sign`: what d was taken with.
// LOW, HIGH: with the input maps 0..3, with 4 and 5.
template <bool LOW, bool HIGH>
__device__ __forceinline__ void col2im_split(const unsigned short* bwd, const unsigned short* rec, float* d_in, float sign, int l) {
  const int q = l >> 4, n16 = l & 15;
  // this quarter's slot groups of a row record and of a pixel record
  const unsigned ga = q == 0 ? bwd_groups(0, true) : q == 1 ? bwd_groups(1, true) : q == 2 ? bwd_groups(2, true) : bwd_groups(3, true);
  const unsigned gb = q == 0 ? bwd_groups(0, false) : q == 1 ? bwd_groups(1, false) : q == 2 ? bwd_groups(2, false) : bwd_groups(3, false);
  const u2v* arow[6];
  u2v bd[4][6];
#pragma unroll
  for (int i = 0; i < 6; ++i) {
    arow[i] = reinterpret_cast<const u2v*>(bwd + BWD_REC * n16) + ((ga >> (4 * i)) & 15);
    const u2v* b = reinterpret_cast<const u2v*>(rec) + n16 * (BWD_REC / 4) + ((gb >> (4 * i)) & 15);
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
      bd[nt][i] = b[16 * nt * (BWD_REC / 4)];
    }
  }
  wave_sync();
  float lo[6], hi[6];  // rows 2m and 2m + 1
  // The tiles tv of tap column V; `u4` is the u = 4 term per pixel tile.  Level 2m has rows 2m and 2m + 1 in the even and
  // the odd lanes, level 2m + 1, with the other sign (bwd_negative), rows 2m + 1 and 2m + 2.
  auto column = [&](auto vc, const f4 (&tv)[4], const float (&u4)[4]) {
    constexpr int V = decltype(vc)::value;
    __builtin_amdgcn_sched_barrier(0);  // two columns' tiles at a time do not fit the registers of the training kernel
    float odd[5];  // levels 2m + 1: (nt = m, u = 1) + (m-1, 3)
#pragma unroll
    for (int m = 0; m < 5; ++m) {
      odd[m] = 0.0f;
      if (m < 4) odd[m] = tv[m < 4 ? m : 0][1];
      if (m >= 1) odd[m] += tv[m >= 1 ? m - 1 : 0][3];
    }
#pragma unroll
    for (int m = 0; m < 6; ++m) {
      // level 2m: (nt = m, u = 0) + (m-1, 2) + (m-2, 4)
      float e = 0.0f;
      if (m < 4) e = tv[m < 4 ? m : 0][0];
      if (m >= 1 && m <= 4) e += tv[m >= 1 ? m - 1 : 0][2];
      if (m >= 2) e += u4[m >= 2 ? m - 2 : 0];
      const float z = n16 & 1 ? (m > 0 ? odd[m > 0 ? m - 1 : 0] : 0.0f) : (m < 5 ? odd[m < 5 ? m : 0] : 0.0f);
      add_column<V>(lo[m], hi[m], e - dpp<0xb1>(z));  // quad_perm [1, 0, 3, 2]
    }
  };
  // the four pixel tiles of one M tile
  auto tiles = [&](int tile, f4 (&out)[4]) {
    u2v a[6];
#pragma unroll
    for (int i = 0; i < 6; ++i) a[i] = arow[i][16 * tile * (BWD_REC / 4)];
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
      f4 d = f4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int k = 0; k < 3; ++k)
        d = mfma_bf16(__builtin_bit_cast(bf8, u4v{a[2 * k].x, a[2 * k].y, a[2 * k + 1].x, a[2 * k + 1].y}),
                      __builtin_bit_cast(bf8, u4v{bd[nt][2 * k].x, bd[nt][2 * k].y, bd[nt][2 * k + 1].x, bd[nt][2 * k + 1].y}), d);
      out[nt] = d;
    }
  };
  float* cell = d_in + DS1_ROW * (n16 & 1) + (n16 >> 1);  // of row 0 or 1, columns 0..7
  f4 tu[4];
  tiles(BWD_PU, tu);
  // ---- input maps 4, 5, packed: lane quarters 0, 1 have them for tap columns 0..2 and quarters 2, 3 for columns 3, 4, in
  //      round s column s or 3 + s (quarters 2, 3 have nothing in round 2: their tile rows are zero).  tu: the u = 4 term of
  //      round s in register s ----
  if constexpr (HIGH) {
    auto round = [&](auto sc) {
      constexpr int S = decltype(sc)::value;
      f4 tv[4];
      tiles(BWD_PV + S, tv);
      float u4[4];
#pragma unroll
      for (int nt = 0; nt < 4; ++nt) u4[nt] = tu[nt][S];
      column(sc, tv, u4);
    };
    round(std::integral_constant<int, 0>{});
    round(std::integral_constant<int, 1>{});
    round(std::integral_constant<int, 2>{});
    float* to = cell + DS1_MAP * (4 + (q & 1)) + (q < 2 ? 0 : 8);
#pragma unroll
    for (int m = 0; m < 6; ++m) {
      // quarters 2, 3: three columns further
      const float h = dpp<0x116, 12>(hi[m], hi[m]) + dpp<0x10a, 12>(0.0f, lo[m]), a = dpp<0x116, 12>(lo[m], lo[m]);
      // the sums over both halves: columns 0..7 in quarters 0, 1 and columns 8..11 in quarters 2, 3
      const u2v s = __builtin_bit_cast(u2v, __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(h), false, false));
      const float v = sign * (__uint_as_float(s.x) + __uint_as_float(s.y));
      to[2 * DS1_ROW * m] = v;
    }
  }
  // ---- input maps 0..3: lane quarter q owns map q; tiles V(0..4) and U4; tap (4, 4) rides in
  //      register 3 of the packed tile PU of the maps 4, 5 above ----
  if constexpr (LOW) {
    f4 t4[4];  // taps (4, v), v < 4, in register v
    tiles(kTileU4, t4);
    auto round = [&](auto vc) {
      constexpr int V = decltype(vc)::value;
      f4 tv[4];  // taps (u, v), u < 4, in register u
      tiles(kTileV0 + V, tv);
      float u4[4];
#pragma unroll
      for (int nt = 0; nt < 4; ++nt) u4[nt] = V < 4 ? t4[nt][V < 4 ? V : 0] : tu[nt][3];
      column(vc, tv, u4);
    };
    round(std::integral_constant<int, 0>{});
    round(std::integral_constant<int, 1>{});
    round(std::integral_constant<int, 2>{});
    round(std::integral_constant<int, 3>{});
    round(std::integral_constant<int, 4>{});
    float* to = cell + DS1_MAP * q;
#pragma unroll
    for (int m = 0; m < 6; ++m) to[2 * DS1_ROW * m] = sign * lo[m];
#pragma unroll
    for (int m = 0; m < 6; ++m) to[2 * DS1_ROW * m + 8] = sign * hi[m];
  }
}

// ---- S2 and its error in LDS: sixteen to a map, seventeen apart (a store or load of a whole tile has lanes 16 apart) ----
constexpr int S2_MAP = 17;
__device__ __forceinline__ int s2_at(int i) { return i + (i >> 4); }
constexpr int S2_WORDS = 12 * S2_MAP;

// ---- output layer -------------------------------------------------------------------------------------------------
// Sums over the wave of ten values per lane, several at a time: a step of the tree adds two values' lanes in one register.
// Lane l holds the sum of value out_of_lane(l); the lanes 0..3, 16..19, 32 and 33 hold the ten in order.
__device__ __forceinline__ float pair32_sum(float a, float b) {  // lanes below 32: a's sum over the lane pair, others: b's
  const u2v r = __builtin_bit_cast(u2v, __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false));
  return __uint_as_float(r.x) + __uint_as_float(r.y);
}
template <int CTRL>
__device__ __forceinline__ float dpp_add(float v) {
  return v + __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}
__device__ __forceinline__ int out_of_lane(int l) { return l < 32 ? 4 * (l >> 4) + (l & 3) : 8 + (l & 1); }
constexpr unsigned long long OUT_LANES = 0x3000F000Full;
__device__ __forceinline__ float wave_sum10(const float (&p)[NY]) {
  const bool odd = threadIdx.x & 1, hi = threadIdx.x & 2;
  float a[5];
#pragma unroll
  for (int k = 0; k < 5; ++k) a[k] = (odd ? p[2 * k + 1] : p[2 * k]) + quad_xor1(odd ? p[2 * k] : p[2 * k + 1]);
  float b[3];
#pragma unroll
  for (int k = 0; k < 2; ++k) b[k] = (hi ? a[2 * k + 1] : a[2 * k]) + quad_xor2(hi ? a[2 * k] : a[2 * k + 1]);
  b[2] = a[4] + quad_xor2(a[4]);
#pragma unroll
  for (int k = 0; k < 3; ++k) b[k] = dpp_add<0x128>(dpp_add<0x124>(b[k]));  // the four quads of a row: rotations by 4 and 8
  return pair32_sum(pair16_sum(b[0], b[1]), pair16_sum(b[2], b[2]));
}

}  // namespace cnn
