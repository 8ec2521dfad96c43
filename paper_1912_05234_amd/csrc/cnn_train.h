// The training step of more than 512 images: ONE WAVEFRONT (64 lanes) OWNS ONE IMAGE from the pixel load to the last
// gradient term, eight waves to a workgroup, two to a SIMD; up to 1024 images, of which a SIMD has one, its two waves share it
// (WavePart).  Definitions: arXiv 1912.05234, Section 3 (forward, conv, mconv, sigmoid, avgpool, backweights, backbias, backin,
// backavgpool); the backward pass is the chain rule over those.
//
// Where the arithmetic runs
//   C1, C2 forward        v_mfma_f32_16x16x32_bf16 on the pieces of the operands (cnn_split.h)
//   C2 weight gradient    the same: M = 12(16) maps, N = 30(32) neighbouring elements of S1 per kernel row, K = 64 pixels
//   C2 input error        the same: T[tap,pixel] = k2^T * d_c2 (K = 12 maps, eight products side by side), then T is
//                         summed over the taps in registers (the col2im form of `backin`: no zero padding)
//   C1 weight gradient    v_mfma_f32_16x16x4_f32: M = 12(16) rows (map, x parity), N = 30(32) shifted taps,
//                         K = 288 pixel pairs; the C1 error is staged in LDS by column tiles of C1
//   FC weight gradient    v_mfma_f32_16x16x4_f32, once per wave over all its images (of a shared one: products in registers)
//   FC, pooling, sigmoid  fp32 VALU
// What bounds it, 60000 images in 577 us (830 with fp32 instructions throughout), 21.8 thousand clocks of a SIMD per image:
// 507 bfloat16 and 144 fp32 matrix instructions are 12.8 thousand of them, about 1810 vector instructions of three clocks
// another 5.4 (few of them under a matrix instruction, see cnn_split.h), the rest are waits that the SIMD's other wave does
// not cover; the LDS is busy for half of the time.  The C1 weight gradient stays on the fp32 instruction: as products of
// pieces it needs 180 instructions, 300 vector instructions for the cutting, and gains nothing.
// Waves with images of their own share the operands in LDS and nothing else; after the barrier that completes them they do
// not synchronise until they join their gradient sums at the end of the kernel.  What two waves of a shared image write, and
// which barrier hands it over, stands at WavePart.
#pragma once

#include "cnn_split.h"

namespace cnn {

// ---- LDS ----------------------------------------------------------------------------------------------------------
// Shared by the workgroup: the items of both convolutions and the records of the input error (cnn_split.h), the FC weights
// as [entry][lane], the biases.
struct __align__(16) TrainOperands {
  u4v items[SPLIT_ITEMS];
  unsigned short bwd[BWD_TILES * 16 * BWD_REC];
  float fc[30 * 64];
  float bias[TAB_BIAS_FLOATS];
  float ones[C1G_ONES];  // 1.0: B operand of the padding columns of the C1 weight-gradient GEMM (c1g_accumulate)
};
// Per wave: the image, and 3120 words that the phases use in turn, exactly one partial row together.  (A shared image has those of
// its FIRST wave; in SECOND's own are the parts that each wave makes for itself.)
//   C1 forward          S1's pieces (first copy) at 0, the image's pieces behind them
//   C2 forward, FC      both copies of S1, s2, d_s2
//   C2 gradients        both copies of S1; then d_s1 and the records of d_c2
//   C1 weight gradient  d_s1, and the C1 error of two column tiles
constexpr int W_S1 = 0;
constexpr int W_PIECES = SPLIT_S1_COPY;                // no longer needed when the second copy takes their place
constexpr int W_S2 = SPLIT_S1_WORDS;                   // s2 as S2_MAP says
constexpr int W_DS2 = W_S2 + S2_WORDS;
constexpr int W_DS1 = 0, W_D2 = 6 * DS1_MAP;
constexpr int W_D1 = W_D2;
constexpr int D1T_HALF = 34, D1T_MAP = 2 * D1T_HALF, D1T_WORDS = 6 * D1T_MAP;
constexpr int W_WORDS = PSTRIDE - NI;
static_assert(W_PIECES % 4 == 0 && W_S2 % 4 == 0 && W_D2 % 4 == 0 && W_D1 % 4 == 0, "alignment");
static_assert(W_PIECES + 3 * SPLIT_IMG_PLANE <= W_WORDS && W_DS2 + S2_WORDS <= W_WORDS && W_D1 + 2 * D1T_WORDS <= W_WORDS && W_D2 + 64 * BWD_REC / 2 <= W_WORDS, "the arrays fit");
struct __align__(16) WaveTrainLds {
  float img[NI];
  float pool[W_WORDS];
};
static_assert(sizeof(WaveTrainLds) == sizeof(float) * PSTRIDE, "a wave's LDS area holds one partial row");

// What the FC weight gradient needs of one image, kept in global memory until the wave has done all
// its images: s2 (192 floats), then delta in [192, 202) and zeros up to 208; rows of 256 floats, so
// that no two images share a cache line.  The gradient is then ONE GEMM per wave over its images,
//   g_fc[o][i] = sum_n delta_n[o] * s2_n[i]                                   (backweights, Section 3)
// with M = 10(16) outputs, N = 192 inputs in twelve tiles, K = the wave's images four at a time:
// three matrix instructions per image instead of thirty multiply-adds on sums that no register or LDS
// space is left for.
constexpr int FC_HIST = 256;        // floats per image
constexpr int FC_HIST_DELTA = 192;  // delta[0..9], then six zeros
// Everything a wave keeps in registers across its images.
struct WaveState {
  float bias2;    // b2[n16]
  f4 acc_k2[10];  // sum over images of d_c2 (x) S1 patches (four times the gradient, with the wave's sign): D[j = 4q+r][16 t + n16] of kernel row u in tile 2 u + t
  f4 acc_k1[2];   // C1 weight gradient GEMM result T[(m,sh) = 4q+r][c = 16 nt + n16]; column 30: the C1 bias gradient
  float g_b;      // FC bias gradient of output out_of_lane(lane)
  float g_b2, loss;
};
__device__ __forceinline__ void wave_init(WaveState& st) {
#pragma unroll
  for (int nt = 0; nt < 10; ++nt) st.acc_k2[nt] = f4{0.0f, 0.0f, 0.0f, 0.0f};
  st.acc_k1[0] = st.acc_k1[1] = f4{0.0f, 0.0f, 0.0f, 0.0f};
  st.g_b2 = st.loss = st.g_b = 0.0f;
}

// The lane index as a phase of the training step sees it: through a register the compiler cannot
// see through, so that the address arithmetic built on it is redone in every phase of every image
// instead of being computed once per kernel and held in (scarce) registers for its whole life.
__device__ __forceinline__ int phase_lane() {
  int l = threadIdx.x & 63;
  asm volatile("" : "+v"(l));
  return l;
}
// What a wave does of an image.  LONE: everything.  Where there is a SIMD for every image and more waves than images
// (train_kernel, PAIR), two waves of a SIMD share one: they take different column tiles of C1, pixel tiles of C2, pixels of the C2 weight
// gradient and input maps of the C2 input error, both make the outputs, and hand over at workgroup barriers (all waves of the workgroup
// pass all of them):
//   in the image's area     written                         read by both behind
//   image and its pieces    place_image, half each          the barrier in train_kernel
//   S1, first copy          C1 forward, tiles 0-4 / 5-8     the first barrier here: the second copy, and with the next one C2
//   S1, second copy         over the image's pieces, halves the second
//   s2                      C2 forward, two pixel tiles each  the third
//   records of d_c2         over S1, which both have done with at the fourth; two pixel tiles each  the fifth
//   d_s1                    col2im, maps 0-3 / 4, 5         the sixth
// and in each wave's own: its d_s2 and its tiles of the C1 error.
enum WavePart { LONE, FIRST, SECOND };
// The image into LDS, as it is and in pieces.
template <WavePart PART>
__device__ __forceinline__ void place_image(WaveTrainLds& s, const Pixels& px) {
  const int l = threadIdx.x & 63;
  if (PART != SECOND) store_pixels(s.img, px);
  unsigned* pieces = reinterpret_cast<unsigned*>(s.pool) + W_PIECES;
  if (PART != SECOND) split_store_pixels(pieces, l, px.a);
  if (PART != FIRST) {
    split_store_pixels(pieces, l + 64, px.b);
    split_store_pixels(pieces, l + 128, px.c);
    if (l < 4) split_store_pixels(pieces, l + 192, px.d);
  }
}
// Touches the 25 cache lines of an image so that they are on their way into the L2 cache; the value
// is not used (the asm keeps the load alive and costs no instruction).
__device__ __forceinline__ void touch_pixels(const float* __restrict__ image) {
  const int l = threadIdx.x & 63;
  float v = image[l < 25 ? 32 * l : 0];
  asm volatile("" ::"v"(v));
}

// The second copy of S1's pieces (cnn_split.h), a word per lane: contiguous, where wider stores would not be aligned.
template <WavePart PART>
__device__ __forceinline__ void s1_second_copy(float* pool) {
  const int l = threadIdx.x & 63;
  const unsigned* from = reinterpret_cast<const unsigned*>(pool) + W_S1 + l;
  unsigned* to = reinterpret_cast<unsigned*>(pool) + W_S1 + SPLIT_S1B + l;
  constexpr int WHOLE = SPLIT_S1_COPY / 64, REST = SPLIT_S1_COPY % 64;
  constexpr int K0 = PART == SECOND ? WHOLE / 2 : 0, K1 = PART == FIRST ? WHOLE / 2 : WHOLE;
  unsigned v[WHOLE + 1];
#pragma unroll
  for (int k = K0; k < K1; ++k) v[k] = from[64 * k];
  if (PART != FIRST && l < REST) v[WHOLE] = from[64 * WHOLE];
#pragma unroll
  for (int k = K0; k < K1; ++k) to[64 * k] = v[k];
  if (PART != FIRST && l < REST) to[64 * WHOLE] = v[WHOLE];
}

// One image through forward and backward.  The image is in s (place_image) on entry and `next_image` (any valid image when
// there is no next one) on return; `hist` is the image's history row (FC_HIST floats).  `sign` (1 or -1): what d_c2 is taken
// with in the bfloat16 products, another in every other wave: the instruction cuts what it aligns towards minus infinity
// (cnn_split.h, bwd_negative), and the sums over images would add that up.
// FIRST and SECOND: `s` is the image's area, `own` the wave's (LONE and FIRST: the same); no next image and no history: SECOND leaves the FC
// weight gradient of its one image in `fc_grad`, of output o and input lane + 64 k.
template <WavePart PART>
__device__ __forceinline__ void wave_image(WaveState& st, WaveTrainLds& s, WaveTrainLds& own, const TrainOperands& ops,
                                           const float* __restrict__ next_image, int label, float sign, float* hist, float (&fc_grad)[NY][3]) {
  constexpr int T0 = PART == SECOND ? 5 : 0, T1 = PART == FIRST ? 5 : 9;  // column tiles of C1
  constexpr int M0 = PART == SECOND ? 2 : 0, MN = PART == LONE ? 4 : 2;   // pixel tiles of C2
  constexpr int S0 = M0 / 2, SN = MN / 2;
  auto hand_over = [&]() {
    if (PART == LONE)
      wave_sync();
    else
      __syncthreads();
  };
  unsigned short* s1 = reinterpret_cast<unsigned short*>(s.pool + W_S1);
  // ---- C1 = sigmoid(mconv(I, k1, b1)), S1 = sums of avgpool's windows (cnn_split.h): lane (q, n16) keeps the six maps
  //      of pixel y = 8 ty + n16 % 8, x = 8 tx + 4 (n16 / 8) + q of the column tiles T = 3 ty + tx --------------------
  float c1[9][6];  // (of the wave's tiles)
  {
    const int l = phase_lane(), n16 = l & 15;
    const C1SLane ln = c1s_lane(reinterpret_cast<const unsigned*>(s.pool) + W_PIECES, l);
    const int es = c1s_lane_s1(l), eh = es + 4 - 2 * (n16 & 1);
    C1SWeights w;
    c1s_load_weights(w, ops.items, l);
    f4 bias1a, bias1b = f4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int i = 0; i < 4; ++i) bias1a[i] = NEG_LOG2E * ops.bias[TAB_BIAS_B1 + i];
#pragma unroll
    for (int i = 0; i < 2; ++i) bias1b[i] = NEG_LOG2E * ops.bias[TAB_BIAS_B1 + 4 + i];
    float low = 0.0f, high = 0.0f;  // of the pair's first tile
    C1SItems it[2];
    c1s_load(it[T0 & 1], ln, T0);
#pragma unroll
    for (int T = T0; T < T1; ++T) {
      if (T < T1 - 1) c1s_load(it[(T + 1) & 1], ln, T + 1);
      f4 d0 = bias1a, d1 = bias1b;
      c1s_gemm(w, it[T & 1], d0, d1);
#pragma unroll
      for (int i = 0; i < 6; ++i) c1[T][i] = logistic_of_scaled(i < 4 ? d0[i & 3] : d1[i & 3]);
      float lo, hi;
      c1s_pool(c1[T], lo, hi);
      if (T == T1 - 1 && ((T1 - T0) & 1)) {
        split_store_s1<false>(s1, es + c1s_tile_s1(T), lo, eh + c1s_tile_s1(T), c1s_pool_rows(hi, hi));
      } else if ((T - T0) & 1) {
        split_store_s1<false>(s1, es + c1s_tile_s1(T - 1), low, es + c1s_tile_s1(T), lo);
        split_store_s1_one<false>(s1, eh + ((n16 & 1) ? c1s_tile_s1(T) : c1s_tile_s1(T - 1)), c1s_pool_rows(high, hi));
      }
      low = lo;
      high = hi;
    }
    // the words behind the planes are read by the last items and meet zero weights (the second copy takes them along)
    if (PART != SECOND && l < 4) s.pool[W_S1 + 3 * SPLIT_S1_PLANE + l] = 0.0f;
  }
  hand_over();
  s1_second_copy<PART>(s.pool);
  hand_over();
  if (PART == LONE) touch_pixels(next_image);
  // ---- C2 = sigmoid(mconv(S1, k2, b2)), S2 = avgpool(C2): a lane's four result registers are one window -------------
  f4 c2v[MN];
  {
    const int l = phase_lane(), q = l >> 4, n16 = l & 15;
#pragma unroll
    for (int mt = 0; mt < MN; ++mt) c2v[mt] = f4{st.bias2, st.bias2, st.bias2, st.bias2};
    c2s_gemm<M0, MN>(c2v, c2s_lane(reinterpret_cast<const unsigned*>(s.pool + W_S1), ops.items, l));
#pragma unroll
    for (int mt = 0; mt < MN; ++mt) {
#pragma unroll
      for (int r = 0; r < 4; ++r) c2v[mt][r] = logistic_of_scaled(c2v[mt][r]);
      if (n16 < 12) s.pool[W_S2 + n16 * S2_MAP + 4 * (M0 + mt) + q] = 0.25f * ((c2v[mt][0] + c2v[mt][1]) + (c2v[mt][2] + c2v[mt][3]));
    }
  }
  hand_over();
  // ---- output = sigmoid(mconv(S2, fc, b)), its error, FC backweights / backbias / backin: the lane owns the inputs lane,
  //      lane + 64, lane + 128 and the output out_of_lane(lane) --------------------------------------------------------
  {
    const int l = phase_lane();
    const bool out_lane = (OUT_LANES >> l) & 1;
    const float* fc = ops.fc + l;
    float sv[3], p[NY];
#pragma unroll
    for (int k = 0; k < 3; ++k) sv[k] = s.pool[W_S2 + s2_at(l + 64 * k)];
#pragma unroll
    for (int o = 0; o < NY; ++o) p[o] = fmaf(fc[(3 * o + 2) * 64], sv[2], fmaf(fc[(3 * o + 1) * 64], sv[1], fc[3 * o * 64] * sv[0]));
    const float y = logistic(wave_sum10(p) + ops.bias[TAB_BIAS_B + out_of_lane(l)]);
    const float e = out_lane ? y - (out_of_lane(l) == label ? 1.0f : 0.0f) : 0.0f;
    const float mine = e * fmaf(-y, y, y);  // y (1 - y) as y - y^2: one instruction
    if (PART != SECOND) {
      st.loss = fmaf(0.5f * e, e, st.loss);
      st.g_b += mine;
    }
    // s2 and delta go to the image's history row, the products are taken once per wave
    if (PART == LONE) {
#pragma unroll
      for (int k = 0; k < 3; ++k) hist[l + 64 * k] = sv[k];
      if (out_lane) hist[FC_HIST_DELTA + out_of_lane(l)] = mine;
      if (l >= 4 && l < 10) hist[FC_HIST_DELTA + 6 + l] = 0.0f;
    }
    float delta[NY];
#pragma unroll
    for (int o = 0; o < NY; ++o)
      delta[o] = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, mine), o < 8 ? 16 * (o >> 2) + (o & 3) : 24 + o));
    if (PART == SECOND)
#pragma unroll
      for (int o = 0; o < NY; ++o)
#pragma unroll
        for (int k = 0; k < 3; ++k) fc_grad[o][k] = delta[o] * sv[k];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      float d = 0.0f;
#pragma unroll
      for (int o = 0; o < NY; ++o) d = fmaf(fc[(3 * o + k) * 64], delta[o], d);
      own.pool[W_DS2 + s2_at(l + 64 * k)] = d;
    }
  }
  wave_sync();
  // ---- backavgpool through S2 and the derivative of C2's sigmoid, in the MFMA result layout; C2 backweights ----------
  u4v d2[2][3];  // pieces k of the tiles 2 S (first two words) and 2 S + 1, registers in pairs
  {
    const int l = phase_lane(), q = l >> 4, n16 = l & 15;
#pragma unroll
    for (int mt = M0; mt < M0 + MN; ++mt) {
      const float up = own.pool[W_DS2 + (n16 < 12 ? n16 : 0) * S2_MAP + 4 * mt + q] * (0.25f * sign);  // (padding rows: map 0's)
      f4 d;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float c = c2v[mt - M0][r];
        d[r] = up * fmaf(-c, c, c);
      }
      st.g_b2 = fmaf(sign, (d[0] + d[1]) + (d[2] + d[3]), st.g_b2);
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const Split2 p = split2(d[2 * h], d[2 * h + 1]);
        d2[mt >> 1][0][2 * (mt & 1) + h] = p.h;
        d2[mt >> 1][1][2 * (mt & 1) + h] = p.m;
        d2[mt >> 1][2][2 * (mt & 1) + h] = p.l;
      }
    }
    k2_gradient<S0, SN>(st.acc_k2, d2, reinterpret_cast<const unsigned*>(s.pool + W_S1), l);
  }
  hand_over();
  // S1 is dead: d_c2 as records of its pixels
  store_records<S0, SN>(reinterpret_cast<unsigned short*>(s.pool + W_D2), d2, phase_lane());
  hand_over();

  // ---- C2 backin into d_s1 -----------------------
  col2im_split<PART != SECOND, PART != FIRST>(ops.bwd, reinterpret_cast<const unsigned short*>(s.pool + W_D2), s.pool + W_DS1, sign, phase_lane());
  hand_over();
  // ---- backavgpool through S1 and the derivative of C1's sigmoid, then C1 backweights as a GEMM over pixel pairs (cnn_wave.h),
  //      column tile by column tile of C1: eight K steps of one row and four pairs.  A tile's error goes to LDS, as
  //      d1[6][x / 2 % 2][8][x / 4][x % 2] with the parts D1T_HALF and D1T_MAP apart (stores and loads of 32 lanes on 32
  //      banks), while the products of the tile before are made from the other buffer -----------------------------------
  {
    const int l = phase_lane(), q = l >> 4, n16 = l & 15, a = (n16 >> 1) & 3, bx = n16 >> 3;
    const float* up = s.pool + W_DS1 + a * DS1_ROW + 2 * bx + (q >> 1);
    float* dst = own.pool + W_D1 + (q >> 1) * D1T_HALF + 4 * (n16 & 7) + 2 * bx + (q & 1);
    float e[2][6];  // the error at S1 over a tile
    auto fetch = [&](int T) {
      const int o = 4 * DS1_ROW * (T / 3) + 4 * (T % 3);
#pragma unroll
      for (int i = 0; i < 6; ++i) e[T & 1][i] = up[i * DS1_MAP + o];
    };
    auto stage = [&](int T) {
#pragma unroll
      for (int i = 0; i < 6; ++i) {
        const float c = c1[T][i];
        // c (1 - c); the pooling's 1/4 is in the weights.  (backbias: the GEMM sums d1 in its padding column.)
        dst[i * D1T_MAP + (T & 1) * D1T_WORDS] = e[T & 1][i] * fmaf(-c, c, c);
      }
    };
    const float* pa = own.pool + W_D1 + ((n16 >> 1) % 6) * D1T_MAP + (q & 1) * D1T_HALF + 2 * (q >> 1) + (n16 & 1);
    const int c0 = n16, c1x = 16 + n16;
    const float* pb0 = s.img + (c0 / 6) * 28 + c0 % 6 + 2 * q;
    const float* pb1 = n16 >= 14 ? ops.ones + 2 * q : s.img + (c1x / 6) * 28 + c1x % 6 + 2 * q;
    const int step1 = n16 >= 14 ? 0 : 1;  // the padding columns 30, 31 read 1.0 whatever the tile
    float oa[2][8], ob0[2][8], ob1[2][8];
    auto load = [&](int T) {
      const int at = 224 * (T / 3) + 8 * (T % 3);
      const float* b1 = pb1 + step1 * at;
#pragma unroll
      for (int y = 0; y < 8; ++y) {
        oa[T & 1][y] = pa[(T & 1) * D1T_WORDS + 4 * y];
        ob0[T & 1][y] = pb0[at + 28 * y];
        ob1[T & 1][y] = b1[28 * y];
      }
    };
    fetch(T0);
    fetch(T0 + 1);
    stage(T0);
    wave_sync();
    load(T0);
    fetch(T0 + 2);
    stage(T0 + 1);
    wave_sync();
    Pixels nx;
    f4 sum[2] = {f4{0.0f, 0.0f, 0.0f, 0.0f}, f4{0.0f, 0.0f, 0.0f, 0.0f}};  // the image's own, as in k2_gradient
    // The products of tile T, the loads of tile T + 1, the stores of tile T + 2 (into the buffer whose loads are done)
    // and the error at S1 for tile T + 3
#pragma unroll
    for (int T = T0; T < T1; ++T) {
      if (T + 3 < T1) fetch(T + 3);
      if (T + 2 < T1) stage(T + 2);
      if (T + 1 < T1) load(T + 1);
      // the next image's pixels (touched into the L2 cache long ago) are fetched under the last products, when the
      // fewest registers are in use (through an offset the compiler cannot see before this point: it would otherwise
      // start the loads, and occupy their sixteen registers, phases earlier)
      if (PART == LONE && T == 7) {
        int zero = 0;
        asm volatile("" : "+v"(zero));
        nx = load_pixels(next_image + zero);
      }
#pragma unroll
      for (int y = 0; y < 8; ++y) {
        sum[0] = mfma16(oa[T & 1][y], ob0[T & 1][y], sum[0]);
        sum[1] = mfma16(oa[T & 1][y], ob1[T & 1][y], sum[1]);
      }
#pragma unroll
      for (int y = 0; y < 8; ++y) {
        __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
        if (T + 2 < T1) __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);
        if (T + 2 < T1) __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
        if (T + 1 < T1) __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
      }
      wave_sync();
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) st.acc_k1[t][r] += sum[t][r];
    if (PART == LONE) {
      place_image<LONE>(s, nx);
      wave_sync();
    }
  }
}

// FC weight gradient of a wave from the history rows of its images (see FC_HIST).  One K step of the
// GEMM takes up to four images: lane (q, n16) supplies A[o = n16][k = q] = delta of the step's q-th
// image and B[k = q][i = n16] = its s2[16 nt + n16] for the twelve tiles nt.  Result tile nt,
// register r of lane (q, n16): g_fc[o = 4 q + r][i = 16 nt + n16].
struct FcStepOperands {
  float a, b[12];
};
// rows[k] points at the row of the step's k-th image, or at any valid row when the step has fewer
// than four (`count` says how many are real: the others contribute delta = 0).
__device__ __forceinline__ void fc_step_load(FcStepOperands& op, const float* const (&rows)[4], int count) {
  const int l = threadIdx.x & 63, q = l >> 4, n16 = l & 15;
  const float* mine = q == 0 ? rows[0] : q == 1 ? rows[1] : q == 2 ? rows[2] : rows[3];
  op.a = mine[FC_HIST_DELTA + n16];
  if (q >= count) op.a = 0.0f;
#pragma unroll
  for (int nt = 0; nt < 12; ++nt) op.b[nt] = mine[16 * nt + n16];
}
__device__ __forceinline__ void fc_step_mfma(f4 (&g_fc)[12], const FcStepOperands& op) {
#pragma unroll
  for (int nt = 0; nt < 12; ++nt) g_fc[nt] = mfma16(op.a, op.b[nt], g_fc[nt]);
}

// Writes the wave's gradient sums as one partial row (PSTRIDE floats in parameter order, the loss
// in LOSS_SLOT, zeros after it) to `row`, every slot by exactly one lane.  `row` may be the start
// of the wave's own LDS area (all of it is dead once the wave's images are done); `park` is
// C1G_PARK floats of LDS outside the row that no other wave uses; the FC weight gradient is `g_fc` (LONE) or `fc_grad` (SECOND; FIRST
// has none, and its row no FC weights).
template <WavePart PART>
__device__ __forceinline__ void wave_flush(WaveState& st, float sign, const f4 (&g_fc)[12], const float (&fc_grad)[NY][3], float* row, float* park) {
  const int l = threadIdx.x & 63, q = l >> 4, n16 = l & 15;
  // The stores are grouped by the lanes that take part (one branch per group, not one per store):
  // FC rows o = 4 q + r < 10 are registers 0, 1 of the quarters 0..2 and registers 2, 3 of the quarters
  // 0, 1; C2 rows j = 4 q + r < 12 are every register of the quarters 0..2, and of the last tap tile
  // only the columns n16 < 6 are taps.
  if (PART == SECOND) {
#pragma unroll
    for (int o = 0; o < NY; ++o)
#pragma unroll
      for (int k = 0; k < 3; ++k) row[OFF_FC + o * NS2 + l + 64 * k] = fc_grad[o][k];
  }
  if (PART == LONE) {
    float* fc = row + OFF_FC + 4 * q * NS2 + n16;
    if (q < 3) {
#pragma unroll
      for (int nt = 0; nt < 12; ++nt)
#pragma unroll
        for (int r = 0; r < 2; ++r) fc[r * NS2 + 16 * nt] = g_fc[nt][r];
    }
    if (q < 2) {
#pragma unroll
      for (int nt = 0; nt < 12; ++nt)
#pragma unroll
        for (int r = 2; r < 4; ++r) fc[r * NS2 + 16 * nt] = g_fc[nt][r];
    }
  }
  if ((OUT_LANES >> l) & 1) row[OFF_B + out_of_lane(l)] = st.g_b;
  const float loss = wave_sum(st.loss);  // lanes without an output hold zero
  if (l < PSTRIDE - LOSS_SLOT) row[LOSS_SLOT + l] = l == 0 ? loss : 0.0f;
  if (q < 3) {
    // column kk = 16 t + n16 of kernel row u is element (v, c) = (kk / 6, kk % 6); S1 was kept as sums of four
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int kk = 16 * t + n16;
      float* k2 = row + OFF_K2 + 4 * q * 150 + (kk % 6) * 25 + kk / 6;
      if (kk < 30) {
#pragma unroll
        for (int u = 0; u < 5; ++u)
#pragma unroll
          for (int r = 0; r < 4; ++r) k2[r * 150 + 5 * u] = (0.25f * sign) * st.acc_k2[2 * u + t][r];
      }
    }
  }
  {
    float v = st.g_b2;  // lane (q, j): sum over the four lane quarters
    v += __shfl_xor(v, 16);
    v += __shfl_xor(v, 32);
    if (q == 0 && n16 < 12) row[OFF_B2 + n16] = v;
  }
  // C1 weights: the two shifted halves of the GEMM result are joined through LDS
  c1g_park(st.acc_k1, park);
  wave_sync();
#pragma unroll
  for (int round = 0; round < 3; ++round) {
    const int e = l + 64 * round;
    if (e < 150) row[OFF_K1 + e] = c1g_combine(park, e);
  }
  // C1 biases: column 30 of the same result holds the sums of d1 by (map, x parity)
  if (l < 6) row[OFF_B1 + l] = park[(2 * l) * 32 + 30] + park[(2 * l + 1) * 32 + 30];
}

}  // namespace cnn
