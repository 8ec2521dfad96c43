// Small-batch form of the fused step: EIGHT WAVEFRONTS (two per SIMD of a compute unit) SHARE ONE
// IMAGE.  Same arithmetic, same operand table, same LDS arrays and the same MFMA formulations as
// cnn_wave.h (arXiv 1912.05234, Section 3); only the division of labour differs, to cut the latency
// of a single image when there are too few images to give every SIMD its own.  Two waves per SIMD
// because one wave alone issues a vector instruction only every ~5 cycles, two reach ~2.4.
//
//   C1 forward and C1 error      GEMM tiles T = wave, wave + 8 (waves 0, 1 also T = wave + 16), cnn_wave.h
//   C1 weight gradient           the GEMM's K steps that belong to the wave's own C1 tiles
//   C2 forward                   waves 0..3: pixel tile mt = wave
//   output layer, C2 error       waves 4..7: each all ten outputs, and pixel tile mt = wave - 4
//   FC weight gradient           waves 4..6 take the three 4-output row tiles
//   C2 input error (col2im)      waves 0..3: input maps 4 cg .. 4 cg + 3, cg = wave % 2, and pixel tiles
//                                nt = 2 h, 2 h + 1, h = wave / 2; half h adds into its own copy of d_s1,
//                                so no two waves ever touch the same cell; the C1 error reads both copies
//   C2 weight gradient           waves 4..7: tap tiles nt = 0-1, 2-3, 4-6, 7-9 over all 64 pixels (each wave
//                                owns whole columns of the result, so nothing has to be added across waves);
//                                of an UPPER workgroup (GroupPart) all eight waves, two or one tile each
//
// Phases that hand data between waves are separated by workgroup barriers (five, plus one in the
// final cross-wave sums).  A workgroup handles exactly one image, and an image has one workgroup (WHOLE) or two
// (LOWER and UPPER).
// Clocks at which the barriers and the end are reached, of the slowest wave, 100 images in two workgroups each / 200 in one:
//   (1) set-up 1.3 LOWER, 1.0 UPPER / 1.3 thousand; (2) C1 5.0, 4.7 / 5.2; (3) C2 7.0, 6.7 / 7.4; (4) outputs and errors 8.3, 8.5 / 9.0;
//   (5) input error 11.0, C2 gradient 11.0 / both 13.3; C1 backward 13.9, - / 16.0; sums and stores 15.1, 12.7 / 18.0.
#pragma once

#include "cnn_split.h"

namespace cnn {

constexpr int GWAVES = 8;  // waves per workgroup of the small-batch kernel
// Second col2im target: [6][12][12] plus the cells behind it that the rows of the padding maps 6, 7
// rewrite with themselves (+ 0.0), as they do behind the first target inside TrainLds.
constexpr int D_S1B_FLOATS = NS1 + 304;

// What a workgroup does of its image's step.  WHOLE: everything.  Where there are two compute units per image (GROUP_PAIR_MAX_BATCH),
// two workgroups share it: both run the forward pass, then LOWER takes the C2 input error and the C1 gradient, UPPER
// the FC and C2 gradients and the loss, and each writes its part of the image's partial row.  Every sum is made in the
// same order in all of them.
enum GroupPart { WHOLE, LOWER, UPPER };

// Tap tiles of the C2 weight gradient owned by wave 4 + i: first tile and count; of UPPER, by wave i.
template <GroupPart PART>
__host__ __device__ constexpr int k2_first(int i) {
  return PART == UPPER ? (i < 2 ? 2 * i : i + 2) : i < 2 ? 2 * i : 3 * i - 2;
}
template <GroupPart PART>
__host__ __device__ constexpr int k2_count(int i) { return PART == UPPER ? (i < 2 ? 2 : 1) : i < 2 ? 2 : 3; }

struct GroupState {
  float bias2;      // b2[n16]
  f4 acc_k2[3];     // waves 4..7 (UPPER: all): C2 weight gradient tiles nt = k2_first(wave - 4 or wave) + k
  f4 acc_k1[2];     // C1 weight gradient GEMM over the K steps of this wave's tiles, T[(m,sh)][c]
  f4 acc_fc[3];     // waves 4..6: FC weight gradient rows o = 4 fw + r, columns lane + 64 k
  float g_bq;       // waves 4..6: FC bias gradient b[4 fw + lane % 4]
  float g_b1[2];    // C1 bias gradient of maps 2q, 2q + 1 over this lane's pixels
  float g_b2, loss;  // (loss: the lane's output's share)
};

// C1 forward + S1 for this wave's NT tiles T = wave + 8 k of the C1 GEMM (cnn_wave.h): returns the
// activations in c1[k].  `c1a` are the eight operand entries, `bias` the table's biases.  All MFMAs
// first (two independent chains at a time), then the sigmoids and the pooling.
template <int NT>
__device__ __forceinline__ void group_c1_forward(const float* c1a, const float* bias, const float* img, float* s1, int wave,
                                                 const C1Lane& ln, f4 (&c1)[3]) {
  const int l = threadIdx.x & 63, q = l >> 4;
  float wa[C1F_KSTEPS];
#pragma unroll
  for (int ks = 0; ks < C1F_KSTEPS; ++ks) wa[ks] = c1a[ks * 64 + l];
  f4 binit = f4{0.0f, 0.0f, 0.0f, 0.0f};
  if (q < 3) {
    const float2 bq = *reinterpret_cast<const float2*>(&bias[TAB_BIAS_B1 + 2 * q]);
    binit = f4{bq.x, bq.x, bq.y, bq.y};
  }
  c1f_gemm_pair(wa, ln, img + c1f_tile_img(wave), img + c1f_tile_img(wave + 8), binit, c1[0], c1[1]);
  if (NT == 3) c1f_gemm_one(wa, ln, img + c1f_tile_img(wave + 16), binit, c1[2]);
#pragma unroll
  for (int k = 0; k < NT; ++k) c1f_finish(c1[k], ln, s1 + c1f_tile_s1(wave + 8 * k));
}

// K steps FIRST .. FIRST + COUNT - 1 of the C2 forward GEMM (cnn_wave.h) for one pixel tile, added to acc;
// `s1` is that tile's origin for this lane's pixel, `bf` the lane's column of the operand entries.
template <int FIRST, int COUNT>
__device__ __forceinline__ void group_c2_steps(const float* s1, const float* bf, f4& acc) {
  const int q = (threadIdx.x & 63) >> 4;
  const float *a12 = s1 + 12 * q, *a1 = s1 + q, *a144 = s1 + 144 * q;
  // operands of step s + AHEAD are read while step s issues: an LDS read takes longer than three
  // matrix instructions, and with eight waves per image there are registers to spare
  constexpr int AHEAD = 6, SLOTS = 8;
  float opa[SLOTS], opw[SLOTS];
  auto load_step = [&](int k, float& oa, float& ow) {
    const int sidx = FIRST + k;
    const float* base = sidx < 30 ? a12 : sidx < 36 ? a1 : a144;
    ow = bf[sidx * 64];
    oa = base[fwd_imm(sidx)];
  };
#pragma unroll
  for (int k = 0; k < AHEAD; ++k) load_step(k, opa[k], opw[k]);
  // even and odd K steps in two sums: a matrix instruction waits for the previous one of its own
  // chain only
  f4 odd = f4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int k = 0; k < COUNT; ++k) {
    if (k + AHEAD < COUNT) load_step(k + AHEAD, opa[(k + AHEAD) % SLOTS], opw[(k + AHEAD) % SLOTS]);
    if (k & 1)
      odd = mfma16(opa[k % SLOTS], opw[k % SLOTS], odd);
    else
      acc = mfma16(opa[k % SLOTS], opw[k % SLOTS], acc);
    if (k + AHEAD < COUNT) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) acc[r] += odd[r];
}

// C1 error of this wave's tiles into the staged d1[6][24][24]; the error at S1 is the sum of the two
// col2im copies.  Lanes q = 3 hold padding rows.
template <int NT>
__device__ __forceinline__ void group_c1_error(GroupState& st, TrainLds& s, const float* d_s1b, int wave,
                                               const C1Lane& ln, const f4 (&c1)[3]) {
  const int q = (threadIdx.x & 63) >> 4;
  if (q < 3) {
#pragma unroll
    for (int k = 0; k < NT; ++k) {
      const int T = wave + 8 * k, o = ln.s1 + c1f_tile_s1(T);
      // (the average pooling's 1/4 is in the col2im operand of the table)
      const float up0 = s.d_s1[o] + d_s1b[o], up1 = s.d_s1[o + 144] + d_s1b[o + 144];
      const f4 c = c1[k];
      const float2 da = float2{up0 * c[0] * (1.0f - c[0]), up0 * c[1] * (1.0f - c[1])};
      const float2 db = float2{up1 * c[2] * (1.0f - c[2]), up1 * c[3] * (1.0f - c[3])};
      st.g_b1[0] += da.x + da.y;
      st.g_b1[1] += db.x + db.y;
      float* dst = s.pool + ln.c1 + c1f_tile_c1(T);
      *reinterpret_cast<float2*>(dst) = da;
      *reinterpret_cast<float2*>(dst + D1_MAP) = db;
    }
  }
}

// C2 weight gradient for COUNT tap tiles over all four pixel tiles: sixteen K steps in one straight
// line (no branches), so that the operand reads of later steps are issued under the MFMAs of
// earlier ones.  bsrc[k] points at the lane's tap of tile k in s1.
template <int COUNT>
__device__ __forceinline__ void group_k2_gradient(f4 (&acc)[3], const TrainLds& s, const float* const (&bsrc)[3]) {
  const int l = threadIdx.x & 63, q = l >> 4, n16 = l & 15;
  f4 a[4];
#pragma unroll
  for (int S = 0; S < 4; ++S) a[S] = *reinterpret_cast<const f4*>(&s.pool[P_D2 + n16 * D2S + 16 * S + 4 * q]);
#pragma unroll
  for (int step = 0; step < 16; ++step) {
    const int S = step >> 2, r = step & 3, off = 24 * S + 12 * (r >> 1) + (r & 1);
#pragma unroll
    for (int k = 0; k < COUNT; ++k) acc[k] = mfma16(a[S][r], bsrc[k][off], acc[k]);
  }
}

// A value of the partial row.  COHERENT (the device-side epoch loop, where other compute units read
// the row during the same kernel): an agent-scope store, written through to memory.
template <bool COHERENT>
__device__ __forceinline__ void put_row(float* p, float v) {
  if (COHERENT)
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else
    *p = v;
}

// A value of the operand table past LDS.  (A function, whose argument is not `restrict`: read through the table's own pointer the loads
// are placed otherwise, and an epoch of 600 steps of 100 images takes 6731 instead of 6717 us.)
__device__ __forceinline__ float table_value(const float* p) { return *p; }

// The whole step for the workgroup's image (`image`, `label` point at it); one partial row, `out`.
// `d_s1b` is the second col2im target (D_S1B_FLOATS floats).  COHERENT: see put_row and TableLoad.
template <bool COHERENT, GroupPart PART>
__device__ __forceinline__ void group_train(const float* __restrict__ image,
                                            const int32_t* __restrict__ label_ptr,
                                            const float* __restrict__ tabg, float* __restrict__ out,
                                            OperandTable<TAB_TRAIN_ENTRIES>& tab, TrainLds& s, float* d_s1b) {
  const int t = threadIdx.x, wave = t >> 6, l = t & 63, q = l >> 4, n16 = l & 15, sub = l & 3;
  const int pp = 12 * ((n16 & 3) >> 1) + 2 * (n16 >> 2) + (n16 & 1);
  const float* tl = tab.e + l;
  const int pix = t < NI / 4 ? t : 0;  // the 16-byte piece of the image this thread moves
  CNN_GROUP_MARK(0);

  f4 px = reinterpret_cast<const f4*>(image)[pix];
  const int label = *label_ptr;  // in flight during the set-up too
  // the C1 forward operands (the table's last entries) and the biases come first: see barrier (1)
  // (the FC weights go to the upper waves' registers, with COHERENT by way of LDS; UPPER has no C2 input error)
  constexpr int SKIPPED = COHERENT ? 0 : (PART == UPPER ? TAB_C1A : TAB_AB) - TAB_FCW;
  TableLoad<TAB_TRAIN_ENTRIES, 64 * GWAVES, COHERENT, TAB_TRAIN_ENTRIES, TAB_C1A, TAB_FCW, SKIPPED> table;
  table.fetch(tabg);
  // every LDS cell that padded GEMM steps may read starts finite, and both col2im targets start at
  // zero (the image area is written below, before the first barrier, so it is left alone here)
  for (int e = t; PART != UPPER && e < D_S1B_FLOATS / 4; e += 64 * GWAVES) {
    if (e < NS1 / 4) reinterpret_cast<f4*>(s.d_s1)[e] = f4{0.0f, 0.0f, 0.0f, 0.0f};
    reinterpret_cast<f4*>(d_s1b)[e] = f4{0.0f, 0.0f, 0.0f, 0.0f};
  }
  for (int e = t; e < POOL_FLOATS / 4; e += 64 * GWAVES) reinterpret_cast<f4*>(s.pool)[e] = f4{0.0f, 0.0f, 0.0f, 0.0f};
  GroupState st;
  const C1Lane ln = c1f_lane();
#pragma unroll
  for (int k = 0; k < 3; ++k) st.acc_k2[k] = f4{0.0f, 0.0f, 0.0f, 0.0f};
  st.acc_k1[0] = st.acc_k1[1] = f4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int k = 0; k < 3; ++k) st.acc_fc[k] = f4{0.0f, 0.0f, 0.0f, 0.0f};
  st.g_bq = 0.0f;
  st.g_b1[0] = st.g_b1[1] = 0.0f;
  st.g_b2 = 0.0f;
  st.loss = 0.0f;
  CNN_GROUP_MARK(1);
  // The lane-invariant address arithmetic of the phases below is independent of the table, so the
  // compiler is free to run it while the table's loads are still in flight; barrier (1) publishes
  // the image together with what the C1 forward pass reads of the table (its own operands and the
  // biases, fetched first); the rest of the table arrives during that pass and is published by
  // barrier (2).
  {
    table.commit_first(tab);
    if (t < NI / 4) reinterpret_cast<f4*>(s.img)[t] = px;
    CNN_GROUP_MARK(2);
    __syncthreads();  // (1) image, C1 forward operands and biases in LDS
    st.bias2 = tab.bias[n16];
    const int fw = wave & 3;
    const float bias3 = tab.bias[TAB_BIAS_B + out_of_lane(l)];

    // ---- C1 forward + S1 for this wave's tiles ---------------------------------------------------------
    f4 c1[3];
    if (wave < 2)
      group_c1_forward<3>(tab.e + TAB_C1A * 64, tab.bias, s.img, s.pool + P_S1, wave, ln, c1);
    else
      group_c1_forward<2>(tab.e + TAB_C1A * 64, tab.bias, s.img, s.pool + P_S1, wave, ln, c1);
    table.commit_rest(tab);
    // The output layer is the upper waves', each for itself (one hand-over between waves costs more than ten outputs): they wait
    // while the lower ones are busy with C2, and their lanes hold the weights of the inputs lane, lane + 64, lane + 128.  They come
    // past LDS, in flight over the barrier, but with COHERENT: beside what that loop over steps keeps they did not fit the registers.
    float fcw[NY][3];
    if (!COHERENT && wave >= 4) {
#pragma unroll
      for (int o = 0; o < NY; ++o)
#pragma unroll
        for (int k = 0; k < 3; ++k) fcw[o][k] = table_value(tabg + (TAB_FCW + 3 * o + k) * 64 + l);
    }
    CNN_GROUP_MARK(3);
    __syncthreads();  // (2) S1 and the operand table complete
    if (COHERENT && wave >= 4) {
#pragma unroll
      for (int o = 0; o < NY; ++o)
#pragma unroll
        for (int k = 0; k < 3; ++k) fcw[o][k] = tl[(TAB_FCW + 3 * o + k) * 64];
    }

    // ---- C2 forward for pixel tile mt = wave, S2 (waves 0..3) -----------------------------------------
    f4 c2v = f4{st.bias2, st.bias2, st.bias2, st.bias2};
    if (wave < 4) {
      group_c2_steps<0, 38>(s.pool + P_S1 + pp + 24 * wave, tl + TAB_BF * 64, c2v);
#pragma unroll
      for (int r = 0; r < 4; ++r) c2v[r] = logistic_of_scaled(c2v[r]);
      if (n16 < 12) s.pool[P_S2 + n16 * 16 + 4 * wave + q] = 0.25f * ((c2v[0] + c2v[1]) + (c2v[2] + c2v[3]));
      *reinterpret_cast<f4*>(&s.pool[P_D2 + n16 * D2S + 16 * wave + 4 * q]) = c2v;  // its error takes this place
    }
    CNN_GROUP_MARK(4);
    __syncthreads();  // (3) S2 and C2 complete

    // ---- output layer, its error, and the error at C2 for pixel tile fw (waves 4..7) ------------------------
    if (wave >= 4) {
      float sv[3], p[NY];
#pragma unroll
      for (int k = 0; k < 3; ++k) sv[k] = s.pool[P_S2 + l + 64 * k];
      f4* const d2 = reinterpret_cast<f4*>(&s.pool[P_D2 + n16 * D2S + 16 * fw + 4 * q]);
      const f4 c2 = *d2;
#pragma unroll
      for (int o = 0; o < NY; ++o) p[o] = fmaf(fcw[o][2], sv[2], fmaf(fcw[o][1], sv[1], fcw[o][0] * sv[0]));
      const bool out_lane = (OUT_LANES >> l) & 1;
      const float y = logistic(wave_sum10(p) + bias3);
      const float e = out_lane ? y - (out_of_lane(l) == label ? 1.0f : 0.0f) : 0.0f;
      const float mine = e * fmaf(-y, y, y);  // y (1 - y) as y - y^2: one instruction
      if (PART != LOWER && fw == 0) st.loss = 0.5f * e * e;
      auto from = [&](int lane) { return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, mine), lane)); };
      // the error at S2, of which the lane takes on element 16 n16 + 4 fw + q; then backavgpool and sigmoid'
      float* const d_s2 = s.pool + P_END + NS2 * fw;
      {
        float up[3] = {0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int o = 0; o < NY; ++o) {
          const float delta = from(o < 8 ? 16 * (o >> 2) + (o & 3) : 24 + o);
#pragma unroll
          for (int k = 0; k < 3; ++k) up[k] = fmaf(fcw[o][k], delta, up[k]);
        }
#pragma unroll
        for (int k = 0; k < 3; ++k) d_s2[l + 64 * k] = up[k];
      }
      wave_sync();
      const float up = 0.25f * d_s2[(n16 < 12 ? 16 * n16 : 0) + 4 * fw + q];
      f4 d2v;
#pragma unroll
      for (int r = 0; r < 4; ++r) d2v[r] = n16 < 12 ? up * c2[r] * (1.0f - c2[r]) : 0.0f;
      *d2 = d2v;
      if (PART != LOWER) {
        st.g_b2 += (d2v[0] + d2v[1]) + (d2v[2] + d2v[3]);
        if (fw < 3) {  // FC backweights / backbias, row tile mt = fw: outputs 4 fw .. 4 fw + 3 (lanes 34, 35 hold zeros)
          float d[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) d[r] = from(16 * fw + r);
          const float aq = (sub & 2) ? ((sub & 1) ? d[3] : d[2]) : ((sub & 1) ? d[1] : d[0]);
          st.g_bq += aq;
#pragma unroll
          for (int k = 0; k < 3; ++k) st.acc_fc[k] = mfma4(aq, sv[k], st.acc_fc[k]);
        }
      }
    }
    // (read before the barrier: the weights of the C2 input error, for input maps 4 cg .. 4 cg + 3)
    const int cg = wave & 1, h = (wave >> 1) & 1;
    float wt[7][3];
    if (PART != UPPER && wave < 4) {
      const float* ta = tl + (cg ? TAB_AB1 : TAB_AB) * 64;
#pragma unroll
      for (int tile = 0; tile < 7; ++tile)
#pragma unroll
        for (int sidx = 0; sidx < 3; ++sidx) wt[tile][sidx] = ta[(tile * 3 + sidx) * 64];
    }
    CNN_GROUP_MARK(6);
    __syncthreads();  // (4) d_c2 complete

    if (PART != UPPER && wave < 4) {
      // ---- C2 input error for input maps 4 cg .. 4 cg + 3 from the pixel tiles nt = 2 h, 2 h + 1
      //      (col2im rounds as in cnn_col2im.h restricted to those tiles: levels 4 h .. 4 h + 6) ---------------
      float bd[3][2];
#pragma unroll
      for (int sidx = 0; sidx < 3; ++sidx)
#pragma unroll
        for (int j = 0; j < 2; ++j) bd[sidx][j] = s.pool[P_D2 + (4 * sidx + q) * D2S + 16 * (2 * h + j) + n16];
      f4 t4[2];
      float t44[2];
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        f4 a = f4{0.0f, 0.0f, 0.0f, 0.0f}, c = a;
#pragma unroll
        for (int sidx = 0; sidx < 3; ++sidx) {
          a = mfma16(wt[kTileU4][sidx], bd[sidx][j], a);
          c = mfma16(wt[kTileC][sidx], bd[sidx][j], c);
        }
        t4[j] = a;
        t44[j] = c[0];
      }
      float* tgt = (h ? d_s1b : s.d_s1) + 144 * q + pp + 576 * cg + 48 * h;
#pragma unroll
      for (int v = 0; v < 5; ++v) {
        f4 tv[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          f4 a = f4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
          for (int sidx = 0; sidx < 3; ++sidx) a = mfma16(wt[kTileV0 + v][sidx], bd[sidx][j], a);
          tv[j] = a;
        }
        const float tu4[2] = {v < 4 ? t4[0][v < 4 ? v : 0] : t44[0], v < 4 ? t4[1][v < 4 ? v : 0] : t44[1]};
        {  // even levels 2 (2 h + mm), mm < 4: (j = mm, u = 0) + (mm - 1, 2) + (mm - 2, 4)
          const float e[4] = {tv[0][0], tv[1][0] + tv[0][2], tv[1][2] + tu4[0], tu4[1]};
          float old[4];
#pragma unroll
          for (int mm = 0; mm < 4; ++mm) old[mm] = tgt[24 * mm + v];
#pragma unroll
          for (int mm = 0; mm < 4; ++mm) tgt[24 * mm + v] = old[mm] + e[mm];
        }
        wave_sync();
        {  // odd levels 2 (2 h + mm) + 1, mm < 3: (j = mm, u = 1) + (mm - 1, 3)
          const float e[3] = {tv[0][1], tv[1][1] + tv[0][3], tv[1][3]};
          float old[3];
#pragma unroll
          for (int mm = 0; mm < 3; ++mm) old[mm] = tgt[24 * mm + 12 + v];
#pragma unroll
          for (int mm = 0; mm < 3; ++mm) tgt[24 * mm + 12 + v] = old[mm] + e[mm];
        }
        wave_sync();
      }
    }
    constexpr int K2_WAVE = PART == UPPER ? 0 : 4;  // the first wave that has tiles of the C2 weight gradient
    if (PART != LOWER && wave >= K2_WAVE) {
      // ---- C2 weight gradient: this wave's tap tiles over all four pixel tiles ---------------------------
      const int first = k2_first<PART>(wave - K2_WAVE), count = k2_count<PART>(wave - K2_WAVE);  // wave-uniform
      const float* bsrc[3];
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const int tap = 16 * (first + (k < count ? k : 0)) + n16;
        const int c = tap / 25, rem = tap - 25 * c, u = rem / 5, v = rem - 5 * u;
        bsrc[k] = s.pool + P_S1 + (tap < 150 ? c * 144 + u * 12 + v : 0) + 2 * q;
      }
      if (count == 3)
        group_k2_gradient<3>(st.acc_k2, s, bsrc);
      else if (count == 2)
        group_k2_gradient<2>(st.acc_k2, s, bsrc);
      else
        group_k2_gradient<1>(st.acc_k2, s, bsrc);
    }
    CNN_GROUP_MARK(7);
    if (PART != UPPER) __syncthreads();  // (5) both d_s1 copies complete; s1, d_c2 no longer needed

    // ---- C1 error for this wave's tiles, then the K steps of the C1 weight gradient GEMM that belong
    //      to the same tiles: a wave reads only the d1 cells it staged itself, so no barrier -------------
    const float* d1t[3];
    const float* imgt[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const int T = wave + 8 * k < C1F_TILES ? wave + 8 * k : wave;
      d1t[k] = s.pool + c1f_tile_c1(T);
      imgt[k] = s.img + c1f_tile_img(T);
    }
    if (PART == UPPER) {
    } else if (wave < 2) {
      group_c1_error<3>(st, s, d_s1b, wave, ln, c1);
      wave_sync();
      c1g_accumulate_tiles<3>(st.acc_k1, d1t, imgt);
    } else {
      group_c1_error<2>(st, s, d_s1b, wave, ln, c1);
      wave_sync();
      c1g_accumulate_tiles<2>(st.acc_k1, d1t, imgt);
    }
    CNN_GROUP_MARK(8);
  }

  const int fw = wave & 3;
  // ---- one partial row per workgroup: cross-wave sums through LDS in a fixed order -------------------
  // The parked values take the storage of the operand table, which nothing has read since barrier (4) but the lower waves of WHOLE
  // and LOWER, and barrier (5) is behind those.
  float* k1s = tab.e;                               // [8 waves][16][32]: parked C1 weight GEMM results
  float* b1s = tab.e + GWAVES * C1G_PARK;           // [8 waves][8]: C1 bias sums (256 floats reserved)
  float* b2s = b1s + 256;                           // [4 waves][64]: per-lane C2 bias sums
  static_assert(GWAVES * C1G_PARK + 256 + 256 <= TAB_TRAIN_ENTRIES * 64, "flush scratch fits the table");
  if (PART != UPPER) {
    c1g_park(st.acc_k1, k1s + wave * C1G_PARK);
    CNN_GROUP_MARK(11);
#pragma unroll
    for (int k = 0; k < 2; ++k) {  // C1 biases: lanes (q, .) hold maps 2q, 2q + 1
      float v = st.g_b1[k];
      v += quad_xor1(v);
      v += quad_xor2(v);
      v += dpp_row_half_mirror(v);
      v += dpp_row_mirror(v);
      if (n16 == 0 && q < 3) b1s[wave * 8 + 2 * q + k] = v;
    }
  }
  if (PART != LOWER && wave >= 4) b2s[fw * 64 + l] = st.g_b2;  // lane (q, j) of this wave's pixel tile
  CNN_GROUP_MARK(9);
  __syncthreads();
  CNN_GROUP_MARK(12);
  // (stores grouped by the lanes that take part: one branch per group, not one per store)
  constexpr int K2_WAVE = PART == UPPER ? 0 : 4;
  if (PART != LOWER && wave >= K2_WAVE) {  // C2 weights: every wave stores the columns (tap tiles) it owns; rows j = 4 q + r < 12
    const int first = k2_first<PART>(wave - K2_WAVE), count = k2_count<PART>(wave - K2_WAVE);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const int tap = 16 * (first + k) + n16;
      if (k < count && q < 3 && tap < 150) {
        float* dst = out + OFF_K2 + 4 * q * 150 + tap;
#pragma unroll
        for (int r = 0; r < 4; ++r) put_row<COHERENT>(dst + r * 150, st.acc_k2[k][r]);
      }
    }
  }
  if (PART != LOWER && wave >= 4 && fw < 3) {  // FC rows o = 4 fw + r < 10: the last wave has two
    float* dst = out + OFF_FC + 4 * fw * NS2;
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
      for (int r = 0; r < 2; ++r) put_row<COHERENT>(dst + r * NS2 + l + 64 * k, st.acc_fc[k][r]);
    if (fw < 2) {
#pragma unroll
      for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int r = 2; r < 4; ++r) put_row<COHERENT>(dst + r * NS2 + l + 64 * k, st.acc_fc[k][r]);
    }
    if (l < 4 && 4 * fw + l < 10) put_row<COHERENT>(out + OFF_B + 4 * fw + l, st.g_bq);
  }
  CNN_GROUP_MARK(13);
  if (PART != UPPER && wave < 3) {
    // one thread per C1 weight: the eight waves' shares of the GEMM, both shifted halves
    const int e = t;
    if (e < 150) {
      float x[GWAVES];
#pragma unroll
      for (int k = 0; k < GWAVES; ++k) x[k] = c1g_combine(k1s + k * C1G_PARK, e);
      put_row<COHERENT>(out + OFF_K1 + e, ((x[0] + x[1]) + (x[2] + x[3])) + ((x[4] + x[5]) + (x[6] + x[7])));
    }
  }
  if (wave == 3) {
    if (PART != UPPER && l < 6) {  // C1 biases: the eight waves' sums
      float x[GWAVES];
#pragma unroll
      for (int k = 0; k < GWAVES; ++k) x[k] = b1s[k * 8 + l];
      put_row<COHERENT>(out + OFF_B1 + l, ((x[0] + x[1]) + (x[2] + x[3])) + ((x[4] + x[5]) + (x[6] + x[7])));
    } else if (PART != LOWER && l >= 16 && l < 28) {  // C2 biases: 4 waves x 4 lane quarters
      const int j = l - 16;
      float x[16];
#pragma unroll
      for (int k = 0; k < 16; ++k) x[k] = b2s[k * 16 + j];
#pragma unroll
      for (int k = 0; k < 16; k += 4) x[k] = (x[k] + x[k + 1]) + (x[k + 2] + x[k + 3]);
      put_row<COHERENT>(out + OFF_B2 + j, (x[0] + x[4]) + (x[8] + x[12]));
    }
  }
  if (PART != LOWER && wave == 4) {
    const float loss = wave_sum(st.loss);
    if (l == 0) put_row<COHERENT>(out + LOSS_SLOT, loss);
  }
  CNN_GROUP_MARK(10);
}

// ---- forward pass alone: the same eight waves on one image -------------------------------------------------
// Here the K steps of C2 are shared too: waves 4..7 take the second half of pixel tile wave - 4's and hand their sums
// over through LDS (600 clocks of matrix instructions for one barrier).  The latency of one image bounds this kernel:
// one memory round trip for the image and the operands, then five short phases.
struct __align__(16) GroupForwardLds {
  float c1a[C1F_KSTEPS * 64];  // operand entries TAB_C1A ..
  float e[TAB_FWD_ENTRIES * 64];  // entries TAB_BF .., TAB_FCW ..
  float bias[TAB_BIAS_FLOATS];
  float img[NI];
  float s1[NS1 + 288];  // maps 6, 7: what the padding rows of C1 leave, finite, read by the padded K steps of C2
  float s2[NS2];
  f4 half[4 * 64];
  float y[16];
};

// yhat of the workgroup's image (`yhat`: its ten outputs in memory, or null) into s.y, complete for the caller after
// a barrier.  DUMP: the activations of image n too.
template <bool DUMP>
__device__ __forceinline__ void group_forward(const float* __restrict__ image, const float* __restrict__ tabg,
                                              float* __restrict__ yhat, GroupForwardLds& s, const DumpPtrs& dump, size_t n) {
  const int t = threadIdx.x, wave = t >> 6, l = t & 63, q = l >> 4, n16 = l & 15;
  const int pp = 12 * ((n16 & 3) >> 1) + 2 * (n16 >> 2) + (n16 & 1);
  // one 16-byte piece per thread of what C1 needs (its operands, the biases, the image), then the other operands
  constexpr int OPS = C1F_KSTEPS * 16, BIAS = TAB_BIAS_FLOATS / 4, FROM = 64 * GWAVES - NI / 4;
  static_assert(OPS + BIAS <= FROM, "one piece per thread");
  const f4* tg = reinterpret_cast<const f4*>(tabg);
  const f4 first = *(t < OPS ? tg + TAB_C1A * 16 + t : t < OPS + BIAS ? tg + TABG_BIAS / 4 + (t - OPS)
                             : t < FROM ? tg : reinterpret_cast<const f4*>(image) + (t - FROM));
  constexpr int PIECES = TAB_FWD_ENTRIES * 16, ROUNDS = (PIECES + 64 * GWAVES - 1) / (64 * GWAVES);
  f4 rest[ROUNDS];
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) rest[r] = tg[t + 64 * GWAVES * r < PIECES ? t + 64 * GWAVES * r : 0];
  const C1Lane ln = c1f_lane();
  if (t < OPS)
    reinterpret_cast<f4*>(s.c1a)[t] = first;
  else if (t < OPS + BIAS)
    reinterpret_cast<f4*>(s.bias)[t - OPS] = first;
  else if (t >= FROM)
    reinterpret_cast<f4*>(s.img)[t - FROM] = first;
  __syncthreads();  // image, C1 operands, biases

  f4 c1[3];
  if (wave < 2)
    group_c1_forward<3>(s.c1a, s.bias, s.img, s.s1, wave, ln, c1);
  else
    group_c1_forward<2>(s.c1a, s.bias, s.img, s.s1, wave, ln, c1);
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r)
    if (t + 64 * GWAVES * r < PIECES) reinterpret_cast<f4*>(s.e)[t + 64 * GWAVES * r] = rest[r];
  if (DUMP && dump.c1 && q < 3) {
#pragma unroll
    for (int k = 0; k < 3; ++k)
      if (wave + 8 * k < C1F_TILES) {
        float* dst = dump.c1 + n * NC1 + ln.c1 + 2 * q * (576 - D1_MAP) + c1f_tile_c1(wave + 8 * k);
        *reinterpret_cast<float2*>(dst) = float2{c1[k][0], c1[k][1]};
        *reinterpret_cast<float2*>(dst + 576) = float2{c1[k][2], c1[k][3]};
      }
  }
  __syncthreads();  // S1, the other operands
  if (DUMP && dump.s1 && t < NS1 / 4) reinterpret_cast<f4*>(dump.s1 + n * NS1)[t] = reinterpret_cast<const f4*>(s.s1)[t];

  const float bias2 = wave < 4 ? s.bias[n16] : 0.0f;
  f4 c2v = f4{bias2, bias2, bias2, bias2};
  const float* s1 = s.s1 + pp + 24 * (wave & 3);
  if (wave < 4) {
    group_c2_steps<0, 19>(s1, s.e + TAB_BF * 64 + l, c2v);
  } else {
    group_c2_steps<19, 19>(s1, s.e + TAB_BF * 64 + l, c2v);
    s.half[t - 256] = c2v;
  }
  __syncthreads();  // the upper waves' sums
  if (wave < 4) {
    const f4 up = s.half[t];
#pragma unroll
    for (int r = 0; r < 4; ++r) c2v[r] = logistic_of_scaled(c2v[r] + up[r]);
    if (n16 < 12) s.s2[n16 * 16 + 4 * wave + q] = 0.25f * ((c2v[0] + c2v[1]) + (c2v[2] + c2v[3]));
    if (DUMP && dump.c2 && n16 < 12) {  // register r: pixel (2 wave + r / 2, 2 q + r % 2)
      float* dst = dump.c2 + n * NC2 + n16 * 64 + 16 * wave + 2 * q;
      *reinterpret_cast<float2*>(dst) = float2{c2v[0], c2v[1]};
      *reinterpret_cast<float2*>(dst + 8) = float2{c2v[2], c2v[3]};
    }
  }
  __syncthreads();  // S2
  if (DUMP && dump.s2 && t < NS2 / 4) reinterpret_cast<f4*>(dump.s2 + n * NS2)[t] = reinterpret_cast<const f4*>(s.s2)[t];
  float sv[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) sv[k] = s.s2[l + 64 * k];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int o = wave + GWAVES * j;  // wave-uniform
    if (o < NY) {
      const float* w = s.e + (TAB_FCW + 3 * o) * 64 + l;
      const float p = fmaf(w[128], sv[2], fmaf(w[64], sv[1], w[0] * sv[0]));
      const float yo = logistic(wave_sum(p) + s.bias[TAB_BIAS_B + o]);
      if (l == 0) {
        s.y[o] = yo;
        if (yhat) yhat[o] = yo;
      }
    }
  }
}

}  // namespace cnn
