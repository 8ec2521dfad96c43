// Convolutions of any shape on the fp32 matrix cores (v_mfma_f32_16x16x4_f32, wave64), tiled over the
// image: a workgroup works on a UNIT = NB whole images, or a band of TH output rows (and, for very wide
// images, a strip of TXC columns) of one image, so nothing has to fit in LDS as a whole.  Definitions:
// arXiv 1912.05234, Section 3 -- listings conv / mconv (forward), backin (input gradient), backweights
// and backbias (weight and bias gradient).
//
// Implicit GEMM in the operand layout, and with the column packing, of cnn_igemm.h.  A fully connected layer is
// the same operation with a kernel as large as its input (Section 3), here H = W = KH = KW = 1.
//
//   forward          M = Cout   K = Cin*KH*KW    N = output pixels
//   input gradient   M = Cin    K = Cout*KH*KW   N = input pixels; the output error is staged with a zero border of
//                    (KH-1, KW-1) and the kernel is read flipped, which turns backin into a forward convolution
//   weight gradient  M = Cout   K = pixels of all images   N = Cin*KH*KW taps
//
// How the work is cut:
//   * the staged operand reaches LDS by direct global-to-LDS loads into two alternating buffers, the
//     next unit's (or the next channel chunk's) loads issued before the current one is multiplied;
//     cells outside the image are written as zeros by the lanes that would load them;
//   * forward form: every wave owns NT column tiles of the unit for MT row tiles at once, so an LDS
//     read of the gathered operand feeds MT instructions and one of the weights NT;
//   * weight gradient: every wave owns ALL tiles of the workgroup (MT x NT accumulators) over its
//     share of the pixels, so the matrix cores are evenly loaded whatever the number of taps; the
//     waves' sums meet in LDS once, at the end.
//
// The gathered operand is addressed as (byte offset of the K index, from a small LDS table) + (byte offset of the
// column), and K is taken in blocks of four steps: dense operand and K offsets of a block are one 16-byte LDS
// read each, the reads of the next block are issued under the matrix instructions of this one.
//
// What bounds it (timed plans, cnn_ops.hip): a block of a column tile costs 144 clocks of its SIMD against the
// 128 of its matrix instructions; around that a unit pays about 500 + 83 NT clocks of staging, addressing and
// stores, and a workgroup one memory round trip (1700 clocks) per unit, the largest share for layers with few
// channels.  500 images 3 -> 16 maps, 32 x 32, 5 x 5: forward 25 us, input gradient 36 us, weight gradient 21.2 + 4.6 us (the
// kernels before, which needed whole images in LDS: 26, 290 and 1540 us); 256 images 16 -> 32, 28 x 28, 3 x 3: 28,
// 35, 33 + 5 us (364, 460, 2020 us).  Without its matrix instructions and operand reads the input gradient of the first
// takes 25 of 46 us, without the weights' way into LDS 33, without staging 40, without stores 45 (before the weights
// were loaded as below).  Small calls are bound by what comes before the first matrix instruction.
#pragma once

#include "cnn_igemm.h"

namespace cnn {
namespace tile {

using igemm::divmod;
using igemm::f2;
using igemm::f4;
using igemm::i4;
using igemm::lds_barrier;
using igemm::mfma16;
using igemm::row_stride;
using igemm::round4;

constexpr int THREADS = 256, WAVES = THREADS / 64;

// Direct loads of this wave have landed (and its earlier stores are done).
__device__ __forceinline__ void wait_loads() { __builtin_amdgcn_s_waitcnt(0x0f70); }  // vmcnt(0)
// ... and everybody's, and all LDS accesses before this point are done.
__device__ __forceinline__ void loads_and_lds_barrier() {
  wait_loads();
  lds_barrier();
}

// Scalar division of n < 2^31 by a fixed d >= 1: the estimate is at most one too small.
struct FastDiv {
  unsigned d, m;
};
inline FastDiv fast_div(long long d) { return FastDiv{(unsigned)d, d <= 1 ? 0xffffffffu : (unsigned)((1ull << 32) / (unsigned long long)d)}; }
__device__ __forceinline__ unsigned divide(unsigned n, FastDiv f, unsigned& rem) {
  unsigned quo = __umulhi(n, f.m);
  rem = n - quo * f.d;
  if (rem >= f.d) ++quo, rem -= f.d;
  return quo;
}

// Buffer accesses check every lane's byte offset against the buffer's size: a load past it (or before
// the base: the offset is unsigned) delivers zero, a store is dropped.  That is how the zeros around
// an image and the ragged ends of units are made, without branches.  FAR marks an offset as outside; two of
// them, or one and any offset inside, still add up to an offset outside, and to one that an int holds.
constexpr int FAR = 0x3ffffffc, FAR_SIZE = 0x3ffffffc;
static_assert(FAR >= FAR_SIZE && FAR <= 0x7fffffff - FAR, "sums of offsets outside stay outside");
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_at(const float* base, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base), 0, bytes, 0x00020000);
}
// Lane i's VB bytes at byte offset `off` (and `at`, the same in every lane) of the buffer to LDS at dst + i VB bytes; dst is
// the same in every lane.
template <int VB>
__device__ __forceinline__ void buffer_to_lds(__amdgpu_buffer_rsrc_t rs, float* dst, unsigned off, int at = 0) {
  static_assert(VB == 16 || VB == 4, "item size");
  __attribute__((address_space(3))) void* to = (__attribute__((address_space(3))) void*)dst;
  if (VB == 16)
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, to, 16, off, at, 0, 0);
  else
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, to, 4, off, at, 0, 0);
}

// Stages runs of consecutive floats: run r of `runs` is `len` floats at src + r * sstride, to LDS floats
// dst + r * dstride.  VB bytes per lane (16: everything a multiple of four floats).  Of a run only the first `valid`
// floats exist (the others are staged as zeros).
template <int VB>
__device__ __forceinline__ void stage_runs(const float* src, float* dst, int runs, int len, size_t sstride,
                                           int dstride, int wave, int l, int valid) {
  constexpr int V = VB / 4, CH = 64 * V;
  const bool spread = runs >= WAVES;  // whole runs to waves, or the pieces of each run
#pragma unroll 1
  for (int r = spread ? wave : 0; r < runs; r += spread ? WAVES : 1) {
    const __amdgpu_buffer_rsrc_t rs = buffer_at(src + r * sstride, 4 * valid);
    float* d = dst + r * dstride;
#pragma unroll 1
    for (int c = (spread ? 0 : wave) * CH; c < len; c += (spread ? 1 : WAVES) * CH)
      if (c + l * V < len) buffer_to_lds<VB>(rs, d + c, 4 * c + VB * l);
  }
}

template <int VB>
__device__ __forceinline__ void stage_runs(const float* src, float* dst, int runs, int len, size_t sstride, int dstride, int wave, int l) {
  stage_runs<VB>(src, dst, runs, len, sstride, dstride, wave, l, len);
}

// ---- forward and input gradient -----------------------------------------------------------------------
struct ConvArgs {
  const float* src;   // [B][SC][SH][SW]
  const float* w;     // [Cout][Cin][KH][KW]
  const float* bias;  // M values or null
  float* dst;         // [B][M][OH][OW]
  int B, M, SC, SH, SW, KH, KW, OH, OW, pady, padx;
  int flip;                // 0: A[m][(c,u,v)] = w[m][c][u][v];  1: A[m][(c,u,v)] = w[c][m][KH-1-u][KW-1-v]
  int P, MR, KWP;          // column packing: pixels per column, rows M*P, shifted taps KW+P-1 
  int NB, TH, TXC;         // a unit: images (1 unless TH covers the image), output rows, columns of P pixels per row
  int groups, bands, strips, units;
  int CC, chunks;          // channels per chunk (one chunk when NB > 1 and the planes have a border)
  int resident;            // the weights of all chunks are in LDS; otherwise every chunk brings its own
  int RH, LW, LP, LI;      // staged rows per plane; LDS strides (floats): row, plane, image
  int K, NBK;              // reduction length of a chunk CC*KH*KWP; blocks of 16
  int SP, SK;              // row strides of the weights and of the K offsets
  int linear;              // planes are staged as runs of memory (no border, full width): 16 or 4 bytes per lane; 0: by rows
  int RPI;                 // rows per staging instruction (by rows)
  int R;                   // rows of A held in LDS: min(16*MT, MR); row R is zero
  float inv_p, inv_khkwp, inv_kwp, inv_cols, inv_txc, inv_lw, inv_khkw, inv_kw, inv_cc;
  FastDiv by_unit, by_strip, by_cc;
};
struct ConvLds {
  int wt, koff, x, buf, total;  // floats; two buffers of `buf` floats at x
};
__host__ __device__ inline ConvLds conv_lds(const ConvArgs& a) {
  ConvLds l;
  l.wt = 0;                                // [R + 1 rows][4: q][SP]: A[row][K index of step s in lane group q] at [s], chunk by chunk when resident
  l.koff = l.wt + (a.R + 1) * 4 * a.SP;    // [4: q][SK] byte offset of that K index
  l.x = l.koff + 4 * a.SK;
  l.buf = round4(a.NB * a.LI + a.P + 4);   // (a padding column may read past the last row)
  l.total = l.x + 2 * l.buf;
  return l;
}

// The order of K inside a block of sixteen: index r of the block is step s of lane group q.  RUN neighbouring indices
// (taps of one kernel row, i.e. neighbouring staged floats) belong to one lane, which reads them as one LDS item.
template <int RUN>
__device__ __forceinline__ void k_place(int r, int& q, int& s) {
  q = RUN == 4 ? r >> 2 : RUN == 2 ? (r >> 1) & 3 : r & 3;
  s = RUN == 4 ? r & 3 : RUN == 2 ? (r >> 3) * 2 + (r & 1) : r >> 2;
}
template <int RUN>
__device__ __forceinline__ int k_index(int q, int s) {
  return RUN == 4 ? 4 * q + s : RUN == 2 ? 8 * (s >> 1) + 2 * q + (s & 1) : 4 * s + q;
}

// Blocks of four K steps, the operands of block i + 1 read under the instructions of block i.
template <int NT, int MT, int RUN>
__device__ __forceinline__ void gemm(f4 (&acc)[MT][NT], const float* wt, const int (&arow)[MT], const i4* koff,
                                     const char* staged, const int (&off)[NT], int nbk) {
  f4 a0[MT], a1[MT];
  float b0[4][NT], b1[4][NT];
  const f4* ap[MT];
#pragma unroll
  for (int m = 0; m < MT; ++m) ap[m] = reinterpret_cast<const f4*>(wt + arow[m]);
  const int last = nbk - 1;
  auto dense = [&](f4 (&a)[MT], int b) {
#pragma unroll
    for (int m = 0; m < MT; ++m) a[m] = ap[m][b];
  };
  auto gather = [&](float (&b)[4][NT], const i4& k) {
#pragma unroll
    for (int s = 0; s < 4; s += RUN)
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        using item = float __attribute__((ext_vector_type(RUN)));
        const item v = *reinterpret_cast<const item*>(staged + k[s] + off[t]);
#pragma unroll
        for (int i = 0; i < RUN; ++i) b[s + i][t] = v[i];
      }
  };
  auto multiply = [&](const f4 (&a)[MT], const float (&b)[4][NT]) {
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int m = 0; m < MT; ++m) acc[m][t] = mfma16(a[m][s], b[s][t], acc[m][t]);
  };
  auto interleave = [&]() {  // one LDS read behind every MT (times RUN) matrix instructions
#pragma unroll
    for (int i = 0; i < 4 * NT / RUN; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, RUN * MT, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x100, MT + 1, 0);
  };
  i4 k0 = koff[0], k1 = koff[min(1, last)];
  dense(a0, 0);
  gather(b0, k0);
  int i = 0;
#pragma unroll 1
  for (; i + 2 < nbk; i += 2) {
    dense(a1, i + 1);
    gather(b1, k1);
    k0 = koff[i + 2];
    multiply(a0, b0);
    interleave();
    dense(a0, i + 2);
    gather(b0, k0);
    k1 = koff[min(i + 3, last)];
    multiply(a1, b1);
    interleave();
  }
  if (i + 2 == nbk) {
    dense(a1, i + 1);
    gather(b1, k1);
    multiply(a0, b0);
    interleave();
    multiply(a1, b1);
  } else {
    multiply(a0, b0);
  }
}

// What a workgroup works on at a time.
struct Unit {
  int b0, y0, x0, nb, th, txp;  // first image, row, column (pixels); images, rows, pixel columns that exist
};
__device__ __forceinline__ Unit unit_at(const ConvArgs& g, unsigned u) {
  unsigned r, strip;
  const unsigned grp = divide(u, g.by_unit, r), band = divide(r, g.by_strip, strip);
  Unit v;
  v.b0 = grp * g.NB;
  v.y0 = band * g.TH;
  v.x0 = strip * g.TXC * g.P;
  v.nb = min(g.NB, g.B - v.b0);
  v.th = min(g.TH, g.OH - v.y0);
  v.txp = min(g.TXC * g.P, g.OW - v.x0);
  return v;
}
// Issues the loads of a unit's channel chunk into the fp32 planes at `buf`.
template <bool BORDER>
__device__ __forceinline__ void stage_unit(const ConvArgs& g, const Unit& u, int chunk, float* buf, int wave, int t) {
  const int plane = g.SH * g.SW;
  const size_t per_image = (size_t)g.SC * plane;
  const int c0 = chunk * g.CC, cc = min(g.CC, g.SC - c0);
  const float* src = g.src + u.b0 * per_image + (size_t)c0 * plane;
  if (!BORDER) {
    const int l = t & 63;
    if (g.bands == 1) {  // whole planes: the channels of an image are one run, and so are all images of the unit if nothing lies between
      const bool one = cc == g.SC && g.LI == g.SC * plane;
      const int runs = one ? 1 : u.nb, len = one ? u.nb * g.LI : cc * plane;
      if (g.linear == 16)
        stage_runs<16>(src, buf, runs, len, per_image, g.LI, wave, l);
      else
        stage_runs<4>(src, buf, runs, len, per_image, g.LI, wave, l);
      return;
    }
    const float* s = src + (size_t)u.y0 * g.SW;
    const int len = min(g.RH, g.SH - u.y0) * g.SW;
    if (g.linear == 16)
      stage_runs<16>(s, buf, cc, len, plane, g.LP, wave, l);
    else
      stage_runs<4>(s, buf, cc, len, plane, g.LP, wave, l);
    return;
  }
  // by rows: RPI rows of LW columns per instruction (or 64 columns of one wide row).  Rows above and
  // below the image fall outside the plane's buffer by themselves, columns beside it are marked.
  const int yb = u.y0 - g.pady, xb = u.x0 - g.padx;
  int l = t & 63;
  asm volatile("" : "+v"(l));  // decoded here, not kept in registers through the main loop
#pragma unroll 1
  for (int cx = 0; cx < g.LW; cx += 64) {
    const int lrr = g.LW <= 64 ? (int)((float)l * g.inv_lw + 1e-4f) : 0, col = g.LW <= 64 ? l - lrr * g.LW : cx + l;
    const bool inside = (unsigned)(xb + col) < (unsigned)g.SW;
    // (bytes as unsigned: rows above and below the image are off by up to three planes of almost FAR_SIZE bytes)
    const unsigned off0 = inside ? 4u * (unsigned)((yb + lrr) * g.SW + xb + col) : FAR, step = inside ? 4u * g.RPI * g.SW : 0;
    if (lrr < g.RPI && col < g.LW) {
#pragma unroll 1
      for (int ic = wave; ic < u.nb * cc; ic += WAVES) {
        unsigned c = ic;
        const unsigned img = u.nb == 1 ? 0 : divide(ic, g.by_cc, c);
        const __amdgpu_buffer_rsrc_t rs = buffer_at(src + img * per_image + (size_t)c * plane, 4 * plane);
        float* d = buf + img * g.LI + c * g.LP + cx;
        unsigned off = off0;
#pragma unroll 1
        for (int r = 0; r < g.RH; r += g.RPI) {
          buffer_to_lds<4>(rs, d, off);
          off += step;
          d += g.RPI * g.LW;
        }
      }
    }
  }
}
// The columns of a wave: tiles wave, wave + 4, ...
template <int NT>
struct Columns {
  int oo[NT], where[NT];  // byte offset in dst (FAR: none); image, row, column inside the unit
};
template <int NT>
__device__ __forceinline__ void columns(const ConvArgs& g, Columns<NT>& c, int wave, int j) {
#pragma unroll
  for (int tt = 0; tt < NT; ++tt) {
    const int n = 16 * (wave + WAVES * tt) + j;
    int img, r, y, xx;
    divmod(n, g.TH * g.TXC, g.inv_cols, img, r);
    divmod(r, g.TXC, g.inv_txc, y, xx);
    const bool have = img < g.NB;
    if (!have) img = y = xx = 0;
    c.oo[tt] = have ? 4 * (img * g.M * g.OH * g.OW + y * g.OW + g.P * xx) : FAR;
    c.where[tt] = (img << 20) | (y << 10) | xx;
  }
}
// The rows of D in a lane's result registers.
template <int MT>
struct Rows {
  int ro[MT][4], shift[4];  // byte offset in dst of result register r (FAR: not a row), its pixel of the column
  f4 binit[MT];             // bias
};
template <int MT>
__device__ __forceinline__ void rows_of(const ConvArgs& g, Rows<MT>& w, int row0, int q) {
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int mrow = row0 + 16 * m + 4 * q + r;
      int ch = mrow, sh = 0;
      if (MT == 1 && g.P > 1) divmod(mrow, g.P, g.inv_p, ch, sh);
      if (m == 0) w.shift[r] = sh;
      w.ro[m][r] = mrow < g.MR ? 4 * (ch * g.OH * g.OW + sh) : FAR;
      w.binit[m][r] = g.bias && mrow < g.MR ? g.bias[ch] : 0.0f;
    }
}
template <int NT, int MT>
__device__ __forceinline__ void store_unit(const ConvArgs& g, const Unit& u, const Columns<NT>& c, const Rows<MT>& w,
                                           const f4 (&acc)[MT][NT]) {
  // how a lane's four result registers of a column lie in memory: one 16-byte item, two of 8 bytes, or single floats
  const int wide = MT > 1 || g.P == 1 ? 1 : (g.P & 3) == 0 && (g.OW & 3) == 0 ? 4 : (g.P & 1) == 0 && (g.OW & 1) == 0 ? 2 : 1;
  const bool ragged_p = MT == 1 && g.OW % g.P != 0;  // the last column of a row has fewer than P pixels
  const __amdgpu_buffer_rsrc_t rs = buffer_at(g.dst + (size_t)u.b0 * g.M * g.OH * g.OW + (size_t)u.y0 * g.OW + u.x0, FAR_SIZE);
  const bool full = u.nb == g.NB && u.th == g.TH && u.txp == g.TXC * g.P;
  int ox[NT], left[NT];
#pragma unroll
  for (int tt = 0; tt < NT; ++tt) {
    left[tt] = u.txp - g.P * (c.where[tt] & 1023);
    ox[tt] = full || ((c.where[tt] >> 20) < u.nb && ((c.where[tt] >> 10) & 1023) < u.th && left[tt] > 0) ? c.oo[tt] : FAR;
  }
  if (wide == 4) {
#pragma unroll
    for (int tt = 0; tt < NT; ++tt) {
      const int off = ragged_p && w.shift[0] >= left[tt] ? FAR : ox[tt] + w.ro[0][0];
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(i4, acc[0][tt]), rs, off, 0, 2);
    }
  } else if (wide == 2) {
#pragma unroll
    for (int r = 0; r < 4; r += 2)
#pragma unroll
      for (int tt = 0; tt < NT; ++tt) {
        using i2 = int __attribute__((ext_vector_type(2)));
        const int off = ragged_p && w.shift[r] >= left[tt] ? FAR : ox[tt] + w.ro[0][r];
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(i2, f2{acc[0][tt][r], acc[0][tt][r + 1]}), rs, off, 0, 0);
      }
  } else {
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int tt = 0; tt < NT; ++tt) {
          const int off = ragged_p && w.shift[r] >= left[tt] ? FAR : ox[tt] + w.ro[m][r];
          __builtin_amdgcn_raw_buffer_store_b32(__float_as_int(acc[m][tt][r]), rs, off, 0, 0);
        }
  }
}

// Waves per SIMD (= workgroups per compute unit) the registers allow; the grid is sized to what is resident.
__host__ __device__ constexpr int conv_residency(int nt, int mt) { return nt * mt <= 4 ? 4 : 3; }

// BORDER: the staged planes have a border (or are strips of a wide image) and are staged by rows.
// RUN: floats of a staged row that a lane reads at once (k_place; KWP, P and the LDS strides are multiples of it): one LDS
// read and one address for RUN matrix instructions.  Kernel times (us, one float at a time -> RUN): input gradient of 500
// images 3 -> 16, 32 x 32, 5 x 5 38.5 -> 35.6 (4); 2585 images 2 -> 10, 22 x 18, 7 x 7 97 -> 94 (2); forward of 1376 images 3 ->
// 3, 28 x 32, 5 x 5 23.6 -> 21.6 (4); the 23 of 120 calls on 60 random shapes that take runs 1.03x.
// ROUND: the reduced-precision form for few channels or little work (cnn_ops.hip): operands are rounded to bfloat16 in LDS,
// their products, exact in fp32, are summed as in the fp32 form.  (As a flag of the launch instead of a kernel of its own it
// cost the small fp32 calls 0.3 us of 5.)
template <int NT, int MT, bool BORDER, int RUN, bool ROUND>
__global__ __launch_bounds__(THREADS, conv_residency(NT, MT)) void conv_kernel(const ConvArgs g) {
  extern __shared__ __align__(16) float lds[];
  const ConvLds L = conv_lds(g);
  float* wt = lds + L.wt;
  int* koff = reinterpret_cast<int*>(lds + L.koff);
  const int t = threadIdx.x, l = t & 63, q = l >> 4, j = l & 15;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int KHKW = g.KH * g.KW, KHKWP = g.KH * g.KWP, row0 = 16 * MT * blockIdx.y;  // first row of A of this workgroup
  auto issue = [&](const Unit& u, int chunk, float* buf) { stage_unit<BORDER>(g, u, chunk, buf, wave, t); };
  // A in LDS: a thread takes a weight's place in the kernels, (channel, tap), of eight maps at a time, all eight loads in
  // flight (the first item's while LDS is cleared and the first unit's loads are issued), and writes each to its P shifted
  // places; the other places are zero from before.  Walking the places of A instead, most of them zeros when packed, eight
  // rows per memory round trip, measured (us, forward / input gradient, then as here): 500 images 3 -> 16, 32 x 32, 5 x 5
  // 25 / 49.5, now 25 / 39; 935 images 2 -> 25, 20 x 11, 5 x 5 12.9 / 50, 11.7 / 35; 115 images 20 -> 4, 31 x 37, 7 x 7
  // 46 / 27, 33 / 27; one image 1 -> 19, 7 x 28, 3 x 3 5.7 / 6.7, 5.0 / 6.4; over 60 random shapes 1.12x / 1.07x.
  const int maps = g.P == 1 ? min(g.R, g.MR - row0) : g.M;  // (packed: one row tile, M * P <= 16)
  const __amdgpu_buffer_rsrc_t ws = buffer_at(g.w, 4 * g.M * g.SC * KHKW);
  struct Item {
    float v[8];
    int m0, kk;
  };
  auto load_item = [&](int chunk, int e, Item& w) {
    const int c0 = chunk * g.CC, cc = g.resident ? g.SC : min(g.CC, g.SC - c0), places = cc * KHKW;
    int grp, r, c, tap, u, x, ck = 0;
    divmod(e, places, 1.0f / (float)places, grp, r);
    divmod(r, KHKW, g.inv_khkw, c, tap);
    divmod(tap, g.KW, g.inv_kw, u, x);
    w.m0 = 8 * grp;
    const int step = (g.flip ? 1 : g.SC) * KHKW, at = g.flip ? ((c0 + c) * g.M + row0) * KHKW + tap : (row0 * g.SC + c0) * KHKW + r;
#pragma unroll
    for (int i = 0; i < 8; ++i)
      w.v[i] = __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(ws, w.m0 + i < maps ? 4 * (at + (w.m0 + i) * step) : FAR, 0, 0));
    if (g.flip) u = g.KH - 1 - u, x = g.KW - 1 - x;
    if (g.resident && g.chunks > 1) {  // chunk ck's blocks lie behind those of the chunks before it
      int rest;
      divmod(c, g.CC, g.inv_cc, ck, rest);
      c = rest;
    }
    w.kk = ck * 16 * g.NBK + c * KHKWP + u * g.KWP + x;
  };
  auto place_item = [&](const Item& w) {
#pragma unroll 1
    for (int sh = 0; sh < g.P; ++sh) {
      const int kk = w.kk + sh;
      int kq, ks;
      k_place<RUN>(kk & 15, kq, ks);
      float* dst = wt + ((w.m0 * g.P + sh) * 4 + kq) * g.SP + 4 * (kk >> 4) + ks;
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if (w.m0 + i < maps) dst[i * g.P * 4 * g.SP] = operand<ROUND>(w.v[i]);
    }
  };
  auto items = [&](int chunk) { return (g.resident ? g.SC : min(g.CC, g.SC - chunk * g.CC)) * KHKW * ((maps + 7) >> 3); };
  // (the next item's loads are in flight while one is written)
  auto weights = [&](int chunk, int e, Item& w) {
    const int n = items(chunk);
#pragma unroll 1
    for (; e < n; e += THREADS) {
      Item next;
      if (e + THREADS < n) load_item(chunk, e + THREADS, next);
      place_item(w);
      w = next;
    }
  };
  auto clear_weights = [&]() {
    for (int e = t; e < (g.R + 1) * g.SP; e += THREADS) reinterpret_cast<f4*>(wt)[e] = f4{0.0f, 0.0f, 0.0f, 0.0f};
  };

  float* const xbuf = lds + L.x;
  Item item;  // in flight while LDS is cleared and the first unit's loads are issued
  if (g.resident && t < items(0)) load_item(0, t, item);
  // every staged cell starts finite: padding K steps and images a ragged unit does not have meet zeros
  for (int e = t; e < 2 * L.buf / 4; e += THREADS) reinterpret_cast<f4*>(xbuf)[e] = f4{0.0f, 0.0f, 0.0f, 0.0f};
  clear_weights();
  lds_barrier();
  unsigned unit = blockIdx.x;
  Unit cur = unit_at(g, unit);
  issue(cur, 0, xbuf);
  for (int e = t; e < 4 * g.SK; e += THREADS) {
    const int qq = e >= 3 * g.SK ? 3 : e >= 2 * g.SK ? 2 : e >= g.SK ? 1 : 0, at = e - qq * g.SK, kk = 16 * (at >> 2) + k_index<RUN>(qq, at & 3);
    int off = 0;
    if (kk < g.K) {
      int c, rem, u, vp;
      divmod(kk, KHKWP, g.inv_khkwp, c, rem);
      divmod(rem, g.KWP, g.inv_kwp, u, vp);
      off = 4 * (c * g.LP + u * g.LW + vp);
    }
    koff[e] = off;
  }
  if (g.resident) weights(0, t, item);

  Columns<NT> col;
  columns(g, col, wave, j);
  int po[NT];  // byte offset of the columns in a buffer
#pragma unroll
  for (int tt = 0; tt < NT; ++tt)
    po[tt] = 4 * ((col.where[tt] >> 20) * g.LI + ((col.where[tt] >> 10) & 1023) * g.LW + g.P * (col.where[tt] & 1023));
  Rows<MT> row;
  rows_of(g, row, row0, q);
  int arow[MT];
#pragma unroll
  for (int m = 0; m < MT; ++m) arow[m] = (min(16 * m + j, g.R) * 4 + q) * g.SP;
  f4 acc[MT][NT];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int tt = 0; tt < NT; ++tt) acc[m][tt] = row.binit[m];
  const i4* kq = reinterpret_cast<const i4*>(koff + q * g.SK);

  int chunk = 0, par = 0;
  wait_loads();
#pragma unroll 1
  while (true) {
    int nchunk = chunk + 1;
    unsigned nunit = unit;
    if (nchunk == g.chunks) nchunk = 0, nunit = unit + gridDim.x;
    const bool more = nunit < (unsigned)g.units;
    lds_barrier();  // this buffer is complete; the other one, and the weights, are no longer read
    if (!g.resident) {
      int e = t;
      asm volatile("" : "+v"(e));  // decoded here, not kept in registers through the main loop
      Item own;
      if (e < items(chunk)) load_item(chunk, e, own);
      if (g.SC - chunk * g.CC < g.CC) {  // fewer channels than the chunk before: what they leave has to be zero
        clear_weights();
        lds_barrier();
      }
      weights(chunk, e, own);
      lds_barrier();
    }
    if (ROUND) {
      f4* x = reinterpret_cast<f4*>(xbuf + par * L.buf);
#pragma unroll 1
      for (int e = t; e < L.buf / 4; e += THREADS) {
        const f4 v = x[e];
        x[e] = f4{round_bf16(v[0]), round_bf16(v[1]), round_bf16(v[2]), round_bf16(v[3])};
      }
      lds_barrier();
    }
    const Unit nxt = nunit == unit || !more ? cur : unit_at(g, nunit);
    if (more) issue(nxt, nchunk, xbuf + (par ^ 1) * L.buf);
    gemm<NT, MT, RUN>(acc, wt + (g.resident ? 4 * g.NBK * chunk : 0), arow, kq, reinterpret_cast<const char*>(xbuf + par * L.buf), po, g.NBK);
    wait_loads();  // before this unit's stores are issued, so that those stay in flight under the next unit's work
    if (nchunk == 0) {
      store_unit(g, cur, col, row, acc);
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int tt = 0; tt < NT; ++tt) acc[m][tt] = row.binit[m];
    }
    if (!more) break;
    cur = nxt, unit = nunit, chunk = nchunk, par ^= 1;
  }
}

// ---- weight and bias gradient --------------------------------------------------------------------------
// T[(co,sh)][tap] = sum over pixel slots (y, X) of d_out[co][y][P X + sh] * in[c][y+u][P X + v'], tap = (c,u,v' < KW+P-1);
// d_k[co][c][u][v] = sum_sh T[(co,sh)][(c,u,v+sh)].  Workgroup (bx, by) sums
// the units bx, bx + gridDim.x, ... for the row tiles MT*mb .. and the tap tiles NT*ntg .. with by = mb * NTG +
// ntg (packed: whole (c,u) groups of KWP taps, as many as fit); it stages only the channels its taps belong to.  K = the unit's pixel slots row by row, padded with
// zeros of d_out to blocks of 16; step s of block b takes, in lane group q, slot 16 b + 4 q + s, so a lane's four
// A values are consecutive floats of a staged row.  Wave w takes the blocks w, w + 4, ...  At the end the
// waves' sums are added in LDS, the P shifts joined, and the workgroup writes its share of ONE row of partial
// sums in the gradient's own order, [bx][d_k ..., d_bias ...], which reduce_rows_kernel adds up (gridDim.x = 1: the
// gradient itself).
struct WgradArgs {
  const float* in;
  const float* d_out;
  float* out_k;          // this workgroup column's sums: a row of partial sums, or (one column) d_k and d_bias themselves
  float* out_b;          // (null: not wanted)
  int B, Cin, H, W, Cout, Ho, Wo, KH, KW;
  int P, MR, KWP, WOP;   // column packing: rows Cout*P, shifted taps KW+P-1, slots per row ceil(Wo/P)
  int K;                 // taps Cin*KH*KWP
  int MT, NT, NTG, TG;   // tiles of the rows and of the taps in all; tap groups and the taps of one
  int RS;                // floats of a row of partial sums, Cout*Cin*KH*KW + Cout: from one workgroup column to the next
  int NB, TH, groups, bands, units;
  int CG;                // most channels a tap group touches
  int RH, LP, LI;        // staged rows; LDS strides (floats) of a plane and an image
  int R;                 // rows of d_out held: min(16*MT of the workgroup, MR); row R is zero
  int N, NBK, NPS;       // slots of a unit, blocks of 16, row stride of the staged d_out
  int vec_x, vec_d;      // bytes per lane of the loads of images and of d_out: 16 or 4
  float inv_khkwp, inv_kwp, inv_slots, inv_wop;
  FastDiv by_band, by_p;
};
struct WgradLds {
  int pb, buf, dy, x, buf_floats, total;
};
__host__ __device__ inline WgradLds wgrad_lds(const WgradArgs& a) {
  WgradLds l;
  l.pb = 0;                     // [4: q][NBK][4] byte offset in x of slot 16 b + 4 q + s
  l.buf = l.pb + 16 * a.NBK;    // two buffers:
  l.dy = 0;                     //   [R + 1][NPS]
  l.x = (a.R + 1) * a.NPS;      //   [NB][LI]
  l.buf_floats = l.x + round4(a.NB * a.LI + a.P);
  l.total = l.buf + 2 * l.buf_floats;
  return l;
}
// LDS at the end of the kernel: the waves' tiles on their way to each other, their row sums, and T.
constexpr int T_STRIDE(int nt) { return 16 * nt + 4; }
constexpr int wgrad_end_floats(int nt, int mt) { return WAVES * WAVES * 256 + WAVES * 16 * mt + 16 * mt * T_STRIDE(nt); }

// The end of a weight-gradient kernel: the waves' accumulators (and row sums of A) are added in LDS in wave order, the
// P shifts joined, and the workgroup's outputs written.  Uses wgrad_end_floats(NT, MT) of LDS from `lds` on.
template <int NT, int MT, typename ARGS>
__device__ __forceinline__ void finish_wgrad(const ARGS& g, const f4 (&acc)[MT][NT], float (&asum)[MT], float* lds, int row0,
                                             int rows, int tap0, int taps, bool sums_bias) {
  const int t = threadIdx.x, l = t & 63, q = l >> 4, j = l & 15;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  // the waves' sums meet in LDS, WAVES tiles at a time: wave w adds tile 4 p + w, in wave order, into T
  float* xch = lds;
  float* bs = xch + WAVES * WAVES * 256;    // [wave][16 MT]
  float* T = bs + WAVES * 16 * MT;          // [16 MT][T_STRIDE]
  constexpr int TS = T_STRIDE(NT);
#pragma unroll
  for (int p = 0; p < (MT * NT + WAVES - 1) / WAVES; ++p) {
    loads_and_lds_barrier();
#pragma unroll
    for (int k = 0; k < WAVES; ++k) {
      const int ti = WAVES * p + k;
      if (ti < MT * NT) {
#pragma unroll
        for (int r = 0; r < 4; ++r) xch[(wave * WAVES + k) * 256 + 64 * r + l] = acc[ti / NT < MT ? ti / NT : 0][ti % NT][r];
      }
    }
    if (p == 0 && sums_bias) {
#pragma unroll
      for (int m = 0; m < MT; ++m) {
        asum[m] += __shfl_xor(asum[m], 16, 64);
        asum[m] += __shfl_xor(asum[m], 32, 64);
        if (q == 0) bs[(wave * MT + m) * 16 + j] = asum[m];
      }
    }
    lds_barrier();
    const int ti = WAVES * p + wave, m = ti / NT, i = ti - m * NT;
    if (m < MT) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float s = 0.0f;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) s += xch[(w * WAVES + wave) * 256 + 64 * r + l];
        T[(16 * m + 4 * q + r) * TS + 16 * i + j] = s;
      }
    }
  }
  lds_barrier();
  // outputs of this workgroup: channels row0 / P .., (c,u) groups tap0 / KWP .., KW taps each
  float* out = g.out_k + (size_t)blockIdx.x * g.RS;
  const int co0 = row0 / g.P, ncu = g.P == 1 ? 1 : taps / g.KWP, per = g.P == 1 ? taps : ncu * g.KW, nco = rows / g.P;
  const int K1 = g.Cin * g.KH * g.KW, first = g.P == 1 ? tap0 : tap0 / g.KWP * g.KW;
  const float inv_per = 1.0f / (float)per, inv_kw = 1.0f / (float)g.KW;
#pragma unroll 1
  for (int e = t; e < nco * per; e += THREADS) {
    int co, k;
    divmod(e, per, inv_per, co, k);
    float s;
    if (g.P == 1) {
      s = T[co * TS + k];
    } else {
      int cu, v;
      divmod(k, g.KW, inv_kw, cu, v);
      const float* tp = T + co * g.P * TS + cu * g.KWP + v;
      s = 0.0f;
#pragma unroll 1
      for (int sh = 0; sh < g.P; ++sh) s += tp[sh * (TS + 1)];
    }
    out[(size_t)(co0 + co) * K1 + first + k] = s;
  }
  if (sums_bias && g.out_b && t < nco) {
    float s = 0.0f;
    for (int sh = 0; sh < g.P; ++sh)
#pragma unroll
      for (int w = 0; w < WAVES; ++w) s += bs[w * MT * 16 + t * g.P + sh];
    g.out_b[(size_t)blockIdx.x * g.RS + co0 + t] = s;
  }
}

// The staged rows of d_out (its base is the first of them in the unit's first image): the first `have` slots exist, the
// others are zeros.  An item of vec_d bytes is of one image: planes are whole items where there are several.
__device__ __forceinline__ void stage_slots(const WgradArgs& g, const float* d, float* buf, int rows, int have, int wave, int l) {
  const int HoWo = g.Ho * g.Wo, V = g.vec_d >> 2, all = 16 * g.NBK;
  const bool by_piece = all > 64 * V * (WAVES - 1);  // waves share out the pieces of a row, or the rows
  const __amdgpu_buffer_rsrc_t rs = buffer_at(d, FAR_SIZE);
#pragma unroll 1
  for (int c = by_piece ? 64 * V * wave : 0; c < all; c += by_piece ? 64 * V * WAVES : 64 * V) {
    const int n = c + V * l;
    int img, r;
    divmod(n, g.TH * g.WOP, g.inv_slots, img, r);
    const int off = n < have ? 4 * (img * g.Cout * HoWo + r) : FAR;
    if (n < all) {
#pragma unroll 1
      for (int row = by_piece ? 0 : wave; row < rows; row += by_piece ? 1 : WAVES) {
        if (V == 4)
          buffer_to_lds<16>(rs, buf + row * g.NPS + c, off, 4 * row * HoWo);
        else
          buffer_to_lds<4>(rs, buf + row * g.NPS + c, off, 4 * row * HoWo);
      }
    }
  }
}

// Waves per SIMD (= workgroups per compute unit) the registers allow, which plans count on: sums, the taps' operands and addresses,
// and with ROUND a block's rounded operands beside those read.  Left unbounded the compiler took up to 28 registers more for two row
// tiles, of eight tap tiles two workgroups were resident instead of three, and plans that asked for three ran a second
// turn: 9770 images 2 -> 23, 8 x 21, 7 x 7 55 us, with the bound 42; 450 images 28 -> 17, 18 x 34, 2 x 2 61 and 43.
__host__ __device__ constexpr int wgrad_residency(int nt, int mt, bool round) {
  const int fit = 512 / (4 * nt * mt + 3 * nt + 60 + (round ? 4 * mt : 0));
  return fit < 4 ? fit : 4;
}

// ROUND: the reduced-precision form for few images (cnn_tile_bf16.h needs eight to fill its operands): operands are
// rounded to bfloat16 as they are read, their products, exact in fp32, are summed as in the fp32 form.
// PACKED: P > 1, a row of d_out is every P-th pixel and is staged float by float.  Otherwise the slots of an image are its
// pixels in order, and come 16 bytes per lane where rows of slots and planes are whole fours (stage_slots).  Kernel times,
// us, float by float -> 16 bytes: 1000 images 1 -> 32, 28 x 28, 3 x 3 47 -> 38; 500 images 3 -> 64, 32 x 32, 3 x 3 68 -> 52;
// 2000 images 4 -> 16, 14 x 14, one tap 22.4 -> 17.6.
template <int NT, int MT, bool ROUND, bool PACKED>
__global__ __launch_bounds__(THREADS, wgrad_residency(NT, MT, ROUND)) void wgrad_kernel(const WgradArgs g) {
  extern __shared__ __align__(16) float lds[];
  const WgradLds L = wgrad_lds(g);
  int* pb = reinterpret_cast<int*>(lds + L.pb);
  const int t = threadIdx.x, l = t & 63, q = l >> 4, j = l & 15;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int KHKWP = g.KH * g.KWP, HoWo = g.Ho * g.Wo, plane = g.H * g.W, SPB = g.TH * g.WOP;
  const int mb = blockIdx.y / g.NTG, ntg = blockIdx.y - mb * g.NTG;
  const int row0 = 16 * MT * mb, rows = min(16 * MT, g.MR - row0);
  const int tap0 = g.TG * ntg, taps = min(g.TG, g.K - tap0);
  int cfirst, clast, rem;
  divmod(tap0, KHKWP, g.inv_khkwp, cfirst, rem);
  divmod(tap0 + taps - 1, KHKWP, g.inv_khkwp, clast, rem);
  cfirst = __builtin_amdgcn_readfirstlane(cfirst), clast = __builtin_amdgcn_readfirstlane(clast);
  const int nc = clast - cfirst + 1;

  for (int e = t; e < 2 * L.buf_floats / 4; e += THREADS) reinterpret_cast<f4*>(lds + L.buf)[e] = f4{0.0f, 0.0f, 0.0f, 0.0f};
  for (int n = t; n < 16 * g.NBK; n += THREADS) {
    int off = 0;
    if (n < g.N) {
      int img, r, y, x;
      divmod(n, SPB, g.inv_slots, img, r);
      divmod(r, g.WOP, g.inv_wop, y, x);
      off = 4 * (img * g.LI + y * g.W + g.P * x);
    }
    pb[((((n >> 2) & 3) * g.NBK + (n >> 4)) << 2) + (n & 3)] = off;
  }
  lds_barrier();

  const int chunks = (16 * g.NBK + 63) >> 6;  // 64-slot pieces of a staged row of d_out
  const bool by_chunk = chunks >= WAVES;      // waves share out the pieces, or the rows
  const bool ragged_p = g.P > 1 && g.Wo % g.P != 0;
  auto issue = [&](unsigned u, float* buf) {
    unsigned band;
    const unsigned grp = divide(u, g.by_band, band);
    const int b0 = grp * g.NB, y0 = band * g.TH, nb = min(g.NB, g.B - b0), th = min(g.TH, g.Ho - y0);
    const float* x = g.in + ((size_t)b0 * g.Cin + cfirst) * plane + (size_t)y0 * g.W;
    const float* d = g.d_out + (size_t)b0 * g.Cout * HoWo + (size_t)y0 * g.Wo;
    const int len = min(g.RH, g.H - y0) * g.W;
    const bool whole = g.bands == 1;  // whole planes: the channels of an image are one run
    const int runs = whole ? nb : nc, rlen = whole ? nc * plane : len, dstride = whole ? g.LI : g.LP;
    const size_t sstride = whole ? (size_t)g.Cin * plane : plane;
    if (g.vec_x == 16)
      stage_runs<16>(x, buf + L.x, runs, rlen, sstride, dstride, wave, l);
    else
      stage_runs<4>(x, buf + L.x, runs, rlen, sstride, dstride, wave, l);
    // d_out: slots that do not exist (and, packed, pixels past the row's end) read as zero
    const int have = g.NB > 1 ? nb * SPB : th * g.WOP;
    if (!PACKED) {
      stage_slots(g, d + (size_t)row0 * HoWo, buf, rows, have, wave, l);
      return;
    }
#pragma unroll 1
    for (int c = by_chunk ? wave : 0; c < chunks; c += by_chunk ? WAVES : 1) {
      const int n = 64 * c + l;
      int img, r, y, xx;
      divmod(n, SPB, g.inv_slots, img, r);
      divmod(r, g.WOP, g.inv_wop, y, xx);
      const int off = n < have ? 4 * (img * g.Cout * HoWo + y * g.Wo + g.P * xx) : FAR, left = g.Wo - g.P * xx;
      if (n < 16 * g.NBK) {
#pragma unroll 1
        for (int row = by_chunk ? 0 : wave; row < rows; row += by_chunk ? 1 : WAVES) {
          unsigned sh;
          const unsigned co = divide(row0 + row, g.by_p, sh);
          const __amdgpu_buffer_rsrc_t rs = buffer_at(d + (size_t)co * HoWo + sh, FAR_SIZE);
          buffer_to_lds<4>(rs, buf + row * g.NPS + 64 * c, ragged_p && (int)sh >= left ? FAR : off);
        }
      }
    }
  };

  int toff[NT];  // byte offset of this lane's tap of each tile (padding taps: the group's first one, never stored)
#pragma unroll
  for (int i = 0; i < NT; ++i) {
    const int tap = tap0 + 16 * i + j;
    int c, r, u, v;
    divmod(16 * i + j < taps ? tap : tap0, KHKWP, g.inv_khkwp, c, r);
    divmod(r, g.KWP, g.inv_kwp, u, v);
    toff[i] = 4 * ((c - cfirst) * g.LP + u * g.W + v);
  }
  f4 acc[MT][NT];
  float asum[MT];
  int arow[MT];
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    asum[m] = 0.0f;
    arow[m] = (16 * m + j < rows ? 16 * m + j : g.R) * g.NPS + 4 * q;
#pragma unroll
    for (int i = 0; i < NT; ++i) acc[m][i] = f4{0.0f, 0.0f, 0.0f, 0.0f};
  }
  const bool sums_bias = ntg == 0;
  const i4* pq = reinterpret_cast<const i4*>(pb) + q * g.NBK;

  int par = 0;
  issue(blockIdx.x, lds + L.buf);
#pragma unroll 1
  for (unsigned u = blockIdx.x; u < (unsigned)g.units; u += gridDim.x, par ^= 1) {
    loads_and_lds_barrier();
    float* buf = lds + L.buf + par * L.buf_floats;
    if (u + gridDim.x < (unsigned)g.units) issue(u + gridDim.x, lds + L.buf + (par ^ 1) * L.buf_floats);
    const char* xb = reinterpret_cast<const char*>(buf + L.x);
    const int last = g.NBK - 1;
    if (wave < g.NBK) {
      // Two blocks a trip; the NT reads of step s + 1 are issued under the instructions of step s, a block's dense operand
      // and slot offsets one block ahead.  Left to itself the compiler puts every read right before its use, and a wave waits
      // for the LDS in every step.  Kernel times, us, with the five tap tiles they now have (before: six and three): 500 images 3 -> 16, 32 x 32,
      // 5 x 5 24.6 -> 21.2; 256 images 16 -> 32, 28 x 28, 3 x 3 38 -> 33.  (Reading two neighbouring slots as one item of eight bytes
      // took 38 and 57: an LDS item that is not aligned to its size is slow.  Taps in another order and planes a few floats further
      // apart, so that no two of a tile share a bank: no gain.)
      i4 k0 = pq[wave], k1;
      f4 a0[MT], a1[MT];
      float b[2][NT];
      auto dense = [&](f4 (&a)[MT], int blk) {
#pragma unroll
        for (int m = 0; m < MT; ++m) a[m] = *reinterpret_cast<const f4*>(buf + arow[m] + 16 * blk);
      };
      auto gather = [&](float (&v)[NT], int at) {
#pragma unroll
        for (int i = 0; i < NT; ++i) v[i] = *reinterpret_cast<const float*>(xb + at + toff[i]);
      };
      auto block = [&](const f4 (&read)[MT], const i4& k, f4 (&an)[MT], i4& kn, int next) {
        f4 a[MT];
#pragma unroll
        for (int m = 0; m < MT; ++m) a[m] = f4{operand<ROUND>(read[m][0]), operand<ROUND>(read[m][1]), operand<ROUND>(read[m][2]), operand<ROUND>(read[m][3])};
        kn = pq[next];
        dense(an, next);
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          gather(b[(s + 1) & 1], s < 3 ? k[s < 3 ? s + 1 : 0] : kn[0]);
#pragma unroll
          for (int i = 0; i < NT; ++i) {
            const float bi = operand<ROUND>(b[s & 1][i]);
#pragma unroll
            for (int m = 0; m < MT; ++m) acc[m][i] = mfma16(a[m][s], bi, acc[m][i]);
          }
        }
        if (sums_bias) {
#pragma unroll
          for (int m = 0; m < MT; ++m) asum[m] += (a[m][0] + a[m][1]) + (a[m][2] + a[m][3]);
        }
        if (!ROUND) {  // (with the rounding in between it is slower: 1083 images 17 -> 5, 13 x 34, 4 x 4 60 -> 70 us)
          __builtin_amdgcn_sched_group_barrier(0x100, 1 + MT, 0);
#pragma unroll
          for (int r = 0; r < 4 * NT; ++r) {  // one LDS read before every MT matrix instructions
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, MT, 0);
          }
        }
      };
      dense(a0, wave);
      gather(b[0], k0[0]);
      int blk = wave;
#pragma unroll 1
      for (; blk + WAVES < g.NBK; blk += 2 * WAVES) {
        block(a0, k0, a1, k1, blk + WAVES);
        block(a1, k1, a0, k0, min(blk + 2 * WAVES, last));
      }
      if (blk < g.NBK) block(a0, k0, a1, k1, last);
    }
  }
  finish_wgrad<NT, MT>(g, acc, asum, lds, row0, rows, tap0, taps, sums_bias);
}

// out[i] = sum over the G rows of part[g][i], i < n: the gradient d_k[0 .. nk) and, if d_bias is not null, d_bias
// behind it.  A workgroup takes COLS columns; its strands walk the rows in ascending order, sixteen loads in flight, and are
// combined by a fixed tree, those of a wave between its lanes.  The walk is bound by load latency, so few columns get many
// strands, and by what comes around it: with 1024 threads and a barrier per level of the tree the three calls of 500 images
// 3 -> 16, 32 x 32, 5 x 5 (512 rows of 1216 floats) took 78.5, now 78.1 us, of 256 images 16 -> 32, 28 x 28, 3 x 3 93.4, now 92.9.
constexpr int REDUCE_THREADS = 512;
template <int COLS>
__global__ __launch_bounds__(REDUCE_THREADS) void reduce_rows_kernel(const float* __restrict__ part, int G, int RS, int nk,
                                                                     float* __restrict__ d_k, float* __restrict__ d_bias) {
  constexpr int STRANDS = REDUCE_THREADS / COLS, HERE = REDUCE_THREADS / 64, DEEP = 16;
  __shared__ float red[HERE][COLS];
  const int t = threadIdx.x, strand = t / COLS, i = blockIdx.x * COLS + t % COLS;
  float sum = 0.0f;
  if (i < RS) {
    const float* p = part + i;
    for (int g = strand; g < G; g += DEEP * STRANDS) {
      float v[DEEP];
#pragma unroll
      for (int k = 0; k < DEEP; ++k) v[k] = g + k * STRANDS < G ? p[(size_t)(g + k * STRANDS) * RS] : 0.0f;
#pragma unroll
      for (int k = 0; k < DEEP; ++k) sum += v[k];
    }
  }
#pragma unroll
  for (int s = COLS; s < 64; s *= 2) sum += __shfl_xor(sum, s);
  if ((t & 63) < COLS) red[t >> 6][t & 63] = sum;
  __syncthreads();
  if (t < COLS && i < RS) {
    float w[HERE];
#pragma unroll
    for (int k = 0; k < HERE; ++k) w[k] = red[k][t];
#pragma unroll
    for (int s = 1; s < HERE; s *= 2)
#pragma unroll
      for (int k = 0; k < HERE; k += 2 * s) w[k] += w[k + s];
    if (i < nk)
      d_k[i] = w[0];
    else if (d_bias)
      d_bias[i - nk] = w[0];
  }
}

}  // namespace tile
}  // namespace cnn
