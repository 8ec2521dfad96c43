// Reduced-precision form of the image-tiled convolutions (cnn_tile.h): operands rounded to bfloat16 (nearest, ties
// to even), products summed in fp32 on v_mfma_f32_16x16x32_bf16.  Tensors in memory stay fp32, NCHW; only the
// arithmetic changes, which is why these are separate entry points with their own tolerance.  (The paper computes
// in `float` throughout, Section 3; this is the reduced-precision matrix-core form of its `conv` / `backin` and of
// `backweights` / `backbias`.)
//
// The instruction takes, per lane, eight consecutive K elements of A's row (lane % 16) and of B's column, K
// elements 8 (lane / 16) .. + 7 of a block of 32.  A lane's eight values of the gathered operand must therefore lie
// together in LDS at every shift (u, v) of the kernel window, which neither the channel planes of an image nor its
// rows do.  So the unit's fp32 data, brought by the direct loads of cnn_tile.h, is turned inside LDS into ITEMS of
// eight bf16 (eight reads of consecutive words, four conversions, one 16-byte write per item):
//   forward, input gradient   item (c / 8, row, column): eight channels of one pixel;  K = (u, v, c), channels padded to eights
//   weight gradient           item (channel, row, column): the same pixel of EIGHT IMAGES;  K = (pixel, image), so that a
//                             shifted window is another item and no shifted copies are needed
// The fp32 buffer is free again once it has been turned, and takes the next unit's loads while the matrix
// instructions run.  LDS traffic bounds these kernels (16 bytes per lane and operand feed an instruction of 16
// clocks), so a wave owns NT column tiles, or all tap tiles, per weight operand it reads.  Measured (forward / input
// gradient / weight gradient, us; in brackets one workgroup per group of whole images, or one thread per element where
// an image did not fit the LDS): 10000 images 6 -> 12 maps, 12 x 12, 5 x 5 taps 21 / 33 / 24.5 + 5 (32, 44, 36), of which a
// copy of the same bytes takes 10.5; 500 images 3 -> 16, 32 x 32, 5 x 5: 17 / 16 / 32 (21, 29, 1840); 256 images 16 -> 32,
// 28 x 28, 3 x 3: 15 / 22 / 45 (24, 870, 2353), the last two weight gradients the fp32 kernel with rounded operands, like forward
// and input gradient where channels are few.
#pragma once

#include "cnn_tile.h"

namespace cnn {
namespace tile16 {

using tile::buffer_at;
using tile::divide;
using tile::divmod;
using tile::f2;
using tile::f4;
using tile::FAR;
using tile::FAR_SIZE;
using tile::FastDiv;
using tile::i4;
using tile::lds_barrier;
using tile::loads_and_lds_barrier;
using tile::round4;
using tile::THREADS;
using tile::wait_loads;
using tile::WAVES;
using bf8 = __bf16 __attribute__((ext_vector_type(8)));

// fp32 -> bf16 bits (nearest, ties to even), two at once: lo in bits 0..15, hi in bits 16..31
__device__ __forceinline__ unsigned pack_bf16(float lo, float hi) {
  using f2v = float __attribute__((ext_vector_type(2)));
  using bf2v = __bf16 __attribute__((ext_vector_type(2)));
  const bf2v r = __builtin_convertvector(f2v{lo, hi}, bf2v);
  return __builtin_bit_cast(unsigned, r);
}

__device__ __forceinline__ f4 mfma32(bf8 a, bf8 b, f4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }
// The item of eight floats `stride` apart; from the count-th on they are zeros, and none at or past `most` is read (the
// same in every lane).
__device__ __forceinline__ void read_item(float (&v)[8], const float* src, int stride, int count, int most) {
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    v[i] = 0.0f;
    if (i < most) {
      v[i] = src[i * stride];
      if (i >= count) v[i] = 0.0f;
    }
  }
}
__device__ __forceinline__ i4 pack_item(const float (&v)[8]) {
  return i4{(int)pack_bf16(v[0], v[1]), (int)pack_bf16(v[2], v[3]), (int)pack_bf16(v[4], v[5]), (int)pack_bf16(v[6], v[7])};
}
// Turns `items` items, two per thread and trip (the reads of both before either is written); `where(e, src, dst, count)`
// says for item e < items where its first float lies, which item it is and how many of its eight values exist.
template <typename WHERE>
__device__ __forceinline__ void turn(int items, int t, i4* out, int stride, int most, WHERE where) {
#pragma unroll 1
  for (int e = t; e < items; e += 2 * THREADS) {
    const float* s0;
    const float* s1;
    int d0, d1, n0, n1;
    float v0[8], v1[8];
    const int e1 = e + THREADS < items ? e + THREADS : e;
    where(e, s0, d0, n0);
    where(e1, s1, d1, n1);
    read_item(v0, s0, stride, n0, most);
    read_item(v1, s1, stride, n1, most);
    out[d0] = pack_item(v0);
    out[d1] = pack_item(v1);
  }
}

// ---- forward and input gradient -----------------------------------------------------------------------
struct ConvArgs {
  // As in the fp32 kernel, with K = KH*KWP*8*C8 of a chunk, NBK blocks of 32, SP and SK unused, LP and LI the fp32 planes
  // as they are staged (rows of SW, no border), LW the pixels of a row of items (with the border).
  tile::ConvArgs t;
  int C8;            // eights of channels of a chunk
  int RS;            // bytes of a weight row, all chunks when resident
  int LPIX;          // items of one channel eight: RH * LW
  // What is turned of a plane: RI rows from item row r0 on, CI columns from item column c0 on; the items around that
  // stay zero from the start.  A band of a bordered image turns all its rows, a strip all its columns: `edges`, cells
  // outside the image are written as zeros.
  int RI, CI, r0, c0, edges;
  float inv_c8, inv_places;  // 1 / C8, 1 / (KH KW eights whose weights are in LDS)
  float inv_plane, inv_ci;  // 1 / (RI CI), 1 / CI
  FastDiv by_c8;
};
struct ConvLds {  // bytes
  int wt, koff, x, item, total;
};
__host__ __device__ inline ConvLds conv_lds(const ConvArgs& a) {
  ConvLds l;
  l.wt = 0;                                  // bf16 [R + 1 rows][RS]
  l.koff = l.wt + (a.t.R + 1) * a.RS;        // int [NBK][4: q] byte offset of K elements 32 b + 8 q ..
  l.x = l.koff + 16 * a.t.NBK;               // fp32 planes [NB][LI]
  l.item = l.x + 4 * round4(a.t.NB * a.t.LI);   // items [NB][C8][LPIX] (a padding column may read past the last row)
  l.total = l.item + 16 * (a.t.NB * a.C8 * a.LPIX + a.t.P + 1);
  return l;
}
// First row of the image that a unit stages, and how many.
__device__ __forceinline__ int first_row(const tile::ConvArgs& g, const tile::Unit& u) { return g.bands == 1 ? 0 : max(0, u.y0 - g.pady); }
// Issues the loads of a unit's channel chunk into the fp32 planes.
__device__ __forceinline__ void stage_planes(const tile::ConvArgs& g, const tile::Unit& u, int chunk, float* buf, int wave, int l) {
  const int plane = g.SH * g.SW, c0 = chunk * g.CC, cc = min(g.CC, g.SC - c0);
  const size_t per_image = (size_t)g.SC * plane;
  const float* src = g.src + u.b0 * per_image + (size_t)c0 * plane;
  int runs, len;
  size_t sstride;
  int dstride;
  if (g.bands == 1) {  // whole planes: the channels of an image are one run, and so are all images of the unit if nothing lies between
    const bool one = cc == g.SC && g.LI == g.SC * plane;
    runs = one ? 1 : u.nb, len = one ? u.nb * g.LI : cc * plane, sstride = per_image, dstride = g.LI;
  } else {
    const int ys = first_row(g, u);
    src += (size_t)ys * g.SW;
    runs = cc, len = (min(g.SH, u.y0 - g.pady + g.RH) - ys) * g.SW, sstride = plane, dstride = g.LP;
  }
  if (g.linear == 16)
    tile::stage_runs<16>(src, buf, runs, len, sstride, dstride, wave, l);
  else
    tile::stage_runs<4>(src, buf, runs, len, sstride, dstride, wave, l);
}

__host__ __device__ constexpr int conv_residency(int nt, int mt) { return nt * mt <= 4 ? 4 : 3; }

// BORDER: the items have a border, or are strips of a wide image; otherwise they lie as the planes do.
template <int NT, int MT, bool BORDER>
__global__ __launch_bounds__(THREADS, conv_residency(NT, MT)) void conv_kernel(const ConvArgs a16) {
  extern __shared__ __align__(16) char smem[];
  const tile::ConvArgs& g = a16.t;
  const ConvLds L = conv_lds(a16);
  int* koff = reinterpret_cast<int*>(smem + L.koff);
  float* const x = reinterpret_cast<float*>(smem + L.x);
  i4* const items = reinterpret_cast<i4*>(smem + L.item);
  const int t = threadIdx.x, l = t & 63, q = l >> 4, j = l & 15;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int KHKW = g.KH * g.KW, OHOW = g.OH * g.OW, C8 = a16.C8;
  const int row0 = 16 * MT * blockIdx.y;
  auto issue = [&](const tile::Unit& u, int chunk) { stage_planes(g, u, chunk, x, wave, l); };
  // A in LDS: a thread takes (tap, eight channels) of two maps at a time, sixteen loads in flight, the first of them while LDS
  // is cleared and the first unit's loads are issued, and writes each eight to its P shifted places; the other places are
  // zero from before (as in the fp32 kernel).  Neighbouring lanes take neighbouring taps, which are neighbours in memory: with
  // the eights of a tap side by side, the order of A, every load met three runs, and forward with seven by seven taps and
  // twenty channels was slower than walking the places of A three rows at a time (115 images, 31 x 37: 23.2 / 27.0 / now 23.2 us;
  // input gradient 35.2 / 37.8 / 34.4).  Against that walk over 60 random shapes 1.06x forward and 1.08x input gradient.  A
  // third map, or a second item in flight, costs registers that the NT = 4 forms spill (5 - 15 % slower forward).
  const int K8 = 4 * g.NBK, maps = g.P == 1 ? min(g.R, g.MR - row0) : g.M;
  const __amdgpu_buffer_rsrc_t ws = buffer_at(g.w, 4 * g.M * g.SC * KHKW);
  const int mstep = 4 * (g.flip ? KHKW : g.SC * KHKW), cstep = 4 * (g.flip ? g.M * KHKW : KHKW);
  const int eights = g.resident ? C8 * g.chunks : C8;  // of all chunks, or of one
  const int n_items = KHKW * eights * ((maps + 1) / 2);
  struct Item {
    float v[2][8];
    int m0, at;  // first map; byte offset of the unshifted place in a weight row
  };
  auto load_item = [&](int chunk, int e, Item& w) {
    int grp, r, tap, c8, u, x0, ck = 0;
    divmod(e, KHKW * eights, a16.inv_places, grp, r);
    divmod(r, KHKW, g.inv_khkw, c8, tap);
    divmod(tap, g.KW, g.inv_kw, u, x0);
    w.m0 = 2 * grp;
    if (g.resident && g.chunks > 1) {
      int rest;
      divmod(c8, C8, a16.inv_c8, ck, rest);
      c8 = rest;
    }
    const int c0 = (chunk + ck) * g.CC, c = c0 + 8 * c8, have = min(8, min(g.SC, c0 + g.CC) - c);  // channels that exist
    const int off = 4 * tap + c * cstep + (row0 + w.m0) * mstep;
#pragma unroll
    for (int n = 0; n < 2; ++n)
#pragma unroll
      for (int i = 0; i < 8; ++i)
        w.v[n][i] = __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(ws, w.m0 + n < maps && i < have ? off + n * mstep + i * cstep : FAR, 0, 0));
    if (g.flip) u = g.KH - 1 - u, x0 = g.KW - 1 - x0;
    w.at = 64 * g.NBK * ck + 16 * ((u * g.KWP + x0) * C8 + c8);
  };
  auto place_item = [&](const Item& w) {
#pragma unroll
    for (int n = 0; n < 2; ++n) {
      if (w.m0 + n < maps) {
        const i4 eight = pack_item(w.v[n]);
        char* dst = smem + L.wt + (w.m0 + n) * g.P * a16.RS + w.at;
#pragma unroll 1
        for (int sh = 0; sh < g.P; ++sh, dst += a16.RS + 16 * C8) *reinterpret_cast<i4*>(dst) = eight;
      }
    }
  };
  // (one item at a time: the registers of a second one would be spilled)
  auto weights = [&](int chunk, int e, Item& w) {
#pragma unroll 1
    while (e < n_items) {
      place_item(w);
      e += THREADS;
      if (e < n_items) load_item(chunk, e, w);
    }
  };

  Item item;
  if (g.resident && t < n_items) load_item(0, t, item);
  for (int e = t; e < (g.R + 1) * a16.RS / 16; e += THREADS) reinterpret_cast<i4*>(smem + L.wt)[e] = i4{0, 0, 0, 0};
  // everything staged starts finite: padding K elements, and images a ragged unit does not have, meet zeros
  for (int e = t; e < (L.total - L.x) / 16; e += THREADS) reinterpret_cast<f4*>(smem + L.x)[e] = f4{0.0f, 0.0f, 0.0f, 0.0f};
  lds_barrier();
  unsigned unit = blockIdx.x;
  tile::Unit cur = tile::unit_at(g, unit);
  issue(cur, 0);
  for (int e = t; e < K8; e += THREADS) {
    int tap, c8, u, vp;
    divmod(e, C8, a16.inv_c8, tap, c8);
    divmod(tap, g.KWP, g.inv_kwp, u, vp);
    koff[e] = u < g.KH ? 16 * (c8 * a16.LPIX + u * g.LW + vp) : 0;
  }
  if (g.resident) weights(0, t, item);

  int po[NT];
  tile::Columns<NT> col;
  tile::columns(g, col, wave, j);
#pragma unroll
  for (int tt = 0; tt < NT; ++tt) {
    const int where = col.where[tt];
    po[tt] = 16 * ((where >> 20) * C8 * a16.LPIX + ((where >> 10) & 1023) * g.LW + g.P * (where & 1023));
  }
  tile::Rows<MT> row;
  tile::rows_of(g, row, row0, q);
  int arow[MT];
#pragma unroll
  for (int m = 0; m < MT; ++m) arow[m] = min(16 * m + j, g.R) * a16.RS + 16 * q;
  f4 acc[MT][NT];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int tt = 0; tt < NT; ++tt) acc[m][tt] = row.binit[m];

  int chunk = 0;
  wait_loads();
#pragma unroll 1
  while (true) {
    int nchunk = chunk + 1;
    unsigned nunit = unit;
    if (nchunk == g.chunks) nchunk = 0, nunit = unit + gridDim.x;
    const bool more = nunit < (unsigned)g.units;
    lds_barrier();  // the fp32 planes are complete, the items and weights no longer read
    if (!g.resident) {
      int e = t;
      asm volatile("" : "+v"(e));  // decoded here, not kept in registers through the main loop
      Item own;
      if (e < n_items) load_item(chunk, e, own);
      weights(chunk, e, own);
    }
    {
      const int cc = min(g.CC, g.SC - chunk * g.CC), per = a16.RI * a16.CI, yb = cur.y0 - g.pady, xb = cur.x0 - g.padx;
      const int ys = first_row(g, cur);
      if (!BORDER) {
        const int most = min(8, cc);
        if (cur.nb * C8 == 1)
          turn(per, t, items, g.LP, most, [&](int e, const float*& src, int& dst, int& count) { src = x + e, dst = e, count = 8; });
        else
          turn(cur.nb * C8 * per, t, items, g.LP, most, [&](int e, const float*& src, int& dst, int& count) {
            int c8, rem, img = 0;
            divmod(e, per, a16.inv_plane, c8, rem);
            if (cur.nb > 1) divmod(c8, C8, a16.inv_c8, img, c8);
            src = x + img * g.LI + 8 * c8 * g.LP + rem, dst = e, count = cc - 8 * c8;
          });
      } else {
        turn(cur.nb * C8 * per, t, items, g.LP, min(8, cc), [&](int e, const float*& src, int& dst, int& count) {
          int c8, rem, ri, ci, img = 0;
          divmod(e, per, a16.inv_plane, c8, rem);
          divmod(rem, a16.CI, a16.inv_ci, ri, ci);
          if (cur.nb > 1) divmod(c8, C8, a16.inv_c8, img, c8);
          const int r = ri + a16.r0, c = ci + a16.c0, y = yb + r, xx = xb + c;
          dst = (img * C8 + c8) * a16.LPIX + r * g.LW + c;
          count = cc - 8 * c8;
          int at = (y - ys) * g.SW + xx;
          if (a16.edges && ((unsigned)y >= (unsigned)g.SH || (unsigned)xx >= (unsigned)g.SW)) count = 0, at = 0;
          src = x + img * g.LI + 8 * c8 * g.LP + at;
        });
      }
    }
    lds_barrier();  // the items are complete, the planes free
    const tile::Unit nxt = nunit == unit || !more ? cur : tile::unit_at(g, nunit);
    if (more) issue(nxt, nchunk);
    {
      const char* wt = smem + L.wt + (g.resident ? 64 * g.NBK * chunk : 0);
      const char* xb = smem + L.item;
      const int* kq = koff + q;
      const int last = g.NBK - 1;
      bf8 a0[MT], a1[MT], b0[NT], b1[NT];
      auto load = [&](bf8 (&a)[MT], bf8 (&b)[NT], int blk, int k) {
#pragma unroll
        for (int m = 0; m < MT; ++m) a[m] = *reinterpret_cast<const bf8*>(wt + arow[m] + 64 * blk);
#pragma unroll
        for (int tt = 0; tt < NT; ++tt) b[tt] = *reinterpret_cast<const bf8*>(xb + po[tt] + k);
      };
      auto multiply = [&](const bf8 (&a)[MT], const bf8 (&b)[NT]) {
#pragma unroll
        for (int tt = 0; tt < NT; ++tt)
#pragma unroll
          for (int m = 0; m < MT; ++m) acc[m][tt] = mfma32(a[m], b[tt], acc[m][tt]);
      };
      // the operands of block b + 1 are read under block b, its offset one block earlier still
      int k1 = kq[4 * min(1, last)], k2;
      load(a0, b0, 0, kq[0]);
      int b = 0;
#pragma unroll 1
      for (; b + 2 < g.NBK; b += 2) {
        k2 = kq[4 * (b + 2)];
        load(a1, b1, b + 1, k1);
        multiply(a0, b0);
        k1 = kq[4 * min(b + 3, last)];
        load(a0, b0, b + 2, k2);
        multiply(a1, b1);
      }
      if (b + 2 == g.NBK) {
        load(a1, b1, b + 1, k1);
        multiply(a0, b0);
        multiply(a1, b1);
      } else {
        multiply(a0, b0);
      }
    }
    wait_loads();  // before this unit's stores are issued, so that those stay in flight under the next unit's work
    if (nchunk == 0) {
      tile::store_unit(g, cur, col, row, acc);
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int tt = 0; tt < NT; ++tt) acc[m][tt] = row.binit[m];
    }
    if (!more) break;
    cur = nxt, unit = nunit, chunk = nchunk;
  }
}

// ---- weight and bias gradient --------------------------------------------------------------------------
// As tile::wgrad_kernel, a unit being EIGHT images (fewer at the end: the others are zeros) and a band of TH output
// rows; K = (pixel slot, image), a block of 32 is four slots; P divides Wo.
struct WgradArgs {
  const float* in;
  const float* d_out;
  float* out_k;          // this workgroup column's sums: a row of partial sums, or (one column) d_k and d_bias themselves
  float* out_b;          // (null: not wanted)
  int B, Cin, H, W, Cout, Ho, Wo, KH, KW;
  int P, MR, KWP, WOP, K;
  int MT, NT, NTG, TG;   // tiles of the rows and of the taps in all; tap groups and the taps of one
  int RS;                // floats of a row of partial sums
  int TH, groups, bands, units;
  int CG, CO;            // most input channels a tap group touches; most output channels of a row block
  int RH, LP, LI;        // rows, and strides (floats, and items) of a staged plane; floats of a staged image
  int DL, DI, DP;        // d_out: floats of a staged plane TH*Wo and image; items of a plane, odd, so that the rows of A start in different banks
  int N, NBK;            // slots of a unit, blocks of four
  int vec_x, vec_d;
  float inv_khkwp, inv_kwp, inv_wop, inv_dl;
  FastDiv by_band;
};
struct WgradLds {  // bytes
  int off, xf, df, xi, di, total;
};
__host__ __device__ inline WgradLds wgrad_lds(const WgradArgs& a) {
  WgradLds l;
  l.off = 0;                              // int2 [4 NBK] byte offsets of a slot: in the items of x, of d_out
  l.xf = l.off + 32 * a.NBK;              // fp32 [8][LI]
  l.df = l.xf + 4 * round4(8 * a.LI);     // fp32 [8][DI]
  l.xi = l.df + 4 * round4(8 * a.DI);     // items [CG][LP] (+ the reach of padding taps)
  l.di = l.xi + 16 * (a.CG * a.LP + a.P);  // items [CO][DP], then one of zeros
  l.total = l.di + 16 * (a.CO * a.DP + 1);
  return l;
}

template <int NT, int MT>
__global__ __launch_bounds__(THREADS) void wgrad_kernel(const WgradArgs g) {
  extern __shared__ __align__(16) char smem[];
  const WgradLds L = wgrad_lds(g);
  int2* slot = reinterpret_cast<int2*>(smem + L.off);
  float* const xf = reinterpret_cast<float*>(smem + L.xf);
  float* const df = reinterpret_cast<float*>(smem + L.df);
  const int t = threadIdx.x, l = t & 63, q = l >> 4, j = l & 15;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int KHKWP = g.KH * g.KWP, HoWo = g.Ho * g.Wo, plane = g.H * g.W;
  const int mb = blockIdx.y / g.NTG, ntg = blockIdx.y - mb * g.NTG;
  const int row0 = 16 * MT * mb, rows = min(16 * MT, g.MR - row0), co0 = row0 / g.P, nco = rows / g.P;
  const int tap0 = g.TG * ntg, taps = min(g.TG, g.K - tap0);
  int cfirst, clast, rem;
  divmod(tap0, KHKWP, g.inv_khkwp, cfirst, rem);
  divmod(tap0 + taps - 1, KHKWP, g.inv_khkwp, clast, rem);
  cfirst = __builtin_amdgcn_readfirstlane(cfirst), clast = __builtin_amdgcn_readfirstlane(clast);
  const int nc = clast - cfirst + 1;

  for (int e = t; e < (L.total - L.xf) / 16; e += THREADS) reinterpret_cast<f4*>(smem + L.xf)[e] = f4{0.0f, 0.0f, 0.0f, 0.0f};
  const int zero_item = 16 * g.CO * g.DP;
  for (int n = t; n < 4 * g.NBK; n += THREADS) {
    int y, xx;
    divmod(n, g.WOP, g.inv_wop, y, xx);
    slot[n] = n < g.N ? int2{16 * (y * g.W + g.P * xx), 16 * (y * g.Wo + g.P * xx)} : int2{0, -1};
  }
  lds_barrier();

  auto issue = [&](unsigned u) {
    unsigned band;
    const unsigned grp = divide(u, g.by_band, band);
    const int b0 = 8 * grp, y0 = band * g.TH, nb = min(8, g.B - b0), th = min(g.TH, g.Ho - y0);
    const float* x = g.in + ((size_t)b0 * g.Cin + cfirst) * plane + (size_t)y0 * g.W;
    const float* d = g.d_out + ((size_t)b0 * g.Cout + co0) * HoWo + (size_t)y0 * g.Wo;
    const int len = min(g.RH, g.H - y0) * g.W;
    if (g.bands == 1) {
      if (g.vec_x == 16)
        tile::stage_runs<16>(x, xf, nb, nc * plane, (size_t)g.Cin * plane, g.LI, wave, l);
      else
        tile::stage_runs<4>(x, xf, nb, nc * plane, (size_t)g.Cin * plane, g.LI, wave, l);
    } else {
#pragma unroll 1
      for (int img = 0; img < nb; ++img) {
        if (g.vec_x == 16)
          tile::stage_runs<16>(x + (size_t)img * g.Cin * plane, xf + img * g.LI, nc, len, plane, g.LP, wave, l);
        else
          tile::stage_runs<4>(x + (size_t)img * g.Cin * plane, xf + img * g.LI, nc, len, plane, g.LP, wave, l);
      }
    }
    // d_out: images and rows that do not exist lie outside the buffer and read as zeros
#pragma unroll 1
    for (int img = 0; img < 8; ++img) {
      const bool have = img < nb;
      const float* di = have ? d + (size_t)img * g.Cout * HoWo : g.d_out;
      const int runs = g.bands == 1 ? 1 : nco, len = g.bands == 1 ? nco * HoWo : g.DL, valid = !have ? 0 : g.bands == 1 ? len : th * g.Wo;
      if (g.vec_d == 16)
        tile::stage_runs<16>(di, df + img * g.DI, runs, len, HoWo, g.DL, wave, l, valid);
      else
        tile::stage_runs<4>(di, df + img * g.DI, runs, len, HoWo, g.DL, wave, l, valid);
    }
  };

  int toff[NT];
#pragma unroll
  for (int i = 0; i < NT; ++i) {
    const int tap = tap0 + 16 * i + j;
    int c, r, u, v;
    divmod(16 * i + j < taps ? tap : tap0, KHKWP, g.inv_khkwp, c, r);
    divmod(r, g.KWP, g.inv_kwp, u, v);
    toff[i] = 16 * ((c - cfirst) * g.LP + u * g.W + v);
  }
  f4 acc[MT][NT];
  float asum[MT];
  int arow[MT];  // byte offset of this lane's row of A in the items of d_out; rows that do not exist read the zero item
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    const int r = 16 * m + j, co = r / g.P;
    arow[m] = r < rows ? 16 * (co * g.DP + r - co * g.P) : -1;
    asum[m] = 0.0f;
#pragma unroll
    for (int i = 0; i < NT; ++i) acc[m][i] = f4{0.0f, 0.0f, 0.0f, 0.0f};
  }
  const bool sums_bias = ntg == 0;
  const char* xi = smem + L.xi;
  const char* di = smem + L.di;

  issue(blockIdx.x);
#pragma unroll 1
  for (unsigned u = blockIdx.x; u < (unsigned)g.units; u += gridDim.x) {
    loads_and_lds_barrier();  // the fp32 data is complete, the items are no longer read
    turn(nc * g.LP, t, reinterpret_cast<i4*>(smem + L.xi), g.LI, 8, [&](int e, const float*& src, int& dst, int& count) { src = xf + e, dst = e, count = 8; });
    turn(nco * g.DL, t, reinterpret_cast<i4*>(smem + L.di), g.DI, 8, [&](int e, const float*& src, int& dst, int& count) {
      int co, r;
      divmod(e, g.DL, g.inv_dl, co, r);
      src = df + e, dst = co * g.DP + r, count = 8;
    });
    lds_barrier();
    if (u + gridDim.x < (unsigned)g.units) issue(u + gridDim.x);
    if (wave < g.NBK) {
      bf8 a0[MT], a1[MT], b0[NT], b1[NT];
      auto load = [&](bf8 (&a)[MT], bf8 (&b)[NT], int2 s) {
#pragma unroll
        for (int m = 0; m < MT; ++m) a[m] = *reinterpret_cast<const bf8*>(di + ((arow[m] | s.y) < 0 ? zero_item : arow[m] + s.y));
#pragma unroll
        for (int i = 0; i < NT; ++i) b[i] = *reinterpret_cast<const bf8*>(xi + toff[i] + s.x);
      };
      auto multiply = [&](const bf8 (&a)[MT], const bf8 (&b)[NT]) {
#pragma unroll
        for (int i = 0; i < NT; ++i)
#pragma unroll
          for (int m = 0; m < MT; ++m) acc[m][i] = mfma32(a[m], b[i], acc[m][i]);
        if (sums_bias) {
#pragma unroll
          for (int m = 0; m < MT; ++m) {
            const i4 bits = __builtin_bit_cast(i4, a[m]);
            float s[4];
#pragma unroll
            for (int h = 0; h < 4; ++h) s[h] = __uint_as_float((unsigned)bits[h] << 16) + __uint_as_float((unsigned)bits[h] & 0xffff0000u);
            asum[m] += (s[0] + s[1]) + (s[2] + s[3]);
          }
        }
      };
      const int last = g.NBK - 1;
      load(a0, b0, slot[4 * wave + q]);
      int2 s1 = slot[4 * min(wave + WAVES, last) + q];
      int blk = wave;
#pragma unroll 1
      for (; blk + 2 * WAVES < g.NBK; blk += 2 * WAVES) {
        const int2 s2 = slot[4 * (blk + 2 * WAVES) + q];
        load(a1, b1, s1);
        multiply(a0, b0);
        s1 = slot[4 * min(blk + 3 * WAVES, last) + q];
        load(a0, b0, s2);
        multiply(a1, b1);
      }
      if (blk + WAVES < g.NBK) {
        load(a1, b1, s1);
        multiply(a0, b0);
        multiply(a1, b1);
      } else {
        multiply(a0, b0);
      }
    }
  }
  tile::finish_wgrad<NT, MT>(g, acc, asum, reinterpret_cast<float*>(smem), row0, rows, tap0, taps, sums_bias);
}

}  // namespace tile16
}  // namespace cnn
