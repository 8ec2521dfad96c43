// Kernels of the fused step, the deterministic gradient reduction with the SGD
// update, and the context-based C entry points.  Definitions: arXiv 1912.05234,
// Section 3 (forward, conv, mconv, sigmoid, avgpool, backweights, backbias,
// backin, backavgpool) and Section 2 (batch gradient descent,
// w := w - eta * sum_i grad F_i).
//
// Large batches: one wavefront owns one image at a time (cnn_train.h, cnn_split.h; of 513 to 1024 images
// two waves own one): the pixels, every activation and every error array stay in LDS and registers; the
// only HBM traffic per image is its 3136-byte pixel block and its label.  Each wave
// keeps its 3898 gradient sums in registers, so no atomics touch memory shared between
// waves and a partial's value does not depend on scheduling.  A second kernel
// adds the partials in a fixed order and applies the update.  Small batches: eight or sixteen
// waves share an image (cnn_group.h).
#include <new>
#include <vector>

#include "cnn_wave.h"
#include "cnn_group.h"
#include "cnn_split.h"
#include "cnn_train.h"

namespace {

using namespace cnn;

constexpr int TRAIN_BLOCKS = 256;  // most workgroups (= gradient partials) of the large-batch training kernel: one per compute unit
// Batches up to this size give each image to a workgroup of eight waves (lower latency per image;
// up to two such workgroups share a compute unit); larger ones give each image to two waves (train_kernel<true>, more images in
// flight).  Gradient of 257 / 384 / 512 / 513 / 576 / 640 images, us: 16.1 / 18.4 / 19.6 / 23.1 / 26.1 / 26.6 with eight waves
// per image (from 513 on a third workgroup has to wait), 21.3 / 21.2 / 21.2 / 21.3 / 21.4 / 21.4 with two.
constexpr int GROUP_MAX_BATCH = 512;
// Up to this size there are two compute units per image, and two workgroups share it.  Step with one workgroup / two, us: 64
// images 11.6 / 10.5, 128 12.1 / 11.0, 129 12.3 / 13.2, 256 13.6 / 15.0, 512 20.7 / 25.8.  Gradient with nothing in the caches:
// 16 images 13.6 / 12.4, 64 13.9 / 12.8, 128 14.6 / 13.6.
constexpr int GROUP_PAIR_MAX_BATCH = 128;
// Beyond GROUP_MAX_BATCH and up to this size there is a SIMD for every image, and two waves of it share one (train_kernel<true>).
constexpr int WAVE_PAIR_MAX_BATCH = 4 * TRAIN_BLOCKS;
// The same choice for the forward pass alone: evaluation of 512 / 768 / 896 / 1024 / 1025 / 1280 images 10.0 / 11.1 / 13.1 / 13.1 /
// 14.6 / 15.3 us with eight waves per image, 12.7 to 13.2 for any number up to 2048 with one (896 and 1024: 12.8, which is 0.3
// less; the line is from before both of them added their pairs in one small workgroup).
constexpr int FWD_GROUP_MAX_BATCH = 1024;
// Device-side epoch loop: one barrier flag per workgroup (a batch of at most EPOCH_MAX_BATCH images:
// thread t of a 512-thread workgroup polls flag t), one flag nobody sets, the error word.
constexpr int EPOCH_MAX_BATCH = 256;
constexpr int SYNC_PHANTOM = EPOCH_MAX_BATCH, SYNC_ERROR = EPOCH_MAX_BATCH + 1, SYNC_WORDS = EPOCH_MAX_BATCH + 2;

// Adds one image's prediction (right: 1) and half its squared error to the two sums.
__device__ __forceinline__ void judge(const float (&y)[10], int label, float& n_ok, float& loss) {
  int best = 0;
  float bestv = y[0], lsum = 0.0f;
#pragma unroll
  for (int o = 0; o < NY; ++o) {
    if (o > 0 && y[o] > bestv) {  // strict '>' keeps the lowest index on ties
      bestv = y[o];
      best = o;
    }
    const float e = y[o] - (o == label ? 1.0f : 0.0f);
    lsum = fmaf(e, e, lsum);
  }
  n_ok += (best == label) ? 1.0f : 0.0f;
  loss = fmaf(0.5f, lsum, loss);
}

// The same for a wave that holds the outputs one per lane (out_of_lane); the sums are the same in every lane.
__device__ __forceinline__ void judge_lanes(float y, bool out_lane, int label, float& n_ok, float& loss) {
  const int l = threadIdx.x & 63;
  const float e = out_lane ? y - (out_of_lane(l) == label ? 1.0f : 0.0f) : 0.0f;
  float sq = e * e, top = out_lane ? y : 0.0f;  // (every output is at least 0)
  sq += quad_xor1(sq);
  sq += quad_xor2(sq);
  top = fmaxf(top, quad_xor1(top));
  top = fmaxf(top, quad_xor2(top));
  auto from = [](float v, int lane) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane));
  };
  top = fmaxf(fmaxf(from(top, 0), from(top, 16)), from(top, 32));
  // the lowest lane is the lowest index; a first output that is NaN stays the answer, as in `judge`
  const unsigned long long best = __ballot(out_lane && (y == top || (l == 0 && y != y)));
  n_ok += best != 0 && __builtin_ctzll(best) == 16 * (label >> 2) + (label & 3) ? 1.0f : 0.0f;
  loss = fmaf(0.5f, (from(sq, 0) + from(sq, 16)) + from(sq, 32), loss);
}

// Forward-only: yhat[B,10], optional activation dump, optional (count, loss) per workgroup.  One wave per image, FWAVES
// waves per workgroup (they share the operands), one workgroup per compute unit; wave w of workgroup b takes the images
// b + blocks * (w + FWAVES k).
// What bounds it: a SIMD's issue.  264 matrix instructions at 6 ns (7.6 alone; a vector instruction hides under half of
// one), about 560 vector instructions at 1.25 and 140 exponentials and reciprocals at 3.45 are 2.8 us of the 3.8 us that
// an image takes a SIMD with two waves; three waves (with fewer registers each) take the same.  In fp32 (152 matrix, 2134
// vector instructions) it was 6.3 us: evaluation of 10000 images 68 -> 42.2 us, of 60000 373 -> 214 us.
constexpr int FWAVES = 8;
struct __align__(16) SplitForwardLds {  // of one wave
  unsigned img[3 * SPLIT_IMG_PLANE];
  unsigned s1[SPLIT_S1_WORDS];
  float s2[S2_WORDS];
};
template <bool DUMP>
__global__ __launch_bounds__(64 * FWAVES) void forward_kernel(const float* __restrict__ images,
                                                             const int32_t* __restrict__ labels, int B,
                                                             const float* __restrict__ w, const float* __restrict__ tabg,
                                                             float* __restrict__ yhat, DumpPtrs dump,
                                                             float* __restrict__ eval_partial) {
  __shared__ u4v items[SPLIT_ITEMS];
  __shared__ __align__(16) float fc[30 * 64];
  __shared__ SplitForwardLds lds[FWAVES];
  const int t = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(t >> 6), l = t & 63, q = l >> 4, n16 = l & 15;
  SplitForwardLds& s = lds[wave];
  const size_t first = (size_t)blockIdx.x + (size_t)gridDim.x * wave, step = (size_t)gridDim.x * FWAVES;
  Pixels px = load_pixels(images + (first < (size_t)B ? first : 0) * NI);  // in flight during the set-up
  SplitLoad<64 * FWAVES, false> weights;
  weights.fetch(w);
  for (int i = t; i < 30 * 16; i += 64 * FWAVES)
    reinterpret_cast<f4*>(fc)[i] = reinterpret_cast<const f4*>(tabg + TAB_FCW * 64)[i];
  // read by the last items, meets zero weights
  if (l < 4) s.s1[3 * SPLIT_S1_PLANE + l] = s.s1[SPLIT_S1B + 3 * SPLIT_S1_PLANE + l] = 0;
  const float* bias = tabg + TABG_BIAS;
  const float bias2 = bias[n16];
  f4 bias1a, bias1b = f4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int i = 0; i < 4; ++i) bias1a[i] = NEG_LOG2E * bias[TAB_BIAS_B1 + i];
#pragma unroll
  for (int i = 0; i < 2; ++i) bias1b[i] = NEG_LOG2E * bias[TAB_BIAS_B1 + 4 + i];
  const float bias3 = bias[TAB_BIAS_B + out_of_lane(l)];
  const bool out_lane = (OUT_LANES >> l) & 1;
  weights.commit(reinterpret_cast<float*>(lds), items);
  __syncthreads();  // the operands are complete; from here on the waves go their own ways
  C1SWeights w1;
  c1s_load_weights(w1, items, l);
  const C1SLane ln = c1s_lane(s.img, l);
  const int es = c1s_lane_s1(l), eh = es + 4 - 2 * (n16 & 1);
  const C2SLane ln2 = c2s_lane(s.s1, items, l);
  unsigned short* s1 = reinterpret_cast<unsigned short*>(s.s1);
  float n_ok = 0.0f, loss = 0.0f;
  for (size_t n = first; n < (size_t)B; n += step) {
    split_store_pixels(s.img, l, px.a);
    split_store_pixels(s.img, l + 64, px.b);
    split_store_pixels(s.img, l + 128, px.c);
    if (l < 4) split_store_pixels(s.img, l + 192, px.d);
    wave_sync();
    if (n + step < (size_t)B) px = load_pixels(images + (n + step) * NI);
    // C1 and S1, column tiles in pairs (the last alone)
    C1SItems it[2];
    c1s_load(it[0], ln, 0);
#pragma unroll
    for (int T = 0; T < 9; T += 2) {
      float low[2], high[2] = {0.0f, 0.0f};
      const int count = T < 8 ? 2 : 1;
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        if (k >= count) continue;
        if (T + k < 8) c1s_load(it[(k + 1) & 1], ln, T + k + 1);
        f4 d0 = bias1a, d1 = bias1b;
        c1s_gemm(w1, it[k], d0, d1);
        float c[6];
#pragma unroll
        for (int i = 0; i < 6; ++i) c[i] = logistic_of_scaled(i < 4 ? d0[i & 3] : d1[i & 3]);
        if (DUMP && dump.c1) {
          const int y = 8 * ((T + k) / 3) + (n16 & 7), x = 8 * ((T + k) % 3) + 4 * (n16 >> 3) + q;
#pragma unroll
          for (int i = 0; i < 6; ++i) dump.c1[n * NC1 + i * 576 + y * 24 + x] = c[i];
        }
        c1s_pool(c, low[k], high[k]);
      }
      const float both = c1s_pool_rows(high[0], count == 2 ? high[1] : high[0]);
      if (count == 2) {
        split_store_s1<true>(s1, es + c1s_tile_s1(T), low[0], es + c1s_tile_s1(T + 1), low[1]);
        const int e = eh + ((n16 & 1) ? c1s_tile_s1(T + 1) : c1s_tile_s1(T));
        split_store_s1_one<true>(s1, e, both);
      } else {
        split_store_s1<true>(s1, es + c1s_tile_s1(T), low[0], eh + c1s_tile_s1(T), both);
      }
    }
    wave_sync();
    if (DUMP && dump.s1)
      for (int e = l; e < NS1; e += 64) dump.s1[n * NS1 + e] = split_s1_value(s1, e);
    // C2 and S2
    f4 c2[4];
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) c2[mt] = f4{bias2, bias2, bias2, bias2};
    c2s_gemm<0, 4>(c2, ln2);
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
#pragma unroll
      for (int r = 0; r < 4; ++r) c2[mt][r] = logistic_of_scaled(c2[mt][r]);
      if (n16 < 12) s.s2[n16 * S2_MAP + 4 * mt + q] = 0.25f * ((c2[mt][0] + c2[mt][1]) + (c2[mt][2] + c2[mt][3]));
      if (DUMP && dump.c2 && n16 < 12)
#pragma unroll
        for (int r = 0; r < 4; ++r) dump.c2[n * NC2 + n16 * 64 + (2 * mt + (r >> 1)) * 8 + 2 * q + (r & 1)] = c2[mt][r];
    }
    wave_sync();
    if (DUMP && dump.s2)
      for (int e = l; e < NS2; e += 64) dump.s2[n * NS2 + e] = s.s2[s2_at(e)];
    // output layer: the lane owns the inputs lane, lane + 64, lane + 128
    float sv[3], p[NY];
#pragma unroll
    for (int k = 0; k < 3; ++k) sv[k] = s.s2[s2_at(l + 64 * k)];
#pragma unroll
    for (int o = 0; o < NY; ++o) {
      const float* f = fc + 3 * o * 64 + l;
      p[o] = fmaf(f[128], sv[2], fmaf(f[64], sv[1], f[0] * sv[0]));
    }
    const float y = logistic(wave_sum10(p) + bias3);
    if (yhat && out_lane) yhat[n * NY + out_of_lane(l)] = y;
    if (labels) judge_lanes(y, out_lane, labels[n], n_ok, loss);
    wave_sync();
  }
  if (!eval_partial) return;
  __shared__ float2 sums[FWAVES];
  if (l == 0) sums[wave] = float2{n_ok, loss};  // (exact: far fewer than 2^24 images per workgroup)
  __syncthreads();
  if (t == 0) {
    float2 all = sums[0];
#pragma unroll
    for (int k = 1; k < FWAVES; ++k) all.x += sums[k].x, all.y += sums[k].y;
    reinterpret_cast<float2*>(eval_partial)[blockIdx.x] = all;
  }
}

// The same for few images: eight waves share one (cnn_group.h), one workgroup per image.
template <bool DUMP>
__global__ __launch_bounds__(64 * GWAVES) void forward_group_kernel(const float* __restrict__ images,
                                                                const int32_t* __restrict__ labels,
                                                                const float* __restrict__ tabg, float* __restrict__ yhat,
                                                                DumpPtrs dump, float* __restrict__ eval_partial) {
  __shared__ GroupForwardLds s;
  const size_t n = blockIdx.x;
  group_forward<DUMP>(images + n * NI, tabg, yhat ? yhat + n * NY : nullptr, s, dump, n);
  if (!eval_partial) return;
  __syncthreads();
  if (threadIdx.x == 0) {
    float y[10], n_ok = 0.0f, loss = 0.0f;
#pragma unroll
    for (int o = 0; o < NY; ++o) y[o] = s.y[o];
    judge(y, labels[n], n_ok, loss);
    eval_partial[2 * n] = n_ok;
    eval_partial[2 * n + 1] = loss;
  }
}

// Sums the G (count, loss) pairs, one per workgroup of the forward kernel: strand t takes the pairs t, t + 256, .. (at most four,
// one memory round trip), then a fixed tree over a wave's lanes and the waves in order.  The counts are whole numbers (each far
// below 2^24, so exact in its float; together no more than the images, which an int counts).  It is bound by the launch and a round trip.
// Evaluation of 1025 / 2048 / 10000 images, us: 13.4 / 14.1 / 42.0 with sixteen waves, a barrier per level of the tree and a pair per
// wave, 13.0 / 13.3 / 41.2 with this.
constexpr int EVAL_REDUCE_THREADS = 256;
__global__ __launch_bounds__(EVAL_REDUCE_THREADS) void eval_reduce_kernel(const float* __restrict__ eval_partial,
                                                                          int G, int64_t* __restrict__ n_correct,
                                                                          float* __restrict__ loss_sum) {
  constexpr int ROUNDS = FWD_GROUP_MAX_BATCH / EVAL_REDUCE_THREADS, WAVES = EVAL_REDUCE_THREADS / 64;
  __shared__ int counts[WAVES];
  __shared__ float losses[WAVES];
  const int t = threadIdx.x;
  float2 pair[ROUNDS];
#pragma unroll
  for (int k = 0; k < ROUNDS; ++k) {
    const int g = t + EVAL_REDUCE_THREADS * k;
    pair[k] = g < G ? reinterpret_cast<const float2*>(eval_partial)[g] : float2{0.0f, 0.0f};
  }
  int ok = 0;
  float loss = 0.0f;
#pragma unroll
  for (int k = 0; k < ROUNDS; ++k) ok += (int)pair[k].x, loss += pair[k].y;
#pragma unroll
  for (int step = 1; step < 64; step *= 2) {
    ok += __shfl_xor(ok, step);
    loss += __shfl_xor(loss, step);
  }
  if ((t & 63) == 0) counts[t >> 6] = ok, losses[t >> 6] = loss;
  __syncthreads();
  if (t == 0) {
    if (n_correct) *n_correct = (int64_t)counts[0] + counts[1] + counts[2] + counts[3];
    if (loss_sum) *loss_sum = (losses[0] + losses[1]) + (losses[2] + losses[3]);
  }
}

// Forward + backward over each wave's images: eight waves per workgroup, one workgroup per compute
// unit, i.e. two waves per SIMD.  (One wave alone issues a vector instruction every 2.4 ns, two
// together one every 1.4 ns, and the matrix instructions of one run under the LDS waits of the
// other; the price is 256 registers and 15.25 KB of LDS per wave.)  Workgroup b owns the images
// b + gridDim.x * k, k < K; WaveShare says which of them each wave takes.  The eight waves then add
// their gradient sums through LDS in a fixed order and the workgroup writes ONE partial row,
// partial[blockIdx.x][PSTRIDE], with 16-byte stores (a wave without images contributes zeros).
constexpr int TWAVES = 8;
// Which of a workgroup's K images each wave takes.  The images are dealt in rounds: a full round
// gives one image to each of the eight waves, a half round one to each of waves 0..3 only; the
// pattern of SHARE_ROUNDS rounds repeats every SHARE_PERIOD images.  A function of K and the wave
// alone, so the grouping of the gradient sums (and with it every rounding) is the same in every run.
// Why not full rounds only: the two waves of a SIMD do not advance at the same rate.  The one in
// the lower slot wins the issue arbitration more often, in every workgroup alike, so an equal split leaves
// the SIMD to one wave for the last part of the kernel.  Where the last rounds are not full ones, the longest wave decides.
// Gradient of so many images, us, an equal split / 4 images to 3 (F F H F) / 3 to 2:
//   2048 and 3072, the same       32 / 32 / 32 and 41 / 41 / 41
//   3073 .. 4096 (13 .. 16 each)  48.5 .. 51.4 / 48.8 .. 51.7 / 51.1 .. 53.9: three to two gives the lower waves a third image
//   4608, 5120, 6144              57.5, 59.2, 72.4 / 57.9, 59.6, 72.3 / 57.3, 59.3, 71.3
//   8448, 9216 (33, 36 each)      97.0, 100.1 / 98.4, 101.1 / 99.4, 103.0
//   10000, 12000                  113, 136 / 110, 131 / 109, 132
//   20000, 60000                  222, 588 / 213, 577 / 211, 575
// One pattern for all sizes, the best of the three from 10000 images on.
// A batch that does not fill the machine (K < 8) still leaves waves 4..7 idle rather than two
// waves on one SIMD and none on another: the first round is a full one.
constexpr unsigned SHARE_PATTERN = 0x5;  // rounds F H F (first round in bit 0): 3 images to 2
constexpr int SHARE_ROUNDS = 3;
constexpr bool share_full(int r) { return (SHARE_PATTERN >> r) & 1; }
constexpr int share_start(int r) {  // first image of round r inside a period
  int at = 0;
  for (int i = 0; i < r; ++i) at += share_full(i) ? 8 : 4;
  return at;
}
constexpr int SHARE_PERIOD = share_start(SHARE_ROUNDS);
constexpr int share_full_rounds() {
  int n = 0;
  for (int r = 0; r < SHARE_ROUNDS; ++r) n += share_full(r);
  return n;
}
constexpr int SHARE_FULL = share_full_rounds();
static_assert(share_full(0), "the first round deals to all eight waves");
struct ShareSlots {  // start of the j-th round that deals to waves 0..3 (every round) / to waves 4..7 (full rounds)
  int low[SHARE_ROUNDS], high[SHARE_ROUNDS];
  constexpr ShareSlots() : low(), high() {
    int nh = 0;
    for (int r = 0; r < SHARE_ROUNDS; ++r) {
      low[r] = share_start(r);
      if (share_full(r)) high[nh++] = share_start(r);
    }
    for (; nh < SHARE_ROUNDS; ++nh) high[nh] = SHARE_PERIOD;  // never reached
  }
};
__device__ constexpr ShareSlots SHARE_SLOTS = ShareSlots();
// How many of K images wave w takes.
__device__ __forceinline__ int share_count(int K, int w) {
  const int per = w < 4 ? SHARE_ROUNDS : SHARE_FULL, rest = K % SHARE_PERIOD;
  int n = per * (K / SHARE_PERIOD);
#pragma unroll
  for (int j = 0; j < SHARE_ROUNDS; ++j)
    if (j < per && (w < 4 ? SHARE_SLOTS.low[j] : SHARE_SLOTS.high[j]) + w < rest) ++n;
  return n;
}
// Walks wave w's images: k() is the current one, left how many remain including it.
struct WaveShare {
  int base, j, per, left, w;
  __device__ __forceinline__ WaveShare(int K, int wave) : base(0), j(0), per(wave < 4 ? SHARE_ROUNDS : SHARE_FULL), left(share_count(K, wave)), w(wave) {}
  __device__ __forceinline__ int k() const { return base + (w < 4 ? SHARE_SLOTS.low[j] : SHARE_SLOTS.high[j]) + w; }
  __device__ __forceinline__ void advance() {
    --left;
    if (++j == per) {
      j = 0;
      base += SHARE_PERIOD;
    }
  }
};
// PAIR: at most four images per workgroup, one for each SIMD; waves w and w + 4 share image w (cnn_train.h).  All waves pass all
// barriers: a pair without an image goes through the first one's and drops what it finds.
template <bool PAIR>
__global__ __launch_bounds__(64 * TWAVES) __attribute__((amdgpu_waves_per_eu(2, 2))) void train_kernel(
    const float* __restrict__ images, const int32_t* __restrict__ labels, int B, const float* __restrict__ w,
    const float* __restrict__ tabg, float* __restrict__ partial, float* fc_hist) {
  __shared__ TrainOperands ops;
  __shared__ WaveTrainLds lds[TWAVES];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // in a scalar register: addresses built on it are wave-uniform
  WaveTrainLds& s = lds[wave];
  WaveState st;
  const int K = B > (int)blockIdx.x ? (B - (int)blockIdx.x + (int)gridDim.x - 1) / (int)gridDim.x : 0;
  WaveShare mine(K, wave);
  const bool has_images = PAIR ? (wave & 3) < K : mine.left > 0;
  const float sign = wave & 1 ? -1.0f : 1.0f;  // see wave_image
  auto image_index = [&](int k) { return (size_t)blockIdx.x + (size_t)gridDim.x * (size_t)k; };
  // every load of the set-up is issued before anything waits for one
  const size_t first = has_images ? image_index(PAIR ? wave & 3 : mine.k()) : PAIR ? image_index(0) : 0;
  const Pixels px = load_pixels(images + first * NI);
  SplitLoad<64 * TWAVES, true> weights;
  weights.fetch(w);
  constexpr int FC_PIECES = 30 * 16;
  static_assert(FC_PIECES <= 64 * TWAVES, "one piece per thread");
  const int t = threadIdx.x;
  const f4 fc = reinterpret_cast<const f4*>(tabg)[TAB_FCW * 16 + (t < FC_PIECES ? t : 0)];
  const float bias = tabg[TABG_BIAS + (t < TAB_BIAS_FLOATS ? t : 0)];
  // waves without images skip their set-up and their row
  if (PAIR || has_images) wave_init(st);
  if (t < C1G_ONES) ops.ones[t] = 1.0f;
  if (t < FC_PIECES) reinterpret_cast<f4*>(ops.fc)[t] = fc;
  if (t < TAB_BIAS_FLOATS) ops.bias[t] = bias;
  weights.commit(lds[0].pool, ops.items, ops.bwd);
  __syncthreads();  // the operands are complete
  float fc_grad[NY][3];  // (PAIR)
  if constexpr (PAIR) {
    WaveTrainLds& area = lds[wave & 3];
    if (wave < 4)
      place_image<FIRST>(area, px);
    else
      place_image<SECOND>(area, px);
    __syncthreads();
    st.bias2 = ops.bias[threadIdx.x & 15];
    if (wave < 4)
      wave_image<FIRST>(st, area, s, ops, images, labels[first], sign, nullptr, fc_grad);
    else
      wave_image<SECOND>(st, area, s, ops, images, labels[first], sign, nullptr, fc_grad);
  } else {
    if (has_images) place_image<LONE>(s, px);
    wave_sync();
    st.bias2 = ops.bias[threadIdx.x & 15];
    while (mine.left > 0) {
      const size_t n = image_index(mine.k());
      mine.advance();
      const size_t nn = mine.left > 0 ? image_index(mine.k()) : n;
      wave_image<LONE>(st, s, s, ops, images + nn * NI, labels[n], sign, fc_hist + n * FC_HIST, fc_grad);
    }
  }
  // FC weight gradient: a second walk over this wave's images, four per K step (the history rows
  // have left the L2 cache by now; a wave that is done early does this while the others still work)
  f4 g_fc[12];
  if (!PAIR && has_images) {
#pragma unroll
    for (int nt = 0; nt < 12; ++nt) g_fc[nt] = f4{0.0f, 0.0f, 0.0f, 0.0f};
    // this wave's stores to its history rows are complete before it reads them back
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    WaveShare again(K, wave);
    const float* row = fc_hist;  // overwritten before use: has_images
    // operands of one K step (the next four images, fewer at the end)
    auto load_step = [&](FcStepOperands& op) {
      const float* rows[4];
      const int count = again.left < 4 ? again.left : 4;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if (again.left > 0) {
          row = fc_hist + image_index(again.k()) * FC_HIST;
          again.advance();
        }
        rows[k] = row;  // past the last image: the last one again (count masks its delta)
      }
      fc_step_load(op, rows, count);
    };
    // eight steps (32 images) at a time while there are that many, then four, two, one: the loads of
    // a group are one memory round trip (the registers of the image loop are free by now)
    auto steps = [&](auto group) {
      constexpr int N = decltype(group)::value;
      FcStepOperands ops[N];
#pragma unroll
      for (int g = 0; g < N; ++g) load_step(ops[g]);
#pragma unroll
      for (int g = 0; g < N; ++g) fc_step_mfma(g_fc, ops[g]);
    };
    while (again.left > 28) steps(std::integral_constant<int, 8>());
    if (again.left > 12) steps(std::integral_constant<int, 4>());
    if (again.left > 12) steps(std::integral_constant<int, 4>());
    if (again.left > 4) steps(std::integral_constant<int, 2>());
    if (again.left > 4) steps(std::integral_constant<int, 2>());
    if (again.left > 0) steps(std::integral_constant<int, 1>());
    if (again.left > 0) steps(std::integral_constant<int, 1>());
  }
  static_assert(OFF_FC % 4 == 0 && OFF_B % 4 == 0, "whole items");
  __syncthreads();  // every wave is done with the operands: their storage parks the C1 GEMM results
  static_assert(TWAVES * C1G_PARK * sizeof(float) <= sizeof(ops.items), "the parked results fit");
  float *const row = reinterpret_cast<float*>(&s), *const park = reinterpret_cast<float*>(ops.items) + wave * C1G_PARK;
  if (!PAIR && has_images) wave_flush<LONE>(st, sign, g_fc, fc_grad, row, park);
  if (PAIR && has_images && wave < 4) wave_flush<FIRST>(st, sign, g_fc, fc_grad, row, park);
  if (PAIR && has_images && wave >= 4) wave_flush<SECOND>(st, sign, g_fc, fc_grad, row, park);
  __syncthreads();
  {
    // rows of the waves that had images in a fixed tree; an idle wave's row counts as zeros (the
    // first round deals image k to wave k, so wave k has images exactly when K > k)
    const f4* r = reinterpret_cast<const f4*>(&lds[0]);
    constexpr int RF4 = PSTRIDE / 4;  // a wave's area is exactly one row
    f4* dst = reinterpret_cast<f4*>(partial + (size_t)blockIdx.x * PSTRIDE);
    const f4 zero = f4{0.0f, 0.0f, 0.0f, 0.0f};
    for (int i = threadIdx.x; i < RF4; i += 64 * TWAVES) {
      f4 v[TWAVES];
#pragma unroll
      for (int k = 0; k < TWAVES; ++k) {
        const bool have = K > (PAIR ? k & 3 : k) && !(PAIR && k < 4 && i >= OFF_FC / 4 && i < OFF_B / 4);  // (FIRST has no FC weights)
        v[k] = have ? r[i + k * RF4] : zero;
      }
      dst[i] = ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
    }
  }
}

// Small batches: eight waves share one image (cnn_group.h); one partial row per workgroup.
// PAIR: two workgroups per image, blocks 0 .. B - 1 and B .. 2 B - 1 (GroupPart).
template <bool PAIR>
__global__ __launch_bounds__(64 * GWAVES) void train_group_kernel(const float* __restrict__ images,
                                                              const int32_t* __restrict__ labels, int B,
                                                              const float* __restrict__ tabg,
                                                              float* __restrict__ partial) {
  __shared__ OperandTable<TAB_TRAIN_ENTRIES> tab;
  __shared__ TrainLds s;
  __shared__ __align__(16) float d_s1b[D_S1B_FLOATS];
  const bool upper = PAIR && blockIdx.x >= (unsigned)B;
  const size_t n = blockIdx.x - (upper ? B : 0);
  const float* image = images + n * NI;
  float* row = partial + n * PSTRIDE;
  if (!PAIR)
    group_train<false, WHOLE>(image, labels + n, tabg, row, tab, s, d_s1b);
  else if (!upper)
    group_train<false, LOWER>(image, labels + n, tabg, row, tab, s, d_s1b);
  else
    group_train<false, UPPER>(image, labels + n, tabg, row, tab, s, d_s1b);
}

// Expanded operand table from the flat parameter vector: tabg[i] = table_scale(i) * w[table_source(i)] or 0.
__global__ __launch_bounds__(256) void expand_kernel(const float* __restrict__ w, float* __restrict__ tabg) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < TABG_FLOATS) {
    const int p = table_source(i);
    tabg[i] = p >= 0 ? table_scale(i) * w[p] : 0.0f;
  }
}

// Adds the G partial rows in a fixed order (sixteen interleaved strands, each summed in row
// order, then a fixed tree over the strands) and either applies  w <- w - scale * g  (grad_out ==
// nullptr) or stores g.  An updated parameter is also written to its slots of the expanded operand
// table, dest[p][0..3] (-1 = none).  One block of work per P parameters, `block` < PSTRIDE / P; neighbouring
// lanes read P consecutive floats of a row, and a strand keeps sixteen row reads in flight.
// THREADS = 16 P: one strand per thread; half of that: every thread takes strands s and s + 8, one after the
// other (same sums, same order).  COHERENT (device-side epoch loop: rows, weights and table are
// written and read by different compute units within one kernel): agent-scope loads and stores.
// What bounds it: the launch and one memory round trip; the rows come from memory, at the rate of the compute units that ask for
// them.  With P = 32 (a cache line of a row) twice as many ask as with 64, and all 256 rows of the largest calls are one trip.
// Step of 256 / 512 / 1000 images, us, with P = 64 13.17 / 20.33 / 22.43, 32 13.08 / 19.96 / 22.27, 16 (half lines) 13.63 /
// 21.13 / 22.88; up to 128 images 32 is as fast as 64.
constexpr int RSTRANDS = 16, REDUCE_PARAMS = 32;
static_assert(PSTRIDE % REDUCE_PARAMS == 0, "whole blocks of parameters");
template <bool COHERENT>
__device__ __forceinline__ float ld_shared(const float* p) {
  return COHERENT ? __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : *p;
}
template <bool COHERENT>
__device__ __forceinline__ void st_shared(float* p, float v) {
  if (COHERENT)
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else
    *p = v;
}
template <int P, int THREADS, bool COHERENT>
__device__ __forceinline__ void reduce_update_block(int block, float (&red)[RSTRANDS][P],
                                                    const float* __restrict__ partial, int G, float scale,
                                                    float* __restrict__ w, const int32_t* __restrict__ dest,
                                                    float* __restrict__ tabg, float* __restrict__ grad_out,
                                                    float* __restrict__ loss_sum) {
  static_assert(THREADS == P * RSTRANDS || THREADS == P * RSTRANDS / 2, "one or two strands per thread");
  constexpr int TOGETHER = THREADS / P, PASSES = RSTRANDS / TOGETHER;
  const int lane = threadIdx.x % P, first = threadIdx.x / P;
  const int p = block * P + lane;
  // what the update needs besides the sum is fetched first, so that it arrives during the reduction
  float w_old = 0.0f;
  int4 d = int4{-1, -1, -1, -1};
  if (first == 0 && !grad_out && p < NPARAM) {
    w_old = ld_shared<COHERENT>(w + p);
    d = reinterpret_cast<const int4*>(dest)[p];
  }
  const float* src = partial + p;
#pragma unroll
  for (int pass = 0; pass < PASSES; ++pass) {
    const int strand = first + TOGETHER * pass;
    // up to sixteen row reads in flight per strand; a row index past G reads nothing and adds 0.0
    float a[8] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
    for (int g = 0; g < G; g += 16 * RSTRANDS) {
      const bool both = g + 8 * RSTRANDS < G;
      float r[16];
      auto fetch = [&](int k) {
        const int row = g + strand + k * RSTRANDS;
        r[k] = row < G ? ld_shared<COHERENT>(src + (size_t)row * PSTRIDE) : 0.0f;
      };
#pragma unroll
      for (int k = 0; k < 8; ++k) fetch(k);
      if (both) {
#pragma unroll
        for (int k = 8; k < 16; ++k) fetch(k);
      }
#pragma unroll
      for (int k = 0; k < 8; ++k) a[k] += r[k];
      if (both) {
#pragma unroll
        for (int k = 0; k < 8; ++k) a[k] += r[8 + k];
      }
    }
    red[strand][lane] = ((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7]));
  }
  __syncthreads();
  if (first == 0) {
    float t[RSTRANDS];
#pragma unroll
    for (int k = 0; k < RSTRANDS; ++k) t[k] = red[k][lane];
#pragma unroll
    for (int step = 1; step < RSTRANDS; step *= 2)
#pragma unroll
      for (int k = 0; k < RSTRANDS; k += 2 * step) t[k] += t[k + step];
    const float total = t[0];
    if (p < NPARAM) {
      if (grad_out) {
        grad_out[p] = total;
      } else {
        const float wn = fmaf(-scale, total, w_old);
        st_shared<COHERENT>(w + p, wn);
        if (d.x >= 0) st_shared<COHERENT>(tabg + d.x, table_scale(d.x) * wn);
        if (d.y >= 0) st_shared<COHERENT>(tabg + d.y, table_scale(d.y) * wn);
        if (d.z >= 0) st_shared<COHERENT>(tabg + d.z, table_scale(d.z) * wn);
        if (d.w >= 0) st_shared<COHERENT>(tabg + d.w, table_scale(d.w) * wn);
      }
    } else if (p == LOSS_SLOT && loss_sum) {
      *loss_sum = total;
    }
  }
}

template <int P>
__global__ __launch_bounds__(P * RSTRANDS) void reduce_update_kernel(const float* __restrict__ partial, int G,
                                                                     float scale, float* __restrict__ w,
                                                                     const int32_t* __restrict__ dest,
                                                                     float* __restrict__ tabg,
                                                                     float* __restrict__ grad_out,
                                                                     float* __restrict__ loss_sum) {
  __shared__ float red[RSTRANDS][P];
  reduce_update_block<P, P * RSTRANDS, false>(blockIdx.x, red, partial, G, scale, w, dest, tabg, grad_out, loss_sum);
}

// ---- device-side epoch loop ---------------------------------------------------------------------------
// Every step of an epoch inside ONE kernel, for batches small enough that all workgroups (one per
// image of a batch, eight waves each) are resident at once.  Per step: the fused forward + backward
// of the workgroup's image (cnn_group.h) -> its partial row; grid barrier; the workgroups 0 ..
// PSTRIDE/64 - 1 sum their 64 parameters over the rows in the order of reduce_update_kernel, update
// them and the expanded operand table; grid barrier; next step (which re-reads the table).
// Rows, weights and table travel between compute units (whose L2 caches are not coherent with each
// other) as agent-scope loads and stores.
//
// Grid barrier: workgroup b publishes the number of the barrier in flags[b] once all its threads'
// stores have completed; thread t < G of every workgroup polls flags[t].  No read-modify-write: a
// central counter costs 3.2 us per barrier at 100 workgroups, this form 2.5 us.  Every wait is
// bounded: after `limit` ticks of the 100 MHz wall clock (or when another workgroup has given up)
// the workgroup sets the error word and leaves; so do, in turn, all others.  flags[phantom] with
// phantom >= 0 is a flag nobody sets: the host's way to force the give-up path in a test.
struct GridSync {
  unsigned* flags;
  unsigned* error;
  unsigned G, epoch;
  long long limit;
  int phantom;
};
__device__ __forceinline__ bool grid_barrier(GridSync& gs, int* dead) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this thread's agent-scope stores have been performed
  __syncthreads();
  ++gs.epoch;
  const unsigned t = threadIdx.x;
  if (t == 0) __hip_atomic_store(&gs.flags[blockIdx.x], gs.epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (t < gs.G || (gs.phantom >= 0 && t == gs.G)) {
    const unsigned* flag = &gs.flags[t < gs.G ? t : (unsigned)gs.phantom];
    const long long t0 = wall_clock64();
    unsigned polls = 0;
    while ((int)(__hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) - gs.epoch) < 0) {
      if ((++polls & 7) == 0 &&
          (wall_clock64() - t0 > gs.limit ||
           __hip_atomic_load(gs.error, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0)) {
        __hip_atomic_store(gs.error, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        *dead = 1;
        break;
      }
      __builtin_amdgcn_s_sleep(1);
    }
  }
  __syncthreads();
  return *dead == 0;
}

__global__ __launch_bounds__(64 * GWAVES) void train_epoch_kernel(const float* __restrict__ images,
                                                              const int32_t* __restrict__ labels, int steps,
                                                              float scale, float* __restrict__ w,
                                                              const int32_t* __restrict__ dest,
                                                              float* __restrict__ tabg,
                                                              float* __restrict__ partial,
                                                              float* __restrict__ loss_sums, unsigned* flags,
                                                              unsigned* error, unsigned epoch_base,
                                                              long long limit, int phantom) {
  __shared__ OperandTable<TAB_TRAIN_ENTRIES> tab;
  __shared__ TrainLds s;
  __shared__ __align__(16) float d_s1b[D_S1B_FLOATS];
  __shared__ float red[RSTRANDS][64];
  __shared__ int dead;
  if (threadIdx.x == 0) dead = 0;
  GridSync gs{flags, error, gridDim.x, epoch_base, limit, phantom};
  const int B = gridDim.x;  // images per step = workgroups
  // a launch that follows one that gave up does nothing (the host resets the error word)
  if (__hip_atomic_load(error, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) return;
  float* row = partial + (size_t)blockIdx.x * PSTRIDE;
  for (int k = 0; k < steps; ++k) {
    const size_t n = (size_t)k * B + blockIdx.x;
    group_train<true, WHOLE>(images + n * NI, labels + n, tabg, row, tab, s, d_s1b);
    if (!grid_barrier(gs, &dead)) return;  // every row of the step is in memory
    for (int j = blockIdx.x; j < PSTRIDE / 64; j += gridDim.x) {  // (a batch below 61 images: several blocks each)
      reduce_update_block<64, 64 * GWAVES, true>(j, red, partial, B, scale, w, dest, tabg, nullptr,
                                            loss_sums ? loss_sums + k : nullptr);
      __syncthreads();  // `red` is free again
    }
    if (!grid_barrier(gs, &dead)) return;  // weights and table of the next step are in memory
  }
}

}  // namespace

// ------------------------------------------------------------------- C ABI
struct cnn_ctx {
  hipStream_t stream;
  int max_batch;
  float* w;             // [PSTRIDE]
  float* tabg;          // [TABG_FLOATS]: the operand table expanded from w, kept in step with it
  int32_t* dest;        // [PSTRIDE][TABLE_MAX_DEST]: slots of tabg that hold parameter p
  float* partial;       // [partial_rows_for(max_batch)][PSTRIDE]
  float* eval_partial;  // [eval_pairs(max_batch)][2]: a pair per workgroup
  float* fc_hist;       // [max_batch][FC_HIST] when max_batch > WAVE_PAIR_MAX_BATCH: per image, what the FC weight gradient needs
  unsigned* sync;       // [SYNC_WORDS]: barrier flags of the device-side epoch loop, then its error word
  int epoch_mode = 0;         // 1: cnn_train_epoch runs as one kernel where it can
  long long wait_ticks = 0;   // longest wait at a grid barrier, in ticks of the 100 MHz wall clock
  int phantom = -1;           // test hook: also wait for this flag, which nobody sets
  unsigned barrier_count = 0; // barriers passed by every workgroup so far (flags hold such counts)
  int resident_limit = -1;    // most workgroups of train_epoch_kernel resident at once (-1: not asked yet)
  std::vector<hipEvent_t> ev;  // 2 per recorded step (before, after the fused kernel)
  int ev_used = 0;             // recorded steps
};

namespace {

constexpr size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// Workgroups of the forward-only kernel for B images: at most one, of FWAVES waves, per compute unit.
inline int forward_blocks(int B) { return B < FWAVES * TRAIN_BLOCKS ? (B + FWAVES - 1) / FWAVES : TRAIN_BLOCKS; }

// (count, loss) pairs an evaluation can write: one per workgroup.
inline int eval_pairs(int max_batch) {
  static_assert(TRAIN_BLOCKS <= FWD_GROUP_MAX_BATCH, "of one wave per image there are fewer");
  return max_batch < FWD_GROUP_MAX_BATCH ? max_batch : FWD_GROUP_MAX_BATCH;
}

struct Layout {
  size_t w, tabg, dest, partial, eval_partial, fc_hist, sync, total;
};

// Partial rows a step can write: one per workgroup of eight waves in the kernels of large batches, one per image in the
// small-batch kernel (one or two workgroups per image).
inline int partial_rows_for(int max_batch) {
  const int by_wave = max_batch < TRAIN_BLOCKS ? max_batch : TRAIN_BLOCKS;
  const int by_group = max_batch < GROUP_MAX_BATCH ? max_batch : GROUP_MAX_BATCH;
  return by_wave > by_group ? by_wave : by_group;
}

inline Layout layout_for(int max_batch) {
  Layout l;
  const size_t g = (size_t)partial_rows_for(max_batch);
  l.w = 0;
  l.tabg = align_up(l.w + sizeof(float) * PSTRIDE, 256);
  l.dest = align_up(l.tabg + sizeof(float) * TABG_FLOATS, 256);
  l.partial = align_up(l.dest + sizeof(int32_t) * TABLE_MAX_DEST * PSTRIDE, 256);
  l.eval_partial = align_up(l.partial + sizeof(float) * PSTRIDE * g, 256);
  l.fc_hist = align_up(l.eval_partial + sizeof(float) * 2 * (size_t)eval_pairs(max_batch), 256);
  // only the kernel with one wave per image writes history rows
  const size_t hist_rows = max_batch > WAVE_PAIR_MAX_BATCH ? (size_t)max_batch : 0;
  l.sync = align_up(l.fc_hist + sizeof(float) * FC_HIST * hist_rows, 256);
  l.total = align_up(l.sync + sizeof(unsigned) * SYNC_WORDS, 256);
  return l;
}

const int kParamOff[6] = {OFF_K1, OFF_B1, OFF_K2, OFF_B2, OFF_FC, OFF_B};
const int kParamLen[6] = {150, 6, 1800, 12, 1920, 10};

inline bool batch_ok(const cnn_ctx* ctx, int B) { return ctx && B >= 1 && B <= ctx->max_batch; }

int run_forward(cnn_ctx* ctx, const float* images, const int32_t* labels, int B, float* yhat, float* c1,
                float* s1, float* c2, float* s2, bool eval) {
  const DumpPtrs dump = {c1, s1, c2, s2};
  const bool dumps = c1 || s1 || c2 || s2;
  float* pairs = eval ? ctx->eval_partial : nullptr;
  if (B <= FWD_GROUP_MAX_BATCH) {
    auto kernel = dumps ? forward_group_kernel<true> : forward_group_kernel<false>;
    kernel<<<B, 64 * GWAVES, 0, ctx->stream>>>(images, labels, ctx->tabg, yhat, dump, pairs);
    return hipGetLastError() == hipSuccess ? B : CNN_EHIP;
  }
  const int blocks = forward_blocks(B);
  auto kernel = dumps ? forward_kernel<true> : forward_kernel<false>;
  kernel<<<blocks, 64 * FWAVES, 0, ctx->stream>>>(images, labels, B, ctx->w, ctx->tabg, yhat, dump, pairs);
  if (hipGetLastError() != hipSuccess) return CNN_EHIP;
  return blocks;
}

int run_backward(cnn_ctx* ctx, const float* images, const int32_t* labels, int B, float scale,
                 float* grad_out, float* loss_sum) {
  const bool grouped = B <= GROUP_MAX_BATCH;
  // small batches: one or two workgroups per image; large ones: one workgroup of eight waves per compute unit
  const int blocks = grouped ? B : (B < TRAIN_BLOCKS ? B : TRAIN_BLOCKS);
  const int G = blocks;  // one partial row per workgroup, or per pair of workgroups
  const bool timed = (size_t)(2 * ctx->ev_used + 1) < ctx->ev.size();
  if (timed) CNN_HIP_TRY(hipEventRecord(ctx->ev[2 * ctx->ev_used], ctx->stream));
  if (grouped && B <= GROUP_PAIR_MAX_BATCH)
    train_group_kernel<true><<<2 * blocks, 64 * GWAVES, 0, ctx->stream>>>(images, labels, B, ctx->tabg, ctx->partial);
  else if (grouped)
    train_group_kernel<false><<<blocks, 64 * GWAVES, 0, ctx->stream>>>(images, labels, B, ctx->tabg, ctx->partial);
  else if (B <= WAVE_PAIR_MAX_BATCH)
    train_kernel<true><<<blocks, 64 * TWAVES, 0, ctx->stream>>>(images, labels, B, ctx->w, ctx->tabg, ctx->partial, ctx->fc_hist);
  else
    train_kernel<false><<<blocks, 64 * TWAVES, 0, ctx->stream>>>(images, labels, B, ctx->w, ctx->tabg, ctx->partial, ctx->fc_hist);
  if (hipGetLastError() != hipSuccess) return CNN_EHIP;
  if (timed) {
    CNN_HIP_TRY(hipEventRecord(ctx->ev[2 * ctx->ev_used + 1], ctx->stream));
    ++ctx->ev_used;
  }
  constexpr int P = REDUCE_PARAMS;
  reduce_update_kernel<P><<<PSTRIDE / P, P * RSTRANDS, 0, ctx->stream>>>(ctx->partial, G, scale, ctx->w, ctx->dest,
                                                              ctx->tabg, grad_out, loss_sum);
  if (hipGetLastError() != hipSuccess) return CNN_EHIP;
  return CNN_OK;
}

}  // namespace

extern "C" {

const char* cnn_strerror(int code) {
  switch (code) {
    case CNN_OK: return "ok";
    case CNN_EINVAL: return "invalid argument (null or misaligned pointer, size out of range)";
    case CNN_EWORKSPACE: return "workspace too small";
    case CNN_EHIP: return "HIP runtime call or kernel launch failed";
    case CNN_ESCRATCH: return "the problem needs more than the library's built-in scratch buffer";
    case CNN_ETIMEOUT: return "a wait between workgroups of the device-side epoch loop was given up";
    default: return "unknown error code";
  }
}

size_t cnn_workspace_bytes(int max_batch) { return max_batch < 1 ? 0 : layout_for(max_batch).total; }

int cnn_set_weights(cnn_ctx* ctx, const float* k1, const float* b1, const float* k2, const float* b2,
                    const float* fc, const float* b) {
  if (!ctx) return CNN_EINVAL;
  const float* src[6] = {k1, b1, k2, b2, fc, b};
  for (int a = 0; a < 6; ++a)
    if (src[a])
      CNN_HIP_TRY(hipMemcpyAsync(ctx->w + kParamOff[a], src[a], sizeof(float) * kParamLen[a],
                                 hipMemcpyDeviceToDevice, ctx->stream));
  expand_kernel<<<(TABG_FLOATS + 255) / 256, 256, 0, ctx->stream>>>(ctx->w, ctx->tabg);
  return hipGetLastError() == hipSuccess ? CNN_OK : CNN_EHIP;
}

int cnn_get_weights(cnn_ctx* ctx, float* k1, float* b1, float* k2, float* b2, float* fc, float* b) {
  if (!ctx) return CNN_EINVAL;
  float* dst[6] = {k1, b1, k2, b2, fc, b};
  for (int a = 0; a < 6; ++a)
    if (dst[a])
      CNN_HIP_TRY(hipMemcpyAsync(dst[a], ctx->w + kParamOff[a], sizeof(float) * kParamLen[a],
                                 hipMemcpyDeviceToDevice, ctx->stream));
  return CNN_OK;
}

int cnn_init(cnn_ctx** out, void* workspace, size_t workspace_bytes, int max_batch, const float* k1,
             const float* b1, const float* k2, const float* b2, const float* fc, const float* b,
             void* hip_stream) {
  if (!out) return CNN_EINVAL;
  *out = nullptr;
  if (!workspace || max_batch < 1 || (reinterpret_cast<uintptr_t>(workspace) & 255u)) return CNN_EINVAL;
  const Layout l = layout_for(max_batch);
  if (workspace_bytes < l.total) return CNN_EWORKSPACE;
  cnn_ctx* ctx = new (std::nothrow) cnn_ctx;
  if (!ctx) return CNN_EINVAL;
  char* base = static_cast<char*>(workspace);
  ctx->stream = (hipStream_t)hip_stream;
  ctx->max_batch = max_batch;
  ctx->w = reinterpret_cast<float*>(base + l.w);
  ctx->tabg = reinterpret_cast<float*>(base + l.tabg);
  ctx->dest = reinterpret_cast<int32_t*>(base + l.dest);
  ctx->partial = reinterpret_cast<float*>(base + l.partial);
  ctx->eval_partial = reinterpret_cast<float*>(base + l.eval_partial);
  ctx->fc_hist = reinterpret_cast<float*>(base + l.fc_hist);
  ctx->sync = reinterpret_cast<unsigned*>(base + l.sync);
  ctx->wait_ticks = 100000000ll;  // one second
  {
    // inverse of table_source: where each parameter sits in the expanded table
    static_assert(TABLE_MAX_DEST == 4 && table_max_multiplicity() <= TABLE_MAX_DEST,
                  "the update kernel reads a parameter's table slots as one int4");
    std::vector<int32_t> dest(TABLE_MAX_DEST * PSTRIDE, -1);
    for (int i = 0; i < TABG_FLOATS; ++i) {
      const int p = table_source(i);
      if (p < 0) continue;
      int k = 0;
      while (dest[TABLE_MAX_DEST * p + k] >= 0) ++k;  // < TABLE_MAX_DEST by the assertion above
      dest[TABLE_MAX_DEST * p + k] = i;
    }
    // synchronous copy: the host vector may go away as soon as the call returns
    if (hipMemcpy(ctx->dest, dest.data(), sizeof(int32_t) * dest.size(), hipMemcpyHostToDevice) != hipSuccess ||
        hipMemsetAsync(ctx->w, 0, sizeof(float) * PSTRIDE, ctx->stream) != hipSuccess ||
        hipMemsetAsync(ctx->sync, 0, sizeof(unsigned) * SYNC_WORDS, ctx->stream) != hipSuccess) {
      (void)hipGetLastError();
      delete ctx;
      return CNN_EHIP;
    }
  }
  const int rc = cnn_set_weights(ctx, k1, b1, k2, b2, fc, b);
  if (rc != CNN_OK) {
    delete ctx;
    return rc;
  }
  *out = ctx;
  return CNN_OK;
}

int cnn_profile_begin(cnn_ctx* ctx, int capacity) {
  if (!ctx || capacity < 0 || capacity > (1 << 20)) return CNN_EINVAL;
  for (hipEvent_t e : ctx->ev) (void)hipEventDestroy(e);
  ctx->ev.clear();
  ctx->ev_used = 0;
  for (int i = 0; i < 2 * capacity; ++i) {
    hipEvent_t e;
    if (hipEventCreate(&e) != hipSuccess) {
      (void)hipGetLastError();
      for (hipEvent_t d : ctx->ev) (void)hipEventDestroy(d);
      ctx->ev.clear();
      return CNN_EHIP;
    }
    ctx->ev.push_back(e);
  }
  return CNN_OK;
}

int cnn_profile_read(cnn_ctx* ctx, float* ms, int capacity, int* n_recorded) {
  if (!ctx || !ms || !n_recorded || capacity < 0) return CNN_EINVAL;
  CNN_HIP_TRY(hipStreamSynchronize(ctx->stream));
  const int n = ctx->ev_used < capacity ? ctx->ev_used : capacity;
  for (int i = 0; i < n; ++i) CNN_HIP_TRY(hipEventElapsedTime(&ms[i], ctx->ev[2 * i], ctx->ev[2 * i + 1]));
  *n_recorded = n;
  ctx->ev_used = 0;
  return CNN_OK;
}

void cnn_destroy(cnn_ctx* ctx) {
  if (!ctx) return;
  for (hipEvent_t e : ctx->ev) (void)hipEventDestroy(e);
  delete ctx;
}

int cnn_forward(cnn_ctx* ctx, const float* images, int B, float* yhat) {
  if (!batch_ok(ctx, B) || !images || !yhat || !aligned16(images) || !aligned16(yhat)) return CNN_EINVAL;
  const int rc = run_forward(ctx, images, nullptr, B, yhat, nullptr, nullptr, nullptr, nullptr, false);
  return rc < 0 ? rc : CNN_OK;
}

int cnn_forward_activations(cnn_ctx* ctx, const float* images, int B, float* c1, float* s1, float* c2,
                            float* s2, float* yhat) {
  if (!batch_ok(ctx, B) || !images || !aligned16(images)) return CNN_EINVAL;
  const float* outs[5] = {c1, s1, c2, s2, yhat};
  for (const float* p : outs)
    if (p && !aligned16(p)) return CNN_EINVAL;
  const int rc = run_forward(ctx, images, nullptr, B, yhat, c1, s1, c2, s2, false);
  return rc < 0 ? rc : CNN_OK;
}

int cnn_evaluate(cnn_ctx* ctx, const float* images, const int32_t* labels, int N, int64_t* n_correct,
                 float* loss_sum) {
  if (!batch_ok(ctx, N) || !images || !labels || !n_correct || !aligned16(images)) return CNN_EINVAL;
  const int G = run_forward(ctx, images, labels, N, nullptr, nullptr, nullptr, nullptr, nullptr, true);
  if (G < 0) return G;
  eval_reduce_kernel<<<1, EVAL_REDUCE_THREADS, 0, ctx->stream>>>(ctx->eval_partial, G, n_correct, loss_sum);
  return hipGetLastError() == hipSuccess ? CNN_OK : CNN_EHIP;
}

int cnn_gradient(cnn_ctx* ctx, const float* images, const int32_t* labels, int B, float* grad,
                 float* loss_sum) {
  if (!batch_ok(ctx, B) || !images || !labels || !grad || !aligned16(images) || !aligned16(grad))
    return CNN_EINVAL;
  return run_backward(ctx, images, labels, B, 0.0f, grad, loss_sum);
}

int cnn_train_batch(cnn_ctx* ctx, const float* images, const int32_t* labels, int B, float lr,
                    float* loss_sum) {
  if (!batch_ok(ctx, B) || !images || !labels || !aligned16(images)) return CNN_EINVAL;
  return run_backward(ctx, images, labels, B, lr / (float)B, nullptr, loss_sum);
}

int cnn_train_epoch(cnn_ctx* ctx, const float* images, const int32_t* labels, int N, int batch, float lr,
                    float* loss_sums) {
  if (!ctx || N < 1 || !batch_ok(ctx, batch) || !images || !labels || !aligned16(images)) return CNN_EINVAL;
  int first = 0, k = 0;
  if (ctx->epoch_mode == 1 && batch <= EPOCH_MAX_BATCH && N >= batch) {
    // the whole steps as ONE kernel, if all its workgroups can be resident at once
    if (ctx->resident_limit < 0) {
      int per_cu = 0, dev = 0, cus = 0;
      CNN_HIP_TRY(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, train_epoch_kernel, 64 * GWAVES, 0));
      CNN_HIP_TRY(hipGetDevice(&dev));
      CNN_HIP_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
      ctx->resident_limit = per_cu * cus;
    }
    const int steps = N / batch;
    if (batch <= ctx->resident_limit && ctx->barrier_count < 0x7f000000u - 2u * (unsigned)steps) {
      train_epoch_kernel<<<batch, 64 * GWAVES, 0, ctx->stream>>>(
          images, labels, steps, lr / (float)batch, ctx->w, ctx->dest, ctx->tabg, ctx->partial, loss_sums,
          ctx->sync, ctx->sync + SYNC_ERROR, ctx->barrier_count, ctx->wait_ticks, ctx->phantom);
      if (hipGetLastError() != hipSuccess) return CNN_EHIP;
      ctx->barrier_count += 2u * (unsigned)steps;
      first = steps * batch;
      k = steps;
    }
  }
  for (; first < N; ++k, first += batch) {
    const int B = N - first < batch ? N - first : batch;
    const int rc = run_backward(ctx, images + (size_t)first * NI, labels + first, B, lr / (float)B, nullptr,
                                loss_sums ? loss_sums + k : nullptr);
    if (rc != CNN_OK) return rc;
  }
  return CNN_OK;
}

int cnn_epoch_mode(cnn_ctx* ctx, int device_loop, double wait_seconds, int never_arrives) {
  if (!ctx || (device_loop != 0 && device_loop != 1) || !(wait_seconds >= 0.0) || wait_seconds > 3600.0)
    return CNN_EINVAL;
  ctx->epoch_mode = device_loop;
  ctx->wait_ticks = (long long)(wait_seconds * 1e8);
  ctx->phantom = never_arrives ? SYNC_PHANTOM : -1;
  return CNN_OK;
}

int cnn_epoch_status(cnn_ctx* ctx) {
  if (!ctx) return CNN_EINVAL;
  unsigned err = 0;
  CNN_HIP_TRY(hipMemcpyAsync(&err, ctx->sync + SYNC_ERROR, sizeof(err), hipMemcpyDeviceToHost, ctx->stream));
  CNN_HIP_TRY(hipStreamSynchronize(ctx->stream));
  if (err == 0) return CNN_OK;
  // start over: the flags of a kernel that gave up hold different counts
  CNN_HIP_TRY(hipMemsetAsync(ctx->sync, 0, sizeof(unsigned) * SYNC_WORDS, ctx->stream));
  ctx->barrier_count = 0;
  return CNN_ETIMEOUT;
}

}  // extern "C"
