// mlp_net.hip -- BF16 MFMA kernels of the 256-512-512-512-5 GELU network.
//
// Every row of the batch passes through all layers on its own, and so does
// its adjoint on the way back; only the weight gradients sum over rows.  So a
// training step is three launches, an inference two:
//   k_mlp_pack    FP32 weights -> BF16 in fragment order (and transposed);
//   k_mlp_rows    a block takes 16 rows through the whole forward pass, the
//                 loss and the whole backward pass, the activations staying
//                 in LDS between layers;
//   k_mlp_update  weight and bias gradients and the AdamW update of the
//                 parameters they belong to, and the loss.
//
// Fragment order.  v_mfma_f32_16x16x32_bf16 takes from lane l the 8 values
// k = 8 (l/16) .. + 8 of row l % 16 of its operand.  A matrix whose rows are
// tiled by 16 and whose K is cut in steps of 32 is stored as
// [tile][step][lane][8], so every operand load of a wave is 1 KiB contiguous.
//
// Sums run over K in ascending steps of 32 in one accumulator per element.
// Rounding points: x, weights, activations and adjoints are rounded to BF16
// (nearest even) before each product; everything else is FP32.
//
// Bound: latency, not rates.  1024 rows are 4.1 GFLOP (3.3 us at the rate of
// a large BF16 product) and 20 MB of parameters and moments; a block reads
// 2.4 MB of weights from L2.  One training step of 1024 rows took 265 us as
// 20 launches (a GEMM kernel per product and layer, casts, column sums,
// AdamW), 52 us now: 4 us packing, 36 us rows, 12 us update.  Inference of
// 4096 rows: 93 -> 25 us.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "device.hpp"
#include "mlp.hpp"

namespace hf {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
// callers' FP32 arrays are only known to be aligned to their values
typedef float f32x4_u __attribute__((ext_vector_type(4), aligned(4)));

__device__ __forceinline__ uint16_t f2bf(float f) {
  return __builtin_bit_cast(uint16_t, static_cast<__bf16>(f));
}

__device__ __forceinline__ bf16x8 frag(const uint16_t* p) {
  return *reinterpret_cast<const bf16x8*>(p);
}

constexpr int kFrag = 64 * 8;  // values of one fragment

// ---------------------------------------------------------------------------
// Weights in fragment order
// ---------------------------------------------------------------------------
struct PackArgs {
  const float* params;
  uint16_t* wb[4];  // rows = outputs, K = inputs: the forward products
  uint16_t* wt[4];  // rows = inputs, K = outputs: the adjoints' products (wt[0] unused)
};

constexpr int kPackBlock = 256;
__host__ __device__ constexpr int pack_blocks(int l) {
  return MlpLayout::kIn[l] * MlpLayout::kOutDim[l] / 8 / kPackBlock;
}

// One lane's 8 values of one fragment per thread: 8 neighbouring weights of a
// row (two 16-byte loads) for wb, or one column of 8 rows (64-byte segments
// per 16 lanes) for wt.
__global__ __launch_bounds__(kPackBlock) void k_mlp_pack(PackArgs g) {
  int blk = blockIdx.x, l = 0;
  bool transposed = false;
  while (blk >= pack_blocks(l)) {  // uniform
    blk -= pack_blocks(l);
    if (++l == 4) {
      l = 1;
      transposed = true;
    }
  }
  const int in = MlpLayout::kIn[l], out = MlpLayout::kOutDim[l];
  const float* w = g.params + MlpLayout::kW[l];
  const int id = blk * kPackBlock + threadIdx.x;
  const int lane = id & 63, f = id >> 6;
  const int steps = (transposed ? out : in) / 32;
  const int row = (f / steps) * 16 + (lane & 15), k = (f % steps) * 32 + (lane >> 4) * 8;
  bf16x8 v;
  if (!transposed) {
    const f32x4_u* p = reinterpret_cast<const f32x4_u*>(w + static_cast<int64_t>(row) * in + k);
    const f32x4_u x = p[0], y = p[1];
    v = bf16x8{(__bf16)x.x, (__bf16)x.y, (__bf16)x.z, (__bf16)x.w,
               (__bf16)y.x, (__bf16)y.y, (__bf16)y.z, (__bf16)y.w};
  } else {
    float x[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) x[j] = w[static_cast<int64_t>(k + j) * in + row];
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = (__bf16)x[j];
  }
  uint16_t* o = (transposed ? g.wt[l] : g.wb[l]) + static_cast<int64_t>(id) * 8;
  *reinterpret_cast<bf16x8*>(o) = v;
}

// ---------------------------------------------------------------------------
// Rows through the network
// ---------------------------------------------------------------------------
struct RowArgs {
  const float* x;       // [B][256]
  const float* target;  // [B][5] (training)
  int B;
  const float* params;  // biases
  MlpWorkspace w;
  float* y;             // [B][32]
};

constexpr int kRowThreads = 512;
constexpr int kRowWaves = kRowThreads / 64;
constexpr int kTiles = kMlpHidden / 16 / kRowWaves;  // column tiles of a hidden layer per wave
constexpr int kLd = kMlpHidden + 8;  // LDS row of activations; the pad spreads 16 rows over the banks
constexpr int kRing = kMlpHidden / 32;  // weight fragments in flight per wave: one column tile

// c[i] = A(rows 16 i..) * W(tile)^T over KS steps of 32; A in LDS, the tile's
// fragments already in `ring`, each of which is replaced by the next tile's
// (NKS steps from `next`) as soon as it is used: a tile's weights arrive
// while the one before it is multiplied and its epilogue runs.
template <int MT, int KS, int NKS>
__device__ __forceinline__ void tile_product(const uint16_t* act, const uint16_t* next,
                                             bf16x8 (&ring)[kRing], f32x4 (&c)[MT]) {
  const int lane = threadIdx.x & 63;
  const uint16_t* ap = act + (lane & 15) * kLd + (lane >> 4) * 8;
#pragma unroll
  for (int i = 0; i < MT; ++i) c[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int ks = 0; ks < kRing; ++ks) {
    if (ks < KS) {
#pragma unroll
      for (int i = 0; i < MT; ++i)
        c[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(frag(ap + 16 * i * kLd + ks * 32), ring[ks],
                                                       c[i], 0, 0, 0);
    }
    if (ks < NKS) ring[ks] = frag(next + ks * kFrag);
  }
}

// Stores ROWS staged rows of N values: row-major at `rm` and, in training,
// in fragment order over the batch (tiles of 16 columns, K = rows) at `fo`.
// The row-major copies are the workspace's documented contents; no kernel
// reads them (14.7 MB for 4096 rows of inference, 3 us at a copy's rate, next to
// the products).
template <int ROWS, int N, bool TRAIN>
__device__ __forceinline__ void store_rows(const uint16_t* act, int64_t row0, int B, uint16_t* rm,
                                           uint16_t* fo) {
  constexpr int C = N / 8;  // 16-byte pieces of a row
  for (int p = threadIdx.x; p < ROWS * C; p += kRowThreads) {
    const int r = p / C, q = p % C;
    *reinterpret_cast<uint4*>(rm + (row0 + r) * N + 8 * q) =
        *reinterpret_cast<const uint4*>(act + r * kLd + 8 * q);
  }
  if constexpr (TRAIN) {
    const int n = threadIdx.x;
    if (n < N) {
#pragma unroll
      for (int h = 0; h < ROWS / 8; ++h) {
        uint32_t v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k)
          v[k] = act[(8 * h + 2 * k) * kLd + n] |
                 static_cast<uint32_t>(act[(8 * h + 2 * k + 1) * kLd + n]) << 16;
        const int64_t b = row0 + 8 * h;
        const int64_t f = static_cast<int64_t>(n >> 4) * (B >> 5) + (b >> 5);
        const int lane = static_cast<int>((b & 31) >> 3) * 16 + (n & 15);
        *reinterpret_cast<uint4*>(fo + f * kFrag + lane * 8) = uint4{v[0], v[1], v[2], v[3]};
      }
    }
  }
}

// One hidden layer of the wave's column tiles.  FORWARD: bias, GELU and
// rounding into the staged rows `out`; in training also z to memory and
// GELU'(z), for which the erf is shared.  Otherwise the adjoint through a
// layer: GELU'(z) times the product, rounded.  The expressions are written
// out without contraction, so that the forward and the adjoint round as
// separate evaluations would.
template <int MT, int KS, int NKS, bool FORWARD, bool TRAIN>
__device__ __forceinline__ void hidden_layer(const uint16_t* act, const uint16_t* w,
                                             const uint16_t* next, bf16x8 (&ring)[kRing],
                                             const float* bias, uint16_t* out, float* z, int64_t row0,
                                             f32x4 (&gp)[kTiles][TRAIN ? MT : 1]) {
#pragma clang fp contract(off)
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int j = 0; j < kTiles; ++j) {
    const int n = (wave * kTiles + j) * 16 + (lane & 15);
    f32x4 c[MT];
    if (j + 1 < kTiles)
      tile_product<MT, KS, KS>(act, w + (j + 1) * KS * kFrag, ring, c);
    else
      tile_product<MT, KS, NKS>(act, next, ring, c);
    const float b = FORWARD ? bias[n] : 0.0f;
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int m = 16 * i + 4 * (lane >> 4) + q;
        if constexpr (FORWARD) {
          const float v = c[i][q] + b;
          const float one = 1.0f + erff(v * 0.70710678118654752f);
          out[m * kLd + n] = f2bf((0.5f * v) * one);
          if constexpr (TRAIN) {
            z[(row0 + m) * kMlpHidden + n] = v;
            gp[j][i][q] = __builtin_fmaf(v * 0.39894228040143268f, expf((-0.5f * v) * v), 0.5f * one);
          }
        } else {
          out[m * kLd + n] = f2bf(c[i][q] * gp[j][i][q]);
        }
      }
  }
}

// A block of 8 waves takes 16 MT rows through the network; wave w computes
// columns [64 w, 64 w + 64) of each hidden layer, tile by tile.  16 rows are
// the least an MFMA takes, and give 4096 rows one block per CU.  Tile by tile
// with a whole tile of weights in flight, the inference kernel takes 22 us
// (4096 rows); all four tiles side by side, a quarter of each in flight, 27.
template <int MT, bool TRAIN>
__global__ __launch_bounds__(kRowThreads) void k_mlp_rows(RowArgs g) {
  constexpr int ROWS = 16 * MT;
  __shared__ __attribute__((aligned(16))) uint16_t act[2][ROWS * kLd];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t row0 = static_cast<int64_t>(blockIdx.x) * ROWS;
  constexpr int KS0 = kMlpIn / 32, KS = kMlpHidden / 32, KSY = kMlpOutPad / 32;
  static_assert(KS <= kRing && KSY == 1, "a tile's fragments fit the ring");
  // this wave's fragments of a weight matrix of `steps` K steps
  auto mine = [&](const uint16_t* w, int steps) {
    return w + static_cast<int64_t>(wave) * kTiles * steps * kFrag + lane * 8;
  };
  const uint16_t *w0 = mine(g.w.wb[0], KS0), *w1 = mine(g.w.wb[1], KS), *w2 = mine(g.w.wb[2], KS);
  // the output layer has two column tiles, taken by waves 0 and 1
  const bool out_wave = wave < kMlpOutPad / 16;
  const uint16_t* w3 = g.w.wb[3] + static_cast<int64_t>(out_wave ? wave : 0) * KS * kFrag + lane * 8;
  bf16x8 ring[kRing];
#pragma unroll
  for (int d = 0; d < KS0; ++d) ring[d] = frag(w0 + d * kFrag);
  for (int p = tid; p < ROWS * kMlpIn / 4; p += kRowThreads) {
    const int r = p / (kMlpIn / 4), q = p % (kMlpIn / 4);
    const f32x4_u v = *reinterpret_cast<const f32x4_u*>(g.x + (row0 + r) * kMlpIn + 4 * q);
    *reinterpret_cast<uint2*>(&act[0][r * kLd + 4 * q]) =
        uint2{f2bf(v.x) | static_cast<uint32_t>(f2bf(v.y)) << 16,
              f2bf(v.z) | static_cast<uint32_t>(f2bf(v.w)) << 16};
  }
  __syncthreads();
  f32x4 gp[TRAIN ? 3 : 1][kTiles][TRAIN ? MT : 1];  // GELU' of the three hidden layers
  const float* par = g.params;
  store_rows<ROWS, kMlpIn, TRAIN>(act[0], row0, g.B, g.w.a[0], g.w.at[0]);
  hidden_layer<MT, KS0, KS, true, TRAIN>(act[0], w0, w1, ring, par + MlpLayout::kB[0], act[1],
                                         g.w.z[1], row0, gp[0]);
  __syncthreads();
  store_rows<ROWS, kMlpHidden, TRAIN>(act[1], row0, g.B, g.w.a[1], g.w.at[1]);
  hidden_layer<MT, KS, KS, true, TRAIN>(act[1], w1, w2, ring, par + MlpLayout::kB[1], act[0],
                                        g.w.z[2], row0, gp[TRAIN ? 1 : 0]);
  __syncthreads();
  store_rows<ROWS, kMlpHidden, TRAIN>(act[0], row0, g.B, g.w.a[2], g.w.at[2]);
  const uint16_t *t1 = nullptr, *t2 = nullptr;
  if constexpr (TRAIN) {
    t2 = mine(g.w.wt[2], KS);
    t1 = mine(g.w.wt[1], KS);
  }
  hidden_layer<MT, KS, KS, true, TRAIN>(act[0], w2, TRAIN && !out_wave ? t2 : w3, ring,
                                        par + MlpLayout::kB[2], act[1], g.w.z[3], row0,
                                        gp[TRAIN ? 2 : 0]);
  __syncthreads();
  bf16x8 ring3[kTiles];  // the output layer's transpose: one K step
  if constexpr (TRAIN) {
    const uint16_t* t3 = mine(g.w.wt[3], KSY);
#pragma unroll
    for (int j = 0; j < kTiles; ++j) ring3[j] = frag(t3 + j * KSY * kFrag);
  }
  store_rows<ROWS, kMlpHidden, TRAIN>(act[1], row0, g.B, g.w.a[3], g.w.at[3]);
  if (out_wave) {
    f32x4 c[MT];
    tile_product<MT, KS, TRAIN ? KS : 0>(act[1], t2, ring, c);
    const int n = wave * 16 + (lane & 15);
    const float b = par[MlpLayout::kB[3] + n];
    const float scale = 2.0f / (5.0f * static_cast<float>(g.B));
    double sq = 0.0;
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int m = 16 * i + 4 * (lane >> 4) + q;
        const float v = c[i][q] + b;
        g.y[(row0 + m) * kMlpOutPad + n] = v;
        if constexpr (TRAIN) {
          // loss = sum over the 5 targets of (y - t)^2 / (5 B)
          float d = 0.0f;
          if (n < kMlpOut) {
            d = v - g.target[(row0 + m) * kMlpOut + n];
            sq += static_cast<double>(d) * d;
          }
          act[0][m * kLd + n] = f2bf(scale * d);
        }
      }
    if constexpr (TRAIN) {
      sq = wave_sum(sq);  // wave 1 holds padding columns only
      if (wave == 0 && lane == 0) g.w.loss_part[blockIdx.x] = sq;
    }
  }
  if constexpr (TRAIN) {
    __syncthreads();
    store_rows<ROWS, kMlpOutPad, true>(act[0], row0, g.B, g.w.dz[4], g.w.dzt[4]);
    {
      const uint16_t* ap = act[0] + (lane & 15) * kLd + (lane >> 4) * 8;
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        const bf16x8 a = frag(ap + 16 * i * kLd);
#pragma unroll
        for (int j = 0; j < kTiles; ++j) {
          const f32x4 c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
              a, ring3[j], f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
#pragma unroll
          for (int q = 0; q < 4; ++q)
            act[1][(16 * i + 4 * (lane >> 4) + q) * kLd + (wave * kTiles + j) * 16 + (lane & 15)] =
                f2bf(c[q] * gp[2][j][i][q]);
        }
      }
    }
    __syncthreads();
    store_rows<ROWS, kMlpHidden, true>(act[1], row0, g.B, g.w.dz[3], g.w.dzt[3]);
    hidden_layer<MT, KS, KS, false, true>(act[1], t2, t1, ring, nullptr, act[0], nullptr, row0, gp[1]);
    __syncthreads();
    store_rows<ROWS, kMlpHidden, true>(act[0], row0, g.B, g.w.dz[2], g.w.dzt[2]);
    hidden_layer<MT, KS, 0, false, true>(act[0], t1, nullptr, ring, nullptr, act[1], nullptr, row0,
                                         gp[0]);
    __syncthreads();
    store_rows<ROWS, kMlpHidden, true>(act[1], row0, g.B, g.w.dz[1], g.w.dzt[1]);
  }
}

// ---------------------------------------------------------------------------
// Gradients of the parameters, AdamW, loss
// ---------------------------------------------------------------------------
struct UpdateArgs {
  MlpWorkspace w;
  int B;
  float *p, *m, *v, *grads, *loss;
  int nparts;  // blocks whose loss partials are summed
  float lr, wd, bc1, bc2;
};

// AdamW with decoupled weight decay (Loshchilov & Hutter), FP32 state.
struct Param {
  float p, m, v;
  __device__ __forceinline__ void load(const UpdateArgs& a, int64_t i) {
    p = a.p[i];
    m = a.m[i];
    v = a.v[i];
  }
  __device__ __forceinline__ void step(const UpdateArgs& a, int64_t i, float gi) const {
    a.grads[i] = gi;
    const float mi = 0.9f * m + 0.1f * gi;
    const float vi = 0.999f * v + 0.001f * gi * gi;
    a.m[i] = mi;
    a.v[i] = vi;
    const float mh = mi / a.bc1, vh = vi / a.bc2;
    a.p[i] = p - a.lr * (mh / (sqrtf(vh) + 1e-8f) + a.wd * p);
  }
};

__host__ __device__ constexpr int update_tiles(int l) {
  return (MlpLayout::kOutDim[l] / 32) * (MlpLayout::kIn[l] / 32);
}
constexpr int kUpdateTiles = update_tiles(0) + update_tiles(1) + update_tiles(2) + update_tiles(3);

// One block of four waves per 32 x 32 tile of a weight gradient, dW[n][k] =
// sum_b dz[b][n] a[b][k]: each wave sums a quarter of the rows, and the four
// sums are added in wave order, every wave finishing a quarter of the tile.
// The blocks of the first column of tiles also sum dz over the rows (a
// product with ones) for the bias.  The last block adds up the loss.
// Bound: latency.  The operands come from the last-level cache (the rows'
// kernel ran on other XCDs), so what counts is how many round trips follow
// each other.  1024 rows: 20.7 us with one wave per tile and the parameters
// read after the products, 16.0 with them requested before, 12.1 with four
// waves per tile (16384 rows: the step went from 285 to 248 us).
constexpr int kUpdateWaves = 4;
__global__ __launch_bounds__(64 * kUpdateWaves) void k_mlp_update(UpdateArgs g) {
  __shared__ f32x4 part[kUpdateWaves][4][64];
  __shared__ f32x4 part_bias[kUpdateWaves][2][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int tile = blockIdx.x, l = 0;
  if (tile == kUpdateTiles) {
    if (wave == 0) {
      double s = 0.0;
      for (int q = lane; q < g.nparts; q += 64) s += g.w.loss_part[q];
      s = wave_sum(s);
      if (lane == 0) g.loss[0] = static_cast<float>(s / (5.0 * g.B));
    }
    return;
  }
  while (tile >= update_tiles(l)) tile -= update_tiles(l++);
  const int in = MlpLayout::kIn[l];
  const int to = tile / (in / 32), ti = tile % (in / 32);
  const int KS = g.B / 32;
  const int k0 = KS * wave / kUpdateWaves, k1 = KS * (wave + 1) / kUpdateWaves;
  const int64_t stride = static_cast<int64_t>(KS) * kFrag;
  const uint16_t* ap = g.w.dzt[l + 1] + 2 * to * stride + lane * 8;
  const uint16_t* bp = g.w.at[l] + 2 * ti * stride + lane * 8;
  constexpr int D = 4;  // K steps in flight
  bf16x8 a0[D], a1[D], b0[D], b1[D];
  auto request = [&](int s, int k) {
    const int64_t o = static_cast<int64_t>(k) * kFrag;
    a0[s] = frag(ap + o);
    a1[s] = frag(ap + stride + o);
    b0[s] = frag(bp + o);
    b1[s] = frag(bp + stride + o);
  };
#pragma unroll
  for (int s = 0; s < D; ++s)
    if (k0 + s < k1) request(s, k0 + s);
  // this wave finishes MFMA tile (i, j) = (wave / 2, wave % 2) of the four:
  // lane holds elements [4 (lane/16) + q][lane % 16] of it
  const bool bias = ti == 0, bias_lane = bias && (wave & 1) == 0 && (lane & 15) == 0;
  const int n = 32 * to + 16 * (wave >> 1) + 4 * (lane >> 4);
  const int64_t iw = MlpLayout::kW[l] + static_cast<int64_t>(n) * in + 32 * ti + 16 * (wave & 1) +
                     (lane & 15);
  const int64_t ib = MlpLayout::kB[l] + n;
  Param pw[4], pb[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    pw[q].load(g, iw + q * in);
    if (bias_lane) pb[q].load(g, ib + q);
  }
  f32x4 c00 = {0.f, 0.f, 0.f, 0.f}, c01 = c00, c10 = c00, c11 = c00, d0 = c00, d1 = c00;
  const __bf16 o = (__bf16)1.0f;
  const bf16x8 ones = {o, o, o, o, o, o, o, o};
  for (int kb = k0; kb < k1; kb += D) {
#pragma unroll
    for (int s = 0; s < D; ++s) {
      const int k = kb + s;
      if (k < k1) {
        c00 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0[s], b0[s], c00, 0, 0, 0);
        c01 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0[s], b1[s], c01, 0, 0, 0);
        c10 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1[s], b0[s], c10, 0, 0, 0);
        c11 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1[s], b1[s], c11, 0, 0, 0);
        if (bias) {
          d0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0[s], ones, d0, 0, 0, 0);
          d1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1[s], ones, d1, 0, 0, 0);
        }
        if (k + D < k1) request(s, k + D);
      }
    }
  }
  part[wave][0][lane] = c00;
  part[wave][1][lane] = c01;
  part[wave][2][lane] = c10;
  part[wave][3][lane] = c11;
  if (bias) {
    part_bias[wave][0][lane] = d0;
    part_bias[wave][1][lane] = d1;
  }
  __syncthreads();
  f32x4 sum = part[0][wave][lane];
#pragma unroll
  for (int w = 1; w < kUpdateWaves; ++w) sum += part[w][wave][lane];
#pragma unroll
  for (int q = 0; q < 4; ++q) pw[q].step(g, iw + q * in, sum[q]);
  if (bias_lane) {
    f32x4 db = part_bias[0][wave >> 1][lane];
#pragma unroll
    for (int w = 1; w < kUpdateWaves; ++w) db += part_bias[w][wave >> 1][lane];
#pragma unroll
    for (int q = 0; q < 4; ++q) pb[q].step(g, ib + q, db[q]);
  }
}

hipError_t pack_weights(const float* params, const MlpWorkspace& w, bool train, hipStream_t s) {
  PackArgs a{};
  a.params = params;
  int blocks = 0;
  for (int l = 0; l < 4; ++l) {
    a.wb[l] = w.wb[l];
    a.wt[l] = w.wt[l];
    blocks += pack_blocks(l);
  }
  if (train) blocks += pack_blocks(1) + pack_blocks(2) + pack_blocks(3);
  hipLaunchKernelGGL(k_mlp_pack, dim3(blocks), dim3(kPackBlock), 0, s, a);
  return hipGetLastError();
}

}  // namespace

// B is a positive multiple of 64 (checked by the caller).
hipError_t mlp_forward(int B, const float* params, const float* x, float* y, void* ws,
                       hipStream_t s) {
  RowArgs r{};
  r.x = x;
  r.B = B;
  r.params = params;
  r.w = mlp_carve(ws, B);
  r.y = y;
  hipError_t e = pack_weights(params, r.w, false, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_mlp_rows<1, false>), dim3(B / 16), dim3(kRowThreads), 0, s, r);
  return hipGetLastError();
}

hipError_t mlp_train_step(int B, float* params, float* m, float* v, int step, float lr, float wd,
                          const float* x, const float* t, float* grads, float* loss, void* ws,
                          hipStream_t s) {
  RowArgs r{};
  r.x = x;
  r.target = t;
  r.B = B;
  r.params = params;
  r.w = mlp_carve(ws, B);
  r.y = r.w.y;
  hipError_t e = pack_weights(params, r.w, true, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_mlp_rows<1, true>), dim3(B / 16), dim3(kRowThreads), 0, s, r);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  UpdateArgs u{};
  u.w = r.w;
  u.B = B;
  u.p = params;
  u.m = m;
  u.v = v;
  u.grads = grads;
  u.loss = loss;
  u.nparts = B / 16;
  u.lr = lr;
  u.wd = wd;
  u.bc1 = 1.0f - powf(0.9f, static_cast<float>(step));
  u.bc2 = 1.0f - powf(0.999f, static_cast<float>(step));
  hipLaunchKernelGGL(k_mlp_update, dim3(kUpdateTiles + 1), dim3(64 * kUpdateWaves), 0, s, u);
  return hipGetLastError();
}

}  // namespace hf
