// Learned pre-screening of partial-evaluation candidates: a small MLP
// (192 -> 128 -> 128 -> 3, ReLU) that predicts the objective deltas of a
// single-point partial change from local features, trained on the exact deltas
// the evaluator produces.  Acceptance still rests on the exact evaluator:
// screening only chooses which candidate is evaluated and whether it is
// evaluated at all.
//
// All matrix products run on gfx950 matrix cores: v_mfma_f32_16x16x32_bf16
// (BF16 operands, FP32 accumulation).  Weights are kept in FP32 (master copy,
// Adam state) and BF16 (operands).  Activations are rounded to BF16 where they
// feed the next product; everything else is FP32.
#include <hip/hip_runtime.h>
#include <math.h>
#include <string.h>

#include <algorithm>
#include <string>
#include <type_traits>
#include <vector>

#include "dsm_internal.h"

namespace dsm {
namespace {

constexpr int kIn = 192, kHid = 128, kOut = 3, kOutPad = 16, kNumFeat = 188;
// parameter layout of the FP32 master copy
constexpr int kW1 = 0, kB1 = kW1 + kHid * kIn, kW2 = kB1 + kHid, kB2 = kW2 + kHid * kHid, kW3 = kB2 + kHid,
              kB3 = kW3 + kOutPad * kHid, kNParams = kB3 + kOutPad;
static_assert(kNParams == 43280, "parameter count");

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));

// FP32 -> BF16, round to nearest even
__device__ __forceinline__ unsigned short f2bf(float x) { return __builtin_bit_cast(unsigned short, (__bf16)x); }
__device__ __forceinline__ float bf2f(unsigned short b) { return __uint_as_float((unsigned)b << 16); }

__device__ __forceinline__ f32x4 mfma(const u16x8& a, const u16x8& b, const f32x4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0,
                                                 0);
}

__device__ __forceinline__ u16x8 load8(const unsigned short* p) { return *(const u16x8*)p; }

__device__ __forceinline__ u16x8 zero8() {
  u16x8 z;
  for (int e = 0; e < 8; ++e) z[e] = 0;
  return z;
}

struct MlpW {
  const unsigned short *w1, *w2, *w3;    // BF16 [128][192], [128][128], [16][128] (out, in)
  const unsigned short *w2t, *w3t;       // BF16 transposes [128][128], [128][16] (in, out)
  const float *b1, *b2, *b3;             // FP32 biases
};

// Forward pass of 64 rows by a workgroup of 4 waves, each computing a
// 32-column slice of a layer for all rows, with its slice of every layer's
// weights in registers: the workgroups are persistent and take tile after tile,
// so the weights are read once per workgroup instead of once per 64 rows (at
// 1.2 M rows that was 1.6 GB from L2 and the longest part of the pass).
constexpr int kXs = kIn + 8;  // padded LDS strides (BF16 elements)
constexpr int kHs = kHid + 8;
constexpr int kTileRows = 64;

struct WaveWeights {
  u16x8 w1[2][kIn / 32], w2[2][kHid / 32], w3[kHid / 32];
  float b1[2], b2[2], b3;
};

__device__ __forceinline__ void load_layer1(const MlpW& w, int wave, int lane, WaveWeights& r) {
  const int i = lane & 15, kb = lane >> 4;
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const int col = 32 * wave + 16 * t + i;
#pragma unroll
    for (int kk = 0; kk < kIn / 32; ++kk) r.w1[t][kk] = load8(w.w1 + (size_t)col * kIn + 32 * kk + 8 * kb);
    r.b1[t] = w.b1[col];
  }
}
__device__ __forceinline__ void load_layers23(const MlpW& w, int wave, int lane, WaveWeights& r) {
  const int i = lane & 15, kb = lane >> 4;
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const int col = 32 * wave + 16 * t + i;
#pragma unroll
    for (int kk = 0; kk < kHid / 32; ++kk) r.w2[t][kk] = load8(w.w2 + (size_t)col * kHid + 32 * kk + 8 * kb);
    r.b2[t] = w.b2[col];
  }
#pragma unroll
  for (int kk = 0; kk < kHid / 32; ++kk) r.w3[kk] = load8(w.w3 + (size_t)i * kHid + 32 * kk + 8 * kb);
  r.b3 = w.b3[i];
}

// out = relu(in W^T + b) for this wave's 32 columns of 64 rows (LDS tiles).
template <int K>
__device__ __forceinline__ void layer64(const unsigned short* in, int in_stride, const u16x8 (&w)[2][K / 32],
                                        const float (&b)[2], unsigned short* out, int wave, int lane) {
  const int i = lane & 15, kb = lane >> 4;
  f32x4 acc[2][4];
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int rb = 0; rb < 4; ++rb) acc[t][rb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int kk = 0; kk < K / 32; ++kk)
#pragma unroll
    for (int rb = 0; rb < 4; ++rb) {
      const u16x8 a = *(const u16x8*)(in + (16 * rb + i) * in_stride + 32 * kk + 8 * kb);
#pragma unroll
      for (int t = 0; t < 2; ++t) acc[t][rb] = mfma(a, w[t][kk], acc[t][rb]);
    }
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int rb = 0; rb < 4; ++rb)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        out[(16 * rb + 4 * kb + r) * kHs + 32 * wave + 16 * t + i] = f2bf(fmaxf(acc[t][rb][r] + b[t], 0.f));
}

// Outputs of a tile's rows from the inputs in xs, all threads of the workgroup,
// after a barrier; xs is overwritten with the second hidden layer.  where(i) is
// the output row of the tile's row i, negative if there is none; rest() loads
// the weights of the later layers where they are not there yet.
template <class Where, class Rest>
__device__ __forceinline__ void mlp_tile(const WaveWeights& w, unsigned short* xs, unsigned short* h1, Where where,
                                         float* __restrict__ out, int wave, int lane, Rest rest) {
  const int i = lane & 15, kb = lane >> 4;
  layer64<kIn>(xs, kXs, w.w1, w.b1, h1, wave, lane);
  rest();
  __syncthreads();  // H1 complete, and every read of the inputs done
  layer64<kHid>(h1, kHs, w.w2, w.b2, xs, wave, lane);
  __syncthreads();
  // layer 3: Y = H2 W3^T + b3, wave -> row block `wave`
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int kk = 0; kk < kHid / 32; ++kk) acc = mfma(*(const u16x8*)(xs + (16 * wave + i) * kHs + 32 * kk + 8 * kb), w.w3[kk], acc);
  if (i < kOut)
    for (int r = 0; r < 4; ++r) {
      const int64_t row = where(16 * wave + 4 * kb + r);
      if (row >= 0) out[(size_t)row * kOut + i] = acc[r] + w.b3;
    }
}

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_mlp_forward(
    MlpW w, const unsigned short* __restrict__ xb, int N, float* __restrict__ out) {
  __shared__ __align__(16) unsigned short xs[kTileRows * kXs];  // inputs, then H2
  __shared__ __align__(16) unsigned short h1[kTileRows * kHs];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  WaveWeights ww;
  load_layer1(w, wave, lane, ww);
  load_layers23(w, wave, lane, ww);
  constexpr int kPer = kTileRows * kIn / 8 / 256;  // 16-byte pieces of a tile per thread
  u16x8 next[kPer];
  auto fetch = [&](int64_t row0) {  // the tile after the current one, in flight while that is computed
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      const int e = tid + 256 * q, r = e / (kIn / 8), c = e % (kIn / 8);
      next[q] = row0 + r < N ? load8(xb + (size_t)(row0 + r) * kIn + 8 * c) : zero8();
    }
  };
  fetch((int64_t)blockIdx.x * kTileRows);
  for (int64_t row0 = (int64_t)blockIdx.x * kTileRows; row0 < N; row0 += (int64_t)gridDim.x * kTileRows) {
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      const int e = tid + 256 * q;
      *(u16x8*)(xs + (e / (kIn / 8)) * kXs + 8 * (e % (kIn / 8))) = next[q];
    }
    fetch(row0 + (int64_t)gridDim.x * kTileRows);
    __syncthreads();
    mlp_tile(ww, xs, h1, [&](int i) { return row0 + i < N ? row0 + i : (int64_t)-1; }, out, wave, lane, [] {});
    __syncthreads();
  }
}

// The same for one tile a workgroup: the weights arrive layer by layer, so the
// first one waits for its own alone, and take 105 instead of 216 registers, so
// more workgroups share a CU.  Up to the 768 tiles of a persistent launch, whose
// workgroups take one tile each as well: 20,000 rows 11.1 us persistent, 9.4 so,
// 40,000 16.2 and 12.0.
__global__ __launch_bounds__(256) void k_mlp_forward_once(MlpW w, const unsigned short* __restrict__ xb, int N,
                                                          float* __restrict__ out) {
  __shared__ __align__(16) unsigned short xs[kTileRows * kXs];  // inputs, then H2
  __shared__ __align__(16) unsigned short h1[kTileRows * kHs];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, row0 = blockIdx.x * kTileRows;
  for (int e = tid; e < kTileRows * kIn / 8; e += 256) {
    const int r = e / (kIn / 8), c = e % (kIn / 8);
    *(u16x8*)(xs + r * kXs + 8 * c) = row0 + r < N ? load8(xb + (size_t)(row0 + r) * kIn + 8 * c) : zero8();
  }
  WaveWeights ww;
  load_layer1(w, wave, lane, ww);
  __syncthreads();
  mlp_tile(ww, xs, h1, [&](int i) { return row0 + i < N ? (int64_t)(row0 + i) : (int64_t)-1; }, out, wave, lane,
           [&] { load_layers23(w, wave, lane, ww); });
}

// Workgroups of a persistent launch over N rows (a multiple of 8): three to a CU.
constexpr int kPersistent = 3 * 256;
unsigned mlp_grid(int64_t N) { return (unsigned)std::min<int64_t>((N + 8 * kTileRows - 1) / (8 * kTileRows) * 8, kPersistent); }

// One training step is two kernels: forward and backward of the minibatch rows
// (k_mlp_rows), then the weight and bias gradients with the update
// (k_mlp_wgrad).  At 4096 rows each is a few microseconds of a chain of
// dependent loads on a mostly idle chip, so the step is bound by the number of
// kernels and by how short each chain is: a step took 150 us as nine kernels
// (three weight-gradient products of 31 us each, one wave per 16x16 tile
// waiting for each step's operands; rows 28; bias sums 16; Adam, operand
// refresh and row draws 5 each), 33.1 us as three (the update apart), 31.7 now.
// The sums over the batch keep their order
// (one accumulator per gradient entry over the whole batch): Adam's first
// steps turn a changed rounding of a small gradient into a change of the
// weights, so slices of the batch summed apart (the faster form by itself)
// moved trained weights by 1e-4 within 8 steps.

// k_mlp_rows writes the transposed BF16 operands of the weight-gradient
// products (inputs X, H1, H2 and output gradients dY, dZ2, dZ1, all
// [features][batch]) and the per-row squared error.  Loss = (1/B) sum_rows
// sum_{3 outputs} (y - t)^2.
struct TrainWs {
  unsigned short *xt, *h1t, *h2t, *dyt, *dz2t, *dz1t;  // [192|128|128|16|128|128][ld]
  float* row_loss;                                      // [B]
  int ld;                                               // B rounded up to a multiple of 32; rows past B are zero
};

// Row of the data that minibatch slot b of a step holds: counter-based
// (splitmix64 of (seed, step, slot)), or slot b itself for step < 0.
__device__ __forceinline__ int batch_row(unsigned long long seed, int step, int N, int b) {
  if (step < 0) return b;
  unsigned long long z = seed + 0x9e3779b97f4a7c15ull * ((unsigned long long)step * 0x100000001ull + (unsigned long long)b + 1);
  z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
  z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
  z ^= z >> 31;
  return (int)(z % (unsigned long long)N);
}

// Stores an LDS tile of 16 rows (stride `stride`) x ncols transposed at
// dst [ncols][ld], columns b0 .. b0 + 15: 16 bytes (8 rows of a column) a store.
__device__ __forceinline__ void store_transposed(const unsigned short* tile, int stride, int ncols, unsigned short* dst,
                                                 int ld, int b0, int tid) {
  for (int e = tid; e < 2 * ncols; e += 256) {
    const int c = e >> 1, r0 = 8 * (e & 1);
    u16x8 v;
#pragma unroll
    for (int r = 0; r < 8; ++r) v[r] = tile[(r0 + r) * stride + c];
    *(u16x8*)(dst + (size_t)c * ld + b0 + r0) = v;  // ld and b0 are multiples of 16
  }
}

// 16 rows per workgroup, each of the 4 waves computing 32 of the 128 columns
// of a layer; its weight fragments are loaded before the rows arrive.
__global__ __launch_bounds__(256) void k_mlp_rows(MlpW w, const unsigned short* __restrict__ xb,
                                                  const float* __restrict__ targets, unsigned long long seed, int step,
                                                  int N, int B, TrainWs ws) {
  __shared__ __align__(16) unsigned short xr[16 * kXs], h1[16 * kHs], h2[16 * kHs], dz2[16 * kHs], dz1[16 * kHs];
  __shared__ __align__(16) unsigned short dy[16 * 32];
  __shared__ float sq[16][4];
  __shared__ int s_idx[16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, i = lane & 15, kb = lane >> 4;
  const int b0 = blockIdx.x * 16;
  u16x8 w1[2][kIn / 32], w2[2][kHid / 32], w2t[2][kHid / 32];
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const int col = 32 * wave + 16 * t + i;
#pragma unroll
    for (int kk = 0; kk < kIn / 32; ++kk) w1[t][kk] = load8(w.w1 + (size_t)col * kIn + 32 * kk + 8 * kb);
#pragma unroll
    for (int kk = 0; kk < kHid / 32; ++kk) {
      w2[t][kk] = load8(w.w2 + (size_t)col * kHid + 32 * kk + 8 * kb);
      w2t[t][kk] = load8(w.w2t + (size_t)col * kHid + 32 * kk + 8 * kb);
    }
  }
  if (tid < 16) s_idx[tid] = b0 + tid < B ? batch_row(seed, step, N, b0 + tid) : 0;
  __syncthreads();
  // gather the 16 input rows into LDS (rows past B are zero)
  for (int e = tid; e < 16 * kIn / 8; e += 256) {
    const int r = e / (kIn / 8), c = e % (kIn / 8);
    const u16x8 v = (b0 + r < B) ? load8(xb + (size_t)s_idx[r] * kIn + 8 * c) : zero8();
    *(u16x8*)(xr + r * kXs + 8 * c) = v;
  }
  __syncthreads();
  // H1 = relu(X W1^T + b1), H2 = relu(H1 W2^T + b2): this lane's columns stay
  // in registers as the ReLU masks of the backward pass
  unsigned short m1[2][4], m2[2][4];
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const int col = 32 * wave + 16 * t + i;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kk = 0; kk < kIn / 32; ++kk) acc = mfma(*(const u16x8*)(xr + i * kXs + 32 * kk + 8 * kb), w1[t][kk], acc);
    const float b = w.b1[col];
    for (int r = 0; r < 4; ++r) h1[(4 * kb + r) * kHs + col] = m1[t][r] = f2bf(fmaxf(acc[r] + b, 0.f));
  }
  __syncthreads();
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const int col = 32 * wave + 16 * t + i;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kk = 0; kk < kHid / 32; ++kk) acc = mfma(*(const u16x8*)(h1 + i * kHs + 32 * kk + 8 * kb), w2[t][kk], acc);
    const float b = w.b2[col];
    for (int r = 0; r < 4; ++r) h2[(4 * kb + r) * kHs + col] = m2[t][r] = f2bf(fmaxf(acc[r] + b, 0.f));
  }
  __syncthreads();
  if (wave == 0) {
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kk = 0; kk < kHid / 32; ++kk)
      acc = mfma(*(const u16x8*)(h2 + i * kHs + 32 * kk + 8 * kb), load8(w.w3 + (size_t)i * kHid + 32 * kk + 8 * kb), acc);
    const float bias = w.b3[i];
    // dY = 2 (y - t) / (3 B), rows past B contribute nothing
    for (int r = 0; r < 4; ++r) {
      const int row = 4 * kb + r;
      float g = 0.f, e2 = 0.f;
      if (i < kOut && b0 + row < B) {
        const float d = acc[r] + bias - targets[(size_t)s_idx[row] * kOut + i];
        e2 = d * d;
        g = 2.f * d / (3.f * (float)B);
      }
      dy[row * 32 + i] = f2bf(g);
      dy[row * 32 + 16 + i] = 0;
      if (i < 4) sq[row][i] = i < kOut ? e2 : 0.f;
    }
  }
  __syncthreads();
  if (tid < 16 && b0 + tid < B) ws.row_loss[b0 + tid] = sq[tid][0] + sq[tid][1] + sq[tid][2];
  // dZ2 = (dY W3) * [H2 > 0]: A = dY [16][32] (columns >= 16 zero), B[o][j] = W3t[j][o]
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const int col = 32 * wave + 16 * t + i;
    const u16x8 bm = kb < 2 ? load8(w.w3t + (size_t)col * kOutPad + 8 * kb) : zero8();
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    acc = mfma(*(const u16x8*)(dy + i * 32 + 8 * kb), bm, acc);
    for (int r = 0; r < 4; ++r) dz2[(4 * kb + r) * kHs + col] = (short)m2[t][r] > 0 ? f2bf(acc[r]) : (unsigned short)0;
  }
  __syncthreads();
  // dZ1 = (dZ2 W2) * [H1 > 0]: B[m][j] = W2t[j][m]
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const int col = 32 * wave + 16 * t + i;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kk = 0; kk < kHid / 32; ++kk) acc = mfma(*(const u16x8*)(dz2 + i * kHs + 32 * kk + 8 * kb), w2t[t][kk], acc);
    for (int r = 0; r < 4; ++r) dz1[(4 * kb + r) * kHs + col] = (short)m1[t][r] > 0 ? f2bf(acc[r]) : (unsigned short)0;
  }
  __syncthreads();
  store_transposed(xr, kXs, kIn, ws.xt, ws.ld, b0, tid);
  store_transposed(h1, kHs, kHid, ws.h1t, ws.ld, b0, tid);
  store_transposed(h2, kHs, kHid, ws.h2t, ws.ld, b0, tid);
  store_transposed(dy, 32, kOutPad, ws.dyt, ws.ld, b0, tid);
  store_transposed(dz2, kHs, kHid, ws.dz2t, ws.ld, b0, tid);
  store_transposed(dz1, kHs, kHid, ws.dz1t, ws.ld, b0, tid);
}

struct Operands {
  unsigned short *w1, *w2, *w3, *w2t, *w3t;
};

__device__ __forceinline__ void refresh_operand(int t, float x, const Operands& o) {
  const unsigned short b = f2bf(x);
  if (t < kB1) {
    o.w1[t] = b;
  } else if (t >= kW2 && t < kB2) {
    const int e = t - kW2;
    o.w2[e] = b;
    o.w2t[(e % kHid) * kHid + e / kHid] = b;
  } else if (t >= kW3 && t < kB3) {
    const int e = t - kW3;
    o.w3[e] = b;
    o.w3t[(e % kHid) * kOutPad + e / kHid] = b;
  }
}

// Adam step on the FP32 master parameters, with the BF16 operand copies.
struct Adam {
  float *p, *m, *v;
  float lr, b1, b2, eps, c1, c2;
  Operands ops;
};
struct AdamState {  // of one parameter
  float p, m, v;
};
__device__ __forceinline__ AdamState load_state(const Adam& ad, int t) { return {ad.p[t], ad.m[t], ad.v[t]}; }
// The roundings of the averages are part of the definition: left to the
// compiler, a sum of two products is contracted on either side, depending on
// the code around it, and an ulp of one bias's average moved trained weights by
// 5e-5 (relative norm) within 8 steps of 4,096 rows.
__device__ __forceinline__ void adam_step(const Adam& ad, int t, const AdamState& s, float gi) {
  const float mi = __fmaf_rn(1.f - ad.b1, gi, __fmul_rn(ad.b1, s.m));
  const float vi = __fmaf_rn(gi, __fmul_rn(1.f - ad.b2, gi), __fmul_rn(ad.b2, s.v));
  ad.m[t] = mi;
  ad.v[t] = vi;
  const float x = s.p - ad.lr * (mi / ad.c1) / (sqrtf(vi / ad.c2) + ad.eps);
  ad.p[t] = x;
  refresh_operand(t, x, ad.ops);
}

// Weight gradients dW[o][c] = sum_b dZt[o][b] At[c][b], one wave per 16x16
// tile of a layer's matrix, and, in further waves, the bias gradients and the
// minibatch loss (lanes over the batch in a fixed order, then a fixed shuffle
// tree).  A tile is one chain of matrix instructions over the batch; the wave
// keeps the operands of kAhead steps of 32 rows in flight in registers, since
// a step's operands take about 40 times as long to arrive from L2 as its
// instruction takes to issue.  With TRAIN the wave that holds an entry's
// gradient updates its parameter too, whose state it has read meanwhile
// (nothing here reads the weights); without, the gradients go to grad.
constexpr int kTiles1 = (kHid / 16) * (kIn / 16), kTiles2 = (kHid / 16) * (kHid / 16), kTiles3 = kHid / 16;
constexpr int kTiles = kTiles1 + kTiles2 + kTiles3, kBiases = 2 * kHid + kOutPad;
constexpr int kAhead = 16;

template <bool TRAIN>
__global__ __launch_bounds__(64) void k_mlp_wgrad(TrainWs ws, int B, float* __restrict__ grad,
                                                  float* __restrict__ loss_out, Adam ad) {
  const int lane = threadIdx.x, i = lane & 15, kb = lane >> 4, ld = ws.ld;
  int tile = blockIdx.x;
  if (tile >= kTiles) {
    const int t = tile - kTiles;
    const int at = t < kHid ? kB1 + t : (t < 2 * kHid ? kB2 + (t - kHid) : kB3 + (t - 2 * kHid));
    AdamState state{};
    float acc = 0.f;
    if (t < kBiases) {
      if (TRAIN) state = load_state(ad, at);
      const unsigned short* src = t < kHid ? ws.dz1t + (size_t)t * ld
                                           : (t < 2 * kHid ? ws.dz2t + (size_t)(t - kHid) * ld
                                                           : ws.dyt + (size_t)(t - 2 * kHid) * ld);
#pragma unroll 16
      for (int b = lane; b < B; b += 64) acc += bf2f(src[b]);
    } else {
      if (!loss_out) return;
#pragma unroll 16
      for (int b = lane; b < B; b += 64) acc += ws.row_loss[b];
    }
    for (int off = 32; off >= 1; off >>= 1) acc += __shfl_xor(acc, off, 64);
    if (lane != 0) return;
    if (t < kBiases && TRAIN)
      adam_step(ad, at, state, acc);
    else if (t < kBiases)
      grad[at] = acc;
    else
      *loss_out = acc / (3.f * (float)B);
    return;
  }
  const unsigned short *dzt, *at;
  int ncols, ow;  // columns of the layer, offset of its weights
  if (tile < kTiles1) {
    dzt = ws.dz1t, at = ws.xt, ncols = kIn, ow = kW1;
  } else if (tile < kTiles1 + kTiles2) {
    tile -= kTiles1;
    dzt = ws.dz2t, at = ws.h1t, ncols = kHid, ow = kW2;
  } else {
    tile -= kTiles1 + kTiles2;
    dzt = ws.dyt, at = ws.h2t, ncols = kHid, ow = kW3;
  }
  const int ot = tile / (ncols / 16), ct = tile % (ncols / 16);
  const unsigned short* pa = dzt + (size_t)(16 * ot + i) * ld + 8 * kb;
  const unsigned short* pb = at + (size_t)(16 * ct + i) * ld + 8 * kb;
  const int nk = ld / 32, last = 32 * (nk - 1);
  const int out = ow + (16 * ot + 4 * kb) * ncols + 16 * ct + i;  // the lane's entries: out, out + ncols, ...
  AdamState state[4];
  if (TRAIN)
    for (int r = 0; r < 4; ++r) state[r] = load_state(ad, out + r * ncols);
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  u16x8 a[kAhead], b[kAhead];
#pragma unroll
  for (int j = 0; j < kAhead; ++j) {  // steps past the last one load it again and are not used
    a[j] = load8(pa + min(32 * j, last));
    b[j] = load8(pb + min(32 * j, last));
  }
  int k = 0;
  for (; k + kAhead <= nk; k += kAhead) {
#pragma unroll
    for (int j = 0; j < kAhead; ++j) {
      acc = mfma(a[j], b[j], acc);
      const int next = min(32 * (k + kAhead + j), last);
      a[j] = load8(pa + next);
      b[j] = load8(pb + next);
    }
  }
#pragma unroll
  for (int j = 0; j < kAhead; ++j)
    if (k + j < nk) acc = mfma(a[j], b[j], acc);
  for (int r = 0; r < 4; ++r) {
    if (TRAIN)
      adam_step(ad, out + r * ncols, state[r], acc[r]);
    else
      grad[out + r * ncols] = acc[r];
  }
}

__global__ void k_refresh_bf16(const float* __restrict__ p, Operands ops) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t < kNParams) refresh_operand(t, p[t], ops);
}

// ---------------------------------------------------------------- features

// trilinear sample of a bordered z-pair image at voxel position p clamped to [0, D-1]
typedef float float4v __attribute__((ext_vector_type(4)));

// (byte offsets fit 32 bits: an image is below 2 GiB)
__device__ __forceinline__ float sample_packed(const DevProblem& pr, __amdgpu_buffer_rsrc_t img, float px, float py, float pz) {
  px = fminf(fmaxf(px, 0.f), (float)(pr.D[0] - 1)) + 1.f;
  py = fminf(fmaxf(py, 0.f), (float)(pr.D[1] - 1)) + 1.f;
  pz = fminf(fmaxf(pz, 0.f), (float)(pr.D[2] - 1)) + 1.f;
  const int ix = (int)px, iy = (int)py, iz = (int)pz;
  const float fx = px - ix, fy = py - iy, fz = pz - iz;
  const unsigned sx8 = 8u * (unsigned)pr.ex, sxy8 = 8u * (unsigned)pr.exy;
  const int at = (int)(__umul24((unsigned)iy, sx8) + (unsigned)iz * sxy8 + ((unsigned)ix << 3));
  // e: (x,y,z),(x,y,z+1),(x+1,y,z),(x+1,y,z+1); f: the same at y+1
  const float4v e = __builtin_bit_cast(float4v, __builtin_amdgcn_raw_buffer_load_b128(img, at, 0, 0));
  const float4v f = __builtin_bit_cast(float4v, __builtin_amdgcn_raw_buffer_load_b128(img, at, (int)sx8, 0));
  const float c00 = e[0] + fx * (e[2] - e[0]), c01 = e[1] + fx * (e[3] - e[1]);
  const float c10 = f[0] + fx * (f[2] - f[0]), c11 = f[1] + fx * (f[3] - f[1]);
  const float c0 = c00 + fy * (c10 - c00), c1 = c01 + fy * (c11 - c01);
  return c0 + fz * (c1 - c0);
}

// Raw features of candidate k of single-point element f of solution s:
//   [0, 6)     candidate minus current position of the point, both grids;
//   [6, 162)   for each of the 26 grid neighbours o (dz, dy, dx in {-1,0,1},
//              dx fastest, centre skipped) and each grid: neighbour position
//              relative to the candidate minus the undeformed relative offset
//              (0 where the neighbour does not exist);
//   [162, 188) source image at (candidate + h o) minus target image at
//              (candidate + h o), h = half the undeformed cube extent per axis;
//   [188, 192) zero.
// Rows are numbered (s, f, k) with k fastest.
struct FeatureArgs {
  DevProblem pr;
  const float* X;
  int S, F, K;
  const int* pts;
  const float* cand;
  const float* ident;  // undeformed grid [P][3]
  float half[3];       // half the undeformed cube extent per axis
  int64_t N;           // rows
};

// The 64 rows of tile `tile` (rows[]: their indices, -1 past the last): the
// rows are taken with the element slowest, then the solution, then the
// candidate, and the tiles are split into 8 contiguous parts, one per XCD.  A
// tile then samples around one point or two, and the tiles that follow on the
// same XCD around the same one in other solutions, so a point's 52 sampled
// neighbourhoods (under 1 MB) come from memory once; in row order every tile
// touched the whole images, and the gathers were bound by what L2 misses: 1320
// us for 1.2 M rows at 512x512x100 in k_screen, 500 us in this order.
__device__ __forceinline__ int64_t tile_row(const FeatureArgs& a, int64_t tile, int i, int& s, int& f) {
  const int64_t q = tile * kTileRows + i;
  s = f = 0;
  if (q >= a.N) return -1;
  int k;
  if (a.N <= 0x7fffffff) {
    const unsigned fs = (unsigned)q / (unsigned)a.K;
    k = (int)((unsigned)q - fs * (unsigned)a.K);
    f = (int)(fs / (unsigned)a.S);
    s = (int)(fs - (unsigned)f * (unsigned)a.S);
  } else {
    const int64_t fs = q / a.K;
    k = (int)(q - fs * a.K);
    f = (int)(fs / a.S);
    s = (int)(fs - (int64_t)f * a.S);
  }
  return ((int64_t)s * a.F + f) * a.K + k;
}

// Tile n of those that workgroup `block` of `blocks` (a multiple of 8) takes, or -1.
__device__ __forceinline__ int64_t tile_of(int64_t tiles, int block, int blocks, int n) {
  const int x = block & 7;
  const int64_t q = tiles >> 3, r = tiles & 7, k = (block >> 3) + (int64_t)n * (blocks >> 3);
  return k < q + (x < r ? 1 : 0) ? x * q + min((int64_t)x, r) + k : -1;
}

// Features of the 64 rows of a tile (absent rows are 0), lane = row: the wave
// takes groups `first`, first + step, ... of the 28 groups of columns (26
// neighbours, the moved point, the padding) and writes lane's row to out(row).  A group's
// offsets and statistics are the same on every lane, so they are scalars, a
// row's indices are worked out once instead of once per group, and the lanes
// of one point's candidates sample next to each other (a gather of the 26
// offsets of one row touches as many cache lines as lanes).  Returns the row's
// index, -1 past the last.  With PACK the values are standardised with the stored
// input statistics and rounded to BF16, bit for bit what k_pack makes of the
// FP32 rows (sums and products are written with explicit rounding, so that
// both forms compute identical FP32 values).
template <bool PACK, class Out>
__device__ __forceinline__ int64_t feature_tile(const FeatureArgs& a, const float* __restrict__ mean,
                                                const float* __restrict__ rstd, int64_t tile_index, int first, int step,
                                                Out where) {
  const DevProblem& pr = a.pr;
  const int lane = threadIdx.x & 63;
  int s, f;
  const int64_t row = tile_row(a, tile_index, lane, s, f);
  const bool exists = row >= 0;
  auto* const out = where(row);
  if (!out) return row;
  const int p = exists ? a.pts[f] : -1;
  const bool valid = p >= 0 && p < pr.P;
  const int pc = valid ? p : 0;  // where rows without a point read
  const float* Xs = a.X + (size_t)s * 6 * pr.P;
  const unsigned pin = pr.pin[pc];
  float c[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (exists)
    for (int k = 0; k < 6; ++k) c[k] = a.cand[row * 6 + k];
  const float u[3] = {a.ident[3 * pc], a.ident[3 * pc + 1], a.ident[3 * pc + 2]};
  const __amdgpu_buffer_rsrc_t img0 = __builtin_amdgcn_make_buffer_rsrc((void*)pr.img[0], (short)0, pr.img_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t img1 = __builtin_amdgcn_make_buffer_rsrc((void*)pr.img[1], (short)0, pr.img_bytes, 0x00020000);
  auto put2 = [&](int col, float v0, float v1) {  // columns col, col + 1 (col even)
    if constexpr (PACK) {
      const unsigned lo = f2bf(__fmul_rn(__fsub_rn(v0, mean[col]), rstd[col]));
      const unsigned hi = f2bf(__fmul_rn(__fsub_rn(v1, mean[col + 1]), rstd[col + 1]));
      *reinterpret_cast<unsigned*>(out + col) = lo | (hi << 16);
    } else {
      out[col] = v0;
      out[col + 1] = v1;
    }
  };
#pragma unroll 2
  for (int j = first; j < 28; j += step) {
    if (j == 27) {
      put2(kNumFeat, 0.f, 0.f);
      put2(kNumFeat + 2, 0.f, 0.f);
      continue;
    }
    float v[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (j == 26) {
      if (valid)
        for (int g = 0; g < 2; ++g)
          for (int k = 0; k < 3; ++k) v[3 * g + k] = __fsub_rn(c[3 * g + k], Xs[((size_t)g * pr.P + p) * 3 + k]);
      for (int e = 0; e < 6; e += 2) put2(e, v[e], v[e + 1]);
      continue;
    }
    const int t = j < 13 ? j : j + 1;  // centre (13) skipped
    const int d[3] = {t % 3 - 1, (t / 3) % 3 - 1, t / 9 - 1};
    bool there = valid;
    for (int k = 0; k < 3; ++k) there = there && !(d[k] < 0 && (pin >> k & 1)) && !(d[k] > 0 && (pin >> (3 + k) & 1));
    if (there) {
      const int q = p + d[0] + pr.n[0] * (d[1] + pr.n[1] * d[2]);
      for (int g = 0; g < 2; ++g)
        for (int k = 0; k < 3; ++k)
          v[3 * g + k] = __fsub_rn(__fsub_rn(Xs[((size_t)g * pr.P + q) * 3 + k], c[3 * g + k]),
                                   __fsub_rn(a.ident[3 * q + k], u[k]));
    }
    float vi = 0.f;
    if (valid) {
      float o[3];
      for (int k = 0; k < 3; ++k) o[k] = __fmul_rn(a.half[k], (float)d[k]);
      const float im = sample_packed(pr, img0, __fadd_rn(c[0], o[0]), __fadd_rn(c[1], o[1]), __fadd_rn(c[2], o[2]));
      const float it = sample_packed(pr, img1, __fadd_rn(c[3], o[0]), __fadd_rn(c[4], o[1]), __fadd_rn(c[5], o[2]));
      vi = __fsub_rn(im, it);
    }
    for (int e = 0; e < 6; e += 2) put2(6 + 6 * j + e, v[e], v[e + 1]);
    if constexpr (PACK)
      out[162 + j] = f2bf(__fmul_rn(__fsub_rn(vi, mean[162 + j]), rstd[162 + j]));
    else
      out[162 + j] = vi;
  }
  return row;
}

// Feature rows as FP32 (out32) or standardised BF16 (out16), written from an LDS
// tile by one workgroup, or, where the grid has kFeatureParts in its second
// dimension, straight to memory with a group to a wave.
constexpr int kFeatureParts = 7;
template <bool PACK>
__global__ __launch_bounds__(256) void k_features(FeatureArgs a, const float* __restrict__ mean,
                                                  const float* __restrict__ rstd, float* __restrict__ out32,
                                                  unsigned short* __restrict__ out16) {
  using T = std::conditional_t<PACK, unsigned short, float>;
  constexpr int kStride = PACK ? kXs : kIn + 4, kPiece = 16 / sizeof(T);  // elements of a 16-byte piece
  __shared__ __align__(16) T tile[kTileRows * kStride];
  __shared__ int64_t s_row[kTileRows];
  const int64_t index = tile_of((a.N + kTileRows - 1) / kTileRows, blockIdx.x, gridDim.x, 0);
  if (index < 0) return;
  T* dst;
  if constexpr (PACK)
    dst = out16;
  else
    dst = out32;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (gridDim.y > 1) {
    feature_tile<PACK>(a, mean, rstd, index, 4 * blockIdx.y + wave, 4 * kFeatureParts,
                       [&](int64_t row) { return row >= 0 ? dst + row * kIn : nullptr; });
    return;
  }
  const int64_t row = feature_tile<PACK>(a, mean, rstd, index, wave, 4, [&](int64_t) { return tile + lane * kStride; });
  if (wave == 0) s_row[lane] = row;
  __syncthreads();
  constexpr int kPieces = kIn / kPiece;  // 16 bytes each: rows of 384 or 768 bytes
  for (int e = threadIdx.x; e < kTileRows * kPieces; e += 256) {
    const int i = e / kPieces, c = kPiece * (e % kPieces);
    if (s_row[i] >= 0) *reinterpret_cast<uint4*>(dst + s_row[i] * kIn + c) = *reinterpret_cast<const uint4*>(tile + i * kStride + c);
  }
}

// Screening: features of 64 rows into LDS and the network on them, without
// rows in memory (0.47 GB written and read again at 1.2 M candidates; the two
// kernels took 1270 and 330 us).  Three waves per SIMD leave 168 registers, of
// which the weights take 101: two values are spilled.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3, 3))) void k_screen(
    MlpW w, FeatureArgs a, const float* __restrict__ mean, const float* __restrict__ rstd, float* __restrict__ out) {
  __shared__ __align__(16) unsigned short xs[kTileRows * kXs];  // inputs, then H2
  __shared__ __align__(16) unsigned short h1[kTileRows * kHs];
  __shared__ int64_t s_row[kTileRows];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  WaveWeights ww;
  load_layer1(w, wave, lane, ww);
  load_layers23(w, wave, lane, ww);
  const int64_t tiles = (a.N + kTileRows - 1) / kTileRows;
  for (int n = 0;; ++n) {
    const int64_t tile = tile_of(tiles, blockIdx.x, gridDim.x, n);
    if (tile < 0) break;
    const int64_t row = feature_tile<true>(a, mean, rstd, tile, __builtin_amdgcn_readfirstlane(wave), 4,
                                           [&](int64_t) { return xs + lane * kXs; });
    if (wave == 0) s_row[lane] = row;
    __syncthreads();
    mlp_tile(ww, xs, h1, [&](int i) { return s_row[i]; }, out, wave, lane, [] {});
    __syncthreads();
  }
}

// Standardise FP32 rows and round to BF16 operands; optionally standardise targets.
__global__ void k_pack(int N, const float* __restrict__ feats, const float* __restrict__ mean, const float* __restrict__ rstd,
                       unsigned short* __restrict__ out) {
  const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (e >= (int64_t)N * kIn) return;
  const int c = (int)(e % kIn);
  out[e] = f2bf(__fmul_rn(__fsub_rn(feats[e], mean[c]), rstd[c]));
}

// Column mean and 1/std of N rows of width `width` (fixed-order FP64 sums, one
// workgroup per column).
__global__ __launch_bounds__(256) void k_column_stats(int N, int width, const float* __restrict__ x, float* mean,
                                                      float* rstd) {
  __shared__ double s1[256], s2[256];
  const int c = blockIdx.x, t = threadIdx.x;
  double a = 0.0, b = 0.0;
  for (int r = t; r < N; r += 256) {
    const double v = x[(size_t)r * width + c];
    a += v;
    b += v * v;
  }
  s1[t] = a;
  s2[t] = b;
  __syncthreads();
  for (int w = 128; w >= 1; w >>= 1) {
    if (t < w) {
      s1[t] += s1[t + w];
      s2[t] += s2[t + w];
    }
    __syncthreads();
  }
  if (t == 0) {
    const double m = N > 0 ? s1[0] / N : 0.0;
    const double var = N > 0 ? fmax(s2[0] / N - m * m, 0.0) : 0.0;
    mean[c] = (float)m;
    rstd[c] = var > 1e-30 ? (float)(1.0 / sqrt(var)) : 1.f;  // constant columns pass through centred
  }
}

// Raw objective deltas (part_new - part_old) of N rows, standardised.
__global__ void k_targets(int N, const double* __restrict__ old, const double* __restrict__ nw, const float* __restrict__ mean,
                          const float* __restrict__ rstd, float* __restrict__ out, float* __restrict__ raw) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= N * kOut) return;
  const float d = (float)(nw[e] - old[e]);
  if (raw) raw[e] = d;
  if (out) out[e] = (d - mean[e % kOut]) * rstd[e % kOut];
}

// Screening: per (solution, element) choose one of K candidates by predicted
// Pareto rank among the K (ties: smallest sum of standardised predictions) and
// flag it for exact evaluation iff its predicted delta would be accepted: it
// improves one objective without worsening another, or it improves one
// objective and the predicted objective vector is not dominated by any archive
// member.  The picked candidates are gathered to cand_pick [S][F][2][3].
// The archive is staged in LDS and G lanes share a pair and its rows.  A pair a
// lane leaves the device idle while each walks the archive row by row (162 us
// for 3,000 rows, however few the pairs); more lanes stage the archive more
// often and repeat the choice among the K.  The whole screening call, in us,
// with 64 / 16 / 4 lanes: 1,600 pairs and 600 rows 30 / - / 80, 32,400 pairs
// and 2,000 rows 118 / 85 / 117, 307,200 pairs and 1,200 rows 1006 / 684 / 583
// (678 with two pairs a lane).  Rows taken 4 at a time, one vote for the 4,
// took the last from 643 to 615 us on new inputs.
constexpr int kSelTile = 512;

template <int G>
__global__ __launch_bounds__(256) void k_select(int S, int F, int K, const float* __restrict__ pred_std,
                                                const float* __restrict__ out_mean, const float* __restrict__ out_scale,
                                                const double* __restrict__ obj, int n_arch,
                                                const double* __restrict__ arch, const float* __restrict__ cand,
                                                float* __restrict__ pred_raw, int* __restrict__ pick,
                                                unsigned char* __restrict__ run_exact, float* __restrict__ cand_pick) {
  __shared__ double s_a[kSelTile][3];
  __shared__ int s_end;
  const int64_t e = (blockIdx.x + (int64_t)gridDim.x * blockIdx.y) * (256 / G) + threadIdx.x / G;
  const int sub = threadIdx.x % G;
  bool accept = false, scan = false;
  double nv[kOut] = {0.0, 0.0, 0.0};
  if (e < (int64_t)S * F) {
    const float* ps = pred_std + (size_t)e * K * kOut;
    int best = 0, best_rank = 1 << 30;
    float best_sum = INFINITY;
    for (int k = 0; k < K; ++k) {
      int rank = 0;
      for (int j = 0; j < K; ++j) {
        if (j == k) continue;
        bool le = true, lt = false;
        for (int o = 0; o < kOut; ++o) {
          le = le && ps[j * kOut + o] <= ps[k * kOut + o];
          lt = lt || ps[j * kOut + o] < ps[k * kOut + o];
        }
        rank += (le && lt) ? 1 : 0;
      }
      const float sum = ps[k * kOut] + ps[k * kOut + 1] + ps[k * kOut + 2];
      if (rank < best_rank || (rank == best_rank && sum < best_sum)) {
        best = k;
        best_rank = rank;
        best_sum = sum;
      }
    }
    double d[kOut];
    for (int k = 0; k < K; ++k)
      for (int o = 0; o < kOut; ++o) {
        const float r = ps[k * kOut + o] * out_scale[o] + out_mean[o];
        if (pred_raw && sub == 0) pred_raw[((size_t)e * K + k) * kOut + o] = r;
        if (k == best) d[o] = r;
      }
    bool le = true, lt = false;
    for (int o = 0; o < kOut; ++o) {
      le = le && d[o] <= 0.0;
      lt = lt || d[o] < 0.0;
    }
    accept = le && lt;
    scan = !accept && lt && obj && n_arch > 0;
    if (scan)
      for (int o = 0; o < kOut; ++o) nv[o] = obj[(size_t)(e / F) * kOut + o] + d[o];
    if (sub == 0) pick[e] = best;
    if (cand_pick && sub == 0)
      for (int c = 0; c < 6; ++c) cand_pick[(size_t)e * 6 + c] = cand[((size_t)e * K + best) * 6 + c];
  }
  bool left = scan;  // still to be tested
  for (int a0 = 0; a0 < n_arch; a0 += kSelTile) {
    if (!__syncthreads_or(left)) break;
    const int na = min(kSelTile, n_arch - a0);
    if (threadIdx.x == 0) s_end = na;
    __syncthreads();
    for (int q = threadIdx.x; q < 3 * na; q += 256) {
      const double x = arch[3 * (size_t)a0 + q];
      s_a[q / 3][q % 3] = x;
      if (q % 3 == 0 && x == INFINITY) atomicMin(&s_end, q / 3);  // padding ends the archive
    }
    __syncthreads();
    const int end = s_end;
    bool dom = false;
    for (int q0 = sub; q0 < end; q0 += 32 * G) {
      if (!__any(left && !dom)) break;
      const int q1 = min(q0 + 32 * G, end);
      for (int q = q0; q < q1; q += 4 * G) {  // 4 rows at a time; past the end the first of them again
        double a[4][3];
#pragma unroll
        for (int u = 0; u < 4; ++u)
          for (int o = 0; o < kOut; ++o) a[u][o] = s_a[q + u * G < end ? q + u * G : q][o];
        bool le[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) le[u] = (a[u][0] <= nv[0]) & (a[u][1] <= nv[1]) & (a[u][2] <= nv[2]);
        if (__any(le[0] | le[1] | le[2] | le[3]))
#pragma unroll
          for (int u = 0; u < 4; ++u) dom |= le[u] & ((a[u][0] < nv[0]) | (a[u][1] < nv[1]) | (a[u][2] < nv[2]));
      }
    }
    dom = (__ballot(dom) >> (threadIdx.x & 63 & ~(G - 1)) & (~0ull >> (64 - G))) != 0;  // of any lane of the pair
    scan = scan && !dom;
    left = left && !dom;
    if (end < na) break;
  }
  if (sub == 0 && e < (int64_t)S * F) run_exact[e] = accept || scan ? 1 : 0;
}

}  // namespace
}  // namespace dsm

using namespace dsm;

struct dsm_surrogate {
  dsm_surrogate_desc desc{};
  int device = 0;
  int64_t step = 0;  // Adam steps taken
  float *d_params = nullptr, *d_m = nullptr, *d_v = nullptr;
  unsigned short *d_w1 = nullptr, *d_w2 = nullptr, *d_w3 = nullptr, *d_w2t = nullptr, *d_w3t = nullptr;
  float *d_in_mean = nullptr, *d_in_rstd = nullptr, *d_out_mean = nullptr, *d_out_rstd = nullptr, *d_out_scale = nullptr;
  // training workspace for max_batch rows (padded to a multiple of 32)
  int bpad = 0;
  unsigned short *d_xt = nullptr, *d_h1t = nullptr, *d_h2t = nullptr, *d_dyt = nullptr, *d_dz2t = nullptr,
                 *d_dz1t = nullptr;
  float* d_row_loss = nullptr;
  float* d_pred = nullptr;  // screening workspace [max_rows][3]
};

namespace {

thread_local std::string s_err;

dsm_status sfail(dsm_status st, const char* msg) {
  s_err = msg;
  return st;
}

MlpW weights(const dsm_surrogate* m) {
  MlpW w;
  w.w1 = m->d_w1;
  w.w2 = m->d_w2;
  w.w3 = m->d_w3;
  w.w2t = m->d_w2t;
  w.w3t = m->d_w3t;
  w.b1 = m->d_params + kB1;
  w.b2 = m->d_params + kB2;
  w.b3 = m->d_params + kB3;
  return w;
}

void free_sur(dsm_surrogate* m) {
  if (!m) return;
  void* bufs[] = {m->d_params,   m->d_m,       m->d_v,        m->d_w1,        m->d_w2,  m->d_w3,  m->d_w2t,
                  m->d_w3t,      m->d_in_mean, m->d_in_rstd,  m->d_out_mean,  m->d_out_rstd, m->d_out_scale,
                  m->d_xt,       m->d_h1t,     m->d_h2t,      m->d_dyt,       m->d_dz2t, m->d_dz1t, m->d_row_loss,
                  m->d_pred};
  for (void* b : bufs)
    if (b) (void)hipFree(b);
  delete m;
}

Operands operands(const dsm_surrogate* m) { return Operands{m->d_w1, m->d_w2, m->d_w3, m->d_w2t, m->d_w3t}; }

FeatureArgs feature_args(const dsm_problem* p, int S, const float* X, int F, const int* pts, int K, const float* cand) {
  FeatureArgs a{};
  a.pr = p->dev;
  a.X = X;
  a.S = S;
  a.F = F;
  a.K = K;
  a.pts = pts;
  a.cand = cand;
  a.ident = p->d_ident;
  for (int k = 0; k < 3; ++k) a.half[k] = (float)p->dev.D[k] / (2.f * (float)(p->dev.n[k] - 1));
  a.N = (int64_t)S * F * K;
  return a;
}

// Grid of k_features for n rows: a workgroup per tile of 64 rows (a multiple of
// 8), or kFeatureParts while the tiles are too few to hide the 7 groups that a
// wave of a tile takes one after the other.  A call by itself in us, one
// workgroup / parts: 2,048 rows 18.2 / 14.9, BF16 8,192 19.0 / 15.8 and 16,038
// 20.3 / 19.8, FP32 8,192 18.7 / 17.5 and 11,664 20.0 / 20.7.
dim3 features_grid(int64_t n, bool packed) {
  return dim3((unsigned)((n + 8 * kTileRows - 1) / (8 * kTileRows) * 8), n <= (packed ? 16384 : 8192) ? kFeatureParts : 1);
}

hipError_t refresh(dsm_surrogate* m, hipStream_t st) {
  k_refresh_bf16<<<(kNParams + 255) / 256, 256, 0, st>>>(m->d_params, operands(m));
  return hipGetLastError();
}

// Forward and backward of B rows (those of minibatch `step` of the N rows, or
// rows 0..B-1 for step < 0); writes the gradient to grad and the loss to loss (or null).
hipError_t gradient_pass(dsm_surrogate* m, const unsigned short* feats, const float* targets, int step, int N, int B,
                         float* loss, float* grad, const Adam* ad, hipStream_t st) {
  const int ld = (B + 31) / 32 * 32;
  TrainWs ws{m->d_xt, m->d_h1t, m->d_h2t, m->d_dyt, m->d_dz2t, m->d_dz1t, m->d_row_loss, ld};
  k_mlp_rows<<<ld / 16, 256, 0, st>>>(weights(m), feats, targets, m->desc.seed, step, N, B, ws);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (ad)
    k_mlp_wgrad<true><<<kTiles + kBiases + 1, 64, 0, st>>>(ws, B, nullptr, loss, *ad);
  else
    k_mlp_wgrad<false><<<kTiles + kBiases + 1, 64, 0, st>>>(ws, B, grad, loss, Adam{});
  return hipGetLastError();
}

}  // namespace

extern "C" {

const char* dsm_surrogate_last_error(void) { return s_err.c_str(); }

dsm_status dsm_surrogate_create(const dsm_surrogate_desc* d, dsm_surrogate** out) {
  s_err.clear();
  if (!out || !d) return sfail(DSM_ERR_ARG, "null argument");
  *out = nullptr;
  if (d->max_rows < 1 || d->max_batch < 32 || d->max_batch % 32 != 0)
    return sfail(DSM_ERR_ARG, "max_rows >= 1 and max_batch a positive multiple of 32 required");
  if (!(d->lr > 0.f) || !(d->beta1 >= 0.f && d->beta1 < 1.f) || !(d->beta2 >= 0.f && d->beta2 < 1.f) || !(d->eps > 0.f))
    return sfail(DSM_ERR_ARG, "bad Adam hyper-parameters");
  auto* m = new dsm_surrogate();
  m->desc = *d;
  m->bpad = d->max_batch;
  hipError_t e = hipGetDevice(&m->device);
#define S_TRY(expr)                                   \
  if (e == hipSuccess) e = (expr);                    \
  if (e != hipSuccess) {                              \
    free_sur(m);                                      \
    return sfail(e == hipErrorOutOfMemory ? DSM_ERR_NOMEM : DSM_ERR_DEVICE, hipGetErrorString(e)); \
  }
  S_TRY(hipMalloc(&m->d_params, sizeof(float) * kNParams));
  S_TRY(hipMalloc(&m->d_m, sizeof(float) * kNParams));
  S_TRY(hipMalloc(&m->d_v, sizeof(float) * kNParams));
  S_TRY(hipMalloc(&m->d_w1, 2 * kHid * kIn));
  S_TRY(hipMalloc(&m->d_w2, 2 * kHid * kHid));
  S_TRY(hipMalloc(&m->d_w3, 2 * kOutPad * kHid));
  S_TRY(hipMalloc(&m->d_w2t, 2 * kHid * kHid));
  S_TRY(hipMalloc(&m->d_w3t, 2 * kOutPad * kHid));
  S_TRY(hipMalloc(&m->d_in_mean, sizeof(float) * kIn));
  S_TRY(hipMalloc(&m->d_in_rstd, sizeof(float) * kIn));
  S_TRY(hipMalloc(&m->d_out_mean, sizeof(float) * kOut));
  S_TRY(hipMalloc(&m->d_out_rstd, sizeof(float) * kOut));
  S_TRY(hipMalloc(&m->d_out_scale, sizeof(float) * kOut));
  const size_t B = m->bpad;
  S_TRY(hipMalloc(&m->d_xt, 2 * kIn * B));
  S_TRY(hipMalloc(&m->d_h1t, 2 * kHid * B));
  S_TRY(hipMalloc(&m->d_h2t, 2 * kHid * B));
  S_TRY(hipMalloc(&m->d_dyt, 2 * kOutPad * B));
  S_TRY(hipMalloc(&m->d_dz2t, 2 * kHid * B));
  S_TRY(hipMalloc(&m->d_dz1t, 2 * kHid * B));
  S_TRY(hipMalloc(&m->d_row_loss, sizeof(float) * B));
  S_TRY(hipMalloc(&m->d_pred, sizeof(float) * kOut * (size_t)d->max_rows));
  // He-uniform initial weights, zero biases (host, from the seed); identity scaling
  std::vector<float> p(kNParams, 0.f);
  unsigned long long z = d->seed;
  auto next = [&z]() {
    z += 0x9e3779b97f4a7c15ull;
    unsigned long long x = z;
    x = (x ^ (x >> 30)) * 0xbf58476d1ce4e5b9ull;
    x = (x ^ (x >> 27)) * 0x94d049bb133111ebull;
    x ^= x >> 31;
    return (double)(x >> 11) * (1.0 / 9007199254740992.0);
  };
  auto fill = [&](int off, int rows, int cols, int fan_in) {
    const double lim = sqrt(6.0 / fan_in);
    for (int r = 0; r < rows; ++r)
      for (int c = 0; c < cols; ++c) p[off + r * cols + c] = (float)((2.0 * next() - 1.0) * lim);
  };
  fill(kW1, kHid, kIn, kIn);
  fill(kW2, kHid, kHid, kHid);
  fill(kW3, kOut, kHid, kHid);  // output rows 3..15 stay zero
  S_TRY(hipMemcpy(m->d_params, p.data(), sizeof(float) * kNParams, hipMemcpyHostToDevice));
  S_TRY(hipMemset(m->d_m, 0, sizeof(float) * kNParams));
  S_TRY(hipMemset(m->d_v, 0, sizeof(float) * kNParams));
  std::vector<float> zeros(kIn, 0.f), ones(kIn, 1.f);
  S_TRY(hipMemcpy(m->d_in_mean, zeros.data(), sizeof(float) * kIn, hipMemcpyHostToDevice));
  S_TRY(hipMemcpy(m->d_in_rstd, ones.data(), sizeof(float) * kIn, hipMemcpyHostToDevice));
  S_TRY(hipMemcpy(m->d_out_mean, zeros.data(), sizeof(float) * kOut, hipMemcpyHostToDevice));
  S_TRY(hipMemcpy(m->d_out_rstd, ones.data(), sizeof(float) * kOut, hipMemcpyHostToDevice));
  S_TRY(hipMemcpy(m->d_out_scale, ones.data(), sizeof(float) * kOut, hipMemcpyHostToDevice));
  S_TRY(refresh(m, nullptr));
  S_TRY(hipDeviceSynchronize());
#undef S_TRY
  *out = m;
  return DSM_OK;
}

dsm_status dsm_surrogate_destroy(dsm_surrogate* m) {
  s_err.clear();
  if (!m) return sfail(DSM_ERR_ARG, "null surrogate");
  free_sur(m);
  return DSM_OK;
}

dsm_status dsm_surrogate_params(dsm_surrogate* m, float* host, int32_t set) {
  s_err.clear();
  if (!m || !host) return sfail(DSM_ERR_ARG, "null argument");
  hipError_t e;
  if (set) {
    e = hipMemcpy(m->d_params, host, sizeof(float) * kNParams, hipMemcpyHostToDevice);
    if (e == hipSuccess) e = refresh(m, nullptr);
    if (e == hipSuccess) e = hipDeviceSynchronize();
  } else {
    e = hipMemcpy(host, m->d_params, sizeof(float) * kNParams, hipMemcpyDeviceToHost);
  }
  return e == hipSuccess ? DSM_OK : sfail(DSM_ERR_DEVICE, hipGetErrorString(e));
}

dsm_status dsm_surrogate_fit_scaling(dsm_surrogate* m, int32_t N, const float* feats, const float* deltas, void* stream) {
  s_err.clear();
  if (!m || !feats || !deltas || N < 1) return sfail(DSM_ERR_ARG, "null argument or N < 1");
  hipStream_t st = (hipStream_t)stream;
  k_column_stats<<<kIn, 256, 0, st>>>(N, kIn, feats, m->d_in_mean, m->d_in_rstd);
  k_column_stats<<<kOut, 256, 0, st>>>(N, kOut, deltas, m->d_out_mean, m->d_out_rstd);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return sfail(DSM_ERR_DEVICE, hipGetErrorString(e));
  // output scale = 1 / rstd (so that raw = std_pred * scale + mean)
  std::vector<float> r(kOut);
  e = hipMemcpyAsync(r.data(), m->d_out_rstd, sizeof(float) * kOut, hipMemcpyDeviceToHost, st);
  if (e == hipSuccess) e = hipStreamSynchronize(st);
  for (float& x : r) x = 1.f / x;
  if (e == hipSuccess) e = hipMemcpy(m->d_out_scale, r.data(), sizeof(float) * kOut, hipMemcpyHostToDevice);
  return e == hipSuccess ? DSM_OK : sfail(DSM_ERR_DEVICE, hipGetErrorString(e));
}

dsm_status dsm_surrogate_get_scaling(dsm_surrogate* m, float* in_mean, float* in_rstd, float* out_mean, float* out_rstd) {
  s_err.clear();
  if (!m) return sfail(DSM_ERR_ARG, "null surrogate");
  hipError_t e = hipSuccess;
  if (in_mean) e = hipMemcpy(in_mean, m->d_in_mean, sizeof(float) * kIn, hipMemcpyDeviceToHost);
  if (e == hipSuccess && in_rstd) e = hipMemcpy(in_rstd, m->d_in_rstd, sizeof(float) * kIn, hipMemcpyDeviceToHost);
  if (e == hipSuccess && out_mean) e = hipMemcpy(out_mean, m->d_out_mean, sizeof(float) * kOut, hipMemcpyDeviceToHost);
  if (e == hipSuccess && out_rstd) e = hipMemcpy(out_rstd, m->d_out_rstd, sizeof(float) * kOut, hipMemcpyDeviceToHost);
  return e == hipSuccess ? DSM_OK : sfail(DSM_ERR_DEVICE, hipGetErrorString(e));
}

dsm_status dsm_surrogate_set_scaling(dsm_surrogate* m, const float* in_mean, const float* in_rstd, const float* out_mean,
                                     const float* out_rstd) {
  s_err.clear();
  if (!m || !in_mean || !in_rstd || !out_mean || !out_rstd) return sfail(DSM_ERR_ARG, "null argument");
  hipError_t e = hipMemcpy(m->d_in_mean, in_mean, sizeof(float) * kIn, hipMemcpyHostToDevice);
  if (e == hipSuccess) e = hipMemcpy(m->d_in_rstd, in_rstd, sizeof(float) * kIn, hipMemcpyHostToDevice);
  if (e == hipSuccess) e = hipMemcpy(m->d_out_mean, out_mean, sizeof(float) * kOut, hipMemcpyHostToDevice);
  if (e == hipSuccess) e = hipMemcpy(m->d_out_rstd, out_rstd, sizeof(float) * kOut, hipMemcpyHostToDevice);
  float sc[kOut];
  for (int o = 0; o < kOut; ++o) sc[o] = 1.f / out_rstd[o];
  if (e == hipSuccess) e = hipMemcpy(m->d_out_scale, sc, sizeof(float) * kOut, hipMemcpyHostToDevice);
  return e == hipSuccess ? DSM_OK : sfail(DSM_ERR_DEVICE, hipGetErrorString(e));
}

dsm_status dsm_surrogate_features(dsm_problem* p, int32_t S, const float* X, int32_t F, const int32_t* fos_pts, int32_t K,
                                  const float* cand, float* feats, void* stream) {
  s_err.clear();
  if (!p || S < 0 || F < 0 || K < 1) return sfail(DSM_ERR_ARG, "null problem or bad sizes");
  const int64_t n = (int64_t)S * F * K;
  if (n == 0) return DSM_OK;
  if (!X || !fos_pts || !cand || !feats) return sfail(DSM_ERR_ARG, "null argument");
  k_features<false><<<features_grid(n, false), 256, 0, (hipStream_t)stream>>>(
      feature_args(p, S, X, F, fos_pts, K, cand), nullptr, nullptr, feats, nullptr);
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? DSM_OK : sfail(DSM_ERR_DEVICE, hipGetErrorString(e));
}

dsm_status dsm_surrogate_features_packed(dsm_surrogate* m, dsm_problem* p, int32_t S, const float* X, int32_t F,
                                         const int32_t* fos_pts, int32_t K, const float* cand, uint16_t* feats_bf16,
                                         void* stream) {
  s_err.clear();
  if (!m || !p || S < 0 || F < 0 || K < 1) return sfail(DSM_ERR_ARG, "null argument or bad sizes");
  const int64_t n = (int64_t)S * F * K;
  if (n == 0) return DSM_OK;
  if (!X || !fos_pts || !cand || !feats_bf16) return sfail(DSM_ERR_ARG, "null argument");
  k_features<true><<<features_grid(n, true), 256, 0, (hipStream_t)stream>>>(
      feature_args(p, S, X, F, fos_pts, K, cand), m->d_in_mean, m->d_in_rstd, nullptr, (unsigned short*)feats_bf16);
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? DSM_OK : sfail(DSM_ERR_DEVICE, hipGetErrorString(e));
}

dsm_status dsm_surrogate_pack(dsm_surrogate* m, int32_t N, const float* feats, uint16_t* feats_bf16, const double* part_old,
                              const double* part_new, float* targets, float* raw_deltas, void* stream) {
  s_err.clear();
  if (!m || N < 0) return sfail(DSM_ERR_ARG, "null surrogate or N < 0");
  if (N == 0) return DSM_OK;
  hipStream_t st = (hipStream_t)stream;
  if (feats && feats_bf16)
    k_pack<<<(unsigned)(((int64_t)N * kIn + 255) / 256), 256, 0, st>>>(N, feats, m->d_in_mean, m->d_in_rstd, feats_bf16);
  if (part_old && part_new && (targets || raw_deltas))
    k_targets<<<(N * kOut + 255) / 256, 256, 0, st>>>(N, part_old, part_new, m->d_out_mean, m->d_out_rstd, targets,
                                                       raw_deltas);
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? DSM_OK : sfail(DSM_ERR_DEVICE, hipGetErrorString(e));
}

dsm_status dsm_surrogate_forward(dsm_surrogate* m, int32_t N, const uint16_t* feats_bf16, float* pred, void* stream) {
  s_err.clear();
  if (!m || !feats_bf16 || !pred || N < 0) return sfail(DSM_ERR_ARG, "null argument");
  if (N == 0) return DSM_OK;
  if (N <= kPersistent * kTileRows)
    k_mlp_forward_once<<<(N + kTileRows - 1) / kTileRows, 256, 0, (hipStream_t)stream>>>(weights(m), (const unsigned short*)feats_bf16,
                                                                                        N, pred);
  else
    k_mlp_forward<<<mlp_grid(N), 256, 0, (hipStream_t)stream>>>(weights(m), (const unsigned short*)feats_bf16, N, pred);
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? DSM_OK : sfail(DSM_ERR_DEVICE, hipGetErrorString(e));
}

dsm_status dsm_surrogate_gradient(dsm_surrogate* m, int32_t N, const uint16_t* feats_bf16, const float* targets, float* grad,
                                  float* loss, void* stream) {
  s_err.clear();
  if (!m || !feats_bf16 || !targets || !grad) return sfail(DSM_ERR_ARG, "null argument");
  if (N < 1 || N > m->bpad) return sfail(DSM_ERR_CAPACITY, "N outside [1, max_batch]");
  hipStream_t st = (hipStream_t)stream;
  const hipError_t e = gradient_pass(m, (const unsigned short*)feats_bf16, targets, -1, N, N, loss, grad, nullptr, st);
  return e == hipSuccess ? DSM_OK : sfail(DSM_ERR_DEVICE, hipGetErrorString(e));
}

dsm_status dsm_surrogate_train(dsm_surrogate* m, int32_t N, const uint16_t* feats_bf16, const float* targets, int32_t steps,
                               int32_t batch, float* loss, void* stream) {
  s_err.clear();
  if (!m || !feats_bf16 || !targets || N < 1 || steps < 0) return sfail(DSM_ERR_ARG, "null argument or bad sizes");
  if (batch < 1 || batch > m->bpad || batch % 32 != 0)
    return sfail(DSM_ERR_CAPACITY, "batch must be a multiple of 32 within max_batch");
  hipStream_t st = (hipStream_t)stream;
  hipError_t e = hipSuccess;
  for (int k = 0; k < steps && e == hipSuccess; ++k) {
    const double n = (double)(m->step + 1);
    const Adam ad{m->d_params, m->d_m, m->d_v, m->desc.lr, m->desc.beta1, m->desc.beta2, m->desc.eps,
                  1.f - powf(m->desc.beta1, (float)n), 1.f - powf(m->desc.beta2, (float)n), operands(m)};
    e = gradient_pass(m, (const unsigned short*)feats_bf16, targets, (int)m->step, N, batch, loss ? loss + k : nullptr,
                      nullptr, &ad, st);
    if (e == hipSuccess) m->step++;
  }
  return e == hipSuccess ? DSM_OK : sfail(DSM_ERR_DEVICE, hipGetErrorString(e));
}

dsm_status dsm_surrogate_screen(dsm_surrogate* m, dsm_problem* p, int32_t S, const float* X, int32_t F, const int32_t* fos_pts,
                                int32_t K, const float* cand, const double* obj, int32_t n_archive, const double* archive,
                                float* pred, int32_t* pick, uint8_t* run_exact, float* cand_pick, void* stream) {
  s_err.clear();
  if (!m || !p || !X || !fos_pts || !cand || !pick || !run_exact) return sfail(DSM_ERR_ARG, "null argument");
  if (S < 0 || F < 0 || K < 1 || n_archive < 0 || (n_archive > 0 && !archive)) return sfail(DSM_ERR_ARG, "bad sizes");
  const int64_t n = (int64_t)S * F * K;
  if (n > m->desc.max_rows) return sfail(DSM_ERR_CAPACITY, "S*F*K exceeds max_rows");
  if (n == 0) return DSM_OK;
  hipStream_t st = (hipStream_t)stream;
  k_screen<<<mlp_grid(n), 256, 0, st>>>(weights(m), feature_args(p, S, X, F, fos_pts, K, cand), m->d_in_mean, m->d_in_rstd,
                                        m->d_pred);
  const int64_t pairs = (int64_t)S * F;
  auto select = [&](auto* kernel, int lanes) {
    kernel<<<wide_grid((pairs * lanes + 255) / 256), 256, 0, st>>>(S, F, K, m->d_pred, m->d_out_mean, m->d_out_scale,
                                                                    obj, n_archive, archive, cand, pred, pick, run_exact,
                                                                    cand_pick);
  };
  if (pairs <= 4096)
    select(k_select<64>, 64);
  else if (pairs <= 65536)
    select(k_select<16>, 16);
  else
    select(k_select<4>, 4);
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? DSM_OK : sfail(DSM_ERR_DEVICE, hipGetErrorString(e));
}

}  // extern "C"
