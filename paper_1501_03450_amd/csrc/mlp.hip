// Spin surrogate network: MLP n_in -> 256 -> 256 -> 256 -> 4 with SiLU
// activations and a normalised output q = y/|y|, trained on the mean squared
// error against one-turn quaternions with Adam.
//
// The two 256×256 layers run on the matrix cores: bf16 operands, fp32
// accumulation, v_mfma_f32_16x16x32_bf16 (A[i][k] in lane i + 16(k/8),
// element k%8; B[k][j] in lane j + 16(k/8); D[i][j] in lane j + 16(i/4),
// element i%4), with the weights as A and the samples as columns of B.  The
// n_in -> 256 layer (and its recomputation and weight gradient in the backward
// pass) runs on the fp32 matrix cores, v_mfma_f32_16x16x4_f32 (A[i][k] in lane
// i + 16k, B[k][j] in lane j + 16k, D as above), so its operands stay fp32.
// The 256 -> 4 layer and its weight gradient use the bf16 matrix cores with the
// fp32 operand (W4, dL/dy) split into three bf16 parts whose sum is exact, so
// those products keep fp32 precision too.
//
// Kernels:
//   infer          all four layers fused, W2 and W3 in registers, activations
//                  kept in LDS
//   train_forward  the same with the loss and dL/dy; stores h1, h2 and dz3
//                  (sample-major) for the weight gradients, silu'(z2) and dz3
//                  for the backward half, and forms the per-workgroup partial
//                  sums of the b3, W4 and b4 gradients
//   train_backward dz3 -> dz2 -> dz1 through W3ᵀ and W2ᵀ in registers, z1
//                  recomputed by the forward half's products; stores dz2 and
//                  forms the partial sums of the b2, b1 and W1 gradients
//   weight_grad    dW2, dW3 = dzᵀ h as split-K MFMA GEMMs over the batch
//   reduce         fixed-order sum of the partials (deterministic)
//   adam           fp32 master weights, then the bf16 copies W and Wᵀ
#include <hip/hip_runtime.h>
#include <hip/hip_bf16.h>

#include <algorithm>
#include <type_traits>

#include "mlp_kernels.h"

namespace st {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

constexpr int W = kMlpWidth;       // 256
constexpr int LDA = W + 8;         // padded LDS row (bf16 elements)
constexpr int NT = 256;            // threads of a weight-gradient workgroup

// σ(z) = 1/(1 + e^-z) with the hardware exponential and reciprocal
// (about 1 ulp each): the activations are rounded to bf16 right after.
__device__ __forceinline__ float sigmoid(float z) {
  return __builtin_amdgcn_rcpf(1.0f + __expf(-z));
}
__device__ __forceinline__ float silu(float z) { return z * sigmoid(z); }
__device__ __forceinline__ float dsilu(float z) {
  const float s = sigmoid(z);
  return s * (1.0f + z * (1.0f - s));
}

__device__ __forceinline__ void zero_acc(f32x4 acc[4][4]) {
#pragma unroll
  for (int mt = 0; mt < 4; ++mt)
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) acc[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
}

// Part `part` (0, 1 or 2) of v split into three bf16 values that sum to v
// exactly: hi = bf16(v), mid = bf16(v - hi), lo = v - hi - mid (each
// difference is exact in fp32, and the last fits in bf16).
__device__ __forceinline__ __bf16 split3(float v, int part) {
  const __bf16 hi = (__bf16)v;
  if (part == 0) return hi;
  const float r = v - (float)hi;
  const __bf16 mid = (__bf16)r;
  if (part == 1) return mid;
  return (__bf16)(r - (float)mid);
}

// Layout of the bf16 copies of a 256×256 matrix: the order in which the waves of
// a workgroup hold it in registers.  Wave n / 32 takes 32 rows as two 16-row
// operand tiles whose rows are interleaved by four, so that a lane's accumulators
// are eight consecutive rows' (features) of one column (sample), one 16-byte
// store; the operands of a (wave, tile, 32-step of k) are 1 KB in lane order.
// Read from row-major copies, 64 bytes of 16 rows per load, the 256 KB took 18000
// cycles per CU.
__device__ __forceinline__ int weight_at(int n, int k) {
  const int r = 4 * (n >> 3 & 3) + (n & 3), ft = n >> 2 & 1;
  return (((n >> 5) * 16 + ft * 8 + (k >> 5)) * 64 + r + 16 * (k >> 3 & 3)) * 8 + (k & 7);
}
// the row of lane r's operand in tile ft of a wave's rows
__device__ __forceinline__ int wave_row(int n_base, int ft, int r) {
  return n_base + 8 * (r >> 2) + 4 * ft + (r & 3);
}
__device__ __forceinline__ void load_weights(bf16x8 (&w)[2][8], const __bf16* src, int wv, int lane) {
  const __bf16* p = src + wv * 32 * W;
#pragma unroll
  for (int ft = 0; ft < 2; ++ft)
#pragma unroll
    for (int k = 0; k < 8; ++k)
      w[ft][k] = *reinterpret_cast<const bf16x8*>(p + (unsigned)(((ft * 8 + k) * 64 + lane) * 8));
}

// acc = rows of w times the 256 inputs of a sample (row: the lane's sample, from
// its first k on)
__device__ __forceinline__ void wave_gemm(const bf16x8 (&w)[2][8], const __bf16* row, f32x4 (&acc)[2]) {
#pragma unroll
  for (int ft = 0; ft < 2; ++ft) acc[ft] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const bf16x8 x = *reinterpret_cast<const bf16x8*>(row + 32 * k);
#pragma unroll
    for (int ft = 0; ft < 2; ++ft)
      acc[ft] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[ft][k], x, acc[ft], 0, 0, 0);
  }
}

// Inference.  One persistent workgroup per compute unit, eight waves; wave wv
// holds rows 32 wv .. 32 wv + 31 of W2 and W3 in registers (128 of them) for
// all its tiles, so that the weights cross L2 once per launch instead of once per
// tile.  Layer 3 of a tile runs beside layer 1 of the next, layer 2 of that beside layer
// 4: two barriers per tile, and work for both the matrix cores and the vector units
// between them.  What bounds it is vector issue, most of it the activation
// (exponential and reciprocal at a fraction of the vector rate): 129 of the 204
// cycles a sample takes on a CU (counters).  2^21 samples: 1256 -> 716 us against a
// workgroup per tile with the weights read from L2 by every tile.
constexpr int kInferWaves = 8;
constexpr int64_t kMlpCus = 256;

template <int TILES>       // samples per tile / 16
__device__ __forceinline__ void infer_hidden(const bf16x8 (&w)[2][8], const float (&bias)[8],
                                             const __bf16* in, __bf16* out, int f0, int lane) {
  const int r = lane & 15, g = lane >> 4;
#pragma unroll
  for (int st = 0; st < TILES; ++st) {
    f32x4 acc[2];
    wave_gemm(w, in + (st * 16 + r) * LDA + 8 * g, acc);
    bf16x8 h;
#pragma unroll
    for (int e = 0; e < 8; ++e) h[e] = (__bf16)silu(acc[e >> 2][e & 3] + bias[e]);
    *reinterpret_cast<bf16x8*>(out + (st * 16 + r) * LDA + f0) = h;
  }
}

template <int TILES>
__global__ void __launch_bounds__(64 * kInferWaves) __attribute__((amdgpu_waves_per_eu(2, 2)))
mlp_infer_kernel(const MlpArgs a) {
  constexpr int M = 16 * TILES, XS = kMlpMaxIn + 1, NTH = 64 * kInferWaves;
  __shared__ __align__(16) __bf16 h1[M * LDA], h2[M * LDA], h3[M * LDA], w4[16 * LDA];
  __shared__ float xs[4][M][XS];
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 15, g = lane >> 4, n_base = 32 * wv, f0 = n_base + 8 * g, nin = a.n_in;
  const int64_t B = a.batch, tiles = (B + M - 1) / M;
  const int count = (int)((tiles - blockIdx.x + gridDim.x - 1) / gridDim.x);
  const float* P = a.params;
  const int xm = tid / kMlpMaxIn, xk = tid % kMlpMaxIn;
  auto load_x = [&](int i) {        // this thread's input of the block's i-th tile
    const int64_t m = ((int64_t)blockIdx.x + (int64_t)i * gridDim.x) * M + xm;
    return i < count && xm < M && m < B && xk < nin ? a.x[m * nin + xk] : 0.0f;
  };
  float x_next = load_x(0);
  float b1[8], b2[8], b3[8], w1[2][2];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    b1[e] = P[a.off.b1 + f0 + e];
    b2[e] = P[a.off.b2 + f0 + e];
    b3[e] = P[a.off.b3 + f0 + e];
  }
#pragma unroll
  for (int ft = 0; ft < 2; ++ft)
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const float v = P[a.off.W1 + wave_row(n_base, ft, r) * nin + min(4 * q + g, nin - 1)];
      w1[ft][q] = 4 * q + g < nin ? v : 0.0f;
    }
  const bf16x8 w4_piece = *reinterpret_cast<const bf16x8*>(a.W4s + tid * 8);
  // (loads arrive in order: what the first layer needs ahead of the weights)
  __builtin_amdgcn_sched_barrier(0);
  bf16x8 w2[2][8], w3[2][8];
  load_weights(w2, a.W2b, wv, lane);
  load_weights(w3, a.W3b, wv, lane);
  __builtin_amdgcn_sched_barrier(0);
  *reinterpret_cast<bf16x8*>(w4 + tid / 32 * LDA + tid % 32 * 8) = w4_piece;
  auto layer1 = [&](int slot) {
#pragma unroll
    for (int st = 0; st < TILES; ++st) {
      const float x0 = xs[slot][st * 16 + r][g], x1 = xs[slot][st * 16 + r][4 + g];
      bf16x8 h;
#pragma unroll
      for (int ft = 0; ft < 2; ++ft) {
        f32x4 d = {0.f, 0.f, 0.f, 0.f};
        d = __builtin_amdgcn_mfma_f32_16x16x4f32(w1[ft][0], x0, d, 0, 0, 0);
        d = __builtin_amdgcn_mfma_f32_16x16x4f32(w1[ft][1], x1, d, 0, 0, 0);
#pragma unroll
        for (int e = 0; e < 4; ++e) h[4 * ft + e] = (__bf16)silu(d[e] + b1[4 * ft + e]);
      }
      *reinterpret_cast<bf16x8*>(h1 + (st * 16 + r) * LDA + f0) = h;
    }
  };
  // wave wv < TILES: 16 samples; lane groups 0, 1 and 2 hold the three parts of
  // the four outputs, and group 0 finishes
  auto layer4 = [&](int i) {
    const __bf16* row = h3 + (wv * 16 + r) * LDA + 8 * g;
    f32x4 y = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < 8; ++k)
      y = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
          *reinterpret_cast<const bf16x8*>(w4 + r * LDA + 32 * k + 8 * g),
          *reinterpret_cast<const bf16x8*>(row + 32 * k), y, 0, 0, 0);
    const float* x = xs[i & 3][wv * 16 + r];
    float u[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float mid = __shfl(y[j], lane + 16, 64), lo = __shfl(y[j], lane + 32, 64);
      const float yj = P[a.off.b4 + j] + ((y[j] + mid) + lo);
      float base = a.out_ref[j];
#pragma unroll
      for (int k = 0; k < kMlpMaxIn; ++k) base = fmaf(a.out_lin[j][k], x[k], base);
      u[j] = fmaf(a.out_scale[j], yj, base);
    }
    const float inv = 1.0f / sqrtf(u[0] * u[0] + u[1] * u[1] + u[2] * u[2] + u[3] * u[3]);
    const int64_t m = ((int64_t)blockIdx.x + (int64_t)i * gridDim.x) * M + wv * 16 + r;
    if (lane < 16 && m < B)
#pragma unroll
      for (int j = 0; j < 4; ++j) a.q_out[m * 4 + j] = u[j] * inv;
  };
  if (xm < M) xs[0][xm][xk] = x_next;
  x_next = load_x(1);
  __syncthreads();
  layer1(0);
  if (xm < M) xs[1][xm][xk] = x_next;
  __syncthreads();
  infer_hidden<TILES>(w2, b2, h1, h2, f0, lane);
  __syncthreads();
  for (int i = 0; i < count; ++i) {
    x_next = load_x(i + 2);
    infer_hidden<TILES>(w3, b3, h2, h3, f0, lane);
    if (i + 1 < count) layer1((i + 1) & 3);
    __syncthreads();
    if (i + 1 < count) infer_hidden<TILES>(w2, b2, h1, h2, f0, lane);
    if (wv < TILES) layer4(i);
    if (xm < M) xs[(i + 2) & 3][xm][xk] = x_next;
    __syncthreads();
  }
}

// Training, forward half.  The workgroups, waves and weights in registers are
// those of inference; the rows of a wave's two weight tiles are interleaved so
// that a lane ends up with eight consecutive features of one sample (f0 ..
// f0 + 7): one 16-byte store to LDS and to HBM (sample-major, as the weight
// gradients read them) per 16 samples.  silu'(z2) goes to HBM in the order the
// backward half's lanes read it, silu'(z3) stays in registers until the tile's
// dL/dy is there, one barrier later; h3 is kept that long for the W4 gradient.
// The b3, W4 and b4 gradients and the loss are summed over the workgroup's tiles
// (at most kTrainTiles, which bounds the length of the sums).  What bounds it is
// vector issue: 7100 of the 13300 cycles that a tile of 65536 samples has on each
// SIMD, the weights' load included (counters).
// A tile of 32 takes all 256 registers and 12 B of scratch a lane; tiles of 64
// samples 536 B (97 us against 57).  Both halves, 65536 samples: 146 us in one kernel
// that read four weight matrices from L2 for every tile -> 98; 1000 samples: 54 ->
// 22.
constexpr int kTrainTile = 32, kTrainTiles = 16;

// Four rows (p, p + ld, ..) of 16 columns, transposed on the way out of LDS: the
// lanes of a 16-lane group address the rows' four-element pieces in order, and
// each gets its column's four elements.
typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) i16x4 lds_i16x4;
__device__ __forceinline__ bf16x4 read_columns(const __bf16* m, int ld, int row, int col, int lane) {
  const int t = lane & 15;
  const __bf16* p = m + (row + (t >> 2)) * ld + col + 4 * (t & 3);
  return __builtin_bit_cast(bf16x4, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)p));
}
// A matrix operand whose k runs down the rows: rows row + 8 g .. + 7 of column
// col + r for lane r + 16 g.
__device__ __forceinline__ bf16x8 read_operand(const __bf16* m, int ld, int row, int col, int lane) {
  const int g = lane >> 4;
  const bf16x4 lo = read_columns(m, ld, row + 8 * g, col, lane);
  const bf16x4 hi = read_columns(m, ld, row + 8 * g + 4, col, lane);
  return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}

__global__ void __launch_bounds__(64 * kInferWaves) __attribute__((amdgpu_waves_per_eu(2, 2)))
mlp_train_forward_kernel(const MlpArgs a) {
  constexpr int M = kTrainTile, TILES = M / 16, XS = kMlpMaxIn + 1, LDY = M + 8;
  __shared__ __align__(16) __bf16 h1[M * LDA], h2[M * LDA], h3[2][M * LDA], w4[16 * LDA];
  __shared__ __align__(16) __bf16 yp[16 * LDY];        // dL/dy in three parts, [4 part + j][sample]
  __shared__ __align__(16) float ys[M][4], ts[M][4], w4f[4 * W], bias[3][W];
  __shared__ f32x4 gb3[2][64 * kInferWaves];           // dL/db3 of a lane's samples and features
  __shared__ float xs[3][M][XS], sums[M][XS];          // sums: dL/dy and the loss of a lane's samples
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 15, g = lane >> 4, n_base = 32 * wv, f0 = n_base + 8 * g, nin = a.n_in;
  const int64_t B = a.batch, tiles = (B + M - 1) / M;
  const int count = (int)((tiles - blockIdx.x + gridDim.x - 1) / gridDim.x);
  const float* P = a.params;
  const int xm = tid / kMlpMaxIn, xk = tid % kMlpMaxIn;
  auto first = [&](int i) { return ((int64_t)blockIdx.x + (int64_t)i * gridDim.x) * M; };
  // the inputs (waves 0 to 3) and targets (0 and 1) of a tile, one value a thread;
  // past the batch or the block's tiles some value of theirs, dropped by keep_x
  auto rows_of = [&](int64_t m0) { return (int)min((int64_t)M, B - m0); };
  auto load_x = [&](int i) {
    const int64_t m0 = min(first(i), B - 1);
    return a.x[m0 * nin + (unsigned)(min(xm, rows_of(m0) - 1) * nin + min(xk, nin - 1))];
  };
  auto keep_x = [&](int i, float v) {
    if (wv < M * kMlpMaxIn / 64) xs[i % 3][xm][xk] = xk < nin && xm < B - first(i) ? v : 0.0f;
  };
  auto load_t = [&](int i) {
    const int64_t m0 = min(first(i), B - 1);
    return a.target[m0 * 4 + (unsigned)min(tid, 4 * rows_of(m0) - 1)];
  };
  // what the first layer needs ahead of the weights: loads arrive in order
  const float x0 = load_x(0), x1 = load_x(1);
  float w1[2][2];
#pragma unroll
  for (int ft = 0; ft < 2; ++ft)
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const float v = P[a.off.W1 + wave_row(n_base, ft, r) * nin + min(4 * q + g, nin - 1)];
      w1[ft][q] = 4 * q + g < nin ? v : 0.0f;
    }
  const int b = min(tid, W - 1);
  const float bias1 = P[a.off.b1 + b], bias2 = P[a.off.b2 + b], bias3 = P[a.off.b3 + b];
  const bf16x8 w4_piece = *reinterpret_cast<const bf16x8*>(a.W4s + tid * 8);
  const float w4_0 = P[a.off.W4 + tid], w4_1 = P[a.off.W4 + tid + 2 * W];
  float b4[4];
#pragma unroll
  for (int j = 0; j < 4; ++j)
    b4[j] = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(
                                          __builtin_bit_cast(int, P[a.off.b4 + j])));
  __builtin_amdgcn_sched_barrier(0);
  bf16x8 w2[2][8], w3[2][8];
  load_weights(w2, a.W2b, wv, lane);
  load_weights(w3, a.W3b, wv, lane);
  __builtin_amdgcn_sched_barrier(0);
  *reinterpret_cast<bf16x8*>(w4 + tid / 32 * LDA + tid % 32 * 8) = w4_piece;
  w4f[tid] = w4_0;
  w4f[tid + 2 * W] = w4_1;
  for (int i = tid; i < 4 * LDY; i += 64 * kInferWaves) yp[12 * LDY + i] = (__bf16)0.0f;
  gb3[0][tid] = gb3[1][tid] = f32x4{0.f, 0.f, 0.f, 0.f};
  if (tid < M * 5) sums[tid / 5][tid % 5] = 0.0f;
  if (tid < W) {
    bias[0][tid] = bias1;
    bias[1][tid] = bias2;
    bias[2][tid] = bias3;
  }
  f32x4 gw4[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
  bf16x8 ds3[TILES];

  // h of a lane's eight features of sample 16 st + r of a tile, zero past the batch
  auto store_h = [&](bf16x8 h, __bf16* lds, int st, __bf16* out, int rows) {
    i32x4 bits = __builtin_bit_cast(i32x4, h);
#pragma unroll
    for (int e = 0; e < 4; ++e) bits[e] = st * 16 + r < rows ? bits[e] : 0;
    h = __builtin_bit_cast(bf16x8, bits);
    *reinterpret_cast<bf16x8*>(lds + (st * 16 + r) * LDA + f0) = h;
    if (out) *reinterpret_cast<bf16x8*>(out + (unsigned)((st * 16 + r) * W + f0)) = h;
  };
  auto load_bias = [&](float (&b)[8], int l) {
#pragma unroll
    for (int e = 0; e < 8; ++e) b[e] = bias[l][f0 + e];
  };
  auto layer1 = [&](int i) {
    const int slot = i % 3;
    const int64_t m0 = first(i);
    float b[8];
    load_bias(b, 0);
#pragma unroll
    for (int st = 0; st < TILES; ++st) {
      const float x0 = xs[slot][st * 16 + r][g], x1 = xs[slot][st * 16 + r][4 + g];
      bf16x8 h;
#pragma unroll
      for (int ft = 0; ft < 2; ++ft) {
        f32x4 d = {0.f, 0.f, 0.f, 0.f};
        d = __builtin_amdgcn_mfma_f32_16x16x4f32(w1[ft][0], x0, d, 0, 0, 0);
        d = __builtin_amdgcn_mfma_f32_16x16x4f32(w1[ft][1], x1, d, 0, 0, 0);
#pragma unroll
        for (int e = 0; e < 4; ++e) h[4 * ft + e] = (__bf16)silu(d[e] + b[4 * ft + e]);
      }
      store_h(h, h1, st, a.h1 + m0 * W, rows_of(m0));
    }
  };
  auto layer = [&](const bf16x8 (&w)[2][8], int l, const __bf16* in, __bf16* out,
                   __bf16* out_global, int64_t m0, auto keep_ds) {
    float b[8];
    load_bias(b, l);
#pragma unroll
    for (int st = 0; st < TILES; ++st) {
      f32x4 acc[2];
      wave_gemm(w, in + (st * 16 + r) * LDA + 8 * g, acc);
      bf16x8 h, ds;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float z = acc[e >> 2][e & 3] + b[e], sg = sigmoid(z);
        h[e] = (__bf16)(z * sg);
        ds[e] = (__bf16)(sg * (1.0f + z * (1.0f - sg)));
      }
      store_h(h, out, st, out_global ? out_global + m0 * W : nullptr, rows_of(m0));
      keep_ds(st, ds);
    }
  };
  auto layer2 = [&](int i) {
    __bf16* out = a.ds2 + first(i) * W;
    layer(w2, 1, h1, h2, a.h2, first(i), [&](int st, bf16x8 ds) {
      *reinterpret_cast<bf16x8*>(out + (unsigned)(((wv * TILES + st) * 64 + lane) * 8)) = ds;
    });
  };
  // outputs, loss and dL/dy of a tile: wave wv < TILES takes 16 samples; lane
  // groups 0, 1 and 2 hold the three parts of the four outputs, group 0 finishes
  auto layer4 = [&](int i) {
    const __bf16* row = h3[i & 1] + (wv * 16 + r) * LDA + 8 * g;
    f32x4 y = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 2
    for (int k = 0; k < 8; ++k)
      y = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
          *reinterpret_cast<const bf16x8*>(w4 + r * LDA + 32 * k + 8 * g),
          *reinterpret_cast<const bf16x8*>(row + 32 * k), y, 0, 0, 0);
    const float* x = xs[i % 3][wv * 16 + r];
    float u[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float mid = __shfl(y[j], lane + 16, 64), lo = __shfl(y[j], lane + 32, 64);
      const float yj = b4[j] + ((y[j] + mid) + lo);
      float base = a.out_ref[j];
#pragma unroll
      for (int k = 0; k < kMlpMaxIn; ++k) base = fmaf(a.out_lin[j][k], x[k], base);
      u[j] = fmaf(a.out_scale[j], yj, base);
    }
    const float inv = 1.0f / sqrtf(u[0] * u[0] + u[1] * u[1] + u[2] * u[2] + u[3] * u[3]);
    const bool in = wv * 16 + r < B - first(i);
    float q[4], dq[4], qd = 0.0f, l = 0.0f;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      q[j] = u[j] * inv;
      const float d = q[j] - ts[wv * 16 + r][j];
      l += d * d;
      dq[j] = 2.0f * d * a.inv_loss_norm;
      qd += q[j] * dq[j];
    }
    float* sum = sums[wv * 16 + r];
    if (lane < 16) sum[4] += in ? l : 0.0f;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float dy = in ? a.out_scale[j] * ((dq[j] - q[j] * qd) * inv) : 0.0f;
      if (lane < 16) {
        sum[j] += dy;
        ys[wv * 16 + r][j] = dy;
#pragma unroll
        for (int part = 0; part < 3; ++part) yp[(4 * part + j) * LDY + wv * 16 + r] = split3(dy, part);
      }
    }
  };
  // dz3 = (dL/dy W4) ⊙ silu'(z3), its bias gradient before rounding, and the W4
  // gradient dL/dyᵀ h3 of the wave's features
  auto finish = [&](int i) {
    const int64_t m0 = first(i);
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      f32x4 w[4], sum = gb3[half][tid];
#pragma unroll
      for (int j = 0; j < 4; ++j) w[j] = *reinterpret_cast<const f32x4*>(w4f + j * W + f0 + 4 * half);
#pragma unroll
      for (int st = 0; st < TILES; ++st) {
        const f32x4 y = *reinterpret_cast<const f32x4*>(ys[st * 16 + r]);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float dh = w[0][e] * y[0] + w[1][e] * y[1] + w[2][e] * y[2] + w[3][e] * y[3];
          const float dz = dh * (float)ds3[st][4 * half + e];
          sum[e] += dz;
          ds3[st][4 * half + e] = (__bf16)dz;
        }
      }
      gb3[half][tid] = sum;
    }
#pragma unroll
    for (int st = 0; st < TILES; ++st)
      *reinterpret_cast<bf16x8*>(a.dz3 + m0 * W + (unsigned)((st * 16 + r) * W + f0)) = ds3[st];
#pragma unroll
    for (int s0 = 0; s0 < M; s0 += 32) {
      const bf16x8 y = *reinterpret_cast<const bf16x8*>(yp + r * LDY + s0 + 8 * g);
#pragma unroll
      for (int t = 0; t < 2; ++t)
        gw4[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
            y, read_operand(h3[i & 1], LDA, s0, n_base + 16 * t, lane), gw4[t], 0, 0, 0);
    }
  };
  keep_x(0, x0);
  keep_x(1, x1);
  __syncthreads();
  float x_next = load_x(2), t_next = load_t(0);
  layer1(0);
  __syncthreads();
  layer2(0);
  __syncthreads();
  // Loads and stores complete in order, so a value is loaded a whole tile ahead,
  // and the last tile is apart: the waits then count past the stores between.
  auto tile = [&](int i, auto more) {
    layer(w3, 2, h2, h3[i & 1], nullptr, first(i), [&](int st, bf16x8 ds) { ds3[st] = ds; });
    keep_x(i + 2, x_next);
    if (wv < 4 * M / 64) ts[tid / 4][tid % 4] = t_next;
    if (more.value) {
      x_next = load_x(i + 3);
      t_next = load_t(i + 1);
      layer1(i + 1);
    }
    __syncthreads();
    if (wv < TILES) layer4(i);
    if (more.value) layer2(i + 1);
    __syncthreads();
    finish(i);
  };
  for (int i = 0; i + 1 < count; ++i) tile(i, std::true_type());
  tile(count - 1, std::false_type());
  const int64_t blk = blockIdx.x;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    float v = gb3[e >> 2][tid][e & 3];
#pragma unroll
    for (int off = 1; off < 16; off <<= 1) v += __shfl_xor(v, off, 64);
    if (r == 0) a.gpart_b3[blk * W + f0 + e] = v;
  }
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float mid = __shfl(gw4[t][j], lane + 16, 64), lo = __shfl(gw4[t][j], lane + 32, 64);
      if (lane < 16) a.gpart_W4[(blk * 4 + j) * W + n_base + 16 * t + r] = (gw4[t][j] + mid) + lo;
    }
  if (tid < 5) {
    float v = 0.0f;
    for (int m = 0; m < M; ++m) v += sums[m][tid];
    if (tid < 4) a.gpart_b4[blk * 4 + tid] = v;
    else         a.loss_part[blk] = v * a.inv_loss_norm;
  }
}

// Training, backward half, with the rows of W3ᵀ and W2ᵀ in registers: dz2 =
// (dz3 W3) ⊙ silu'(z2) and dz1 = (dz2 W2) ⊙ silu'(z1), z1 recomputed by the
// forward half's products.  dz1 is only needed by the wave that forms it, for the
// W1 and b1 gradients (fp32 matrix cores, samples taken four by four in the
// order that the transposed read gives them).
__global__ void __launch_bounds__(64 * kInferWaves) __attribute__((amdgpu_waves_per_eu(2, 2)))
mlp_train_backward_kernel(const MlpArgs a) {
  constexpr int M = kTrainTile, TILES = M / 16, XS = kMlpMaxIn + 1, NTH = 64 * kInferWaves, LD1 = 48;
  constexpr int Q = M * W / 8 / NTH;       // 16-byte pieces of a tile per thread
  __shared__ __align__(16) __bf16 d3[M * LDA], d2[M * LDA], d1[kInferWaves][M * LD1];
  __shared__ float xs[2][M][XS];
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = lane & 15, g = lane >> 4, n_base = 32 * wv, f0 = n_base + 8 * g, nin = a.n_in;
  const int64_t B = a.batch, tiles = (B + M - 1) / M;
  const int count = (int)((tiles - blockIdx.x + gridDim.x - 1) / gridDim.x);
  const float* P = a.params;
  const int xm = tid / kMlpMaxIn, xk = tid % kMlpMaxIn;
  auto first = [&](int i) { return ((int64_t)blockIdx.x + (int64_t)i * gridDim.x) * M; };
  float x_next;
  bf16x8 next[Q], ds2[TILES];
  // (past the last tile: that one again, so that every wait counts the same loads)
  auto load_tile = [&](int i) {
    const int64_t m0 = first(min(i, count - 1));
    const int rows = (int)min((int64_t)M, B - m0);
    x_next = a.x[m0 * nin + (unsigned)(min(xm, rows - 1) * nin + min(xk, nin - 1))];
#pragma unroll
    for (int q = 0; q < Q; ++q)
      next[q] = *reinterpret_cast<const bf16x8*>(a.dz3 + m0 * W + (unsigned)((tid + q * NTH) * 8));
  };
  auto store_tile = [&](int i) {
    if (wv < M * kMlpMaxIn / 64)
      xs[i & 1][xm][xk] = xk < nin && xm < B - first(i) ? x_next : 0.0f;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int c = tid + q * NTH;
      *reinterpret_cast<bf16x8*>(d3 + c / (W / 8) * LDA + c % (W / 8) * 8) = next[q];
    }
  };
  auto load_ds = [&](int i) {
    const __bf16* src = a.ds2 + first(min(i, count - 1)) * W;
#pragma unroll
    for (int st = 0; st < TILES; ++st)
      ds2[st] = *reinterpret_cast<const bf16x8*>(src + (unsigned)(((wv * TILES + st) * 64 + lane) * 8));
  };
  load_tile(0);
  __builtin_amdgcn_sched_barrier(0);
  bf16x8 w3[2][8], w2[2][8];
  load_weights(w3, a.W3Tb, wv, lane);
  load_ds(0);
  load_weights(w2, a.W2Tb, wv, lane);
  float b1[8], w1[2][2];
#pragma unroll
  for (int e = 0; e < 8; ++e) b1[e] = P[a.off.b1 + f0 + e];
#pragma unroll
  for (int ft = 0; ft < 2; ++ft)
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const float v = P[a.off.W1 + wave_row(n_base, ft, r) * nin + min(4 * q + g, nin - 1)];
      w1[ft][q] = 4 * q + g < nin ? v : 0.0f;
    }
  __builtin_amdgcn_sched_barrier(0);
  float gb2[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  f32x4 gw1[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
  __bf16* const own = d1[wv];
  // the W1 and b1 gradients of a tile whose dz1 the wave has left in LDS
  auto grad1 = [&](int i) {
    const float (*x)[XS] = xs[i & 1];
#pragma unroll
    for (int st = 0; st < TILES; ++st) {
      bf16x4 v[2];
#pragma unroll
      for (int ft = 0; ft < 2; ++ft) v[ft] = read_columns(own, LD1, 16 * st + 4 * g, 16 * ft, lane);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float xv = x[16 * st + 4 * g + e][min(r, nin - 1)];
        const float in = r < nin ? xv : r == nin ? 1.0f : 0.0f;
#pragma unroll
        for (int ft = 0; ft < 2; ++ft)
          gw1[ft] = __builtin_amdgcn_mfma_f32_16x16x4f32((float)v[ft][e], in, gw1[ft], 0, 0, 0);
      }
    }
  };
  store_tile(0);
  __syncthreads();
  for (int i = 0; i < count; ++i) {
    const int64_t m0 = first(i);
    load_tile(i + 1);
    if (i > 0) grad1(i - 1);
#pragma unroll
    for (int st = 0; st < TILES; ++st) {
      f32x4 acc[2];
      wave_gemm(w3, d3 + (st * 16 + r) * LDA + 8 * g, acc);
      bf16x8 v;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        v[e] = (__bf16)(acc[e >> 2][e & 3] * (float)ds2[st][e]);
        gb2[e] += (float)v[e];
      }
      *reinterpret_cast<bf16x8*>(d2 + (st * 16 + r) * LDA + f0) = v;
      *reinterpret_cast<bf16x8*>(a.dz2 + m0 * W + (unsigned)((st * 16 + r) * W + f0)) = v;
    }
    __syncthreads();
    load_ds(i + 1);
    const float (*x)[XS] = xs[i & 1];
#pragma unroll
    for (int st = 0; st < TILES; ++st) {
      f32x4 acc[2];
      wave_gemm(w2, d2 + (st * 16 + r) * LDA + 8 * g, acc);
      const float x0 = x[st * 16 + r][g], x1 = x[st * 16 + r][4 + g];
      bf16x8 v;
#pragma unroll
      for (int ft = 0; ft < 2; ++ft) {
        f32x4 z = {0.f, 0.f, 0.f, 0.f};
        z = __builtin_amdgcn_mfma_f32_16x16x4f32(w1[ft][0], x0, z, 0, 0, 0);
        z = __builtin_amdgcn_mfma_f32_16x16x4f32(w1[ft][1], x1, z, 0, 0, 0);
#pragma unroll
        for (int e = 0; e < 4; ++e)
          v[4 * ft + e] = (__bf16)(acc[ft][e] * dsilu(z[e] + b1[4 * ft + e]));
      }
      *reinterpret_cast<bf16x8*>(own + (st * 16 + r) * LD1 + 8 * g) = v;
    }
    store_tile(i + 1);
    __syncthreads();
  }
  grad1(count - 1);
  const int64_t blk = blockIdx.x;
#pragma unroll
  for (int e = 0; e < 8; ++e)
#pragma unroll
    for (int off = 1; off < 16; off <<= 1) gb2[e] += __shfl_xor(gb2[e], off, 64);
  if (r == 0)
#pragma unroll
    for (int e = 0; e < 8; ++e) a.gpart_b2[blk * W + f0 + e] = gb2[e];
#pragma unroll
  for (int ft = 0; ft < 2; ++ft)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int64_t n = n_base + 16 * ft + 4 * g + e;
      if (r < nin) a.gpart_W1[(blk * W + n) * nin + r] = gw1[ft][e];
      else if (r == nin) a.gpart_b1[blk * W + n] = gw1[ft][e];
    }
}

// Weight gradients of the two 256×256 layers: gW[n][k] = Σ_b dz[b][n] h[b][k]
// over one split (a contiguous range of samples).  A workgroup computes a
// 128×128 tile of one split, each wave a 64×64 quarter of it; every 32-sample
// step stages the tile's 128 columns of both operands in LDS (double-buffered),
// from where they are read transposed (rows padded to 288 B: the four row pieces
// of a transposed read lie in different banks), and the next step's global loads
// are in flight during the current step's sixteen MFMAs.  The four tiles of a
// (layer, split) group read the same operands, so the launch keeps a group on
// one XCD (workgroups are dealt to the 8 XCDs in turn), where they share the
// XCD's L2.
constexpr int kWgTile = 128, kWgRow = kWgTile + 16;
__global__ void __launch_bounds__(NT) mlp_weight_grad_kernel(const MlpArgs a) {
  __shared__ __align__(16) __bf16 As[2][32 * kWgRow];
  __shared__ __align__(16) __bf16 Bs[2][32 * kWgRow];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int id = blockIdx.x, xcd = id % 8, slot = id / 8;
  const int group = xcd + 8 * (slot / 4), tile = slot % 4;
  const int which = group & 1, split = group >> 1;
  const __bf16* dz = which == 0 ? a.dz2 : a.dz3;
  const __bf16* h = which == 0 ? a.h1 : a.h2;
  float* out = (which == 0 ? a.gpart_W2 : a.gpart_W3) + (size_t)split * W * W;
  const int n0 = (tile >> 1) * kWgTile, k0 = (tile & 1) * kWgTile;
  const int wn = (wv >> 1) * 64, wk = (wv & 1) * 64;
  const int64_t bs = (int64_t)split * a.split_chunk, be = min(a.ld, bs + a.split_chunk);
  const int nsteps = be > bs ? (int)((be - bs) / 32) : 0;
  // staging: thread t moves 16 bytes of samples t/16 and 16 + t/16, piece t%16
  const int sr = tid >> 4, sc = (tid & 15) * 8;
  const __bf16* ga = dz + (bs + sr) * W + n0 + sc;
  const __bf16* gb = h + (bs + sr) * W + k0 + sc;
  const int so0 = sr * kWgRow + sc, so1 = so0 + 16 * kWgRow;
  f32x4 acc[4][4];
  zero_acc(acc);
  bf16x8 xa0, xa1, xb0, xb1;
  if (nsteps > 0) {
    xa0 = *reinterpret_cast<const bf16x8*>(ga);
    xa1 = *reinterpret_cast<const bf16x8*>(ga + 16 * W);
    xb0 = *reinterpret_cast<const bf16x8*>(gb);
    xb1 = *reinterpret_cast<const bf16x8*>(gb + 16 * W);
    *reinterpret_cast<bf16x8*>(&As[0][so0]) = xa0;
    *reinterpret_cast<bf16x8*>(&As[0][so1]) = xa1;
    *reinterpret_cast<bf16x8*>(&Bs[0][so0]) = xb0;
    *reinterpret_cast<bf16x8*>(&Bs[0][so1]) = xb1;
  }
  __syncthreads();
  for (int st = 0; st < nsteps; ++st) {
    const int cur = st & 1;
    const bool more = st + 1 < nsteps;
    if (more) {
      const int64_t off = (int64_t)(st + 1) * 32 * W;
      xa0 = *reinterpret_cast<const bf16x8*>(ga + off);
      xa1 = *reinterpret_cast<const bf16x8*>(ga + off + 16 * W);
      xb0 = *reinterpret_cast<const bf16x8*>(gb + off);
      xb1 = *reinterpret_cast<const bf16x8*>(gb + off + 16 * W);
    }
    bf16x8 av[4], bv[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      av[i] = read_operand(As[cur], kWgRow, 0, wn + i * 16, lane);
      bv[i] = read_operand(Bs[cur], kWgRow, 0, wk + i * 16, lane);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[i], bv[j], acc[i][j], 0, 0, 0);
    if (more) {
      *reinterpret_cast<bf16x8*>(&As[cur ^ 1][so0]) = xa0;
      *reinterpret_cast<bf16x8*>(&As[cur ^ 1][so1]) = xa1;
      *reinterpret_cast<bf16x8*>(&Bs[cur ^ 1][so0]) = xb0;
      *reinterpret_cast<bf16x8*>(&Bs[cur ^ 1][so1]) = xb1;
    }
    __syncthreads();
  }
  const int c = lane & 15, rq = 4 * (lane >> 4);
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        out[(size_t)(n0 + wn + i * 16 + rq + e) * W + k0 + wk + j * 16 + c] = acc[i][j][e];
}

// Column sums of row-major partials [rows][len], 64 rows per workgroup and
// pass: a workgroup covers C columns (C = 64, or fewer for short rows) with
// 256/C threads per column; every thread sums a strided subset of the rows
// and the subsets are combined in LDS in thread order, so the result does not
// depend on scheduling.  Several independent sums share a launch: the blocks
// of segment k are numbered from first[k].
struct SumPass {
  int nseg;
  struct {
    const float* src;
    float* dst;
    int64_t len, first;
    int rows, C, gx;
  } seg[kMaxSumSegments];
};

__global__ void __launch_bounds__(256) sum_partials_multi_kernel(const SumPass p) {
  __shared__ float acc[256];
  int k = 0;
  while (k + 1 < p.nseg && (int64_t)blockIdx.x >= p.seg[k + 1].first) ++k;
  const int64_t b = (int64_t)blockIdx.x - p.seg[k].first;
  const int C = p.seg[k].C, gx = p.seg[k].gx, rows = p.seg[k].rows;
  const int64_t len = p.seg[k].len;
  const int64_t bx = b % gx, by = b / gx;
  const int t = threadIdx.x, c = t % C, g = t / C, G = 256 / C;
  const int64_t i = bx * C + c;
  const int r0 = (int)by * 64, r1 = min(rows, r0 + 64);
  const float* part = p.seg[k].src;
  float s = 0.0f;
  if (i < len)
#pragma unroll 4
    for (int r = r0 + g; r < r1; r += G) s += part[(size_t)r * len + i];
  acc[t] = s;
  __syncthreads();
  if (g == 0 && i < len) {
    float v = 0.0f;
    for (int q = 0; q < G; ++q) v += acc[q * C + c];
    p.seg[k].dst[(size_t)by * len + i] = v;
  }
}

__global__ void __launch_bounds__(256) adam_kernel(const MlpArgs a, float lr, float c1, float c2,
                                                   const AdamPending pend) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i == 0 && pend.loss_rows > 0) {
    float l = 0.0f;
    for (int r = 0; r < pend.loss_rows; ++r) l += pend.loss_src[r];
    *pend.loss_out = l;
  }
  if (i >= a.n_params) return;
  float g = a.grad[i];
  for (int k = 0; k < pend.n; ++k) {
    const int64_t e = i - pend.seg[k].off;
    if (e >= 0 && e < pend.seg[k].len) {
      g = 0.0f;
      for (int r = 0; r < pend.seg[k].rows; ++r) g += pend.seg[k].src[(int64_t)r * pend.seg[k].len + e];
      a.grad[i] = g;
    }
  }
  const float m = fmaf(kAdamBeta1, a.adam_m[i] - g, g);      // β1 m + (1 - β1) g
  const float v = fmaf(kAdamBeta2, a.adam_v[i] - g * g, g * g);
  a.adam_m[i] = m;
  a.adam_v[i] = v;
  const float p = a.params_rw[i] - lr * (m * c1) / (sqrtf(v * c2) + kAdamEps);
  a.params_rw[i] = p;
  if (i >= a.off.W2 && i < a.off.W2 + W * W) {
    const int64_t e = i - a.off.W2, n = e / W, k = e % W;
    a.W2b_rw[weight_at((int)n, (int)k)] = (__bf16)p;
    a.W2Tb_rw[weight_at((int)k, (int)n)] = (__bf16)p;
  } else if (i >= a.off.W3 && i < a.off.W3 + W * W) {
    const int64_t e = i - a.off.W3, n = e / W, k = e % W;
    a.W3b_rw[weight_at((int)n, (int)k)] = (__bf16)p;
    a.W3Tb_rw[weight_at((int)k, (int)n)] = (__bf16)p;
  } else if (i >= a.off.W4 && i < a.off.W4 + 4 * W) {
    const int64_t e = i - a.off.W4, j = e / W, k = e % W;
#pragma unroll
    for (int part = 0; part < 3; ++part) a.W4s_rw[(4 * part + j) * W + k] = split3(p, part);
  }
}

// Rewrite the bf16 copies from the master weights (after a parameter upload):
// W2, W3, their transposes and the three-part W4.
__global__ void __launch_bounds__(256) refresh_bf16_kernel(const MlpArgs a) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= W * W) return;
  const int64_t n = e / W, k = e % W;
  const float p2 = a.params[a.off.W2 + e], p3 = a.params[a.off.W3 + e];
  const int at = weight_at((int)n, (int)k), at_t = weight_at((int)k, (int)n);
  a.W2b_rw[at] = (__bf16)p2;
  a.W2Tb_rw[at_t] = (__bf16)p2;
  a.W3b_rw[at] = (__bf16)p3;
  a.W3Tb_rw[at_t] = (__bf16)p3;
  if (e < 16 * W) {        // W4 in three parts, rows 12-15 zero
    const int64_t row = e / W;
    a.W4s_rw[e] = row < 12 ? split3(a.params[a.off.W4 + (row & 3) * W + k], (int)(row >> 2))
                           : (__bf16)0.0f;
  }
}

}  // namespace

TrainShape mlp_train_shape(int64_t batch) {
  const int64_t tiles = (batch + kTrainTile - 1) / kTrainTile;
  return {kTrainTile, (int)std::min(tiles, mlp_train_rows(batch))};
}
int64_t mlp_train_rows(int64_t ld) {
  const int64_t tiles = (ld + kTrainTile - 1) / kTrainTile, per = kMlpCus * kTrainTiles;
  return kMlpCus * ((tiles + per - 1) / per);
}

hipError_t launch_mlp_infer(const MlpArgs& a, hipStream_t s) {
  // A workgroup per CU.  Tiles of 32 samples spread a small batch over more of
  // them; from four such rounds on, the two barriers per tile weigh more: 32
  // against 64 samples a tile, 13.1 / 15.8 us for 1000, 19.5 / 21.4 for 24576,
  // 22.6 / 21.4 for 32768, 833 / 735 for 2^21.
  const int64_t small = (a.batch + 31) / 32, large = (a.batch + 63) / 64;
  const dim3 block(64 * kInferWaves);
  if (small <= 3 * kMlpCus)
    hipLaunchKernelGGL(mlp_infer_kernel<2>, dim3((unsigned)std::min(kMlpCus, small)), block, 0, s, a);
  else
    hipLaunchKernelGGL(mlp_infer_kernel<4>, dim3((unsigned)std::min(kMlpCus, large)), block, 0, s, a);
  return hipGetLastError();
}

hipError_t launch_mlp_train(const MlpArgs& a, hipStream_t s) {
  const TrainShape t = mlp_train_shape(a.batch);
  if (a.ld % t.tile != 0 || a.ld < a.batch) return hipErrorInvalidValue;
  const dim3 grid((unsigned)t.blocks), block(64 * kInferWaves);
  hipLaunchKernelGGL(mlp_train_forward_kernel, grid, block, 0, s, a);
  hipLaunchKernelGGL(mlp_train_backward_kernel, grid, block, 0, s, a);
  return hipGetLastError();
}

hipError_t launch_mlp_weight_grad(const MlpArgs& a, hipStream_t s) {
  // 4 tiles × 2 layers × n_splits splits; the kernel maps the linear block
  // index to (group, tile) so that each group stays on one XCD
  if (a.n_splits % 4 != 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(mlp_weight_grad_kernel, dim3(4u * 2u * (unsigned)a.n_splits), dim3(NT), 0, s, a);
  return hipGetLastError();
}

size_t sum_partials_tmp(int64_t len, int parts) {
  return parts > 64 ? 2 * (size_t)len * (size_t)((parts + 63) / 64) : 0;
}

hipError_t launch_sum_partials_multi(const SumSegment* segs, int nseg, float* tmp, hipStream_t s,
                                     int max_passes, SumLeft* left) {
  if (nseg < 0 || nseg > kMaxSumSegments) return hipErrorInvalidValue;
  struct State { const float* src; int rows; float* tmp; size_t half; int C; int gx; bool done; };
  State st[kMaxSumSegments];
  size_t off = 0;
  for (int k = 0; k < nseg; ++k) {
    const SumSegment& g = segs[k];
    int C = 64;
    while (C > 1 && C / 2 >= g.len) C /= 2;
    st[k] = {g.part, g.parts, tmp + off, sum_partials_tmp(g.len, g.parts) / 2, C,
             (int)((g.len + C - 1) / C), g.len <= 0};
    off += sum_partials_tmp(g.len, g.parts);
  }
  for (int pass = 0;; ++pass) {
    if (pass == max_passes) {
      for (int k = 0; k < nseg; ++k)
        if (left) left[k] = {st[k].src, segs[k].len, st[k].done ? 0 : st[k].rows};
      return hipSuccess;
    }
    SumPass p;
    p.nseg = 0;
    int64_t blocks = 0;
    int idx[kMaxSumSegments];
    for (int k = 0; k < nseg; ++k) {
      if (st[k].done) continue;
      const bool last = st[k].rows <= 64;
      const int next = last ? 1 : (st[k].rows + 63) / 64;
      auto& q = p.seg[p.nseg];
      q.src = st[k].src;
      q.dst = last ? segs[k].out : st[k].tmp + (pass & 1) * st[k].half;
      q.len = segs[k].len;
      q.first = blocks;
      q.rows = st[k].rows;
      q.C = st[k].C;
      q.gx = st[k].gx;
      idx[p.nseg++] = k;
      blocks += (int64_t)st[k].gx * next;
    }
    if (p.nseg == 0) {
      if (left)
        for (int k = 0; k < nseg; ++k) left[k] = {st[k].src, segs[k].len, 0};
      return hipSuccess;
    }
    hipLaunchKernelGGL(sum_partials_multi_kernel, dim3((unsigned)blocks), dim3(256), 0, s, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    for (int j = 0; j < p.nseg; ++j) {
      State& x = st[idx[j]];
      if (x.rows <= 64) {
        x.done = true;
      } else {
        x.src = p.seg[j].dst;
        x.rows = (x.rows + 63) / 64;
      }
    }
  }
}

hipError_t launch_adam(const MlpArgs& a, float lr, float c1, float c2, hipStream_t s,
                       const AdamPending* pending) {
  AdamPending none{};
  const AdamPending& p = pending ? *pending : none;
  hipLaunchKernelGGL(adam_kernel, dim3((unsigned)((a.n_params + 255) / 256)), dim3(256), 0, s, a, lr,
                     c1, c2, p);
  return hipGetLastError();
}

hipError_t launch_refresh_bf16(const MlpArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(refresh_bf16_kernel, dim3((W * W + 255) / 256), dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace st

namespace st {
namespace {

__global__ void __launch_bounds__(256) features_kernel(const double* z, int64_t n, FeatureMap f,
                                                       int n_in, float* x) {
  const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (j >= n) return;
  for (int i = 0; i < 6 && i < n_in; ++i)
    x[j * n_in + i] = (float)((z[(size_t)i * n + j] - f.center[i]) * f.inv_scale[i]);
  if (n_in == 7) x[j * n_in + 6] = (float)f.extra;
}

__global__ void __launch_bounds__(256) targets_kernel(const double* q, int64_t n, double r0, double r1,
                                                      double r2, double r3, float* t) {
  const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (j >= n) return;
  const double w = q[j], x = q[n + j], y = q[2 * n + j], z = q[3 * n + j];
  const double s = (w * r0 + x * r1 + y * r2 + z * r3) < 0.0 ? -1.0 : 1.0;
  t[j * 4 + 0] = (float)(s * w);
  t[j * 4 + 1] = (float)(s * x);
  t[j * 4 + 2] = (float)(s * y);
  t[j * 4 + 3] = (float)(s * z);
}

// Frame fit.  Four launches with one wait at their end: moments, solve,
// residuals, finish; what bounds it is the two passes over x and t (42 MB for
// 2^20 samples of six inputs: 15.6 and 12.3 us) and the launches themselves (12
// us in the solve, one wave's chain).  2^20 samples: 142 -> 64 us a call against
// two launches with an allocation, two copies and the solve on the host between
// them.
//
// Moments.  With Z = [1, x, t] (1 + n_in + 4 <= 13 columns, zero-padded to 16)
// the normal equations are parts of ZᵀZ, a sum over samples of outer products:
// v_mfma_f64_16x16x4 takes four samples per instruction, and since A = Zᵀ and
// B = Z the same register is both operands (lane l holds column l & 15 of
// sample l >> 4).  A wave sums a contiguous range of samples in order over four
// accumulators, with the next 32 samples' loads in flight, a block its sixteen
// waves in order.
typedef double f64x4 __attribute__((ext_vector_type(4)));
constexpr int kFitWaves = 16;

__global__ void __launch_bounds__(64 * kFitWaves) fit_moments_kernel(const float* x, const float* t,
                                                                     int64_t n, int n_in,
                                                                     double* part) {
  __shared__ double sum[kFitWaves][256];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int col = lane & 15, k = lane >> 4, C = 1 + n_in + 4;
  const int64_t waves = (int64_t)gridDim.x * kFitWaves, w = (int64_t)blockIdx.x * kFitWaves + wv;
  const int64_t per = ((n + waves - 1) / waves + 3) / 4 * 4;
  const int64_t lo = min(n, w * per), hi = min(n, lo + per);
  const bool from_x = col >= 1 && col <= n_in, from_t = col > n_in && col < C;
  const float* src = from_x ? x + (col - 1) : from_t ? t + (col - 1 - n_in) : x;
  const int64_t stride = from_t ? 4 : n_in;
  const float scale = from_x || from_t ? 1.0f : 0.0f, shift = col == 0 ? 1.0f : 0.0f;
  f64x4 acc[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) acc[u] = f64x4{0.0, 0.0, 0.0, 0.0};
  const int64_t full = lo + (hi - lo) / 32 * 32;
  const float* at = src + (lo + k) * stride;
  float v[8];
  if (lo < full)
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = at[4 * u * stride];
  for (int64_t s = lo; s < full; s += 32) {
    if (s + 32 < full) at += 32 * stride;     // (the last round loads its own samples again)
    float next[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) next[u] = at[4 * u * stride];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const double z = (double)fmaf(v[u], scale, shift);
      acc[u & 3] = __builtin_amdgcn_mfma_f64_16x16x4f64(z, z, acc[u & 3], 0, 0, 0);
      v[u] = next[u];
    }
  }
  for (int64_t s = full; s < hi; s += 4) {
    const double z = s + k < hi ? (double)fmaf(src[(s + k) * stride], scale, shift) : 0.0;
    acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(z, z, acc[0], 0, 0, 0);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i)      // entry (4 i + lane / 16, lane % 16)
    sum[wv][(4 * i + k) * 16 + col] = (acc[0][i] + acc[1][i]) + (acc[2][i] + acc[3][i]);
  __syncthreads();
  if (threadIdx.x < 256) {
    double v = 0.0;
    for (int q = 0; q < kFitWaves; ++q) v += sum[q][threadIdx.x];
    part[(int64_t)blockIdx.x * 256 + threadIdx.x] = v;
  }
}

// The blocks' partials summed in block order (seven groups of rows, then the
// groups), and the least-squares coefficients: elimination of the symmetric
// equations [G | R] without pivoting (its pivots are the squared diagonal of the
// Cholesky factor, all positive where the equations are positive definite), one
// row per lane in registers, with a ridge of 1e-12 of the mean diagonal on the
// input columns, which keeps a constant-zero input (a band of one energy)
// solvable with coefficient 0.
__global__ void __launch_bounds__(1024) fit_solve_kernel(const double* part, int nb, int n_in,
                                                         FitResult* out) {
  constexpr int M = kMlpMaxIn + 1, kGroups = 1024 / (16 * M);
  __shared__ double red[kGroups][16 * M];
  __shared__ double G[M][16];
  const int tid = threadIdx.x, D = n_in + 1, e = tid % (16 * M), g = tid / (16 * M);
  const int per = (nb + kGroups - 1) / kGroups, b1 = min(nb, (g + 1) * per);
  if (g < kGroups) {
    double s = 0.0;
    if (e < 16 * D)
#pragma unroll 20
      for (int b = g * per; b < b1; ++b) s += part[(int64_t)b * 256 + e];
    red[g][e] = s;
  }
  __syncthreads();
  if (tid < 16 * M) {
    double v = red[0][tid];
    for (int q = 1; q < kGroups; ++q) v += red[q][tid];
    G[tid >> 4][tid & 15] = v;
  }
  __syncthreads();
  if (tid >= 64) return;
  // lane p: row p, the right-hand sides in the last four columns; rows past D
  // are those of the identity
  const int p = min(tid, M - 1);
  double row[M + 4], trace = 0.0;
  for (int k = 0; k < D; ++k) trace += G[k][k];
#pragma unroll
  for (int k = 0; k < M; ++k) row[k] = p < D && k < D ? G[p][k] : p == k ? 1.0 : 0.0;
#pragma unroll
  for (int c = 0; c < 4; ++c) row[M + c] = p < D ? G[p][D + c] : 0.0;
#pragma unroll
  for (int k = 1; k < M; ++k)
    if (p == k && k < D) row[k] += 1e-12 * trace / D;
  bool bad = false;
#pragma unroll
  for (int k = 0; k < M; ++k) {
    const double pivot = __shfl(row[k], k, 64);
    bad |= !(pivot > 0.0);
    const double f = tid == k ? 0.0 : row[k] / pivot;
#pragma unroll
    for (int q = k; q < M + 4; ++q) row[q] = fma(-f, __shfl(row[q], k, 64), row[q]);
  }
#pragma unroll
  for (int k = 0; k < M; ++k)
    if (tid == k && k < D)
#pragma unroll
      for (int c = 0; c < 4; ++c) out->coef[c][k] = row[M + c] / row[k];
  if (tid == 0) out->bad = bad;
}

// Squared residuals of each component and their largest magnitude over one
// block's range of samples; sums in a fixed order (a thread's samples, the
// wave's lanes by halving, the waves).
template <int NIN>
__global__ void __launch_bounds__(256) fit_residual_kernel(const float* x, const float* t, int64_t n,
                                                           const FitResult* fit, double* part) {
  __shared__ double red[4][8];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  double cf[4][NIN + 1];
#pragma unroll
  for (int c = 0; c < 4; ++c)
#pragma unroll
    for (int k = 0; k <= NIN; ++k) cf[c][k] = fit->coef[c][k];
  double v[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  for (int64_t j = (int64_t)blockIdx.x * 256 + tid; j < n; j += (int64_t)gridDim.x * 256) {
    float xv[NIN], tv[4];
#pragma unroll
    for (int k = 0; k < NIN; ++k) xv[k] = x[j * NIN + k];
#pragma unroll
    for (int c = 0; c < 4; ++c) tv[c] = t[j * 4 + c];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      double f = cf[c][0];
#pragma unroll
      for (int k = 0; k < NIN; ++k) f = fma(cf[c][1 + k], (double)xv[k], f);
      const double r = (double)tv[c] - f;
      v[c] = fma(r, r, v[c]);
      v[4 + c] = fmax(v[4 + c], fabs(r));
    }
  }
  for (int w = 32; w > 0; w >>= 1)
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      const double o = __shfl_xor(v[c], w, 64);
      v[c] = c < 4 ? v[c] + o : fmax(v[c], o);
    }
  if (lane == 0)
    for (int c = 0; c < 8; ++c) red[wv][c] = v[c];
  __syncthreads();
  if (tid < 8) {
    double r = red[0][tid];
    for (int q = 1; q < 4; ++q) r = tid < 4 ? r + red[q][tid] : fmax(r, red[q][tid]);
    part[(int64_t)blockIdx.x * 8 + tid] = r;
  }
}

// The residuals' partials in block order, and the whole result into host memory.
__global__ void __launch_bounds__(256) fit_finish_kernel(const double* part, int nb,
                                                         const FitResult* fit, FitResult* host) {
  __shared__ double red[32][8];
  const int tid = threadIdx.x, c = tid & 7, g = tid >> 3;
  const int per = (nb + 31) / 32, b1 = min(nb, (g + 1) * per);
  double r = 0.0;
#pragma unroll 8
  for (int b = g * per; b < b1; ++b) {
    const double o = part[(int64_t)b * 8 + c];
    r = c < 4 ? r + o : fmax(r, o);
  }
  red[g][c] = r;
  __syncthreads();
  if (tid < 8) {
    r = red[0][tid];
    for (int q = 1; q < 32; ++q) r = tid < 4 ? r + red[q][tid] : fmax(r, red[q][tid]);
    if (tid < 4) host->ss[tid] = r;
    else         host->mx[tid - 4] = r;
  }
  if (tid >= 64 && tid < 64 + 4 * (kMlpMaxIn + 1))
    (&host->coef[0][0])[tid - 64] = (&fit->coef[0][0])[tid - 64];
  if (tid == 128) host->bad = fit->bad;
}

}  // namespace

hipError_t launch_fit(const float* x, const float* t, int64_t n, int n_in, FitWork* work,
                      FitResult* host, hipStream_t s) {
  // enough samples per wave that the blocks' own sums stay small beside them
  const int nb = (int)std::min<int64_t>(kFitBlocks, (n + 32 * kFitWaves - 1) / (32 * kFitWaves));
  const int rb = (int)std::min<int64_t>(kFitResidualBlocks, (n + 255) / 256);
  hipLaunchKernelGGL(fit_moments_kernel, dim3(nb), dim3(64 * kFitWaves), 0, s, x, t, n, n_in,
                     work->moments);
  hipLaunchKernelGGL(fit_solve_kernel, dim3(1), dim3(1024), 0, s, work->moments, nb, n_in,
                     &work->result);
  switch (n_in) {
#define ST_FIT_RESIDUAL(N)                                                                        \
  case N:                                                                                         \
    hipLaunchKernelGGL(fit_residual_kernel<N>, dim3(rb), dim3(256), 0, s, x, t, n, &work->result, \
                       work->residuals);                                                          \
    break;
    ST_FIT_RESIDUAL(1) ST_FIT_RESIDUAL(2) ST_FIT_RESIDUAL(3) ST_FIT_RESIDUAL(4)
    ST_FIT_RESIDUAL(5) ST_FIT_RESIDUAL(6) ST_FIT_RESIDUAL(7) ST_FIT_RESIDUAL(8)
#undef ST_FIT_RESIDUAL
  }
  hipLaunchKernelGGL(fit_finish_kernel, dim3(1), dim3(256), 0, s, work->residuals, rb,
                     &work->result, host);
  return hipGetLastError();
}

hipError_t launch_features(const double* z, int64_t n, const FeatureMap& f, int n_in, float* x,
                           hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(features_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, z, n, f,
                     n_in, x);
  return hipGetLastError();
}

hipError_t launch_targets(const double* q, int64_t n, const double* ref, float* t, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(targets_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, q, n, ref[0],
                     ref[1], ref[2], ref[3], t);
  return hipGetLastError();
}

}  // namespace st
