// Kernels of the b_n continuation network: 16 -> 256 -> 256 -> 16 with GELU,
// BF16 operands on the MFMA units (v_mfma_f32_16x16x32_bf16) with FP32
// accumulation, FP32 master weights and Adam.
//
// Matrix-core lane layout (wave64) of v_mfma_f32_16x16x32_bf16, A 16x32,
// B 32x16, D 16x16 fp32:
//   A: lane l holds row l%16, k = 8*(l/16) .. 8*(l/16)+7
//   B: lane l holds column l%16, k = 8*(l/16) .. 8*(l/16)+7
//   D: lane l holds column l%16, rows 4*(l/16) .. 4*(l/16)+3
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "device_common.hpp"

namespace pauli {
namespace mlp {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float floatx4;

constexpr int NIN = 16, NHID = 256, NOUT = 16;
constexpr int64_t NPARAM = NHID * NIN + NHID + NHID * NHID + NHID + NOUT * NHID + NOUT;
// offsets in the flat parameter vector
constexpr int64_t OFF_W1 = 0, OFF_B1 = OFF_W1 + NHID * NIN;
constexpr int64_t OFF_W2 = OFF_B1 + NHID, OFF_B2 = OFF_W2 + NHID * NHID;
constexpr int64_t OFF_W3 = OFF_B2 + NHID, OFF_B3 = OFF_W3 + NOUT * NHID;

// float -> bfloat16, round to nearest even (finite inputs)
__device__ __forceinline__ uint16_t f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// GELU(x) = x Phi(x) = x (1 + erf(x / sqrt 2)) / 2 and its derivative
// Phi(x) + x phi(x).
__device__ __forceinline__ float gelu(float x) { return 0.5f * x * (1.0f + erff(x * 0.70710678118654752f)); }
__device__ __forceinline__ float gelu_grad(float x) {
  const float cdf = 0.5f * (1.0f + erff(x * 0.70710678118654752f));
  const float pdf = 0.39894228040143268f * expf(-0.5f * x * x);
  return cdf + x * pdf;
}

enum Epilogue : int { EP_STORE = 0, EP_BIAS = 1, EP_BIAS_GELU = 2 };

struct GemmArgs {
  const uint16_t* A;  // A(m,k) = transA ? A[k*lda + m] : A[m*lda + k]
  const uint16_t* B;  // B(k,n) = transB ? B[n*ldb + k] : B[k*ldb + n]
  float* C;           // C[m*ldc + n]
  uint16_t* Cb;       // bf16 of GELU(C) (EP_BIAS_GELU) or nullptr
  const float* bias;  // [n]
  int lda, ldb, ldc;
  int transA, transB;
  int M, N, K;        // M, N multiples of 16; k >= K reads as zero
  int epilogue;
};

// One 64-thread wave per 16x16 output tile, four waves per 32x32 block tile.
__global__ __launch_bounds__(256) void k_gemm_bf16(GemmArgs g) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int m0 = blockIdx.y * 32 + (wv >> 1) * 16;
  const int n0 = blockIdx.x * 32 + (wv & 1) * 16;
  if (m0 >= g.M || n0 >= g.N) return;
  const int r = lane & 15, kq = (lane >> 4) * 8;
  floatx4 acc = {0.f, 0.f, 0.f, 0.f};
  for (int k0 = 0; k0 < g.K; k0 += 32) {
    bf16x8 a, b;
#pragma unroll
    for (int q = 0; q < 8; q++) {
      const int k = k0 + kq + q;
      uint16_t av = 0, bv = 0;
      if (k < g.K) {
        av = g.transA ? g.A[(size_t)k * g.lda + (m0 + r)] : g.A[(size_t)(m0 + r) * g.lda + k];
        bv = g.transB ? g.B[(size_t)(n0 + r) * g.ldb + k] : g.B[(size_t)k * g.ldb + (n0 + r)];
      }
      a[q] = __builtin_bit_cast(__bf16, av);
      b[q] = __builtin_bit_cast(__bf16, bv);
    }
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc, 0, 0, 0);
  }
  const int n = n0 + r;
#pragma unroll
  for (int q = 0; q < 4; q++) {
    const int m = m0 + (lane >> 4) * 4 + q;
    float v = acc[q];
    if (g.epilogue != EP_STORE) v = v + g.bias[n];
    g.C[(size_t)m * g.ldc + n] = v;
    if (g.epilogue == EP_BIAS_GELU) g.Cb[(size_t)m * g.ldc + n] = f2bf(gelu(v));
  }
}

// The same product, operands in their k order (A row-major, B by columns) and
// rows aligned to 16 bytes, which is every product of a forward pass: a wave
// takes 16 rows by NT_TILES column tiles, so A is read once for all of them
// and a lane's eight operands come in one load; the four waves of a block
// share the columns, whose operands then come from the CU's cache.  Bound by
// those reads and the FP32 and BF16 output: the single tiles above, which load
// 16 bits at a time, took 85 us for each of the three products of 15,360 rows
// (16 -> 256, 256 -> 256, 256 -> 16); a training run of four epochs, which ends
// with one forward pass, went from 6.18 to 5.96 ms.  The products of a tile are
// added in the same order as there.
constexpr int NT_TILES = 4;
__global__ __launch_bounds__(256) void k_gemm_nt(GemmArgs g) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int m0 = (blockIdx.y * 4 + wv) * 16;
  const int n0 = blockIdx.x * (NT_TILES * 16);
  if (m0 >= g.M) return;
  const int r = lane & 15, kq = (lane >> 4) * 8;
  const uint16_t* pa = g.A + (size_t)(m0 + r) * g.lda;
  const uint16_t* pb = g.B + (size_t)(n0 + r) * g.ldb;
  const bf16x8 zero = {};
  floatx4 acc[NT_TILES] = {};
  for (int k0 = 0; k0 < g.K; k0 += 32) {
    const int k = k0 + kq;
    const bool in = k < g.K;  // K is a multiple of 8
    const bf16x8 a = in ? *(const bf16x8*)(pa + k) : zero;
#pragma unroll
    for (int j = 0; j < NT_TILES; j++) {
      if (n0 + j * 16 >= g.N) break;
      const bf16x8 b = in ? *(const bf16x8*)(pb + (size_t)(j * 16) * g.ldb + k) : zero;
      acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc[j], 0, 0, 0);
    }
  }
#pragma unroll
  for (int j = 0; j < NT_TILES; j++) {
    const int n = n0 + j * 16 + r;
    if (n0 + j * 16 >= g.N) break;
    const float bias = g.epilogue != EP_STORE ? g.bias[n] : 0.f;
#pragma unroll
    for (int q = 0; q < 4; q++) {
      const int m = m0 + (lane >> 4) * 4 + q;
      float v = acc[j][q];
      if (g.epilogue != EP_STORE) v = v + bias;
      g.C[(size_t)m * g.ldc + n] = v;
      if (g.epilogue == EP_BIAS_GELU) g.Cb[(size_t)m * g.ldc + n] = f2bf(gelu(v));
    }
  }
}

__global__ void k_bf_to_f(const uint16_t* x, float* y, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) y[i] = bf2f(x[i]);
}

__global__ void k_to_bf16(const float* x, uint16_t* y, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) y[i] = f2bf(x[i]);
}

// Masked mean-squared error: per-row partial sums of mask*(y-t)^2 and of the
// mask (fixed order), and dL/dy = 2 mask (y - t) / sum(mask) rounded to bf16.
__global__ void k_mse_rows(const float* y, const float* t, const float* mask, int64_t rows,
                           double* row_err, double* row_cnt) {
  const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= rows) return;
  double e = 0.0, c = 0.0;
  for (int j = 0; j < NOUT; j++) {
    const double m = mask[b * NOUT + j];
    const double d = (double)y[b * NOUT + j] - (double)t[b * NOUT + j];
    e += m * d * d;
    c += m;
  }
  row_err[b] = e;
  row_cnt[b] = c;
}

__global__ void k_sum_rows(const double* row_err, const double* row_cnt, int64_t rows,
                           double* out) {
  __shared__ double se[256], sc[256];
  const int t = threadIdx.x;
  double e = 0.0, c = 0.0;
  for (int64_t b = t; b < rows; b += 256) {
    e += row_err[b];
    c += row_cnt[b];
  }
  se[t] = e;
  sc[t] = c;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (t < s) {
      se[t] += se[t + s];
      sc[t] += sc[t + s];
    }
    __syncthreads();
  }
  if (t == 0) {
    out[0] = sc[0] > 0 ? se[0] / sc[0] : 0.0;
    out[1] = sc[0];
  }
}

__global__ void k_mse_grad(const float* y, const float* t, const float* mask, int64_t n,
                           const double* loss_cnt, float* dy, uint16_t* dyb) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double cnt = loss_cnt[1];
  const float g = cnt > 0 ? (float)(2.0 * (double)mask[i] * ((double)y[i] - (double)t[i]) / cnt) : 0.f;
  dy[i] = g;
  dyb[i] = f2bf(g);
}

// dZ = dY * GELU'(Z), in fp32 and bf16.
__global__ void k_gelu_back(const float* dy, const float* z, int64_t n, float* dz, uint16_t* dzb) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float g = dy[i] * gelu_grad(z[i]);
  dz[i] = g;
  dzb[i] = f2bf(g);
}

// Bias gradient: column sums of d[rows][cols] in a fixed order (one thread
// per column, rows in ascending order).
__global__ void k_col_sum(const float* d, int64_t rows, int cols, float* out) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= cols) return;
  float s = 0.f;
  for (int64_t b = 0; b < rows; b++) s += d[b * cols + c];
  out[c] = s;
}

// Adam on the flat fp32 parameter vector; refreshes the bf16 copy.  The
// complements 1-b1 and 1-b2 come from the host in double precision: formed
// in float from a rounded b2 = 0.999 they would be off by 1.3e-5 relative.
__global__ void k_adam(float* p, const float* g, float* m, float* v, uint16_t* pb, int64_t n,
                       float lr, float b1, float omb1, float b2, float omb2, float eps, float c1,
                       float c2) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + omb1 * gi;
  const float vi = b2 * v[i] + omb2 * gi * gi;
  m[i] = mi;
  v[i] = vi;
  const float mh = mi / c1, vh = vi / c2;
  const float pi = p[i] - lr * mh / (sqrtf(vh) + eps);
  p[i] = pi;
  pb[i] = f2bf(pi);
}

// ---------------------------------------------------------------------------
// Fused training step, two kernels per minibatch (row i of the minibatch is row
// order[i] of the training set; the operands, FP32 accumulation and epilogues
// are those of the layer-by-layer kernels above).
//
// k_mlp_step: one block of 1024 threads (sixteen waves, wave w on hidden columns
// 16 w .. 16 w + 15) takes SB rows through forward, masked MSE and backward
// with the activations in LDS and every product on the matrix cores, and
// leaves what the weight gradients need in memory (StepOut; rows beyond the
// minibatch are zero with zero mask, so they contribute nothing).
// k_mlp_grad_adam: one wave per 16 x 16 tile of a weight gradient (K = the
// minibatch, in shares of SR rows that are added in order) or per eight bias
// columns takes the gradient and the Adam step at once.
//
// Bound: the chain of six dependent products with a barrier after each, on as
// many CUs as the minibatch has SB-row blocks.  Four waves that walked the tiles of 32 rows
// in turn, with operands read as single 16-bit words, took 50.7 us for 256 rows
// and 4.9 us for the sum of the blocks' gradient shares and Adam; sixteen waves
// with 16-byte operand reads 22.7 us; 16-row blocks that leave the weight
// gradients to the second kernel (no gradient shares are written or read) 15.1
// and 6.2 us. (240 such minibatches: 14.4 -> 6.2 ms with the launches.)
// ---------------------------------------------------------------------------
constexpr int SR = 32;  // rows of a gradient share
constexpr int SB = 16;  // rows of a block of k_mlp_step
constexpr int STEP_THREADS = 1024;

// Activations of a minibatch padded to Bp rows (a multiple of SR): by columns
// [column][Bp] in bf16, the operands of the weight gradients, and by rows in
// FP32, for the bias gradients; and the squared errors.
struct StepOut {
  uint16_t *x, *y1, *y2, *dz1, *dz2, *dy;
  float *fz1, *fz2, *fy;
  double* err;  // [Bp][16]
  double* cnt;  // sum of the mask
  int Bp;
};
constexpr size_t step_out_bytes(size_t Bp) {
  return Bp * (2 * (NIN + 4 * NHID + NOUT) + 4 * (2 * NHID + NOUT) + 8 * NOUT) + 8;
}

struct StepArgs {
  const float* params;   // fp32 master weights (biases)
  const uint16_t* pb;    // bf16 weights
  const uint16_t* w2t;   // bf16 W2 transposed (nullptr: read from pb by columns)
  const float* X;        // [n][16] training inputs
  const float* T;        // [n][16] targets
  const float* Mk;       // [n][16] target mask
  const int32_t* order;  // the minibatch's rows, `rows` entries
  int rows;
  StepOut o;
};

__device__ __forceinline__ bf16x8 bf8_lds(const uint16_t* p) {
  return *reinterpret_cast<const bf16x8*>(p);
}
__device__ __forceinline__ bf16x8 bf8_zero() {
  bf16x8 v;
#pragma unroll
  for (int q = 0; q < 8; q++) v[q] = __builtin_bit_cast(__bf16, (uint16_t)0);
  return v;
}
// 8 bf16 values p[0], p[stride], ..., p[7 stride]
__device__ __forceinline__ bf16x8 bf8_strided(const uint16_t* p, int stride) {
  bf16x8 v;
#pragma unroll
  for (int q = 0; q < 8; q++) v[q] = __builtin_bit_cast(__bf16, p[q * stride]);
  return v;
}
// 8 consecutive bf16 weights, in one load where ALIGNED says that the weights start on 16 bytes
template <bool ALIGNED>
__device__ __forceinline__ bf16x8 bf8_weights(const uint16_t* p) {
  if constexpr (ALIGNED) return *reinterpret_cast<const bf16x8*>(p);
  else return bf8_strided(p, 1);
}
__device__ __forceinline__ floatx4 mfma(bf16x8 a, bf16x8 b, floatx4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
// Barrier that orders the block's LDS accesses only: loads from memory stay in
// flight across it (__syncthreads waits for them).
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}
// d[0] = d[0] + ... + d[255]: d[t] += d[t + s] for s = 128, ..., 1, from s = 32
// on inside the first wave
__device__ __forceinline__ void tree256(double* d, int tid) {
  lds_barrier();
  if (tid < 64) {
    double v = (d[tid] + d[tid + 128]) + (d[tid + 64] + d[tid + 192]);
#pragma unroll
    for (int s = 32; s > 0; s >>= 1) v += __shfl_down(v, s, 64);
    if (tid == 0) d[0] = v;
  }
  lds_barrier();
}

// ALIGNED: the caller's bf16 weights start on 16 bytes (each matrix of the
// vector then does, see the offsets)
static_assert(OFF_W1 % 8 == 0 && OFF_W2 % 8 == 0 && OFF_W3 % 8 == 0, "whole 16-byte words");
template <bool ALIGNED>
__global__ __launch_bounds__(STEP_THREADS) void k_mlp_step(StepArgs a) {
  constexpr int RS = NHID + 8;  // row of a tile (16-bit words; 16-byte aligned, off the bank stride)
  static_assert(NHID == 16 * (STEP_THREADS / 64) && SB == 16, "one column tile per wave, one row tile");
  __shared__ __align__(16) uint16_t xb[SB][NIN];
  __shared__ __align__(16) uint16_t y1b[SB][RS];   // bf16 GELU(Z1)
  __shared__ __align__(16) uint16_t y2b[SB][RS];   // bf16 GELU(Z2), then bf16 dZ2
  __shared__ float yv[SB][NOUT];
  __shared__ __align__(16) uint16_t dyb[SB][NOUT];
  __shared__ double dred[256];
  __shared__ float mk[4096];                       // mask values, 256 rows at a time
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const int r = lane & 15, kq = (lane >> 4) * 8, rq = (lane >> 4) * 4;
  const int row0 = blockIdx.x * SB;
  const StepOut& o = a.o;
  const size_t Bp = (size_t)o.Bp;
  const uint16_t* W1 = a.pb + OFF_W1;
  const uint16_t* W2 = a.pb + OFF_W2;
  const uint16_t* W3 = a.pb + OFF_W3;
  const int n = wv * 16 + r;  // this lane's hidden column
  // this lane's four rows of column c of a tile, by columns and by rows
  auto put = [&](uint16_t* by_col, int c, ushort4 t) {
    *reinterpret_cast<ushort4*>(by_col + (size_t)c * Bp + row0 + rq) = t;
  };

  // Loads in two rounds: the rows of this block and of the minibatch's mask
  // (every index clamped, so that no branch comes between loads) with the
  // forward weights of this wave's columns, then what those rows hold.
  // Thread t of the first quarter takes input and output t % 16 of row t / 16.
  static_assert(NIN == NOUT && SB * NIN == STEP_THREADS / 4, "one input and one output per thread");
  const int xr = (tid & 255) / NIN, xj = tid % NIN;
  const bool have = tid < SB * NIN && row0 + xr < a.rows;
  const int id = a.order[min(row0 + xr, a.rows - 1)];
  const int nmask = a.rows * NOUT;
  int mid[4];
#pragma unroll
  for (int q = 0; q < 4; q++) mid[q] = a.order[min(q * STEP_THREADS + tid, nmask - 1) / NOUT];
  const bf16x8 w1 = kq < NIN ? bf8_weights<ALIGNED>(W1 + n * NIN + kq) : bf8_zero();
  const float bias1 = a.params[OFF_B1 + n], bias2 = a.params[OFF_B2 + n];
  bf16x8 w2[NHID / 32], w2c[NHID / 32];
#pragma unroll
  for (int k = 0; k < NHID / 32; k++)
    w2[k] = bf8_weights<ALIGNED>(W2 + n * NHID + k * 32 + kq);
  const float tx = a.X[(size_t)id * NIN + xj];
  const float tt = a.T[(size_t)id * NOUT + xj], tm = a.Mk[(size_t)id * NOUT + xj];
  // the minibatch's mask, summed further down (every block sums the same
  // values in the same order)
  float mv[4];
#pragma unroll
  for (int q = 0; q < 4; q++) mv[q] = a.Mk[(size_t)mid[q] * NOUT + tid % NOUT];
  if (tid < SB * NIN) {
    const uint16_t v = have ? f2bf(tx) : (uint16_t)0;
    xb[xr][xj] = v;
    o.x[(size_t)xj * Bp + row0 + xr] = v;
  }
  lds_barrier();

  // Z1 = Xb W1^T + b1 (K = 16: lanes of k >= 16 supply zeros), Y1 = GELU(Z1)
  float z1[4], z2[4];
  {
    const bf16x8 av = kq < NIN ? bf8_lds(&xb[r][kq]) : bf8_zero();
    const floatx4 acc = mfma(av, w1, floatx4{0.f, 0.f, 0.f, 0.f});
    ushort4 t;
    uint16_t* tv = reinterpret_cast<uint16_t*>(&t);
#pragma unroll
    for (int q = 0; q < 4; q++) {
      z1[q] = acc[q] + bias1;
      tv[q] = f2bf(gelu(z1[q]));
      y1b[rq + q][n] = tv[q];
    }
    put(o.y1, n, t);
  }
  // the backward weights: W2 and W3 by columns
#pragma unroll
  for (int k = 0; k < NHID / 32; k++)
    w2c[k] = a.w2t ? *reinterpret_cast<const bf16x8*>(a.w2t + n * NHID + k * 32 + kq)
                   : bf8_strided(W2 + (size_t)(k * 32 + kq) * NHID + n, NHID);
  const bf16x8 w3 = kq < NOUT ? bf8_strided(W3 + (size_t)kq * NHID + n, NHID) : bf8_zero();
  lds_barrier();
  // Z2 = Y1b W2^T + b2, Y2 = GELU(Z2)
  {
    floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < NHID / 32; k++) acc = mfma(bf8_lds(&y1b[r][k * 32 + kq]), w2[k], acc);
    ushort4 t;
    uint16_t* tv = reinterpret_cast<uint16_t*>(&t);
#pragma unroll
    for (int q = 0; q < 4; q++) {
      z2[q] = acc[q] + bias2;
      tv[q] = f2bf(gelu(z2[q]));
      y2b[rq + q][n] = tv[q];
    }
    put(o.y2, n, t);
  }
#pragma unroll
  for (int q = 0; q < 4; q++)
    mk[q * STEP_THREADS + tid] = q * STEP_THREADS + tid < nmask ? mv[q] : 0.f;
  lds_barrier();
  // Y = Y2b W3^T + b3
  if (wv == 0) {
    floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k0 = 0; k0 < NHID; k0 += 32)
      acc = mfma(bf8_lds(&y2b[r][k0 + kq]), bf8_weights<ALIGNED>(W3 + r * NHID + k0 + kq), acc);
    const float bias3 = a.params[OFF_B3 + r];
#pragma unroll
    for (int q = 0; q < 4; q++) yv[rq + q][r] = acc[q] + bias3;
  }
  // the minibatch's mask count: thread t < 256 adds entries t, t + 256, ...
  double c = 0.0;
  for (int e0 = 0; e0 < nmask; e0 += 4096) {
    if (e0) {
      lds_barrier();
#pragma unroll
      for (int q = 0; q < 4; q++) {
        const int e = e0 + q * STEP_THREADS + tid;
        mk[q * STEP_THREADS + tid] = e < nmask ? a.Mk[(size_t)a.order[e / NOUT] * NOUT + e % NOUT] : 0.f;
      }
      lds_barrier();
    }
    if (tid >= 768)  // (not the wave of the product above)
#pragma unroll
      for (int q = 0; q < 16; q++) c += (double)mk[q * 256 + tid - 768];
  }
  if (tid >= 768) dred[tid - 768] = c;
  tree256(dred, tid);
  const double cnt = dred[0];
  // squared errors and dY = 2 mask (y - t) / sum(mask)
  if (tid < SB * NOUT) {
    double err = 0.0;
    float g = 0.f;
    if (have) {
      const double m = tm;
      const double d = (double)yv[xr][xj] - (double)tt;
      err = m * d * d;
      g = cnt > 0 ? (float)(2.0 * m * d / cnt) : 0.f;
    }
    const uint16_t gb = f2bf(g);
    dyb[xr][xj] = gb;
    o.err[(size_t)(row0 + xr) * NOUT + xj] = err;
    o.fy[(size_t)(row0 + xr) * NOUT + xj] = g;
    o.dy[(size_t)xj * Bp + row0 + xr] = gb;
  }
  if (blockIdx.x == 0 && tid == 0) *o.cnt = cnt;
  lds_barrier();
  // dY2 = dYb W3 (K = 16), dZ2 = dY2 GELU'(Z2); its bf16 copy replaces Y2
  // (y2b was read before the last barriers)
  {
    const bf16x8 av = kq < NOUT ? bf8_lds(&dyb[r][kq]) : bf8_zero();
    const floatx4 acc = mfma(av, w3, floatx4{0.f, 0.f, 0.f, 0.f});
    ushort4 t;
    uint16_t* tv = reinterpret_cast<uint16_t*>(&t);
#pragma unroll
    for (int q = 0; q < 4; q++) {
      const float g = acc[q] * gelu_grad(z2[q]);
      tv[q] = f2bf(g);
      y2b[rq + q][n] = tv[q];
      o.fz2[(size_t)(row0 + rq + q) * NHID + n] = g;
    }
    put(o.dz2, n, t);
  }
  lds_barrier();
  // dY1 = dZ2b W2, dZ1 = dY1 GELU'(Z1)
  {
    floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < NHID / 32; k++) acc = mfma(bf8_lds(&y2b[r][k * 32 + kq]), w2c[k], acc);
    ushort4 t;
    uint16_t* tv = reinterpret_cast<uint16_t*>(&t);
#pragma unroll
    for (int q = 0; q < 4; q++) {
      const float g = acc[q] * gelu_grad(z1[q]);
      tv[q] = f2bf(g);
      o.fz1[(size_t)(row0 + rq + q) * NHID + n] = g;
    }
    put(o.dz1, n, t);
  }
}

// bf16 W2, transposed (see StepArgs::w2t; k_mlp_grad_adam keeps it current).
__global__ void k_w2_transpose(const uint16_t* pb, uint16_t* w2t) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;  // over W2, row-major
  if (i < NHID * NHID) w2t[(i % NHID) * NHID + i / NHID] = pb[OFF_W2 + i];
}

struct GradArgs {
  StepOut o;
  float *grads, *p, *m, *v;
  uint16_t* pb;
  uint16_t* w2t;
  float lr, b1, omb1, b2, omb2, eps, c1, c2;
  double* loss;
};
// the Adam step of parameter i with gradient g; returns the bf16 copy
__device__ __forceinline__ uint16_t adam_step(const GradArgs& a, int64_t i, float g) {
  a.grads[i] = g;
  const float mi = a.b1 * a.m[i] + a.omb1 * g;
  const float vi = a.b2 * a.v[i] + a.omb2 * g * g;
  a.m[i] = mi;
  a.v[i] = vi;
  const float mh = mi / a.c1, vh = vi / a.c2;
  const float pi = a.p[i] - a.lr * mh / (sqrtf(vh) + a.eps);
  a.p[i] = pi;
  const uint16_t b = f2bf(pi);
  a.pb[i] = b;
  return b;
}

// Gradient = the SR-row shares summed in order, then the Adam step; the
// minibatch loss (the shares' squared errors over the mask count) into *loss.
// Blocks of one wave: W2_TILES + 32 weight tiles, BIAS_BLOCKS bias blocks, one
// for the loss.
constexpr int HT = NHID / 16, W2_TILES = HT * HT, BIAS_BLOCKS = (2 * NHID + NOUT) / 8;
constexpr int GRAD_BLOCKS = W2_TILES + 2 * HT + BIAS_BLOCKS + 1;
__global__ __launch_bounds__(64) void k_mlp_grad_adam(GradArgs a) {
  const int lane = threadIdx.x, r = lane & 15, kq = (lane >> 4) * 8, rq = (lane >> 4) * 4;
  const int blk = blockIdx.x;
  const size_t Bp = (size_t)a.o.Bp;
  const int nsh = a.o.Bp / SR;
  if (blk < W2_TILES + 2 * HT) {
    // rows of the tile: columns m0 of A; columns of the tile: columns n0 of B
    const uint16_t *A, *B;
    int m0, n0, ld;
    int64_t off;
    bool is_w2 = false;
    if (blk < W2_TILES) {
      A = a.o.dz2, B = a.o.y1, m0 = blk / HT * 16, n0 = blk % HT * 16, ld = NHID, off = OFF_W2;
      is_w2 = true;
    } else if (blk < W2_TILES + HT) {
      A = a.o.dz1, B = a.o.x, m0 = (blk - W2_TILES) * 16, n0 = 0, ld = NIN, off = OFF_W1;
    } else {
      A = a.o.dy, B = a.o.y2, m0 = 0, n0 = (blk - W2_TILES - HT) * 16, ld = NHID, off = OFF_W3;
    }
    const uint16_t* pa = A + (size_t)(m0 + r) * Bp + kq;
    const uint16_t* pbv = B + (size_t)(n0 + r) * Bp + kq;
    floatx4 g = {0.f, 0.f, 0.f, 0.f};
    for (int s0 = 0; s0 < nsh; s0 += 8) {
      bf16x8 av[8], bv[8];
#pragma unroll
      for (int u = 0; u < 8; u++) {
        const int s = min(s0 + u, nsh - 1);
        av[u] = *reinterpret_cast<const bf16x8*>(pa + s * SR);
        bv[u] = *reinterpret_cast<const bf16x8*>(pbv + s * SR);
      }
#pragma unroll
      for (int u = 0; u < 8; u++)
        if (s0 + u < nsh) {
          const floatx4 d = mfma(av[u], bv[u], floatx4{0.f, 0.f, 0.f, 0.f});
#pragma unroll
          for (int q = 0; q < 4; q++) g[q] += d[q];
        }
    }
    ushort4 t;
    uint16_t* tv = reinterpret_cast<uint16_t*>(&t);
#pragma unroll
    for (int q = 0; q < 4; q++) tv[q] = adam_step(a, off + (int64_t)(m0 + rq + q) * ld + n0 + r, g[q]);
    if (is_w2 && a.w2t)
      *reinterpret_cast<ushort4*>(a.w2t + (size_t)(n0 + r) * NHID + m0 + rq) = t;
  } else if (blk < W2_TILES + 2 * HT + BIAS_BLOCKS) {
    // eight columns, one share per lane of a column at a time
    const int col = (blk - W2_TILES - 2 * HT) * 8 + (lane & 7), sl = lane >> 3;
    const float* src;
    int ld;
    int64_t i;
    if (col < NHID) {
      src = a.o.fz1 + col, ld = NHID, i = OFF_B1 + col;
    } else if (col < 2 * NHID) {
      src = a.o.fz2 + col - NHID, ld = NHID, i = OFF_B2 + col - NHID;
    } else {
      src = a.o.fy + col - 2 * NHID, ld = NOUT, i = OFF_B3 + col - 2 * NHID;
    }
    float g = 0.f;
    for (int s0 = 0; s0 < nsh; s0 += 8) {
      const int s = min(s0 + sl, nsh - 1);
      float e[SR];
#pragma unroll
      for (int k = 0; k < SR; k++) e[k] = src[(size_t)(s * SR + k) * ld];
      float sm = 0.f;
#pragma unroll
      for (int k = 0; k < SR; k++) sm += e[k];
#pragma unroll
      for (int u = 0; u < 8; u++) {
        const float x = __shfl(sm, u * 8 + (lane & 7), 64);
        if (s0 + u < nsh) g += x;
      }
    }
    if (sl == 0) adam_step(a, i, g);
  } else {
    double e = 0.0;
    for (int s = 0; s < nsh; s++) {
      const double* d = a.o.err + (size_t)s * SR * NOUT;
      double q[4];
#pragma unroll
      for (int u = 0; u < 4; u++) q[u] = d[lane + 64 * u] + d[lane + 64 * u + 256];
      double v = (q[0] + q[2]) + (q[1] + q[3]);
#pragma unroll
      for (int h = 32; h > 0; h >>= 1) v += __shfl_down(v, h, 64);
      e += v;
    }
    const double cnt = *a.o.cnt;
    if (lane == 0) *a.loss = cnt > 0 ? e / cnt : 0.0;
  }
}

}  // namespace mlp
}  // namespace pauli
