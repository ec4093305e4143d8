// k_mlp.h -- the warm-start network: a fully connected 6 -> 128 -> 128 -> 32
// map with GELU (z Phi(z), Phi from erff) after the two hidden layers, FP32,
// trained with a mean-squared-error loss and Adam.  Two kernels:
//   k_mlp       a workgroup takes sixteen rows at a time through the whole
//               network and, when training, back through it; the weight and
//               bias gradients accumulate in registers over its rows and go
//               to one partial gradient per workgroup
//   k_mlp_grad  the partial gradients summed in a fixed order, and the Adam
//               update with bias correction
// All products run on the FP32 matrix instruction (16 x 16 x 4): exact FP32
// products, FP32 accumulation, as the vector units give.
//
// What bounds it: a training pass over 3506 rows is 0.45 GFLOP on 86 KB of
// weights, a few microseconds of matrix work, so the launches and the length
// of each workgroup's chain of layers decide.  Separate kernels per product
// (fourteen launches, the weight gradients on one to four workgroups, the
// bias gradients one serial chain over the rows per column) took 4.2 ms per
// Adam step; these two take 23 + 7 us.
#pragma once
#include <hip/hip_runtime.h>

namespace lb {

constexpr int MLP_IN = 6, MLP_H = 128, MLP_OUT = 32;
// parameter layout: W1 [H][IN], b1 [H], W2 [H][H], b2 [H], W3 [OUT][H], b3 [OUT]
constexpr int MLP_B1 = MLP_H * MLP_IN, MLP_W2 = MLP_B1 + MLP_H, MLP_B2 = MLP_W2 + MLP_H * MLP_H;
constexpr int MLP_W3 = MLP_B2 + MLP_H, MLP_B3 = MLP_W3 + MLP_OUT * MLP_H, MLP_NPARAM = MLP_B3 + MLP_OUT;
constexpr int MLP_ROWS = 16;    // rows of one matrix tile
// workgroups of a training pass: each writes one partial gradient (86 KB), so
// fewer workgroups with more rows each trade the chain's length against the
// partials' traffic.  At 3506 rows (220 tiles) one tile per workgroup takes
// 23 + 7 us, two tiles (128 workgroups) 39 + 5 us; beyond one workgroup per
// CU the rows of a workgroup follow each other.
constexpr int MLP_PARTS = 256;

__device__ __forceinline__ float gelu(float z) { return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f)); }
__device__ __forceinline__ float gelu_grad(float z) {
  return 0.5f * (1.0f + erff(z * 0.70710678118654752f)) + z * 0.39894228040143268f * expf(-0.5f * z * z);
}

typedef float f32x4 __attribute__((ext_vector_type(4)));
// four floats at any multiple of four bytes (a caller's parameter array)
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));

// one product step: lane l holds A[l & 15][l >> 4] and B[l >> 4][l & 15];
// register r of the result is C[4 (l >> 4) + r][l & 15]
__device__ __forceinline__ f32x4 mma(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Rows [16 q, 16 q + 16) for q = blockIdx.x, + gridDim.x, ...: 256 threads,
// wave w the hidden columns [32 w, 32 w + 32) (two tiles).  Rows past B are
// zero and neither stored nor counted.  Y may be null when training.
// STAGED (one workgroup): all inputs are taken into LDS first, for an output
// array that lies over them.
template <bool TRAIN, bool STAGED = false>
__global__ __launch_bounds__(256) void k_mlp(const float* __restrict__ prm, const float* __restrict__ X,
                                             const float* __restrict__ T, int B, float invB,
                                             float* __restrict__ Y, float* __restrict__ part,
                                             double* __restrict__ lpart) {
  constexpr int LH = MLP_H + 4, LO = MLP_OUT + 4;  // padded rows: sixteen lanes of a column step through the banks
  __shared__ float sX[MLP_ROWS][16];  // inputs, zero beyond MLP_IN
  __shared__ __attribute__((aligned(16))) float sA1[MLP_ROWS][LH], sA2[MLP_ROWS][LH];
  __shared__ float sG1[TRAIN ? MLP_ROWS : 1][LH], sG2[TRAIN ? MLP_ROWS : 1][LH];  // GELU', then dZ
  __shared__ float sDY[TRAIN ? MLP_ROWS : 1][LO];
  __shared__ double sL[4];
  extern __shared__ float sAll[];  // STAGED: B * MLP_IN
  const float *W1 = prm, *b1 = prm + MLP_B1, *W2 = prm + MLP_W2, *b2 = prm + MLP_B2, *W3 = prm + MLP_W3,
              *b3 = prm + MLP_B3;
  const int t = threadIdx.x, w = t >> 6, l = t & 63, li = l & 15, lg = l >> 4;
  f32x4 g2[TRAIN ? 2 : 1][8] = {}, g3[2][2] = {}, g1[2] = {};
  float gb1 = 0.0f, gb2 = 0.0f, gb3 = 0.0f;
  double loss = 0.0;
  if constexpr (STAGED) {
    for (int i = t; i < B * MLP_IN; i += 256) sAll[i] = X[i];
    __syncthreads();
  }
  for (int q = blockIdx.x; q * MLP_ROWS < B; q += gridDim.x) {
    const int r0 = q * MLP_ROWS;
    {
      const int i = t >> 4, c = t & 15;
      float x = 0.0f;
      if (c < MLP_IN && r0 + i < B)
        x = STAGED ? sAll[(r0 + i) * MLP_IN + c] : X[(long long)(r0 + i) * MLP_IN + c];
      sX[i][c] = x;
    }
    __syncthreads();
    // layer 1
#pragma unroll
    for (int u = 0; u < 2; u++) {
      const int n = 32 * w + 16 * u + li;
      f32x4 c = {};
#pragma unroll
      for (int s = 0; s < 2; s++) {
        const int k = 4 * s + lg;
        c = mma(sX[li][k], k < MLP_IN ? W1[n * MLP_IN + k] : 0.0f, c);
      }
      const float bias = b1[n];
#pragma unroll
      for (int r = 0; r < 4; r++) {
        const float z = c[r] + bias;
        sA1[4 * lg + r][n] = gelu(z);
        if (TRAIN) sG1[4 * lg + r][n] = gelu_grad(z);
      }
    }
    __syncthreads();
    // layers 2 and 3: the order of the reduction is free, so lane group lg
    // takes entries 16 s + 4 lg .. + 3 of both operands with one 16-byte load
#pragma unroll
    for (int u = 0; u < 2; u++) {
      const int n = 32 * w + 16 * u + li;
      f32x4 c = {};
#pragma unroll
      for (int s = 0; s < 8; s++) {
        const f32x4 a = *(const f32x4*)&sA1[li][16 * s + 4 * lg];
        const f32x4 v = *(const f32x4u*)&W2[n * MLP_H + 16 * s + 4 * lg];
#pragma unroll
        for (int r = 0; r < 4; r++) c = mma(a[r], v[r], c);
      }
      const float bias = b2[n];
#pragma unroll
      for (int r = 0; r < 4; r++) {
        const float z = c[r] + bias;
        sA2[4 * lg + r][n] = gelu(z);
        if (TRAIN) sG2[4 * lg + r][n] = gelu_grad(z);
      }
    }
    __syncthreads();
    if (w < 2) {
      const int n = 16 * w + li;
      f32x4 c = {};
#pragma unroll
      for (int s = 0; s < 8; s++) {
        const f32x4 a = *(const f32x4*)&sA2[li][16 * s + 4 * lg];
        const f32x4 v = *(const f32x4u*)&W3[n * MLP_H + 16 * s + 4 * lg];
#pragma unroll
        for (int r = 0; r < 4; r++) c = mma(a[r], v[r], c);
      }
      const float bias = b3[n];
#pragma unroll
      for (int r = 0; r < 4; r++) {
        const int row = r0 + 4 * lg + r;
        const float y = c[r] + bias;
        if (TRAIN) {
          const float e = row < B ? y - T[(long long)row * MLP_OUT + n] : 0.0f;
          sDY[4 * lg + r][n] = e * invB;
          loss += (double)e * (double)e;
        } else if (row < B) {
          Y[(long long)row * MLP_OUT + n] = y;
        }
      }
    }
    if constexpr (TRAIN) {
      __syncthreads();
      // dZ2 = (dY W3) GELU'(Z2), in place of GELU'(Z2) (each lane its own entries)
#pragma unroll
      for (int u = 0; u < 2; u++) {
        const int n = 32 * w + 16 * u + li;
        f32x4 c = {};
#pragma unroll
        for (int s = 0; s < 8; s++) c = mma(sDY[li][4 * s + lg], W3[(4 * s + lg) * MLP_H + n], c);
#pragma unroll
        for (int r = 0; r < 4; r++) sG2[4 * lg + r][n] *= c[r];
      }
      __syncthreads();
      // dZ1 = (dZ2 W2) GELU'(Z1)
#pragma unroll
      for (int u = 0; u < 2; u++) {
        const int n = 32 * w + 16 * u + li;
        f32x4 c = {};
#pragma unroll
        for (int s = 0; s < 32; s++) c = mma(sG2[li][4 * s + lg], W2[(4 * s + lg) * MLP_H + n], c);
#pragma unroll
        for (int r = 0; r < 4; r++) sG1[4 * lg + r][n] *= c[r];
      }
      __syncthreads();
      // gradients: dW2 = dZ2^T A1, dW3 = dY^T A2, dW1 = dZ1^T X over the rows
#pragma unroll
      for (int s = 0; s < 4; s++) {
        const int i = 4 * s + lg;
        float a2[2], a1[2];
#pragma unroll
        for (int u = 0; u < 2; u++) {
          a2[u] = sG2[i][32 * w + 16 * u + li];
          a1[u] = sG1[i][32 * w + 16 * u + li];
        }
#pragma unroll
        for (int v = 0; v < 8; v++) {
          const float bv = sA1[i][16 * v + li];
#pragma unroll
          for (int u = 0; u < 2; u++) g2[u][v] = mma(a2[u], bv, g2[u][v]);
        }
        const float xv = sX[i][li];
#pragma unroll
        for (int u = 0; u < 2; u++) {
          g1[u] = mma(a1[u], xv, g1[u]);
          const float dy = sDY[i][16 * u + li];
#pragma unroll
          for (int v = 0; v < 2; v++) g3[u][v] = mma(dy, sA2[i][32 * w + 16 * v + li], g3[u][v]);
        }
      }
      if (t < MLP_H) {
#pragma unroll
        for (int i = 0; i < MLP_ROWS; i++) {
          gb1 += sG1[i][t];
          gb2 += sG2[i][t];
        }
      } else if (t < MLP_H + MLP_OUT) {
#pragma unroll
        for (int i = 0; i < MLP_ROWS; i++) gb3 += sDY[i][t - MLP_H];
      }
    }
    __syncthreads();  // the next rows overwrite the staged ones
  }
  if constexpr (TRAIN) {
    float* g = part + (size_t)blockIdx.x * MLP_NPARAM;
#pragma unroll
    for (int r = 0; r < 4; r++) {
      const int m = 4 * lg + r;
#pragma unroll
      for (int u = 0; u < 2; u++) {
        const int n = 32 * w + 16 * u + m;
        if (li < MLP_IN) g[n * MLP_IN + li] = g1[u][r];
#pragma unroll
        for (int v = 0; v < 8; v++) g[MLP_W2 + n * MLP_H + 16 * v + li] = g2[u][v][r];
#pragma unroll
        for (int v = 0; v < 2; v++) g[MLP_W3 + (16 * u + m) * MLP_H + 32 * w + 16 * v + li] = g3[u][v][r];
      }
    }
    if (t < MLP_H) {
      g[MLP_B1 + t] = gb1;
      g[MLP_B2 + t] = gb2;
    } else if (t < MLP_H + MLP_OUT) {
      g[MLP_B3 + t - MLP_H] = gb3;
    }
    for (int o = 32; o > 0; o >>= 1) loss += __shfl_down(loss, o, 64);
    if (l == 0) sL[w] = loss;
    __syncthreads();
    if (t == 0) lpart[blockIdx.x] = sL[0] + sL[1];  // waves 0 and 1 hold the outputs
  }
}

// g = the sum of nparts partial gradients (four interleaved runs per
// parameter, then their sum: a fixed order); with ADAM the update
// m = b1 m + (1-b1) g, v = b2 v + (1-b2) g^2,
// p -= lr * (m / (1 - b1^t)) / (sqrt(v / (1 - b2^t)) + eps)
template <bool ADAM>
__global__ __launch_bounds__(256) void k_mlp_grad(const float* __restrict__ part, int nparts, float* __restrict__ g,
                                                  float* __restrict__ p, float* __restrict__ m,
                                                  float* __restrict__ v, float lr, float b1, float b2, float eps,
                                                  float c1, float c2) {
  __shared__ float sh[4][64];
  const int j = threadIdx.x & 63, run = threadIdx.x >> 6, k = blockIdx.x * 64 + j;
  float s = 0.0f;
  if (k < MLP_NPARAM)
#pragma unroll 8
    for (int i = run; i < nparts; i += 4) s += part[(size_t)i * MLP_NPARAM + k];
  sh[run][j] = s;
  __syncthreads();
  if (run != 0 || k >= MLP_NPARAM) return;
  const float gk = (sh[0][j] + sh[1][j]) + (sh[2][j] + sh[3][j]);
  g[k] = gk;
  if constexpr (ADAM) {
    const float mk = b1 * m[k] + (1.0f - b1) * gk;
    const float vk = b2 * v[k] + (1.0f - b2) * gk * gk;
    m[k] = mk;
    v[k] = vk;
    p[k] -= lr * (mk / c1) / (sqrtf(vk / c2) + eps);
  }
}

}  // namespace lb
