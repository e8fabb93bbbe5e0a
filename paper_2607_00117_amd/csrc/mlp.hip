// Surrogate MLP of chi^2(theta): 12 -> 256 -> 256 -> 256 -> 1, SiLU on the
// hidden layers.  Training kernels (forward with cached activations,
// backward, Adam) work in fp32; inference runs one fused kernel with bf16
// weights and fp32 accumulation.
//
// Parameter packing (fp32): [W1 (256x12), b1 (256), W2 (256x256), b2, W3 (256x256), b3, W4 (1x256), b4 (1)],
// weights row-major [out][in].
#include <hip/hip_runtime.h>

#include "common.h"

namespace sw {

constexpr int kIn = 12, kHid = 256;
constexpr int64_t kOffW1 = 0, kOffB1 = kOffW1 + kHid * kIn, kOffW2 = kOffB1 + kHid, kOffB2 = kOffW2 + kHid * kHid,
                  kOffW3 = kOffB2 + kHid, kOffB3 = kOffW3 + kHid * kHid, kOffW4 = kOffB3 + kHid,
                  kOffB4 = kOffW4 + kHid, kNParam = kOffB4 + 1;

__device__ __forceinline__ float sigmoidf_(float z) { return 1.0f / (1.0f + __expf(-z)); }

// ---------------------------------------------------------------------------
// Matrix products on fp32 MFMA (v_mfma_f32_16x16x4f32: fp32 operands and
// sums).  Lane l supplies A[l % 16][k] and B[k][l % 16] for k = l / 16 of four
// and holds D[4 (l / 16) + r][l % 16].  The order of the inner index is free, so
// each lane takes runs of consecutive k (or consecutive columns) and reads them
// with one wide load; the loads need 4-byte alignment only (f4u, f2u).
//
// A training step was 11 launches of a 64 x 64-tile GEMM on 4 to 32 workgroups
// and four serial column sums; what bounds it is latency, not the 0.4 GFLOP.
// Now one launch carries 16 samples per workgroup through all layers (their
// activations never leave LDS between layers), one carries the gradient back
// through them, and one forms every weight and bias gradient.  Batch 512, one
// step with mlp_mse_grad and mlp_adam_step: 994 us before, 56 us now.
// ---------------------------------------------------------------------------
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
typedef float f2u __attribute__((ext_vector_type(2), aligned(4)));
constexpr int kRows = 16;         // samples per workgroup
constexpr int kLd = kHid + 4;     // LDS row stride: the 16 rows of an operand read fall in distinct banks
constexpr int kThr = 512;         // 8 waves, 32 columns each

// acc[t] = sum_k h[row][k] W[n][k] for the 16 rows of h (LDS) and the columns
// n = n0 + 16 t + l % 16 of this wave, W row-major [out][in]
__device__ __forceinline__ void layer_fwd(const float (*h)[kLd], const float* __restrict__ W, int n0, int lane,
                                          f32x4 (&acc)[2]) {
  const int i = lane & 15, g = lane >> 4;
  const float* w0 = W + (int64_t)(n0 + i) * kHid + 4 * g;
  const float* w1 = w0 + 16 * kHid;
  acc[0] = acc[1] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 8
  for (int k = 0; k < kHid; k += 16) {
    const f4u b0 = *reinterpret_cast<const f4u*>(w0 + k), b1 = *reinterpret_cast<const f4u*>(w1 + k);
    const f32x4 a = *reinterpret_cast<const f32x4*>(&h[i][k + 4 * g]);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      acc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[j], b0[j], acc[0], 0, 0, 0);
      acc[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[j], b1[j], acc[1], 0, 0, 0);
    }
  }
}

// acc[t] = sum_n h[row][n] W[n][c] for the columns c = c0 + 2 (l % 16) + t
__device__ __forceinline__ void layer_bwd(const float (*h)[kLd], const float* __restrict__ W, int c0, int lane,
                                          f32x4 (&acc)[2]) {
  const int i = lane & 15, g = lane >> 4;
  const float* w = W + (int64_t)(4 * g) * kHid + c0 + 2 * i;
  acc[0] = acc[1] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 4
  for (int k = 0; k < kHid; k += 16) {
    f2u b[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) b[j] = *reinterpret_cast<const f2u*>(w + (int64_t)(k + j) * kHid);
    const f32x4 a = *reinterpret_cast<const f32x4*>(&h[i][k + 4 * g]);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      acc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[j], b[j][0], acc[0], 0, 0, 0);
      acc[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[j], b[j][1], acc[1], 0, 0, 0);
    }
  }
}

// Forward pass of 16 samples per workgroup; keeps a_l = silu(z_l) and
// d_l = silu'(z_l) of the hidden layers (act: a_1, a_2, a_3, d_1, d_2, d_3, [B][256] each).
__global__ __launch_bounds__(kThr) void k_mlp_fwd(const float* __restrict__ p, const float* __restrict__ x, int64_t B,
                                                  float* __restrict__ y, float* __restrict__ act) {
  __shared__ __attribute__((aligned(16))) float h[2][kRows][kLd];
  __shared__ float xin[kRows][kIn];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int64_t r0 = (int64_t)blockIdx.x * kRows, S = B * kHid;
  const int nr = (int)(B - r0 < kRows ? B - r0 : kRows);
  if (tid < kRows * kIn) xin[tid / kIn][tid % kIn] = tid < nr * kIn ? x[r0 * kIn + tid] : 0.0f;
  __syncthreads();
  // hidden unit n of layer l, row r
  auto put = [&](int l, int buf, int r, int n, float z) {
    const float s = sigmoidf_(z), a = z * s;
    h[buf][r][n] = a;
    if (r < nr) {
      const int64_t at = (r0 + r) * kHid + n;
      act[l * S + at] = a;
      act[(l + 3) * S + at] = s * (1.0f + z * (1.0f - s));
    }
  };
  {
    const int n = tid & (kHid - 1);
    float wr[kIn];
#pragma unroll
    for (int c = 0; c < kIn; ++c) wr[c] = p[kOffW1 + n * kIn + c];
    const float bb = p[kOffB1 + n];
    for (int r = tid / kHid; r < kRows; r += kThr / kHid) {
      float z = 0.0f;
#pragma unroll
      for (int c = 0; c < kIn; ++c) z += wr[c] * xin[r][c];
      put(0, 0, r, n, z + bb);
    }
  }
  __syncthreads();
#pragma unroll
  for (int l = 1; l < 3; ++l) {
    f32x4 acc[2];
    layer_fwd(h[l - 1], p + (l == 1 ? kOffW2 : kOffW3), 32 * w, lane, acc);
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int n = 32 * w + 16 * t + (lane & 15);
      const float bb = p[(l == 1 ? kOffB2 : kOffB3) + n];
#pragma unroll
      for (int r = 0; r < 4; ++r) put(l, l & 1, 4 * (lane >> 4) + r, n, acc[t][r] + bb);
    }
    __syncthreads();
  }
  for (int r = w; r < nr; r += kThr / 64) {
    float v = 0.0f;
#pragma unroll
    for (int j = 0; j < 4; ++j) v += h[0][r][4 * lane + j] * p[kOffW4 + 4 * lane + j];
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    if (lane == 0) y[r0 + r] = v + p[kOffB4];
  }
}

// dL/dz of the hidden layers for 16 samples per workgroup: dz_3 = dy w_4 d_3 (formed
// again where it is needed), dz_2 = (dz_3 W_3) d_2 and dz_1 = (dz_2 W_2) d_1 kept
__global__ __launch_bounds__(kThr) void k_mlp_bwd(const float* __restrict__ p, const float* __restrict__ dy, int64_t B,
                                                  const float* __restrict__ act, float* __restrict__ dz1,
                                                  float* __restrict__ dz2) {
  __shared__ __attribute__((aligned(16))) float h[2][kRows][kLd];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int64_t r0 = (int64_t)blockIdx.x * kRows, S = B * kHid;
  const int nr = (int)(B - r0 < kRows ? B - r0 : kRows);
  {
    const int n = tid & (kHid - 1);
    const float w4 = p[kOffW4 + n];
#pragma unroll
    for (int q = 0; q < kRows / 2; ++q) {
      const int r = tid / kHid + 2 * q;
      h[0][r][n] = r < nr ? dy[r0 + r] * w4 * act[5 * S + (r0 + r) * kHid + n] : 0.0f;
    }
  }
  __syncthreads();
#pragma unroll
  for (int l = 0; l < 2; ++l) {  // through W_3, then W_2
    f32x4 acc[2];
    layer_bwd(h[l], p + (l == 0 ? kOffW3 : kOffW2), 32 * w, lane, acc);
    const float* d = act + (l == 0 ? 4 : 3) * S;
    float* out = l == 0 ? dz2 : dz1;
    const int c = 32 * w + 2 * (lane & 15);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = 4 * (lane >> 4) + r;
      f2u v = {0.0f, 0.0f};
      if (row < nr) {
        const int64_t at = (r0 + row) * kHid + c;
        const f2u dd = *reinterpret_cast<const f2u*>(d + at);
        v = f2u{acc[0][r] * dd[0], acc[1][r] * dd[1]};
        *reinterpret_cast<f2u*>(out + at) = v;
      }
      h[l ^ 1][row][c] = v[0];
      h[l ^ 1][row][c + 1] = v[1];
    }
    __syncthreads();
  }
}

// Gradients of the parameters.  Workgroups 0..127: a 32 x 32 tile of dW_3 (then
// dW_2), dW[n][k] = sum_b dz[b][n] a[b][k], the samples dealt to the 8 waves in
// runs of four and the waves' sums added in order.  The last 16: 16 columns each
// of the bias gradients, dW_4 and dW_1, 32 sample slices added by a fixed tree.
constexpr int kGradTiles = (kHid / 32) * (kHid / 32);
constexpr int kSumCols = 16, kSlices = kThr / kSumCols, kSums = 5 + kIn;

__global__ __launch_bounds__(kThr) void k_mlp_grad(const float* __restrict__ p, const float* __restrict__ x,
                                                   const float* __restrict__ dy, int64_t B,
                                                   const float* __restrict__ act, const float* __restrict__ dz1,
                                                   const float* __restrict__ dz2, float* __restrict__ grad) {
  __shared__ float red[kThr * kSums];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int64_t S = B * kHid;
  if (blockIdx.x < 2 * kGradTiles) {
    const bool top = blockIdx.x < kGradTiles;  // layer 3, whose dz is formed here
    const int q = blockIdx.x % kGradTiles;
    const int m0 = (q / (kHid / 32)) * 32, c0 = (q % (kHid / 32)) * 32, i = lane & 15, g = lane >> 4;
    const float* dz = (top ? act + 5 * S : dz2) + m0 + 2 * i;
    const float* a = act + (top ? S : 0) + c0 + 2 * i;
    const f2u w4 = *reinterpret_cast<const f2u*>(p + kOffW4 + m0 + 2 * i);
    f32x4 acc[2][2];
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[t >> 1][t & 1] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    constexpr int U = 4;  // sample runs in flight
    for (int64_t b0 = 4 * w; b0 < B; b0 += 4 * 8 * U) {
      f2u dv[U], av[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t b = b0 + 32 * u + g;
        const bool ok = b < B;
        const int64_t at = (ok ? b : 0) * kHid;
        dv[u] = *reinterpret_cast<const f2u*>(dz + at);
        av[u] = *reinterpret_cast<const f2u*>(a + at);
        const float s = dy[ok ? b : 0];
        if (top) dv[u] = f2u{s * w4[0] * dv[u][0], s * w4[1] * dv[u][1]};
        if (!ok) dv[u] = av[u] = f2u{0.0f, 0.0f};
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int t = 0; t < 4; ++t)
          acc[t >> 1][t & 1] =
              __builtin_amdgcn_mfma_f32_16x16x4f32(dv[u][t >> 1], av[u][t & 1], acc[t >> 1][t & 1], 0, 0, 0);
    }
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        red[w * 1024 + (2 * (4 * g + r) + (t >> 1)) * 32 + 2 * i + (t & 1)] = acc[t >> 1][t & 1][r];
    __syncthreads();
    float* out = grad + (top ? kOffW3 : kOffW2);
    for (int e = tid; e < 1024; e += kThr) {
      float v = red[e];
#pragma unroll
      for (int u = 1; u < 8; ++u) v += red[u * 1024 + e];
      out[(int64_t)(m0 + e / 32) * kHid + c0 + e % 32] = v;
    }
    return;
  }
  const int n = (blockIdx.x - 2 * kGradTiles) * kSumCols + tid % kSumCols, sl = tid / kSumCols;
  const float w4 = p[kOffW4 + n];
  float s[kSums] = {};  // db_1, db_2, db_3, dW_4, db_4, dW_1
#pragma unroll 4
  for (int64_t b = sl; b < B; b += kSlices) {
    const int64_t at = b * kHid + n;
    const float e = dy[b], d1 = dz1[at];
    s[0] += d1;
    s[1] += dz2[at];
    s[2] += e * w4 * act[5 * S + at];
    s[3] += e * act[2 * S + at];
    s[4] += e;
#pragma unroll
    for (int c = 0; c < kIn; ++c) s[5 + c] += d1 * x[b * kIn + c];
  }
#pragma unroll
  for (int k = 0; k < kSums; ++k) red[k * kThr + tid] = s[k];
  __syncthreads();
  for (int o = kSlices / 2; o > 0; o >>= 1) {
    if (sl < o)
      for (int k = 0; k < kSums; ++k) red[k * kThr + tid] += red[k * kThr + tid + o * kSumCols];
    __syncthreads();
  }
  if (sl == 0) {
    grad[kOffB1 + n] = red[tid];
    grad[kOffB2 + n] = red[kThr + tid];
    grad[kOffB3 + n] = red[2 * kThr + tid];
    grad[kOffW4 + n] = red[3 * kThr + tid];
    if (n == 0) grad[kOffB4] = red[4 * kThr];
    for (int c = 0; c < kIn; ++c) grad[kOffW1 + n * kIn + c] = red[(5 + c) * kThr + tid];
  }
}

__global__ void k_adam(float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m, float* __restrict__ v,
                       int64_t n, float lr, float b1, float b2, float eps, float c1, float c2) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.0f - b1) * gi;
  const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

__global__ void k_mse_grad(const float* __restrict__ y, const float* __restrict__ t, int64_t B,
                           float* __restrict__ dy) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < B) dy[i] = 2.0f * (y[i] - t[i]) / (float)B;
}

__global__ void k_to_bf16(const float* __restrict__ p, __bf16* __restrict__ q, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) q[i] = (__bf16)p[i];
}

// Fused inference, 16 samples per workgroup through all layers in LDS; bf16
// weights widened exactly and multiplied in fp32 on MFMA with fp32 sums.  A lane
// reads 8 consecutive weights of a row at a time (16 rows x 64 bytes per wave);
// the previous kernel's lanes walked one row each, 512 bytes apart.  32 samples
// (the sampler's screen) are two workgroups and bound by latency: 87 us before,
// 15.5 us now (50,000: 137 us).
typedef __bf16 bf8u __attribute__((ext_vector_type(8), aligned(2)));

__global__ __launch_bounds__(kThr) void k_mlp_infer_bf16(const __bf16* __restrict__ q, const float* __restrict__ x,
                                                         int64_t B, float* __restrict__ y) {
  __shared__ __attribute__((aligned(16))) float h[2][kRows][kLd];
  __shared__ float xin[kRows][kIn];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, i = lane & 15, g = lane >> 4;
  const int64_t r0 = (int64_t)blockIdx.x * kRows;
  const int nr = (int)(B - r0 < kRows ? B - r0 : kRows);
  if (tid < kRows * kIn) xin[tid / kIn][tid % kIn] = tid < nr * kIn ? x[r0 * kIn + tid] : 0.0f;
  __syncthreads();
  {
    const int n = tid & (kHid - 1);
    float wr[kIn];
#pragma unroll
    for (int c = 0; c < kIn; ++c) wr[c] = (float)q[kOffW1 + n * kIn + c];
    const float bb = (float)q[kOffB1 + n];
    for (int r = tid / kHid; r < kRows; r += kThr / kHid) {
      float z = bb;
#pragma unroll
      for (int c = 0; c < kIn; ++c) z += wr[c] * xin[r][c];
      h[0][r][n] = z * sigmoidf_(z);
    }
  }
  __syncthreads();
#pragma unroll
  for (int l = 1; l < 3; ++l) {
    const __bf16* w0 = q + (l == 1 ? kOffW2 : kOffW3) + (int64_t)(32 * w + i) * kHid + 8 * g;
    const float* hr = &h[l - 1][i][8 * g];
    f32x4 acc[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const float bb = (float)q[(l == 1 ? kOffB2 : kOffB3) + 32 * w + 16 * t + i];
      acc[t] = f32x4{bb, bb, bb, bb};
    }
#pragma unroll
    for (int k = 0; k < kHid; k += 32) {
      const bf8u b0 = *reinterpret_cast<const bf8u*>(w0 + k);
      const bf8u b1 = *reinterpret_cast<const bf8u*>(w0 + 16 * kHid + k);
      const f32x4 a0 = *reinterpret_cast<const f32x4*>(hr + k), a1 = *reinterpret_cast<const f32x4*>(hr + k + 4);
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const float a = j < 4 ? a0[j & 3] : a1[j & 3];
        acc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, (float)b0[j], acc[0], 0, 0, 0);
        acc[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, (float)b1[j], acc[1], 0, 0, 0);
      }
    }
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) h[l & 1][4 * g + r][32 * w + 16 * t + i] = acc[t][r] * sigmoidf_(acc[t][r]);
    __syncthreads();
  }
  for (int r = w; r < nr; r += kThr / 64) {
    float v = 0.0f;
#pragma unroll
    for (int j = 0; j < 4; ++j) v += h[0][r][4 * lane + j] * (float)q[kOffW4 + 4 * lane + j];
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    if (lane == 0) y[r0 + r] = v + (float)q[kOffB4];
  }
}

// workspace: a_1, a_2, a_3, d_1, d_2, d_3 of mlp_forward, then dz_1, dz_2 of mlp_backward ([B][256] each)
static size_t act_bytes(int64_t B) { return (size_t)B * kHid * 4; }

}  // namespace sw

using namespace sw;

extern "C" int64_t mlp_param_count(void) { return kNParam; }

extern "C" size_t mlp_workspace_bytes(int64_t batch) { return batch > 0 ? 8 * act_bytes(batch) : 0; }

extern "C" int mlp_forward(const float* params, const float* x, int64_t B, float* y, void* workspace, size_t ws_bytes,
                           void* stream) {
  SW_CHECK(params && x && y && workspace, "mlp_forward: null argument");
  SW_CHECK(B > 0 && B < (1 << 30), "mlp_forward: bad batch");
  SW_CHECK(ws_bytes >= mlp_workspace_bytes(B), "mlp_forward: workspace too small");
  hipStream_t st = (hipStream_t)stream;
  hipLaunchKernelGGL(k_mlp_fwd, dim3((unsigned)((B + kRows - 1) / kRows)), dim3(kThr), 0, st, params, x, B, y,
                     (float*)workspace);
  SW_HIP(hipGetLastError());
  return SW_OK;
}

// Gradients of sum_b dy[b] * y[b] with respect to the parameters, using the
// activations cached by mlp_forward on the same x and params.
extern "C" int mlp_backward(const float* params, const float* x, int64_t B, const float* dy, float* grad,
                            void* workspace, size_t ws_bytes, void* stream) {
  SW_CHECK(params && x && dy && grad && workspace, "mlp_backward: null argument");
  SW_CHECK(B > 0 && B < (1 << 30), "mlp_backward: bad batch");
  SW_CHECK(ws_bytes >= mlp_workspace_bytes(B), "mlp_backward: workspace too small");
  hipStream_t st = (hipStream_t)stream;
  float* act = (float*)workspace;
  float *dz1 = act + 6 * B * kHid, *dz2 = act + 7 * B * kHid;
  hipLaunchKernelGGL(k_mlp_bwd, dim3((unsigned)((B + kRows - 1) / kRows)), dim3(kThr), 0, st, params, dy, B,
                     (const float*)act, dz1, dz2);
  hipLaunchKernelGGL(k_mlp_grad, dim3(2 * kGradTiles + kHid / kSumCols), dim3(kThr), 0, st, params, x, dy, B,
                     (const float*)act, (const float*)dz1, (const float*)dz2, grad);
  SW_HIP(hipGetLastError());
  return SW_OK;
}

extern "C" int mlp_adam_step(float* params, const float* grad, float* m, float* v, int64_t n, int32_t t, float lr,
                             float beta1, float beta2, float eps, void* stream) {
  SW_CHECK(params && grad && m && v, "mlp_adam_step: null argument");
  SW_CHECK(n > 0 && t >= 1, "mlp_adam_step: need n > 0 and t >= 1");
  const float c1 = 1.0f - powf(beta1, (float)t), c2 = 1.0f - powf(beta2, (float)t);
  hipLaunchKernelGGL(k_adam, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, (hipStream_t)stream, params, grad, m, v,
                     n, lr, beta1, beta2, eps, c1, c2);
  SW_HIP(hipGetLastError());
  return SW_OK;
}

// dL/dy of L = mean_b (y_b - t_b)^2
extern "C" int mlp_mse_grad(const float* y, const float* t, int64_t B, float* dy, void* stream) {
  SW_CHECK(y && t && dy && B > 0, "mlp_mse_grad: bad argument");
  hipLaunchKernelGGL(k_mse_grad, dim3((unsigned)((B + 255) / 256)), dim3(256), 0, (hipStream_t)stream, y, t, B, dy);
  SW_HIP(hipGetLastError());
  return SW_OK;
}

extern "C" int mlp_pack_bf16(const float* params, void* packed, void* stream) {
  SW_CHECK(params && packed, "mlp_pack_bf16: null argument");
  hipLaunchKernelGGL(k_to_bf16, dim3((unsigned)((kNParam + 255) / 256)), dim3(256), 0, (hipStream_t)stream, params,
                     (__bf16*)packed, kNParam);
  SW_HIP(hipGetLastError());
  return SW_OK;
}

extern "C" int mlp_infer_bf16(const void* packed, const float* x, int64_t B, float* y, void* stream) {
  SW_CHECK(packed && x && y, "mlp_infer_bf16: null argument");
  SW_CHECK(B >= 0, "mlp_infer_bf16: bad batch");
  if (B == 0) return SW_OK;
  // a launch of 2^32 threads or more (32 a sample) would start their number modulo 2^32
  constexpr int64_t kPer = (int64_t)1 << 26;
  for (int64_t b = 0; b < B; b += kPer) {
    const int64_t n = B - b < kPer ? B - b : kPer;
    hipLaunchKernelGGL(k_mlp_infer_bf16, dim3((unsigned)((n + kRows - 1) / kRows)), dim3(kThr), 0,
                       (hipStream_t)stream, (const __bf16*)packed, x + b * kIn, n, y + b);
    SW_HIP(hipGetLastError());
  }
  return SW_OK;
}
