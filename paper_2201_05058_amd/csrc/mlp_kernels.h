// Kernels of the surrogate MLP (included by mlp.hip).
#pragma once

// Learned surrogate for sphere queries: an n_in -> 4 x 128 SiLU -> 1 MLP
// (n_in <= 32 inputs, padded to 32 columns) with BF16 operands and FP32
// accumulation on the matrix cores, its input gradient by reverse mode,
// and its training (weight gradients + Adam).
//
// Every product of the network is a dense contraction with one dimension
// of 128, so each layer is one MFMA GEMM over a batch of rows:
//   forward    Z_l  = A_l W_l^T + b_l,   A_{l+1} = bf16(SiLU(Z_l)),
//                                       D_l     = bf16(SiLU'(Z_l));
//   backward   dA_l = dZ_l W_l,          dZ_{l-1} = bf16(dA_l * D_{l-1});
//   weights    dW_l = dZ_l^T A_l (a reduction over the batch).
// The BF16 rounding points are exactly those of the CPU oracle.
//
// Matrix-core tile: v_mfma_f32_32x32x16_bf16.  For a 32-row by 32-column
// output block and a 16-deep slice of the contraction, lane l supplies
// A[row l%32][k 8*(l/32) .. +7] and B[k 8*(l/32) .. +7][col l%32] as eight
// BF16 values each, and receives output element
// (row 8*(r/4) + 4*(l/32) + r%4, col l%32) in accumulator register r.
// A wave owns 32 rows of the batch and all 128 units of every layer, with
// the weights as the first operand, so that a lane's accumulators are
// units of its own row and the next layer's operand is built from them in
// registers (mlp_rows.h).
#include <cmath>
#include <cstring>
#include <vector>

#include "internal.h"

namespace pcsdf {

constexpr int kInPad = 32, kHid = 128, kLayers = 4;
// Parameters of a network with n_in inputs: W0 [128][n_in] and the rest.
__host__ __device__ constexpr int mlp_nparam(int n_in) {
  return kHid * n_in + kHid + 3 * (kHid * kHid + kHid) + kHid + 1;
}

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ uint16_t to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);  // round to nearest, ties to even
  return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float from_bf16(uint16_t h) {
  return __uint_as_float((uint32_t)h << 16);
}
__device__ __forceinline__ f32x16 mfma(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ bf16x8 load8(const uint16_t *p) {
  return *reinterpret_cast<const bf16x8 *>(p);
}

// The BF16 weight copies of the hidden layers lie in the order in which the
// matrix cores read them: for the 16-deep contraction slice ks and the
// 32-unit block ub the 64 lanes' operands of eight values are consecutive
// (fragment ks * (units / 32) + ub, 1 KB), so that a wave's operand is one
// contiguous 1 KB read, from memory or from LDS without bank conflicts.
// Element (unit u, contraction index c) of a matrix of `units` rows:
__host__ __device__ constexpr int frag_at(int u, int c, int units) {
  return (((c >> 4) * (units >> 5) + (u >> 5)) * 64 + (u & 31) +
          32 * ((c >> 3) & 1)) * 8 + (c & 7);
}
constexpr int kFrag = 64 * 8;  // elements of one fragment

// Two fp32 values to BF16 by round-to-nearest-even in one hardware
// conversion (the same rounding as to_bf16 for finite values): a in the
// low half, b in the high half.
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t cvt2(float a, float b) {
  const f32x2_t v = {a, b};
  const bf16x2_t r = __builtin_convertvector(v, bf16x2_t);
  return __builtin_bit_cast(uint32_t, r);
}
__device__ __forceinline__ uint16_t lo16(uint32_t v) { return (uint16_t)v; }
__device__ __forceinline__ uint16_t hi16(uint32_t v) {
  return (uint16_t)(v >> 16);
}

// Per-layer geometry of the flat parameter vector.
struct LayerDesc {
  int w_off, b_off, out, in, in_pad;
};
__host__ __device__ inline LayerDesc layer_desc(int l, int n_in) {
  // W0[128][n_in] b0 W1 b1 W2 b2 W3 b3 W4[1][128] b4
  const int sizes_in[5] = {n_in, kHid, kHid, kHid, kHid};
  const int sizes_out[5] = {kHid, kHid, kHid, kHid, 1};
  int off = 0;
  for (int q = 0; q < l; ++q) off += sizes_out[q] * sizes_in[q] + sizes_out[q];
  LayerDesc d;
  d.w_off = off;
  d.b_off = off + sizes_out[l] * sizes_in[l];
  d.out = sizes_out[l];
  d.in = sizes_in[l];
  d.in_pad = l == 0 ? kInPad : sizes_in[l];
  return d;
}

// Adam on the fp32 masters, then refresh the BF16 weights W_l (rows: units,
// contraction over the inputs) and their transposes Wt_l (rows: inputs,
// contraction over the units), in fragment order; W_4 [128] plain.  Padding
// inputs stay zero.
__global__ __launch_bounds__(256) void k_adam(
    float *__restrict__ p, const float *__restrict__ g, float *__restrict__ m1,
    float *__restrict__ m2, float lr, float b1, float b2, float eps,
    float c1, float c2, uint16_t *__restrict__ wbf, uint16_t *__restrict__ wtbf,
    const int *__restrict__ wofs, int n_in) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= mlp_nparam(n_in)) return;
  const float gi = g[i];
  const float a = b1 * m1[i] + (1.f - b1) * gi;
  const float v = b2 * m2[i] + (1.f - b2) * gi * gi;
  m1[i] = a;
  m2[i] = v;
  const float th = p[i] - lr * (a / c1) / (sqrtf(v / c2) + eps);
  p[i] = th;
  for (int l = 0; l <= kLayers; ++l) {
    const LayerDesc d = layer_desc(l, n_in);
    if (i >= d.w_off && i < d.b_off) {
      const int o = (i - d.w_off) / d.in, c = (i - d.w_off) - o * d.in;
      const uint16_t hb = to_bf16(th);
      wbf[wofs[l] + (l < kLayers ? frag_at(o, c, kHid) : c)] = hb;
      if (l < kLayers) wtbf[wofs[l] + frag_at(c, o, d.in_pad)] = hb;
    }
  }
}

// BF16 copies of every weight matrix from the fp32 masters.
__global__ __launch_bounds__(256) void k_cast_weights(
    const float *__restrict__ p, uint16_t *__restrict__ wbf,
    uint16_t *__restrict__ wtbf, const int *__restrict__ wofs, int n_in) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= mlp_nparam(n_in)) return;
  for (int l = 0; l <= kLayers; ++l) {
    const LayerDesc d = layer_desc(l, n_in);
    if (i >= d.w_off && i < d.b_off) {
      const int o = (i - d.w_off) / d.in, c = (i - d.w_off) - o * d.in;
      const uint16_t hb = to_bf16(p[i]);
      wbf[wofs[l] + (l < kLayers ? frag_at(o, c, kHid) : c)] = hb;
      if (l < kLayers) wtbf[wofs[l] + frag_at(c, o, d.in_pad)] = hb;
    }
  }
}

}  // namespace pcsdf
