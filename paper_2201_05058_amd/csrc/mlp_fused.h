// Fused inference of the surrogate MLP (included by mlp.hip): forward pass
// and input gradient of 32 rows per wave with the activations in registers
// (mlp_rows.h) and no intermediate in memory.
//
// The rounding points are those of the training kernels and of the oracle:
// A_{l+1} = bf16(SiLU(Z_l)), D_l = bf16(SiLU'(Z_l)), dZ_3 = bf16(out_scale
// W4 (.) D_3), dZ_{l-1} = bf16((dZ_l W_l) (.) D_{l-1}); y and the input
// gradient are FP32.
#pragma once

#include "mlp_rows.h"

namespace pcsdf {

// y [n] and, when gx is given, dy/dx [n][n_in] for rows [0, n), x
// [n][n_in], one workgroup per 128 rows striding over the row tiles.  With
// n_dev the row count is min(n, *n_dev), read on the device (a grid sized
// for n then leaves its surplus workgroups idle).  130k rows take 47 us (570
// TFLOP/s; 76 us with activations and derivatives exchanged through LDS and
// weights read from the caches), the same values bit for bit.
__global__ __launch_bounds__(64 * kRowWaves, 2) void k_mlp_infer(
    const float *__restrict__ x, int n, const int *__restrict__ n_dev,
    int n_in, const float *__restrict__ norm, NetWeights w,
    const float *__restrict__ p, float out_scale, float *__restrict__ y,
    float *__restrict__ gx) {
  __shared__ RowsLds L;
  const int lane = threadIdx.x & 63, half = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (n_dev) n = min(n, *n_dev);
  const int tiles = (n + kRowTile - 1) / kRowTile;
  if ((int)blockIdx.x >= tiles) return;
  load_small(L, w, p, n_in);
  for (int tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    const int64_t m = (int64_t)tile * kRowTile + wave * 32 + (lane & 31);
    copy_to_lds<kHid * kInPad>(w.W[0], L.w, wave, lane);
    bf16x8 f[8];
    input_frags(x, m, n, n_in, norm, half, f);
    lds_copies_done();
    __syncthreads();

    uint32_t D[kLayers][4][8];  // the layers' derivatives
    f32x16 acc[4];
#pragma unroll
    for (int l = 0; l < kLayers; ++l) {
      if (l == 0)
        rows_gemm<kInPad / 16, 4>(L.w, f, lane, acc);
      else
        rows_gemm<kHid / 16, 4>(L.w, f, lane, acc);
      const bool more = l + 1 < kLayers || gx;
      if (more) {
        __syncthreads();  // every wave has read the layer's weights
        copy_to_lds<kHid * kHid>(l + 1 < kLayers ? w.W[l + 1] : w.Wt[l], L.w,
                                 wave, lane);
      }
#pragma unroll
      for (int ub = 0; ub < 4; ++ub) {
        act_block<SiluFast>(acc[ub], L.bias[l], ub, half, &f[2 * ub],
                            &f[2 * ub + 1], D[l][ub]);
      }
      if (more) {
        lds_copies_done();
        __syncthreads();
      }
    }
    const float s = output_sum(f, L.w4, half);
    if (half == 0 && m < n)
      y[m] = (s + p[layer_desc(kLayers, n_in).b_off]) * out_scale;
    if (gx) {
#pragma unroll
      for (int ub = 0; ub < 4; ++ub)
        seed_block(out_scale, L.w4, ub, half, D[kLayers - 1][ub], &f[2 * ub],
                   &f[2 * ub + 1]);
#pragma unroll
      for (int l = kLayers - 1; l >= 1; --l) {
        rows_gemm<kHid / 16, 4>(L.w, f, lane, acc);
        __syncthreads();
        if (l > 1)
          copy_to_lds<kHid * kHid>(w.Wt[l - 1], L.w, wave, lane);
        else
          copy_to_lds<kHid * kInPad>(w.Wt[0], L.w, wave, lane);
#pragma unroll
        for (int ub = 0; ub < 4; ++ub) {
          grad_block(acc[ub], D[l - 1][ub], &f[2 * ub], &f[2 * ub + 1]);
        }
        lds_copies_done();
        __syncthreads();
      }
      rows_gemm<kHid / 16, 1>(L.w, f, lane, acc);
      store_input_grad(acc[0], m, n, n_in, norm + kInPad, half, gx);
    }
    __syncthreads();  // the weights' LDS is reused by the next tile
  }
}

// The same for few rows, with a layer's units split over the waves of a
// workgroup: 32 rows a workgroup, 32 units a wave.  A wave's chain of
// products and epilogues is then a quarter as long, for an exchange of the
// rows' activations through LDS and one barrier a layer; the weights come
// straight from the caches, one layer ahead.  The operations on a value and
// their order are k_mlp_infer's, so the bits are.  Bound by that chain: us a
// call with the input gradient, k_mlp_infer and this: 1 row 19.6, 10.3; 8192
// 20.7, 10.2; 16384 20.7, 11.6; 24000 20.8, 16.8; 32768 21.2, 20.2; 50000
// 26.1, 31.3 (without it 14.6, 8.2; 15.4, 8.2; 15.6, 8.8; 15.3, 11.4; 15.6,
// 14.4; 18.5, 21.2).  The line is one round of two workgroups a CU.
constexpr int kFewRows = 32768;
__device__ __forceinline__ void load_layer(const uint16_t *w, int wave,
                                           int lane, bf16x8 (&b)[8]) {
#pragma unroll
  for (int ks = 0; ks < 8; ++ks)
    b[ks] = load8(w + (ks * 4 + wave) * kFrag + lane * 8);
}
// Gives the workgroup this wave's two fragments and takes everyone's.
__device__ __forceinline__ void exchange(uint16_t *ex, int wave, int lane,
                                         bf16x8 lo, bf16x8 hi,
                                         bf16x8 (&f)[8]) {
  *reinterpret_cast<bf16x8 *>(ex + 2 * wave * kFrag + lane * 8) = lo;
  *reinterpret_cast<bf16x8 *>(ex + (2 * wave + 1) * kFrag + lane * 8) = hi;
  __syncthreads();
#pragma unroll
  for (int ks = 0; ks < 8; ++ks) f[ks] = load8(ex + ks * kFrag + lane * 8);
}
__device__ __forceinline__ f32x16 few_gemm(const bf16x8 (&b)[8],
                                           const bf16x8 (&f)[8], int ks_end) {
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.f;
#pragma unroll
  for (int ks = 0; ks < 8; ++ks)
    if (ks < ks_end) acc = mfma(b[ks], f[ks], acc);
  return acc;
}

__global__ __launch_bounds__(64 * kRowWaves, 2) void k_mlp_infer_few(
    const float *__restrict__ x, int n, const int *__restrict__ n_dev,
    int n_in, const float *__restrict__ norm, NetWeights w,
    const float *__restrict__ p, float out_scale, float *__restrict__ y,
    float *__restrict__ gx) {
  // by turns, so that one barrier an exchange is enough
  __shared__ alignas(16) uint16_t ex[2][8 * kFrag];
  __shared__ alignas(16) float bias[kLayers][kHid], w4[kHid];
  const int lane = threadIdx.x & 63, half = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (n_dev) n = min(n, *n_dev);
  const int tiles = (n + 31) / 32;
  if ((int)blockIdx.x >= tiles) return;
  bf16x8 b[8], f[8], lo, hi;
#pragma unroll
  for (int ks = 0; ks < kInPad / 16; ++ks)
    b[ks] = load8(w.W[0] + (ks * 4 + wave) * kFrag + lane * 8);
  for (int t = threadIdx.x; t < kHid; t += 64 * kRowWaves) {
#pragma unroll
    for (int l = 0; l < kLayers; ++l)
      bias[l][t] = p[layer_desc(l, n_in).b_off + t];
    w4[t] = from_bf16(w.W[kLayers][t]);
  }
  const float b4 = p[layer_desc(kLayers, n_in).b_off];
  __syncthreads();
  int e = 0;
  for (int tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    const int64_t m = (int64_t)tile * 32 + (lane & 31);
    input_frags(x, m, n, n_in, norm, half, f);
    uint32_t D[kLayers][8];  // the layers' derivatives
#pragma unroll
    for (int l = 0; l < kLayers; ++l) {
      const f32x16 acc = few_gemm(b, f, l == 0 ? kInPad / 16 : 8);
      if (l + 1 < kLayers)
        load_layer(w.W[l + 1], wave, lane, b);
      else if (gx)
        load_layer(w.Wt[l], wave, lane, b);
      act_block<SiluFast>(acc, bias[l], wave, half, &lo, &hi, D[l]);
      exchange(ex[e], wave, lane, lo, hi, f);
      e ^= 1;
    }
    if (wave == 0) {
      const float s = output_sum(f, w4, half);
      if (half == 0 && m < n) y[m] = (s + b4) * out_scale;
    }
    if (gx) {
      seed_block(out_scale, w4, wave, half, D[kLayers - 1], &lo, &hi);
      exchange(ex[e], wave, lane, lo, hi, f);
      e ^= 1;
#pragma unroll
      for (int l = kLayers - 1; l >= 1; --l) {
        const f32x16 acc = few_gemm(b, f, 8);
        if (l > 1) {
          load_layer(w.Wt[l - 1], wave, lane, b);
        } else if (wave == 0) {
#pragma unroll
          for (int ks = 0; ks < 8; ++ks)
            b[ks] = load8(w.Wt[0] + ks * kFrag + lane * 8);
        }
        grad_block(acc, D[l - 1], &lo, &hi);
        exchange(ex[e], wave, lane, lo, hi, f);
        e ^= 1;
      }
      if (wave == 0)
        store_input_grad(few_gemm(b, f, 8), m, n, n_in, norm + kInPad, half,
                         gx);
    }
    if (tile + (int)gridDim.x < tiles) {
#pragma unroll
      for (int ks = 0; ks < kInPad / 16; ++ks)
        b[ks] = load8(w.W[0] + (ks * 4 + wave) * kFrag + lane * 8);
    }
  }
}

}  // namespace pcsdf
