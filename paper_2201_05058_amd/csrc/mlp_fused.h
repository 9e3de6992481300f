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

}  // namespace pcsdf
