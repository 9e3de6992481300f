// Gradients of the surrogate MLP over a batch (included by mlp.hip), in
// three launches:
//   k_mlp_train_rows  forward, loss seed and backward of 32 rows per wave
//                     with the activations in registers (mlp_rows.h);
//                     leaves A_0..A_4 and dZ_0..dZ_3 (bf16, in the order of
//                     the fragments) and the output seed in memory;
//   k_mlp_wgrad       per chunk of rows the products dZ_l^T A_l of every
//                     layer and the biases' sums, into partial gradients;
//   k_grad_sum        the partials summed in a fixed order.
#pragma once

#include "mlp_rows.h"

namespace pcsdf {

// Layout of one chunk's partial gradient (fp32): W1, W2, W3 [128][128],
// W0 [128][32], b0..b3 [128], W4 [128], b4.
constexpr int kPartW0 = 3 * kHid * kHid;
constexpr int kPartB = kPartW0 + kHid * kInPad;
constexpr int kPartW4 = kPartB + kLayers * kHid;
constexpr int kPartLen = kPartW4 + kHid + 4;

// A layer's activations or gradients in memory: per 32 rows the KS
// fragments of the wave that holds them, 1 KB each, so that a wave stores
// and a slab is copied in whole cache lines (row-major stores, 32 bytes per
// row and instruction, cost the row kernel 3 us more at 65,536 rows).
// Element (row r of the 32, unit u) of such a block:
__device__ __forceinline__ int block_at(int r, int u) {
  return ((u >> 4) * 64 + r + 32 * ((u >> 3) & 1)) * 8 + (u & 7);
}
template <int KS>
__device__ __forceinline__ void store_frags(uint16_t *__restrict__ dst,
                                            int64_t block, int lane,
                                            const bf16x8 (&f)[8]) {
  uint16_t *at = dst + block * (KS * kFrag) + lane * 8;
#pragma unroll
  for (int ks = 0; ks < KS; ++ks)
    *reinterpret_cast<bf16x8 *>(at + ks * kFrag) = f[ks];
}

// Rows [0, npad), npad = 128 gridDim.x; rows at or beyond n are zero
// inputs with a zero seed.  The seed is 2 (y - tgt) / n, or dy[m] when dy
// is given; sbuf[m] = seed * out_scale; lpart[wave] = the wave's sum of
// squared residuals.  act and dz hold 4 layers of `stride` elements.
//
// Bound by vector instructions and, as much again, by waits that two waves
// per SIMD do not cover: per 64 values of a layer the SiLU pair is 15
// instructions and two transcendentals (about 90 cycles) against 26 matrix
// cycles forward and back; of 41 us for 65,536 rows of 16 inputs (490
// TFLOP/s) a SIMD issues vector instructions for 19 and runs the matrix unit
// for 5, and 28 % of the waves' cycles wait for a layer's weights or for the
// barriers around them.  222 registers hold the four layers' derivatives
// (128), the accumulators (64) and one layer's fragments.  The
// layer-by-layer kernels this replaces, with activations in memory between
// them, took 135 us for the same work.
__global__ __launch_bounds__(64 * kRowWaves, 2) void k_mlp_train_rows(
    const float *__restrict__ x, int n, int n_in,
    const float *__restrict__ norm, NetWeights w, const float *__restrict__ p,
    float out_scale, const float *__restrict__ tgt,
    const float *__restrict__ dy, uint16_t *__restrict__ a0,
    uint16_t *__restrict__ act, uint16_t *__restrict__ dz, int64_t stride,
    float *__restrict__ sbuf, float *__restrict__ lpart,
    float *__restrict__ gx) {
  __shared__ RowsLds L;
  const int lane = threadIdx.x & 63, half = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t m =
      (int64_t)blockIdx.x * kRowTile + wave * 32 + (lane & 31);
  copy_to_lds<kHid * kInPad>(w.W[0], L.w, wave, lane);
  load_small(L, w, p, n_in);
  bf16x8 f[8];
  input_frags(x, m, n, n_in, norm, half, f);
  lds_copies_done();
  __syncthreads();
  const int64_t block = (int64_t)blockIdx.x * kRowWaves + wave;
  store_frags<kInPad / 16>(a0, block, lane, f);

  uint32_t D[kLayers][4][8];  // the layers' derivatives
  f32x16 acc[4];
#pragma unroll
  for (int l = 0; l < kLayers; ++l) {
    if (l == 0)
      rows_gemm<kInPad / 16, 4>(L.w, f, lane, acc);
    else
      rows_gemm<kHid / 16, 4>(L.w, f, lane, acc);
    __syncthreads();  // every wave has read the layer's weights
    copy_to_lds<kHid * kHid>(l + 1 < kLayers ? w.W[l + 1] : w.Wt[l], L.w,
                             wave, lane);
#pragma unroll
    for (int ub = 0; ub < 4; ++ub) {
      act_block<SiluTrain>(acc[ub], L.bias[l], ub, half, &f[2 * ub],
                           &f[2 * ub + 1], D[l][ub]);
    }
    lds_copies_done();
    __syncthreads();
    // stored here, so that the wait above never waits for them: they have
    // the next product and epilogue to complete
    store_frags<8>(act + l * stride, block, lane, f);
  }

  const float y =
      (output_sum(f, L.w4, half) + p[layer_desc(kLayers, n_in).b_off]) *
      out_scale;
  float seed = 0.f, r2 = 0.f;
  if (m < n) {
    if (dy) {
      seed = dy[m];
    } else {
      const float r = y - tgt[m];
      seed = 2.f * r / (float)n;
      r2 = half == 0 ? r * r : 0.f;
    }
  }
  const float s = seed * out_scale;
  if (half == 0) sbuf[m] = s;
  for (int d = 32; d > 0; d >>= 1) r2 += __shfl_xor(r2, d);
  if (lane == 0) lpart[blockIdx.x * kRowWaves + wave] = r2;

#pragma unroll
  for (int ub = 0; ub < 4; ++ub)
    seed_block(s, L.w4, ub, half, D[kLayers - 1][ub], &f[2 * ub], &f[2 * ub + 1]);
  store_frags<8>(dz + 3 * stride, block, lane, f);
#pragma unroll
  for (int l = kLayers - 1; l >= 1; --l) {
    rows_gemm<kHid / 16, 4>(L.w, f, lane, acc);
    if (l > 1 || gx) {
      __syncthreads();
      if (l > 1)
        copy_to_lds<kHid * kHid>(w.Wt[l - 1], L.w, wave, lane);
      else
        copy_to_lds<kHid * kInPad>(w.Wt[0], L.w, wave, lane);
    }
#pragma unroll
    for (int ub = 0; ub < 4; ++ub) {
      grad_block(acc[ub], D[l - 1][ub], &f[2 * ub], &f[2 * ub + 1]);
    }
    if (l > 1 || gx) {
      lds_copies_done();
      __syncthreads();
    }
    store_frags<8>(dz + (l - 1) * stride, block, lane, f);
  }
  if (gx) {
    rows_gemm<kHid / 16, 1>(L.w, f, lane, acc);
    store_input_grad(acc[0], m, n, n_in, norm + kInPad, half, gx);
  }
}

// ------------------------------------------------------ weight gradients

// A slab is one 32-row block of a layer (128 columns 8 KB, 32 columns 2 KB)
// in LDS, as it lies in memory.
constexpr int kSlabRows = 32;
// Copies of 1 KB per wave for a slab of K columns; the 32-column slab's two
// are made twice, by waves 0, 1 and waves 2, 3 (the same bytes), so that
// every wave has the same number in flight.
template <int K>
constexpr int slab_copies() {
  return K == kHid ? kHid / 16 / kRowWaves : 1;
}
template <int K>
__device__ __forceinline__ void copy_slab(const uint16_t *src, uint16_t *dst,
                                          int wave, int lane) {
  typedef const __attribute__((address_space(1))) char *gptr;
  const uint32_t off = (uint32_t)lane * 16u;
#pragma unroll
  for (int q = 0; q < slab_copies<K>(); ++q) {
    const int frag = K == kHid ? q * kRowWaves + wave : wave & 1;
    __builtin_amdgcn_global_load_lds(
        (const __attribute__((address_space(1))) void *)(
            (gptr)src + frag * (kFrag * 2) + off),
        (__attribute__((address_space(3))) void *)(dst + frag * kFrag), 16, 0,
        0);
  }
}

// MFMA operand of columns 32 cb .. 32 cb + 31 and slab rows 16 kk .. + 15:
// lane l gets column l % 32, rows 8 (l / 32) .. + 7 of the sixteen.  Two
// transposed reads of four rows; each group of 16 lanes reads four rows x
// 16 columns (8 bytes a lane) and receives them by column.
typedef short s16x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ bf16x8 slab_operand(const uint16_t *slab, int kk,
                                               int cb, int lane) {
  const int i = lane & 15, h = lane >> 5, cg = (lane >> 4) & 1;
  const uint16_t *p = slab + block_at(16 * kk + 8 * h + (i >> 2),
                                      32 * cb + 16 * cg + 4 * (i & 3));
  typedef __attribute__((address_space(3))) s16x4 *lds4;
  s16x4 v[2];
  v[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4)p);
  v[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4)(p + 4 * 8));
  return __builtin_bit_cast(bf16x8, v);
}

// Register r of a 32x32 accumulator holds row 8 (r / 4) + 4 half + r % 4
// of the first operand.
__device__ __forceinline__ int acc_row(int r, int half) {
  return 8 * (r >> 2) + 4 * half + (r & 3);
}

// Partial products of one layer over `rows` rows (a multiple of 32) at Z
// and A, and the biases' sums.  kFirst: layer 0 (128 x 32, 32 output units
// per wave); else 128 x 128, one 64 x 64 quadrant per wave.  Slabs of 32
// rows pass through three LDS buffers, two copies in flight while one is
// multiplied.
constexpr int kSlabBufs = 3;
template <bool kFirst>
__device__ __forceinline__ void wgrad_layer(
    const uint16_t *__restrict__ Z, const uint16_t *__restrict__ A, int rows,
    uint16_t (&zs)[kSlabBufs][kSlabRows * kHid],
    uint16_t (&as)[kSlabBufs][kSlabRows * kHid], int wave, int lane,
    float *__restrict__ W, float *__restrict__ bias) {
  constexpr int K = kFirst ? kInPad : kHid;
  constexpr int NB = kFirst ? 1 : 2;
  constexpr int kCopies = slab_copies<kHid>() + slab_copies<K>();
  const int slabs = rows / kSlabRows;
  auto start = [&](int q) {
    copy_slab<kHid>(Z + q * (kSlabRows * kHid), zs[q % kSlabBufs], wave, lane);
    copy_slab<K>(A + q * (kSlabRows * K), as[q % kSlabBufs], wave, lane);
  };
  f32x16 acc[NB][NB], accb;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int c = 0; c < NB; ++c) acc[b][c][r] = 0.f;
    accb[r] = 0.f;
  }
  bf16x8 ones;
#pragma unroll
  for (int e = 0; e < 8; ++e) ones[e] = (__bf16)1.0f;
  const int oq = wave >> 1, iq = wave & 1;  // quadrant
  start(0);
  if (slabs > 1) start(1);
  for (int q = 0; q < slabs; ++q) {
    // Slab q is complete when at most slab q + 1's copies are outstanding.
    asm volatile("" ::: "memory");
    if (q + 1 < slabs)
      __builtin_amdgcn_s_waitcnt(0x0F70 | kCopies);  // vmcnt(kCopies)
    else
      __builtin_amdgcn_s_waitcnt(0x0F70);
    asm volatile("" ::: "memory");
    __syncthreads();
    if (q + 2 < slabs) start(q + 2);  // into the buffer read at q - 1
    const uint16_t *zq = zs[q % kSlabBufs], *aq = as[q % kSlabBufs];
#pragma unroll
    for (int kk = 0; kk < kSlabRows / 16; ++kk) {
      if constexpr (kFirst) {
        const bf16x8 z = slab_operand(zq, kk, wave, lane);
        acc[0][0] = mfma(z, slab_operand(aq, kk, 0, lane), acc[0][0]);
        accb = mfma(z, ones, accb);
      } else {
        bf16x8 z[2], a[2];
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          z[b] = slab_operand(zq, kk, 2 * oq + b, lane);
          a[b] = slab_operand(aq, kk, 2 * iq + b, lane);
        }
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
          for (int c = 0; c < 2; ++c)
            acc[b][c] = mfma(z[b], a[c], acc[b][c]);
        // the two waves of a row of quadrants sum one unit block each
        accb = mfma(iq ? z[1] : z[0], ones, accb);
      }
    }
  }
  const int col = lane & 31, half = lane >> 5;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int row = acc_row(r, half);
    if constexpr (kFirst) {
      W[(32 * wave + row) * K + col] = acc[0][0][r];
      if (col == 0) bias[32 * wave + row] = accb[r];
    } else {
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int c = 0; c < 2; ++c)
          W[(64 * oq + 32 * b + row) * K + 64 * iq + 32 * c + col] =
              acc[b][c][r];
      if (col == 0) bias[64 * oq + 32 * iq + row] = accb[r];
    }
  }
}

// Partial gradients of rows [R blockIdx.x, + R) of the padded batch (R a
// multiple of 32; the last chunk may be shorter).  blockIdx.y: 0..2 the
// layers 1..3, 3 layer 0, 4 the output layer.  Bound by memory: each row's
// 512 bytes per layer are read once for 16 K multiply-adds (16 rows cost a
// wave 128 matrix cycles and, at the CU's share of the memory rate, about
// a thousand).  65,536 rows: 156 MB in 26 us, 6 TB/s (partly from the
// Infinity Cache); staging 16-row slices element by element, in 64
// workgroups per layer, took 640 us.
__global__ __launch_bounds__(256, 2) void k_mlp_wgrad(
    const uint16_t *__restrict__ a0, const uint16_t *__restrict__ act,
    const uint16_t *__restrict__ dz, int64_t stride,
    const float *__restrict__ sbuf, int npad, int R,
    float *__restrict__ part) {
  __shared__ alignas(16) uint16_t zs[kSlabBufs][kSlabRows * kHid];
  __shared__ alignas(16) uint16_t as[kSlabBufs][kSlabRows * kHid];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t r0 = (int64_t)blockIdx.x * R;
  const int rows = (int)min((int64_t)R, npad - r0);
  float *out = part + (int64_t)blockIdx.x * kPartLen;
  const int job = blockIdx.y;
  if (job < 3) {
    wgrad_layer<false>(dz + (job + 1) * stride + r0 * kHid,
                       act + job * stride + r0 * kHid, rows, zs, as, wave,
                       lane, out + job * kHid * kHid,
                       out + kPartB + (job + 1) * kHid);
  } else if (job == 3) {
    wgrad_layer<true>(dz + r0 * kHid, a0 + r0 * kInPad, rows, zs, as, wave,
                      lane, out + kPartW0, out + kPartB);
  } else {
    // W4: sum of s[m] A4[m][c]; thread t takes the eight columns of chunk
    // t % 16 and every 16th row.
    const uint16_t *A4 = act + 3 * stride + r0 * kHid;
    const int c = threadIdx.x & 15, rg = threadIdx.x >> 4;
    float acc[8] = {}, sb = 0.f;
#pragma unroll 4
    for (int q = rg; q < rows; q += 16) {
      const float s = sbuf[r0 + q];
      const uint4 v = *reinterpret_cast<const uint4 *>(
          A4 + (q >> 5) * (kSlabRows * kHid) + block_at(q & 31, 8 * c));
      const uint32_t u[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        acc[2 * e] += s * from_bf16(lo16(u[e]));
        acc[2 * e + 1] += s * from_bf16(hi16(u[e]));
      }
      sb += s;
    }
    constexpr int kRow = kHid + 4;
    float *red = reinterpret_cast<float *>(&zs[0][0]);  // [16][kRow]
#pragma unroll
    for (int e = 0; e < 8; ++e) red[rg * kRow + 8 * c + e] = acc[e];
    if (c == 0) red[rg * kRow + kHid] = sb;
    __syncthreads();
    if (threadIdx.x <= kHid) {
      float s = 0.f;
      for (int q = 0; q < 16; ++q) s += red[q * kRow + threadIdx.x];
      out[kPartW4 + threadIdx.x] = s;
    }
  }
}

// Sums the chunks' partials into the flat gradient vector (fixed order:
// four interleaved sums per value, then their sum), one block per 64
// positions of the partial's layout; the last block sums the loss.  7.5 us
// for 128 partials (28 MB); a sum per layer and bias in launches of their
// own took 130 us.
__global__ __launch_bounds__(256) void k_grad_sum(
    const float *__restrict__ part, int chunks, int n_in,
    float *__restrict__ g, const float *__restrict__ lpart, int nlpart,
    float inv_n, float *__restrict__ loss) {
  __shared__ float red[256];
  const int t = threadIdx.x & 63, q = threadIdx.x >> 6;
  float s = 0.f;
  if (blockIdx.x == gridDim.x - 1) {
    if (!loss) return;  // uniform over the block
    for (int i = threadIdx.x; i < nlpart; i += 256) s += lpart[i];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int d = 128; d > 0; d >>= 1) {
      if ((int)threadIdx.x < d) red[threadIdx.x] += red[threadIdx.x + d];
      __syncthreads();
    }
    if (threadIdx.x == 0) loss[0] = red[0] * inv_n;
    return;
  }
  const int at = blockIdx.x * 64 + t;
  if (at < kPartLen) {
#pragma unroll 8
    for (int c = q; c < chunks; c += 4) s += part[(int64_t)c * kPartLen + at];
  }
  red[threadIdx.x] = s;
  __syncthreads();
  if (q != 0 || at >= kPartLen) return;
  s = (red[t] + red[64 + t]) + (red[128 + t] + red[192 + t]);
  if (at < kPartW0) {
    const int l = at / (kHid * kHid);
    g[layer_desc(l + 1, n_in).w_off + at - l * kHid * kHid] = s;
  } else if (at < kPartB) {
    const int o = (at - kPartW0) / kInPad, i = (at - kPartW0) % kInPad;
    if (i < n_in) g[o * n_in + i] = s;
  } else if (at < kPartW4) {
    const int l = (at - kPartB) / kHid;
    g[layer_desc(l, n_in).b_off + (at - kPartB) % kHid] = s;
  } else if (at - kPartW4 <= kHid) {
    g[layer_desc(kLayers, n_in).w_off + at - kPartW4] = s;
  }
}

}  // namespace pcsdf
