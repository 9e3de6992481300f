// The network on 32 rows per wave with the activations in registers: the
// core of the fused inference and training kernels.
//
// Every product takes the weights as the first MFMA operand and the rows
// as the second, so the accumulators of lane l are units of row l % 32:
// register r of unit block ub holds unit 32 ub + 8 (r / 4) + 4 (l / 32) +
// r % 4.  The next product wants eight consecutive units of the same row
// in each lane, which the lane and its partner in the other half hold
// between them: after the epilogue two values share a word, and one
// v_permlane32_swap per word pair puts them in place (pack_block).  So an
// activation never leaves the registers between layers, and the four waves
// of a workgroup share nothing but the layer's weights, 32 KB in LDS in
// fragment order, copied there by direct loads to LDS that run under the
// previous layer's epilogue.
#pragma once

#include "mlp_kernels.h"

namespace pcsdf {

constexpr int kRowWaves = 4;                 // waves per workgroup
constexpr int kRowTile = 32 * kRowWaves;     // rows per workgroup

struct NetWeights {
  const uint16_t *W[kLayers + 1];  // W_l in fragment order (W4: [128])
  const uint16_t *Wt[kLayers];     // W_l^T in fragment order
};

// Starts the copy of kElems BF16 values (a multiple of 2048; 16 bytes a
// lane and step) from global memory into LDS by the whole workgroup; both
// are 16-byte aligned.  The copies are complete after every wave's
// lds_copies_done() and a barrier.  The lane's part of the address is one
// 32-bit offset, the rest uniform.
template <int kElems>
__device__ __forceinline__ void copy_to_lds(const uint16_t *src, uint16_t *dst,
                                            int wave, int lane) {
  typedef const __attribute__((address_space(1))) char *gptr;
  // opaque, so that the copies' addresses are formed where they are used
  // instead of all being kept in registers
  uint32_t off = (uint32_t)lane * 16u;
  asm volatile("" : "+v"(off));
  const gptr from = (gptr)src + wave * (kFrag * 2);
#pragma unroll
  for (int q = 0; q < kElems / (kRowWaves * kFrag); ++q)
    __builtin_amdgcn_global_load_lds(
        (const __attribute__((address_space(1))) void *)(
            from + q * (kRowWaves * kFrag * 2) + off),
        (__attribute__((address_space(3))) void *)(
            dst + (q * kRowWaves + wave) * kFrag),
        16, 0, 0);
}
// Waits for this wave's outstanding vector memory operations, the copies
// to LDS among them (vmcnt = 0, the other counters at their maximum).
__device__ __forceinline__ void lds_copies_done() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0x0F70);
  asm volatile("" ::: "memory");
}

// Keeps the compiler from moving instructions across: the products' operand
// reads and the epilogues' blocks, all independent, would otherwise be
// started together and spill.
__device__ __forceinline__ void sched_fence() {
  __builtin_amdgcn_sched_barrier(0);
}

// acc[nb] = weights (NB blocks of 32 units, KS contraction slices, in LDS)
// times this wave's rows; a slice's operands are read one slice ahead.
template <int KS, int NB>
__device__ __forceinline__ void rows_gemm(const uint16_t *w,
                                          const bf16x8 (&f)[8], int lane,
                                          f32x16 (&acc)[4]) {
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[nb][r] = 0.f;
  bf16x8 b[2][NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) b[0][nb] = load8(w + nb * kFrag + lane * 8);
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    if (ks + 1 < KS) {
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
        b[(ks + 1) & 1][nb] =
            load8(w + ((ks + 1) * NB + nb) * kFrag + lane * 8);
    }
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
      acc[nb] = mfma(b[ks & 1][nb], f[ks], acc[nb]);
    sched_fence();
  }
}

// Exchanges the upper half-wave of *a with the lower half-wave of *b.
__device__ __forceinline__ void swap_halves(uint32_t *a, uint32_t *b) {
  const auto r = __builtin_amdgcn_permlane32_swap(*a, *b, false, false);
  *a = r[0];
  *b = r[1];
}

// The two operand fragments of a unit block from its 16 values in
// accumulator order, two per word: v[0..1] are units 4h .. 4h+3 (h: the
// lane's half), v[2..3] units 8+4h .. 8+4h+3, v[4..7] the same of the next
// 16 units.
__device__ __forceinline__ void pack_block(uint32_t (&v)[8], bf16x8 *lo,
                                           bf16x8 *hi) {
#pragma unroll
  for (int q = 0; q < 8; q += 4) {
    swap_halves(&v[q], &v[q + 2]);
    swap_halves(&v[q + 1], &v[q + 3]);
    const uint4 u = make_uint4(v[q], v[q + 1], v[q + 2], v[q + 3]);
    *(q ? hi : lo) = __builtin_bit_cast(bf16x8, u);
  }
  sched_fence();
}

// A0 fragments of row m (zero beyond n_in columns and n rows): lane half
// h holds columns 16 ks + 8 h .. + 7.
__device__ __forceinline__ void input_frags(const float *__restrict__ x,
                                            int64_t m, int n, int n_in,
                                            const float *__restrict__ norm,
                                            int half, bf16x8 (&f)[8]) {
  const bool vec = !(n_in & 7) && !((uintptr_t)x & 15);
#pragma unroll
  for (int ks = 0; ks < kInPad / 16; ++ks) {
    const int c0 = 16 * ks + 8 * half;
    uint32_t u[4] = {0, 0, 0, 0};
    if (m < n && c0 < n_in) {
      float v[8];
      const float *row = x + m * n_in + c0;
      if (vec) {
        const float4 a = *reinterpret_cast<const float4 *>(row);
        const float4 b = *reinterpret_cast<const float4 *>(row + 4);
        v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
        v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = c0 + e < n_in ? row[e] : 0.f;
      }
#pragma unroll
      for (int e = 0; e < 8; ++e)
        v[e] = c0 + e < n_in ? (v[e] - norm[c0 + e]) * norm[kInPad + c0 + e]
                             : 0.f;
#pragma unroll
      for (int e = 0; e < 4; ++e) u[e] = cvt2(v[2 * e], v[2 * e + 1]);
    }
    f[ks] = __builtin_bit_cast(bf16x8, make_uint4(u[0], u[1], u[2], u[3]));
  }
}

// sum over units of A4 W4 for this lane's row, in the order: units 0..63
// by the lower half, 64..127 by the upper, then their sum (both halves get
// it).  w4: [128] floats in LDS.
__device__ __forceinline__ float output_sum(const bf16x8 (&f)[8],
                                            const float *w4, int half) {
  float s = 0.f;
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) {
    const uint4 a = __builtin_bit_cast(uint4, f[ks]);
    const uint4 b = __builtin_bit_cast(uint4, f[ks + 4]);
    uint32_t p[4] = {a.x, a.y, a.z, a.w}, q[4] = {b.x, b.y, b.z, b.w};
    // p: units 16 ks + 64 half + 0..7, q: the next eight
#pragma unroll
    for (int j = 0; j < 4; ++j) swap_halves(&p[j], &q[j]);
    const float *w = w4 + 64 * half + 16 * ks;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      s += from_bf16(lo16(p[j])) * w[2 * j];
      s += from_bf16(hi16(p[j])) * w[2 * j + 1];
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      s += from_bf16(lo16(q[j])) * w[8 + 2 * j];
      s += from_bf16(hi16(q[j])) * w[8 + 2 * j + 1];
    }
  }
  return s + __shfl_xor(s, 32);
}

// SiLU and its derivative from one logistic value.  Inference: with the
// hardware's approximate exponential and reciprocal (a few ulp of fp32;
// the results are rounded to BF16 next, whose unit is 2^16 fp32 ulps).
struct SiluFast {
  __device__ __forceinline__ static void eval(float z, float *a, float *d) {
    const float e = __expf(-z);
    const float sg = __builtin_amdgcn_rcpf(1.f + e);
    *a = z * sg;
    *d = sg * (1.f + z * (1.f - sg));
  }
};
// Training: the same to about one fp32 ulp.  exp(-z) = 2^t (1 + ln2 rem)
// with t + rem = -z log2(e), t the rounded product and rem what it and the
// constant leave out; the reciprocal gets one Newton step.  So that no
// intermediate leaves fp32's range z is taken at 87 beyond it, where the
// logistic is 1, and at -88.5 beyond that, where its reciprocal, 3.7e-39, is
// subnormal: the hardware's is zero there (from -87.3 on), and SiLU and its
// derivative then are, of any finite z.
struct SiluTrain {
  __device__ __forceinline__ static void eval(float z, float *a, float *d) {
    constexpr float kL = 1.44269504088896341f;          // log2 e, fp32
    constexpr float kLlo = 1.92596299112661746887e-8f;  // log2 e - kL
    constexpr float kLn2 = 0.693147180559945309f;
    const float zc = __builtin_amdgcn_fmed3f(z, -88.5f, 87.f);
    const float t = -zc * kL;
    const float e0 = __builtin_amdgcn_exp2f(t);
    const float rem = __builtin_fmaf(-zc, kLlo, __builtin_fmaf(-zc, kL, -t));
    const float den = 1.f + __builtin_fmaf(e0, rem * kLn2, e0);
    const float r0 = __builtin_amdgcn_rcpf(den);
    const float sg = __builtin_fmaf(__builtin_fmaf(-den, r0, 1.f), r0, r0);
    *a = z * sg;
    *d = sg * __builtin_fmaf(z, 1.f - sg, 1.f);
  }
};

// Epilogue of a hidden layer's unit block ub: A = bf16(SiLU(z + b)) as the
// next layer's fragments, D = bf16(SiLU'(z + b)) in accumulator order.
// bias: the layer's [128] floats in LDS.
template <class Act>
__device__ __forceinline__ void act_block(const f32x16 &acc, const float *bias,
                                          int ub, int half, bf16x8 *lo,
                                          bf16x8 *hi, uint32_t (&D)[8]) {
  uint32_t v[8];
#pragma unroll
  for (int r = 0; r < 16; r += 4) {
    const float4 b = *reinterpret_cast<const float4 *>(
        bias + 32 * ub + 2 * r + 4 * half);
    const float bb[4] = {b.x, b.y, b.z, b.w};
    float a[4], d[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) Act::eval(acc[r + e] + bb[e], &a[e], &d[e]);
    v[r / 2] = cvt2(a[0], a[1]);
    v[r / 2 + 1] = cvt2(a[2], a[3]);
    D[r / 2] = cvt2(d[0], d[1]);
    D[r / 2 + 1] = cvt2(d[2], d[3]);
    // opaque: the packed words are what waits for the backward pass, not
    // the fp32 values they are computed from
    asm volatile("" : "+v"(D[r / 2]), "+v"(D[r / 2 + 1]));
    sched_fence();
  }
  pack_block(v, lo, hi);
}

// bf16(acc (.) D) of a unit block as fragments.
__device__ __forceinline__ void grad_block(const f32x16 &acc,
                                           const uint32_t (&D)[8], bf16x8 *lo,
                                           bf16x8 *hi) {
  uint32_t v[8];
#pragma unroll
  for (int q = 0; q < 8; ++q)
    v[q] = cvt2(acc[2 * q] * from_bf16(lo16(D[q])),
                acc[2 * q + 1] * from_bf16(hi16(D[q])));
  pack_block(v, lo, hi);
}

// dZ3 = bf16(s W4 (.) D3) of a unit block as fragments; s = dLoss/dy times
// the output scale of this lane's row.
__device__ __forceinline__ void seed_block(float s, const float *w4, int ub,
                                           int half, const uint32_t (&D)[8],
                                           bf16x8 *lo, bf16x8 *hi) {
  uint32_t v[8];
#pragma unroll
  for (int r = 0; r < 16; r += 4) {
    const float4 w = *reinterpret_cast<const float4 *>(
        w4 + 32 * ub + 2 * r + 4 * half);
    v[r / 2] = cvt2(s * w.x * from_bf16(lo16(D[r / 2])),
                    s * w.y * from_bf16(hi16(D[r / 2])));
    v[r / 2 + 1] = cvt2(s * w.z * from_bf16(lo16(D[r / 2 + 1])),
                        s * w.w * from_bf16(hi16(D[r / 2 + 1])));
  }
  pack_block(v, lo, hi);
}

// Input gradient of row m from the last product (columns in accumulator
// order), scaled back to the caller's units.
__device__ __forceinline__ void store_input_grad(const f32x16 &g, int64_t m,
                                                 int n, int n_in,
                                                 const float *__restrict__ scale,
                                                 int half,
                                                 float *__restrict__ gx) {
  if (m >= n) return;
  const bool vec = !(n_in & 3) && !((uintptr_t)gx & 15);
#pragma unroll
  for (int r = 0; r < 16; r += 4) {
    const int c = 2 * r + 4 * half;
    if (c >= n_in) continue;
    float *dst = gx + m * n_in + c;
    if (vec) {
      *reinterpret_cast<float4 *>(dst) =
          make_float4(g[r] * scale[c], g[r + 1] * scale[c + 1],
                      g[r + 2] * scale[c + 2], g[r + 3] * scale[c + 3]);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (c + e < n_in) dst[e] = g[r + e] * scale[c + e];
    }
  }
}

// LDS of one workgroup: the current layer's weights, biases and the output
// weights.
struct RowsLds {
  alignas(16) uint16_t w[kHid * kHid];
  alignas(16) float bias[kLayers][kHid];
  alignas(16) float w4[kHid];
};

__device__ __forceinline__ void load_small(RowsLds &L, const NetWeights &w,
                                           const float *__restrict__ p,
                                           int n_in) {
  for (int t = threadIdx.x; t < kHid; t += 64 * kRowWaves) {
#pragma unroll
    for (int l = 0; l < kLayers; ++l)
      L.bias[l][t] = p[layer_desc(l, n_in).b_off + t];
    L.w4[t] = from_bf16(w.W[kLayers][t]);
  }
}

}  // namespace pcsdf
