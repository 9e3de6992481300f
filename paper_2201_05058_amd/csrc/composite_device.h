// The composite epilogue shared by the single-scene kernel (composite.hip)
// and the batched workers (batch_device.h): for four consecutive voxels
// of the flattened [nz][ny][nx] grid, read the static field once and write
// min(static, humans' value) for a range of slices.
//
// The static field and the outputs are flat streams, written in packs of
// four voxels per lane, 1 KB per wave and stream.  Where every slice starts
// on a cache line (32 divides nx ny nz and the outputs are so aligned) and
// four divides nx ny, packs are aligned in every stream and lie in one layer
// (composite_pack).  Everywhere else each slice's packs are cut where that
// slice's output meets a cache line, and the static and planar values, which
// come from the caches, are read as unaligned vectors
// (composite_pack_shifted).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "device_common.h"

namespace pcsdf {

// Packs of VEC int32 or fp32 values, and their loads as global memory
// instructions.  Pointers read from memory (the batch's scene
// table) would otherwise be accessed with flat instructions, which the
// compiler cannot count in order: every wait for one of them then waits
// for all outstanding loads and stores.  The casts are written per
// concrete type because a global address space on a template-dependent
// type is not kept.
#if defined(__clang__)
#define PCSDF_GLOBAL_AS __attribute__((address_space(1)))
typedef int32_t pk_i32x4 __attribute__((ext_vector_type(4)));
typedef int32_t pk_i32x2 __attribute__((ext_vector_type(2)));
typedef int32_t pk_i32x1 __attribute__((ext_vector_type(1)));
typedef float pk_f32x4 __attribute__((ext_vector_type(4)));
// the same four values, and four 16-bit ones, at the alignment of one
typedef int32_t pk_i32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef float pk_f32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef int16_t pk_i16x4u __attribute__((ext_vector_type(4), aligned(2)));
#else  // a host compiler building the device code for CPU tests
#define PCSDF_GLOBAL_AS
template <class T, int N>
struct HostPack {
  T v[N];
  T &operator[](int i) { return v[i]; }
  const T &operator[](int i) const { return v[i]; }
};
typedef HostPack<int32_t, 4> pk_i32x4;
typedef HostPack<int32_t, 2> pk_i32x2;
typedef HostPack<int32_t, 1> pk_i32x1;
typedef HostPack<float, 4> pk_f32x4;
typedef pk_i32x4 pk_i32x4u;
typedef pk_f32x4 pk_f32x4u;
typedef HostPack<int16_t, 4> pk_i16x4u;
#endif

#define PCSDF_GLOBAL_IO(T)                                           \
  __device__ __forceinline__ T ld_global(const T *p) {              \
    return *(PCSDF_GLOBAL_AS const T *)p;                            \
  }
PCSDF_GLOBAL_IO(pk_i32x4)
PCSDF_GLOBAL_IO(pk_i32x2)
PCSDF_GLOBAL_IO(pk_i32x1)
#undef PCSDF_GLOBAL_IO

__device__ __forceinline__ pk_i32x4 load_i32x4(const int32_t *p) {
  return ld_global(reinterpret_cast<const pk_i32x4 *>(p));
}
__device__ __forceinline__ int32_t load_i32(const int32_t *p) {
  return ld_global(reinterpret_cast<const pk_i32x1 *>(p))[0];
}
// Four values from an address that is a multiple of one (the hardware
// reads such vectors in one instruction).
__device__ __forceinline__ pk_i32x4 load_i32x4u(const int32_t *p) {
  const pk_i32x4u v = *(PCSDF_GLOBAL_AS const pk_i32x4u *)p;
  pk_i32x4 r;
#pragma unroll
  for (int e = 0; e < 4; ++e) r[e] = v[e];
  return r;
}
// The outputs are written once and not read back by the kernel: stores
// with the nontemporal hint (no write-allocation in the caches; measured
// as fast at 256 x 256 x 128 and up to a quarter faster on smaller grids).
__device__ __forceinline__ void store_i32x4(int32_t *p, pk_i32x4 v) {
  __builtin_nontemporal_store(v, reinterpret_cast<pk_i32x4 *>(p));
}
__device__ __forceinline__ void store_f32x4(float *p, pk_f32x4 v) {
  __builtin_nontemporal_store(v, reinterpret_cast<pk_f32x4 *>(p));
}
__device__ __forceinline__ void store_f32x4u(float *p, pk_f32x4 v) {
  pk_f32x4u r;
#pragma unroll
  for (int e = 0; e < 4; ++e) r[e] = v[e];
  __builtin_nontemporal_store(
      r, (PCSDF_GLOBAL_AS pk_f32x4u *)p);
}

// Voxels of an output in one 128-byte line.
constexpr uint32_t kLineVoxels = 32;

// Whether every pack of four is aligned in all streams and lies in one
// layer, and every slice of the outputs starts on a line.
__host__ __device__ inline bool packs_aligned(int64_t plane, int64_t V,
                                              const void *S, const void *oc,
                                              const void *of) {
  return plane % 4 == 0 && V % kLineVoxels == 0 && !((uintptr_t)S & 15) &&
         !(((uintptr_t)oc | (uintptr_t)of) & 127);
}

// Voxels spanned by a slice's packs: V, or a line less one more where the
// packs start before voxel 0 (composite_pack_shifted).
__host__ __device__ inline uint32_t pack_span(uint32_t V, bool aligned) {
  return aligned ? V : V + kLineVoxels - 1;
}

// Order of the (slice group, voxel chunk) blocks of one scene.  The blocks
// run span by span, a span being `span` consecutive slice groups; within a
// span, eight chunks (one per XCD: the dispatcher places block b on XCD b
// mod 8) run their groups in succession before the next eight.  So a
// chunk's static values are re-read from the L2 of the XCD that has them,
// and the blocks in flight write only the span's slices.  The number of
// chunks is rounded up to eight (the surplus does nothing).
//
// Slices per span for single-slice groups, measured as written bytes on a
// streaming kernel of this shape (two outputs, nontemporal stores; write-only
// 6.4-6.6 TB/s at every size):
//  - up to 6.3 M voxels an XCD's eighth of the static field stays in its 4
//    MB L2 from one slice to the next, so one slice at a time: 2.5 M voxels
//    6.5 TB/s (all slices in one span 6.0), 6.3 M 6.4 (6.1);
//  - larger fields do not: 8.4 M voxels run one slice at a time at 4.9
//    TB/s, in spans of 10 at 6.3; 16.8 M 4.9 and 6.3;
//  - from 15 2^21 voxels the outputs of a long span compete (a slice is 120
//    MB or more apart): 33 M voxels x 40 slices spans of 4 6.4 TB/s, of 10
//    6.1, of 40 5.3; 31.5 M x 20 784 us and 820, 512 x 512 x 127 x 40 1945
//    and 2208;
//  - from kLargeVoxels on, where the static field alone fills the Infinity
//    Cache, 67 M x 50 with the 16-bit copy spans of 2 6.25, of 10 5.6, of 50
//    5.1; up to four slices are still one span (67 M x 3 278 us, 338 in two).
// A span is at most n and spans of one grid are about equally long.
constexpr int64_t kLargeVoxels = 15LL << 22;  // 240 MiB of the 256
constexpr int64_t kSpanVoxels = 1LL << 26;    // single slices up to here
__host__ __device__ inline int slices_per_span(int64_t V, int n) {
  const int most = V <= (3LL << 21)   ? 1
                   : V < (15LL << 21) ? 10
                   : V < kLargeVoxels ? 4
                   : n <= 4           ? n
                                      : 2;
  const int spans = (n + most - 1) / most;
  return (n + spans - 1) / spans;
}

// Element `byte_off` bytes past a base pointer.  With a base that is the
// same for the whole wave and a 32-bit offset, the access is a global
// instruction with the base in scalar registers and only the offset in a
// vector register, so no 64-bit address arithmetic runs per lane.
template <class T>
__device__ __forceinline__ T *at_bytes(T *base, uint32_t byte_off) {
  return reinterpret_cast<T *>(
      reinterpret_cast<typename std::conditional<
          std::is_const<T>::value, const char, char>::type *>(base) +
      byte_off);
}

// Slices whose planar packs one lane loads before it stores any of them.
constexpr int kPackSlices = 8;

// The 16-bit copy of the static field (k_static16): values in
// [-32767, 32767] as they are, every other value as kS16Far, which sends
// the reader to the int32 field.
constexpr int32_t kS16Far = -32768;

// The static values of an aligned pack from the 16-bit copy, sign-extended
// (kS16Far where the int32 field must be read).
__device__ __forceinline__ pk_i32x4 load_s16x4(const int16_t *p) {
  const pk_i32x2 w = ld_global(reinterpret_cast<const pk_i32x2 *>(p));
  pk_i32x4 s;
  s[0] = (int32_t)(int16_t)(w[0] & 0xFFFF);
  s[1] = w[0] >> 16;
  s[2] = (int32_t)(int16_t)(w[1] & 0xFFFF);
  s[3] = w[1] >> 16;
  return s;
}
__device__ __forceinline__ pk_i32x4 load_s16x4u(const int16_t *p) {
  const pk_i16x4u w = *(PCSDF_GLOBAL_AS const pk_i16x4u *)p;
  pk_i32x4 s;
#pragma unroll
  for (int e = 0; e < 4; ++e) s[e] = w[e];
  return s;
}

__device__ __forceinline__ HumanLayer human_layer_opaque(int k, int Kt,
                                                         int has_above) {
  HumanLayer hl = human_layer(k, Kt, has_above);
#if defined(__clang__)
  // Opaque to the optimiser, which would otherwise apply the addition
  // under a select of its own in the loop (one more instruction per voxel
  // and slice).
  asm("" : "+v"(hl.lo), "+v"(hl.add));
#endif
  return hl;
}

// Voxels v0 .. v0+3 (v0 a multiple of four, all in [0, V)) of an aligned
// grid (packs_aligned) for slices [s_begin, s_end); with kNeed, slices with
// need[sl] == 0 are skipped (a template parameter so that without it the
// stores are unconditional).
//
// One counter tracks a wave's outstanding vector loads and stores in issue
// order, so a load issued after a store can only be waited for together
// with that store.  The lane therefore issues the static load and the
// planar loads of up to kPackSlices slices first, and only then computes
// and stores them, so that no load waits behind the lane's own stores.
// (Longer slice groups still measure slower than groups of two or three:
// the blocks in flight then write more slices' outputs at once.)
//
// With S16 (the 16-bit copy of the static field, k_static16) the static
// values come from it and only the far ones from S: every slice group
// reads the static values again, and the copy is half their bytes.
template <bool kSsq, bool kSdf, bool kNeed = false>
__device__ __forceinline__ void composite_pack(
    const int32_t *__restrict__ S, const int32_t *__restrict__ P,
    const int32_t *__restrict__ need, int32_t *__restrict__ oc,
    float *__restrict__ of, const FastDiv &pd, uint32_t V, uint32_t v0,
    int s_begin, int s_end, int Kt, int has_above, float hf,
    const int16_t *__restrict__ S16 = nullptr) {
  const uint32_t plane = pd.d;
  const uint32_t k = quotient(v0, pd);
  const uint32_t pix = v0 - k * plane;
  const HumanLayer hl = human_layer_opaque((int)k, Kt, has_above);
  // V <= 2^30, so byte offsets within one slice fit in 32 bits.
  const uint32_t vb = v0 * 4u;
  pk_i32x4 s = S16 ? load_s16x4(at_bytes(S16, v0 * 2u))
                   : load_i32x4(at_bytes(S, vb));
  for (int sl0 = s_begin; sl0 < s_end; sl0 += kPackSlices) {
    const int cnt = min(kPackSlices, s_end - sl0);
    pk_i32x4 p[kPackSlices];
#pragma unroll
    for (int j = 0; j < kPackSlices; ++j)
      if (j < cnt && !(kNeed && need[sl0 + j] == 0))
        p[j] = load_i32x4(at_bytes(P + (size_t)(sl0 + j) * plane, pix * 4u));
    if (S16 && sl0 == s_begin) {
      // the far values from the int32 field (after the planar loads are
      // issued, so that only the static load is waited for)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (s[e] == kS16Far) s[e] = load_i32(at_bytes(S, vb + 4u * e));
    }
#pragma unroll
    for (int j = 0; j < kPackSlices; ++j) {
      if (j >= cnt) break;
      const int sl = sl0 + j;
      if (kNeed && need[sl] == 0) continue;
      pk_i32x4 c;
#pragma unroll
      for (int e = 0; e < 4; ++e) c[e] = min(s[e], human_value(p[j][e], hl));
      if (kSsq) store_i32x4(at_bytes(oc + (size_t)sl * V, vb), c);
      if (kSdf) {
        pk_f32x4 f;
#pragma unroll
        for (int e = 0; e < 4; ++e) f[e] = ssq_to_metres(c[e], hf);
        store_f32x4(at_bytes(of + (size_t)sl * V, vb), f);
      }
    }
  }
}

// The same for any grid and any 4-byte aligned buffers.  With v4 a multiple
// of four in [0, V + 31), the lane writes of each slice the voxels v4 - a ..
// v4 - a + 3 that lie in [0, V), where a in [0, 31] is the slice's own shift
// that puts voxel v4 - a on the same place of a 128-byte line as v4 is of a
// line of 32 voxels: the packs of a wave are whole lines of the output (the
// int32 one, else the fp32 one; the other is stored unaligned where the
// bases differ).  The static and planar values are unaligned vector reads
// from the caches.  A pack that leaves the slice or crosses a layer boundary
// is done voxel by voxel.
//
// Lines split between waves are what this avoids: 255 x 241 x 127 x 20
// slices, both fields, 205 us (6.2 TB/s), with packs cut at 16 bytes 262,
// with the fp32 stream alone off the lines 249, and gathering single voxels
// into aligned packs of the flattened outputs 324.
constexpr int kShiftSlices = 2;
template <bool kSsq, bool kSdf, bool kNeed = false>
__device__ __forceinline__ void composite_pack_shifted(
    const int32_t *__restrict__ S, const int32_t *__restrict__ P,
    const int32_t *__restrict__ need, int32_t *__restrict__ oc,
    float *__restrict__ of, const FastDiv &pd, uint32_t V, uint32_t v4,
    int s_begin, int s_end, int Kt, int has_above, float hf,
    const int16_t *__restrict__ S16 = nullptr) {
  const uint32_t base =
      (uint32_t)((kSsq ? (uintptr_t)oc : (uintptr_t)of) >> 2);
  const uint32_t plane = pd.d;
  const uint32_t k4 = quotient(v4, pd);
  const uint32_t pix4 = v4 - k4 * plane;
  for (int sl0 = s_begin; sl0 < s_end; sl0 += kShiftSlices) {
    pk_i32x4 s[kShiftSlices], p[kShiftSlices];
    uint32_t shift[kShiftSlices];
    bool whole[kShiftSlices], down[kShiftSlices];
#pragma unroll
    for (int j = 0; j < kShiftSlices; ++j) {
      const int sl = sl0 + j;
      const uint32_t a = (base + (uint32_t)sl * V) & (kLineVoxels - 1);
      shift[j] = a;
      // the shift leads into v4's layer or, from its first pixels, into the
      // one below (planes of fewer pixels than a line: voxel by voxel)
      down[j] = pix4 < a;
      const uint32_t pix = pix4 - a + (down[j] ? plane : 0u);
      whole[j] = sl < s_end && v4 >= a && v4 - a + 3 < V &&
                 pix + 3 < plane && plane >= kLineVoxels;
      if (kNeed && whole[j]) whole[j] = need[sl] != 0;
      if (whole[j]) {
        p[j] = load_i32x4u(at_bytes(P + (size_t)sl * plane, pix * 4u));
        s[j] = S16 ? load_s16x4u(at_bytes(S16, (v4 - a) * 2u))
                   : load_i32x4u(at_bytes(S, (v4 - a) * 4u));
      }
    }
#pragma unroll
    for (int j = 0; j < kShiftSlices; ++j) {
      const int sl = sl0 + j;
      if (sl >= s_end) break;
      if (kNeed && need[sl] == 0) continue;
      int32_t *ocs = oc + (size_t)sl * V;
      float *ofs = of + (size_t)sl * V;
      if (whole[j]) {
        const uint32_t vb = (v4 - shift[j]) * 4u;
        if (S16) {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (s[j][e] == kS16Far)
              s[j][e] = load_i32(at_bytes(S, vb + 4u * e));
        }
        const HumanLayer hl = human_layer_opaque(
            (int)k4 - (down[j] ? 1 : 0), Kt, has_above);
        pk_i32x4 c;
#pragma unroll
        for (int e = 0; e < 4; ++e)
          c[e] = min(s[j][e], human_value(p[j][e], hl));
        if (kSsq) store_i32x4(at_bytes(ocs, vb), c);
        if (kSdf) {
          pk_f32x4 f;
#pragma unroll
          for (int e = 0; e < 4; ++e) f[e] = ssq_to_metres(c[e], hf);
          if (kSsq)
            store_f32x4u(at_bytes(ofs, vb), f);
          else
            store_f32x4(at_bytes(ofs, vb), f);
        }
      } else {
        for (uint32_t e = 0; e < 4; ++e) {
          const uint32_t v = v4 - shift[j] + e;  // wraps below zero
          if (v >= V) continue;
          const uint32_t k = quotient(v, pd);
          const int32_t c =
              min(S[v], human_value(P[(size_t)sl * plane + (v - k * plane)],
                                    human_layer((int)k, Kt, has_above)));
          if (kSsq) ocs[v] = c;
          if (kSdf) ofs[v] = ssq_to_metres(c, hf);
        }
      }
    }
  }
}

}  // namespace pcsdf
