// The static EDT's column passes by propagation (included by edt.hip), for
// volumes in which no voxel is farther than kReachMax voxels from the other
// type's set, or has none to be near to; and, in 32 bits (kWide), for short
// columns whatever the distances.
//
// g(q) = min over p of f(p) + (q - p)^2 along a column.  Moving one step
// further from a site costs 1, 3, 5, ...: after iterations k = 1 .. K of
//   u(q) <- min(u(q), u(q-1) + 2k - 1, u(q+1) + 2k - 1)
// u(q) is the minimum over |q - p| <= K (a site d steps away pays least by
// moving in the first d iterations, 1 + 3 + .. + (2d-1) = d^2), and an
// iteration that changes nothing is followed by none that does, its step
// being dearer.  The column is in registers: neighbours in the column are
// neighbouring registers, and an iteration is an addition and a minimum of
// three for two columns, packed.
//
// How far to go.  k_pass_x_coarse and k_reach bound every voxel's distance
// from the occupancy.  The nearest site of a voxel v bounded by B is at most
// B away along each axis, so the partial values on its way come from rows
// within B of v along y and z, in at most B iterations: a row takes part in
// as many as the largest B of the voxels (of its x tile) that it is that near
// to, and any value above that is as good as none.  Without a bound the y
// pass would go on for hundreds of steps in layers with few sites, for values
// that the z pass then takes from another layer.
//
// Both channels run in one array: a voxel holds the distance to the other
// type's set, and a row of the other type is a site of value 0.  The first
// iteration (done as the rows are loaded) so gives 1, the least there is, to
// both sides of every border between the types.  No later iteration is
// masked: nothing gets past a border, where it would arrive with 1 + 3 or
// more, and a site beyond a border is never the nearest, the border's is.
//
// Values are whole numbers in 16 bits, two columns a register, exact up to
// kReachMax^2; the signed distances of the x pass and the signed squares
// between the passes are 16-bit too, half the traffic of 32.  In registers
// they are offset by kBias, which makes each the bit pattern of a normal
// fp16 number: these compare as the integers do, and the minimum of three
// is an fp16 instruction (16-bit integers have none).
//
// Measured, 512 x 512 x 256 with 200 boxes of 10-80 voxels (distances up to
// 107, bounds up to 142): y pass 279 us, z pass 228 (with both outputs, 671
// MB), where the envelopes and the search beside them took 587 and 582.  The
// passes are bound by the packed instructions, 4.5 cycles each, of about 20
// rounds of four iterations; 64 rows a wave (fewer halo rows, half the waves)
// took 307 and 244, an unpacked pair 3 x 2.4 cycles a voxel instead of 4.6.
#pragma once

#include "device_common.h"
#include "internal.h"

namespace pcsdf {

constexpr int kReachMax = 169;
constexpr int kFarDist = kReachMax + 1;     // any distance beyond
constexpr int kFar16 = kFarDist * kFarDist; // any square beyond
constexpr int kBias = 1024;                 // the least normal fp16 pattern
constexpr uint32_t kPairs = 0x00010001u;    // n * kPairs: n in both halves
// the largest value meant for a comparison is a finite fp16 number
static_assert(kFar16 + kBias + 2 * (kReachMax + 8) < 0x7C00, "fp16 patterns");

// ------------------------------------------------------------- the bound

constexpr int kPropCols = 128;  // columns per workgroup, two per lane
constexpr int kCoarse = 16;     // edge of a block along y and z

// The x pass (k_pass_x_vec's row, with distances of 16 bits as its result),
// and the occupancy of blocks of VPL (at most 64 along x, a lane each) by 16
// by 4 voxels, which it has in its hands: bit bx of occ_bits[r]
// (free_bits[r]): block (bx, r) has an occupied (a free) voxel; r = bz cy +
// by.  Grid: one workgroup per r, a wave per layer of it.
constexpr int kXLayers = 4;

template <int VPL>
__global__ __launch_bounds__(64 * kXLayers) void k_pass_x_coarse(
    const uint8_t *__restrict__ occ, int16_t *__restrict__ out, int nx, int ny,
    int nz, int cy, uint64_t *__restrict__ occ_bits,
    uint64_t *__restrict__ free_bits) {
  __shared__ uint64_t any[2][kXLayers];
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int bz = blockIdx.x / cy, y0 = (blockIdx.x - bz * cy) * kCoarse;
  const int z = bz * kXLayers + w;
  uint64_t has_occ = 0, has_free = 0;
  if (z < nz) {
    const int rows = min(kCoarse, ny - y0), i0 = lane * VPL;
    const int64_t at = ((int64_t)z * ny + y0) * nx;
    const uint8_t *src = occ + at;
    int16_t *dst = out + at;
    // two rows' occupancy is on its way while a row is done
    typename BytePack<VPL>::T raw = x_load<VPL>(src, nx, lane);
    typename BytePack<VPL>::T next =
        x_load<VPL>(src + min(1, rows - 1) * nx, nx, lane);
    for (int r = 0; r < rows; ++r) {
      const typename BytePack<VPL>::T after =
          x_load<VPL>(src + min(r + 2, rows - 1) * nx, nx, lane);
      int d[VPL];
      uint32_t mo;
      uint64_t lo, lf;
      x_row<VPL>(raw, nx, lane, d, &mo, &lo, &lf);
      raw = next;
      next = after;
      has_occ |= lo;
      has_free |= lf;
      uint32_t v[VPL / 2];
      x_words<VPL>(d, mo, v);
      if (i0 < nx) x_store<VPL>(dst + i0, v);
      dst += nx;
    }
  }
  if (lane == 0) {
    any[0][w] = has_occ;
    any[1][w] = has_free;
  }
  __syncthreads();
  if (threadIdx.x < 2) {
    uint64_t v = 0;
    for (int q = 0; q < kXLayers; ++q) v |= any[threadIdx.x][q];
    (threadIdx.x ? free_bits : occ_bits)[blockIdx.x] = v;
  }
}

// Bound of every voxel's distance.  The marked blocks are grown, by turns to
// the six neighbours and to the 3x3x3 surroundings (along x by as many blocks
// as make 16 voxels), until they hold every block that has a voxel of the
// other type.  After a steps of the second kind and b of the first, a block
// in the grown set is at most 16 (a + b, a, a) voxels (in some order) from a
// marked one, and any two voxels of theirs at most 15 more along each axis.
// One workgroup, a thread per row of blocks of 16^2 (cy cz <= 1024) made of
// those of k_pass_x_coarse, of which there are cq layers.  bound: for each
// 128 voxels of a row of blocks the largest bound, [tiles][cy cz].
__global__ __launch_bounds__(1024) void k_reach(
    const uint64_t *__restrict__ occ_bits,
    const uint64_t *__restrict__ free_bits, int fx, int cy, int cz, int cq,
    int tiles, int32_t *__restrict__ bound, EdtPlan *plan) {
  // rows put for the neighbours to read, into one of two by turns, so that
  // one barrier a time is enough
  __shared__ uint64_t grown[2][2][1024];
  // whether a needed block is open still, of three steps by turns
  __shared__ int blank[3];
  const int n = cy * cz, r = threadIdx.x;
  const int z = r / cy, y = r - z * cy;
  const bool in = r < n;
  uint64_t occ = 0, fre = 0;
  constexpr int kPer = kCoarse / kXLayers;
  {
    uint64_t o[kPer], f[kPer];
#pragma unroll
    for (int e = 0; e < kPer; ++e) {
      const int q = in ? min(z * kPer + e, cq - 1) * cy + y : 0;
      o[e] = occ_bits[q];
      f[e] = free_bits[q];
    }
#pragma unroll
    for (int e = 0; e < kPer; ++e) {
      occ |= in ? o[e] : 0ull;
      fre |= in ? f[e] : 0ull;
    }
  }
  const uint64_t need_occ = fre, need_free = occ;
  if (threadIdx.x < 3) blank[threadIdx.x] = 0;
  __syncthreads();
  // (bits beyond the last block may be set: no voxel needs them)
  auto wide = [&](uint64_t v) {
    v |= v << 1 | v >> 1;
    if (fx < 16) v |= v << 1 | v >> 1;
    return fx < 8 ? v | v << 2 | v >> 2 : v;
  };
  int turn = 0;
  auto put = [&]() {
    turn ^= 1;
    grown[turn][0][r] = occ;
    grown[turn][1][r] = fre;
  };
  // a neighbouring row, or (no branches) the own one where there is none
  auto take = [&](int c, int row) { return grown[turn][c][row]; };
  const int up = in && y > 0 ? r - 1 : r;
  const int down = in && y + 1 < cy ? r + 1 : r;
  const int front = in && z > 0 ? r - cy : r;
  const int back = in && z + 1 < cz ? r + cy : r;
  const int per = kPropCols / fx;  // blocks of a tile
  bool found = false;
  uint64_t open = need_occ | need_free;  // blocks whose bound is not known
  for (int step = 0, a = 0, b = 0;; ++step) {
    const int far = kCoarse * (a + b + 1) - 1, near = kCoarse * (a + 1) - 1;
    const int bound2 = far * far + 2 * near * near;
    int reach = (int)__builtin_amdgcn_sqrtf((float)bound2);
    while (reach * reach < bound2) ++reach;
    if (reach > kReachMax) break;
    const uint64_t left = (need_occ & ~occ) | (need_free & ~fre);
    if (const uint64_t now = open & ~left)
      for (int t = 0; t < tiles; ++t)
        if (now >> (t * per) & (~0ull >> (64 - per))) bound[t * n + r] = reach;
    open = left;
    if (left) blank[step % 3] = 1;
    const bool cube = step & 1;
    const uint64_t wo = wide(occ), wf = wide(fre);
    if (cube) {
      occ = wo;
      fre = wf;
    }
    put();
    __syncthreads();
    if (blank[step % 3] == 0) {
      found = true;
      break;
    }
    // (read a barrier ago at the latest, written again after another)
    if (threadIdx.x == 0) blank[(step + 2) % 3] = 0;
    if (cube) {
      ++a;
      occ |= take(0, up) | take(0, down);
      fre |= take(1, up) | take(1, down);
      put();
      __syncthreads();
      occ |= take(0, front) | take(0, back);
      fre |= take(1, front) | take(1, back);
    } else {
      ++b;
      occ = wo | take(0, up) | take(0, down) | take(0, front) | take(0, back);
      fre = wf | take(1, up) | take(1, down) | take(1, front) | take(1, back);
    }
  }
  if (threadIdx.x == 0) plan->near = found;
}

// ------------------------------------------------------------ the passes

constexpr int kPropRows = 32;   // rows per wave (R; 48 where one is enough)
constexpr int kPropWaves = 16;  // waves per workgroup, at most
constexpr int kPropHalo = 4;    // rows from either neighbour, iterations
                                // between exchanges
constexpr int kPropBatch = 7;   // rows loaded together

typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
typedef int16_t i16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t pair16 __attribute__((aligned(2)));  // two 16-bit elements
typedef int32_t i32x2u __attribute__((ext_vector_type(2), aligned(4)));
typedef float f32x2u __attribute__((ext_vector_type(2), aligned(4)));

template <class T>
__device__ __forceinline__ T as(uint32_t v) {
  return __builtin_bit_cast(T, v);
}
template <class T>
__device__ __forceinline__ uint32_t bits(T v) {
  return __builtin_bit_cast(uint32_t, v);
}
__device__ __forceinline__ uint32_t add2(uint32_t a, uint32_t b) {
  return bits(as<u16x2>(a) + as<u16x2>(b));
}
// Minimum of three: of positive fp16 patterns in both halves, or (kWide) of
// whole words.
template <bool kWide>
__device__ __forceinline__ uint32_t min3(uint32_t a, uint32_t b, uint32_t c) {
  if constexpr (kWide) return min(min(a, b), c);
  return bits(__builtin_elementwise_minimum(
      __builtin_elementwise_minimum(as<f16x2>(a), as<f16x2>(b)),
      as<f16x2>(c)));
}

// 32-bit values, one column a lane: no distance is too far for them.
constexpr int32_t kNone32 = 1 << 30;

// One iteration over rows 1 .. N-2 of u (the outermost rows only give), step
// cost c in both halves; with kTrack, the bits that changed in the own rows.
// A row's new value takes the register that the row before it in the sweep
// left; sweeps up and down in turn leave every row where it was.
template <bool kWide, int N, bool kUp, bool kTrack>
__device__ __forceinline__ uint32_t prop_step(uint32_t (&u)[N], uint32_t c) {
  constexpr int H = kPropHalo, d = kUp ? -1 : 1;
  if constexpr (kWide) {
    uint32_t prev = kUp ? u[N - 1] : u[0], acc = 0;
    asm volatile("" : "+s"(c));  // one sum per row, not of three
#pragma unroll
    for (int e = 1; e < N - 1; ++e) {
      const int j = (kUp ? N - 1 : 0) + d * e;
      const uint32_t x = u[j];
      uint32_t v = min(x, min(prev, u[j + d]) + c);
      // (or the compiler forms sums of two iterations, and runs out of
      // registers)
      asm volatile("" : "+v"(v));
      u[j] = v;
      if (kTrack && j >= H && j < N - H) acc |= u[j] ^ x;
      prev = x;
    }
    return acc;
  }
  constexpr int first = kUp ? N - 1 : 0;
  uint32_t before = add2(u[first], c), acc = 0;
  uint32_t here = add2(u[first + d], c), after = add2(u[first + 2 * d], c);
#pragma unroll
  for (int e = 1; e < N - 1; ++e) {
    const int j = first + d * e;
    // (the sum for the next row first: an instruction on packed values
    // cannot follow one that it depends on at once)
    const uint32_t ahead = e < N - 2 ? add2(u[j + 2 * d], c) : 0u;
    const uint32_t x = u[j];
    u[j] = min3<false>(x, before, after);
    if (kTrack && j >= H && j < N - H) acc |= u[j] ^ x;
    before = here;
    here = after;
    after = ahead;
  }
  return acc;
}

// Dynamic LDS of a workgroup: above, between and below its waves, twice
// (rounds alternate), the last rows of the one and the first of the other.
inline int prop_lds(int waves) { return (waves + 1) * 2 * 2 * kPropHalo * 256; }

// in_: columns of m rows at `stride`, element i of outer index o's row q at
// o * outer_stride + q * stride + i, i < nfast (2 at least).  In pairs, in_
// holds with kFirst the x pass's signed 16-bit distances, else signed
// squares; the result, out_, is 16-bit squares again or, with kLast, 32-bit
// ones and (kSdf) sdf.  kWide: squares of 32 bits in and out, whatever
// their size, one column a lane.  Grid: (tiles of 128 columns, kWide: 64) x
// nouter; block: ceil(m / R) waves.
template <bool kWide, int R, bool kFirst, bool kLast, bool kSdf>
__global__ __launch_bounds__(64 * kPropWaves) void k_pass_col_prop(
    const void *__restrict__ in_, void *__restrict__ out_,
    float *__restrict__ sdf, float hf, int nfast, int m, int64_t stride,
    int64_t outer_stride, int tiles, int cy, int cz,
    const int32_t *__restrict__ bound, const EdtPlan *__restrict__ plan) {
  constexpr int H = kPropHalo, N = R + 2 * H;
  constexpr int kSigns = kWide ? 32 : 16, B = (R + kSigns - 1) / kSigns;  // rows a word
  constexpr int kCols = kWide ? 1 : 2;                     // per lane
  typedef typename std::conditional<kWide, int32_t, int16_t>::type T;
  extern __shared__ uint32_t edge[];  // [2][waves + 1][2][H][64]
  __shared__ int flag[2][kPropWaves];
  if (!kWide && plan && !plan->near) return;
  __shared__ int limits[kPropWaves];
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int waves = blockDim.x >> 6;
  const int o = blockIdx.x / tiles, tile = blockIdx.x - o * tiles;
  const int i0 = kCols * (tile * 64 + lane);
  // lanes at or past the last column take the last (two) again; one with an
  // odd last column so has it as its pair's second
  const int ip = min(i0, nfast - kCols);
  const bool pair = i0 + 1 < nfast, single = i0 + 1 == nfast;
  const int q0 = w * R;
  const int64_t base = o * outer_stride;

  // The iterations of this wave's rows, and the workgroup's most.  The
  // column runs along y (kFirst) or z; along the other axis it is at o.
  // Without a plan, none is left out.
  int limit = m, longest = m;
  if (!kWide && plan) {
    limit = longest = 0;
    const int n = cy * cz;
    for (int c = lane; c < n; c += 64) {
      const int b = bound[tile * n + c];
      const int bz = c / cy, by = c - bz * cy;
      auto gap = [](int cell, int first, int last) {
        return max(max(cell * kCoarse - last, first - cell * kCoarse -
                                                  (kCoarse - 1)), 0);
      };
      const int along = gap(kFirst ? by : bz, q0, min(q0 + R, m) - 1);
      const int across = gap(kFirst ? bz : by, o, o);
      if (along <= b && (kFirst ? across <= b : across == 0))
        limit = max(limit, b);
    }
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) limit = max(limit, __shfl_xor(limit, d));
    limit = __builtin_amdgcn_readfirstlane(limit);
    if (lane == 0) limits[w] = limit;
    __syncthreads();
    for (int q = 0; q < waves; ++q) longest = max(longest, limits[q]);
    longest = __builtin_amdgcn_readfirstlane(longest);
  }

  constexpr uint32_t kCap =
      kWide ? (uint32_t)kNone32 : kPairs * (kBias + kFar16);  // none
  uint32_t u[N];
  uint32_t neg[B] = {};  // the own rows' signs, a row per bit of a half
  {
    // Rows q0 - H - 1 .. q0 + R + H, one more on either side than u holds:
    // after the first iteration all of u is exact.
    const T *row = static_cast<const T *>(in_) + base +
                   max(q0 - H - 1, 0) * stride;  // uniform
    // next to a border, and anywhere
    constexpr uint32_t kCap1 = kWide ? 1u : kPairs * (kBias + 1);
    uint32_t above = 0, type_above = 0;  // of the row above: value + 1, type
    // kPropBatch rows' loads are in flight while as many are taken in
    uint32_t x[2][kPropBatch];
    auto load = [&](int j0) {
#pragma unroll
      for (int e = 0; e < kPropBatch; ++e) {
        if (j0 + e >= N + 2) break;
        const int q = q0 - H - 1 + j0 + e;
        if constexpr (kWide)
          x[(j0 / kPropBatch) & 1][e] = (uint32_t)row[(uint32_t)ip];
        else
          x[(j0 / kPropBatch) & 1][e] =
              *reinterpret_cast<const pair16 *>(row + (uint32_t)ip);
        // on to row q + 1, if q and it are rows (no branches: masks)
        row += stride & ~(int64_t)((q | (m - 2 - q)) >> 31);
      }
    };
    load(0);
#pragma unroll
    for (int j0 = 0; j0 < N + 2; j0 += kPropBatch) {
      if (j0 + kPropBatch < N + 2) load(j0 + kPropBatch);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int e = 0; e < kPropBatch; ++e) {
        const int j = j0 + e, q = q0 - H - 1 + j;  // u[j - 1] is row q
        if (j >= N + 2) break;
        const uint32_t in = x[(j0 / kPropBatch) & 1][e];
        // beyond the column there is no site (and, rows repeated, no border)
        const uint32_t gone = (uint32_t)((q | (m - 1 - q)) >> 31);
        uint32_t type, v, step;  // type: all ones where occupied
        if constexpr (kWide) {
          type = (uint32_t)((int32_t)in >> 31);
          v = (uint32_t)max((int32_t)in, -(int32_t)in) | (gone >> 1);
          v = min(v, (uint32_t)kNone32);
          step = v + 1;
        } else {
          const i16x2 s = as<i16x2>(in);
          type = bits(s >> 15);
          v = bits(__builtin_elementwise_max(s, -s)) | (gone & 0x7FFF7FFFu);
          v = bits(__builtin_elementwise_min(
              as<u16x2>(v),
              as<u16x2>(kPairs * (uint32_t)(kFirst ? kFarDist : kFar16))));
          if (kFirst) v = bits(as<u16x2>(v) * as<u16x2>(v));
          v = add2(v, kPairs * kBias);
          step = add2(v, kPairs);
        }
        const uint32_t differ = type ^ type_above;
        const uint32_t cap = (differ & kCap1) | (~differ & kCap);
        if (j >= 2) u[j - 2] = min3<kWide>(u[j - 2], step, cap);
        if (j >= 1 && j <= N) u[j - 1] = min3<kWide>(v, above, cap);
        above = step;
        type_above = type;
        if (j > H && j <= R + H)
          neg[(j - H - 1) / kSigns] |=
              type & ((kWide ? 1u : kPairs) << ((j - H - 1) % kSigns));
      }
      // computed here, not where they are first used
#pragma unroll
      for (int e = 0; e < kPropBatch; ++e)
        if (j0 + e >= 1 && j0 + e <= N) asm volatile("" : "+v"(u[j0 + e - 1]));
#pragma unroll
      for (int e = 0; e < B; ++e) asm volatile("" : "+v"(neg[e]));
      __builtin_amdgcn_sched_barrier(0);
    }
  }

  // Rounds of iterations k .. k + 3.  A row changes only in the iteration
  // after a change of a row next to it, so a wave sits four out if
  // in the last one neither its rows changed nor its neighbours'; the
  // workgroup ends when in the last one no row did, or at its limits.
  bool run = true, was = true;
  uint32_t *const above = edge + w * (2 * H * 64) + lane;
  uint32_t *const below = above + 2 * H * 64;
  const int other = (waves + 1) * (2 * H * 64);
#pragma unroll
  for (int e = 0; e < H; ++e) {  // no rows beyond the column
    if (w == 0)
      above[e * 64] = above[other + e * 64] = kCap;
    if (w == waves - 1)
      below[(H + e) * 64] = below[other + (H + e) * 64] = kCap;
  }
  int p = 0, buf = 0;
  for (int k = 2;; k += H) {
    bool ch = false;
    if (run) {
      constexpr uint32_t kOne = kWide ? 1u : kPairs;
      const uint32_t c = kOne * (uint32_t)(2 * k - 1);
      prop_step<kWide, N, false, false>(u, c);
      prop_step<kWide, N, true, false>(u, c + 2 * kOne);
      prop_step<kWide, N, false, false>(u, c + 4 * kOne);
      uint32_t acc = prop_step<kWide, N, true, true>(u, c + 6 * kOne);
      asm volatile("" : "+v"(acc));  // one word, not a flag per row
      ch = __ballot(acc != 0) != 0;
    }
    if (k + H > longest) break;
    // (written once more after the last change, into the other buffer)
    if (run || was) {
#pragma unroll
      for (int e = 0; e < H; ++e) {
        below[buf + e * 64] = u[R + e];
        above[buf + (H + e) * 64] = u[H + e];
      }
    }
    was = run;
    if (lane == 0) flag[p][w] = ch;
    __syncthreads();
    const uint64_t mask =
        __ballot(lane < waves && flag[p][lane & (kPropWaves - 1)]);
    if (mask == 0) break;
    run = (((mask << 1) >> w) & 7) != 0 && k + H <= limit;
    if (run) {
#pragma unroll
      for (int e = 0; e < H; ++e) {
        u[e] = above[buf + e * 64];
        u[R + H + e] = below[buf + (H + e) * 64];
      }
    }
    p ^= 1;
    buf = other - buf;
  }

  const int64_t at = base + q0 * stride;  // uniform
  int16_t *dst16 = static_cast<int16_t *>(out_) + at;
  int32_t *dst = static_cast<int32_t *>(out_) + at;
  float *fdst = kSdf ? sdf + at : nullptr;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    if (q0 + r < m) {  // uniform
      const uint32_t v = u[H + r];
      if constexpr (kWide) {
        int32_t a = (int32_t)v;
        a = a >= kNone32 ? kInf : a;
        const int32_t sa = (int32_t)(neg[r / 32] << (31 - r % 32)) >> 31;
        a = (a ^ sa) - sa;
        if (i0 < nfast) {
          dst[(uint32_t)i0] = a;
          if (kSdf) fdst[(uint32_t)i0] = ssq_to_metres(a, hf);
        }
      } else if (!kLast) {
        const i16x2 s = as<i16x2>(neg[r / 16] << (15 - r % 16)) >> 15;
        const i16x2 x = as<i16x2>(v) - (int16_t)kBias;
        const uint32_t sv = bits((x ^ s) - s);
        if (pair)
          *reinterpret_cast<pair16 *>(dst16 + (uint32_t)i0) = sv;
        else if (single)
          dst16[(uint32_t)i0] = (int16_t)(sv >> 16);
      } else {
        // (kFar16 is left where there is no site at all)
        int32_t a = (int32_t)(v & 0xFFFFu) - kBias;
        int32_t b = (int32_t)(v >> 16) - kBias;
        a = a == kFar16 ? kInf : a;
        b = b == kFar16 ? kInf : b;
        const int32_t sa = (int32_t)(neg[r / 16] << (31 - r % 16)) >> 31;
        const int32_t sb = (int32_t)(neg[r / 16] << (15 - r % 16)) >> 31;
        const int32_t va = (a ^ sa) - sa, vb = (b ^ sb) - sb;
        if (pair) {
          *reinterpret_cast<i32x2u *>(dst + (uint32_t)i0) = i32x2u{va, vb};
          if (kSdf)
            *reinterpret_cast<f32x2u *>(fdst + (uint32_t)i0) =
                f32x2u{ssq_to_metres(va, hf), ssq_to_metres(vb, hf)};
        } else if (single) {
          dst[(uint32_t)i0] = vb;
          if (kSdf) fdst[(uint32_t)i0] = ssq_to_metres(vb, hf);
        }
      }
    }
    if (!kWide && !kLast) dst16 += stride;
    if (kWide || kLast) dst += stride;
    if (kSdf) fdst += stride;
  }
}

}  // namespace pcsdf
