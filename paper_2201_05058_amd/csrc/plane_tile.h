// Planar signed field of a slice's disks in one step, tile by tile: the
// workgroup builds the chords of the slice's disks in LDS (only the rows a
// disk covers), then each wave evaluates 64 columns x 8 rows of pixels, a
// lane holding the eight rows of its column (G = 8 below; small calls take
// fewer, planes.hip).  Shared by the per-call kernel
// (planes.hip) and the batch's planar items (batch_device.h).
//
// A chord serves a whole wave: the row's index is uniform, the distance of
// the lane's column to the chord is formed once (four instructions) and
// offered to the eight rows of the column (an add and half a three-way min
// each), where one pixel per lane did the same work, and the tests around
// it, for every pixel.  Disks nearest first, rows outward from the tile; a
// disk, or the rest of its rows, is left out once no lane's values can still
// fall.  Pixels covered by a chord come out as distance zero: those get the
// distance to the nearest uncovered pixel, row by row outward, each row's
// value again formed once per column, from bits of the row's coverage (and,
// where a covered run is longer than the words, from its end, found once per
// row and wave).  Both are the definition of the squared distance written
// row by row (planes.hip), so the result is exact.
//
// Bound by instruction issue (512 x 512 x 50 x 8 issues in about every cycle of
// its SIMDs, three vector to two scalar instructions): about 110 vector
// instructions per four rows of a disk and 512 pixels; where one round of
// waves covers the launch, by the waves that hold covered pixels (about 25
// rows of 75 instructions more), which wait half their cycles on the chords'
// table.  Planar fields of a call: 256 x 256 x 20 slices x 3 discs 19 us in
// one launch (chords, row pass and one pixel per lane: 40 us in three), 512
// x 512 x 50 x 8 128-141 us (265 by coverage and column passes beside the
// other kernels of the call), 16 uneven rooms of a batch 57 us (326).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "plane_device.h"

namespace pcsdf {

constexpr int kTileCols = 64;  // a wave's columns
constexpr int kTileRows = 8;   // rows of a column per lane
constexpr int kTileWaves = 4;  // waves per workgroup, one above the other
constexpr int kTilePlaneMax = 2048;  // pixels per axis (see kNoChord)
// An empty chord's ends: farther from every column than any squared
// distance within kTilePlaneMax pixels (2 * 2047^2 < kTileFar <
// (kNoChord - 2047)^2), and its square fits in 32 bits.
constexpr int kNoChord = 8192;
constexpr int32_t kTileFar = 1 << 24;
constexpr int32_t kTileUnset = 1 << 30;

// Rows on either side of a wave's own whose coverage it holds as bits, one
// row per lane, with G rows of a column per lane.
constexpr int tile_reach(int G) { return (64 - G) / 2; }
constexpr int kTileReach = tile_reach(kTileRows);

// Tiles of a plane, numbered row-major.
__host__ __device__ inline int plane_tiles_x(int nx) {
  return (nx + kTileCols - 1) / kTileCols;
}
__host__ __device__ inline int plane_tiles(int nx, int ny,
                                           int G = kTileRows) {
  return plane_tiles_x(nx) *
         ((ny + G * kTileWaves - 1) / (G * kTileWaves));
}
// Rows a disk of fixed-point radius R can cover in ny rows, and the LDS
// bytes of K such disks (box, then chords, per disk).
__host__ __device__ inline int disk_rows(int64_t R, int ny) {
  const int64_t r = ((2 * R) >> 16) + 1;  // odd multiples of 2^15 in [-R, R]
  return (int)(r < ny ? r : ny);
}
// kEdge empty chords before a disk's first row and after its last let four
// rows be read at once without a test.
constexpr int kEdge = 3;
__host__ __device__ inline int64_t tile_lds(int K, int rows) {
  return (int64_t)K * 16 + (int64_t)K * (rows + 2 * kEdge) * 8;
}

// Uniform values and votes of a wave; a host build has one lane per wave.
#if defined(__clang__)
__device__ __forceinline__ int uni(int v) {
  return __builtin_amdgcn_readfirstlane(v);
}
__device__ __forceinline__ bool any_lane(bool b) { return __ballot(b) != 0; }
#else
inline int uni(int v) { return v; }
inline bool any_lane(bool b) { return b; }
#endif

// The slice's disks in LDS: boxes [K] and chords [K][stride], kEdge rows
// from before each box's first; empty chords hold (kNoChord, -kNoChord).
struct TileDisks {
  const int4 *box;
  const int2 *ch;
  int K, stride;
  // Disk k's chord of row z + q, -kEdge <= q < stride - kEdge.
  __device__ __forceinline__ int2 chord(int k, int q) const {
    return ch[k * stride + kEdge + q];
  }
};

// Fills the tables (all lanes of the workgroup; a barrier follows).  XY(k)
// gives disk k's centre.
template <class XY>
__device__ __forceinline__ TileDisks tile_disks(int4 *lds, int K, int rows,
                                                int64_t R, int nx, int ny,
                                                const XY &xy) {
  int4 *box = lds;
  int2 *ch = reinterpret_cast<int2 *>(lds + K);
  const int stride = rows + 2 * kEdge;
  for (int t = threadIdx.x; t < K * stride; t += blockDim.x) {
    const int k = t / stride, q = t - k * stride - kEdge;
    const int64_t X = xy(2 * k), Y = xy(2 * k + 1);
    const int4 b = disk_box(X, Y, R, nx, ny);
    if (q == 0) box[k] = b;
    int2 c = make_int2(1, 0);
    if (q >= 0 && b.z + q <= b.w) c = disk_chord(X, Y, R, nx, b.z + q);
    if (c.x > c.y) c = make_int2(kNoChord, -kNoChord);
    ch[t] = c;
  }
  return TileDisks{box, ch, K, stride};
}

// A lane's eight values are held less g^2 for row j0 + g: with t = r - j0, a
// row r at distance f along x gives row g the value f + (t - g)^2, that is
// (f + t^2) - 2 t g + g^2, so one uniform 2 t steps through the rows and no
// square is formed per row.  kTileSkip, below every such value, stays.
constexpr int32_t kTileSkip = -1000;

// The largest of the values.
template <int G>
__device__ __forceinline__ int32_t max_of(const int32_t (&v)[G]) {
  int32_t m = v[0];
#pragma unroll
  for (int g = 1; g < G; ++g) m = max(m, v[g] + g * g);
  return m;
}
// At least the largest of the values, by less than G^2.
template <int G>
__device__ __forceinline__ int32_t bound_of(const int32_t (&v)[G]) {
  int32_t m = v[0];
#pragma unroll
  for (int g = 1; g < G; ++g) m = max(m, v[g]);
  return m + (G - 1) * (G - 1);
}
// Offers a row at distance f along x, t rows from j0.
template <int G>
__device__ __forceinline__ void offer_row(int32_t f, int t, int32_t (&v)[G]) {
  int32_t c = f + t * t;
#pragma unroll
  for (int g = 0; g < G; ++g) {
    v[g] = min(v[g], c);
    c -= 2 * t;
  }
}

// Offers the chords of four rows rr, rr + dir, ... of disk k (first row z;
// rr one of its rows) to the column's rows j0 .. j0 + 7; returns the last
// row's distance from the column to its chord (over kNoChord / 2: none).
template <int G>
__device__ __forceinline__ int offer_rows(const TileDisks &d, int k, int z,
                                          int rr, int dir, int i, int j0,
                                          int32_t (&best)[G]) {
  int dx[4];
  int32_t dx2[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int2 c = d.chord(k, rr - z + u * dir);
    dx[u] = max(0, max(c.x - i, i - c.y));
    dx2[u] = sq24(dx[u]);
  }
  const int t = rr - j0;  // uniform
  int32_t c0 = dx2[0] + t * t;
  int32_t c1 = dx2[1] + (t + dir) * (t + dir);
  int32_t c2 = dx2[2] + (t + 2 * dir) * (t + 2 * dir);
  int32_t c3 = dx2[3] + (t + 3 * dir) * (t + 3 * dir);
#pragma unroll
  for (int g = 0; g < G; ++g) {
    best[g] = min(min(best[g], min(c0, c1)), min(c2, c3));
    c0 -= 2 * t;
    c1 -= 2 * (t + dir);
    c2 -= 2 * (t + 2 * dir);
    c3 -= 2 * (t + 3 * dir);
  }
  return dx[3];
}

// Lowers best by disk k where it can: its rows outward from the tile in each
// direction, four at a time, until in every lane either the box is too far
// or the distance can only grow.  The squared distance from a pixel to the
// disk's points of height r is convex in r (least over x of a convex
// function on a convex set), at most the chord's dx^2 + dy^2, and more than
// (dx - 1)^2 + dy^2, since the chord's end is the first pixel centre inside
// the disk.  So if that lower bound at a step's last row reaches the value
// at the previous step's last row, the convex function has begun to rise:
// no later row is below a value already offered.  The bounds' difference
// over four rows, 8 dist - 16 + (dx - 1)^2 - dx_prev^2, is least for the
// row of the tile nearest to the chord (dist rows away).
template <int G>
__device__ __forceinline__ void offer_disk(const TileDisks &d, int k, int i,
                                           int j0, int32_t (&best)[G]) {
  const int4 b = d.box[k];
  const int z = uni(b.z), w = uni(b.w);
  const int32_t dxb2 = sq24(max(0, max(b.x - i, i - b.y)));
  const int r0 = min(max(j0 + G / 2, z), w);
  auto rising = [](int dist, int dx, int prev) {
    const int m = max(dx - 1, 0);
    return dx < kNoChord / 2 && prev < kNoChord / 2 &&
           8 * dist - 16 + sq24(m) - sq24(prev) >= 0;
  };
  // one copy of the loop for both directions: this code runs once per wave
  // in most launches, from a cold instruction cache
  for (int dir = 1; dir >= -1; dir -= 2) {
    int prev = kNoChord;
    bool done = false;
    const int end = dir > 0 ? w : -z;
    for (int rr = dir > 0 ? r0 : r0 - 1; rr * dir <= end; rr += 4 * dir) {
      // rows between the tile and rr, and after the step's last row
      const int gap = dir > 0 ? rr - (j0 + G - 1) : j0 - rr;
      const int dy = max(0, gap);
      if (!any_lane(!done && bound_of(best) > dy * dy + dxb2)) break;
      const int dx = offer_rows(d, k, z, rr, dir, i, j0, best);
      done = done || rising(gap + 3, dx, prev);
      prev = dx;
    }
  }
}

// The free pixels of 64 rows from r0 around a wave's columns, one bit each:
// word q holds columns i0 - 64 + 64 q .. + 63 (columns outside the plane
// are not free), and the distances from column i0 to the nearest free one to
// the left of the words and to the right (kNoChord: none, or not needed, the
// outer word having one).  On the device lane l holds row r0 + l and at(r)
// reads a row's words into scalar registers; a host build forms the row
// asked for.
struct RowBits {
  uint64_t w[3];
  int left, right;
};
struct FreeBits {
#if defined(__clang__)
  RowBits b;
  bool outer;  // uniform: some row has a distance beyond the words
#else
  const TileDisks *d;
  int i0, nx, ny;
#endif
  int r0;
};
// Bits a .. b of word q (bit 0 is position 64 q); none when a > b.
__device__ __forceinline__ uint64_t bit_range(int a, int b, int q) {
  const int lo = max(a - 64 * q, 0), hi = min(b - 64 * q, 63);
  return lo <= hi ? (~0ull >> (63 - (hi - lo))) << lo : 0ull;
}
__device__ __forceinline__ RowBits free_row(const TileDisks &d, int r, int i0,
                                            int nx, int ny) {
  RowBits f;
#pragma unroll
  for (int q = 0; q < 3; ++q)
    f.w[q] = bit_range(64 - i0, 64 - i0 + nx - 1, q);
  for (int k = 0; k < d.K; ++k) {
    const int4 b = d.box[k];
    if (b.x > b.y || r < b.z || r > b.w) continue;
    const int2 c = d.chord(k, r - b.z);
#pragma unroll
    for (int q = 0; q < 3; ++q)
      f.w[q] &= ~bit_range(c.x - i0 + 64, c.y - i0 + 64, q);
  }
  f.left = f.right = kNoChord;
  return f;
}
// The distances beyond the words, where an outer word has no free bit and the
// plane goes on: the covered run's end, chord by chord.
__device__ __forceinline__ bool free_beyond(const TileDisks &d, int r, int i0,
                                            int nx, RowBits *f) {
  const bool row = r >= 0;
  const bool need_l = row && i0 > 64 && f->w[0] == 0;
  const bool need_r = row && i0 + 128 < nx && f->w[2] == 0;
  if (!any_lane(need_l || need_r)) return false;
  int lo = i0 - 65, hi = i0 + 128;
  for (bool moved = true; any_lane(moved);) {
    moved = false;
    for (int k = 0; k < d.K; ++k) {
      const int4 b = d.box[k];
      if (b.x > b.y || r < b.z || r > b.w) continue;
      const int2 c = d.chord(k, r - b.z);
      if (need_l && lo >= c.x && lo <= c.y) {
        lo = c.x - 1;
        moved = true;
      }
      if (need_r && hi >= c.x && hi <= c.y) {
        hi = c.y + 1;
        moved = true;
      }
    }
  }
  if (need_l && lo >= 0) f->left = i0 - lo;
  if (need_r && hi < nx) f->right = hi - i0;
  return true;
}
__device__ __forceinline__ FreeBits free_bits(const TileDisks &d, int r0,
                                              int i0, int nx, int ny) {
  FreeBits f;
  f.r0 = r0;
#if defined(__clang__)
  const int r = r0 + (int)(threadIdx.x & 63);
  f.b = free_row(d, r, i0, nx, ny);
  f.outer = free_beyond(d, r, i0, nx, &f.b);
#else
  f.d = &d;
  f.i0 = i0;
  f.nx = nx;
  f.ny = ny;
#endif
  return f;
}
__device__ __forceinline__ RowBits bits_at(const FreeBits &f, int r) {
#if defined(__clang__)
  RowBits b;
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    const uint32_t lo =
        __builtin_amdgcn_readlane((uint32_t)f.b.w[q], r - f.r0);
    const uint32_t hi =
        __builtin_amdgcn_readlane((uint32_t)(f.b.w[q] >> 32), r - f.r0);
    b.w[q] = (uint64_t)hi << 32 | lo;
  }
  b.left = b.right = kNoChord;
  if (f.outer) {
    b.left = __builtin_amdgcn_readlane(f.b.left, r - f.r0);
    b.right = __builtin_amdgcn_readlane(f.b.right, r - f.r0);
  }
  return b;
#else
  RowBits b = free_row(*f.d, r, f.i0, f.nx, f.ny);
  free_beyond(*f.d, r, f.i0, f.nx, &b);
  return b;
#endif
}
// Squared distance along a row from column i0 + l (l in [0, 64)) to its
// nearest free pixel; kTileUnset when the row has none.
__device__ __forceinline__ int32_t row_free2(const RowBits &b, int l) {
  // the nearest bits beside the lane's word are the same for all lanes; a
  // lane's own word first (bit 0 or 63 set where it has none: the value is
  // not used)
  const int c0 = b.w[0] ? 1 + __builtin_clzll(b.w[0]) : b.left;
  const int c2 = b.w[2] ? 64 + __builtin_ctzll(b.w[2]) : b.right;
  const uint64_t le = b.w[1] & (~0ull >> (63 - l));
  const uint64_t ge = b.w[1] & (~0ull << l);
  const int own_l = l - 63 + __builtin_clzll(le | 1);
  const int own_r = __builtin_ctzll(ge | 1ull << 63) - l;
  const int dl = le ? own_l : l + c0;
  const int dr = ge ? own_r : c2 - l;
  const int m = min(dl, dr);
  return m >= kNoChord / 2 ? kTileUnset : sq24(m);
}

// The same from the chords, for rows beyond the lanes': squared distances
// along eight rows from column i to each row's nearest pixel that no chord
// covers (0: column i itself; kTileUnset: none), the rows r0 + u for u < 4
// and r1 + u for the others.  The covered run through i grows until no chord
// overlaps or touches it; eight rows at a time, so that their reads of the
// table overlap.  Rows outside the table's disks read as uncovered.
__device__ __forceinline__ void tile_rows_free(const TileDisks &d, int r0,
                                               int r1, int nx, int i, bool in,
                                               int32_t (&f)[8]) {
  int lo[8], hi[8];  // empty so far: hi < i
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    lo[u] = i;
    hi[u] = i - 1;
  }
  bool grew = in;
  while (any_lane(grew)) {
    grew = false;
    for (int k = 0; k < d.K; ++k) {
      const int4 b = d.box[k];
      const int z = uni(b.z), w = uni(b.w);
      if (uni(b.x) > uni(b.y) || z > w || r0 > w ||
          (r0 + 3 < z && r1 > w) || r1 + 3 < z)
        continue;
      int2 c[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int r = (u < 4 ? r0 : r1 - 4) + u;
        c[u] = d.chord(k, min(max(r - z, -1), w - z + 1));
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const bool none = hi[u] < i;
        const bool meets = c[u].x <= (none ? i : hi[u] + 1) &&
                           c[u].y >= (none ? i : lo[u] - 1);
        const int l = min(lo[u], c[u].x), h = max(hi[u], c[u].y);
        if (in && meets && (l < lo[u] || h > hi[u])) {
          lo[u] = l;
          hi[u] = h;
          grew = true;
        }
      }
    }
  }
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    const int dl = lo[u] >= 1 ? i - lo[u] + 1 : kNoChord;
    const int dr = hi[u] <= nx - 2 ? hi[u] + 1 - i : kNoChord;
    const int m = min(dl, dr);
    f[u] = hi[u] < i ? 0 : (m == kNoChord ? kTileUnset : sq24(m));
  }
}

// Pixels (i, j0 .. j0 + 7) of the plane P [ny][nx]; i0 is the wave's first
// column.
template <int G>
__device__ __forceinline__ void plane_column(const TileDisks &d, int nx,
                                             int ny, int i0, int i, int j0,
                                             int32_t *__restrict__ P) {
  int32_t best[G];
#pragma unroll
  for (int g = 0; g < G; ++g)
    best[g] = i < nx && j0 + g < ny ? kTileUnset : kTileSkip;
  // the disk whose box is nearest to the wave's tile first
  int kb = -1;
  int32_t near = INT32_MAX;
  for (int k = 0; k < d.K; ++k) {
    const int4 b = d.box[k];
    const int x = uni(b.x), y = uni(b.y), z = uni(b.z), w = uni(b.w);
    if (x > y || z > w) continue;
    const int dx = max(0, max(x - (i0 + kTileCols - 1), i0 - y));
    const int dy = max(0, max(z - (j0 + G - 1), j0 - w));
    const int32_t lb = dx * dx + dy * dy;
    if (lb < near) {
      near = lb;
      kb = k;
    }
  }
  for (int q = kb < 0 ? d.K : -1; q < d.K; ++q) {
    const int k = q < 0 ? kb : q;
    const int4 b = d.box[k];
    if (q == kb || uni(b.x) > uni(b.y) || uni(b.z) > uni(b.w)) continue;
    offer_disk(d, k, i, j0, best);
  }
  // pixels at distance zero are covered
  bool in = false;
#pragma unroll
  for (int g = 0; g < G; ++g) {
    best[g] = best[g] >= kTileFar ? kInfP : best[g] + g * g;
    in = in || best[g] == 0;
  }
  if (any_lane(in)) {
    int32_t free2[G];  // kTileUnset only where it is needed
#pragma unroll
    for (int g = 0; g < G; ++g)
      free2[g] = best[g] == 0 ? kTileUnset : kTileSkip;
    const FreeBits bits = free_bits(d, j0 - tile_reach(G), i0, nx, ny);
    auto offer = [&](int r) {
      offer_row(row_free2(bits_at(bits, r), i - i0), r - j0, free2);
    };
    for (int r = j0; r < min(ny, j0 + G); ++r) offer(r);
    int q = 1;
    bool more = true;
    for (; q < tile_reach(G); q += 2) {
      const int lo = j0 - q, hi = j0 + G - 1 + q;
      more = (lo >= 0 || hi < ny) && any_lane(max_of(free2) > q * q);
      if (!more) break;
      if (lo >= 0) offer(lo);
      if (hi < ny) offer(hi);
      if (lo >= 1) offer(lo - 1);
      if (hi + 1 < ny) offer(hi + 1);
    }
    if (more) {  // deeper rows: from the chords
      auto offer8 = [&](int r0, int r1) {
        int32_t f[8];
        tile_rows_free(d, r0, r1, nx, i, in, f);
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int r = (u < 4 ? r0 : r1 - 4) + u;
          if (r < 0 || r >= ny) continue;  // uniform
          offer_row(f[u], r - j0, free2);
        }
      };
      for (;; q += 4) {
        const int lo = j0 - q, hi = j0 + G - 1 + q;
        if (lo < 0 && hi >= ny) break;
        if (!any_lane(max_of(free2) > q * q)) break;
        offer8(lo - 3, hi);
      }
    }
#pragma unroll
    for (int g = 0; g < G; ++g)
      if (best[g] == 0)
        best[g] = free2[g] >= kTileFar ? -kInfP : -(free2[g] + g * g);
  }
#pragma unroll
  for (int g = 0; g < G; ++g)
    if (i < nx && j0 + g < ny) P[(j0 + g) * nx + i] = best[g];
}

// Tile `tile` of one slice's plane; all 64 kTileWaves lanes of the workgroup
// (a host build's one lane loops over the pixels).
template <int G = kTileRows, class XY>
__device__ __forceinline__ void plane_tile(int4 *lds, int K, int rows,
                                           int64_t R, int nx, int ny,
                                           int tile, const XY &xy,
                                           int32_t *__restrict__ P) {
  const TileDisks d = tile_disks(lds, K, rows, R, nx, ny, xy);
  __syncthreads();
  const int tx = plane_tiles_x(nx);
  const int ty = tile / tx;
  const int i0 = (tile - ty * tx) * kTileCols;
#if defined(__clang__)
  // one lane per column and one wave per G rows
  const int j0 = (ty * kTileWaves + uni((int)threadIdx.x >> 6)) * G;
  if (j0 < ny)
    plane_column<G>(d, nx, ny, i0, i0 + (int)(threadIdx.x & 63), j0, P);
#else
  for (int w = 0; w < kTileWaves; ++w)
    for (int c = 0; c < kTileCols; ++c)
      if ((ty * kTileWaves + w) * G < ny)
        plane_column<G>(d, nx, ny, i0, i0 + c, (ty * kTileWaves + w) * G,
                     P);
#endif
}

}  // namespace pcsdf
