// Planar signed EDT of the humans' disk union, one plane per slice.
//
// A slice's human voxels are D x Z (see composite.hip), with D the union of
// the voxelised disks.  Each disk is convex, so its voxels in grid row j
// form one integer interval, a chord [a, b] of the closed predicate
//   (2^15(2i+1) - X)^2 + (2^15(2j+1) - Y)^2 <= R^2:
// with dy = 2^15(2j+1) - Y and W = floor(sqrt(R^2 - dy^2)), a voxel is in
// the chord iff |2^15(2i+1) - X| <= W, i.e. 2i+1 lies in
// [ceil((X-W)/2^15), floor((X+W)/2^15)].  All of this is exact integer
// arithmetic (divisions by powers of two are arithmetic shifts).
//
// With the chords in hand every pixel is independent.  Most calls evaluate
// them by tiles, chords and all in one launch (plane_tile.h).  Large stacks
// of slices with many chords take the static build's passes, and the rest is
// computed one pixel per lane:
//   outside D:  E_D(i,j) = min over disks, over the disk's rows jj, of
//               (j-jj)^2 + (distance from i to the chord)^2,
//               pruned by each disk's bounding box and by (j-jj)^2 >= best;
//   inside D:   E_{Gxy\D}(i,j) = min over rows jj of
//               (j-jj)^2 + (distance from i to the nearest uncovered pixel
//               of row jj)^2, searching rows outward from j and stopping
//               once (j-jj)^2 reaches the best value; in a row the covered
//               run through i is the union of the chords that overlap or
//               touch it.
// Both are the definition of the squared distance written row by row
// (the x term of the nearest voxel in row jj is the distance to the
// nearest chord end), so the result is exact.
#include <algorithm>
#include <type_traits>

#include "internal.h"
#include "plane_tile.h"

namespace pcsdf {

// The tiled kernel's limits.  Disks of more rows than its coverage words
// reach (kTileReach either side) would take its slow path, row by row from
// the chords, at every pixel they cover; so would dense crowds, whose disks
// join.  Against the paths below (us a call of 1000 direct queries; 51 rows
// per disk at 512 x 512, 26 at 256 x 256):
//   512 x 512 x 50 slices: 1, 8, 16, 32 disks 50, 107, 151, 420 against 141,
//   213, 236, 282 by coverage and column passes;
//   256 x 256 x 20: 3, 16, 64, 128 disks 22, 46, 112, 1245 against 39, 95,
//   360, 774 per pixel;  512 x 512 x 2: 8, 32, 64 disks 30, 50, 505 against
//   36, 82, 164.
// The lines are drawn in chords per slice, disks times rows.
// Crowds on small planes are the same when their discs are large for the
// plane: covered pixels then lie deeper than the words' rows.  The depth goes
// with how often the boxes cover the plane, times the rows of a disk: above
// kTileDepth tiles lose (us a call, tiles and the path below: 64 x 64 x 12, 8
// disks of 41 rows, 134, 82, 37; 100 x 100 x 12, 16 of 41, 110, 229, 59; 128 x
// 96 x 12, 8 of 51, 86, 48, 40; 48 x 64 x 12, 16 of 25, 81, 69, 51), under it
// they win (64 x 100 x 12, 32 of 25, 78, 53, 74; 48 x 64 x 12, 8 of 31, 77, 29,
// 34; 140 x 140 x 12, 16 of 41, 56, 52, 59; 48 x 64 x 12, 40 of 17, 64, 58, 80).
constexpr int64_t kTileLds = 48 * 1024;
constexpr int64_t kTileDepth = 80;
constexpr int kTileMaxRows = 2 * kTileReach;
constexpr int kTileChords = 1664;
constexpr int kTileChordsStack = 1024;  // where the column passes apply

// Workgroups up to which a lane holds two rows of its column instead of
// eight: such a call is over after one round of waves, whose chains of
// dependent steps are then less than half as long.  Us a call, eight rows
// against two: 80 x 68 x 2 slices, 4 and 8 disks 25, 34 against 19, 25 (22, 27
// by the paths below); 147 x 104 x 2, 7 disks 28, 22; 308 x 84 x 11 (165
// workgroups) 55, 53; but 512 x 512 x 2, 8 disks (256) 30, 35.  In larger
// calls on crowded planes, where most waves hold covered pixels, four rows:
// 100 x 100, 8 disks of 42 rows, 25 and 100 slices 64, 124 against 48, 107 (53,
// 124); 130 x 130 x 50 101, 88; elsewhere eight are as good or better.
constexpr int kTileFew = 192;

// chords[s][k][j] = (a, b), empty when a > b.
// Slices whose entry in `need` is zero are skipped (all slices when `need`
// is null) by this kernel and the two below.
// Rs[s] is slice s's fixed-point disk radius.
__global__ __launch_bounds__(256) void k_chords(Centres C, int K, int nx,
                                                int ny, int64_t total,
                                                const int32_t *__restrict__ need,
                                                int2 *__restrict__ chords) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (t >= total) return;
  const int j = (int)(t % ny);
  const int64_t sk = t / ny;  // s*K + k
  if (need && need[sk / K] == 0) return;
  const int64_t X = centre_word(C, 2 * sk), Y = centre_word(C, 2 * sk + 1);
  const int2 c = disk_chord(X, Y, radius_of(C, sk / K), nx, j);
  chords[t] = c;
}

// Row pass of the free-set channel for every pixel of every slice:
// F1[s][j][i] = squared distance along row j to the nearest uncovered
// pixel (0 when (i, j) is uncovered, kInf when the whole row is covered).
// Block b takes pixels 256 (b mod bpr) + 0..255 of row b / bpr of all
// slices' rows: the row, and so its chords, is uniform over the block.
__global__ __launch_bounds__(256) void k_rowfree(
    const int2 *__restrict__ chords, int K, int nx, int ny, int bpr,
    const int32_t *__restrict__ need, int32_t *__restrict__ F1) {
  const int row = (int)(blockIdx.x / (unsigned)bpr);  // s*ny + j
  const int i = (int)(blockIdx.x - (unsigned)row * bpr) * 256 + threadIdx.x;
  const int s = row / ny;
  if (i >= nx || (need && need[s] == 0)) return;
  const int j = row - s * ny;
  const GlobalTab ch{chords + (int64_t)s * K * ny};
  F1[(int64_t)row * nx + i] = row_free_dist(ch, K, ny, nx, j, i);
}

// Coverage of every pixel of every slice by the disks, one byte per pixel
// (1: covered): the map whose 2-D signed EDT is the planar field.  One
// block per row of one slice (nx <= 1024): the row's K chords are staged
// in LDS, and each lane marks 4 adjacent pixels, stored as one word when
// the row allows it.
__global__ __launch_bounds__(256) void k_cover(
    const int2 *__restrict__ chords, int K, int nx, int ny,
    uint8_t *__restrict__ cov) {
  __shared__ int2 rc[kMaxHumans];
  const int row = blockIdx.x;  // s*ny + j
  const int s = row / ny, j = row - s * ny;
  const int2 *ch = chords + (int64_t)s * K * ny + j;
  for (int k = threadIdx.x; k < K; k += 256) rc[k] = ch[k * ny];
  __syncthreads();
  const int i0 = 4 * threadIdx.x;
  if (i0 >= nx) return;
  uint32_t m = 0;  // bit e: pixel i0 + e is covered
  for (int k = 0; k < K; ++k) {
    const int2 c = rc[k];
#pragma unroll
    for (int e = 0; e < 4; ++e)
      m |= (c.x <= i0 + e && i0 + e <= c.y) ? 1u << e : 0u;
  }
  uint8_t *dst = cov + (int64_t)row * nx + i0;
  if (nx % 4 == 0) {  // the word is inside the row and 4-byte aligned
    *reinterpret_cast<uint32_t *>(dst) =
        (m & 1u) | ((m & 2u) << 7) | ((m & 4u) << 14) | ((m & 8u) << 21);
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (i0 + e < nx) dst[e] = (m >> e) & 1u;
  }
}

// One block per (tile, slice).  The slice's chords (K*ny pairs) are staged
// in LDS when they fit (kLds), else read through the cache from global
// memory; the disks' bounding boxes always live in LDS.  Blocks of 16
// waves: two share a CU's waves at 33 KB of LDS each for 8 humans x 512
// rows (blocks of 4 waves would be limited to 16 waves per CU by LDS),
// and the per-pixel row scans are chains of LDS round trips.
constexpr int kPlaneThreads = 1024;
template <bool kLds>
__global__ __launch_bounds__(kPlaneThreads) void k_planes(
    const int2 *__restrict__ chords, Centres C, int K, int nx, int ny,
    int tiles, const int32_t *__restrict__ F1,
    const int32_t *__restrict__ need, int32_t *__restrict__ P) {
  extern __shared__ int4 sh4[];
  const int s = blockIdx.x / tiles;
  const int tile = blockIdx.x - s * tiles;
  if (need && need[s] == 0) return;  // uniform over the block
  const int64_t R = radius_of(C, s);
  const int2 *gch = chords + (int64_t)s * K * ny;
  int4 *box = sh4;                                   // K boxes
  int2 *lch = reinterpret_cast<int2 *>(sh4 + K);     // K*ny chords
  if (kLds)
    for (int t = threadIdx.x; t < K * ny; t += kPlaneThreads) lch[t] = gch[t];
  for (int k = threadIdx.x; k < K; k += kPlaneThreads) {
    const int64_t X = centre_word(C, 2 * ((int64_t)s * K + k));
    const int64_t Y = centre_word(C, 2 * ((int64_t)s * K + k) + 1);
    const int4 b = disk_box(X, Y, R, nx, ny);
    box[k] = b;
  }
  __syncthreads();
  typename std::conditional<kLds, LdsTab, GlobalTab>::type ch{kLds ? lch
                                                                   : gch};

  const int npx = nx * ny;
  for (int p = tile * kPlaneThreads + threadIdx.x; p < npx;
       p += tiles * kPlaneThreads) {
    const int j = p / nx;
    const int i = p - j * nx;
    const int32_t out = plane_value(ch, box, F1 + (int64_t)s * npx + i, K, nx,
                                    ny, i, j);
    P[(int64_t)s * npx + p] = out;
  }
}

// Tile blockIdx.x of slice blockIdx.y (+ 65535 blockIdx.z).
template <int G>
__global__ __launch_bounds__(64 * kTileWaves) void k_plane_tiles(
    Centres C, int K, int rows, int nx, int ny, int n_slices,
    const int32_t *__restrict__ need, int32_t *__restrict__ P) {
  extern __shared__ int4 sh4[];
  const int s = blockIdx.z * 65535 + blockIdx.y;
  if (s >= n_slices || (need && need[s] == 0)) return;  // uniform
  const int64_t at = 2 * (int64_t)s * K;
  plane_tile<G>(sh4, K, rows, radius_of(C, s), nx, ny, blockIdx.x,
                [&](int q) { return centre_word(C, at + q); },
                P + (int64_t)s * nx * ny);
}

static int launch_chords(Handle *h, const Centres &C, int K, int2 *chords,
                         int nx, int ny, int n_slices, const int32_t *need,
                         hipStream_t s) {
  const int64_t total = (int64_t)n_slices * K * ny;
  if (total <= 0) return PCSDF_OK;
  launch_timed(h, k_chords, dim3((unsigned)((total + 255) / 256)), dim3(256),
               0u, s, C, K, nx, ny, total, need, chords);
  return check_launch(h, "chords");
}

int launch_planes(Handle *h, const Centres &C, int K, bool empty,
                  int64_t max_R, int2 *chords, int32_t *P, int nx, int ny,
                  int n_slices, const int32_t *need, hipStream_t s) {
  const int Keff = empty ? 0 : K;
  const int rows = disk_rows(max_R, ny);
  const int64_t lds = tile_lds(Keff, rows);
  // a stack with a workgroup of column segments (64 columns of a slice) per
  // CU, in columns whose envelopes stay in LDS (16-bit entries), of planes no
  // wider than a grid: k_cover, the row pass and the entries' 10-bit roots
  // end at 1024 columns, and a template's window may have more
  const bool stack = !need && Keff > 0 && ny <= 512 && nx <= kMaxDim &&
                     h->tuning.static_segments == 0 &&
                     (int64_t)((nx + 63) / 64) * n_slices >= 256;
  // such a stack of planes wider than a tile whose disks' boxes together
  // cover them: nearly every wave holds covered pixels, many deep (100 x 100,
  // 8 disks of 42 rows, 130, 200 and 400 slices 150, 206, 349 us a call by
  // tiles, 140, 179, 293 by the column passes; 300 x 50 x 100, 20 of 32
  // rows, 167, 108; but 64 x 64 x 260, 8 of 41, 101, 117)
  const bool dense = stack && nx > kTileCols &&
                     (int64_t)Keff * rows * rows >= (int64_t)nx * ny;
  const bool deep =
      (int64_t)Keff * rows * rows * rows >= kTileDepth * nx * ny;
  if (nx <= kTilePlaneMax && ny <= kTilePlaneMax && rows <= kTileMaxRows &&
      (int64_t)Keff * rows <= (stack ? kTileChordsStack : kTileChords) &&
      lds <= kTileLds && !dense && !deep) {
    auto go = [&](auto kernel, int G) {
      launch_timed(h, kernel,
                   dim3((unsigned)plane_tiles(nx, ny, G),
                        (unsigned)std::min(n_slices, 65535),
                        (unsigned)((n_slices + 65534) / 65535)),
                   dim3(64 * kTileWaves), (uint32_t)lds, s, C, Keff, rows, nx,
                   ny, n_slices, need, P);
      return check_launch(h, "plane_tiles");
    };
    if ((int64_t)plane_tiles(nx, ny) * n_slices <= kTileFew)
      return go(&k_plane_tiles<2>, 2);
    // a crowd: the disks' boxes together cover two fifths of the plane
    if (5LL * Keff * rows * rows >= 2LL * nx * ny)
      return go(&k_plane_tiles<4>, 4);
    return go(&k_plane_tiles<kTileRows>, kTileRows);
  }
  int rc0 = launch_chords(h, C, Keff, chords, nx, ny, n_slices, need, s);
  if (rc0) return rc0;
  const int npx = nx * ny;
  int32_t *F1 = P + (int64_t)n_slices * npx;
  const int64_t npix = (int64_t)n_slices * npx;
  if (stack) {
    // Every slice of a large stack: the planar field is the 2-D signed EDT
    // of the disks' coverage, by the static build's row pass and y column
    // pass over the stack of slices (each slice a z layer of an
    // nx x ny x n grid).  The coverage bytes use the front of P, the row
    // pass's output the back.  With the default segment counts (a static
    // build tuning sends the planes to the per-pixel kernel) no workspace
    // is allocated.
    uint8_t *cov = reinterpret_cast<uint8_t *>(P);
    launch_timed(h, k_cover, dim3((unsigned)(npix / nx)), dim3(256), 0u, s,
                 chords, Keff, nx, ny, cov);
    int rc = check_launch(h, "cover");
    if (!rc) rc = launch_pass_x_u8(h, cov, F1, nx, (int64_t)n_slices * ny, s);
    if (!rc)
      rc = launch_pass_col(h, F1, P, nullptr, 1.0f, nx, n_slices, ny, nx,
                           (int64_t)npx, true, false, s);
    return rc;
  }
  if (Keff > 0) {
    const int bpr = (nx + 255) / 256;
    launch_timed(h, k_rowfree, dim3((unsigned)(npix / nx * bpr)), dim3(256),
                 0, s, chords, Keff, nx, ny, bpr, need, F1);
    int rc = check_launch(h, "rowfree");
    if (rc) return rc;
  }
  int tiles = (512 + n_slices - 1) / n_slices;
  const int maxt = (npx + kPlaneThreads - 1) / kPlaneThreads;
  if (tiles > maxt) tiles = maxt;
  if (tiles < 1) tiles = 1;
  const size_t box_bytes = (size_t)Keff * sizeof(int4);
  const size_t ch_bytes = (size_t)Keff * ny * sizeof(int2);
  const bool use_lds = box_bytes + ch_bytes <= 48 * 1024;
  const dim3 grid((unsigned)((int64_t)tiles * n_slices)),
      block(kPlaneThreads);
  if (use_lds)
    launch_timed(h, k_planes<true>, grid, block,
                 (uint32_t)(box_bytes + ch_bytes), s, chords, C, Keff, nx, ny,
                 tiles, F1, need, P);
  else
    launch_timed(h, k_planes<false>, grid, block, (uint32_t)box_bytes, s,
                 chords, C, Keff, nx, ny, tiles, F1, need, P);
  return check_launch(h, "planes");
}

}  // namespace pcsdf
