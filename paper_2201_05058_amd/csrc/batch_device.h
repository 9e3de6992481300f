// Device side of the batched composite (see batch.hip): scene table entry,
// planar-field item, composite chunk and the worker loops.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "composite_device.h"
#include "device_common.h"
#include "plane_tile.h"

namespace pcsdf {

struct SceneDev {
  const int32_t *S;
  int32_t *oc;
  float *of;
  const int64_t *xy;  // [n][K][2] fixed-point centres
  int2 *chords;       // [n][K][ny] (used when the table exceeds LDS)
  int32_t *P;         // [n][ny][nx] planar fields
  int32_t *F1;        // [n][ny][nx] row pass of the free set
  int64_t R;
  uint32_t V;
  int nx, ny, nz, n, K, Kt, has_above;
  int aligned;  // every composite pack is aligned (packs_aligned)
  float hf;
  uint32_t item0;   // first composite item of the scene
  uint32_t items;   // its composite items: slice groups x voxel chunks
  uint32_t span;    // slice groups per span of items
  uint32_t octet;   // log2 of the chunks that run together, 3 or less
  int fold;         // an item holds this many times the plan's slices
  FastDiv plane;    // nx ny
  FastDiv per_span, per_oct;  // items per span, per 2^octet chunks in one
};

// Composite items are numbered scene by scene, each scene's count padded
// to a multiple of kItemGroup, so that one table entry per kItemGroup
// items names the scene (padding items do nothing).
constexpr int kItemGroupShift = 6;
constexpr int kItemGroup = 1 << kItemGroupShift;

// One scene-table entry, read field by field through the constant address
// space: the compiler takes a pointer loaded from there to be global, so
// every access through it is a global instruction rather than a flat one
// (a wait for a flat access cannot be counted in order and so waits for
// all outstanding loads and stores).  A whole-struct copy would lose the
// address space.
template <class T>
__device__ __forceinline__ void load_div(FastDiv *d, T *c) {
  d->d = c->d;
  d->m = c->m;
  d->s1 = c->s1;
  d->s2 = c->s2;
}
__device__ __forceinline__ SceneDev load_scene(const SceneDev *scenes, int q) {
#if defined(__clang__)
  typedef __attribute__((address_space(4))) const SceneDev ConstScene;
#else  // a host compiler building the device code for CPU tests
  typedef const SceneDev ConstScene;
#endif
  ConstScene *c = (ConstScene *)(scenes + q);
  SceneDev d;
  d.S = c->S;
  d.oc = c->oc;
  d.of = c->of;
  d.xy = c->xy;
  d.chords = c->chords;
  d.P = c->P;
  d.F1 = c->F1;
  d.R = c->R;
  d.V = c->V;
  d.nx = c->nx;
  d.ny = c->ny;
  d.nz = c->nz;
  d.n = c->n;
  d.K = c->K;
  d.Kt = c->Kt;
  d.has_above = c->has_above;
  d.aligned = c->aligned;
  d.hf = c->hf;
  d.item0 = c->item0;
  d.items = c->items;
  d.span = c->span;
  d.octet = c->octet;
  d.fold = c->fold;
  load_div(&d.plane, &c->plane);
  load_div(&d.per_span, &c->per_span);
  load_div(&d.per_oct, &c->per_oct);
  return d;
}

constexpr int kItemPlane = 0;

// Whether a scene's planar items are tiles with the slice's disks in LDS.
// The single call's limits on rows and chords (planes.hip) do not apply: what
// it falls back to is not at hand here, and beside the items of one pixel per
// lane with the chords in LDS, or of a whole slice without, tiles win at any
// disks.  Us a batch of 16 rooms of about 200 x 200 x 64 x 20 slices, those
// items and tiles: 8 disks of 81 rows 10990, 1802, 4 of 201 rows 14238, 3329,
// 26 of 41 22767, 1598, 128 of 27 28276, 2988; 1 of 61 1174, 1087.
__host__ __device__ inline bool planes_tiled(int K, int64_t R, int ny,
                                             int lds_cap) {
  return tile_lds(K, disk_rows(R, ny)) <= lds_cap;
}

// ------------------------------------------------------------ device side

// Planar field of slice s: one tile of it (plane_tile.h), or, when the
// slice's chords exceed the LDS, the whole slice with the chords and the
// row pass in global memory.
__device__ inline void plane_item(const SceneDev &sc, int s, int tile,
                                  int4 *lds, int lds_cap) {
  const int K = sc.K, nx = sc.nx, ny = sc.ny;
  const int npx = nx * ny;
  const int64_t *xy = sc.xy + (int64_t)s * K * 2;
  if (planes_tiled(K, sc.R, ny, lds_cap)) {
    plane_tile(lds, K, disk_rows(sc.R, ny), sc.R, nx, ny, tile,
               [&](int q) { return xy[q]; }, sc.P + (int64_t)s * npx);
    return;
  }
  int4 *box = lds;
  int2 *gch = sc.chords + (int64_t)s * K * ny;
  for (int t = threadIdx.x; t < K; t += blockDim.x)
    box[t] = disk_box(xy[2 * t], xy[2 * t + 1], sc.R, nx, ny);
  for (int t = threadIdx.x; t < K * ny; t += blockDim.x) {
    const int k = t / ny, j = t - k * ny;
    gch[t] = disk_chord(xy[2 * k], xy[2 * k + 1], sc.R, nx, j);
  }
  __threadfence();
  __syncthreads();
  int32_t *f1 = sc.F1 + (int64_t)s * npx;
  int32_t *P = sc.P + (int64_t)s * npx;
  {
    const GlobalTab ch{gch};
    for (int p = threadIdx.x; p < npx; p += blockDim.x) {
      const int j = p / nx, i = p - j * nx;
      f1[p] = row_free_dist(ch, K, ny, nx, j, i);
    }
    __threadfence();
    __syncthreads();
    for (int p = threadIdx.x; p < npx; p += blockDim.x) {
      const int j = p / nx, i = p - j * nx;
      P[p] = plane_value(ch, box, f1 + i, K, nx, ny, i, j);
    }
  }
}

// Composite of `count` consecutive voxels from v0 (four per lane) for slices
// [s0, s1); v0 is a multiple of the chunk size, itself a multiple of 4.
// Each lane runs the same epilogue as the single-scene kernel; with the
// tuned chunk of 256 lanes x 4 voxels a lane handles one pack and exits.
// (A loop that loads the next step's data ahead of the current stores was
// measured slower for these short item lengths, and persistent grids
// slower than one workgroup per item.)
template <bool kAligned, bool kSsq, bool kSdf>
__device__ inline void composite_chunk(const SceneDev &sc, uint32_t v0,
                                       uint32_t count, int s0, int s1) {
  const uint32_t end = min(pack_span(sc.V, kAligned), v0 + count);
  for (uint32_t v = v0 + threadIdx.x * 4; v < end; v += blockDim.x * 4) {
    if (kAligned)
      composite_pack<kSsq, kSdf>(sc.S, sc.P, nullptr, sc.oc, sc.of, sc.plane,
                                 sc.V, v, s0, s1, sc.Kt, sc.has_above, sc.hf);
    else
      composite_pack_shifted<kSsq, kSdf>(sc.S, sc.P, nullptr, sc.oc, sc.of,
                                         sc.plane, sc.V, v, s0, s1, sc.Kt,
                                         sc.has_above, sc.hf);
  }
}

template <bool kAligned>
__device__ inline void composite_chunk_any(const SceneDev &sc, uint32_t v0,
                                           uint32_t count, int s0, int s1) {
  if (sc.oc && sc.of)
    composite_chunk<kAligned, true, true>(sc, v0, count, s0, s1);
  else if (sc.oc)
    composite_chunk<kAligned, true, false>(sc, v0, count, s0, s1);
  else
    composite_chunk<kAligned, false, true>(sc, v0, count, s0, s1);
}

// Workers.  A grid strides over a list of work items; nothing waits on
// anything, so every workgroup runs a bounded number of bounded items.
// The planar items of a batch are run by one launch and its composite
// items by the next on the same stream, so stream order is the only
// dependency between them.
__device__ inline void batch_planes(const SceneDev *__restrict__ scenes,
                                    const int4 *__restrict__ items,
                                    int n_items, int lds_cap, int4 *lds) {
  for (int it = blockIdx.x; it < n_items; it += gridDim.x) {
    const int4 w = items[it];
    plane_item(load_scene(scenes, w.y), w.z, w.w, lds, lds_cap);
    __syncthreads();  // the next item reuses the LDS
  }
}

// Composite item `it` belongs to scene q = scene_of[it / kItemGroup]; its
// number within the scene, it - item0 (item0 is a multiple of eight), counts
// spans, octets of chunks (2, 4 or one where the scene has no eight), the
// span's slice groups and the octet's chunks, the last fastest (the order of
// slices_per_span's comment); it is padding when it - item0 >= items.
__device__ inline void batch_composites(const SceneDev *__restrict__ scenes,
                                        const int32_t *__restrict__ scene_of,
                                        uint32_t total, int G,
                                        uint32_t chunk_voxels) {
  for (uint32_t it = blockIdx.x; it < total; it += gridDim.x) {
    const SceneDev sc = load_scene(scenes, scene_of[it >> kItemGroupShift]);
    const uint32_t local = it - sc.item0;
    if (local >= sc.items) continue;
    const uint32_t sp = quotient(local, sc.per_span);
    const uint32_t in_span = local - sp * sc.per_span.d;
    const uint32_t oct = quotient(in_span, sc.per_oct);
    const uint32_t in_oct = in_span - oct * sc.per_oct.d;
    const uint32_t group = in_oct >> sc.octet;
    const uint32_t v0 =
        ((oct << sc.octet) + in_oct - (group << sc.octet)) * chunk_voxels;
    const int slices = G * sc.fold;
    const int s0 = (int)((sp * sc.span + group) * (uint32_t)slices);
    const int s1 = min(sc.n, s0 + slices);
    if (s0 >= s1 || v0 >= pack_span(sc.V, sc.aligned)) continue;
    if (sc.aligned)
      composite_chunk_any<true>(sc, v0, chunk_voxels, s0, s1);
    else
      composite_chunk_any<false>(sc, v0, chunk_voxels, s0, s1);
  }
}

}  // namespace pcsdf
