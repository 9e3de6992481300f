// Predicted composite fields: one exact signed field of the humans per
// time slice, min-composited with the environment field (mapping section:
// a parallel min between the environment field and the humans' fields at
// their predicted positions; RHAP-GPMP2 section: a sequence of n such
// fields, one per slice).
//
// The humans are vertical cylinders sharing one radius and height, all
// standing on the grid's floor, so a slice's human voxels form a product
// set O_h = D x Z: D is the union of voxelised disks in the xy plane and
// Z = {0..Kt} the voxel layers whose centres lie under the cylinder top.
// The squared distance to a product set splits into one term per factor,
// so for every voxel (i, j, k):
//   outside:  E_{O_h}(i,j,k)    = E_D(i,j) + max(0, k - Kt)^2
//   inside:   E_{G\O_h}(i,j,k)  = min(E_{Gxy\D}(i,j), (Kt + 1 - k)^2)
// (the complement of D x Z in the grid is (Gxy\D) x Gz  union  Gxy x (Gz\Z),
// and the second term is absent when Z reaches the grid top).  This is
// the z pass of the separable EDT done in closed form: the column input
// is constant on 0..Kt and empty elsewhere, and its lower envelope is that
// constant plus the squared distance to the interval.  So the exact 3-D
// field of the humans needs only a 2-D signed EDT per slice (planes.hip:
// each disk's chord per row from an exact integer square root of the
// voxelisation predicate, a row pass giving every pixel's distance to the
// nearest pixel outside the disks, and a bounded per-pixel search over
// rows for both signs), and the per-voxel work is a streaming epilogue:
//   read the static field once, then for every slice compute the humans'
//   value from the slice's plane, take the signed min, convert to metres
//   and write both outputs.
// The epilogue moves the compulsory bytes only: 4 B of static field per
// voxel (read once for all slices) and 8 B per voxel-slice of output; the
// planes (nx*ny*4 B per slice) stay in cache.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>
#include <vector>

#include "composite_device.h"
#include "device_common.h"
#include "internal.h"

namespace pcsdf {

// The 16-bit copy of the static field: S16[v] = S[v] where |S[v]| <=
// 32767, else kS16Far.  Thread t converts voxels 4t .. 4t+3 (S16 is
// 256-byte aligned; S is read in 16-byte packs when it is so aligned).
__global__ __launch_bounds__(256) void k_static16(
    const int32_t *__restrict__ S, int16_t *__restrict__ S16, uint32_t V) {
  const uint32_t v = (blockIdx.x * 256u + threadIdx.x) * 4u;
  if (v >= V) return;
  auto c16 = [](int32_t x) -> uint32_t {
    return (uint32_t)(uint16_t)(x >= -32767 && x <= 32767 ? x : kS16Far);
  };
  if (v + 3 < V && !((uintptr_t)S & 15)) {
    const pk_i32x4 x = ld_global(reinterpret_cast<const pk_i32x4 *>(S + v));
    pk_i32x2 w;
    w[0] = (int32_t)(c16(x[0]) | c16(x[1]) << 16);
    w[1] = (int32_t)(c16(x[2]) | c16(x[3]) << 16);
    *reinterpret_cast<pk_i32x2 *>(S16 + v) = w;
  } else {
    for (uint32_t e = v; e < V && e < v + 4; ++e) S16[e] = (int16_t)c16(S[e]);
  }
}

// Slices with need[sl] == 0 are skipped when `need` is non-null.  Thread g
// handles the packs at voxel 4 g (composite_pack, or with !kAligned
// composite_pack_shifted); with S16 the static values come from the 16-bit
// copy.
template <bool kAligned, bool kSsq, bool kSdf>
__global__ __launch_bounds__(256) void k_composite(
    const int32_t *__restrict__ S, const int32_t *__restrict__ P,
    const int32_t *__restrict__ need,
    int32_t *__restrict__ oc, float *__restrict__ of, FastDiv plane,
    int n_slices, int G, int Kt, int has_above, float hf, uint32_t V,
    FastDiv parts, const int16_t *__restrict__ S16) {
  // The order of slices_per_span's comment: blockIdx.x is the XCD plus eight
  // times the slice group within its span, y the chunk's octet, z the span
  // (times the parts of the octets where y holds too few, `parts`).
  const uint32_t sp = quotient(blockIdx.z, parts);
  const uint32_t oct =
      blockIdx.y + gridDim.y * (blockIdx.z - sp * parts.d);
  const uint32_t chunk = oct * 8 + (blockIdx.x & 7);
  const uint32_t v0 = (chunk * 256u + threadIdx.x) * 4;
  if (v0 >= pack_span(V, kAligned)) return;
  const int s_begin = (int)(sp * (gridDim.x >> 3) + (blockIdx.x >> 3)) * G;
  const int s_end = min(n_slices, s_begin + G);
  if (s_begin >= s_end) return;
  if (need) {  // skip the static read when none of the block's slices is due
    bool any = false;
    for (int sl = s_begin; sl < s_end; ++sl) any = any || need[sl] != 0;
    if (!any) return;
  }
#define PCSDF_PACK(fn, kNeed, copy)                                       \
  fn<kSsq, kSdf, kNeed>(S, P, need, oc, of, plane, V, v0, s_begin, s_end, \
                        Kt, has_above, hf, copy)
  if constexpr (kAligned) {
    if (need)
      PCSDF_PACK(composite_pack, true, nullptr);
    else
      PCSDF_PACK(composite_pack, false, S16);
  } else {
    if (need)
      PCSDF_PACK(composite_pack_shifted, true, nullptr);
    else
      PCSDF_PACK(composite_pack_shifted, false, S16);
  }
#undef PCSDF_PACK
}

template <bool kAligned>
static void launch_comp(Handle *h, const int32_t *S, const int32_t *P,
                        const int32_t *need, int32_t *oc, float *of,
                        uint32_t plane, int n, int G, int span, int Kt,
                        int has_above, float hf, uint32_t V,
                        const int16_t *S16, hipStream_t s) {
  const uint32_t nthreads = (pack_span(V, kAligned) + 3) / 4;
  const uint32_t octets = ((nthreads + 255) / 256 + 7) / 8;
  const int groups = (n + G - 1) / G;
  const uint32_t parts = (octets + 65534) / 65535;
  const dim3 grid(8 * (uint32_t)span, (octets + parts - 1) / parts,
                  (unsigned)((groups + span - 1) / span) * parts);
  const dim3 block(256);
  const FastDiv pd = fast_div(plane);
  if (oc && of)
    launch_timed(h, k_composite<kAligned, true, true>, grid, block, 0u, s, S,
                 P, need, oc, of, pd, n, G, Kt, has_above, hf, V, fast_div(parts),
                 S16);
  else if (oc)
    launch_timed(h, k_composite<kAligned, true, false>, grid, block, 0u, s, S,
                 P, need, oc, of, pd, n, G, Kt, has_above, hf, V, fast_div(parts),
                 S16);
  else
    launch_timed(h, k_composite<kAligned, false, true>, grid, block, 0u, s, S,
                 P, need, oc, of, pd, n, G, Kt, has_above, hf, V, fast_div(parts),
                 S16);
}

// Fixed-point conversion of a coordinate to the 2^-16 voxel lattice:
// rint(((p - o)/h) * 2^16), each step an IEEE fp64 operation.
static bool to_fixed(double p, double o, double h, int64_t *out) {
  double t = p - o;
  t = t / h;
  t = t * 65536.0;
  if (!std::isfinite(t) || std::fabs(t) >= 4611686018427387904.0) return false;
  *out = (int64_t)std::nearbyint(t);
  return true;
}

// Validates the humans of every slice and converts them to the fixed-point
// lattice: words [0, 2 n_slices n_humans) are the centres, then one radius
// per slice.  `w` must hold humans_words() values.
static size_t humans_words(int32_t n_slices, int32_t n_humans) {
  return 2 * (size_t)n_slices * (size_t)n_humans + (size_t)n_slices;
}

static int humans_fixed(Handle *h, const pcsdf_grid *g, int32_t n_slices,
                        int32_t n_humans, const double *human_xy_host,
                        double radius_m, const double *radius_per_slice,
                        double height_m, int64_t *w, int *Kt_out) {
  const double hv = g->voxel_m;
  if (!std::isfinite(height_m) || height_m < 0)
    return fail(h, PCSDF_ERR_NUMERIC, "height_m must be finite, >= 0");
  int64_t Hq;
  if (!to_fixed(height_m, 0.0, hv, &Hq))
    return fail(h, PCSDF_ERR_NUMERIC, "height out of range");
  const size_t ncent = (size_t)n_slices * n_humans;
  // Fixed-point radius of every slice.
  for (int32_t j = 0; j < n_slices; ++j) {
    const double r = radius_per_slice ? radius_per_slice[j] : radius_m;
    if (!std::isfinite(r) || r < 0)
      return fail(h, PCSDF_ERR_NUMERIC, "radius must be finite, >= 0");
    int64_t R;
    if (!to_fixed(r, 0.0, hv, &R))
      return fail(h, PCSDF_ERR_NUMERIC, "radius out of range");
    if (R >= (1LL << 31))
      return fail(h, PCSDF_ERR_NUMERIC, "radius/voxel_m must be < 32768");
    w[2 * ncent + j] = R;
  }
  // Highest layer whose centre lies at or under the cylinder top.
  *Kt_out = Hq >= 32768
                ? (int)std::min<int64_t>((Hq - 32768) / 65536, g->nz - 1)
                : -1;
  // Fixed-point centres, validated on the host before anything is queued.
  for (size_t t = 0; t < ncent; ++t) {
    if (!to_fixed(human_xy_host[2 * t], g->origin_m[0], hv, &w[2 * t]) ||
        !to_fixed(human_xy_host[2 * t + 1], g->origin_m[1], hv,
                  &w[2 * t + 1]))
      return fail(h, PCSDF_ERR_NUMERIC,
                  "human position non-finite or out of range at index " +
                      std::to_string(t));
  }
  return PCSDF_OK;
}

static int check_human_args(Handle *h, int32_t n_slices, int32_t n_humans,
                            const double *human_xy_host) {
  if (n_slices < 1)
    return fail(h, PCSDF_ERR_INVALID_ARG, "n_slices must be >= 1");
  if (n_humans < 0 || n_humans > kMaxHumans)
    return fail(h, PCSDF_ERR_INVALID_ARG, "n_humans must be in [0, 256]");
  if (n_humans > 0 && !human_xy_host)
    return fail(h, PCSDF_ERR_INVALID_ARG, "human_xy_host is required");
  return PCSDF_OK;
}

int humans_upload(Handle *h, const pcsdf_grid *g, int32_t n_slices,
                  int32_t n_humans, const double *human_xy_host,
                  double radius_m, const double *radius_per_slice,
                  double height_m, hipStream_t s, HumanSet *out) {
  int rc = check_human_args(h, n_slices, n_humans, human_xy_host);
  if (rc) return rc;
  const int ny = g->ny;
  const size_t ncent = (size_t)n_slices * n_humans;
  std::vector<int64_t> &xy = h->host_xy;
  xy.resize(humans_words(n_slices, n_humans));
  int Kt;
  if ((rc = humans_fixed(h, g, n_slices, n_humans, human_xy_host, radius_m,
                         radius_per_slice, height_m, xy.data(), &Kt)))
    return rc;
  const bool empty = Kt < 0 || n_humans == 0;
  if ((rc = bind_device(h))) return rc;
  const size_t xy_bytes = xy.size() * sizeof(int64_t);
  const size_t chord_bytes =
      (size_t)n_slices * (n_humans > 0 ? n_humans : 1) * ny * sizeof(int2);
  if ((rc = ensure_buffer(h, h->chord_buf, chord_bytes, s))) return rc;
  if (xy.size() <= (size_t)kCentresInArgs) {
    // small sets travel in the planar kernels' arguments
    out->C.xy = nullptr;
    out->C.Rs = nullptr;
    out->C.rs_off = (int32_t)(2 * ncent);
    std::memcpy(out->C.w, xy.data(), xy_bytes);
  } else {
    if ((rc = ensure_buffer(h, h->param_buf, xy_bytes, s))) return rc;
    int64_t *xy_dev = reinterpret_cast<int64_t *>(h->param_buf.ptr);
    if ((rc = acquire_staging(h, xy_bytes))) return rc;
    std::memcpy(h->pinned, xy.data(), xy_bytes);
    if (hipMemcpyAsync(xy_dev, h->pinned, xy_bytes, hipMemcpyHostToDevice,
                       s) != hipSuccess)
      return fail(h, PCSDF_ERR_HIP, "upload of human positions failed");
    if ((rc = release_staging(h, s))) return rc;
    out->C.xy = xy_dev;
    out->C.Rs = xy_dev + 2 * ncent;
  }
  out->max_R = *std::max_element(xy.begin() + 2 * ncent, xy.end());
  out->chords = reinterpret_cast<int2 *>(h->chord_buf.ptr);
  out->K = empty ? 0 : n_humans;
  out->Kt = empty ? -1 : Kt;
  out->has_above = out->Kt + 1 <= g->nz - 1;
  return PCSDF_OK;
}

int planes_from(Handle *h, const pcsdf_grid *g, const HumanSet &hs,
                int32_t n_slices, int32_t n_humans, const int32_t *need,
                hipStream_t s, PlaneSet *out) {
  const int nx = g->nx, ny = g->ny;
  const size_t plane_bytes = (size_t)n_slices * nx * ny * sizeof(int32_t);
  int rc;
  if ((rc = ensure_buffer(h, h->plane_buf, 2 * plane_bytes, s))) return rc;
  int32_t *p2 = reinterpret_cast<int32_t *>(h->plane_buf.ptr);
  // Planar signed field of the disk union, per slice.
  ProfScope pp(h, PCSDF_KERNEL_PLANES, s, true);
  if ((rc = launch_planes(h, hs.C, n_humans, hs.K == 0, hs.max_R, hs.chords,
                          p2, nx, ny, n_slices, need, s)))
    return rc;
  out->P = p2;
  out->Kt = hs.Kt;
  out->has_above = hs.has_above;
  return PCSDF_OK;
}

int planes_run(Handle *h, const pcsdf_grid *g, int32_t n_slices,
               int32_t n_humans, const double *human_xy_host, double radius_m,
               const double *radius_per_slice, double height_m,
               const int32_t *need, hipStream_t s, PlaneSet *out) {
  HumanSet hs;
  int rc = humans_upload(h, g, n_slices, n_humans, human_xy_host, radius_m,
                         radius_per_slice, height_m, s, &hs);
  if (rc) return rc;
  return planes_from(h, g, hs, n_slices, n_humans, need, s, out);
}

int composite_run(Handle *h, const pcsdf_grid *g,
                  const int32_t *static_ssq_dev, int32_t n_slices,
                  int32_t n_humans, const double *human_xy_host,
                  double radius_m, const double *radius_per_slice,
                  double height_m, int32_t *out_ssq_dev, float *out_sdf_dev,
                  const int32_t *need, hipStream_t s) {
  int rc = check_grid(h, g);
  if (rc) return rc;
  if (!static_ssq_dev)
    return fail(h, PCSDF_ERR_INVALID_ARG, "static_ssq_dev is required");
  if (!out_ssq_dev && !out_sdf_dev)
    return fail(h, PCSDF_ERR_INVALID_ARG,
                "at least one of out_ssq_dev / out_sdf_dev is required");
  if (((uintptr_t)static_ssq_dev & 3) || ((uintptr_t)out_ssq_dev & 3) ||
      ((uintptr_t)out_sdf_dev & 3))
    return fail(h, PCSDF_ERR_ALIGN, "device buffers must be 4-byte aligned");
  PlaneSet ps_;
  if ((rc = planes_run(h, g, n_slices, n_humans, human_xy_host, radius_m,
                       radius_per_slice, height_m, need, s, &ps_)))
    return rc;
  ProfScope ps(h, PCSDF_KERNEL_COMPOSITE, s, true);
  return launch_composite(h, g, static_ssq_dev, ps_.P, need, ps_.Kt,
                          ps_.has_above, n_slices, out_ssq_dev, out_sdf_dev,
                          s, true);
}

// Grids beyond the caches.  The 256 MiB Infinity Cache holds the static field
// up to about kLargeVoxels and its 16-bit copy up to about twice that, beside
// the outputs that stream through it, so the best shape changes within a few
// layers of the grid.  Kernel us (both fields; f the field, c the copy, then
// slices per block x groups per span; the copy's own time included):
//   voxels x slices   f1x4   c1x2   c2x1   f4x1   f6x1
//   58.7 M x 40       2978   3050   3261   3291
//   65.5 M x 40       3827   3514   3570   3680
//   71.3 M x 40       4691   3799   4037   4669   4687
//   77.6 M x 24       3797   2848   2690   3104   2861
//   83.9 M x 30       5291   4899   4150   4394   3865
//   105 M x 30        6637   7463   7012   5480   4803
//   134 M x 40       12165  13021  11499   9723   9213
//   315 M x 10        6831   7801   6885   5531   5312
// and, with packs off the lines, 75 M x 40 c1x2 4121, c2x1 3953; 109 M x 10
// f1x2 1974, f4x1 2383, c2x1 2565.  One field: 75.5 M x 40 f4x1 2844, c2x1
// 2720, c4x1 2324; 105 M x 20 2104, 2835, 2552, off the lines 127 M x 30 f2x1
// 4479, f4x1 5148.
constexpr int64_t kCopyVoxels = 5LL << 24;  // the copy up to here

// Slices per block where the tuning leaves them.  Small and middle grids: one
// slice, in the rule's spans, or two where only one field is written (a lane's
// address and layer work, not the stores, then bounds a block of one slice:
// 160 x 144 x 96 x 20 slices 31 against 36 us, 255 x 241 x 127 x 20 119
// against 153, with both fields 57 and 56, 270 and 248).
static int block_slices(int64_t V, bool both, bool aligned, bool may_copy) {
  if (V <= kSpanVoxels) return both ? 1 : V < kLargeVoxels ? 2 : 4;
  if (V <= kCopyVoxels && may_copy) return both ? 2 : 4;
  if (!aligned) return both ? 1 : 2;
  return both ? 6 : 4;
}

// Whether the packs read the 16-bit static copy: the tuning's choice, else
// where the field exceeds the caches and the copy does not.  The copy costs 6
// B per voxel once (66 us at 67 M voxels) and saves 2 B per voxel and slice
// group, little where some of the field stays cached (65.5 M voxels: x 10
// slices c1x2 961, f1x2 910; x 24 2153, 2202; one field x 20 c4x1 945, f4x1
// 936, x 40 1766, 1930) and much beyond (73.4 M x 12 c2x1 1297, f2x1 1585).
// Where the tuning has the groups apart (order 0) nothing of the field stays
// cached between them (65.5 M x 40, three slices 3585, 3758), and single
// slices read it that often from 2^25 voxels on (50 M x 40 2851, 3307).
static bool use_static16(const Handle *h, int64_t V, int G, int groups,
                         bool both) {
  const pcsdf_tuning &tu = h->tuning;
  if (tu.composite_static16 != 0) return tu.composite_static16 == 2;
  const bool apart =
      tu.composite_slices_per_block > 0 && tu.composite_order == 0;
  const int64_t least = apart && G == 1 ? 1LL << 25 : kLargeVoxels;
  return V >= least && V <= kCopyVoxels &&
         groups >= (apart || V > kSpanVoxels ? 4 : both ? 16 : 8);
}

int launch_composite(Handle *h, const pcsdf_grid *g,
                     const int32_t *static_ssq_dev, const int32_t *P,
                     const int32_t *need, int Kt, int has_above,
                     int32_t n_slices, int32_t *out_ssq_dev,
                     float *out_sdf_dev, hipStream_t s, bool static_copy) {
  const int nx = g->nx, ny = g->ny, nz = g->nz;
  const int64_t V = (int64_t)nx * ny * nz;
  // Streaming epilogue over all voxels and slices.
  const float hf = (float)g->voxel_m;
  // Slices per block and slice groups per span: the rules', or the tuning's
  // slices per block in spans of one group (order 0) or of the rule's slices
  // (order 1).
  const pcsdf_tuning &tu = h->tuning;
  const bool both = out_ssq_dev && out_sdf_dev;
  const bool aligned = packs_aligned((int64_t)nx * ny, V, static_ssq_dev,
                                     out_ssq_dev, out_sdf_dev);
  const bool may_copy =
      static_copy && !need && tu.composite_static16 != 1;
  const bool chosen = tu.composite_slices_per_block > 0;
  const int G = std::min(chosen ? tu.composite_slices_per_block
                                : block_slices(V, both, aligned, may_copy),
                         n_slices);
  const int groups = (n_slices + G - 1) / G;
  const bool copy16 = may_copy && use_static16(h, V, G, groups, both);
  int span = 1;
  if (!chosen || tu.composite_order == 1)
    span = std::max(1, (slices_per_span(V, n_slices) + G - 1) / G);
  // gridDim.z, which also holds up to 3 parts of the octets
  while ((groups + span - 1) / span > 65535 / 3) ++span;
  const uint32_t plane = (uint32_t)nx * (uint32_t)ny;
  const uint32_t Vu = (uint32_t)V;
  const int16_t *S16 = nullptr;
  if (copy16) {
    // the copy lives in the static build's intermediate buffer, which is
    // free between builds
    int rc = ensure_buffer(h, h->tmp_buf, (size_t)V * 2, s);
    if (rc) return rc;
    int16_t *c = reinterpret_cast<int16_t *>(h->tmp_buf.ptr);
    launch_timed(h, k_static16, dim3((unsigned)(((Vu + 3) / 4 + 255) / 256)),
                 dim3(256), 0u, s, static_ssq_dev, c, Vu);
    if ((rc = check_launch(h, "static16"))) return rc;
    S16 = c;
  }
  if (aligned)
    launch_comp<true>(h, static_ssq_dev, P, need, out_ssq_dev, out_sdf_dev,
                      plane, n_slices, G, span, Kt, has_above, hf, Vu, S16, s);
  else
    launch_comp<false>(h, static_ssq_dev, P, need, out_ssq_dev, out_sdf_dev,
                       plane, n_slices, G, span, Kt, has_above, hf, Vu, S16, s);
  return check_launch(h, "composite");
}

}  // namespace pcsdf

using namespace pcsdf;

extern "C" int pcsdf_predicted_composite_sdf(
    pcsdf_handle *hp, const pcsdf_grid *g, const int32_t *static_ssq_dev,
    int32_t n_slices, int32_t n_humans, const double *human_xy_host,
    double radius_m, double height_m, int32_t *out_ssq_dev,
    float *out_sdf_dev, void *stream) {
  Handle *h = reinterpret_cast<Handle *>(hp);
  if (!h) return PCSDF_ERR_INVALID_ARG;
  return composite_run(h, g, static_ssq_dev, n_slices, n_humans,
                       human_xy_host, radius_m, nullptr, height_m,
                       out_ssq_dev, out_sdf_dev, nullptr,
                       reinterpret_cast<hipStream_t>(stream));
}

extern "C" int pcsdf_predicted_composite_sdf_growing(
    pcsdf_handle *hp, const pcsdf_grid *g, const int32_t *static_ssq_dev,
    int32_t n_slices, int32_t n_humans, const double *human_xy_host,
    const double *radius_per_slice_m, double height_m, int32_t *out_ssq_dev,
    float *out_sdf_dev, void *stream) {
  Handle *h = reinterpret_cast<Handle *>(hp);
  if (!h) return PCSDF_ERR_INVALID_ARG;
  if (!radius_per_slice_m)
    return fail(h, PCSDF_ERR_INVALID_ARG, "radius_per_slice_m is required");
  return composite_run(h, g, static_ssq_dev, n_slices, n_humans,
                       human_xy_host, 0.0, radius_per_slice_m, height_m,
                       out_ssq_dev, out_sdf_dev, nullptr,
                       reinterpret_cast<hipStream_t>(stream));
}

// ---- The composite without allocation -----------------------------------
// One call's planar fields, row passes and chords live in a file-scope
// device array instead of the handle's workspace, for callers that cannot
// allocate device memory (graph capture, serving loops).  Each device the
// library runs on holds its own copy of the array until the process ends;
// every call on a device shares it, so calls that overlap on one device
// race.  Nothing in it needs to start at zero: each call writes every
// chord, row-pass value and plane pixel before it reads them.
namespace pcsdf {

constexpr size_t kNoAllocScratchBytes = (size_t)64 << 20;
constexpr int kNoAllocMaxDevices = 64;

static __device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];

static std::mutex g_scratch_mu;
static void *g_scratch_ptr[kNoAllocMaxDevices];

// The device address of `scratch` on the handle's (current) device, taken
// once per device: in host code the array's name is not a device address.
static int scratch_address(Handle *h, unsigned char **out) {
  if (h->device < 0 || h->device >= kNoAllocMaxDevices)
    return fail(h, PCSDF_ERR_INVALID_ARG,
                "device index beyond the no-allocation entry point's table");
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  void *&p = g_scratch_ptr[h->device];
  if (!p) {
    void *q = nullptr;
    const hipError_t e = hipGetSymbolAddress(&q, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !q) {
      (void)hipGetLastError();
      return fail(h, PCSDF_ERR_HIP,
                  std::string("hipGetSymbolAddress(scratch): ") +
                      hipGetErrorString(e));
    }
    p = q;
  }
  *out = static_cast<unsigned char *>(p);
  return PCSDF_OK;
}

}  // namespace pcsdf

extern "C" int pcsdf_predicted_composite_sdf_noalloc(
    pcsdf_handle *hp, const pcsdf_grid *g, const int32_t *static_ssq_dev,
    int32_t n_slices, int32_t n_humans, const double *human_xy_host,
    double radius_m, double height_m, int32_t *out_ssq_dev,
    float *out_sdf_dev, void *stream) {
  Handle *h = reinterpret_cast<Handle *>(hp);
  if (!h) return PCSDF_ERR_INVALID_ARG;
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  int rc = check_grid(h, g);
  if (rc) return rc;
  if (!static_ssq_dev)
    return fail(h, PCSDF_ERR_INVALID_ARG, "static_ssq_dev is required");
  if (!out_ssq_dev && !out_sdf_dev)
    return fail(h, PCSDF_ERR_INVALID_ARG,
                "at least one of out_ssq_dev / out_sdf_dev is required");
  if (((uintptr_t)static_ssq_dev & 3) || ((uintptr_t)out_ssq_dev & 3) ||
      ((uintptr_t)out_sdf_dev & 3))
    return fail(h, PCSDF_ERR_ALIGN, "device buffers must be 4-byte aligned");
  if ((rc = check_human_args(h, n_slices, n_humans, human_xy_host))) return rc;
  const size_t words = humans_words(n_slices, n_humans);
  if (words > (size_t)kCentresInArgs)
    return fail(h, PCSDF_ERR_INVALID_ARG,
                "no-allocation composite: 2*n_slices*n_humans + n_slices = " +
                    std::to_string(words) + " exceeds " +
                    std::to_string(kCentresInArgs));
  const int nx = g->nx, ny = g->ny;
  const size_t plane_bytes = (size_t)n_slices * nx * ny * sizeof(int32_t);
  const size_t chord_off = align_up(2 * plane_bytes, 256);
  const size_t chord_bytes =
      (size_t)n_slices * (n_humans > 0 ? n_humans : 1) * ny * sizeof(int2);
  if (chord_off + chord_bytes > kNoAllocScratchBytes)
    return fail(h, PCSDF_ERR_INVALID_ARG,
                "no-allocation composite: needs " +
                    std::to_string(chord_off + chord_bytes) +
                    " bytes of scratch (8*n_slices*nx*ny, then "
                    "8*n_slices*max(n_humans,1)*ny), the maximum is " +
                    std::to_string(kNoAllocScratchBytes));
  Centres C;
  C.xy = nullptr;
  C.Rs = nullptr;
  C.rs_off = (int32_t)(2 * (size_t)n_slices * n_humans);
  int Kt;
  if ((rc = humans_fixed(h, g, n_slices, n_humans, human_xy_host, radius_m,
                         nullptr, height_m, C.w, &Kt)))
    return rc;
  if ((rc = bind_device(h))) return rc;
  unsigned char *base;
  if ((rc = scratch_address(h, &base))) return rc;
  const bool empty = Kt < 0 || n_humans == 0;
  int32_t *P = reinterpret_cast<int32_t *>(base);
  int2 *chords = reinterpret_cast<int2 *>(base + chord_off);
  if ((rc = launch_planes(h, C, n_humans, empty,
                          *std::max_element(C.w + C.rs_off,
                                            C.w + C.rs_off + n_slices),
                          chords, P, nx, ny, n_slices, nullptr, s)))
    return rc;
  const int Kt_eff = empty ? -1 : Kt;
  return launch_composite(h, g, static_ssq_dev, P, nullptr, Kt_eff,
                          Kt_eff + 1 <= g->nz - 1, n_slices, out_ssq_dev,
                          out_sdf_dev, s);
}
