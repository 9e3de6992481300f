// Prints the composite items that the batch planner gives one scene, of the
// fields asked for: nx ny nz n_slices ssq sdf.  Test infrastructure only.
#define main harness_main
#include "harness.cpp"
#undef main

int main(int argc, char **argv) {
  if (argc != 7) return 2;
  int a[6];
  for (int q = 0; q < 6; ++q) a[q] = atoi(argv[q + 1]);
  // addresses on a cache line, not accessed
  alignas(128) static int32_t line[32];
  pcsdf_scene sc = {};
  sc.grid.nx = a[0];
  sc.grid.ny = a[1];
  sc.grid.nz = a[2];
  sc.grid.voxel_m = 0.05;
  sc.static_ssq_dev = line;
  sc.n_slices = a[3];
  sc.radius_m = 0.2;
  sc.height_m = 1.0;
  sc.out_ssq_dev = a[4] ? line : nullptr;
  sc.out_sdf_dev = a[5] ? reinterpret_cast<float *>(line) : nullptr;
  Handle h;
  BatchPlan bp;
  if (plan_batch(&h, 1, &sc, pcsdf_tuning{}, 1, &bp)) return 1;
  printf("%u\n", bp.composite_items);
  return 0;
}
