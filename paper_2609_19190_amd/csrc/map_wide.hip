// Map kernels of radius 4 and 5: the fused per-voxel body of the smaller
// radii with larger tables (one instance for both raw types).  One wavefront
// per voxel, 32 or 64 present levels; MCC problems of at most 32 levels in
// the stash for plain calls with room for it, solved in the kernel
// otherwise and for batched and served jobs.  LDS (16 to 35 KB a workgroup)
// and registers (two waves a SIMD) set the occupancy, VALU issue the rate, as
// at the smaller radii.  A PET VOI of 6,007 voxels, radius 4, Ng 32, 93 maps:
// 8.28 ms on the generic kernel (one 256-thread workgroup a voxel, tables in
// global memory), 0.44 ms here when it came in, 0.25 now.
#include "map_body.h"

namespace fr {
namespace {

template <int R, int LMAX>
hipError_t launch_w(const MapArgs& a, bool debug, hipStream_t st) {
  // the instance without a stash dumps the matrices when a.d_glcm is set
  return a.mcc && !debug ? launch_i<AnyRaw, R, LMAX, false, true>(a, st)
                         : launch_i<AnyRaw, R, LMAX, true, false>(a, st);
}

}  // namespace

hipError_t launch_map_batch_wide(const BatchJob* jobs, const DiscParams* params, const int2* items,
                                 int32_t n_items, const int32_t* items_count, int32_t vpw, int radius, int lmax,
                                 int grid, int2* over, int32_t* over_count, int32_t* queue, int64_t part_n,
                                 hipStream_t st) {
  auto f = radius == 4 ? (lmax <= 32 ? launch_b<AnyRaw, 4, 32> : launch_b<AnyRaw, 4, 64>)
                       : (lmax <= 32 ? launch_b<AnyRaw, 5, 32> : launch_b<AnyRaw, 5, 64>);
  return f(jobs, params, items, n_items, items_count, vpw, grid, over, over_count, queue, part_n, st);
}

int map_batch_wide_blocks_per_cu(int radius, int lmax) {
  if (radius == 4) return lmax <= 32 ? occ_b<AnyRaw, 4, 32>() : occ_b<AnyRaw, 4, 64>();
  return lmax <= 32 ? occ_b<AnyRaw, 5, 32>() : occ_b<AnyRaw, 5, 64>();
}

hipError_t launch_map_wide(const MapArgs& a, int radius, int lmax, bool debug, hipStream_t st) {
  if (radius == 4) return lmax <= 32 ? launch_w<4, 32>(a, debug, st) : launch_w<4, 64>(a, debug, st);
  return lmax <= 32 ? launch_w<5, 32>(a, debug, st) : launch_w<5, 64>(a, debug, st);
}

}  // namespace fr
