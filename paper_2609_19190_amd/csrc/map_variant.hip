// Map kernels of the merged extraction variants (GLCM distance, GLDM alpha)
// at every radius: the fused per-voxel body with the variant's counting, MCC
// problems solved in the kernel.  8,000 voxels, radius 2, Ng 32, tolerance 1:
// 0.15 ms; 100 voxels of radius 4 with two levels 0.19 (the generic kernel,
// which has four waves a voxel, 0.18).
#include "map_body.h"

namespace fr {

hipError_t launch_map_variant(const MapArgs& a, int radius, int lmax, hipStream_t st) {
  return a.opt.averaged ? launch_map_averaged(a, radius, lmax, st) : launch_v<kMerged>(a, radius, lmax, st);
}

}  // namespace fr
