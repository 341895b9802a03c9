// Map kernels of the direction-averaged variant (GLCM and GLRLM features per
// direction, then their mean) at every radius: the fused per-voxel body with
// 13 GLCM and GLRLM passes a voxel.  Up to 13 MCC problems a voxel, solved
// in the kernel four at a time, bound it (two waves a SIMD).  4,007 voxels, radius 2, Ng 32:
// 29.0 ms on the generic kernel (one 256-thread workgroup a voxel, tables
// in global memory), 0.94 ms here when it came in, 0.58 now.
#include "map_body.h"

namespace fr {

hipError_t launch_map_averaged(const MapArgs& a, int radius, int lmax, hipStream_t st) {
  return launch_v<kAveraged>(a, radius, lmax, st);
}

}  // namespace fr
