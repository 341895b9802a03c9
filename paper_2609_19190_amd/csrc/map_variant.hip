// Map kernels of the merged extraction variants (GLCM distance, GLDM alpha)
// at every radius: the fused per-voxel body with the variant's counting, MCC
// problems solved in the kernel.
#include "map_body.h"

namespace fr {

hipError_t launch_map_variant(const MapArgs& a, int radius, int lmax, hipStream_t st) {
  return a.opt.averaged ? launch_map_averaged(a, radius, lmax, st) : launch_v<kMerged>(a, radius, lmax, st);
}

}  // namespace fr
