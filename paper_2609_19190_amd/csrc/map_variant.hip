// Map kernels of the extraction variants (GLCM distance, GLDM alpha,
// direction-averaged GLCM and GLRLM) at every radius: the fused per-voxel
// body with the variant's counting.  MCC problems are solved in the kernel
// (up to 13 per voxel when averaged, flushed four at a time; they bound the
// averaged form).  4,007 voxels, radius 2, Ng 32, averaged: 29.0 ms on the
// generic kernel, 0.94 ms here.
#include "map_body.h"

namespace fr {
namespace {

template <int R, int LMAX>
hipError_t launch_v(const MapArgs& a, hipStream_t st) {
  return a.opt.averaged ? launch_i<AnyRaw, R, LMAX, true, false, kAveraged>(a, st)
                        : launch_i<AnyRaw, R, LMAX, true, false, kMerged>(a, st);
}

}  // namespace

hipError_t launch_map_variant(const MapArgs& a, int radius, int lmax, hipStream_t st) {
  switch (radius) {
    case 1: return launch_v<1, 32>(a, st);
    case 2: return lmax <= 32 ? launch_v<2, 32>(a, st) : launch_v<2, 64>(a, st);
    case 3: return lmax <= 32 ? launch_v<3, 32>(a, st) : launch_v<3, 64>(a, st);
    case 4: return lmax <= 32 ? launch_v<4, 32>(a, st) : launch_v<4, 64>(a, st);
    default: return lmax <= 32 ? launch_v<5, 32>(a, st) : launch_v<5, 64>(a, st);
  }
}

}  // namespace fr
