// Plain map kernels of radius 1..3 for float volumes.
#include "map_body.h"

namespace fr {

hipError_t launch_map_f32(const MapArgs& a, int radius, int lmax, bool debug, hipStream_t st) {
  return launch_r<float>(a, radius, lmax, debug, st);
}

}  // namespace fr
