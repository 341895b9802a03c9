// Plain map kernels of radius 1..3 for int16 volumes.
#include "map_body.h"

namespace fr {

hipError_t launch_map_i16(const MapArgs& a, int radius, int lmax, bool debug, hipStream_t st) {
  return launch_r<int16_t>(a, radius, lmax, debug, st);
}

}  // namespace fr
