// Batched map kernels of radius 1..3 for int16 volumes (one persistent pass per
// radius, as served jobs take it).
#include "map_body.h"

namespace fr {

hipError_t launch_map_batch_i16(const BatchJob* jobs, const DiscParams* params, const int2* items, int32_t n_items,
                                const int32_t* items_count, int32_t vpw, int radius, int lmax, int grid, int2* over,
                                int32_t* over_count, int32_t* queue, int64_t part_n, hipStream_t st) {
  return launch_b_r<int16_t>(jobs, params, items, n_items, items_count, vpw, radius, lmax, grid, over, over_count,
                           queue, part_n, st);
}

int map_batch_i16_blocks_per_cu(int radius, int lmax) { return occ_b_r<int16_t>(radius, lmax); }

}  // namespace fr
