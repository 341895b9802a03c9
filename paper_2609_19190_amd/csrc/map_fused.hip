// The fused batched pass over every radius 1..3.
#include "map_body.h"

namespace fr {
namespace {

// The fused batched pass: every fixed radius of one raw type in one
// persistent kernel.  The LDS holds one radius's layout at a time (a union
// of the three); a workgroup switches layout when its next item's job has
// another radius (items come grouped by radius, so rarely), after flushing
// the MCC problems stashed in the old layout (64-level form).  The 32-level
// form asks for four waves per SIMD (128 VGPRs, some fifteen spilled): its
// LDS allows fifteen waves per CU, three per SIMD left a fifth of them out
// (a batch of 16 scans: 2.48 -> 2.37 ms).
struct FusedNone {};
template <int LMAX, bool MOUT>
union FusedSmem {
  std::conditional_t<LMAX == 32, Smem<1, 32, MOUT>, FusedNone> s1;
  Smem<2, LMAX, MOUT> s2;
  Smem<3, LMAX, MOUT> s3;
};

template <typename T, int LMAX>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(LMAX == 32 ? 4 : 2))) void k_map_fused(
    const BatchJob* __restrict__ jobs, const DiscParams* __restrict__ params,
    const int2* __restrict__ items, int32_t n_items_host, const int32_t* __restrict__ items_count,
    int2* over, int32_t* over_count, int32_t* queue, unsigned char* mcc, int64_t part_n,
    int32_t* mcc_count) {
  constexpr bool MOUT = true;  // problems with <= 32 levels go to the stash
  __shared__ FusedSmem<LMAX, MOUT> sm;
  int part = (int)blockIdx.x % kParts, left = kParts;
  int cur = 0;         // radius whose layout the LDS holds (0: none yet)
  int ns = 0, nq = 0;  // deferred MCC problems (64-level form)
  bool big = false;
  auto flush = [&](bool) FR_INLINE {
    if constexpr (LMAX > 32) {  // a problem with more than 32 levels, solved here
      if (big) {
        if (cur == 2)
          mcc_flush(sm.s2, 0, 0, true);
        else
          mcc_flush(sm.s3, 0, 0, true);
        big = false;
      }
    }
  };
  int64_t m = 0, m1 = 0;
  MapArgs a;
  const BatchJob* J = nullptr;
  for (;;) {
    int R = cur;
    while (m >= m1) {  // next item of a job without error
      const int64_t w = take_item(queue, items_count, part_n, n_items_host, part, left);
      if (w < 0) break;
      const int2 it2 = items[w];
      const DiscParams& P = params[it2.x];
      if (P.err != kJobOk) continue;
      J = &jobs[it2.x];
      a.params = &P;
      a.vol = J->vol;
      a.levels = J->levels;
      a.list = J->list;
      a.sample = nullptr;
      a.out = J->out;
      a.stage = J->stage;
      a.n_out = J->n_mask;
      a.n_items = J->n_mask;
      a.n_list = J->n_mask;
      a.nx = J->nx;
      a.ny = J->ny;
      a.nz = J->nz;
      a.ng = P.ng;
      a.families = J->families;
      a.voxel_volume = J->voxel_volume;
      a.nblk = 0;
      a.d_glcm = a.d_glrlm = a.d_glszm = a.d_gldm = a.d_ngn = a.d_hist = nullptr;
      a.d_ngS = nullptr;
      a.items = nullptr;
      a.items_count = nullptr;
      a.over = over;
      a.over_count = over_count;
      a.over_job = it2.x;
      a.radius = J->radius;
      a.opt = J->opt;
      a.mcc = mcc;
      a.part_n = part_n;
      a.key0 = J->key0;
      a.mcc_count = mcc_count;
      R = __builtin_amdgcn_readfirstlane(J->radius);
      m = it2.y;
      m1 = (int64_t)it2.y + (LMAX == 32 ? J->vpw : 1);
      if (m1 > J->n_mask) m1 = J->n_mask;
    }
    const bool more = m < m1;
    if (!more || R != cur) {  // end, or another radius's layout
      flush(true);
      if (!more) break;
      if (R == 1) {
        if constexpr (LMAX == 32) smem_layout(sm.s1);
      } else if (R == 2) {
        smem_layout(sm.s2);
      } else {
        smem_layout(sm.s3);
      }
      cur = R;
    }
    if (R == 1) {
      if constexpr (LMAX == 32) map_voxel<T, 1, 32, false, MOUT>(sm.s1, a, a.list[m], m, ns, nq, big);
    } else if (R == 2) {
      map_voxel<T, 2, LMAX, false, MOUT>(sm.s2, a, a.list[m], m, ns, nq, big);
    } else {
      map_voxel<T, 3, LMAX, false, MOUT>(sm.s3, a, a.list[m], m, ns, nq, big);
    }
    ++m;
    flush(false);
  }
}


template <typename T, int LMAX>
int occ_f() {
  int nb = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, (const void*)k_map_fused<T, LMAX>, 64, 0) != hipSuccess)
    return 1;
  return nb > 0 ? nb : 1;
}

}  // namespace

hipError_t launch_map_fused(const BatchJob* jobs, const DiscParams* params, const int2* items,
                            int32_t n_items, const int32_t* items_count, int dtype, int lmax,
                            int grid, int2* over, int32_t* over_count, int32_t* queue,
                            unsigned char* mcc, int64_t part_n, int32_t* mcc_count, hipStream_t st) {
  if (n_items <= 0 && !items_count) return hipSuccess;
  const dim3 g((unsigned)grid), b(64);
  if (dtype == 1) {
    if (lmax <= 32)
      hipLaunchKernelGGL((k_map_fused<int16_t, 32>), g, b, 0, st, jobs, params, items, n_items, items_count,
                         over, over_count, queue, mcc, part_n, mcc_count);
    else
      hipLaunchKernelGGL((k_map_fused<int16_t, 64>), g, b, 0, st, jobs, params, items, n_items, items_count,
                         over, over_count, queue, mcc, part_n, mcc_count);
  } else {
    if (lmax <= 32)
      hipLaunchKernelGGL((k_map_fused<float, 32>), g, b, 0, st, jobs, params, items, n_items, items_count,
                         over, over_count, queue, mcc, part_n, mcc_count);
    else
      hipLaunchKernelGGL((k_map_fused<float, 64>), g, b, 0, st, jobs, params, items, n_items, items_count,
                         over, over_count, queue, mcc, part_n, mcc_count);
  }
  return hipGetLastError();
}

int map_fused_blocks_per_cu(int dtype, int lmax) {
  if (dtype == 1) return lmax <= 32 ? occ_f<int16_t, 32>() : occ_f<int16_t, 64>();
  return lmax <= 32 ? occ_f<float, 32>() : occ_f<float, 64>();
}

}  // namespace fr
