// The MCC kernel, the staging transposes and the choice of a plain map kernel.
#include "map_body.h"

namespace fr {
namespace {

// The MCC of the problems a map pass stashed: groups of four problems of
// one kind per wave (a 16-lane row each), the <= 16-level ones first; each
// result goes to its problem's output address.  A problem's result depends
// only on the problem, as in the in-kernel flush.
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(3))) void k_mcc(
    const int32_t* __restrict__ counts, const int32_t* __restrict__ err,
    const unsigned char* __restrict__ stash, int64_t part_n, bool fine) {
  if (err && *err != kJobOk) return;
  // workgroup b takes every per-th group of partition b mod kParts
  const int p = (int)blockIdx.x % kParts, per = ((int)gridDim.x - p + kParts - 1) / kParts;
  const int nn = counts[p * kPartStride + kCntNarrow], nw = counts[p * kPartStride + kCntWide];
  const unsigned char* first = stash + part_base(part_n, p) * kMccProblemBytes;
  const unsigned char* past = stash + part_base(part_n, p + 1) * kMccProblemBytes;
  const int gn = (nn + 3) / 4, gw = (nw + 3) / 4;
  for (int g = (int)blockIdx.x / kParts; g < gn + gw; g += per) {
    if (g < gn) {
      const int c = min(4, nn - 4 * g);
      mcc_narrow((const McSmall*)first + 4 * g, (1u << c) - 1u, fine);
    } else {
      // wide problem k is the (k + 1)-th entry from the end: slot s of the
      // group's window is problem k0 + c - 1 - s
      const int k0 = 4 * (g - gn), c = min(4, nw - k0);
      const McProblem* win = (const McProblem*)past - (k0 + c);
      mcc_wide(win, (1u << c) - 1u, fine);
    }
  }
}

// Tile transpose of the staging rows: 64 voxels x up to 96 maps per block
// through LDS, so both the row reads (16 bytes a lane, all of a thread's in
// flight together) and the per-map writes (64 consecutive floats) are
// contiguous.
__device__ inline void transpose_tile(const float* __restrict__ stage, float* __restrict__ out, int64_t n, int64_t m0,
                                      int count) {
  __shared__ float tile[64][kStageStride + 1];
  constexpr int Q = kStageStride / 4, PER = 64 * Q / 256;
  const int t = threadIdx.x;
  float4 r[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int e = t + 256 * i, v = e / Q, k = 4 * (e % Q);
    r[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (m0 + v < n && k < count) r[i] = *(const float4*)(stage + (m0 + v) * kStageStride + k);
  }
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int e = t + 256 * i, v = e / Q, k = 4 * (e % Q);
    tile[v][k] = r[i].x;
    tile[v][k + 1] = r[i].y;
    tile[v][k + 2] = r[i].z;
    tile[v][k + 3] = r[i].w;
  }
  __syncthreads();
  const int v = t % 64;
  if (m0 + v < n) {
#pragma unroll 4
    for (int k = t / 64; k < count; k += 4) out[(int64_t)k * n + m0 + v] = tile[v][k];
  }
}

__global__ __launch_bounds__(256) void k_transpose(const float* __restrict__ stage,
                                                   float* __restrict__ out, int64_t n,
                                                   int count, const DiscParams* __restrict__ params) {
  if (params->err != kJobOk) return;
  transpose_tile(stage, out, n, (int64_t)blockIdx.x * 64, count);
}

__global__ __launch_bounds__(256) void k_transpose_batch(const BatchJob* __restrict__ jobs,
                                                         const DiscParams* __restrict__ params,
                                                         const int2* __restrict__ items) {
  const int2 it2 = items ? items[blockIdx.x] : make_int2(0, (int)blockIdx.x * 64);
  const BatchJob& J = jobs[it2.x];
  if (params[it2.x].err != kJobOk) return;
  transpose_tile(J.stage, J.out, J.n_mask, it2.y, J.count);
}

}  // namespace

hipError_t launch_transpose_batch(const BatchJob* jobs, const DiscParams* params, const int2* items,
                                  int32_t n_items, hipStream_t st) {
  if (n_items <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_transpose_batch, dim3((unsigned)n_items), dim3(256), 0, st, jobs, params, items);
  return hipGetLastError();
}

hipError_t launch_mcc(const int32_t* counts, const int32_t* err, const unsigned char* stash,
                      int64_t part_n, bool fine, hipStream_t st) {
  static int grid = 0;  // resident workgroups of k_mcc: a persistent grid
  if (grid == 0) {
    int dev = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void*)k_mcc, 64, 0) != hipSuccess) {
      (void)hipGetLastError();
      cus = 256;
      per_cu = 1;
    }
    grid = (per_cu > 0 ? per_cu : 1) * (cus > 0 ? cus : 1);
    if (grid < kParts) grid = kParts;
  }
  hipLaunchKernelGGL(k_mcc, dim3((unsigned)grid), dim3(64), 0, st, counts, err, stash, part_n, fine);
  return hipGetLastError();
}

hipError_t launch_transpose(const float* stage, float* out, int64_t n, int count,
                            const DiscParams* params, hipStream_t st) {
  const int64_t nb = (n + 63) / 64;
  hipLaunchKernelGGL(k_transpose, dim3((unsigned)nb), dim3(256), 0, st, stage, out, n, count, params);
  return hipGetLastError();
}

hipError_t launch_map(const MapArgs& a, int dtype, int radius, int lmax, bool debug, hipStream_t st) {
  if (a.opt.glcm_dist != 1 || a.opt.gldm_alpha != 0 || a.opt.averaged)
    return launch_map_variant(a, radius, lmax, st);
  if (radius > 3) return launch_map_wide(a, radius, lmax, debug, st);
  return dtype == 1 ? launch_map_i16(a, radius, lmax, debug, st) : launch_map_f32(a, radius, lmax, debug, st);
}

hipError_t launch_map_batch(const BatchJob* jobs, const DiscParams* params, const int2* items,
                            int32_t n_items, const int32_t* items_count, int32_t vpw, int dtype,
                            int radius, int lmax, int grid, int2* over, int32_t* over_count,
                            int32_t* queue, int64_t part_n, hipStream_t st) {
  if (n_items <= 0 && !items_count) return hipSuccess;
  if (radius > 3)
    return launch_map_batch_wide(jobs, params, items, n_items, items_count, vpw, radius, lmax, grid, over,
                                 over_count, queue, part_n, st);
  auto f = dtype == 1 ? launch_map_batch_i16 : launch_map_batch_f32;
  return f(jobs, params, items, n_items, items_count, vpw, radius, lmax, grid, over, over_count, queue, part_n, st);
}

int map_batch_blocks_per_cu(int dtype, int radius, int lmax) {
  if (radius > 3) return map_batch_wide_blocks_per_cu(radius, lmax);
  return dtype == 1 ? map_batch_i16_blocks_per_cu(radius, lmax) : map_batch_f32_blocks_per_cu(radius, lmax);
}

}  // namespace fr
