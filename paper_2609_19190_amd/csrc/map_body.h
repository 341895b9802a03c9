#pragma once
// Fused spatial-mapping kernel for gfx950 (CDNA4, wave64).
//
// What it computes: for every VOI voxel c, the features of its cubic
// neighbourhood V(c) = cube(2r+1) ∩ image ∩ mask (paper: "Software design
// and extraction modes" -- spatial maps; Table 2 -- 18 first-order, 24 GLCM,
// 16 GLRLM, 16 GLSZM, 14 GLDM, 5 NGTDM maps; feature equations per IBSI as
// the paper defers to it, with the readings stated in fr.h).
//
// How: one wavefront (= one workgroup) handles the voxels of its part of the
// list one after another, all 64 lanes on one voxel:
//   gather   lane per cube position: levels and raw values, all loads in
//            flight together
//   levels   local compaction of the levels present (L <= LMAX), so every
//            table is L-sized instead of Ng-sized
//   first order  order statistics by sorting the values of their own levels
//   count    lane per cube position, the 26 neighbours as nine rows of three
//            bytes: equal-level neighbour bitmask, GLCM counts (13 forward
//            offsets, LDS atomics), GLCM row sums, GLDM dependence, NGTDM
//            exact integer sums (from row sums of the levels)
//   zones    union of the equal-level neighbours that no other one implies
//   runs     a run starts where the backward neighbour bit is clear; runs of
//            one voxel are counted from the masks, the others walked
//   features FP64, DPP reductions; integer numerators kept exact where a
//            feature is a ratio of integer sums; GLCM features via the
//            sum/difference histograms; MCC as the spectral radius of
//            D^-1/2 P D^-1/2 - v v^T (v = sqrt(px)), by Householder
//            tridiagonalisation and Sturm-count multisection
// The modes kMerged and kAveraged (distance, tolerance, averaged matrices)
// take the same body with their own counting.  Nothing here is a dense
// contraction, so no MFMA; the bound is VALU issue, and the latency and
// bandwidth of LDS where fewer than four waves share a SIMD.
#include <math.h>
#include <stddef.h>

#include <type_traits>
#include <utility>

#include "fr_internal.h"
#include "map_device.h"

namespace fr {
namespace {

constexpr int kNFO = 18, kNGLCM = 24, kNGLRLM = 16, kNGLSZM = 16, kNGLDM = 14, kNNGTDM = 5;

// Raw-value access: T is int16_t or float, or AnyRaw for instances shared by
// both raw types (the type is then read from the arguments, one
// wave-uniform branch per load).
struct AnyRaw {};
template <typename T>
__device__ inline float raw_at(const MapArgs& a, int64_t i) {
  if constexpr (std::is_same_v<T, AnyRaw>)
    return a.dtype == 1 ? (float)((const int16_t*)a.vol)[i] : ((const float*)a.vol)[i];
  else
    return (float)((const T*)a.vol)[i];
}

// What map_voxel counts: the defaults (kPlain), any GLCM distance and GLDM
// alpha with merged directions (kMerged), or GLCM and GLRLM features
// averaged over the directions (kAveraged).
enum { kPlain = 0, kMerged = 1, kAveraged = 2 };
// Sums over the directions of one voxel (kAveraged).
struct AvgMem {
  double glcm[24];  // GLCM features
  double mcc[13];   // MCC of each direction
};

// One deferred MCC problem: a neighbourhood with 2..NL present levels whose
// MCC is computed later, together with up to three others (one per 16-lane
// row of the wave).
template <int NL>
struct McProblemT {
  float* dst;  // address of this voxel's MCC map value
  int n;       // number of present levels
  // co-occurrence counts of the present levels, upper triangle (entry
  // (a, b), a <= b, at b (b + 1) / 2 + a; the row sums and N_P follow from
  // them exactly)
  uint16_t g[NL * (NL + 1) / 2];
};
using McProblem = McProblemT<32>;  // 17..32 levels (or 2..32 without a small pool)
using McSmall = McProblemT<16>;    // 2..16 levels
template <typename P, int N>
struct McSlots {
  P s[N];
};
template <typename P>
struct McSlots<P, 0> {};
static_assert(sizeof(McProblem) == kMccProblemBytes, "stash entry size");
static_assert(sizeof(McSmall) <= sizeof(McProblem), "stash entry size");

// Every neighbourhood with at most 32 present levels defers its MCC: four
// problems per flush.  A problem's result depends only on the problem (not
// on the instance or on what shares its flush).  Wider problems (64-level
// instances) are computed at the flush that follows their voxel, from the
// GLCM that is still in LDS.
template <int R, int LMAX>
constexpr int kMcSlots = 4;
// Problems with <= 16 levels have a pool of their own (four small slots),
// so both kinds of flush run with four problems; the radius-3, 32-level
// instance (whose LDS budget is tighter: eight workgroups per CU) keeps
// them in its large slots instead.
template <int R, int LMAX>
constexpr int kSmallSlots = (R == 3 && LMAX == 32) ? 0 : 4;

// MOUT: the MCC problems with <= 32 levels go to a global stash for the
// MCC kernel (no deferred-problem slots in LDS).
template <int R, int LMAX, bool MOUT = false>
struct Smem {
  static constexpr int S = 2 * R + 1;
  static constexpr int C = S * S * S;
  static constexpr int CP = (C + 63) / 64 * 64;
  // sort size, 64 * pow2 >= C
  static constexpr int SP = R == 1 ? 64 : R == 2 ? 128 : R == 3 ? 512 : R == 4 ? 1024 : 2048;
  // zone hash slots: more than the distinct (level, size) pairs, which are
  // at most |V| (27, 125) or, for radius 3, 178 (sizes 1, 2 for 64 levels
  // and 3 for 50 use 342 voxels), likewise 273 for radius 4 (sizes 1..4 for
  // 64 levels, 5 for 17) and 381 for radius 5 (1..5 for 64, 6 for 61)
  static constexpr int HT = R == 1 ? 64 : R == 2 ? 128 : R == 3 ? 256 : 512;
  // above radius 2 the hash overlays the equal-level masks, free by then
  static constexpr bool kHashInSame = R > 2;
  // GLCM |i-j| and i+j histograms over level values 1..Ng (Ng <= 255)
  static constexpr int PD = 256;
  static constexpr int PS = 512;
  // The co-occurrence counts, 16 bits each.  Up to 32 levels: counts of
  // (voxel's level l, forward neighbour's level m), levels l and l ^ 1 in
  // the halves of word (l >> 1) kRowWords + m + 1; column 0 takes the
  // neighbours outside V, so that counting needs neither a test nor an
  // order of the two.  More levels (where the table would cost occupancy):
  // the packed upper triangle of the symmetric counts.
  static constexpr bool kFullGlcm = LMAX <= 32;
  static constexpr int kRowWords = LMAX + 1;
  static constexpr int kGlcmWords = kFullGlcm ? LMAX / 2 * kRowWords : (LMAX * (LMAX + 1) / 2 + 1) / 2;
  // words in use for L present levels
  __device__ static int glcm_words(int L) { return kFullGlcm ? (L + 1) / 2 * kRowWords : (L * (L + 1) / 2 + 1) / 2; }
  // words of a level's 27 packed dependence counts: odd, so that lanes
  // reading a row each meet no bank conflicts
  static constexpr int kGldmWords = 15;
  static constexpr int SQ = S + 2;                                // padded cube side
  static constexpr int SX = (SQ + 3) / 4 * 4;                     // bytes of a padded cube row
  static constexpr int PC = SQ * SQ * SX + 4;                     // 8-byte reads end past the last row
  uint8_t cl[CP];        // compact level + 1 per cube position (0: not in V)
  // The regions below are shared by what lives at different times, because
  // LDS sets the occupancy at radius 3: 13.2 -> 10.7 KB is 15 workgroups a
  // CU instead of 12 (14.3 -> 12.2 ms for 1 M voxels).
  // One region (nb) in turn holds
  //   the same in a cube with a zero border of 1, rows from 4-byte
  //   boundaries (clp), and per position of the cube and of its border rows
  //   the level values of the position and its two neighbours along x,
  //   summed, times 32, plus how many of the three are in V (cw);
  //   after the counting pass, the zone pass's edge list (16-bit entries, at
  //   most three a voxel); the list of runs; the zone sizes at roots and
  //   the zones per size (zcnt, zps: 16-bit, packed); this voxel's maps,
  //   over the zone sizes or behind both.
  static constexpr int CWB = 2 * SQ * SQ * S;  // bytes of cw
  static constexpr int kZoneBytes = CP * 4;    // of zcnt and zps
  static constexpr int kFeatAt = CP * 2 >= 384 ? 0 : kZoneBytes;
  static constexpr int cmax(int a, int b) { return a > b ? a : b; }
  static constexpr int NB = (cmax(cmax(PC + CWB, 6 * C), cmax(kZoneBytes, kFeatAt + 384)) + 15) / 16 * 16;
  alignas(16) uint8_t nb[NB];
  __device__ uint8_t* clp() { return nb; }
  __device__ uint16_t* cw() { return (uint16_t*)(nb + PC); }
  __device__ uint16_t* list() { return (uint16_t*)nb; }
  __device__ uint32_t* zcnt() { return (uint32_t*)nb; }
  __device__ uint32_t* zps() { return (uint32_t*)nb + CP / 2; }
  __device__ float* feat() { return (float*)(nb + kFeatAt); }
  // level values 1..255; at most LMAX of them present in one neighbourhood
  // (a neighbourhood with more is handed to a wider instance)
  static constexpr int LV = 256;
  static constexpr int LVW = LV / 4;
  // per bit of the equal-level mask: what the zone pass covers with that
  // neighbour (dir_cover; zone bits), its distance in the cube (zone bits),
  // and the distance of a forward bit
  // (entries that are no bit of theirs hold 0)
  uint32_t zcov[32];
  uint8_t zoff[32], foff[32];
  uint8_t lval[LMAX];    // compact index -> level
  uint32_t hist[LMAX];   // level histogram
  uint32_t pxc[LMAX];    // GLCM row sums
  // maps taken before the others: first order, GLDM, NGTDM
  float early[kNFO + kNGLDM + kNNGTDM];
  McSlots<McProblem, MOUT ? 0 : kMcSlots<R, LMAX>> mq;  // deferred MCC problems
  McSlots<McSmall, MOUT ? 0 : kSmallSlots<R, LMAX>> ms;  // deferred MCC problems, <= 16 levels
  // The counting tables (a), the GLCM feature histograms (c) and the MCC
  // work space (b) share one region; b and c keep a.glcm in place and put
  // their arrays past it, over tables whose features are already done.
  union U {
    struct A {
      alignas(16) uint32_t glcm[kGlcmWords];
      // first the map of level values to compact indices (bytes); then the
      // equal-level masks; then the zone hash (kHashInSame)
      alignas(16) uint32_t same[CP];
      uint32_t parent[CP]; // raw values to sort; zone forest; the list of its roots
      // GLDM and NGTDM counts; once their maps are taken, the runs, the
      // zones per level and (kHashInSame false) the zone hash
      union {
        struct {
          alignas(16) uint32_t gldm[LMAX * kGldmWords];  // 16-bit counts, packed, kGldmWords words a level
          uint32_t ngn[LMAX];
          unsigned long long ngS[LMAX];
        };
        struct {
          alignas(16) uint32_t glrlm[LMAX * S];
          uint32_t zpl[LMAX];
          uint32_t hash_m[kHashInSame ? 1 : HT + HT / 2];
        };
      };
    } a;
    struct C {
      uint32_t glcm[kGlcmWords];  // a.glcm
      uint32_t pd[PD];                 // |i-j| histogram of the GLCM
      uint32_t ps[PS];                 // i+j histogram of the GLCM
    } c;
    struct B {
      uint32_t glcm[kGlcmWords];  // a.glcm, still read by the MCC
      int pl[LMAX];                    // compact level of present level i
      double d[LMAX];                  // tridiagonal form: diagonal
      double e2[LMAX];                 // and squared sub-diagonal
      float* big_dst;                  // a pending problem with > 32 levels
      int big_n;
    } b;
  } u;
  // zone hash: keys, then zones per (level, size) key (16-bit, packed)
  __device__ uint32_t* hkey() { return kHashInSame ? u.a.same : u.a.hash_m; }
  __device__ uint32_t* hcnt() { return hkey() + HT; }
};


// What a workgroup's tables hold before its first voxel.
template <int R, int LMAX, bool MOUT>
__device__ FR_INLINE inline void smem_layout(Smem<R, LMAX, MOUT>& sm) {
  using SM = Smem<R, LMAX, MOUT>;
  const int lane = threadIdx.x;
  if (lane < 32) {
    sm.zcov[lane] = 0u;
    sm.zoff[lane] = 0;
    sm.foff[lane] = 0;
  }
  __syncthreads();
  if (lane < 13) {
    const int off = (kDir[lane][2] * SM::S + kDir[lane][1]) * SM::S + kDir[lane][0];
    sm.zcov[zone_bit(lane)] = kDirCover[lane];
    sm.zoff[zone_bit(lane)] = (uint8_t)off;
    sm.foff[fwd_bit(lane)] = (uint8_t)off;
  }
  __syncthreads();
}
// Zeroes n bytes (rounded up to 16; the arrays that follow a cleared one are
// cleared or written later) from a 16-byte boundary.
__device__ FR_INLINE inline void clear16(void* p, int n, int lane) {
  for (int e = lane; e < (n + 15) / 16; e += 64) ((uint4*)p)[e] = make_uint4(0u, 0u, 0u, 0u);
}

// Packed 16-bit counts (GLCM, GLDM, zone tables): entry e in half e & 1 of
// word e >> 1; every count stays below 2^16 (at most 26 (2r+1)^3 = 34,606).
__device__ inline void gadd(uint32_t* g, int e, uint32_t v) {
  atomicAdd(&g[e >> 1], v << ((e & 1) << 4));
}
__device__ inline uint32_t gget(const uint32_t* g, int e) {
  return (g[e >> 1] >> ((e & 1) << 4)) & 0xffffu;
}
// Entry (r, c), r <= c, of a packed upper triangle.
__device__ inline int tri(int r, int c) { return c * (c + 1) / 2 + r; }
// The symmetric co-occurrence count of present levels r and c.
template <typename SM>
__device__ inline uint32_t gsym(const uint32_t* g, int r, int c) {
  if constexpr (SM::kFullGlcm)
    return ((g[(r >> 1) * SM::kRowWords + c + 1] >> ((r & 1) << 4)) & 0xffffu) +
           ((g[(c >> 1) * SM::kRowWords + r + 1] >> ((c & 1) << 4)) & 0xffffu);
  return gget(g, r <= c ? tri(r, c) : tri(c, r));
}
// One pair of neighbours of levels l and m.
template <typename SM>
__device__ inline void gpair(uint32_t* g, int l, int m) {
  if constexpr (SM::kFullGlcm)
    atomicAdd(&g[(l >> 1) * SM::kRowWords + m + 1], 1u << ((l & 1) << 4));
  else
    gadd(g, l < m ? tri(l, m) : tri(m, l), l == m ? 2u : 1u);
}
// Lanes below this one in m.
__device__ inline int below(uint64_t m) {
  return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Wavefront reductions on the VALU (DPP), every call site with all 64
// lanes active; the result is a wave-uniform scalar.
__device__ inline double readlane_d(double x, int l) {
  const long long b = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_readlane((int)b, l);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
__device__ inline long long readlane_l(long long x, int l) {
  const int lo = __builtin_amdgcn_readlane((int)x, l);
  const int hi = __builtin_amdgcn_readlane((int)(x >> 32), l);
  return ((long long)hi << 32) | (unsigned)lo;
}
// the two values a 64-bit x takes after a permlane16 (R16) or permlane32
// swap of a register with itself: lane i gets x of lane i and of i ^ 16 (32)
template <bool R16>
__device__ inline void swap_pair(long long b, long long& p0, long long& p1) {
  if (R16) {
    const auto lo = __builtin_amdgcn_permlane16_swap((int)b, (int)b, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((int)(b >> 32), (int)(b >> 32), false, false);
    p0 = ((long long)hi[0] << 32) | (unsigned)lo[0];
    p1 = ((long long)hi[1] << 32) | (unsigned)lo[1];
  } else {
    const auto lo = __builtin_amdgcn_permlane32_swap((int)b, (int)b, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((int)(b >> 32), (int)(b >> 32), false, false);
    p0 = ((long long)hi[0] << 32) | (unsigned)lo[0];
    p1 = ((long long)hi[1] << 32) | (unsigned)lo[1];
  }
}
// One DPP step on a 64-bit value (bit moves): a single 64-bit move for the
// row broadcasts (row_newbcast), two 32-bit moves for the other patterns.
// Steps that write every lane need no identity; the row broadcasts of
// row_bcast:15/31 write only some rows and give the identity bits `id` to
// the others.
template <int CTRL>
__device__ inline long long dpp64(long long b) {
  return __builtin_amdgcn_mov_dpp(b, CTRL, 0xf, 0xf, true);
}
template <int CTRL, int ROWMASK>
__device__ inline long long dpp64m(long long b, long long id) {
  return __builtin_amdgcn_update_dpp(id, b, CTRL, ROWMASK, 0xf, false);
}
// Reduce across the wavefront: four steps inside each row of 16 lanes
// (quad_perm twice, half-row mirror, row mirror: every lane then holds its
// row total), then two row broadcasts fold rows 0..3 into lane 63, which is
// read back as a uniform scalar.
template <typename Op>
__device__ inline long long wfold64(long long v, long long id, Op op) {
  v = op(v, dpp64<0xb1>(v));             // quad_perm [1,0,3,2]
  v = op(v, dpp64<0x4e>(v));             // quad_perm [2,3,0,1]
  v = op(v, dpp64<0x141>(v));            // row_half_mirror
  v = op(v, dpp64<0x140>(v));            // row_mirror
  v = op(v, dpp64m<0x142, 0xa>(v, id));  // row_bcast:15 into rows 1, 3
  v = op(v, dpp64m<0x143, 0xc>(v, id));  // row_bcast:31 into rows 2, 3
  return readlane_l(v, 63);
}
__device__ inline double wsum(double v) {
  return __longlong_as_double(wfold64(__double_as_longlong(v), 0ll, [](long long a, long long b) {
    return __double_as_longlong(__longlong_as_double(a) + __longlong_as_double(b));
  }));
}
__device__ inline long long wsumi(long long v) {
  return wfold64(v, 0ll, [](long long a, long long b) { return a + b; });
}
__device__ inline double wmaxd_nonneg(double v) {  // identity 0.0: inputs are >= 0
  return __longlong_as_double(wfold64(__double_as_longlong(v), 0ll, [](long long a, long long b) {
    return __double_as_longlong(fmax(__longlong_as_double(a), __longlong_as_double(b)));
  }));
}
__device__ inline unsigned wmaxu(unsigned v) {
  v = max(v, (unsigned)__builtin_amdgcn_mov_dpp((int)v, 0xb1, 0xf, 0xf, true));
  v = max(v, (unsigned)__builtin_amdgcn_mov_dpp((int)v, 0x4e, 0xf, 0xf, true));
  v = max(v, (unsigned)__builtin_amdgcn_mov_dpp((int)v, 0x141, 0xf, 0xf, true));
  v = max(v, (unsigned)__builtin_amdgcn_mov_dpp((int)v, 0x140, 0xf, 0xf, true));
  v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false));
  v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false));
  return (unsigned)__builtin_amdgcn_readlane((int)v, 63);
}
template <typename Op>
__device__ inline float wfold_f(float x, Op op) {  // x of idle lanes: the identity
  auto dpp = [&](auto ctrl) FR_INLINE {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), decltype(ctrl)::value, 0xf, 0xf, true));
  };
  x = op(x, dpp(std::integral_constant<int, 0xb1>{}));
  x = op(x, dpp(std::integral_constant<int, 0x4e>{}));
  x = op(x, dpp(std::integral_constant<int, 0x141>{}));
  x = op(x, dpp(std::integral_constant<int, 0x140>{}));
  const auto h = __builtin_amdgcn_permlane16_swap(__float_as_int(x), __float_as_int(x), false, false);
  x = op(__int_as_float(h[0]), __int_as_float(h[1]));
  const auto w = __builtin_amdgcn_permlane32_swap(__float_as_int(x), __float_as_int(x), false, false);
  return op(__int_as_float(w[0]), __int_as_float(w[1]));
}
__device__ inline int wscan_excl(int v, int lane, int* total) {
  // inclusive scan by DPP (no LDS round trips): shifts by 1, 2, 4, 8 inside
  // each 16-lane row (zero shifted in), then lane 15 of a row added to the
  // next row (rows 1, 3) and lane 31 to rows 2 and 3; every lane active
  (void)lane;
  int x = v;
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, true);  // row_shr:1
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, true);  // row_shr:2
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, true);  // row_shr:4
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, true);  // row_shr:8
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);  // row_bcast:15
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);  // row_bcast:31
  *total = __builtin_amdgcn_readlane(x, 63);
  return x - v;
}

// Eight wavefront sums at once.  A permlane32 swap adds lanes l and l+32
// while keeping values 0-3 in the low half and 4-7 in the high half; a
// permlane16 swap does the same for row pairs; each row then holds two
// values, reduced in its two 8-lane halves by DPP (row mirror, half-row
// mirror, quad permutes).  Total k ends in lane 8 k.
__device__ inline double fold32d(double x, double y) {
  const long long bx = __double_as_longlong(x), by = __double_as_longlong(y);
  const auto lo = __builtin_amdgcn_permlane32_swap((int)bx, (int)by, false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((int)(bx >> 32), (int)(by >> 32), false, false);
  return __longlong_as_double(((long long)hi[0] << 32) | (unsigned)lo[0]) +
         __longlong_as_double(((long long)hi[1] << 32) | (unsigned)lo[1]);
}
__device__ inline double fold16d(double x, double y) {
  const long long bx = __double_as_longlong(x), by = __double_as_longlong(y);
  const auto lo = __builtin_amdgcn_permlane16_swap((int)bx, (int)by, false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap((int)(bx >> 32), (int)(by >> 32), false, false);
  return __longlong_as_double(((long long)hi[0] << 32) | (unsigned)lo[0]) +
         __longlong_as_double(((long long)hi[1] << 32) | (unsigned)lo[1]);
}
template <int CTRL>
__device__ inline double dppd(double x) {
  return __longlong_as_double(dpp64<CTRL>(__double_as_longlong(x)));
}
__device__ inline void wsum8d(double (&v)[8]) {
  const double a0 = fold32d(v[0], v[4]), a1 = fold32d(v[1], v[5]);
  const double a2 = fold32d(v[2], v[6]), a3 = fold32d(v[3], v[7]);
  const double b0 = fold16d(a0, a2), b1 = fold16d(a1, a3);  // row r: values 2r', 2r'+1
  const bool hi8 = (threadIdx.x & 8) != 0;
  double c = (hi8 ? b1 : b0) + dppd<0x140>(hi8 ? b0 : b1);  // row_mirror
  c += dppd<0x141>(c);                                        // row_half_mirror
  c += dppd<0x4e>(c);
  c += dppd<0xb1>(c);
#pragma unroll
  for (int k = 0; k < 8; ++k) v[k] = readlane_d(c, 8 * k);
}
__device__ inline int fold32i(int x, int y) {
  const auto r = __builtin_amdgcn_permlane32_swap(x, y, false, false);
  return r[0] + r[1];
}
__device__ inline int fold16i(int x, int y) {
  const auto r = __builtin_amdgcn_permlane16_swap(x, y, false, false);
  return r[0] + r[1];
}
// 32-bit integer version (callers guarantee every total fits in int32).
__device__ inline void wsum8i(int (&v)[8]) {
  const int a0 = fold32i(v[0], v[4]), a1 = fold32i(v[1], v[5]);
  const int a2 = fold32i(v[2], v[6]), a3 = fold32i(v[3], v[7]);
  const int b0 = fold16i(a0, a2), b1 = fold16i(a1, a3);
  const bool hi8 = (threadIdx.x & 8) != 0;
  int c = (hi8 ? b1 : b0) + __builtin_amdgcn_mov_dpp(hi8 ? b0 : b1, 0x140, 0xf, 0xf, true);
  c += __builtin_amdgcn_mov_dpp(c, 0x141, 0xf, 0xf, true);
  c += __builtin_amdgcn_mov_dpp(c, 0x4e, 0xf, 0xf, true);
  c += __builtin_amdgcn_mov_dpp(c, 0xb1, 0xf, 0xf, true);
#pragma unroll
  for (int k = 0; k < 8; ++k) v[k] = __builtin_amdgcn_readlane(c, 8 * k);
}

// ---- MCC of four neighbourhoods at once --------------------------------
// Row r of 16 lanes holds problem r; lane j of the row is column j.  Values
// move inside a row by DPP (row broadcast of lane I, row mirrors), so the
// four problems never mix and each one's result does not depend on its row.
// The lane index through an opaque move: nothing derived from it is
// hoisted out of the voxel loop, where it would stay live (and spill)
// across the large MCC flush.
__device__ FR_INLINE inline int opaque_lane() {
  int lane;
  asm volatile("v_mov_b32 %0, %1" : "=v"(lane) : "v"((int)threadIdx.x));
  return lane;
}
template <int I>
__device__ inline double rbc(double v) {  // lane I of this row
  return __longlong_as_double(dpp64<0x150 + I>(__double_as_longlong(v)));
}
__device__ inline double rsum(double v) {  // row total in every lane of the row
  long long b = __double_as_longlong(v);
  b = __double_as_longlong(__longlong_as_double(b) + __longlong_as_double(dpp64<0xb1>(b)));
  b = __double_as_longlong(__longlong_as_double(b) + __longlong_as_double(dpp64<0x4e>(b)));
  b = __double_as_longlong(__longlong_as_double(b) + __longlong_as_double(dpp64<0x141>(b)));
  b = __double_as_longlong(__longlong_as_double(b) + __longlong_as_double(dpp64<0x140>(b)));
  return __longlong_as_double(b);
}
__device__ inline double rmax(double v) {
  long long b = __double_as_longlong(v);
  b = __double_as_longlong(fmax(__longlong_as_double(b), __longlong_as_double(dpp64<0xb1>(b))));
  b = __double_as_longlong(fmax(__longlong_as_double(b), __longlong_as_double(dpp64<0x4e>(b))));
  b = __double_as_longlong(fmax(__longlong_as_double(b), __longlong_as_double(dpp64<0x141>(b))));
  b = __double_as_longlong(fmax(__longlong_as_double(b), __longlong_as_double(dpp64<0x140>(b))));
  return __longlong_as_double(b);
}

// Slot of the stash that row r takes: the r-th set bit of mask (-1: none).
__device__ inline int row_slot(unsigned mask, int r) {
  int slot = -1, c = 0;
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    if ((mask >> s) & 1u) {
      if (c == r) slot = s;
      ++c;
    }
  }
  return slot;
}

// Rounds of 17-way Sturm multisection of [0, min(gb, 1)] for the row's
// tridiagonal (16 probes per row): 6, to a width <= 1 / 17^6, or, fine (radii
// 4 and 5, the variants), 8 (1 / 17^8, an error below 8e-11); the spectrum
// of B lies in [-1, 1] (that of D^-1/2 P D^-1/2 without its top eigenvalue 1).
template <typename F>
__device__ FR_INLINE inline double multisect_row(double gb, int r, int j, bool fine, F&& count_is_n,
                                                 double* lo_out) {
  double lo = 0.0, hi = fmin(gb, 1.0) * (1.0 + 1e-12) + 1e-300;
  const double frac = (double)(j + 1) / 17.0;
  const int rounds = fine ? kRowRounds<true> : kRowRounds<false>;
  const double wabs = fine ? 0.0 : 1e-8, wrel = fine ? 2e-9 : 2e-6;
  bool done = false;
#pragma unroll 1
  for (int round = 0; round < rounds; ++round) {
    // a row stops refining once its bracket is below 1e-8 + 2e-6 lo (the
    // midpoint then errs by under 5e-9 + 1e-6 of the value, far inside
    // the parity bound; fine: 2e-9 lo, below seven rounds' 1 / 17^7) or
    // after the last round; so its result depends on its own problem only.
    // The wave stops when every row has.
    done = done || (hi - lo) <= wabs + wrel * lo;
    if (__ballot(!done) == 0ull) break;
    const double x = lo + (hi - lo) * frac;
    const uint64_t bal = __ballot(count_is_n(x));
    const uint32_t rb = (uint32_t)(bal >> (16 * r)) & 0xffffu;
    if (done) {
    } else if (rb == 0u) {
      lo = lo + (hi - lo) * ((double)16 / 17.0);
    } else {
      const int t = __ffs(rb) - 1;
      const double xt = lo + (hi - lo) * ((double)(t + 1) / 17.0);
      const double xp = t > 0 ? lo + (hi - lo) * ((double)t / 17.0) : lo;
      hi = xt;
      lo = xp;
    }
  }
  if (lo_out) *lo_out = lo;
  return 0.5 * (lo + hi);
}

// The MCC of the row's problem: the spectral radius of its tridiagonal.
// First the multisection on the largest eigenvalue alone (one Sturm
// sequence a probe); when no eigenvalue lies below minus the lower end of
// its final bracket, the largest eigenvalue is the radius and every probe
// gave what the two-sided count of [-x, x) gives (a probe above the largest
// eigenvalue is above minus the smallest), so the result is the two-sided
// search's.  Otherwise the two-sided search runs (for the whole wave; a row
// keeps the result of the search its own problem calls for).
template <int N>
__device__ FR_INLINE inline double radius_row(const double (&D)[N], const double (&E2)[N], int n, double gb, int r,
                                              int j, bool fine) {
  double lo = 0.0;
  double m = multisect_row(gb, r, j, fine, [&](double x) FR_INLINE { return sturm_row<N, 1>(D, E2, x) == n; }, &lo);
  const bool ok = sturm_row<N, 2>(D, E2, lo) == 0;
  if (__ballot(!ok) != 0ull) {
    const double m2 =
        multisect_row(gb, r, j, fine, [&](double x) FR_INLINE { return sturm_row<N, 3>(D, E2, x) == n; }, nullptr);
    if (!ok) m = m2;
  }
  return m;
}

// Eight rows of a Householder step (rows 8b .. 8b + 7 of B) with the row
// broadcast fused into the FMA: v_fmac_f64 with a
// row_newbcast operand, one instruction per product where the compiler
// emits a DPP move and an FMA.  H: the rows are lanes 8..15 of their 16-row
// copy instead of 0..7.  mv8 adds col[t] * v_{8b+t} to pp[t & 3]; up8
// subtracts q_{8b+t} v + v_{8b+t} q from col[t] (in that order, the
// rounding of the two-FMA form).  The leading s_nop 4 covers the DPP read
// hazards after a VALU write of the broadcast source (2 wait states) or of
// EXEC (5).
#define FR_MV(L, A, C) "v_fmac_f64_dpp " A ", %4, " C " row_newbcast:" #L " row_mask:0xf bank_mask:0xf\n\t"
template <bool H>
__device__ FR_INLINE inline void mv8(double (&pp)[4], double vr, const double* c) {
  if constexpr (!H)
    asm volatile("s_nop 4\n\t" FR_MV(0, "%0", "%5") FR_MV(1, "%1", "%6") FR_MV(2, "%2", "%7") FR_MV(3, "%3", "%8")
                 FR_MV(4, "%0", "%9") FR_MV(5, "%1", "%10") FR_MV(6, "%2", "%11") FR_MV(7, "%3", "%12")
                 : "+v"(pp[0]), "+v"(pp[1]), "+v"(pp[2]), "+v"(pp[3])
                 : "v"(vr), "v"(c[0]), "v"(c[1]), "v"(c[2]), "v"(c[3]), "v"(c[4]), "v"(c[5]), "v"(c[6]), "v"(c[7]));
  else
    asm volatile("s_nop 4\n\t" FR_MV(8, "%0", "%5") FR_MV(9, "%1", "%6") FR_MV(10, "%2", "%7") FR_MV(11, "%3", "%8")
                 FR_MV(12, "%0", "%9") FR_MV(13, "%1", "%10") FR_MV(14, "%2", "%11") FR_MV(15, "%3", "%12")
                 : "+v"(pp[0]), "+v"(pp[1]), "+v"(pp[2]), "+v"(pp[3])
                 : "v"(vr), "v"(c[0]), "v"(c[1]), "v"(c[2]), "v"(c[3]), "v"(c[4]), "v"(c[5]), "v"(c[6]), "v"(c[7]));
}
#undef FR_MV
// c[t] += bq_t (-v) + bv_t (-q) for the eight rows, in that order.
#define FR_UP(L, C) "v_fmac_f64_dpp " C ", %9, %10 row_newbcast:" #L " row_mask:0xf bank_mask:0xf\n\t" \
                    "v_fmac_f64_dpp " C ", %8, %11 row_newbcast:" #L " row_mask:0xf bank_mask:0xf\n\t"
template <bool H>
__device__ FR_INLINE inline void up8(double* c, double vr, double qr, double nv, double nq) {
  if constexpr (!H)
    asm volatile("s_nop 4\n\t" FR_UP(0, "%0") FR_UP(1, "%1") FR_UP(2, "%2") FR_UP(3, "%3") FR_UP(4, "%4")
                 FR_UP(5, "%5") FR_UP(6, "%6") FR_UP(7, "%7")
                 : "+v"(c[0]), "+v"(c[1]), "+v"(c[2]), "+v"(c[3]), "+v"(c[4]), "+v"(c[5]), "+v"(c[6]), "+v"(c[7])
                 : "v"(vr), "v"(qr), "v"(nv), "v"(nq));
  else
    asm volatile("s_nop 4\n\t" FR_UP(8, "%0") FR_UP(9, "%1") FR_UP(10, "%2") FR_UP(11, "%3") FR_UP(12, "%4")
                 FR_UP(13, "%5") FR_UP(14, "%6") FR_UP(15, "%7")
                 : "+v"(c[0]), "+v"(c[1]), "+v"(c[2]), "+v"(c[3]), "+v"(c[4]), "+v"(c[5]), "+v"(c[6]), "+v"(c[7])
                 : "v"(vr), "v"(qr), "v"(nv), "v"(nq));
}
#undef FR_UP
// The same for two columns per lane (cA, cB: columns j and j + 16 of a
// 17..32-level problem in a 16-lane row), each broadcast feeding both.
#define FR_MV2(L, A, B, CA, CB)                                                    \
  "v_fmac_f64_dpp " A ", %4, " CA " row_newbcast:" #L " row_mask:0xf bank_mask:0xf\n\t" \
  "v_fmac_f64_dpp " B ", %4, " CB " row_newbcast:" #L " row_mask:0xf bank_mask:0xf\n\t"
#define FR_MV2_ALL(L0, L1, L2, L3, L4, L5, L6, L7)                                              \
  "s_nop 4\n\t" FR_MV2(L0, "%0", "%2", "%5", "%13") FR_MV2(L1, "%1", "%3", "%6", "%14")           \
      FR_MV2(L2, "%0", "%2", "%7", "%15") FR_MV2(L3, "%1", "%3", "%8", "%16")                      \
          FR_MV2(L4, "%0", "%2", "%9", "%17") FR_MV2(L5, "%1", "%3", "%10", "%18")                 \
              FR_MV2(L6, "%0", "%2", "%11", "%19") FR_MV2(L7, "%1", "%3", "%12", "%20")
template <bool H>
__device__ FR_INLINE inline void mv8w(double (&pA)[2], double (&pB)[2], double vsrc, const double* cA,
                                      const double* cB) {
  if constexpr (!H)
    asm volatile(FR_MV2_ALL(0, 1, 2, 3, 4, 5, 6, 7)
                 : "+v"(pA[0]), "+v"(pA[1]), "+v"(pB[0]), "+v"(pB[1])
                 : "v"(vsrc), "v"(cA[0]), "v"(cA[1]), "v"(cA[2]), "v"(cA[3]), "v"(cA[4]), "v"(cA[5]), "v"(cA[6]),
                   "v"(cA[7]), "v"(cB[0]), "v"(cB[1]), "v"(cB[2]), "v"(cB[3]), "v"(cB[4]), "v"(cB[5]), "v"(cB[6]),
                   "v"(cB[7]));
  else
    asm volatile(FR_MV2_ALL(8, 9, 10, 11, 12, 13, 14, 15)
                 : "+v"(pA[0]), "+v"(pA[1]), "+v"(pB[0]), "+v"(pB[1])
                 : "v"(vsrc), "v"(cA[0]), "v"(cA[1]), "v"(cA[2]), "v"(cA[3]), "v"(cA[4]), "v"(cA[5]), "v"(cA[6]),
                   "v"(cA[7]), "v"(cB[0]), "v"(cB[1]), "v"(cB[2]), "v"(cB[3]), "v"(cB[4]), "v"(cB[5]), "v"(cB[6]),
                   "v"(cB[7]));
}
#undef FR_MV2_ALL
#undef FR_MV2
// cA[t] += q_i (-vA) + v_i (-qA), cB[t] += q_i (-vB) + v_i (-qB), i the
// row of t; %16 / %17: v and q sources, %18..%21: -vA, -vB, -qA, -qB.
#define FR_UP2(L, CA, CB)                                                            \
  "v_fmac_f64_dpp " CA ", %17, %18 row_newbcast:" #L " row_mask:0xf bank_mask:0xf\n\t" \
  "v_fmac_f64_dpp " CB ", %17, %19 row_newbcast:" #L " row_mask:0xf bank_mask:0xf\n\t" \
  "v_fmac_f64_dpp " CA ", %16, %20 row_newbcast:" #L " row_mask:0xf bank_mask:0xf\n\t" \
  "v_fmac_f64_dpp " CB ", %16, %21 row_newbcast:" #L " row_mask:0xf bank_mask:0xf\n\t"
#define FR_UP2_ALL(L0, L1, L2, L3, L4, L5, L6, L7)                                                   \
  "s_nop 4\n\t" FR_UP2(L0, "%0", "%8") FR_UP2(L1, "%1", "%9") FR_UP2(L2, "%2", "%10") FR_UP2(L3, "%3", "%11") \
      FR_UP2(L4, "%4", "%12") FR_UP2(L5, "%5", "%13") FR_UP2(L6, "%6", "%14") FR_UP2(L7, "%7", "%15")
template <bool H>
__device__ FR_INLINE inline void up8w(double* cA, double* cB, double vsrc, double qsrc, double nvA, double nvB,
                                      double nqA, double nqB) {
  if constexpr (!H)
    asm volatile(FR_UP2_ALL(0, 1, 2, 3, 4, 5, 6, 7)
                 : "+v"(cA[0]), "+v"(cA[1]), "+v"(cA[2]), "+v"(cA[3]), "+v"(cA[4]), "+v"(cA[5]), "+v"(cA[6]),
                   "+v"(cA[7]), "+v"(cB[0]), "+v"(cB[1]), "+v"(cB[2]), "+v"(cB[3]), "+v"(cB[4]), "+v"(cB[5]),
                   "+v"(cB[6]), "+v"(cB[7])
                 : "v"(vsrc), "v"(qsrc), "v"(nvA), "v"(nvB), "v"(nqA), "v"(nqB));
  else
    asm volatile(FR_UP2_ALL(8, 9, 10, 11, 12, 13, 14, 15)
                 : "+v"(cA[0]), "+v"(cA[1]), "+v"(cA[2]), "+v"(cA[3]), "+v"(cA[4]), "+v"(cA[5]), "+v"(cA[6]),
                   "+v"(cA[7]), "+v"(cB[0]), "+v"(cB[1]), "+v"(cB[2]), "+v"(cB[3]), "+v"(cB[4]), "+v"(cB[5]),
                   "+v"(cB[6]), "+v"(cB[7])
                 : "v"(vsrc), "v"(qsrc), "v"(nvA), "v"(nvB), "v"(nqA), "v"(nqB));
}
#undef FR_UP2_ALL
#undef FR_UP2

// MCC (spectral radius of B = D^-1/2 P D^-1/2 - v v^T over the present
// levels) of up to four stashed problems with n <= 16, row r taking the
// r-th slot of mask: Householder tridiagonalisation with one column per
// lane, then the row's Sturm multisection; row r writes its value to dst.
// O: type the result is stored as (double: one direction's MCC, kAveraged).
// fine: see multisect_row.
template <typename O = float, typename P>
__device__ FR_INLINE inline void mcc_narrow(const P* slots, unsigned mask, bool fine) {
  const int lane = opaque_lane(), r = lane >> 4, j = lane & 15;
  const int slot = row_slot(mask, r);
  const P& q = slots[slot >= 0 ? slot : 0];
  const int n = slot >= 0 ? q.n : 0;
  const bool lok = j < n;
  const int tj = j * (j + 1) / 2;
  uint32_t gc[16];  // column j of the counts
  uint32_t rowc = 0;
  static_for<0, 16>([&](auto ac) FR_INLINE {
    constexpr int a = decltype(ac)::value;
    const int e = a <= j ? tj + a : a * (a + 1) / 2 + j;  // in the slot for any a, j
    gc[a] = (a < n && lok) ? (uint32_t)q.g[e] : 0u;
    rowc += gc[a];
  });
  const double rtb = sqrt((double)rowc), irtb = lok ? 1.0 / rtb : 0.0;
  const double invN = 1.0 / rsum((double)rowc);  // N_P
  double col[16];
  static_for<0, 16>([&](auto ac) FR_INLINE {
    constexpr int a = decltype(ac)::value;
    const double rta = rbc<a>(rtb), irta = rbc<a>(irtb);
    col[a] = (a < n && lok) ? (double)gc[a] * (irta * irtb) - rta * rtb * invN : 0.0;
  });
  double e_lane = 0.0;
  // steps past the wave's largest n - 2 change nothing in any row: skipped
  const int kend = (int)wmaxu((unsigned)n) - 1;
  static_for<0, 14>([&](auto kc) FR_INLINE {
    constexpr int k = decltype(kc)::value;
    if (k >= kend) return;
    const double xi = (j > k && j < n) ? col[k] : 0.0;
    const double a2 = rsum(xi * xi);
    const double x0 = rbc<k + 1>(xi);
    const double alpha = a2 < kNoColumn ? 0.0 : -copysign(fsqrt(a2), x0);
    const double beta = a2 < kNoColumn ? 0.0 : rcp64(a2 - x0 * alpha);  // 2 / v.v
    const double vi = j == k + 1 ? x0 - alpha : xi;
    // rows in blocks of eight, the finished ones (v_i = q_i = 0) along
    double pp[4] = {0.0, 0.0, 0.0, 0.0};
    if constexpr (k < 7) mv8<false>(pp, vi, &col[0]);
    mv8<true>(pp, vi, &col[8]);
    const double pj = ((pp[0] + pp[1]) + (pp[2] + pp[3])) * beta;  // p = beta T v
    const double Kc = 0.5 * beta * rsum(vi * pj);
    // 0 on the finished columns (whose v is 0 too): they stay unchanged
    const double qj = j > k ? pj - Kc * vi : 0.0;
    const double nv = -vi, nq = -qj;
    if constexpr (k < 7) up8<false>(&col[0], vi, qj, nv, nq);  // T -= v q^T + q v^T
    up8<true>(&col[8], vi, qj, nv, nq);
    if (j == k) e_lane = alpha;  // also the last step k = n - 2 (a sign flip)
  });
  double d = 0.0;
  static_for<0, 16>([&](auto ic) FR_INLINE {
    constexpr int i = decltype(ic)::value;
    if (j == i) d = col[i];
  });
  if (n == 16 && j == 14) e_lane = col[15];  // last sub-diagonal entry (step 14 not run)
  const double dl = lok ? d : 0.0;
  const double el = j < n - 1 ? e_lane : 0.0;
  const double em = __longlong_as_double(dpp64<0x111>(__double_as_longlong(el)));  // e_{j-1}
  const double gb = rmax(lok ? fabs(dl) + fabs(el) + (j >= 1 ? fabs(em) : 0.0) : 0.0);
  const double e2l = el * el, dp = lok ? d : kPastN;
  double Db[16], Eb[16];  // the row's d_i and e_i^2, in every lane of the row
  static_for<0, 16>([&](auto ic) FR_INLINE {
    constexpr int i = decltype(ic)::value;
    Db[i] = rbc<i>(dp);
    Eb[i] = rbc<i>(e2l);
  });
  // the two-sided search directly: with at most 16 levels the smallest
  // eigenvalue dominates often enough that searching the largest first
  // costs more than it saves (measured)
  const double mcc =
      multisect_row(gb, r, j, fine, [&](double x) FR_INLINE { return sturm_row<16, 3>(Db, Eb, x) == n; }, nullptr);
  if (j == 0 && slot >= 0) *(O*)q.dst = (O)mcc;
}

// The same for problems with 17 <= n <= 32: lane j of row r holds columns
// j (cA) and j + 16 (cB) of its problem.
template <typename O = float>
__device__ FR_INLINE inline void mcc_wide(const McProblem* slots, unsigned mask, bool fine) {
  const int lane = opaque_lane(), r = lane >> 4, j = lane & 15, jb = j + 16;
  const int slot = row_slot(mask, r);
  const McProblem& q = slots[slot >= 0 ? slot : 0];
  const int n = slot >= 0 ? q.n : 0;
  const bool okA = j < n, okB = jb < n;
  const int tA = j * (j + 1) / 2, tB = jb * (jb + 1) / 2;
  uint32_t gcA[32], gcB[32];  // columns j and j + 16 of the counts
  uint32_t rcA = 0, rcB = 0;
  static_for<0, 32>([&](auto ac) FR_INLINE {
    constexpr int a = decltype(ac)::value;
    const int eA = a <= j ? tA + a : a * (a + 1) / 2 + j;  // in the slot for any a, j
    const int eB = a <= jb ? tB + a : a * (a + 1) / 2 + jb;
    gcA[a] = (a < n && okA) ? (uint32_t)q.g[eA] : 0u;
    gcB[a] = (a < n && okB) ? (uint32_t)q.g[eB] : 0u;
    rcA += gcA[a];
    rcB += gcB[a];
  });
  const double rtA = sqrt((double)rcA), irtA = okA ? 1.0 / rtA : 0.0;
  const double rtB = sqrt((double)rcB), irtB = okB ? 1.0 / rtB : 0.0;
  const double invN = 1.0 / rsum((double)rcA + (double)rcB);  // N_P
  double cA[32], cB[32];
  static_for<0, 32>([&](auto ac) FR_INLINE {
    constexpr int a = decltype(ac)::value;
    const double rta = a < 16 ? rbc<a & 15>(rtA) : rbc<a & 15>(rtB);
    const double irta = a < 16 ? rbc<a & 15>(irtA) : rbc<a & 15>(irtB);
    cA[a] = (a < n && okA) ? (double)gcA[a] * (irta * irtA) - rta * rtA * invN : 0.0;
    cB[a] = (a < n && okB) ? (double)gcB[a] * (irta * irtB) - rta * rtB * invN : 0.0;
  });
  double eA = 0.0, eB = 0.0;
  // steps k = 0 .. nmax - 2 (a step past a problem's own n - 2 changes
  // nothing in it); runtime loops over four groups of steps, each group's
  // body covering the rows from its first step on (rows <= k get v_i = 0
  // and q_i = 0, so they are unchanged) -- a quarter of the code of a full
  // unroll
  const int nmax = (int)wmaxu((unsigned)n);
  const int kend = nmax - 1;
  auto steps = [&](auto k0c, auto k1c) FR_INLINE {
    constexpr int K0 = decltype(k0c)::value, K1 = decltype(k1c)::value;
#pragma unroll 1
    for (int k = K0; k < K1 && k < kend; ++k) {
      // row k of the lane's columns and its entry k + 1 (a branch, not
      // selects: the empty statement keeps the moves inside it)
      double ckA = 0.0, ckB = 0.0, x0 = 0.0;
      static_for<K0, K1>([&](auto cc) FR_INLINE {
        constexpr int c = decltype(cc)::value;
        if (k == c) {
          ckA = cA[c];
          ckB = cB[c];
          x0 = c + 1 < 16 ? rbc<(c + 1) & 15>(ckA) : rbc<(c + 1) & 15>(ckB);
          asm volatile("" : "+v"(ckA), "+v"(ckB), "+v"(x0));
        }
      });
      // column k below the diagonal; by symmetry B[i][k] = cA[k] of lane i
      const double xA = (j > k && j < n) ? ckA : 0.0;
      const double xB = (jb > k && jb < n) ? ckB : 0.0;
      const double a2 = rsum(xA * xA + xB * xB);
      const double alpha = a2 < kNoColumn ? 0.0 : -copysign(fsqrt(a2), x0);
      const double beta = a2 < kNoColumn ? 0.0 : rcp64(a2 - x0 * alpha);  // 2 / v.v
      const double vA = j == k + 1 ? x0 - alpha : xA;
      const double vB = jb == k + 1 ? x0 - alpha : xB;
      // rows from K0 on, in blocks of eight behind one uniform branch each
      // (block b only if 8 b < nmax: rows past every problem's n hold zeros,
      // as v and q of the finished rows); two partial sums per column for
      // latency
      double pA2[2] = {0.0, 0.0}, pB2[2] = {0.0, 0.0};
      static_for<K0 / 8, 4>([&](auto bc) FR_INLINE {
        constexpr int b = decltype(bc)::value;
        if (8 * b < nmax) mv8w<(b & 1) != 0>(pA2, pB2, b < 2 ? vA : vB, &cA[8 * b], &cB[8 * b]);
      });
      const double pA = (pA2[0] + pA2[1]) * beta;  // p = beta T v
      const double pB = (pB2[0] + pB2[1]) * beta;
      const double Kc = 0.5 * beta * rsum(vA * pA + vB * pB);
      // q = p - K v on the trailing columns, 0 on the finished ones (whose
      // v is 0 too), so the update leaves those unchanged
      const double qA = j > k ? pA - Kc * vA : 0.0, qB = jb > k ? pB - Kc * vB : 0.0;
      const double nvA = -vA, nvB = -vB, nqA = -qA, nqB = -qB;
      static_for<K0 / 8, 4>([&](auto bc) FR_INLINE {  // T -= v q^T + q v^T
        constexpr int b = decltype(bc)::value;
        if (8 * b < nmax)
          up8w<(b & 1) != 0>(&cA[8 * b], &cB[8 * b], b < 2 ? vA : vB, b < 2 ? qA : qB, nvA, nvB, nqA, nqB);
      });
      if (j == k) eA = alpha;  // also the last step k = n - 2 (a sign flip)
      if (jb == k) eB = alpha;
    }
  };
  steps(std::integral_constant<int, 0>{}, std::integral_constant<int, 8>{});
  steps(std::integral_constant<int, 8>{}, std::integral_constant<int, 16>{});
  steps(std::integral_constant<int, 16>{}, std::integral_constant<int, 24>{});
  steps(std::integral_constant<int, 24>{}, std::integral_constant<int, 30>{});
  double dA = 0.0, dB = 0.0;
  static_for<0, 32>([&](auto ic) FR_INLINE {
    constexpr int i = decltype(ic)::value;
    if (j == i) dA = cA[i];
    if (jb == i) dB = cB[i];
  });
  if (n == 32 && j == 14) eB = cB[31];  // last sub-diagonal entry (step 30 not run)
  const double dlA = okA ? dA : 0.0, dlB = okB ? dB : 0.0;
  const double elA = j < n - 1 ? eA : 0.0, elB = jb < n - 1 ? eB : 0.0;
  // e_{j-1} and e_{j+15}: lane 0 of the B half takes e_15 from lane 15 of A
  const double emA = __longlong_as_double(dpp64<0x111>(__double_as_longlong(elA)));
  double emB = __longlong_as_double(dpp64<0x111>(__double_as_longlong(elB)));
  const double e15 = rbc<15>(elA);
  if (j == 0) emB = e15;
  const double gA = okA ? fabs(dlA) + fabs(elA) + (j >= 1 ? fabs(emA) : 0.0) : 0.0;
  const double gB = okB ? fabs(dlB) + fabs(elB) + fabs(emB) : 0.0;
  const double gb = rmax(fmax(gA, gB));
  const double e2A = elA * elA, e2B = elB * elB;
  const double dpA = okA ? dA : kPastN, dpB = okB ? dB : kPastN;
  double Db[32], Eb[32];  // the row's d_i and e_i^2, in every lane of the row
  static_for<0, 16>([&](auto ic) FR_INLINE {
    constexpr int i = decltype(ic)::value;
    Db[i] = rbc<i>(dpA);
    Eb[i] = rbc<i>(e2A);
    Db[i + 16] = rbc<i>(dpB);
    Eb[i + 16] = rbc<i>(e2B);
  });
  const double mcc = radius_row<32>(Db, Eb, n, gb, r, j, fine);
  if (j == 0 && slot >= 0) *(O*)q.dst = (O)mcc;
}


// MCC of the pending problem with 33 <= n <= 64 present levels (64-level
// instances), straight from the GLCM still in LDS: one problem per wave,
// lane j holding column j of B in registers.  Each step stages v (then q)
// in LDS and reads it back so that lane n of every 16-lane row holds
// v_n, v_{16+n}, v_{32+n}, v_{48+n}; a row broadcast of lane i & 15 of copy
// i >> 4 then gives v_i to every lane, fused into the FMA that uses it
// (mv8, up8; a single 64-bit DPP move on the partial blocks).  Householder
// steps in runtime loops over groups of eight (each group's body covers the
// rows from its first step on; rows <= k get v_i = q_i = 0 and stay
// unchanged), then 4 rounds of 65-way Sturm multisection on the tridiagonal
// form (width <= 1 / 65^4), 6 if FINE (1 / 65^6).
template <typename O, bool FINE, int R, int LMAX, bool MOUT>
__device__ FR_INLINE inline void mcc_big(Smem<R, LMAX, MOUT>& sm) {
  const int lane = opaque_lane();
  const int n = __builtin_amdgcn_readfirstlane(sm.u.b.big_n);
  const bool ok = lane < n;
  const int plj = ok ? sm.u.b.pl[lane] : 0;
  const uint32_t rowc = ok ? sm.pxc[plj] : 0u;  // GLCM row sum of present level j
  const double rtj = sqrt((double)rowc), irtj = ok ? 1.0 / rtj : 0.0;
  const double invN = 1.0 / wsum((double)rowc);  // N_P
  // rt and 1/rt are 0 past n, so every entry outside n x n is 0 without a
  // select (and the code stays free of branches)
  uint32_t gv[64];  // column j of the counts: all LDS reads issued first
  static_for<0, 64>([&](auto ac) FR_INLINE {
    constexpr int a = decltype(ac)::value;
    gv[a] = gsym<Smem<R, LMAX, MOUT>>(sm.u.a.glcm, __builtin_amdgcn_readlane(plj, a), plj);
  });
  __builtin_amdgcn_sched_barrier(0);
  double col[64];
  static_for<0, 64>([&](auto ac) FR_INLINE {
    constexpr int a = decltype(ac)::value;
    const double rta = readlane_d(rtj, a), irta = readlane_d(irtj, a);
    col[a] = (double)gv[a] * (irta * irtj) - rta * rtj * invN;
  });
  double e_lane = 0.0;
  double* hv = sm.u.b.d;  // staging of v and q (the tridiagonal form comes later)
  double* hq = sm.u.b.e2;
  const int ln = lane & 15;
  const int kend = n - 1 < 62 ? n - 1 : 62;  // steps k <= n - 2 (k = 62 is not needed)
  auto steps = [&](auto k0c, auto k1c) FR_INLINE {
    constexpr int K0 = decltype(k0c)::value, K1 = decltype(k1c)::value;
#pragma unroll 1
    for (int k = K0; k < K1 && k < kend; ++k) {
      double ck = 0.0;  // row k of the lane's column
      static_for<K0, K1>([&](auto cc) FR_INLINE {
        constexpr int c = decltype(cc)::value;
        if (k == c) {  // a branch, as in mcc_wide
          ck = col[c];
          asm volatile("" : "+v"(ck));
        }
      });
      // column k below the diagonal; by symmetry B[i][k] = col[k] of lane i
      const double x = lane > k ? ck : 0.0;
      const double a2 = wsum(x * x);
      const double x0 = readlane_d(x, k + 1);
      const double alpha = a2 < kNoColumn ? 0.0 : -copysign(fsqrt(a2), x0);
      const double beta = a2 < kNoColumn ? 0.0 : rcp64(a2 - x0 * alpha);  // 2 / v.v
      const double v = lane == k + 1 ? x0 - alpha : x;
      double vr[4];  // vr[m] = v_{16 m + n} in lane n of every row
      hv[lane] = v;
      __syncthreads();
      static_for<0, 4>([&](auto mc) FR_INLINE { vr[decltype(mc)::value] = hv[16 * decltype(mc)::value + ln]; });
      // rows from K0 on, in blocks of eight behind one uniform branch each
      // (block b only if 8 b < n); rows past n inside a block hold zeros,
      // and v_i = q_i = 0 there and in the finished rows.  Four independent
      // sums for latency.
      double pp[4] = {0.0, 0.0, 0.0, 0.0};
      static_for<K0 / 8, 8>([&](auto bc) FR_INLINE {
        constexpr int b = decltype(bc)::value;
        if (8 * b < n) mv8<(b & 1) != 0>(pp, vr[b >> 1], &col[8 * b]);
      });
      double p = (pp[0] + pp[1]) + (pp[2] + pp[3]);
      p *= beta;  // p = beta T v
      const double Kc = 0.5 * beta * wsum(v * p);
      const double q = lane > k ? p - Kc * v : 0.0;
      double qr[4];  // the same copies of q
      hq[lane] = q;
      __syncthreads();
      static_for<0, 4>([&](auto mc) FR_INLINE { qr[decltype(mc)::value] = hq[16 * decltype(mc)::value + ln]; });
      const double nv = -v, nq = -q;
      static_for<K0 / 8, 8>([&](auto bc) FR_INLINE {  // T -= v q^T + q v^T
        constexpr int b = decltype(bc)::value;
        if (8 * b < n) up8<(b & 1) != 0>(&col[8 * b], vr[b >> 1], qr[b >> 1], nv, nq);
      });
      if (lane == k) e_lane = alpha;  // also the last step k = n - 2 (a sign flip)
    }
  };
  steps(std::integral_constant<int, 0>{}, std::integral_constant<int, 8>{});
  steps(std::integral_constant<int, 8>{}, std::integral_constant<int, 16>{});
  steps(std::integral_constant<int, 16>{}, std::integral_constant<int, 24>{});
  steps(std::integral_constant<int, 24>{}, std::integral_constant<int, 32>{});
  steps(std::integral_constant<int, 32>{}, std::integral_constant<int, 40>{});
  steps(std::integral_constant<int, 40>{}, std::integral_constant<int, 48>{});
  steps(std::integral_constant<int, 48>{}, std::integral_constant<int, 56>{});
  steps(std::integral_constant<int, 56>{}, std::integral_constant<int, 62>{});
  double d = 0.0;
  static_for<0, 64>([&](auto ic) FR_INLINE {
    constexpr int i = decltype(ic)::value;
    if (lane == i) d = col[i];
  });
  if (n == 64 && lane == 62) e_lane = col[63];  // last sub-diagonal entry (step 62 not run)
  const double dl = ok ? d : 0.0;
  const double el = lane < n - 1 ? e_lane : 0.0;
  const double em = __shfl_up(el, 1);  // e_{lane-1}
  const double gb = wmaxd_nonneg(ok ? fabs(dl) + fabs(el) + (lane >= 1 ? fabs(em) : 0.0) : 0.0);
  __syncthreads();  // the last step's reads of hv and hq are done
  if (ok) {
    sm.u.b.d[lane] = dl;
    sm.u.b.e2[lane] = el * el;
  }
  __syncthreads();
  // the spectrum of B lies in [-1, 1]; the largest eigenvalue alone first,
  // the two-sided count only when the smallest may be the larger in size
  // (as radius_row)
  const double hi0 = fmin(gb, 1.0) * (1.0 + 1e-12) + 1e-300;
  const double frac = (double)(lane + 1) / 65.0;
  auto search = [&](auto seqc, double& lo, double& hi) FR_INLINE {
    constexpr int SEQ = decltype(seqc)::value;
    lo = 0.0;
    hi = hi0;
#pragma unroll 1
    for (int round = 0; round < kBigRounds<FINE>; ++round) {
      const double xr = lo + (hi - lo) * frac;
      const uint64_t bal = __ballot(sturm_span_r<SEQ>(sm.u.b.d, sm.u.b.e2, n, xr) == n);
      if (bal == 0ull) {
        lo = readlane_d(xr, 63);
      } else {
        const int t = __ffsll((unsigned long long)bal) - 1;
        const double xt = readlane_d(xr, t);
        const double xp = t > 0 ? readlane_d(xr, t - 1) : lo;
        hi = xt;
        lo = xp;
      }
    }
  };
  double lo, hi;
  search(std::integral_constant<int, 1>{}, lo, hi);
  if (sturm_span_r<2>(sm.u.b.d, sm.u.b.e2, n, lo) != 0) search(std::integral_constant<int, 3>{}, lo, hi);
  if (lane == 0) *(O*)sm.u.b.big_dst = (O)(0.5 * (lo + hi));
}

// Computes the pending MCC problems: the one with more than 32 levels (if
// big), the first ns problems of the small pool and the first nq of the
// large pool (a large slot with <= 16 levels goes to the one-column pass).
// Which routine takes a problem depends only on its n, so a result does
// not depend on the other problems of the flush.
template <typename O = float, bool FINE = false, int R, int LMAX, bool MOUT>
__device__ FR_INLINE inline void mcc_flush(Smem<R, LMAX, MOUT>& sm, int ns, int nq, bool big) {
  __syncthreads();
  if constexpr (LMAX > 32) {
    if (big) mcc_big<O, FINE>(sm);
  }
  if constexpr (!MOUT) mcc_flush_pools<O, FINE>(sm, ns, nq);
  __syncthreads();
}

// The LDS pools' problems of a flush (see mcc_flush).
template <typename O, bool FINE, int R, int LMAX>
__device__ FR_INLINE inline void mcc_flush_pools(Smem<R, LMAX, false>& sm, int ns, int nq) {
  if constexpr (kSmallSlots<R, LMAX> > 0) {
    if (ns) mcc_narrow<O>(sm.ms.s, (1u << ns) - 1u, FINE);
  }
  if (nq) {
    unsigned narrow = 0u, wide = 0u;
    for (int s = 0; s < nq; ++s) {
      if (sm.mq.s[s].n <= 16)
        narrow |= 1u << s;
      else
        wide |= 1u << s;
    }
    if constexpr (kSmallSlots<R, LMAX> == 0) {
      if (narrow) mcc_narrow<O>(sm.mq.s, narrow, FINE);
    }
    if (wide) mcc_wide<O>(sm.mq.s, wide, FINE);
  }
}

// Bitonic sort of 64 NPL values held in registers, the NIN values of each
// lane's `in` first (+inf beyond; +inf sorts last), element e = lane * NPL
// + r: stages whose partner is in the same lane are register
// compare-exchanges, the others exchange with lane ^ (j / NPL).  No
// barriers.  Writes the first NOUT of the sorted values to srt.
// x of lane (lane ^ M), M a power of two below 64, without the LDS
// crossbar: DPP quad permutes (1, 2), row rotates (4: by 4 or 12 depending
// on lane bit 2; 8), and the gfx950 row / half swaps (16, 32).
template <int M>
__device__ inline float xor_lane(float x, int lane) {
  const int b = __float_as_int(x);
  if constexpr (M == 1) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(b, 0xb1, 0xf, 0xf, false));
  } else if constexpr (M == 2) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(b, 0x4e, 0xf, 0xf, false));
  } else if constexpr (M == 4) {
    // row_ror:12 (lane + 4), then row_ror:4 (lane - 4) into banks 1 and 3
    const int r12 = __builtin_amdgcn_mov_dpp(b, 0x12c, 0xf, 0xf, false);
    return __int_as_float(__builtin_amdgcn_update_dpp(r12, b, 0x124, 0xf, 0xa, false));
  } else if constexpr (M == 8) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(b, 0x128, 0xf, 0xf, false));  // row_ror:8
  } else if constexpr (M == 16) {
    // swapping a register with itself: the odd rows find the partner in the
    // first result, the even rows in the second
    const auto r = __builtin_amdgcn_permlane16_swap(b, b, false, false);
    return __int_as_float((lane & 16) ? r[0] : r[1]);
  } else {
    static_assert(M == 32, "xor_lane: M in 1..32");
    const auto r = __builtin_amdgcn_permlane32_swap(b, b, false, false);  // halves, likewise
    return __int_as_float((lane & 32) ? r[0] : r[1]);
  }
}
// The smaller (lim = -inf) or larger (+inf) of x and its value in lane ^ M;
// no NaN.  A swap of a register with itself leaves both in every lane.
template <int M>
__device__ inline float med_lane(float x, int lane, float lim) {
  if constexpr (M == 16) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_int(x), __float_as_int(x), false, false);
    return __builtin_amdgcn_fmed3f(__int_as_float(r[0]), __int_as_float(r[1]), lim);
  } else if constexpr (M == 32) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_int(x), __float_as_int(x), false, false);
    return __builtin_amdgcn_fmed3f(__int_as_float(r[0]), __int_as_float(r[1]), lim);
  } else {
    return __builtin_amdgcn_fmed3f(x, xor_lane<M>(x, lane), lim);
  }
}

// MED: for values without NaN, minimum or maximum by a median with -inf or
// +inf (one instruction where a selection of the two takes three).
template <int NPL, int NIN, int NOUT, bool MED = false>
__device__ inline void sort_regs(const float (&in)[NIN], float* srt, int lane) {
  constexpr int NE = 64 * NPL;
  static_assert(NE <= 2048 && NIN <= NPL, "sort size");
  float v[NPL];
#pragma unroll
  for (int r = 0; r < NPL; ++r) v[r] = r < NIN ? in[r] : INFINITY;
  static_for<1, 12>([&](auto kl) FR_INLINE {  // k = 2^kl up to NE <= 2048
    constexpr int k = 1 << decltype(kl)::value;
    if constexpr (k <= NE) {
    const bool up = ((lane * NPL) & k) == 0 || k < NPL;
    static_for<0, decltype(kl)::value>([&](auto jl) FR_INLINE {  // j = k / 2, k / 4, ..., 1
      constexpr int j = k >> (1 + decltype(jl)::value);
      if constexpr (j >= NPL) {
        constexpr int m = j / NPL;
        const bool keep_lo = ((lane & m) == 0) == up;
        const float lim = keep_lo ? -INFINITY : INFINITY;
#pragma unroll
        for (int r = 0; r < NPL; ++r) {
          if constexpr (MED) {
            v[r] = med_lane<m>(v[r], lane, lim);
          } else {
            const float y = xor_lane<m>(v[r], lane);
            v[r] = keep_lo ? fminf(v[r], y) : fmaxf(v[r], y);
          }
        }
      } else {
#pragma unroll
        for (int r = 0; r < NPL; ++r) {
          if (r & j) continue;
          const bool u = k < NPL ? ((r & k) == 0) : up;
          const float a = v[r], b = v[r | j];
          if (MED && k >= NPL) {
            const float lim = up ? -INFINITY : INFINITY;
            v[r] = __builtin_amdgcn_fmed3f(a, b, lim);
            v[r | j] = __builtin_amdgcn_fmed3f(a, b, -lim);
          } else {
            v[r] = u ? fminf(a, b) : fmaxf(a, b);
            v[r | j] = u ? fmaxf(a, b) : fminf(a, b);
          }
        }
      }
    });
    }
  });
#pragma unroll
  for (int r = 0; r < NPL; ++r)
    if (lane * NPL + r < NOUT) srt[lane * NPL + r] = v[r];
}

// Run/zone/dependence emphasis features from per-entry sums.
struct Emph {
  long long n, si, si2, sj, sj2;  // totals (after emph_reduce)
  double si2j2;                   // total of c i^2 j^2, an integer below 2^53
  uint32_t pn, psi, psi2, psj, psj2;  // the lane's partial sums
  double psi2j2;
  double invj2, invi2, invi2j2, i2invj2, j2invi2, clogc;
};
// One matrix entry (its entropy term apart): count c (at most 13 (2r+1)^3 < 2^24) at level value i
// (<= 255) and index j (run length, zone size or dependence count, <= 1331).
// The sums of c, c i, c i^2, c j, c j^2 stay below 2^31 (at most 13|V| =
// 17,303 entries, c i <= 4.5e6, c i^2 <= 1.2e9): 32-bit arithmetic, 24-bit
// multiplies.  Sum c i^2 j^2 does not (a uniform 7^3 neighbourhood at level
// 255 gives 5.9e9 for the dependence counts): it is summed in FP64, where
// every term and partial sum is an integer below 2^53, so exactly and in
// any order.
__device__ inline void emph_add(Emph& a, uint32_t c, int i, int j) {
  const double ci = (double)c;
  const uint32_t ui = (uint32_t)i, uj = (uint32_t)j;
  const uint32_t i2u = __umul24(ui, ui), j2u = __umul24(uj, uj);
  const double i2 = (double)i2u, j2 = (double)j2u;
  const double ri2 = kInvSq.v[ui], rj2 = kInvSq.v[uj];
  const uint32_t cis = __umul24(c, ui), cjs = __umul24(c, uj);
  a.pn += c;
  a.psi += cis;
  a.psi2 += __umul24(cis, ui);
  a.psj += cjs;
  a.psj2 += __umul24(cjs, uj);
  a.psi2j2 += ci * (i2 * j2);
  a.invj2 += ci * rj2;
  a.invi2 += ci * ri2;
  a.invi2j2 += ci * ri2 * rj2;
  a.i2invj2 += ci * i2 * rj2;
  a.j2invi2 += ci * j2 * ri2;
}
// The integer sums fit in 32 bits (see emph_add); x1, x2: two more
// per-lane integer partials (squared row / column totals, each total below
// 2^31) reduced in the same pass.
__device__ inline void emph_reduce(Emph& a, long long& x1, long long& x2) {
  int vi[8] = {(int)a.pn, (int)a.psi, (int)a.psi2, (int)a.psj, (int)a.psj2, 0, (int)x1, (int)x2};
  wsum8i(vi);
  a.n = vi[0];
  a.si = vi[1];
  a.si2 = vi[2];
  a.sj = vi[3];
  a.sj2 = vi[4];
  x1 = vi[6];
  x2 = vi[7];
  double vd[8] = {a.invj2, a.invi2, a.invi2j2, a.i2invj2, a.j2invi2, a.clogc, a.psi2j2, 0.0};
  wsum8d(vd);
  a.invj2 = vd[0];
  a.invi2 = vd[1];
  a.invi2j2 = vd[2];
  a.i2invj2 = vd[3];
  a.j2invi2 = vd[4];
  a.clogc = vd[5];
  a.si2j2 = vd[6];
}
// The feature sums are VALU-issue bound.  Tables (map_device.h) for c log2 c
// and 1 / n^2, run and dependence sums taken along rows instead of entry by
// entry, and fewer wave reductions for the co-occurrence features: 12.1 k ->
// 10.8 k VALU instructions a voxel and 22.4 -> 20.9 ms for the 1 M-voxel
// radius-3 workload, 6.3 k -> 5.4 k and 1.39 -> 1.27 ms for the 100 k-voxel
// radius-2 one.
// The present level of a lane in a pass over a [level][size] table: with at
// most 32 levels, the two halves of the wave share a level and take every
// other column; with more, a lane takes the whole row.
template <int LMAX>
struct LevelRow {
  static constexpr int H = LMAX <= 32 ? 2 : 1;  // lanes per level
  int l, part;   // compact level; first column of the lane
  bool ok;       // the level is present
  uint32_t i;    // level value
  double i2, ri2;  // i^2, 1 / i^2
  __device__ LevelRow(const uint8_t* lval, int L, int lane) {
    l = H == 2 ? lane & 31 : lane;
    part = H == 2 ? lane >> 5 : 0;
    ok = l < L;
    i = ok ? lval[l] : 1u;
    i2 = (double)__umul24(i, i);
    ri2 = kInvSq.v[i];
  }
};
// Sums over the columns of a lane's row (or half row).
struct RowSums {
  uint32_t n, j1, j2;  // of c, c j, c j^2
  double invj2, clogc;  // of c / j^2, c log2 c
};
template <int R>
__device__ inline void row_add(RowSums& r, uint32_t c, uint32_t j) {
  r.n += c;
  r.j1 += __umul24(c, j);
  r.j2 += __umul24(c, __umul24(j, j));
  r.invj2 = fma((double)c, kInvSq.v[j], r.invj2);
  r.clogc += xlog2x<R>(c);
}
// The emphasis sums of the lane's entries: every one is a row sum times a
// power of the level (the bounds are those of emph_add).
template <int LMAX>
__device__ inline void emph_rows(Emph& a, const RowSums& r, const LevelRow<LMAX>& lr) {
  const double n = (double)r.n, j2 = (double)r.j2;
  a.pn = r.n;
  a.psi = __umul24(r.n, lr.i);
  a.psi2 = __umul24(a.psi, lr.i);
  a.psj = r.j1;
  a.psj2 = r.j2;
  a.psi2j2 = j2 * lr.i2;
  a.invj2 = r.invj2;
  a.invi2 = n * lr.ri2;
  a.invi2j2 = r.invj2 * lr.ri2;
  a.i2invj2 = r.invj2 * lr.i2;
  a.j2invi2 = j2 * lr.ri2;
  a.clogc = r.clogc;
}
// The row total of the lane's level (both halves of a split row).
template <int LMAX>
__device__ inline uint32_t row_total(uint32_t n) {
  if constexpr (LMAX > 32) return n;
  const auto r = __builtin_amdgcn_permlane32_swap((int)n, (int)n, false, false);
  return (uint32_t)(r[0] + r[1]);
}

// The 16-value set shared by GLRLM and GLSZM: gln/rln are the sums of
// squared row/column totals; units = Np (13|V| for runs) or Nv (|V|).
template <typename O>
__device__ inline void emph16(const Emph& a, long long gln, long long rln, double units, double nlogn, O* f) {
  const double N = (double)a.n;
  const double rN = rcp64(N), rN2 = rN * rN;  // one reciprocal; the rest multiply
  f[0] = (O)(a.invj2 * rN);
  f[1] = (O)((double)a.sj2 * rN);
  f[2] = (O)((double)gln * rN);
  f[3] = (O)((double)gln * rN2);
  f[4] = (O)((double)rln * rN);
  f[5] = (O)((double)rln * rN2);
  f[6] = (O)fdiv(N, units);
  f[7] = (O)((double)(a.n * a.si2 - a.si * a.si) * rN2);
  f[8] = (O)((double)(a.n * a.sj2 - a.sj * a.sj) * rN2);
  f[9] = (O)((nlogn - a.clogc) * rN);  // nlogn = N log2 N
  f[10] = (O)(a.invi2 * rN);
  f[11] = (O)((double)a.si2 * rN);
  f[12] = (O)(a.invi2j2 * rN);
  f[13] = (O)(a.i2invj2 * rN);
  f[14] = (O)(a.j2invi2 * rN);
  f[15] = (O)(a.si2j2 * rN);
}

// Instances that search the MCC to the finer width.
template <int R, int MODE>
constexpr bool kFineMcc = R > 3 || MODE != kPlain;

// The 16 GLRLM maps of the counts glrlm [L][S] (compact level, run length
// - 1).  Rows by lane (LevelRow): the sums over a level's lengths first,
// the level's powers once a row; the tables' loads together.
template <int R, int LMAX, typename O>
__device__ FR_INLINE inline void runs_features(const uint32_t* glrlm, const LevelRow<LMAX>& lr, int L, int lane,
                                               double units, O* f) {
  constexpr int S = 2 * R + 1, H = LevelRow<LMAX>::H, NT = (S + H - 1) / H;
  RowSums rs = {};
  long long gln = 0, rln = 0;
  uint32_t cs[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int j = t * H + lr.part;
    cs[t] = lr.ok && j < S ? glrlm[lr.l * S + j] : 0u;
  }
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int j = t * H + lr.part;
    const uint32_t c = cs[t];
    row_add<R>(rs, c, (uint32_t)(j < S ? j : 0) + 1u);
    // the length's total over the levels: in the last lane of each half
    // wave (H 2, one column per half) or of the wave
    int v = (int)c;
    v += __builtin_amdgcn_mov_dpp(v, 0xb1, 0xf, 0xf, true);
    v += __builtin_amdgcn_mov_dpp(v, 0x4e, 0xf, 0xf, true);
    v += __builtin_amdgcn_mov_dpp(v, 0x141, 0xf, 0xf, true);
    v += __builtin_amdgcn_mov_dpp(v, 0x140, 0xf, 0xf, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);
    if constexpr (H == 1) v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);
    rln += (long long)v * v;
  }
  rln = (H == 2 ? (lane & 31) == 31 : lane == 63) ? rln : 0;
  const uint32_t tot = row_total<LMAX>(rs.n);
  if (lr.part == 0) gln = (long long)tot * tot;
  Emph er = {};
  emph_rows(er, rs, lr);
  emph_reduce(er, gln, rln);
  emph16(er, gln, rln, units, xlog2x<R>((uint32_t)er.n), f);
}

template <typename T, int R, int LMAX, bool DEBUG, bool MOUT = false, int MODE = kPlain>
__device__ __attribute__((always_inline)) inline void map_voxel(Smem<R, LMAX, MOUT>& sm, const MapArgs& a, int32_t lin, int64_t it,
                                                               int& ns, int& nq, bool& big, AvgMem* av = nullptr) {
  // an AnyRaw instance dumps the matrices only when asked to
  const bool dbg = DEBUG && (!std::is_same_v<T, AnyRaw> || a.d_glcm != nullptr);
  using SM = Smem<R, LMAX, MOUT>;
  constexpr int S = SM::S, C = SM::C, CP = SM::CP, SP = SM::SP, HT = SM::HT;
  constexpr int NIT = CP / 64;
  const int lane = opaque_lane();
  const uint32_t fam = a.families;
  const bool fFO = fam & 1u, fGLCM = fam & 2u, fGLRLM = fam & 4u, fGLSZM = fam & 8u,
             fGLDM = fam & 16u, fNGTDM = fam & 32u;
  const int nx = a.nx, ny = a.ny, nz = a.nz;
  const int cx = lin % nx, cy = (lin / nx) % ny, cz = lin / (nx * ny);

  // ---- gather the cube ------------------------------------------------
  // the raw values (xq) and levels (gl) stay in registers until the
  // first-order maps are done; the sums for the moments are taken here
  uint8_t* lflag = reinterpret_cast<uint8_t*>(sm.u.a.glcm);  // level present in V (before the counts)
  clear16(lflag, SM::LV, lane);
  clear16(sm.nb, SM::PC + SM::CWB, lane);
  int K = 0;
  float xq[NIT];
  double s1 = 0.0, s2 = 0.0;
  // every load of the cube first (levels and raw values of the positions
  // inside the image, whatever their level), so that they are all in
  // flight together instead of one round trip per position
  // The coordinates come from a table, and one comparison a byte (7 bits a
  // coordinate, the top one for the sign) tests them against the part of the
  // cube that lies inside the image.
  int gl[NIT];
  float xl[NIT];
  {
    constexpr uint32_t kTop = 0x808080u;
    auto first = [](int at) FR_INLINE { return (uint32_t)max(0, R - at); };
    auto last = [](int at, int n) FR_INLINE { return (uint32_t)min(S - 1, n - 1 - at + R); };
    const uint32_t lo = first(cx) | first(cy) << 8 | first(cz) << 16;
    const uint32_t hi = last(cx, nx) | last(cy, ny) << 8 | last(cz, nz) << 16 | kTop;
    // an image holds less than 2^31 voxels: the index is exact modulo 2^32
    const uint32_t unx = (uint32_t)nx, unxy = unx * (uint32_t)ny;
    const uint32_t corner = (uint32_t)lin - (uint32_t)R * (unxy + unx + 1u);
#pragma unroll
    for (int q = 0; q < NIT; ++q) {
      const uint32_t pos = kPos<R>.v[lane + 64 * q];
      gl[q] = 0;
      xl[q] = INFINITY;
      if (((((pos | kTop) - lo) & (hi - (pos & 0xffffffu))) & kTop) == kTop) {
        const uint32_t gi = corner + ((pos >> 16) & 0xffu) * unxy + ((pos >> 8) & 0xffu) * unx + (pos & 0xffu);
        gl[q] = a.levels[gi];
        xl[q] = raw_at<T>(a, gi);
      }
    }
  }
#pragma unroll
  for (int q = 0; q < NIT; ++q) {
    const int g = gl[q];
    const float xr = g ? xl[q] : INFINITY;
    if (g) lflag[g] = 1;
    xq[q] = xr;
    if (fFO) {
      const double xd = (double)(g ? xl[q] : 0.f);
      s1 += xd;
      s2 = fma(xd, xd, s2);
    }
    K += __popcll(__ballot(g != 0));
  }
  __syncthreads();

  // ---- local level compaction -----------------------------------------
  int L;
  uint8_t* lmap = reinterpret_cast<uint8_t*>(sm.u.a.same);  // level -> compact index
  static_assert(sizeof(SM::U::A::same) >= (size_t)SM::LV, "the level map fits the masks' place");
  {
    const uint32_t fw = lane < SM::LVW ? ((const uint32_t*)lflag)[lane] : 0u;
    const int f0 = (fw & 0xffu) != 0, f1 = (fw & 0xff00u) != 0, f2 = (fw & 0xff0000u) != 0,
              f3 = (fw & 0xff000000u) != 0;
    int pre = wscan_excl(f0 + f1 + f2 + f3, lane, &L);
    if (f0) { lmap[4 * lane] = (uint8_t)pre; sm.lval[pre++] = (uint8_t)(4 * lane); }
    if (f1) { lmap[4 * lane + 1] = (uint8_t)pre; sm.lval[pre++] = (uint8_t)(4 * lane + 1); }
    if (f2) { lmap[4 * lane + 2] = (uint8_t)pre; sm.lval[pre++] = (uint8_t)(4 * lane + 2); }
    if (f3) { lmap[4 * lane + 3] = (uint8_t)pre; sm.lval[pre++] = (uint8_t)(4 * lane + 3); }
  }
  if constexpr (C > LMAX) {
    if (L > LMAX) {  // more present levels than these tables hold: a wider pass maps it
      if (lane == 0) {
        const int p = (int)(it + a.key0) % kParts;
        a.over[part_base(a.part_n, p) + atomicAdd(&a.over_count[p * kPartStride], 1)] = make_int2(a.over_job, (int)it);
      }
      return;
    }
  }
  // clear the L-sized tables
  clear16(sm.u.a.glcm, SM::glcm_words(L) * 4, lane);
  static_assert(offsetof(typename SM::U::A, same) % 16 == 0 && (SM::kGlcmWords * 4 + 15) / 16 * 16 <= (int)offsetof(typename SM::U::A, same),
                "clearing the counts stays clear of the level map");
  clear16(sm.u.a.gldm, L * SM::kGldmWords * 4, lane);
  if (lane < L) {
    sm.hist[lane] = 0;
    sm.pxc[lane] = 0;
    sm.u.a.ngn[lane] = 0;
    sm.u.a.ngS[lane] = 0ull;
  }
  __syncthreads();

  // compact levels into the cubes, row sums of the level values, level
  // histogram
  uint16_t* lev = reinterpret_cast<uint16_t*>(sm.u.a.parent);  // position c at c + 1: level * 32 + 1, or 0
#pragma unroll
  for (int q = 0; q < NIT; ++q) {
    const int c = lane + 64 * q;
    lev[c + 1] = (uint16_t)(gl[q] * 32 + min(gl[q], 1));
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < NIT; ++q) {
    const int c = lane + 64 * q;
    const int g = gl[q];
    int l1 = 0;
    if (g) {
      const int l = lmap[g];
      l1 = l + 1;
      atomicAdd(&sm.hist[l], 1u);
    }
    gl[q] = l1;
    sm.cl[c] = (uint8_t)l1;
    if (c < C) {
      const uint32_t pos = kPos<R>.v[c];
      const int x = (int)(pos & 0xffu), row = (int)(pos >> 24);
      const uint32_t left = lev[c], right = lev[c + 2];
      sm.clp()[row * SM::SX + (x + 1)] = (uint8_t)l1;
      sm.cw()[row * S + x] = (uint16_t)((x > 0 ? left : 0u) + (g * 32 + min(g, 1)) + (x < S - 1 ? right : 0u));
    }
  }
  __syncthreads();

  // ---- first order ----------------------------------------------------
  // Levels grow with the raw value, so the ten order statistics lie in at
  // most ten levels: only the values of those are sorted (typically a
  // quarter of V), not V.  With a NaN among the values, or too many to
  // sort this way, V is sorted as it stands.  (Sorting V had been about
  // 1,000 VALU instructions a voxel at radius 3, this is about 300.)
  const double Kd = (double)K;
  if (fFO) {
    const double rKd = rcp64(Kd);  // one reciprocal; the rest multiply
    float* srt = reinterpret_cast<float*>(sm.u.a.parent);
    const double rank[5] = {(double)(K - 1) * 0.10, (double)(K - 1) * 0.25, (double)(K - 1) * 0.50,
                            (double)(K - 1) * 0.75, (double)(K - 1) * 0.90};
    int at0[5], at1[5];  // positions of the ranks' two order statistics in srt
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      at0[k] = __builtin_amdgcn_readfirstlane((int)rank[k]);
      at1[k] = min(at0[k] + 1, K - 1);
    }
    float lo = INFINITY, hi = -INFINITY;
    bool nan = false;
#pragma unroll
    for (int q = 0; q < NIT; ++q) {
      if (gl[q]) {
        lo = fminf(lo, xq[q]);
        hi = fmaxf(hi, xq[q]);
        nan |= xq[q] != xq[q];
      }
    }
    const int h = lane < L ? (int)sm.hist[lane] : 0;
    int M = K;  // values to sort
    bool part = __ballot(nan) == 0ull;
    if constexpr (R > 1) {
      if (part) {
        int tot;
        const int pre = wscan_excl(h, lane, &tot);
        bool mark = false;
#pragma unroll
        for (int k = 0; k < 5; ++k)
          mark |= (uint32_t)(at0[k] - pre) < (uint32_t)h || (uint32_t)(at1[k] - pre) < (uint32_t)h;
        const uint64_t bins = __ballot(mark);
        const int shift = wscan_excl(mark ? h : 0, lane, &M) - pre;
        constexpr int kMost = R == 2 ? 128 : R == 3 ? 256 : 512;
        part = M <= kMost;
        if (part) {
          int n = 0;
#pragma unroll
          for (int q = 0; q < NIT; ++q) {
            bool in = false;
            if (gl[q]) in = LMAX <= 32 ? ((uint32_t)bins >> (gl[q] - 1)) & 1u : (bins >> (gl[q] - 1)) & 1ull;
            const uint64_t m = __ballot(in);
            if (in) srt[n + below(m)] = xq[q];
            n += __popcll(m);
          }
          // a rank's place among the kept values: that of its level
#pragma unroll
          for (int k = 0; k < 5; ++k) {
            const uint64_t m0 = __ballot((uint32_t)(at0[k] - pre) < (uint32_t)h);
            const uint64_t m1 = __ballot((uint32_t)(at1[k] - pre) < (uint32_t)h);
            at0[k] += __builtin_amdgcn_readlane(shift, __ffsll((unsigned long long)m0) - 1);
            at1[k] += __builtin_amdgcn_readlane(shift, __ffsll((unsigned long long)m1) - 1);
          }
          __syncthreads();
          auto sort = [&](auto npl) FR_INLINE {
            constexpr int N = decltype(npl)::value;
            float v[N];
#pragma unroll
            for (int r = 0; r < N; ++r) v[r] = lane + 64 * r < M ? srt[lane + 64 * r] : INFINITY;
            sort_regs<N, N, 64 * N, true>(v, srt, lane);
          };
          if (M <= 64)
            sort(std::integral_constant<int, 1>{});
          else if (M <= 128)
            sort(std::integral_constant<int, 2>{});
          else if constexpr (R > 2) {
            if (R == 3 || M <= 256)
              sort(std::integral_constant<int, 4>{});
            else if constexpr (R > 3)
              sort(std::integral_constant<int, 8>{});
          }
        }
      }
    } else {
      if (part) sort_regs<1, 1, 64, true>(xq, srt, lane);
    }
    if (!part) sort_regs<SP / 64, NIT, CP>(xq, srt, lane);
    __syncthreads();
    if (!part) {
#pragma unroll
      for (int q = 0; q < NIT; ++q) {
        const int c = lane + 64 * q;
        xq[q] = srt[c];
        gl[q] = c < K;
      }
    }
    const float mnf = part ? wfold_f(lo, [](float x, float y) { return __builtin_amdgcn_fmed3f(x, y, -INFINITY); }) : srt[0];
    const float mxf = part ? wfold_f(hi, [](float x, float y) { return __builtin_amdgcn_fmed3f(x, y, INFINITY); }) : srt[K - 1];
    double pct[5];
#pragma unroll
    for (int k = 0; k < 5; ++k) {  // (the second statistic equals the first where there is none)
      const double a0 = srt[at0[k]], a1 = srt[at1[k]];
      pct[k] = at1[k] == at0[k] ? a0 : a0 + (rank[k] - floor(rank[k])) * (a1 - a0);
    }
    const double mn = mnf, mx = mxf;
    const double p10 = pct[0], p25 = pct[1], p50 = pct[2], p75 = pct[3], p90 = pct[4];
    double ent = 0.0, uni = 0.0;
    if (lane < L) {
      const double p = (double)h * rKd;
      ent = xlog2x<R>((uint32_t)h);
      uni = p * p;
    }
    double r1[8] = {s1, s2, ent, uni, 0.0, 0.0, 0.0, 0.0};
    wsum8d(r1);
    const double S1 = r1[0], S2 = r1[1];
    // (no value at all, where every voxel is a NaN that got no level: entropy 0)
    ent = K ? (xlog2x<R>((uint32_t)K) - r1[2]) * rKd : 0.0;
    uni = r1[3];
    const double mu = S1 * rKd;
    double m2 = 0, m3 = 0, m4 = 0, mad = 0, rs = 0, rn = 0;
#pragma unroll
    for (int q = 0; q < NIT; ++q) {
      if (gl[q]) {
        const double x = xq[q];
        const double d = x - mu;
        const double d2 = d * d;
        m2 += d2;
        m3 += d2 * d;
        m4 += d2 * d2;
        mad += fabs(d);
        if (x >= p10 && x <= p90) {
          rs += x;
          rn += 1.0;
        }
      }
    }
    double r2[8] = {m2, m3, m4, mad, rs, rn, 0.0, 0.0};
    wsum8d(r2);
    m2 = r2[0] * rKd;
    m3 = r2[1] * rKd;
    m4 = r2[2] * rKd;
    mad = r2[3] * rKd;
    rs = r2[4];
    rn = r2[5];
    double rmad = NAN;
    if (rn > 0.0) {
      const double rrn = rcp64(rn), rmu = rs * rrn;
      double acc = 0.0;
#pragma unroll
      for (int q = 0; q < NIT; ++q) {
        if (gl[q]) {
          const double x = xq[q];
          if (x >= p10 && x <= p90) acc += fabs(x - rmu);
        }
      }
      rmad = wsum(acc) * rrn;
    }
    const bool flat = (mn == mx);
    if (lane == 0) {
      float* f = sm.early;
      f[0] = (float)S2;
      f[1] = (float)(a.voxel_volume * S2);
      f[2] = (float)ent;
      f[3] = (float)mn;
      f[4] = (float)p10;
      f[5] = (float)p90;
      f[6] = (float)mx;
      f[7] = (float)mu;
      f[8] = (float)p50;
      f[9] = (float)(p75 - p25);
      f[10] = (float)(mx - mn);
      f[11] = (float)mad;
      f[12] = (float)rmad;
      f[13] = (float)(S2 > 0.0 && S2 < (double)INFINITY ? fsqrt(S2 * rKd) : S2 * rKd);
      f[14] = flat ? 0.f : (float)fdiv(m3, m2 * fsqrt(m2));  // m2^1.5
      f[15] = flat ? 0.f : (float)(fdiv(m4, m2 * m2) - 3.0);
      f[16] = (float)m2;
      f[17] = (float)uni;
    }
    __syncthreads();
  }

  // ---- counting pass: lane per cube position --------------------------
  // The neighbourhood as nine rows of three compact levels, each out of two
  // aligned words of the zero-bordered cube (no bounds tests; byte 3 is not
  // looked at; unaligned 4-byte reads measured 1.3 times the kernel's time).
  // Compact levels plus one are below 128: adding 0x7f to each byte sets
  // its top bit where the byte is not zero.  Level sums and neighbour
  // counts are nine more reads.  With the sorted values above: 7.9 k ->
  // 6.0 k VALU instructions a voxel at radius 3 (16.6 -> 14.9 ms for 1 M
  // voxels), 4.0 k -> 3.7 k at radius 2.
  constexpr int SQ = SM::SQ;
  // The variants.  A tolerance: the levels that a level depends on are
  // neighbours of it in the (sorted) list of the present ones, so a
  // neighbour is tested by its compact level, all of a row at a time.
  [[maybe_unused]] const bool tolerant = MODE != kPlain && fGLDM && a.opt.gldm_alpha > 0;
  [[maybe_unused]] uint32_t* range = sm.u.a.parent;  // per level: the first compact level + 1, the last one's << 8
  if constexpr (MODE != kPlain) {
    if (tolerant) {
      const int g = lane < L ? (int)sm.lval[lane] : 0;
      uint32_t first = 1, last = 0;
      for (int m = 0; m < L; ++m) {
        const int d = __builtin_amdgcn_readlane(g, m) - g;
        first += d < -a.opt.gldm_alpha;
        last += d <= a.opt.gldm_alpha;
      }
      if (lane < L) range[lane] = first | last << 8;
      __syncthreads();
    }
  }
  // at distance 1 the merged GLCM is the plain one
  const bool nearest = MODE == kPlain || (MODE == kMerged && a.opt.glcm_dist == 1);
#pragma unroll 1
  for (int q = 0; q < NIT; ++q) {
    const int c = lane + 64 * q;
    const uint32_t l1 = (c < C) ? sm.cl[c] : 0u;
    if (l1) {
      const uint32_t pos = kPos<R>.v[c];
      const int x = (int)(pos & 0xffu), row0 = (int)(pos >> 24);
      const uint32_t* words = reinterpret_cast<const uint32_t*>(&sm.clp()[row0 * SM::SX + (x & ~3)]);
      const uint16_t* sums = &sm.cw()[row0 * S + x];
      uint32_t rw[9], wsum = 0;
#pragma unroll
      for (int r = 0; r < 9; ++r) {  // rows opposite to the forward ones, forward rows, the own one
        const int dy = r == 8 ? 0 : r < 4 ? -fdy(r) : fdy(r - 4), dz = r == 8 ? 0 : r < 4 ? -fdz(r) : fdz(r - 4);
        const int o = dz * SQ + dy;
        rw[r] = __builtin_amdgcn_alignbyte(words[o * (SM::SX / 4) + 1], words[o * (SM::SX / 4)], (uint32_t)x & 3u);
        wsum += sums[o * S];
      }
      const uint32_t l4 = l1 * 0x01010101u;
      uint32_t ne = 0;  // bit r of byte dx + 1: row r's level differs
#pragma unroll
      for (int r = 0; r < 8; ++r) ne = (ne >> 1) | (((rw[r] ^ l4) + 0x7f7f7f7fu) & 0x80808080u);
      const uint32_t own = ~((rw[8] ^ l4) + 0x7f7f7f7fu);
      const uint32_t same = (~ne & 0x00ffffffu) | ((own & 0x80u) << 20) | ((own & 0x800000u) << 8);
      const int l = (int)l1 - 1, g = sm.lval[l];
      const int cnt = (int)(wsum & 31u) - 1, lsum = (int)(wsum >> 5) - g;
      sm.u.a.same[c] = same;
      if (nearest && fGLCM) {
        if constexpr (SM::kFullGlcm) {
          uint32_t* row = &sm.u.a.glcm[(l >> 1) * SM::kRowWords];
          const int shift = (l & 1) << 4;
          const uint32_t one = 1u << shift;
          // Lanes that add to one word take turns, a cycle each.  Where half
          // the positions have four equal forward neighbours or more
          // (smooth images), those are counted together and the neighbours
          // outside V not at all: the GLCM of 30,000 voxels of a uniform
          // image at radius 3 takes 304 us, 538 without this (noise in 8
          // levels 364 and 382, in more the same).
          const int eq = __popc(same & kFwdBits);
          if (2 * __popcll(__ballot(eq >= 4)) >= __popcll(__ballot(true))) {
#pragma unroll
            for (int d = 0; d < 13; ++d) {
              const uint32_t m1 = d < 12 ? (rw[4 + d % 4] >> (8 * (d / 4))) & 0xffu : (rw[8] >> 16) & 0xffu;
              if (m1 != 0 && m1 != l1) atomicAdd(&row[m1], one);
            }
            if (eq) atomicAdd(&row[l1], (uint32_t)eq << shift);
          } else {
#pragma unroll
            for (int d = 0; d < 12; ++d) atomicAdd(&row[(rw[4 + d % 4] >> (8 * (d / 4))) & 0xffu], one);
            atomicAdd(&row[(rw[8] >> 16) & 0xffu], one);
          }
        } else {
#pragma unroll
          for (int d = 0; d < 13; ++d) {
            const uint32_t m1 = d < 12 ? (rw[4 + d % 4] >> (8 * (d / 4))) & 0xffu : (rw[8] >> 16) & 0xffu;
            if (m1 != 0 && m1 != l1) {
              const int m = (int)m1 - 1;
              gadd(sm.u.a.glcm, l < m ? tri(l, m) : tri(m, l), 1u);
            }
          }
          const int eq = __popc(same & kFwdBits);
          if (eq) gadd(sm.u.a.glcm, tri(l, l), 2u * eq);
        }
        atomicAdd(&sm.pxc[l], (uint32_t)cnt);
      }
      if (fGLDM) {
        int dep = __popc(same);
        if constexpr (MODE != kPlain) {
          if (tolerant) {
            // top bit of a byte: not below the first level of the range, not
            // above the last (bytes of 0 lie below)
            const uint32_t w = range[l], lo4 = (w & 0xffu) * 0x01010101u, hi4 = (0x7fu - (w >> 8)) * 0x01010101u;
            auto inside = [&](uint32_t r) FR_INLINE { return ((r | 0x80808080u) - lo4) & ~(r + hi4) & 0x00808080u; };
            uint32_t in = 0;
#pragma unroll
            for (int r = 0; r < 8; ++r) in = (in >> 1) | inside(rw[r]);
            dep = __popc(in) + __popc(inside(rw[8]) & 0x00800080u);
          }
        }
        gadd(sm.u.a.gldm, l * (2 * SM::kGldmWords) + dep, 1u);
      }
      if (fNGTDM && cnt) {
        atomicAdd(&sm.u.a.ngn[l], 1u);
        const int dd = g * cnt - lsum;
        atomicAdd(&sm.u.a.ngS[l], (unsigned long long)(dd < 0 ? -dd : dd) * kLcmOver[cnt]);
      }
    }
  }
  __syncthreads();

  // GLCM of the variants.  The neighbour's compact level + 1 (0: none) at
  // `dist` along a direction, its bounds tested.
  [[maybe_unused]] auto neighbour = [&](uint32_t pos, int dist, int dx, int dy, int dz) FR_INLINE {
    const uint32_t ux = (pos & 0xffu) + dist * dx, uy = ((pos >> 8) & 0xffu) + dist * dy, uz = ((pos >> 16) & 0xffu) + dist * dz;
    const bool in = ux < (uint32_t)S && uy < (uint32_t)S && uz < (uint32_t)S;
    const uint32_t m1 = sm.cl[in ? (uz * S + uy) * S + ux : 0u];
    return in ? (int)m1 : 0;
  };
  // One direction's pairs (kAveraged); an entry off the diagonal is added
  // once, at (min, max).
  [[maybe_unused]] auto count_direction = [&](int d) FR_INLINE {
#pragma unroll 1
    for (int q = 0; q < NIT; ++q) {
      const int c = lane + 64 * q;
      const int l1 = (c < C) ? sm.cl[c] : 0;
      if (l1) {
        const int m1 = neighbour(kPos<R>.v[c], a.opt.glcm_dist, kDir[d][0], kDir[d][1], kDir[d][2]);
        if (m1) {
          gpair<SM>(sm.u.a.glcm, l1 - 1, m1 - 1);
          atomicAdd(&sm.pxc[l1 - 1], 1u);
          atomicAdd(&sm.pxc[m1 - 1], 1u);
        }
      }
    }
    __syncthreads();
  };
  if constexpr (MODE == kMerged) {
    // every direction's pairs, a position's neighbours read together; the
    // row sums from the table
    if (fGLCM && !nearest) {
#pragma unroll 1
      for (int q = 0; q < NIT; ++q) {
        const int c = lane + 64 * q;
        const int l1 = (c < C) ? sm.cl[c] : 0;
        if (l1) {
          const uint32_t pos = kPos<R>.v[c];
          int m1[13];
#pragma unroll
          for (int d = 0; d < 13; ++d) m1[d] = neighbour(pos, a.opt.glcm_dist, fdx(d), fdy(d), fdz(d));
#pragma unroll
          for (int d = 0; d < 13; ++d)
            if (m1[d]) gpair<SM>(sm.u.a.glcm, l1 - 1, m1[d] - 1);
        }
      }
      __syncthreads();
      if (lane < L) {
        uint32_t sum = 0;
        for (int m = 0; m < L; ++m) sum += gsym<SM>(sm.u.a.glcm, lane, m);
        sm.pxc[lane] = sum;
      }
      __syncthreads();
    }
  }

  const LevelRow<LMAX> lrow(sm.lval, L, lane);
  if (dbg) {
    const int ng = a.ng;
    for (int e = lane; e < L * 27; e += 64) {
      const int l = e / 27, j = e % 27;
      a.d_gldm[it * ng * 27 + (int64_t)(sm.lval[l] - 1) * 27 + j] = (int32_t)gget(sm.u.a.gldm, l * (2 * SM::kGldmWords) + j);
    }
    if (lane < L) {
      const int64_t o = it * ng + (sm.lval[lane] - 1);
      a.d_ngn[o] = (int32_t)sm.u.a.ngn[lane];
      a.d_ngS[o] = (int64_t)sm.u.a.ngS[lane];
      a.d_hist[o] = (int32_t)sm.hist[lane];
    }
  }

  // ---- GLDM -----------------------------------------------------------
  if (fGLDM) {
    Emph ed = {};
    if (L <= 2) {  // a level to each half of the wave, a dependence to a lane
      const int l = lane >> 5, d = lane & 31;
      const uint32_t c = l < L && d < 27 ? gget(sm.u.a.gldm, l * (2 * SM::kGldmWords) + d) : 0u;
      emph_add(ed, c, l < L ? sm.lval[l] : 1, d + 1);
      ed.clogc = xlog2x<R>(c);
    } else {
      // rows by lane, as the runs; two dependences a word
      constexpr int H = LevelRow<LMAX>::H, NT = (14 + H - 1) / H;
      RowSums rs = {};
      uint32_t cs[NT];
#pragma unroll
      for (int t = 0; t < NT; ++t)
        cs[t] = lrow.ok ? sm.u.a.gldm[lrow.l * SM::kGldmWords + t * H + lrow.part] : 0u;
      auto add = [&](int t) FR_INLINE {
        const uint32_t w = (uint32_t)(t * H + lrow.part);
        row_add<R>(rs, cs[t] & 0xffffu, 2u * w + 1u);
        row_add<R>(rs, cs[t] >> 16, 2u * w + 2u);
      };
      // up to 8 (of 27) equal neighbours together, each more if any level has it
      constexpr int T0 = 4 / H;
      uint32_t rest = 0;
#pragma unroll
      for (int t = T0; t < NT; ++t) rest |= cs[t];
#pragma unroll
      for (int t = 0; t < T0; ++t) add(t);
      if (__ballot(rest != 0u) != 0ull) {
#pragma unroll
        for (int t = T0; t < NT; ++t)
          if (__ballot(cs[t] != 0u) != 0ull) add(t);
      }
      emph_rows(ed, rs, lrow);
    }
    // voxels per dependence: the columns' sums, two (16 bits each) to a lane
    // of each row of 16, which takes every fourth level.  (They had been
    // counted by atomics, on few addresses.  With this, one or two levels by
    // lanes and no passes over dependences that no level has, GLDM maps of
    // 30,000 voxels of a uniform image at radius 3 take 197 us, 228 before;
    // of blocks 198 and 214; of 60,000 of noise in 32 levels 262 and 290.)
    uint32_t col = 0;
    if ((lane & 15) < 14) {
#pragma unroll 4
      for (int l = lane >> 4; l < L; l += 4) col += sm.u.a.gldm[l * SM::kGldmWords + (lane & 15)];
    }
    col = (uint32_t)fold16i((int)col, (int)col);
    col = (uint32_t)fold32i((int)col, (int)col);
    long long gln = 0, dn = 0;
    if (lane < L) {
      const long long t = sm.hist[lane];
      gln = t * t;
    }
    if (lane < 14) dn = (long long)(__umul24(col & 0xffffu, col & 0xffffu) + __umul24(col >> 16, col >> 16));
    emph_reduce(ed, gln, dn);
    const double N = (double)ed.n;
    const double rN = rcp64(N), rN2 = rN * rN;  // one reciprocal; the rest multiply
    if (lane == 0) {
      float* f = sm.early + kNFO;
      f[0] = (float)(ed.invj2 * rN);
      f[1] = (float)((double)ed.sj2 * rN);
      f[2] = (float)((double)gln * rN);
      f[3] = (float)((double)dn * rN);
      f[4] = (float)((double)dn * rN2);
      f[5] = (float)((double)(ed.n * ed.si2 - ed.si * ed.si) * rN2);
      f[6] = (float)((double)(ed.n * ed.sj2 - ed.sj * ed.sj) * rN2);
      f[7] = (float)((xlog2x<R>((uint32_t)ed.n) - ed.clogc) * rN);
      f[8] = (float)(ed.invi2 * rN);
      f[9] = (float)((double)ed.si2 * rN);
      f[10] = (float)(ed.invi2j2 * rN);
      f[11] = (float)(ed.i2invj2 * rN);
      f[12] = (float)(ed.j2invi2 * rN);
      f[13] = (float)(ed.si2j2 * rN);
    }
  }

  // ---- NGTDM ----------------------------------------------------------
  if (fNGTDM) {
    long long n_i = 0, sum_n = 0, sum_ni = 0, sum_ni2 = 0, pres = 0, pj = 0, pj2 = 0;
    double s_i = 0.0, ps_acc = 0.0;
    int i_lev = 0, anys = 0;
    // s_i as a double in place of its integer numerator (no later reader of
    // the integer), so the pairwise terms read it converted once per level
    double* sd = reinterpret_cast<double*>(sm.u.a.ngS);
    if (lane < L) {
      n_i = sm.u.a.ngn[lane];
      const unsigned long long Si = sm.u.a.ngS[lane];
      i_lev = sm.lval[lane];
      s_i = (double)Si * kRcpLcm26;
      sd[lane] = s_i;
      if (n_i) {
        pres = 1;
        pj = i_lev;
        pj2 = (long long)i_lev * i_lev;
        anys = Si != 0ull;
      }
      sum_n = n_i;
      sum_ni = n_i * i_lev;
      sum_ni2 = n_i * i_lev * i_lev;
      ps_acc = (double)n_i * s_i;
    }
    // pairwise terms over present levels: both terms are symmetric in
    // (i, j) and vanish for i = j, so the pairs i < j, enumerated compactly
    // (e = j (j - 1) / 2 + i), one per lane, count twice
    long long bden = 0;
    double cplx = 0.0;
    __syncthreads();  // sd complete
    {
      const int npair = L * (L - 1) / 2;
      for (int e0 = 0; e0 < npair; e0 += 64) {
        const int e = e0 + lane;
        if (e < npair) {
          const uint32_t rc = kTri.v[e];
          const int i = (int)(rc & 0xffu), jc = (int)(rc >> 8) + 1;
          // counts <= (2r+1)^3 and levels <= 255: the products fit in 32 bits
          const int ni = (int)sm.u.a.ngn[i], nj = (int)sm.u.a.ngn[jc];
          if (ni && nj) {
            const int il = sm.lval[i], jl = sm.lval[jc];
            const int t = il * ni - jl * nj;
            bden += 2 * (t < 0 ? -t : t);
            const double si = sd[i], sj = sd[jc];
            cplx += 2.0 * fabs((double)(il - jl)) * ((double)ni * si + (double)nj * sj) *
                    frcp((double)(ni + nj));
          }
        }
      }
    }
    // every integer total is below 2^31: |V| <= 1,331, at most 64 present
    // levels of value <= 255 (sum n_i i^2 <= 8.7e7, bden <= 2 (L - 1) sum
    // n_i i <= 4.3e7)
    int ri[8] = {(int)sum_n, (int)pres, (int)pj, (int)pj2, (int)sum_ni, (int)sum_ni2, (int)bden, 0};
    wsum8i(ri);
    double rd[8] = {s_i, ps_acc, cplx, 0.0, 0.0, 0.0, 0.0, 0.0};
    wsum8d(rd);
    const long long Nvc = ri[0];
    if (Nvc == 0) {
      if (lane < kNNGTDM) sm.early[kNFO + kNGLDM + lane] = NAN;
    } else {
      const long long Ngp = ri[1], A1 = ri[2], A2 = ri[3];
      const long long Sn1 = ri[4], Sn2 = ri[5];
      const double ssum = rd[0];
      const double Nd = (double)Nvc;
      const double rNd = rcp64(Nd);      // one reciprocal; the rest multiply
      const double psum = rd[1] * rNd;  // sum_i p_i s_i
      const bool any_s = __ballot(anys) != 0ull;
      bden = ri[6];
      cplx = rd[2];
      if (lane == 0) {
        float* f = sm.early + kNFO + kNGLDM;
        // sum_ij p_i p_j (i-j)^2 = 2 Var_p(i);  sum_ij (p_i+p_j)(i-j)^2 =
        // 2 sum_i p_i (Ngp i^2 - 2 i A1 + A2)
        const double c1 = 2.0 * (double)(Nvc * Sn2 - Sn1 * Sn1) * (rNd * rNd);
        const double strn = 2.0 * (double)(Ngp * Sn2 - 2 * A1 * Sn1 + A2 * Nvc) * rNd;
        f[0] = any_s ? (float)rcp64(psum) : 1e6f;
        f[1] = Ngp <= 1 ? 0.f : (float)(fdiv(c1, (double)(Ngp * (Ngp - 1))) * (ssum * rNd));
        f[2] = bden == 0 ? 0.f : (float)fdiv(rd[1], (double)bden);
        f[3] = (float)(cplx * rNd);
        f[4] = any_s ? (float)fdiv(strn, ssum) : 0.f;
      }
    }
  }

  // the place of those counts is the runs' and zones' now
  __syncthreads();
  clear16(sm.u.a.glrlm, L * S * 4, lane);
  if (lane < L) sm.u.a.zpl[lane] = 0;
  if constexpr (!SM::kHashInSame) {
    for (int e = lane; e < HT + HT / 2; e += 64) sm.u.a.hash_m[e] = 0;
  }
  __syncthreads();

  // ---- zones: union of the listed edges -------------------------------
  // parent[c] <= c names a voxel of c's zone: a forest whose roots are the
  // zones' smallest cube indices once every edge's ends share a root.  An
  // edge lowers the parent of its larger end; an end that had another
  // parent goes on with that one, so no connection is lost.  A pass of
  // minimum labels over all 26 neighbours, repeated until nothing changed
  // (about four times), had been 14 % of the kernel's VALU instructions and
  // half its LDS ones; with the runs below counted by kind: 10.8 k -> 7.9 k
  // VALU and 1,346 -> 790 LDS instructions a voxel, 20.9 -> 16.7 ms for
  // 1 M voxels of radius 3.
  //
  // This pass and the following ones take QB positions a lane at a time,
  // their LDS reads issued together (14.9 -> 14.3 ms for 1 M voxels of
  // radius 3).
  using UA = typename SM::U::A;
  constexpr int QB = NIT < 6 ? NIT : 6;
  uint16_t* elist = sm.list();
  static_assert(SM::NB >= 6 * C, "the edge list holds three edges a voxel");
  static_assert(C <= 2048, "an entry is a cube index of 11 bits and a mask bit of 5");
  // levels (compact + 1) and masks of positions 64 (q0 + k) + lane, 0 where
  // there is no member
  auto load_masks = [&](int q0, uint32_t(&l1)[QB], uint32_t(&same)[QB]) FR_INLINE {
#pragma unroll
    for (int k = 0; k < QB; ++k) {
      const int c = lane + 64 * (q0 + k), cc = min(c, CP - 1);
      l1[k] = c < C ? sm.cl[cc] : 0u;
      same[k] = sm.u.a.same[cc];
    }
#pragma unroll
    for (int k = 0; k < QB; ++k) same[k] = l1[k] ? same[k] : 0u;
  };
  if (fGLSZM) {
    uint32_t* parent = sm.u.a.parent;
    int n_edge = 0;
#pragma unroll 1
    for (int q0 = 0; q0 < NIT; q0 += QB) {
      uint32_t l1[QB], back[QB], cov[QB];
      load_masks(q0, l1, back);
      // the first equal-level neighbour before c is its parent (backward
      // bits, dx = 0 first: zone bits); no bit: entry 31, 0
#pragma unroll
      for (int k = 0; k < QB; ++k) {
        back[k] = __builtin_amdgcn_perm(0u, back[k] & kBackBits, 0x03020001u);
        const int b = (__ffs(back[k]) - 1) & 31, c = lane + 64 * (q0 + k);
        cov[k] = sm.zcov[b];
        const uint32_t off = sm.zoff[b];
        if (l1[k]) parent[c] = (uint32_t)c - off;
      }
      // the neighbours that no earlier one taken is a neighbour of: edges
      // (at most three more: four of the half neighbourhood are pairwise
      // no neighbours)
      for (;;) {
        bool any = false;
#pragma unroll
        for (int k = 0; k < QB; ++k) {
          back[k] &= ~cov[k];
          const uint64_t m = __ballot(back[k] != 0u);
          const int b = (__ffs(back[k]) - 1) & 31;
          cov[k] = sm.zcov[b];
          if (back[k]) elist[n_edge + below(m)] = (uint16_t)((lane + 64 * (q0 + k)) | b << 11);
          n_edge += __popcll(m);
          any |= m != 0ull;
        }
        if (!any) break;
      }
    }
    __syncthreads();
    for (int e0 = 0; e0 < n_edge; e0 += 64) {
      if (e0 + lane < n_edge) {
        const uint32_t w = elist[e0 + lane];
        uint32_t u = w & 0x7ffu, v = u - sm.zoff[w >> 11];
        while (u != v) {
          const uint32_t hi = max(u, v), lo = min(u, v);
          const uint32_t old = atomicMin(&parent[hi], lo);
          if (old == hi) break;
          u = old;
          v = lo;
        }
      }
    }
    __syncthreads();
  }

  // ---- runs -----------------------------------------------------------
  // A run of direction d starts where the backward neighbour is not of this
  // level.  Runs of one voxel (most of them, in images with noise) are
  // counted together; the longer ones are listed and walked, one a lane.
  // (Positions with many of them had been walked all directions together:
  // the GLRLM of 30,000 voxels of a uniform or piecewise constant image at
  // radius 3 took 393 and 364 us, listed 320 and 313; of noise in 8 levels
  // 336, listed 287.)
  if (MODE != kAveraged && fGLRLM) {
    uint16_t* rlist = sm.list();
    constexpr int kCap = SM::NB / 2;
    static_assert(kCap >= 64 * QB, "a round of run starts fits the list");
    int n_run = 0;
#pragma unroll 1
    for (int q0 = 0; q0 < NIT; q0 += QB) {
      uint32_t l1[QB], act[QB];
      load_masks(q0, l1, act);
#pragma unroll
      for (int k = 0; k < QB; ++k) {
        const uint32_t same = act[k];
        // (the backward bits moved to their opposites: bytes 0 and 2 swapped)
        const uint32_t starts = ~(__builtin_amdgcn_perm(0u, same, 0x03000102u) << 4) & kFwdBits;
        act[k] = starts & same;
        const int single = __popc(starts & ~same);
        if (l1[k] && single) atomicAdd(&sm.u.a.glrlm[((int)l1[k] - 1) * S], (uint32_t)single);
      }
      for (bool any = true; any;) {  // one run of every position a round
        any = false;
#pragma unroll
        for (int k = 0; k < QB; ++k) {
          const uint64_t m = __ballot(act[k] != 0u);
          if (act[k]) rlist[n_run + below(m)] = (uint16_t)((lane + 64 * (q0 + k)) | (__ffs(act[k]) - 1) << 11);
          act[k] &= act[k] - 1u;
          n_run += __popcll(m);
          any |= m != 0ull;
        }
        if (n_run > 0 && (n_run > kCap - 64 * QB || (!any && q0 + QB >= NIT))) {
          __syncthreads();
          for (int e0 = 0; e0 < n_run; e0 += 64) {
            if (e0 + lane < n_run) {
              const uint32_t w = rlist[e0 + lane];
              const int c = (int)(w & 0x7ffu), b = (int)(w >> 11);
              const uint32_t step = sm.foff[b];
              uint32_t* row = &sm.u.a.glrlm[((int)sm.cl[c] - 1) * S];
              uint32_t u = (uint32_t)c + step;
              int len = 1;
              while ((sm.u.a.same[u] >> b) & 1u) {
                u += step;
                ++len;
              }
              atomicAdd(&row[len], 1u);
            }
          }
          __syncthreads();
          n_run = 0;
        }
      }
    }
    __syncthreads();
  }
  // GLRLM averaged over the directions: each direction's runs counted and
  // reduced in turn; lane k < 16 keeps the sum of feature k
  double rl_acc = 0.0;
  if constexpr (MODE == kAveraged) {
    if (fGLRLM) {
#pragma unroll 1
      for (int d = 0; d < 13; ++d) {
        __syncthreads();
        for (int e = lane; e < L * S; e += 64) sm.u.a.glrlm[e] = 0;
        __syncthreads();
        const int step = (kDir[d][2] * S + kDir[d][1]) * S + kDir[d][0];
#pragma unroll 1
        for (int q = 0; q < NIT; ++q) {
          const int c = lane + 64 * q;
          const int l1 = (c < C) ? sm.cl[c] : 0;
          if (!l1) continue;
          uint32_t sb = sm.u.a.same[c];
          if ((sb >> back_bit(d)) & 1u) continue;  // not the start of a run
          int len = 0, u = c;
          while ((sb >> fwd_bit(d)) & 1u) {
            u += step;
            sb = sm.u.a.same[u];
            ++len;
          }
          atomicAdd(&sm.u.a.glrlm[(l1 - 1) * S + len], 1u);
        }
        __syncthreads();
        if (dbg)
          for (int e = lane; e < L * S; e += 64)
            a.d_glrlm[it * a.ng * S + (int64_t)(sm.lval[e / S] - 1) * S + e % S] += (int32_t)sm.u.a.glrlm[e];
        double f[16];
        runs_features<R>(sm.u.a.glrlm, lrow, L, lane, (double)K, f);
        double own = 0.0;
#pragma unroll
        for (int k = 0; k < 16; ++k) own = lane == k ? f[k] : own;
        rl_acc += own;
      }
    }
  }
  __syncthreads();

  // ---- zone sizes, then the zones, a lane each ------------------------
  Emph ez = {};
  if (fGLSZM) {
    // the run list's place and the hash; the masks are no longer read
    clear16(sm.zcnt(), SM::kZoneBytes, lane);
    if constexpr (SM::kHashInSame) {
      static_assert(sizeof(UA::same) >= 6u * HT, "the hash fits the masks' place");
      clear16(sm.u.a.same, 6 * HT, lane);
    }
    __syncthreads();
    uint32_t* parent = sm.u.a.parent;
    uint64_t roots[NIT];
#pragma unroll
    for (int q0 = 0; q0 < NIT; q0 += QB) {
      uint32_t l1[QB], r[QB];
#pragma unroll
      for (int k = 0; k < QB && q0 + k < NIT; ++k) {
        const int c = lane + 64 * (q0 + k);
        l1[k] = c < C ? sm.cl[c] : 0u;
        r[k] = parent[c];
      }
#pragma unroll
      for (int k = 0; k < QB && q0 + k < NIT; ++k) {
        const uint32_t c = (uint32_t)(lane + 64 * (q0 + k));
        roots[q0 + k] = __ballot(l1[k] && r[k] == c);
        r[k] = l1[k] ? r[k] : c;
      }
      for (bool moved = true; moved;) {
        uint32_t up[QB];
        moved = false;
#pragma unroll
        for (int k = 0; k < QB && q0 + k < NIT; ++k) up[k] = parent[r[k]];
#pragma unroll
        for (int k = 0; k < QB && q0 + k < NIT; ++k) {
          moved |= l1[k] && up[k] != r[k];
          r[k] = l1[k] ? up[k] : r[k];
        }
        moved = __ballot(moved) != 0ull;
      }
#pragma unroll
      for (int k = 0; k < QB && q0 + k < NIT; ++k)
        if (l1[k]) gadd(sm.zcnt(), (int)r[k], 1u);
    }
    __syncthreads();
    // the roots listed in place of the forest
    int n_root = 0;
#pragma unroll
    for (int q = 0; q < NIT; ++q) {
      if ((roots[q] >> lane) & 1ull) parent[n_root + below(roots[q])] = (uint32_t)(lane + 64 * q);
      n_root += __popcll(roots[q]);
    }
    __syncthreads();
#pragma unroll 1
    for (int k0 = 0; k0 < n_root; k0 += 64) {
      if (k0 + lane < n_root) {
        const int c = (int)parent[k0 + lane];
        const int l = (int)sm.cl[c] - 1, g = sm.lval[l];
        const int s = (int)gget(sm.zcnt(), c);
        emph_add(ez, 1, g, s);  // c log2 c = 0 for c = 1; the entropy comes from the hash
        atomicAdd(&sm.u.a.zpl[l], 1u);
        gadd(sm.zps(), s - 1, 1u);
        const uint32_t key = ((uint32_t)l << 16 | (uint32_t)s) + 1u;
        // multiplicative hash: the product's high bits mix level and size
        uint32_t h = (key * 2654435761u) >> (32 - __builtin_ctz((unsigned)HT));
        while (true) {
          const uint32_t old = atomicCAS(&sm.hkey()[h], 0u, key);
          if (old == 0u || old == key) {
            gadd(sm.hcnt(), (int)h, 1u);
            break;
          }
          h = (h + 1) & (HT - 1);
        }
        if (dbg) {
          const int64_t base = it * (int64_t)a.ng * C;
          atomicAdd(&a.d_glszm[base + (int64_t)(g - 1) * C + (s - 1)], 1);
        }
      }
    }
  }
  __syncthreads();

  // adds this pass's co-occurrence counts to the dense table (lane e mod 64
  // owns entry e in every pass)
  auto dump_glcm = [&]() FR_INLINE {
    const int ng = a.ng;
    for (int e = lane; e < L * L; e += 64) {
      const int l = e / L, m = e % L;
      a.d_glcm[it * ng * ng + (int64_t)(sm.lval[l] - 1) * ng + (sm.lval[m] - 1)] += (int32_t)gsym<SM>(sm.u.a.glcm, l, m);
    }
  };
  if (dbg) {
    const int ng = a.ng;
    if constexpr (MODE != kAveraged) {
      dump_glcm();
      for (int e = lane; e < L * S; e += 64) {
        const int l = e / S, j = e % S;
        a.d_glrlm[it * ng * S + (int64_t)(sm.lval[l] - 1) * S + j] = (int32_t)sm.u.a.glrlm[e];
      }
    }
  }

  // map offsets of the families in the output
  int off = 0;
  const int oFO = off;    off += fFO ? kNFO : 0;
  const int oGLCM = off;  off += fGLCM ? kNGLCM : 0;
  const int oGLRLM = off; off += fGLRLM ? kNGLRLM : 0;
  const int oGLSZM = off; off += fGLSZM ? kNGLSZM : 0;
  const int oGLDM = off;  off += fGLDM ? kNGLDM : 0;
  const int oNGTDM = off; off += fNGTDM ? kNNGTDM : 0;
  const int count = off;
  float* F = sm.feat();
  if (fFO && lane < kNFO) F[oFO + lane] = sm.early[lane];
  if (fGLDM && lane < kNGLDM) F[oGLDM + lane] = sm.early[kNFO + lane];
  if (fNGTDM && lane < kNNGTDM) F[oNGTDM + lane] = sm.early[kNFO + kNGLDM + lane];

  // ---- GLRLM ----------------------------------------------------------
  if (fGLRLM) {
    if constexpr (MODE == kAveraged) {
      if (lane < 16) F[oGLRLM + lane] = (float)(rl_acc / 13.0);
    } else {
      float f[16];
      runs_features<R>(sm.u.a.glrlm, lrow, L, lane, 13.0 * Kd, f);
      if (lane == 0)
        for (int k = 0; k < 16; ++k) F[oGLRLM + k] = f[k];
    }
  }

  // ---- GLSZM ----------------------------------------------------------
  if (fGLSZM) {
    double hl = 0.0;
#pragma unroll
    for (int t = 0; t < HT / 2; t += 64) {  // two counts a word; 0 log 0 = 0
      const uint32_t w = t + lane < HT / 2 ? sm.hcnt()[t + lane] : 0u;
      hl += xlog2x<R>(w & 0xffffu) + xlog2x<R>(w >> 16);
    }
    ez.clogc = hl;  // zones count once each; the entropy term comes from the hash
    long long gln = 0;
    if (lane < L) {
      const long long t = sm.u.a.zpl[lane];
      gln = t * t;
    }
    uint32_t szs = 0;  // total at most C^2 = 1.8e6
    for (int e = lane; e < CP / 2; e += 64) {
      const uint32_t w = sm.zps()[e];
      szs += __umul24(w & 0xffffu, w & 0xffffu) + __umul24(w >> 16, w >> 16);
    }
    long long szn = szs;
    emph_reduce(ez, gln, szn);
    float f[16];
    emph16(ez, gln, szn, Kd, xlog2x<R>((uint32_t)ez.n), f);
    if (lane == 0)
      for (int k = 0; k < 16; ++k) F[oGLSZM + k] = f[k];
  }

  // ---- GLCM (last: its eigen work space overlays the tables above) -----
  if (fGLCM) {
    [[maybe_unused]] uint32_t defined = 0;  // kAveraged: directions with a pair
    if constexpr (MODE == kAveraged) {
      if (lane < 24) av->glcm[lane] = 0.0;
    }
#pragma unroll 1
    for (int pass = 0; pass < (MODE == kAveraged ? 13 : 1); ++pass) {
    if constexpr (MODE == kAveraged) {
      __syncthreads();
      for (int e = lane; e < SM::glcm_words(L); e += 64) sm.u.a.glcm[e] = 0;
      if (lane < L) sm.pxc[lane] = 0;
      __syncthreads();
      count_direction(pass);
      if (dbg) dump_glcm();
    }
    __syncthreads();
    // the |i-j| and i+j histograms overlay tables whose features are done:
    // clear the ranges the features read (|i-j| < Ng, i+j <= 2 Ng)
    for (int e = lane; e < a.ng; e += 64) sm.u.c.pd[e] = 0;
    for (int e = lane; e <= 2 * a.ng; e += 64) sm.u.c.ps[e] = 0;
    __syncthreads();
    uint32_t rowc = 0;
    double hxp = 0.0;
    int ri[8] = {};  // N_P, sum i, sum i^2: totals below 2^31
    if (lane < L) {
      rowc = sm.pxc[lane];
      const uint32_t lv = sm.lval[lane];
      ri[0] = (int)rowc;
      ri[1] = (int)__umul24(rowc, lv);
      ri[2] = (int)__umul24((uint32_t)ri[1], lv);
      hxp = xlog2x<R>(rowc);
    }
    wsum8i(ri);
    const long long NP = ri[0], S1x = ri[1], S2x = ri[2];
    if (NP == 0) {
      if constexpr (MODE != kAveraged) {
        if (lane < kNGLCM) F[oGLCM + lane] = NAN;
      }
    } else {
      defined |= 1u << pass;
      const uint64_t presb = __ballot(lane < L && rowc > 0);
      const int nlev = __popcll(presb);
      const double Nd = (double)NP;
      const double nlogn = xlog2x<R>((uint32_t)NP);
      // MCC: spectral radius of B = D^-1/2 P D^-1/2 - v v^T over present
      // levels.  The place of a problem with up to 32 levels, which a flush
      // (or the MCC kernel) computes four at a time
      const bool defer = nlev > 1 && nlev <= 32;
      uint16_t* gq = nullptr;
      float** dq = nullptr;
      int* nqp = nullptr;
      if (defer) {
        if constexpr (MOUT) {
          // problems with <= 16 levels fill the voxel's partition of the
          // stash from its start, wider ones from its end (one problem per
          // voxel at most, so the two never meet)
          const bool small = nlev <= 16;
          const int p = (int)(it + a.key0) % kParts;
          int slot = 0;
          if (lane == 0) slot = atomicAdd(&a.mcc_count[p * kPartStride + (small ? kCntNarrow : kCntWide)], 1);
          slot = __builtin_amdgcn_readfirstlane(slot);
          if (small) {
            McSmall* q = (McSmall*)(a.mcc + part_base(a.part_n, p) * kMccProblemBytes) + slot;
            gq = q->g, dq = &q->dst, nqp = &q->n;
          } else {
            McProblem* q = (McProblem*)(a.mcc + part_base(a.part_n, p + 1) * kMccProblemBytes) - (slot + 1);
            gq = q->g, dq = &q->dst, nqp = &q->n;
          }
        } else {
          bool to_small = false;
          if constexpr (kSmallSlots<R, LMAX> > 0) to_small = nlev <= 16;
          if (to_small) {
            if constexpr (kSmallSlots<R, LMAX> > 0) gq = sm.ms.s[ns].g, dq = &sm.ms.s[ns].dst, nqp = &sm.ms.s[ns].n;
            ++ns;
          } else {
            gq = sm.mq.s[nq].g, dq = &sm.mq.s[nq].dst, nqp = &sm.mq.s[nq].n;
            ++nq;
          }
        }
      }
      // every level has a pair (all but isolated ones do): the problem's
      // entries are those of the pass below, in its order
      const bool whole = defer && nlev == L;
      // entries of the upper triangle (r <= c), one per lane, enumerated
      // compactly (e = c (c + 1) / 2 + r); an entry off the diagonal stands
      // for the two symmetric ones (weight 2)
      const int ntri = L * (L + 1) / 2;
      uint32_t e2 = 0;  // total at most N_P^2 = 8.1e8
      double plogp = 0.0;
      unsigned pmax = 0;
      for (int e0 = 0; e0 < ntri; e0 += 64) {
        const int e = e0 + lane;
        if (e < ntri) {
          const uint32_t rc = kTri.v[e];
          const int r = (int)(rc & 0xffu), c = (int)(rc >> 8);
          const uint32_t P = gsym<SM>(sm.u.a.glcm, r, c);
          if (whole) gq[e] = (uint16_t)P;
          if (P) {
            const uint32_t w = r == c ? 1u : 2u;
            e2 += __umul24(w * P, P);
            plogp = fma((double)w, xlog2x<R>(P), plogp);
            pmax = max(pmax, P);
            const int i = sm.lval[r], j = sm.lval[c];
            atomicAdd(&sm.u.c.pd[i > j ? i - j : j - i], w * P);
            atomicAdd(&sm.u.c.ps[i + j], w * P);
          }
        }
      }
      pmax = wmaxu(pmax);
      __syncthreads();
      const int ng = a.ng;
      const double rNd = rcp64(Nd), rN2 = rNd * rNd;  // one reciprocal; the rest multiply
      const double mu = (double)S1x * rNd;
      uint32_t sd1 = 0, sd2 = 0, ss1 = 0;
      std::conditional_t<(R > 3), double, uint32_t> ss2 = 0;
      double dlog = 0, slog = 0, iv = 0, idm = 0, idmn = 0, id = 0, idn = 0, ct = 0, cs = 0, cp = 0;
      const double ngd = (double)ng;
      const double rng = rcp64(ngd), rng2 = rng * rng;
      for (int k = lane; k < ng; k += 64) {
        const uint32_t c = sm.u.c.pd[k];
        if (c) {
          const double cd = (double)c, kd = (double)k;
          const uint32_t ck = __umul24(c, (uint32_t)k);
          sd1 += ck;
          sd2 += __umul24(ck, (uint32_t)k);
          dlog += xlog2x<R>(c);
          iv += cd * kInvSq.v[k];  // the table's entry 0 is 0
          idm += cd * frcp(1.0 + kd * kd);
          idmn += cd * frcp(1.0 + kd * kd * rng2);
          id += cd * frcp(1.0 + kd);
          idn += cd * frcp(1.0 + kd * rng);
        }
      }
      for (int k = 2 + lane; k <= 2 * ng; k += 64) {
        const uint32_t c = sm.u.c.ps[k];
        if (c) {
          const double cd = (double)c, t = (double)k - 2.0 * mu;
          const uint32_t ck = __umul24(c, (uint32_t)k);
          ss1 += ck;
          if constexpr (R > 3)
            ss2 += (double)ck * (double)k;
          else
            ss2 += __umul24(ck, (uint32_t)k);
          slog += xlog2x<R>(c);
          ct += cd * t * t;
          cs += cd * t * t * t;
          cp += cd * t * t * t * t;
        }
      }
      // totals below 2^31: the largest, sum over i+j of c k^2, is at most
      // N_P (2 Ng)^2 = 6,516 x 510^2 = 1.7e9 for a 7^3 cube; above radius 3
      // (28,460 x 510^2 = 7.4e9) that one is summed in FP64, exactly
      int hi[8] = {(int)sd1, (int)sd2, (int)ss1, R > 3 ? 0 : (int)ss2, (int)e2, 0, 0, 0};
      wsum8i(hi);
      const long long Sd1 = hi[0], Sd2 = hi[1], Ss1 = hi[2], E2 = hi[4];
      double h1[8] = {dlog, slog, iv, idm, idmn, id, idn, ct};
      wsum8d(h1);
      dlog = h1[0];
      slog = h1[1];
      iv = h1[2];
      idm = h1[3];
      idmn = h1[4];
      id = h1[5];
      idn = h1[6];
      ct = h1[7];
      double h2[8] = {cs, cp, R > 3 ? (double)ss2 : 0.0, hxp, plogp, 0.0, 0.0, 0.0};
      wsum8d(h2);
      const long long Ss2 = R > 3 ? (long long)h2[2] : (long long)hi[3];
      cs = h2[0];
      cp = h2[1];
      const long long sij = (Ss2 - Sd2) / 4;  // sum_ij i j P
      const double HX = (nlogn - h2[3]) * rNd, HXY = (nlogn - h2[4]) * rNd;

      double mcc = 1.0;
      if (nlev > 1) {
        mcc = NAN;
        if (!whole) {
          if (lane < L && rowc > 0) {
            const int pos = __popcll(presb & ((lane == 0) ? 0ull : (~0ull >> (64 - lane))));
            sm.u.b.pl[pos] = lane;
          }
          __syncthreads();
        }
        if (defer) {
          if (!whole) {
            // upper triangle, column c of the lower half-wave and column
            // n - 1 - c of the upper one per pass
            const int l = lane & 31, n = nlev;
            const int plr = l < n ? sm.u.b.pl[l] : 0;
            for (int c0 = 0; 2 * c0 < n; ++c0) {
              const int c = lane < 32 ? c0 : n - 1 - c0;
              if (l <= c && (lane < 32 || c > c0))
                gq[c * (c + 1) / 2 + l] = (uint16_t)gsym<SM>(sm.u.a.glcm, plr, sm.u.b.pl[c]);
            }
          }
          if (lane == 0) {
            *nqp = nlev;
            if constexpr (MODE == kAveraged)
              *dq = (float*)&av->mcc[pass];
            else
              *dq = a.stage ? a.stage + it * kStageStride + (oGLCM + 15)
                            : a.out + (int64_t)(oGLCM + 15) * a.n_out + it;
          }
        }
        if constexpr (LMAX > 32) {
          if (!defer) {  // > 32 levels: computed at the flush after this voxel
            if (lane == 0) {
              sm.u.b.big_n = nlev;
              if constexpr (MODE == kAveraged)
                sm.u.b.big_dst = (float*)&av->mcc[pass];
              else
                sm.u.b.big_dst = a.stage ? a.stage + it * kStageStride + (oGLCM + 15)
                                       : a.out + (int64_t)(oGLCM + 15) * a.n_out + it;
            }
            big = true;
          }
        }
      }

      if (lane == 0) {
        // a feature of this pass: its map, or one term of its mean
        auto put = [&](int k, double v) FR_INLINE {
          if constexpr (MODE == kAveraged)
            av->glcm[k] += v;
          else
            F[oGLCM + k] = (float)v;
        };
        put(0, (double)sij * rNd);
        put(1, mu);
        put(2, cp * rNd);
        put(3, cs * rNd);
        put(4, ct * rNd);
        put(5, (double)Sd2 * rNd);
        put(6, nlev <= 1 ? 1.0
                         : fdiv((double)(NP * sij - S1x * S1x), (double)(NP * S2x - S1x * S1x)));
        put(7, (double)Sd1 * rNd);
        put(8, (nlogn - dlog) * rNd);
        put(9, (double)(NP * Sd2 - Sd1 * Sd1) * rN2);
        put(10, (double)E2 * rN2);
        put(11, HXY);
        put(12, nlev <= 1 ? 0.0 : fdiv(HXY - 2.0 * HX, HX));
        const double t = 1.0 - exp(-2.0 * (2.0 * HX - HXY));
        put(13, t > 0.0 ? fsqrt(t) : 0.0);
        put(14, idm * rNd);
        if constexpr (MODE == kAveraged) {
          if (nlev <= 1) av->mcc[pass] = 1.0;
        } else {
          put(15, mcc);
        }
        put(16, idmn * rNd);
        put(17, id * rNd);
        put(18, idn * rNd);
        put(19, iv * rNd);
        put(20, (double)pmax * rNd);
        put(21, (double)Ss1 * rNd);
        put(22, (nlogn - slog) * rNd);
        put(23, (double)(NP * S2x - S1x * S1x) * rN2);
      }
    }
    if constexpr (MODE == kAveraged) {  // one flush site for the pending problems of the directions so far
      const int fs = (ns == kSmallSlots<R, LMAX> || pass == 12) ? ns : 0;
      const int fq = (nq == kMcSlots<R, LMAX> || pass == 12) ? nq : 0;
      if (big || fs || fq) {
        mcc_flush<double, kFineMcc<R, MODE>>(sm, fs, fq, big);
        ns -= fs;
        nq -= fq;
        big = false;
      }
    }
    }
    if constexpr (MODE == kAveraged) {  // mean over the directions that have a pair
      __syncthreads();
      if (lane < kNGLCM) {
        double t = av->glcm[lane];
        if (lane == 15)
          for (int d = 0; d < 13; ++d)
            if ((defined >> d) & 1u) t += av->mcc[d];
        F[oGLCM + lane] = defined ? (float)(t / (double)__popc(defined)) : NAN;
      }
    }
  }

  __syncthreads();
  if (a.stage) {  // one contiguous row per voxel; the transpose kernel scatters it
    // whole rows (a deferred MCC is a placeholder here; the flush overwrites it
    // after its barrier, whose release fence completes these stores first)
    float* row = a.stage + it * kStageStride;
    for (int k = lane; k < count; k += 64) row[k] = F[k];
  } else {
    for (int k = lane; k < count; k += 64) a.out[(int64_t)k * a.n_out + it] = F[k];
  }
  __syncthreads();
}

// Waves per SIMD that an instance's registers are held to.  The production
// instances (MOUT: the MCC problems with <= 32 levels go to the stash of
// a.mcc, so there are no LDS slots for them) with at most 32 levels hold no
// MCC code.  Five below radius 3 (96 VGPRs, a few of them spilled): the
// latency of the zone and run walks shows there; 100 k voxels at radius 2
// take 0.90 ms, 0.95 with four waves.  Four at radius 3 (128 VGPRs, none
// spilled), where the tables in LDS allow fifteen waves per CU: 1 M voxels
// take 11.4 ms, 12.2 with three.  Two for the 64-level ones, which solve
// wider problems themselves, a column of 64 doubles a lane (three spill
// thirty registers: 60 k voxels of 33 levels and more, 3.2 -> 4.8 ms), and
// for all others.
template <int R, int LMAX, bool MOUT>
constexpr int kMapWaves = !MOUT || LMAX > 32 || R > 3 ? 2 : R == 3 ? 4 : 5;
template <typename T, int R, int LMAX, bool DEBUG, bool MOUT, int MODE = kPlain>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(kMapWaves<R, LMAX, MOUT>))) void k_map(MapArgs arg) {
  static_assert(!MOUT || (!DEBUG && MODE == kPlain), "stash only from production instances");
  __shared__ Smem<R, LMAX, MOUT> sm;
  __shared__ std::conditional_t<MODE == kAveraged, AvgMem, char> av;
  const bool dbg = DEBUG && (!std::is_same_v<T, AnyRaw> || arg.d_glcm != nullptr);
  const DiscParams* P = arg.params;
  if (P->err != kJobOk) return;  // a data error of the discretisation: write nothing
  MapArgs a = arg;
  a.ng = P->ng;
  smem_layout(sm);
  int ns = 0, nq = 0;  // deferred MCC problems in sm.ms and sm.mq
  bool big = false;    // a problem with > 32 levels pending
  // balanced shares of the voxels (n < 2^31): the counts differ by at most
  // one; of an item list, workgroup b takes every per-th entry of partition
  // b mod kParts, as the previous pass left it (launch_i: nblk >= kParts)
  int64_t k = (int64_t)blockIdx.x * a.n_items / a.nblk, kend = ((int64_t)blockIdx.x + 1) * a.n_items / a.nblk;
  int64_t kstep = 1;
  const int2* items = nullptr;
  if (a.items) {
    const int p = (int)blockIdx.x % kParts;
    items = a.items + part_base(a.part_n, p);
    kend = a.items_count[p * kPartStride];
    k = (int)blockIdx.x / kParts;
    kstep = (a.nblk - p + kParts - 1) / kParts;
  }
  for (; k < kend; k += kstep) {
    const int64_t it = items ? (int64_t)items[k].y : k;
    const int64_t m = dbg ? a.sample[it] : it;
    if (m < 0 || m >= a.n_list) {  // out-of-range sample index: NaN maps, no matrices
      for (int q = threadIdx.x; q < 93; q += 64)
        if (q < __popc(a.families & 1u) * 18 + __popc(a.families & 2u) * 24 +
                    __popc(a.families & 4u) * 16 + __popc(a.families & 8u) * 16 +
                    __popc(a.families & 16u) * 14 + __popc(a.families & 32u) * 5)
          a.out[(int64_t)q * a.n_out + it] = NAN;
    } else {
      map_voxel<T, R, LMAX, DEBUG, MOUT, MODE>(sm, a, a.list[m], it, ns, nq, big, (AvgMem*)&av);
    }
    if constexpr (MODE == kAveraged) {  // every problem was solved with its voxel
    } else if constexpr (!MOUT) {
      // one flush site (the flush code is large): after a voxel with more
      // than 32 levels, when a pool is full, and after the last voxel
      const bool last = k + kstep >= kend;
      const int fs = (ns == kSmallSlots<R, LMAX> || last) ? ns : 0;
      const int fq = (nq == kMcSlots<R, LMAX> || last) ? nq : 0;
      if (big || fs || fq) {
        mcc_flush<float, kFineMcc<R, MODE>>(sm, fs, fq, big);
        ns -= fs;
        nq -= fq;
        big = false;
      }
    } else if constexpr (LMAX > 32) {
      if (big) {  // the smaller problems went to the stash
        mcc_flush<float, kFineMcc<R, MODE>>(sm, 0, 0, true);
        big = false;
      }
    }
  }
}

// Workgroups for n voxels: a whole number of waves of the resident
// workgroups (so no partial last wave leaves CUs idle), at least 8 voxels
// each (a sweep over 4..48 on the PET workload put the optimum there) and
// at most 8 waves.  Fewer voxels than resident workgroups get one each
// where the MCC problems leave the kernel (or are solved with their voxel):
// with the other stages as they were then, a call of 1,537 voxels at radius 2
// took 186 us with four each, 109 us with one (61 now); of 2,176 at radius 1,
// 84 and 76 (34 now).  An instance that flushes its deferred problems itself
// keeps four voxels per workgroup (minv 4), which fill the rows of its
// flushes.
inline int64_t plain_blocks(int64_t n, int64_t resident, int64_t minv) {
  if (resident < 1) resident = 1;
  int64_t per = (n + resident * 8 - 1) / (resident * 8);
  if (per < 8) per = 8;
  const int64_t waves = (n + resident * per - 1) / (resident * per);
  int64_t nblk = waves * resident;
  const int64_t cap = (n + minv - 1) / minv;
  if (nblk > cap) nblk = cap;
  return nblk < 1 ? 1 : nblk;
}

template <typename T, int R, int LMAX, bool DEBUG, bool MOUT, int MODE = kPlain>
int resident_t() {
  static int resident = 0;  // resident workgroups of this instance on the device
  if (resident == 0) {
    int dev = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void*)k_map<T, R, LMAX, DEBUG, MOUT, MODE>, 64,
                                                     0) != hipSuccess) {
      (void)hipGetLastError();
      cus = 256;
      per_cu = 1;
    }
    resident = (per_cu > 0 ? per_cu : 1) * (cus > 0 ? cus : 1);
  }
  return resident;
}

// One launch of an instance: a whole number of waves over a.n_items voxels,
// or, over an item list whose length only the device knows, one wave of
// resident workgroups, each taking its share of whatever the list holds.
template <typename T, int R, int LMAX, bool DEBUG, bool MOUT, int MODE = kPlain>
hipError_t launch_i(MapArgs a, hipStream_t st) {
  const int resident = resident_t<T, R, LMAX, DEBUG, MOUT, MODE>();
  a.nblk = a.items ? (resident > kParts ? resident : kParts) : plain_blocks(a.n_items, resident, MOUT || MODE == kAveraged ? 1 : 4);
  hipLaunchKernelGGL((k_map<T, R, LMAX, DEBUG, MOUT, MODE>), dim3((unsigned)a.nblk), dim3(64), 0, st, a);
  return hipGetLastError();
}

template <typename T, int R, int LMAX>
hipError_t launch_t(const MapArgs& a, bool debug, hipStream_t st) {
  if (debug) return launch_i<T, R, LMAX, true, false>(a, st);
  return a.mcc ? launch_i<T, R, LMAX, false, true>(a, st) : launch_i<T, R, LMAX, false, false>(a, st);
}

template <typename T>
hipError_t launch_r(const MapArgs& a, int radius, int lmax, bool debug, hipStream_t st) {
  if (radius == 1) return launch_t<T, 1, 32>(a, debug, st);
  if (radius == 2) return lmax <= 32 ? launch_t<T, 2, 32>(a, debug, st) : launch_t<T, 2, 64>(a, debug, st);
  return lmax <= 32 ? launch_t<T, 3, 32>(a, debug, st) : launch_t<T, 3, 64>(a, debug, st);
}

// An extraction variant's launch (any radius, both raw types).
template <int MODE>
hipError_t launch_v(const MapArgs& a, int radius, int lmax, hipStream_t st) {
  const bool l32 = lmax <= 32;
  switch (radius) {
    case 1: return launch_i<AnyRaw, 1, 32, true, false, MODE>(a, st);
    case 2: return l32 ? launch_i<AnyRaw, 2, 32, true, false, MODE>(a, st) : launch_i<AnyRaw, 2, 64, true, false, MODE>(a, st);
    case 3: return l32 ? launch_i<AnyRaw, 3, 32, true, false, MODE>(a, st) : launch_i<AnyRaw, 3, 64, true, false, MODE>(a, st);
    case 4: return l32 ? launch_i<AnyRaw, 4, 32, true, false, MODE>(a, st) : launch_i<AnyRaw, 4, 64, true, false, MODE>(a, st);
    default: return l32 ? launch_i<AnyRaw, 5, 32, true, false, MODE>(a, st) : launch_i<AnyRaw, 5, 64, true, false, MODE>(a, st);
  }
}

// The next item of a workgroup from the partitioned queue: of a host-made
// list of n_items (item w in partition w mod kParts, so that the list's order
// is kept across them), or of an earlier pass's partitioned list (counts).
// p: the workgroup's partition, left: how many it has not found empty yet;
// an exhausted one is left for the next.  -1 once all are.
__device__ inline int64_t take_item(int32_t* queue, const int32_t* counts, int64_t part_n, int32_t n_items, int& p,
                                    int& left) {
  for (; left > 0; --left, p = (p + 1) % kParts) {
    const int n = counts ? counts[p * kPartStride] : (n_items - p + kParts - 1) / kParts;
    int q = n;
    if (threadIdx.x == 0 &&
        __hip_atomic_load(&queue[p * kPartStride], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < n)
      q = atomicAdd(&queue[p * kPartStride], 1);
    q = __builtin_amdgcn_readfirstlane(q);
    if (q < n) return counts ? part_base(part_n, p) + q : (int64_t)q * kParts + p;
  }
  return -1;
}

template <typename T, int R, int LMAX>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(kMapWaves<R, LMAX, false>))) void k_map_batch(
    const BatchJob* __restrict__ jobs, const DiscParams* __restrict__ params,
    const int2* __restrict__ items, int32_t n_items_host, const int32_t* __restrict__ items_count,
    int32_t vpw, int2* over, int32_t* over_count, int32_t* queue, int64_t part_n) {
  __shared__ Smem<R, LMAX, false> sm;
  smem_layout(sm);
  int ns = 0, nq = 0;  // deferred MCC problems in sm.ms and sm.mq
  bool big = false;    // a problem with > 32 levels pending
  // work distribution: items blockIdx.x, + gridDim.x, ... (static), or the
  // next item of the queue (dynamic); one loop over their voxels, so that
  // the flush has a single site
  int64_t w = (int64_t)blockIdx.x - (int64_t)gridDim.x;
  int part = (int)blockIdx.x % kParts, left = kParts;
  bool more = true;
  int64_t m = 0, m1 = 0;
  MapArgs a;
  const BatchJob* J = nullptr;
  for (;;) {
    while (m >= m1) {  // next item of a job without error
      if (queue) {
        w = take_item(queue, items_count, part_n, n_items_host, part, left);
        more = w >= 0;
      } else {
        w += gridDim.x;
        more = w < n_items_host;
      }
      if (!more) break;
      // no item table: one job (index 0), item w starts at voxel w * vpw
      const int2 it2 = items ? items[w] : make_int2(0, w * vpw);
      const DiscParams& P = params[it2.x];
      if (P.err != kJobOk) continue;
      J = &jobs[it2.x];
      a.params = &P;
      a.vol = J->vol;
      a.dtype = J->dtype;
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
      a.mcc = nullptr;
      a.part_n = part_n;
      a.key0 = J->key0;
      a.mcc_count = nullptr;
      m = it2.y;
      m1 = (int64_t)it2.y + vpw;
      if (m1 > J->n_mask) m1 = J->n_mask;
    }
    if (more) {
      map_voxel<T, R, LMAX, false, false>(sm, a, a.list[m], m, ns, nq, big);
      ++m;
    }
    const int fs = (ns == kSmallSlots<R, LMAX> || !more) ? ns : 0;
    const int fq = (nq == kMcSlots<R, LMAX> || !more) ? nq : 0;
    if (big || fs || fq) {
      mcc_flush<float, kFineMcc<R, kPlain>>(sm, fs, fq, big);
      ns -= fs;
      nq -= fq;
      big = false;
    }
    if (!more) break;
  }
}

template <typename T, int R, int LMAX>
hipError_t launch_b(const BatchJob* jobs, const DiscParams* params, const int2* items,
                    int32_t n_items, const int32_t* items_count, int32_t vpw, int grid, int2* over,
                    int32_t* over_count, int32_t* queue, int64_t part_n, hipStream_t st) {
  hipLaunchKernelGGL((k_map_batch<T, R, LMAX>), dim3((unsigned)grid), dim3(64), 0, st, jobs, params,
                     items, n_items, items_count, vpw, over, over_count, queue, part_n);
  return hipGetLastError();
}

template <typename T, int R, int LMAX>
int occ_b() {
  int nb = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, (const void*)k_map_batch<T, R, LMAX>, 64, 0) !=
      hipSuccess)
    return 1;
  return nb > 0 ? nb : 1;
}

template <typename T>
hipError_t launch_b_r(const BatchJob* jobs, const DiscParams* params, const int2* items,
                      int32_t n_items, const int32_t* items_count, int32_t vpw, int radius,
                      int lmax, int grid, int2* over, int32_t* over_count, int32_t* queue,
                      int64_t part_n, hipStream_t st) {
  const bool l32 = lmax <= 32;
  auto f = radius == 1   ? launch_b<T, 1, 32>
           : radius == 2 ? (l32 ? launch_b<T, 2, 32> : launch_b<T, 2, 64>)
                         : (l32 ? launch_b<T, 3, 32> : launch_b<T, 3, 64>);
  return f(jobs, params, items, n_items, items_count, vpw, grid, over, over_count, queue, part_n, st);
}

template <typename T>
int occ_b_r(int radius, int lmax) {
  if (radius == 1) return occ_b<T, 1, 32>();
  if (radius == 2) return lmax > 32 ? occ_b<T, 2, 64>() : occ_b<T, 2, 32>();
  return lmax > 32 ? occ_b<T, 3, 64>() : occ_b<T, 3, 32>();
}

}  // namespace
}  // namespace fr
