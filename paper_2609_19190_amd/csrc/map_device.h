// Device helpers shared by the map kernels of this library (the fused
// fixed-radius kernel and the generic kernel): the 13 GLCM/GLRLM direction
// representatives, the exact NGTDM scale table and two FP64 primitives.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

namespace fr {
namespace {

// lcm(1..26) / c for c = 1..26: NGTDM differences |g c - sum| scaled by it
// are exact integers (s_i * lcm(1..26)).
__constant__ unsigned long long kLcmOver[27] = {
    0ull,           26771144400ull, 13385572200ull, 8923714800ull, 6692786100ull,
    5354228880ull,  4461857400ull,  3824449200ull,  3346393050ull, 2974571600ull,
    2677114440ull,  2433740400ull,  2230928700ull,  2059318800ull, 1912224600ull,
    1784742960ull,  1673196525ull,  1574773200ull,  1487285800ull, 1409007600ull,
    1338557220ull,  1274816400ull,  1216870200ull,  1163962800ull, 1115464350ull,
    1070845776ull,  1029659400ull};
constexpr double kLcm26 = 26771144400.0;
constexpr double kRcpLcm26 = 1.0 / kLcm26;

// 13 forward neighbour offsets (dx, dy, dz), one of each +/- pair, each the
// larger cube index of its pair.
// Directions 0..11 are dx = d / 4 - 1 on the forward rows (dy, dz) = (0, 1),
// (1, 0), (1, 1), (-1, 1); direction 12 is (1, 0, 0).
__host__ __device__ constexpr int fdx(int d) { return d == 12 ? 1 : d / 4 - 1; }
__host__ __device__ constexpr int fdy(int d) { return d == 12 || d % 4 == 0 ? 0 : d % 4 == 3 ? -1 : 1; }
__host__ __device__ constexpr int fdz(int d) { return d == 12 || d % 4 == 1 ? 0 : 1; }
// The equal-level mask of a voxel: byte dx + 1 (bits 0..23) holds the eight
// neighbour rows, bit r < 4 the row opposite to forward row r, bit 4 + r
// forward row r; the voxel's own row has bit 27 (dx = -1) and 31 (dx = 1).
constexpr uint32_t kFwdBits = 0x80f0f0f0u, kBackBits = 0x080f0f0fu;
__host__ __device__ constexpr int fwd_bit(int d) { return d == 12 ? 31 : 8 * (d / 4) + 4 + d % 4; }
__host__ __device__ constexpr int back_bit(int d) { return d == 12 ? 27 : 8 * (2 - d / 4) + d % 4; }
// The backward bits with the dx = 0 byte first, so that the lowest set bit
// is the neighbour that most of the others are neighbours of: bit position
// of direction d's opposite in that order.
__host__ __device__ constexpr int zone_bit(int d) {
  return d == 12 ? 27 : (d / 4 == 1 ? 0 : d / 4 == 2 ? 8 : 16) + d % 4;
}
// Zone bits of the opposites that are neighbours of direction d's opposite
// (or are it).
__host__ __device__ constexpr uint32_t dir_cover(int d) {
  uint32_t m = 0;
  for (int n = 0; n < 13; ++n) {
    const int x = fdx(n) - fdx(d), y = fdy(n) - fdy(d), z = fdz(n) - fdz(d);
    if (x >= -1 && x <= 1 && y >= -1 && y <= 1 && z >= -1 && z <= 1) m |= 1u << zone_bit(n);
  }
  return m;
}
// The same as tables, for a direction known only at run time.
__constant__ signed char kDir[13][3] = {
    {fdx(0), fdy(0), fdz(0)},    {fdx(1), fdy(1), fdz(1)},    {fdx(2), fdy(2), fdz(2)},
    {fdx(3), fdy(3), fdz(3)},    {fdx(4), fdy(4), fdz(4)},    {fdx(5), fdy(5), fdz(5)},
    {fdx(6), fdy(6), fdz(6)},    {fdx(7), fdy(7), fdz(7)},    {fdx(8), fdy(8), fdz(8)},
    {fdx(9), fdy(9), fdz(9)},    {fdx(10), fdy(10), fdz(10)}, {fdx(11), fdy(11), fdz(11)},
    {fdx(12), fdy(12), fdz(12)}};
__constant__ uint32_t kDirCover[13] = {dir_cover(0), dir_cover(1), dir_cover(2),  dir_cover(3),  dir_cover(4),
                                       dir_cover(5), dir_cover(6), dir_cover(7),  dir_cover(8),  dir_cover(9),
                                       dir_cover(10), dir_cover(11), dir_cover(12)};
__host__ __device__ constexpr int ndx(int n) { return n < 13 ? fdx(n) : -fdx(n - 13); }
__host__ __device__ constexpr int ndy(int n) { return n < 13 ? fdy(n) : -fdy(n - 13); }
__host__ __device__ constexpr int ndz(int n) { return n < 13 ? fdz(n) : -fdz(n - 13); }

// 1/x from the hardware reciprocal refined by one Newton step (relative
// error ~1e-16; used where a quotient feeds a sum or a sign test).
__device__ inline double frcp(double x) {
  const double r0 = __builtin_amdgcn_rcp(x);
  return fma(fma(-x, r0, 1.0), r0, r0);
}

// a / b of normal b != 0 from frcp and one correction of the quotient (the
// residual is exact in the FMA): six instructions where the division, which
// scales for the range's ends, takes eleven.  A voxel has some twenty
// quotients and roots; with them so, the positions and triangles from
// tables (below) and the co-occurrence counts handed to the MCC kernel in
// the pass that sums them, 5.9 k -> 4.7 k VALU instructions a voxel at
// radius 3 (12.2 -> 11.4 ms for 1 M voxels, LDS and latency then showing),
// 3.7 k -> 3.0 k at radius 2 (100 k voxels: 0.77 -> 0.68 ms).
__device__ inline double fdiv(double a, double b) {
  const double r = frcp(b), q = a * r;
  return fma(fma(-b, q, a), r, q);
}

// sqrt(x) of a positive normal x from the hardware reciprocal square root
// and one Newton step (relative error ~1e-16).
__device__ inline double fsqrt(double x) {
  const double r = __builtin_amdgcn_rsq(x), g = x * r;
  return fma(g, fma(-0.5 * r, g, 0.5), g);
}

// log2 of a positive finite normal x, for the entropy terms: x = m 2^e with
// m in [1/sqrt 2, sqrt 2), ln m = 2 atanh(s), s = (m - 1) / (m + 1) (|s| <=
// 0.1716), by the odd series of atanh to s^15.  The first omitted term,
// 2 s^17 / 17 <= 1.2e-14 in ln m, bounds the error at about 2e-14 absolute
// in log2 (some hundred ulps near m = sqrt 2; the entropies it feeds are
// compared at 1e-5 relative).  Exact for powers of two.  About a third of
// the instructions of the library's double-double log2.
__device__ inline double flog2(double x) {
  int e;
  double m = frexp(x, &e);  // m in [0.5, 1)
  if (m < 0.70710678118654752) {
    m *= 2.0;
    e -= 1;
  }
  const double s = (m - 1.0) * frcp(m + 1.0), s2 = s * s;
  double t = 1.0 / 15.0;
  t = fma(t, s2, 1.0 / 13.0);
  t = fma(t, s2, 1.0 / 11.0);
  t = fma(t, s2, 1.0 / 9.0);
  t = fma(t, s2, 1.0 / 7.0);
  t = fma(t, s2, 1.0 / 5.0);
  t = fma(t, s2, 1.0 / 3.0);
  t = fma(t, s2, 1.0);
  constexpr double k2OverLn2 = 2.8853900817779268;  // 2 / ln 2
  return fma(s * t, k2OverLn2, (double)e);
}

// Tables of the integer arguments that the feature sums take: a load that
// the vector cache serves in place of the instructions of a logarithm
// (about 28) or a reciprocal (6).
template <int N>
struct Table {
  double v[N];
};
// log2 of c >= 1 for the table: c = m 2^e, m in [1, 2), halved above sqrt 2,
// then the series of flog2 to s^31 (its remainder is below 1e-26).
constexpr double table_log2(unsigned c) {
  int e = 0;
  while ((c >> (e + 1)) != 0u) ++e;
  double m = (double)c / (double)(1u << e);
  if (m > 1.4142135623730951) {
    m *= 0.5;
    ++e;
  }
  const double s = (m - 1.0) / (m + 1.0), s2 = s * s;
  double t = 0.0;
  for (int k = 31; k >= 1; k -= 2) t = t * s2 + 1.0 / k;
  return (double)e + s * t * 2.8853900817779268;  // 2 / ln 2
}
// c log2 c for every count of a neighbourhood of radius 3 or less (the
// largest, the co-occurrence total of a full 7^3 cube, is 6,516).
constexpr int kXLogN = 6528;
constexpr Table<kXLogN> make_xlog2x() {
  Table<kXLogN> t{};
  for (int c = 2; c < kXLogN; ++c)
    t.v[c] = (c & 1) ? c * table_log2(c) : 2.0 * t.v[c / 2] + c;  // 2k log2 2k = 2 (k log2 k) + 2k, exact scaling
  return t;
}
__device__ const Table<kXLogN> kXLog2X = make_xlog2x();
// 1 / n^2 for levels and run, zone and dependence sizes (at most 11^3).
constexpr int kInvSqN = 1332;
constexpr Table<kInvSqN> make_inv_sq() {
  Table<kInvSqN> t{};
  for (int c = 1; c < kInvSqN; ++c) t.v[c] = 1.0 / ((double)c * c);
  return t;
}
__device__ const Table<kInvSqN> kInvSq = make_inv_sq();
// Positions of a (2R+1)^3 cube, x fastest: x, y, z and the row of the
// bordered cube, (z + 1)(2R + 3) + y + 1, a byte each; beyond the cube (up to
// the next multiple of 64) coordinates that no bounds admit.  A load in
// place of the divisions by the side (17 instructions a position).
template <int R>
struct PosTable {
  static constexpr int S = 2 * R + 1, C = S * S * S, N = (C + 63) / 64 * 64;
  uint32_t v[N];
};
template <int R>
constexpr PosTable<R> make_positions() {
  using P = PosTable<R>;
  PosTable<R> t{};
  for (int c = 0; c < P::N; ++c) {
    const uint32_t x = c % P::S, y = c / P::S % P::S, z = c / (P::S * P::S);
    t.v[c] = c < P::C ? x | y << 8 | z << 16 | ((z + 1) * (P::S + 2) + y + 1) << 24 : 0x7f7f7fu;
  }
  return t;
}
template <int R>
__device__ const PosTable<R> kPos = make_positions<R>();
// Entries of an upper triangle of up to 64 columns, e = c (c + 1) / 2 + r:
// r and c, a byte each (a load in place of nine instructions).
constexpr int kTriN = 64 * 65 / 2;
struct TriTable {
  uint16_t v[kTriN];
};
constexpr TriTable make_triangle() {
  TriTable t{};
  int e = 0;
  for (int c = 0; c < 64; ++c)
    for (int r = 0; r <= c; ++r) t.v[e++] = (uint16_t)(r | c << 8);
  return t;
}
__device__ const TriTable kTri = make_triangle();
// c log2 c of a count of a radius-R neighbourhood (0 for c = 0).
template <int R>
__device__ inline double xlog2x(uint32_t c) {
  if constexpr (R <= 3) return kXLog2X.v[c];
  return c < (uint32_t)kXLogN ? kXLog2X.v[c] : (double)c * flog2((double)c);
}

}  // namespace
}  // namespace fr
