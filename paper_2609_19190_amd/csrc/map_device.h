// Device helpers shared by the map kernels of this library (the fused
// fixed-radius kernel and the generic kernel): the 13 GLCM/GLRLM direction
// representatives, the exact NGTDM scale table, FP64 primitives and the
// Sturm counts of the MCC.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>

namespace fr {
namespace {

#define FR_INLINE __attribute__((always_inline))
template <int B, int E, typename F>
__host__ __device__ FR_INLINE inline void static_for(F&& f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    static_for<B + 1, E>(f);
  }
}

// A column with a smaller sum of squares is left as it is by the
// tridiagonalisation of the MCC's matrix (whose entries are of order 1): that
// changes no eigenvalue by more than 1e-30.  Levels with equal rows of
// counts leave a trailing block of nothing but rounding, of one rank itself,
// so that each reflection leaves 1e-16 of it: after ten of them 2 / v.v
// overflows, and the infinity spreads over the whole form.
constexpr double kNoColumn = 1e-60;

// ---- Sturm counts of the MCC searches (host code calls them in a test) ----
// Eigenvalues of the symmetric tridiagonal (d, e) inside [-x, x): the sign
// changes of the leading principal minors
//   p_0 = 1, p_1 = d_0 - y, p_i = (d_{i-1} - y) p_{i-1} - e_{i-2}^2 p_{i-2}
// count the eigenvalues below y; the sequences for y = x and y = -x run
// interleaved, without divisions.  Every minor has kMinorShift added, so
// that a zero minor counts as positive: right between two minors of opposite
// sign, and off by the eigenvalue that equals y otherwise, a probe exactly at
// a bracket's end.  The range: the spectrum and |y| lie within [-1, 1] but
// for rounding (an entry past a problem's end, kPastN, within 3 of y), so a
// step multiplies a minor by at most 3, and, with an m-fold eigenvalue a (m
// equal rows of a co-occurrence matrix; near a matrix of rank one a = 0), by
// as little as |a - y|.  The sequences start at kMinorOne and, past
// kMinorRun minors, go on from there again: a run of them stays between
// kMinorOne 3^32 = 2^951 and, down to |a - y| = 3e-18, above the shift.
// (From 1, without a second start, 64 levels lost the sign at |a - y| =
// 3e-5: MCCs off by that much.)
// The signs are shifted into a word as they come (one instruction a minor)
// and the changes counted at the end: four instructions a minor instead of
// ten.  With the reflections' reciprocals and roots by Newton steps 2.6 k ->
// 2.1 k VALU instructions a problem of 17..32 levels (k_mcc of 1 M voxels 5.4
// -> 4.5 ms; 2.0 k and 4.3 now), 1.1 k -> 0.8 k of the radius-2 workload (249
// -> 190 us).
constexpr double kMinorShift = 1e-290;
constexpr int kMinorOneExp = 900, kMinorRun = 32;
constexpr double kMinorOne = 0x1p900;
// acc with the top bit of h shifted in (one instruction on the GPU, where the
// general expression becomes two and its registers spill).
__host__ __device__ inline uint32_t push_bit(uint32_t acc, uint32_t h) {
#ifdef __HIP_DEVICE_COMPILE__
  return __builtin_amdgcn_alignbit(acc, h, 31);
#else
  return acc << 1 | h >> 31;
#endif
}
__host__ __device__ inline uint32_t push_sign(uint32_t acc, double p) {
  return push_bit(acc, (uint32_t)(__builtin_bit_cast(uint64_t, p) >> 32));
}
// The last two minors of a sequence, the larger one brought back to kMinorOne.
__host__ __device__ inline void minors_rescale(double& a, double& b) {
  int e;
  (void)frexp(fmax(fabs(a), fabs(b)), &e);
  a = ldexp(a, kMinorOneExp - e);
  b = ldexp(b, kMinorOneExp - e);
}
// Rounds of the searches: 17-way (16 probes a row) for up to 32 levels, 65-way
// (a probe a lane) beyond.  FINE (radii 4 and 5 and the extraction variants):
// no wider a last bracket than the generic kernel's, 1 / 257^4.
template <bool FINE>
constexpr int kRowRounds = FINE ? 8 : 6;
template <bool FINE>
constexpr int kBigRounds = FINE ? 6 : 4;
// n <= 64; D[i] = d_i and E2[i] = e_i^2 are (LDS) arrays, read as broadcasts.
// SEQ 3: Sturm count of [-x, x) (eigenvalues below x minus those below -x);
// SEQ 1: eigenvalues below x only; SEQ 2: eigenvalues below -x only.  The
// counts of 1 and 2 are the two terms of 3, computed the same way.
template <int SEQ = 3>
__host__ __device__ inline int sturm_span_r(const double* D, const double* E2, int n, double x) {
  const double d0 = D[0];
  double ap = (d0 - x) * kMinorOne, am = (d0 + x) * kMinorOne, bp = kMinorOne, bm = kMinorOne;
  uint32_t hp = 0, lp = push_sign(0, ap), hm = 0, lm = push_sign(0, am);
  auto run = [&](int i0, int i1) FR_INLINE {
#pragma unroll 4
    for (int i = i0; i < i1; ++i) {
      const double di = D[i], e2 = E2[i - 1];
      if constexpr (SEQ & 1) {
        const double np = fma(di - x, ap, fma(-e2, bp, kMinorShift));
        hp = push_bit(hp, lp);
        lp = push_sign(lp, np);
        bp = ap;
        ap = np;
      }
      if constexpr (SEQ & 2) {
        const double nm = fma(di + x, am, fma(-e2, bm, kMinorShift));
        hm = push_bit(hm, lm);
        lm = push_sign(lm, nm);
        bm = am;
        am = nm;
      }
    }
  };
  run(1, n < kMinorRun ? n : kMinorRun);
  if (n > kMinorRun) {
    if constexpr (SEQ & 1) minors_rescale(ap, bp);
    if constexpr (SEQ & 2) minors_rescale(am, bm);
    run(kMinorRun, n);
  }
  auto changes = [](uint32_t h, uint32_t l) FR_INLINE {
    return __builtin_popcount(h ^ (h >> 1)) + __builtin_popcount(l ^ (l >> 1 | h << 31));
  };
  const int cp = SEQ & 1 ? changes(hp, lp) : 0, cm = SEQ & 2 ? changes(hm, lm) : 0;
  return SEQ == 3 ? cp - cm : cp + cm;
}
// The same for a row's tridiagonal (D[i] = d_i and E2[i] = e_i^2 already
// broadcast to every lane of the row), N = 16 or 32 entries; past a
// problem's n they hold kPastN and 0, an eigenvalue above every probe, so
// that no entry needs a test.
constexpr double kPastN = 2.0;
template <int N, int SEQ = 3>
__host__ __device__ FR_INLINE inline int sturm_row(const double (&D)[N], const double (&E2)[N], double x) {
  static_assert(N <= 32 && N <= kMinorRun, "the signs fit a word, the minors their range");
  const double d0 = D[0];
  double ap = (d0 - x) * kMinorOne, am = (d0 + x) * kMinorOne, bp = kMinorOne, bm = kMinorOne;
  uint32_t sp = push_sign(0, ap), sm = push_sign(0, am);
  static_for<1, N>([&](auto ic) FR_INLINE {
    constexpr int i = decltype(ic)::value;
    const double di = D[i], e2 = E2[i - 1];
    if constexpr (SEQ & 1) {
      const double np = fma(di - x, ap, fma(-e2, bp, kMinorShift));
      sp = push_sign(sp, np);
      bp = ap;
      ap = np;
    }
    if constexpr (SEQ & 2) {
      const double nm = fma(di + x, am, fma(-e2, bm, kMinorShift));
      sm = push_sign(sm, nm);
      bm = am;
      am = nm;
    }
  });
  const int cp = SEQ & 1 ? __builtin_popcount(sp ^ (sp >> 1)) : 0, cm = SEQ & 2 ? __builtin_popcount(sm ^ (sm >> 1)) : 0;
  return SEQ == 3 ? cp - cm : cp + cm;
}

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

// Reciprocal and root from a seed r (the hardware's: relative errors up to
// 4.7e-8 and 5.3e-8 measured here, 2^-23 documented), by two Newton steps:
// correctly rounded but for a hair, a relative error of 2^-53 as 1 / x and
// sqrt have (one step leaves 2.2e-15 and 4.2e-15, 20 and 38 times as much).
// x normal and positive for the root.
__host__ __device__ inline double rcp_refine(double x, double r) {
  r = fma(fma(-x, r, 1.0), r, r);
  return fma(fma(-x, r, 1.0), r, r);
}
__host__ __device__ inline double sqrt_refine(double x, double r) {
  double g = x * r, h = 0.5 * r;
  const double e = fma(-h, g, 0.5);
  g = fma(g, e, g);
  h = fma(h, e, h);
  return fma(fma(-g, g, x), h, g);
}
__device__ inline double rcp64(double x) { return rcp_refine(x, __builtin_amdgcn_rcp(x)); }
__device__ inline double fsqrt(double x) { return sqrt_refine(x, __builtin_amdgcn_rsq(x)); }

// 1/x by one Newton step (relative error up to 2.2e-15): for terms of the
// sums where every entry takes one, and fdiv.
__device__ inline double frcp(double x) {
  const double r0 = __builtin_amdgcn_rcp(x);
  return fma(fma(-x, r0, 1.0), r0, r0);
}

// a / b of normal b != 0 from frcp and one correction of the quotient (the
// residual is exact in the FMA; 2^-53, as a / b): six instructions where the
// division, which scales for the range's ends, takes eleven.  A voxel has some twenty
// quotients and roots; with them so, the positions and triangles from
// tables (below) and the co-occurrence counts handed to the MCC kernel in
// the pass that sums them, 5.9 k -> 4.7 k VALU instructions a voxel at
// radius 3 (12.2 -> 11.4 ms for 1 M voxels, LDS and latency then showing),
// 3.7 k -> 3.0 k at radius 2 (100 k voxels: 0.77 -> 0.68 ms).
__device__ inline double fdiv(double a, double b) {
  const double r = frcp(b), q = a * r;
  return fma(fma(-b, q, a), r, q);
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
