"""The MCC's eigenvalue searches on the CPU: the kernels' own Sturm counts
(csrc/map_device.h, compiled for the host) in the kernels' brackets, on
tridiagonals whose spectral radius is known; and the reciprocals and roots of
its reflections from seeds as coarse as the hardware's may be."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from paper_2609_19190_amd import build

SOURCE = r"""
#include "map_device.h"
using namespace fr;
template <typename F>
static void search(int width, int rounds, double& lo, double& hi, F is_n) {
  for (int r = 0; r < rounds; ++r) {
    double at = lo, past = hi;
    bool found = false;
    for (int p = 1; p < width && !found; ++p) {
      const double x = lo + (hi - lo) * ((double)p / width);
      if (is_n(x)) past = x, found = true;
      else at = x;
    }
    lo = at;
    hi = past;
  }
}
template <typename C1, typename C2, typename C3>
static double radius(int width, int rounds, double gb, int n, C1 c1, C2 c2, C3 c3) {
  const double top = fmin(gb, 1.0) * (1.0 + 1e-12) + 1e-300;
  double lo = 0.0, hi = top;
  search(width, rounds, lo, hi, [&](double x) { return c1(x) == n; });
  if (c2(lo) != 0) {
    lo = 0.0, hi = top;
    search(width, rounds, lo, hi, [&](double x) { return c3(x) == n; });
  }
  return 0.5 * (lo + hi);
}
extern "C" double radius_span(const double* d, const double* e2, int n, double gb, int rounds) {
  return radius(65, rounds, gb, n, [&](double x) { return sturm_span_r<1>(d, e2, n, x); },
                [&](double x) { return sturm_span_r<2>(d, e2, n, x); },
                [&](double x) { return sturm_span_r<3>(d, e2, n, x); });
}
template <int N>
static double radius_row(const double* d, const double* e2, int n, double gb, int rounds) {
  double D[N], E[N];
  for (int i = 0; i < N; ++i) D[i] = i < n ? d[i] : kPastN, E[i] = i < n - 1 ? e2[i] : 0.0;
  return radius(17, rounds, gb, n, [&](double x) { return sturm_row<N, 1>(D, E, x); },
                [&](double x) { return sturm_row<N, 2>(D, E, x); }, [&](double x) { return sturm_row<N, 3>(D, E, x); });
}
extern "C" double rcp(double x, double r) { return rcp_refine(x, r); }
extern "C" double root(double x, double r) { return sqrt_refine(x, r); }
extern "C" int rounds(int rows, int fine) {
  return rows ? (fine ? kRowRounds<true> : kRowRounds<false>) : fine ? kBigRounds<true> : kBigRounds<false>;
}
extern "C" double radius_rows(const double* d, const double* e2, int n, double gb, int rounds) {
  return n <= 16 ? radius_row<16>(d, e2, n, gb, rounds) : radius_row<32>(d, e2, n, gb, rounds);
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("mcc")
    src, so = d / "search.hip", d / "search.so"
    src.write_text(SOURCE)
    r = subprocess.run([build.HIPCC, *build.FLAGS, "-O1", "-I", build.CSRC, "-shared", str(src), "-o", str(so)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    L = ctypes.CDLL(os.fspath(so))
    for f in (L.radius_span, L.radius_rows):
        f.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_int, ctypes.c_double, ctypes.c_int]
        f.restype = ctypes.c_double
    for f in (L.rcp, L.root):
        f.argtypes = [ctypes.c_double, ctypes.c_double]
        f.restype = ctypes.c_double
    return L


def run(f, d, e, rounds):
    d, e2 = np.ascontiguousarray(d, np.float64), np.ascontiguousarray(np.append(e, 0.0) ** 2, np.float64)
    a = np.abs(np.concatenate(([0.0], e, [0.0])))
    gb = float((np.abs(d) + a[:-1] + a[1:]).max())
    return f(d.ctypes.data, e2.ctypes.data, len(d), gb, rounds)


# the rounds the kernels run with: 65-way to 1 / 65^4, 17-way to 1 / 17^6
@pytest.mark.parametrize("n", [2, 3, 16, 17, 31, 32, 33, 48, 63, 64])
@pytest.mark.parametrize("top", [1.0, 0.3, 1.0 / 63, 1e-6, 1e-12, 0.0])
@pytest.mark.parametrize("kind", ["equal", "negative", "one", "noise"])
def test_radius_of_multiple_eigenvalues(lib, n, top, kind):
    """n or n - 1 eigenvalues of one size: equal rows of a co-occurrence
    matrix, or, with a radius near 0, one of rank one."""
    d, e = np.full(n, top), np.zeros(n - 1)
    if kind == "negative":
        d = -d
    elif kind == "one":  # the other eigenvalue is 0, as that of I - v v^T
        d[0], d[1], e[0] = 0.75 * top, 0.25 * top, np.sqrt(0.1875) * top
    elif kind == "noise":  # what rounding leaves beside them
        r = np.random.default_rng(n)
        d = d + r.uniform(-1, 1, n) * 1e-17
        e = r.uniform(-1, 1, n - 1) * 1e-17
    f, width = (lib.radius_rows, 17.0 ** -6) if n <= 32 else (lib.radius_span, 65.0 ** -4)
    got = run(f, d, e, 6 if n <= 32 else 4)
    # half the last bracket of one that began no wider than three radii
    # (Gershgorin), and the rounding of a bracket's end
    assert abs(got - top) <= 1.5 * top * width + 2e-12 * top + 1e-16


@pytest.mark.parametrize("n", [2, 9, 16, 17, 32, 33, 50, 64])
def test_radius_of_random_tridiagonals(lib, n):
    for seed in range(6):
        r = np.random.default_rng(100 * n + seed)
        d, e = r.uniform(-0.3, 0.3, n), r.uniform(-0.3, 0.3, n - 1)
        want = np.abs(np.linalg.eigvalsh(np.diag(d) + np.diag(e, 1) + np.diag(e, -1))).max()
        f, rounds, width = (lib.radius_rows, 6, 17.0 ** -6) if n <= 32 else (lib.radius_span, 4, 65.0 ** -4)
        assert abs(run(f, d, e, rounds) - want) <= 0.5 * width + 1e-13


@pytest.mark.parametrize("n", [2, 16, 20, 32, 33, 47, 64])
def test_finer_searches_err_no_more_than_the_generic_kernels(lib, n):
    """Radii 4 and 5 and the extraction variants: half of 1 / 257^4, the
    generic kernel's last bracket."""
    for seed in range(8):
        r = np.random.default_rng(1000 * n + seed)
        d, e = r.uniform(-0.4, 0.4, n), r.uniform(-0.3, 0.3, n - 1)
        want = np.abs(np.linalg.eigvalsh(np.diag(d) + np.diag(e, 1) + np.diag(e, -1))).max()
        f, rows = (lib.radius_rows, 1) if n <= 32 else (lib.radius_span, 0)
        assert abs(run(f, d, e, lib.rounds(rows, 1)) - want) <= 0.5 * 257.0 ** -4 + 1e-13
        width = 17.0 ** -6 if rows else 65.0 ** -4
        assert abs(run(f, d, e, lib.rounds(rows, 0)) - want) <= 0.5 * width + 1e-13


@pytest.mark.parametrize("seed_error", [0.0, 2.0 ** -23, -2.0 ** -23, 5.3e-8, -5.3e-8, 2.0 ** -30])
def test_reciprocals_and_roots_are_as_near_as_ieee_ones(lib, seed_error):
    """One rounding: 2^-53, and what two Newton steps leave of the seed's
    error (below 2^-88)."""
    r = np.random.default_rng(3)
    x = np.concatenate((r.uniform(1.0, 4.0, 3000), np.arange(1.0, 2000.0), 10.0 ** r.uniform(-40, 40, 500)))
    for v in x:
        v = np.longdouble(float(v))
        got = np.longdouble(lib.rcp(float(v), float((1 / v) * (1 + np.longdouble(seed_error)))))
        assert abs(got * v - 1) <= 2.0 ** -53 * (1 + 1e-3)
        got = np.longdouble(lib.root(float(v), float((1 / np.sqrt(v)) * (1 + np.longdouble(seed_error)))))
        assert abs(got / np.sqrt(v) - 1) <= 2.0 ** -53 * (1 + 1e-3)
