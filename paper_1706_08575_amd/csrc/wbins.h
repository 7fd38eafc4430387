// Neighbour bins of the frame-weight sum: bin lookup and the row-grouped
// sample record of the 2D two-level sort (shared by the weight and the
// binning sources).
#pragma once

#include "ftcg_internal.h"

namespace ftcg {

// bin of a sample that passed the input check
template <int DIM>
__device__ inline int wbin_of(const double* x, const WBinGeom& g, int* b) {
  int id = 0;
  for (int a = 0; a < DIM; ++a) {
    int v = (int)floor((x[a] - g.kmin[a]) / g.h);
    v = v < 0 ? 0 : (v >= g.nb[a] ? g.nb[a] - 1 : v);
    b[a] = v;
    id = id * g.nb[a] + v;
  }
  return id;
}

// a sample grouped by bin row: coordinates, caller index, bin column
struct RowRec {
  double k0, k1;
  int32_t j, b1;
};

// bin row and column of sample j, clamped in floating point (a NaN lands in
// the last row or column), so both are in range for any input: the row
// binning runs before the host has seen the input check
__device__ inline int wbin_row_col(const double* __restrict__ k, int64_t j, const WBinGeom& g, int* b1,
                                   double* x) {
  x[0] = k[2 * j];
  x[1] = k[2 * j + 1];
  int b[2];
  for (int a = 0; a < 2; ++a)
    b[a] = (int)fmax(0.0, fmin(floor((x[a] - g.kmin[a]) / g.h), (double)(g.nb[a] - 1)));
  *b1 = b[1];
  return b[0];
}

// 1/x: hardware float64 reciprocal estimate refined by one Newton step, which
// leaves an error of a few units in the last place
__device__ inline double rcp64(double x) {
  const double r = __builtin_amdgcn_rcp(x);
  return fma(r, fma(-x, r, 1.0), r);
}

// pi^(2 DIM) T_in^2 of one candidate i for sample n = (x, sn, cs), 0 outside
// the box (the kernels divide pi^(2 DIM) by the sum). Per axis, T factors into
// sin(pi d) / (pi d) with d = k_i - k_n; here num = sin(pi d) + pi eps and
// den = d + eps with eps = 2^-500. For d = 0, sin(pi d) comes out exactly 0
// (the per-sample sin and cos are equal bit for bit, and the two products are
// rounded separately, never fused), so num / den = pi: the factor pi * sinc(0)
// with no compare or select. For |d| >= 2^-447, d + eps == d and
// sin(pi d) + pi eps == sin(pi d) exactly, so nothing changes; eps^2 and
// (pi eps)^2 stay normal numbers. This keeps the loop body to plain float64
// arithmetic.
constexpr double WEPS = 0x1p-500;
constexpr double WPI_EPS = WPI * WEPS;

// pi^DIM T_in by the select-free form, or a value whose square is 0 when
// ||k_i - k_n||_inf > R
template <int DIM>
__device__ inline double pair_term(const WSample<DIM>& o, const double* x, const double* sn, const double* cs,
                                   double R) {
#pragma clang fp contract(off)
  double num = 1.0, den = 1.0, dmax = 0.0;
#pragma unroll
  for (int a = 0; a < DIM; ++a) {
    const double d = o.k[a] - x[a];
    dmax = a == 0 ? fabs(d) : fmax(dmax, fabs(d));
    // sin(pi (k_i - k_n)) = sin(pi k_i) cos(pi k_n) - cos(pi k_i) sin(pi k_n)
    const double p1 = o.sc[a][0] * cs[a];
    const double p2 = o.sc[a][1] * sn[a];
    num *= (p1 - p2) + WPI_EPS;
    den *= d + WEPS;
  }
  const double q = num * rcp64(den);
  // outside the box: clear the high word, which leaves at most 2^-1042, whose
  // square is 0
  const int hi = dmax <= R ? __double2hiint(q) : 0;
  return __hiloint2double(hi, __double2loint(q));
}

// acc + (pi^DIM T_in)^2, the square rounded to the sums' quantum (wq_square)
template <int DIM>
__device__ inline double pair_add(double acc, const WSample<DIM>& o, const double* x, const double* sn,
                                  const double* cs, double R) {
  return acc + wq_square(pair_term<DIM>(o, x, sn, cs, R));
}


// Bin edge h = R / span with span in [2, 16] chosen for about BIN_TARGET
// samples per bin at the raster's mean density over its bounding box, so the
// 2 span + 1 bins of a row range end at the box of radius R; at most 4096
// bins per axis in 2D (4M in 1D). Finer bins waste fewer out-of-box
// candidates but cut the candidates into more, shorter row ranges: measured
// on SAS rasters of 2^17, 2^20 and 2^23 samples (span 3 against span 4), the
// weight kernel took 0.053 / 0.507 / 2.23 ms against 0.058 / 0.528 / 2.21 ms.
constexpr double BIN_TARGET = 4.5;
constexpr double KMAX_ABS = 1099511627776.0;   // 2^40

__device__ inline double decode_ordered_dev(unsigned long long o) {
  const unsigned long long b = (o & 0x8000000000000000ull) ? (o & 0x7fffffffffffffffull) : ~o;
  return __longlong_as_double((long long)b);
}

// the answer of the input check from its reduced words (non-finite flag, per-axis
// minimum and maximum as order-preserving integers): points are rejected when one
// is non-finite or farther than 2^40 from the origin on an axis, and a rejected
// set still gets a valid one-bin geometry
__device__ inline CheckOut check_finish(const unsigned long long (&v)[5], int dim, int64_t m, double R) {
  CheckOut o;
  bool bad = v[0] != 0;
  for (int a = 0; a < 2; ++a) {
    o.kmin[a] = a < dim ? decode_ordered_dev(v[1 + a]) : 0.0;
    o.kmax[a] = a < dim ? decode_ordered_dev(v[3 + a]) : 0.0;
    bad = bad || !(o.kmin[a] >= -KMAX_ABS && o.kmax[a] <= KMAX_ABS);
  }
  WBinGeom g;
  g.R = R;
  if (bad) {
    g.kmin[0] = g.kmin[1] = 0.0;
    g.h = 1.0;
    g.nb[0] = g.nb[1] = 1;
    g.span = 1;
  } else {
    // bins of about BIN_TARGET samples at the mean density of the box, with
    // h = R / span exactly, so the 2 span + 1 bins of a row range end on the
    // box of radius R; at most max_bins bins per axis
    double vol = 1.0;
    for (int a = 0; a < 2; ++a)
      if (a < dim) vol *= fmax(o.kmax[a] - o.kmin[a], 1e-9);
    const double rho = (double)m / vol;
    const double h_target = dim == 2 ? sqrt(BIN_TARGET / rho) : BIN_TARGET / rho;
    const double sp = fmin(fmax(floor(R / h_target + 0.5), 2.0), 16.0);
    double h = R / sp;
    const double max_bins = dim == 1 ? (double)(1 << 22) : (double)WROW_MAX;
    for (int a = 0; a < 2; ++a) {
      const double ext = o.kmax[a] - o.kmin[a];
      if (a < dim && ext / h + 1.0 > max_bins) h = ext / (max_bins - 1.0);
    }
    g.h = h;
    g.span = (int)ceil(R / h);
    for (int a = 0; a < 2; ++a) {
      g.kmin[a] = a < dim ? o.kmin[a] : 0.0;
      g.nb[a] = a < dim ? (int)fmin(fmax(floor((o.kmax[a] - o.kmin[a]) / h) + 1.0, 1.0), max_bins) : 1;
    }
  }
  o.g = g;
  o.bad = bad ? 1 : 0;
  return o;
}

}  // namespace ftcg
