// Banded FTCG coefficient matrix C (Sec. III-C eq:ftcg, eq:cr; Sec. IV
// eq:twodftcg) and its application c = C fhat ahead of the spreading
// (tau = Omega C fhat).
//
// C is the band-constrained minimiser of ||T C - I||_F, T the truncated Gram
// matrix of the data frame (T_in = prod_a sinc(k_ia - k_na) within
// ||k_i - k_n||_inf <= R) and the band J(n) = {n - r + 1 .. n + r - 1} in
// the caller's sample (raster) order. Column n solves the least-squares
// problem min ||T[:, J(n)] c - e_n||, i.e. the normal equations
//   (T_J^T T_J) c = T_J^T e_n = (T_{n,j})_{j in J(n)}.
// Every entry of T_J^T T_J is an entry of the band of T^2 of half-width
// 2r - 2: (T^2)_{a,b} for a, b in J(n). So:
//   1. P[a][e] = pi^(2 DIM) (T^2)_{a, a+e}, e = 0 .. 2r-2. 2D: k_band_gram_mm,
//      a wavefront per run of consecutive samples, the contraction over the
//      candidates on the matrix cores; runs whose samples lie too far apart
//      for that, and 1D: k_band_gram, one thread per sample a, walking
//      a's neighbour bins once per pass of up to BAND_NC offsets e (each
//      candidate i: T_ia and T_{i,a+e}; T_ia = 0 outside a's box, so a's box
//      is the whole sum), every product rounded to a multiple of 2^-36
//      (wq_product), so that its sums are exact in any order;
//   2. k_band_solve: per column n, the (2r-1)^2 normal matrix gathered from
//      P, the right-hand side from the pair terms of n, and a float64
//      elimination over 16 lanes; writes C by columns;
//   3. k_band_apply: c_i = sum_{|n - i| < r} C[i, n] fhat_n in float64, one
//      thread per sample, the columns of its neighbours through LDS.
#include <algorithm>

#include "ftcg_internal.h"
#include "wbins.h"

namespace ftcg {

constexpr int BAND_BLOCK = 256;
constexpr int BAND_NC = 8;   // band offsets per pass of the T^2 kernel

__device__ inline double rcp64b(double x) {
  const double r = __builtin_amdgcn_rcp(x);
  return fma(r, fma(-x, r, 1.0), r);
}

// pi^DIM T_in of candidate o for sample (x, sn, cs), exactly 0 outside the
// box ||k_i - k_n||_inf <= R. Per axis sin(pi d) comes from the per-sample
// sine and cosine by the difference formula, products rounded separately, so
// the value does not depend on which of the two samples is the candidate;
// num / den with eps = 2^-500 added gives pi at d = 0 (as for the diagonal
// weights).
template <int DIM>
__device__ inline double band_term(const WSample<DIM>& o, const double* x, const double* sn, const double* cs,
                                   double R) {
#pragma clang fp contract(off)
  double num = 1.0, den = 1.0, dmax = 0.0;
#pragma unroll
  for (int a = 0; a < DIM; ++a) {
    const double d = o.k[a] - x[a];
    dmax = a == 0 ? fabs(d) : fmax(dmax, fabs(d));
    const double p1 = o.sc[a][0] * cs[a];
    const double p2 = o.sc[a][1] * sn[a];
    num *= (p1 - p2) + 0x1p-500 * WPI;
    den *= d + 0x1p-500;
  }
  const double q = num * rcp64b(den);
  return dmax <= R ? q : 0.0;
}

// a * b rounded to a multiple of 2^-36 (|a b| <= pi^4 < 2^16)
__device__ inline double wq_product(double a, double b) { return fma(a, b, WQ_MAGIC) - WQ_MAGIC; }

template <int DIM>
__device__ inline void load_sample(const WSample<DIM>& w, double* x, double* sn, double* cs) {
#pragma unroll
  for (int a = 0; a < DIM; ++a) {
    x[a] = w.k[a];
    sn[a] = w.sc[a][0];
    cs[a] = w.sc[a][1];
  }
}

template <int DIM, int NC>
__global__ __launch_bounds__(BAND_BLOCK) void k_band_gram(const WSample<DIM>* __restrict__ ss,
                                                         const int32_t* __restrict__ inv,
                                                         const int32_t* __restrict__ boff, int64_t m, WBinGeom g,
                                                         int nband, const int32_t* __restrict__ run_far, int stride,
                                                         int* __restrict__ bad, double* __restrict__ P) {
  const int64_t a = (int64_t)blockIdx.x * BAND_BLOCK + threadIdx.x;
  const int e0 = blockIdx.y * NC;
  if (a == 0 && e0 == 0) *bad = 0;   // counted by the solve
  if (a >= m || (run_far && !run_far[a / stride])) return;
  double x[DIM], sn[DIM], cs[DIM];
  load_sample<DIM>(ss[inv[a]], x, sn, cs);
  double cx[NC][DIM], csn[NC][DIM], ccs[NC][DIM], acc[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int64_t j = std::min<int64_t>(a + e0 + c, m - 1);   // past the end: repeated, never stored
    load_sample<DIM>(ss[inv[j]], cx[c], csn[c], ccs[c]);
    acc[c] = 0.0;
  }
  int b[DIM];
  wbin_of<DIM>(x, g, b);
  const int lo0 = max(b[0] - g.span, 0), hi0 = min(b[0] + g.span, g.nb[0] - 1);
  const int lo1 = DIM == 2 ? max(b[DIM - 1] - g.span, 0) : 0;
  const int hi1 = DIM == 2 ? min(b[DIM - 1] + g.span, g.nb[DIM - 1] - 1) : 0;
  for (int b0 = lo0; b0 <= hi0; ++b0) {
    const int first = DIM == 2 ? b0 * g.nb[1] + lo1 : b0;
    const int last = DIM == 2 ? b0 * g.nb[1] + hi1 : b0;
    const int beg = boff[first], end = boff[last + 1];
    for (int i = beg; i < end; ++i) {
      const WSample<DIM> o = ss[i];
      const double qa = band_term<DIM>(o, x, sn, cs, g.R);
      if (qa == 0.0) continue;   // outside a's box: every product is 0
#pragma unroll
      for (int c = 0; c < NC; ++c) acc[c] += wq_product(qa, band_term<DIM>(o, cx[c], csn[c], ccs[c], g.R));
    }
  }
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int e = e0 + c;
    if (e < nband && a + e < m) P[a * nband + e] = acc[c];
  }
}

// The band of T^2 of one run of consecutive samples per wavefront: samples
// a0 .. a0 + 16 NBK - 1 in NBK blocks of 16, P[a][e] for the first `stride` of
// them (a + e stays inside the blocks). Each step takes four candidates: lane (c, g)
// forms T_{i,j} of candidate g with sample c of every block, which is the
// operand layout of v_mfma_f64_16x16x4_f64 for both factors, and one
// instruction per block adds T_ia T_ij over the four candidates for 16 x 16
// pairs (a, j). So each T_{i,j} is formed once per run instead of once per sample
// whose band holds it. The candidates are the bins around the run's
// bounding box; a run that jumps by more than 2R between two samples (the end of a
// pulse) is walked in parts, each with its own box and its samples alone as
// the left factor. A run whose parts hold more bins than the samples' own
// windows are worth (each sample's window once for its own terms, and about
// half of it in the box for the band's; both counted in T terms) is left to
// k_band_gram (run_far). Fixed order of addition. Float64 issue bounds it: at 512^2
// with r = 8, 2^17 samples, 191 us against 687 us for one thread per
// sample.
typedef double double4_t __attribute__((ext_vector_type(4)));

// numerator and denominator of band_term, and its box test; the shift of the
// denominators is 2^-160 here, so that the product of three blocks' is normal
// (2^-960 at least; the shift vanishes against any |k_i - k_n| above 2^-107)
__device__ inline bool pair_parts(const WSample<2>& o, const double* x, const double* sn, const double* cs, double R,
                                  double* num, double* den) {
#pragma clang fp contract(off)
  constexpr double EPS = 0x1p-160;
  double nu = 1.0, de = 1.0, dmax = 0.0;
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    const double d = o.k[a] - x[a];
    dmax = a == 0 ? fabs(d) : fmax(dmax, fabs(d));
    const double p1 = o.sc[a][0] * cs[a];
    const double p2 = o.sc[a][1] * sn[a];
    nu *= (p1 - p2) + EPS * WPI;
    de *= d + EPS;
  }
  *num = nu;
  *den = de;
  return dmax <= R;
}

// num / den of N pairs with one reciprocal, of the product of the denominators
template <int N>
__device__ inline void quotients(const double* num, const double* den, double* t) {
  double pre[N];
  pre[0] = den[0];
#pragma unroll
  for (int b = 1; b < N; ++b) pre[b] = pre[b - 1] * den[b];
  double r = rcp64b(pre[N - 1]);
#pragma unroll
  for (int b = N - 1; b > 0; --b) {
    t[b] = num[b] * (r * pre[b - 1]);
    r *= den[b];
  }
  t[0] = num[0] * r;
}

template <int NBK>
__global__ __launch_bounds__(BAND_BLOCK, NBK == 1 ? 8 : NBK == 2 ? 6 : 4) void k_band_gram_mm(const WSample<2>* __restrict__ ss,
                                                            const int32_t* __restrict__ inv,
                                                            const int32_t* __restrict__ boff, int64_t m, WBinGeom g,
                                                            int nband, int stride, int32_t* __restrict__ run_far,
                                                            double* __restrict__ P) {
  const int lane = threadIdx.x & 63, c = lane & 15, q = lane >> 4;
  const int64_t run = xcd_block(blockIdx.x, gridDim.x) * (BAND_BLOCK / 64) + (threadIdx.x >> 6);
  const int64_t a0 = run * stride;
  if (a0 >= m) return;   // no barrier below: wavefronts are independent
  double x[NBK][2], sn[NBK][2], cs[NBK][2];
  bool ok[NBK];
#pragma unroll
  for (int b = 0; b < NBK; ++b) {
    const int64_t j = a0 + 16 * b + c;
    ok[b] = j < m;
    load_sample<2>(ss[inv[std::min<int64_t>(j, m - 1)]], x[b], sn[b], cs[b]);
  }
  int bin[2];
  wbin_of<2>(x[0], g, bin);
  const int na = (int)std::min<int64_t>(stride, m - a0);
  const double px = __shfl(x[0][0], (lane - 1) & 63), py = __shfl(x[0][1], (lane - 1) & 63);
  const bool brk = c < na && (c == 0 || fmax(fabs(x[0][0] - px), fabs(x[0][1] - py)) > 2.0 * g.R);
  const unsigned starts = (unsigned)__ballot(brk) & 0xffffu;
  // bins around the part of the run that starts at sample s: rows, columns
  auto part = [&](int s, int e, int* lo, int* hi) {
    const bool in = c >= s && c < e;
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      int l = in ? bin[a] : 1 << 30, h = in ? bin[a] : -1;
#pragma unroll
      for (int o = 1; o < 16; o <<= 1) {
        l = min(l, __shfl_xor(l, o));
        h = max(h, __shfl_xor(h, o));
      }
      lo[a] = __builtin_amdgcn_readfirstlane(max(l - g.span, 0));
      hi[a] = __builtin_amdgcn_readfirstlane(min(h + g.span, g.nb[a] - 1));
    }
  };
  auto next = [&](int s) {   // end of the part that starts at s
    const unsigned later = starts & ~((2u << s) - 1u);
    return later ? __ffs(later) - 1 : na;
  };
  int64_t cells = 0;
  for (int s = 0; s < na;) {
    const int e = next(s);
    int lo[2], hi[2];
    part(s, e, lo, hi);
    cells += (int64_t)(hi[0] - lo[0] + 1) * (hi[1] - lo[1] + 1);
    s = e;
  }
  const int w = 2 * g.span + 1;
  const bool far = 2 * cells * 16 * NBK > (int64_t)na * w * w * (2 + nband);
  if (lane == 0) run_far[run] = far;
  if (far) return;
  double4_t acc[NBK];
#pragma unroll
  for (int b = 0; b < NBK; ++b) acc[b] = (double4_t){0.0, 0.0, 0.0, 0.0};
  for (int s = 0; s < na;) {
    const int e = next(s);
    const bool in = c >= s && c < e;
    int lo[2], hi[2];
    part(s, e, lo, hi);
    for (int b0 = lo[0]; b0 <= hi[0]; ++b0) {
      const int beg = boff[b0 * g.nb[1] + lo[1]], end = boff[b0 * g.nb[1] + hi[1] + 1];
      for (int i0 = beg; i0 < end; i0 += 4) {
        const int i = i0 + q;
        const WSample<2> o = ss[min(i, end - 1)];
        const double dx = o.k[0] - x[0][0], dy = o.k[1] - x[0][1];
        const bool left = in && i < end && fmax(fabs(dx), fabs(dy)) <= g.R;
        if (!__any(left)) continue;
        double num[NBK], den[NBK], t[NBK];
        bool box[NBK];
#pragma unroll
        for (int b = 0; b < NBK; ++b) box[b] = pair_parts(o, x[b], sn[b], cs[b], g.R, &num[b], &den[b]) && ok[b];
        quotients<NBK>(num, den, t);
        const double ta = left ? t[0] : 0.0;   // past the row's end and for other parts' samples: 0
#pragma unroll
        for (int b = 0; b < NBK; ++b)
          acc[b] = __builtin_amdgcn_mfma_f64_16x16x4f64(ta, box[b] ? t[b] : 0.0, acc[b], 0, 0, 0);
      }
    }
    s = e;
  }
#pragma unroll
  for (int b = 0; b < NBK; ++b)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int a = 4 * v + q, e = 16 * b + c - a;   // accumulator v of lane (c, q): row 4v + q, column c
      if (a < na && e >= 0 && e < nband && a0 + a + e < m) P[(a0 + a) * nband + e] = acc[b][v];
    }
}

// element K of a group of GW lanes (a row of 16, or four), in every lane of the group
template <int K, int GW>
__device__ inline double row_bcast(double v) {
  static_assert(GW == 16 || GW == 4, "DPP broadcasts within a row or a quad");
  constexpr int CTRL = GW == 16 ? 0x150 + K : K * 0x55;
  const long long b = __builtin_bit_cast(long long, v);
  const int lo = __builtin_amdgcn_mov_dpp((int)b, CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xf, 0xf, true);
  return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned)lo);
}

// Step K of the elimination: every other row loses its entry in column K
// (columns K + 1 .. and the right-hand side are kept up to date). Row p is in
// lane p % GW, set p / GW. ok clears when the pivot vanishes.
template <int K, int NBP, int NS, int GW>
__device__ inline void band_step(double (&A)[NS][NBP], double (&y)[NS], double (&ip)[NS], const double (&d0)[NS],
                                 int c, bool& ok) {
  constexpr int S = K / GW, KL = K % GW;
  __builtin_amdgcn_sched_barrier(0);   // the next steps' broadcasts would not fit the registers
  const double piv = row_bcast<KL, GW>(A[S][K]);
  ok = ok && piv > 1e-13 * row_bcast<KL, GW>(d0[S]);
  double r = rcp64b(piv);
  r = fma(r, fma(-piv, r, 1.0), r);
  double f[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const bool self = s == S && c == KL;
    f[s] = self ? 0.0 : A[s][K] * r;
    if (self) ip[s] = r;
  }
#pragma unroll
  for (int t = K + 1; t < NBP; ++t) {
    const double e = row_bcast<KL, GW>(A[S][t]);
#pragma unroll
    for (int s = 0; s < NS; ++s) A[s][t] = fma(-f[s], e, A[s][t]);
  }
  const double e = row_bcast<KL, GW>(y[S]);
#pragma unroll
  for (int s = 0; s < NS; ++s) y[s] = fma(-f[s], e, y[s]);
  if constexpr (K + 1 < NBP) band_step<K + 1, NBP, NS, GW>(A, y, ip, d0, c, ok);
}

// Column n of C per group of GW lanes (16; four for r <= 2): the L x L normal matrix of J(n), padded
// to NBP with the identity, row p in the registers of lane p % GW (set
// p / GW), eliminated in place without a back substitution (in lockstep lanes
// the rows above the pivot cost nothing extra). Pivots are the Cholesky
// factorisation's (its squared diagonal); one vanishing against the
// matrix's diagonal entry reports a column without full rank. Measured at 2^17
// columns, r = 8: 51 us, against 241 us for one thread per column with the
// triangle in LDS (69 KB per wavefront, two wavefronts per compute unit).
template <int DIM, int NBP, int GW>
__global__ __launch_bounds__(BAND_BLOCK) void k_band_solve(const double* __restrict__ P,
                                                          const WSample<DIM>* __restrict__ ss,
                                                          const int32_t* __restrict__ inv, int64_t m, int r, double R,
                                                          double* __restrict__ bcol, int* __restrict__ bad) {
  constexpr int NS = (NBP + GW - 1) / GW;
  const int c = threadIdx.x % GW;
  const int64_t n = ((int64_t)blockIdx.x * BAND_BLOCK + threadIdx.x) / GW;
  if (n >= m) return;   // whole groups of lanes; no barrier below
  const int nb = 2 * r - 1;
  const int64_t lo = std::max<int64_t>(0, n - r + 1), hi = std::min<int64_t>(m - 1, n + r - 1);
  const int L = (int)(hi - lo + 1);
  const int off = (int)(lo - (n - r + 1));   // band position of J(n)'s first member
  double A[NS][NBP], y[NS], ip[NS], d0[NS];
  double x[DIM], sn[DIM], cs[DIM];
  load_sample<DIM>(ss[inv[n]], x, sn, cs);
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const int p = GW * s + c;
    const bool row = p < L;
#pragma unroll
    for (int t = 0; t < NBP; ++t) {
      const bool on = row && t < L;
      const double v = P[on ? (lo + min(p, t)) * nb + abs(p - t) : lo * nb];
      A[s][t] = on ? v : (p == t ? 1.0 : 0.0);
    }
    d0[s] = row ? P[(lo + p) * nb] : 1.0;
    y[s] = row ? band_term<DIM>(ss[inv[lo + p]], x, sn, cs, R) : 0.0;
    ip[s] = 1.0;
  }
  bool ok = true;
  band_step<0, NBP, NS, GW>(A, y, ip, d0, c, ok);
  if (!ok && c == 0) atomicAdd(bad, 1);
  // the sums carry pi^(2 DIM), the right-hand side pi^DIM: C = pi^DIM x
  constexpr double SC = DIM == 1 ? WPI : WPI * WPI;
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const int p = GW * s + c;
    if (p < L) bcol[n * nb + off + p] = ok ? SC * (y[s] * ip[s]) : 0.0;
    if (p < nb && (p < off || p >= off + L)) bcol[n * nb + p] = 0.0;
  }
}

// c_i: C[i, n] at [n][i - n + r - 1] of the column form. A workgroup's columns
// are read once, in order, and each thread takes its anti-diagonal from
// LDS (odd row length: no bank conflicts).
constexpr int APPLY_NT = 128;
template <class cx>
__global__ __launch_bounds__(APPLY_NT) void k_band_apply(const double* __restrict__ bcol,
                                                        const cx* __restrict__ fhat, int64_t m, int r,
                                                        cx* __restrict__ out) {
  extern __shared__ double sc[];   // (APPLY_NT + 2 (r - 1)) x (2r - 1)
  const int64_t i0 = (int64_t)blockIdx.x * APPLY_NT, i = i0 + threadIdx.x;
  const int nb = 2 * r - 1, rows = APPLY_NT + 2 * (r - 1);
  const int64_t first = (i0 - (r - 1)) * nb;
#pragma unroll 4
  for (int t = threadIdx.x; t < rows * nb; t += APPLY_NT) {
    const int64_t at = first + t;
    const bool on = at >= 0 && at < m * nb;
    const double v = bcol[on ? at : 0];
    sc[t] = on ? v : 0.0;
  }
  __syncthreads();
  if (i >= m) return;
  double re = 0.0, im = 0.0;
#pragma unroll 4
  for (int e = 0; e < nb; ++e) {
    const int64_t n = i + e - (r - 1);
    const bool on = n >= 0 && n < m;
    const double c = sc[(threadIdx.x + e) * nb + (nb - 1 - e)];
    const cx v = fhat[on ? n : i];
    re = fma(c, on ? (double)v.x : 0.0, re);
    im = fma(c, on ? (double)v.y : 0.0, im);
  }
  cx o;
  o.x = (decltype(o.x))re;
  o.y = (decltype(o.y))im;
  out[i] = o;
}

// samples per run of the matrix-core band: blocks of 16, and how many of the
// first have their whole band inside them (one block up to r = 5, where 16 -
// 2(r - 1) >= 8 samples per block still beat forming a second one; two up to r = 9)
static int run_blocks(int r) { return r <= 5 ? 1 : r <= 9 ? 2 : 3; }
static int run_stride(int r) { return std::min(16, 16 * run_blocks(r) - 2 * (r - 1)); }

// Bands of r <= 3 have at most five offsets, which k_band_gram forms in one pass
// with each T_{i,j} formed at most five times; a run of 12 or 14 samples then
// gains nothing over its wider box and leaves a good part of the runs to that
// kernel all the same. 59 515 samples on 448^2, points: r = 2 330 us by runs,
// 240 without; r = 3 281 and 244; r = 4 203 and 254; r = 5 152 and 412.
static bool band_by_runs(int r) { return r > 3; }

template <int DIM>
static void launch_band(ftcg_plan p) {
  const int64_t m = p->m;
  const int r = p->band_r, nb = 2 * r - 1;
  hipStream_t s = p->stream;
  const WSample<DIM>* ss = p->ws_k.as<WSample<DIM>>();
  const int32_t* inv = p->ws_inv.as<int32_t>();
  const unsigned gb = (unsigned)((m + BAND_BLOCK - 1) / BAND_BLOCK);
  const int32_t* boff = p->wb_off.as<int32_t>();
  double* P = p->band_P.as<double>();
  int* bad = reinterpret_cast<int*>(p->flags.as<double>() + 8);
  timing_begin(p, STEP_BAND_GRAM);
  const int32_t* far = nullptr;
  const int stride = run_stride(r);
  if constexpr (DIM == 2) {
    if (band_by_runs(r)) {
      const int64_t runs = (m + stride - 1) / stride;
      p->band_far.ensure(sizeof(int32_t) * runs);
      const int nbk = run_blocks(r);
      hipLaunchKernelGGL(nbk == 1 ? k_band_gram_mm<1> : nbk == 2 ? k_band_gram_mm<2> : k_band_gram_mm<3>,
                         dim3((unsigned)((runs + BAND_BLOCK / 64 - 1) / (BAND_BLOCK / 64))), dim3(BAND_BLOCK), 0, s,
                         ss, inv, boff, m, p->wgeom, nb, stride, p->band_far.as<int32_t>(), P);
      far = p->band_far.as<int32_t>();
    }
  }
  hipLaunchKernelGGL((k_band_gram<DIM, BAND_NC>), dim3(gb, (unsigned)((nb + BAND_NC - 1) / BAND_NC)), dim3(BAND_BLOCK),
                     0, s, ss, inv, boff, m, p->wgeom, nb, far, stride, bad, P);
  FTCG_HIP(hipGetLastError());
  timing_end(p, STEP_BAND_GRAM);
  timing_begin(p, STEP_BAND_SOLVE);
  const int gw = r <= 2 ? 4 : 16;
  const unsigned gs = (unsigned)((m * gw + BAND_BLOCK - 1) / BAND_BLOCK);
  hipLaunchKernelGGL((r <= 2    ? k_band_solve<DIM, 3, 4>
                      : r <= 3  ? k_band_solve<DIM, 5, 16>
                      : r <= 4  ? k_band_solve<DIM, 7, 16>
                      : r <= 8  ? k_band_solve<DIM, 15, 16>
                      : r <= 12 ? k_band_solve<DIM, 23, 16>
                                : k_band_solve<DIM, 31, 16>),
                     dim3(gs), dim3(BAND_BLOCK), 0, s, P, ss, inv, m, r, p->R, p->band_col.as<double>(), bad);
  FTCG_HIP(hipGetLastError());
  timing_end(p, STEP_BAND_SOLVE);
  // columns whose normal matrix is not positive definite (T[:, J(n)] without
  // full column rank, e.g. two samples at the same location within r
  // positions): reported as an error of set_points
  int* hb = reinterpret_cast<int*>(p->host_flags + 8);
  FTCG_HIP(hipMemcpyAsync(hb, bad, sizeof(int), hipMemcpyDeviceToHost, s));
  FTCG_HIP(hipStreamSynchronize(s));
  p->band_bad = *hb;
  if (p->band_bad) throw StatusError{FTCG_EINVAL};
}

void run_band_weights(ftcg_plan p) {
  const int64_t m = p->m;
  const int nb = 2 * p->band_r - 1;
  p->band_P.ensure(sizeof(double) * m * nb);
  p->band_col.ensure(sizeof(double) * m * nb);
  p->band_c.ensure((p->dtype == FTCG_F64 ? 16 : 8) * (size_t)m);
  if (p->dim == 1)
    launch_band<1>(p);
  else
    launch_band<2>(p);
}

void band_apply(ftcg_plan p, const void* fhat) {
  const unsigned gb = (unsigned)((p->m + APPLY_NT - 1) / APPLY_NT);
  const int r = p->band_r;
  const size_t lds = sizeof(double) * (APPLY_NT + 2 * (r - 1)) * (2 * r - 1);   // r <= 16: 39 KiB
  timing_begin(p, STEP_BAND_APPLY);
  if (p->dtype == FTCG_F64)
    hipLaunchKernelGGL(k_band_apply<double2>, dim3(gb), dim3(APPLY_NT), lds, p->stream, p->band_col.as<double>(),
                       static_cast<const double2*>(fhat), p->m, r, p->band_c.as<double2>());
  else
    hipLaunchKernelGGL(k_band_apply<float2>, dim3(gb), dim3(APPLY_NT), lds, p->stream, p->band_col.as<double>(),
                       static_cast<const float2*>(fhat), p->m, r, p->band_c.as<float2>());
  FTCG_HIP(hipGetLastError());
  timing_end(p, STEP_BAND_APPLY);
}

}  // namespace ftcg
