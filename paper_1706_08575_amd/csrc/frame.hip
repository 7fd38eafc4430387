// Dense frame approximation A_fr (Sec. III-B eq:binv, eq:afr, eq:afrm; 2D
// Sec. IV eq:twodframe, eq:twodframeB), the accuracy reference that the
// banded FTCG approximates, for small rasters.
//
//   zeta_n(x) = exp(2 pi i n . x) / w(x), modes n_a in -N/2 .. N/2 - 1 (the
//               admissible frame of eq:newadm on the pixel frequencies),
//               w(x) = Phi(x / sigma) per axis (the window the path divides by);
//   Psi_{j,n} = <phi_j, zeta_n> = prod_a g(k_ja - n_a),
//               g(t) = int_{-1/2}^{1/2} cos(2 pi t x) / w(x) dx;
//   beta      = Psi^dagger fhat (least squares when the samples are at
//               least as many as the modes, minimum norm otherwise);
//   A_fr(x_p) = sum_n beta_n exp(2 pi i n . x_p) / w(x_p).
//
// Steps, all float64:
//   1. k_gl_nodes: Gauss-Legendre nodes and weights of order Q = 4N + 64 on
//      [-1/2, 1/2] (Newton's method on P_Q from the three-term recurrence,
//      one thread per node), the weights divided by w at the nodes;
//   2. k_frame_axis: the per-axis tables g(k_ja - n_a) (one thread per entry);
//   3. the tall matrix of the QR: Psi with the real and imaginary parts of
//      fhat as two extra columns (m >= N^d), or Psi^T (m < N^d);
//   4. Householder QR: up to 4096 rows in tiles and panels (k_frame_tiles,
//      qr.hip); taller matrices column-major (k_frame_assemble) and one
//      column at a time, as their rows do not fit one workgroup's registers: k_house forms the unit reflector of column j in
//      place (R_jj apart), k_reflect applies it to every later column (one
//      workgroup per column);
//   5. the triangular solve (least squares: R beta = Q^T fhat; minimum norm:
//      R^T y = fhat, beta = Q [y; 0]), one workgroup (qr.hip);
//   6. the inverse DFT of beta on the N^d mode grid and the division by w:
//      the grid-to-image passes with G = N (no crop).
// The quadrature's nodes and the mode grid's twiddles depend on the plan
// alone and are formed by its first call.
#include "ftcg_internal.h"
#include "qr.h"

namespace ftcg {

constexpr int FR_BLOCK = 256;

// node i of Gauss-Legendre order Q (x in (-1, 1), weight), mapped to
// [-1/2, 1/2]; the weight is divided by w(x) = sqrt(pi / beta) e^{-pi^2 (x / sigma)^2 / beta}
__global__ void k_gl_nodes(int Q, double sigma, double beta, double* __restrict__ xq, double* __restrict__ cw) {
  // coefficients of P_j = a_j x P_{j-1} - b_j P_{j-2}, off the recurrence's
  // serial chain (with the division in it: 61 us at Q = 192)
  extern __shared__ double2 ab[];
  for (int j = 2 + threadIdx.x; j <= Q; j += blockDim.x) ab[j] = make_double2((2.0 * j - 1.0) / j, (j - 1.0) / j);
  __syncthreads();
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= Q) return;
  auto legendre = [&](double x, double* prev) {
    double p0 = 1.0, p1 = x;
    for (int j = 2; j <= Q; ++j) {
      const double p2 = fma(ab[j].x * x, p1, -ab[j].y * p0);
      p0 = p1;
      p1 = p2;
    }
    *prev = p0;
    return p1;
  };
  double x = cos(WPI * (i + 0.75) / (Q + 0.5));   // initial guess near the i-th root
  double dp = 1.0, p0;
  for (int it = 0; it < 100; ++it) {
    const double p1 = legendre(x, &p0);
    dp = Q * (x * p1 - p0) / (x * x - 1.0);       // P_Q'(x)
    const double dx = p1 / dp;
    x -= dx;
    if (fabs(dx) < 1e-16) break;
  }
  {
    const double p1 = legendre(x, &p0);
    dp = Q * (x * p1 - p0) / (x * x - 1.0);
  }
  const double wgt = 2.0 / ((1.0 - x * x) * dp * dp);
  const double xh = 0.5 * x;
  const double t = xh / sigma;
  const double w = sqrt(WPI / beta) * exp(-WPI * WPI * t * t / beta);
  xq[i] = xh;
  cw[i] = 0.5 * wgt / w;
}

// G[a][j][i] = g(k_ja - (i - N/2)), a < dim; four lanes share an entry's
// quadrature (one lane per entry left two wavefronts per SIMD to hide the
// chain of Q cosines: 35 us at 900 samples, N = 32)
constexpr int AXIS_LANES = 4;
__global__ void k_frame_axis(const double* __restrict__ k, int64_t m, int dim, int N, int Q,
                             const double* __restrict__ xq, const double* __restrict__ cw, double* __restrict__ G) {
  const int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t t = u / AXIS_LANES;
  if (t >= (int64_t)dim * m * N) return;   // whole groups of lanes
  const int i = (int)(t % N);
  const int64_t j = (t / N) % m;
  const int a = (int)(t / ((int64_t)N * m));
  const double d = k[j * dim + a] - (double)(i - N / 2);
  double s = 0.0;
  for (int q = (int)(u % AXIS_LANES); q < Q; q += AXIS_LANES) s += cw[q] * cospi(2.0 * d * xq[q]);
  for (int o = 1; o < AXIS_LANES; o <<= 1) s += __shfl_xor(s, o);
  if (u % AXIS_LANES == 0) G[t] = s;
}

// entry (sample j, mode col) of Psi from the per-axis tables
__device__ inline double psi_at(const double* __restrict__ G, int64_t m, int dim, int N, int64_t j, int64_t col) {
  if (dim == 1) return G[j * N + col];
  const int n0 = (int)(col / N), n1 = (int)(col % N);
  return G[j * N + n0] * G[(m + j) * N + n1];
}

// A (m x (NM + 2), column-major) = [Psi | Re fhat | Im fhat]
__global__ void k_frame_assemble(const double* __restrict__ G, const double2* __restrict__ fhat, int64_t m, int dim,
                                 int N, int64_t NM, double* __restrict__ A) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= m * NM) return;
  const int64_t j = t / NM, col = t % NM;
  A[col * m + j] = psi_at(G, m, dim, N, j, col);
  if (col == 0) {
    A[NM * m + j] = fhat[j].x;
    A[(NM + 1) * m + j] = fhat[j].y;
  }
}

// The same in 16 x 16 tiles (a workgroup each, zeros past the edges), the two
// right-hand sides in a tile column of their own; !over: Psi^T, and fhat to f.
__global__ __launch_bounds__(256) void k_frame_tiles(const double* __restrict__ G, const double2* __restrict__ fhat,
                                                     int64_t m, int dim, int N, int64_t NM, int over, int nrb,
                                                     int npanel, double* __restrict__ A, double2* __restrict__ f) {
  const int ct = blockIdx.x / nrb, rb = blockIdx.x % nrb;
  const int64_t i = 16 * (int64_t)rb + (threadIdx.x & 15), k = 16 * (int64_t)ct + (threadIdx.x >> 4);
  double v = 0.0;
  if (over) {
    if (i < m && k < NM) v = psi_at(G, m, dim, N, i, k);
    if (i < m && ct == npanel && k - 16 * (int64_t)npanel < 2) v = (k & 15) == 0 ? fhat[i].x : fhat[i].y;
  } else if (i < NM && k < m) {
    v = psi_at(G, m, dim, N, k, i);
  }
  A[(int64_t)blockIdx.x * 256 + threadIdx.x] = v;
  if (!over && rb == 0 && threadIdx.x < 16) {   // the forward substitution's own copy of fhat
    const int64_t j = 16 * (int64_t)ct + threadIdx.x;
    f[j] = j < m ? fhat[j] : make_double2(0.0, 0.0);
  }
}

__global__ void k_set_int(int* __restrict__ p, int v) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *p = v;
}

__device__ inline double block_sum(double v, double* red) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  const int w = threadIdx.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[w] = v;
  __syncthreads();
  double s = 0.0;
  for (int i = 0; i < (int)blockDim.x / 64; ++i) s += red[i];
  return s;
}

// unit Householder vector of column j (rows j..r-1) in place, R_jj to diag[j]
__global__ __launch_bounds__(FR_BLOCK) void k_house(double* __restrict__ A, int64_t r, int j,
                                                    double* __restrict__ diag) {
  __shared__ double red[FR_BLOCK / 64];
  double* col = A + (int64_t)j * r;
  double s2 = 0.0;
  for (int64_t i = j + 1 + threadIdx.x; i < r; i += FR_BLOCK) s2 += col[i] * col[i];
  s2 = block_sum(s2, red);
  const double alpha = col[j];
  const double nrm = sqrt(alpha * alpha + s2);
  if (nrm == 0.0) {
    if (threadIdx.x == 0) diag[j] = 0.0;
    return;   // a zero column: the reflector stays 0 (identity); the solve reports it
  }
  const double rjj = alpha >= 0.0 ? -nrm : nrm;
  const double v0 = alpha - rjj;                  // |v0| = |alpha| + nrm: no cancellation
  const double inv = 1.0 / sqrt(v0 * v0 + s2);
  __syncthreads();
  for (int64_t i = j + 1 + threadIdx.x; i < r; i += FR_BLOCK) col[i] *= inv;
  if (threadIdx.x == 0) {
    col[j] = v0 * inv;
    diag[j] = rjj;
  }
}

// columns jc = j + 1 + block: A[j:, jc] -= 2 (v . A[j:, jc]) v
__global__ __launch_bounds__(FR_BLOCK) void k_reflect(double* __restrict__ A, int64_t r, int j) {
  __shared__ double red[FR_BLOCK / 64];
  const double* v = A + (int64_t)j * r;
  double* c = A + (int64_t)(j + 1 + blockIdx.x) * r;
  double s = 0.0;
  for (int64_t i = j + threadIdx.x; i < r; i += FR_BLOCK) s += v[i] * c[i];
  s = 2.0 * block_sum(s, red);
  for (int64_t i = j + threadIdx.x; i < r; i += FR_BLOCK) c[i] -= s * v[i];
}

void frame_approx(ftcg_plan p, int64_t m, const double* k, const void* fhat, void* image) {
  const int dim = p->dim;
  const int N = (int)p->n;
  int64_t NM = N;
  for (int a = 1; a < dim; ++a) NM *= N;
  const bool over = m >= NM;
  const int64_t r = over ? m : NM, c = over ? NM : m;
  hipStream_t s = p->stream;
  const int Q = 4 * N + 64;
  // tiles up to QR_ROWS rows, else (over: only there are the rows the samples) column-major
  const bool tiled = r <= QR_ROWS;
  const int npanel = (int)qr_panels(c), nrb = (int)((r + QR_NB - 1) / QR_NB), nct = npanel + (over ? 1 : 0);
  p->fa_gl.ensure(sizeof(double) * 2 * Q);
  p->fa_G.ensure(sizeof(double) * (size_t)dim * m * N);
  p->fa_A.ensure(sizeof(double) * (tiled ? (size_t)nrb * nct * QR_NB * QR_NB : (size_t)(r * (c + 2))));
  p->fa_diag.ensure((sizeof(double) + 2 * sizeof(double2)) * (size_t)npanel * QR_NB);
  p->fa_beta.ensure(sizeof(double2) * (size_t)NM);
  p->fa_tw.ensure(sizeof(double2) * (size_t)twiddle_entries(N));
  p->fa_tmp.ensure(sizeof(double2) * (size_t)NM);
  p->fa_T.ensure(sizeof(double) * QR_NB * QR_NB * (size_t)npanel);
  double* xq = p->fa_gl.as<double>();
  double* cw = xq + Q;
  int* bad = reinterpret_cast<int*>(p->flags.as<double>() + 10);
  timing_begin(p, STEP_FRAME);
  if (!p->fa_ready) {
    hipLaunchKernelGGL(k_gl_nodes, dim3((Q + 63) / 64), dim3(64), sizeof(double2) * (Q + 1), s, Q, p->sigma, p->beta,
                       xq, cw);
    compute_twiddles(p->fa_tw.p, N, true, s);
    FTCG_HIP(hipGetLastError());
    p->fa_ready = true;
  }
  const int64_t ng = (int64_t)dim * m * N;
  hipLaunchKernelGGL(k_frame_axis, dim3((unsigned)((AXIS_LANES * ng + FR_BLOCK - 1) / FR_BLOCK)), dim3(FR_BLOCK), 0,
                     s, k, m, dim, N, Q, xq, cw, p->fa_G.as<double>());
  double* A = p->fa_A.as<double>();
  double* diag = p->fa_diag.as<double>();
  const double2* f = static_cast<const double2*>(fhat);
  double2* beta = p->fa_beta.as<double2>();
  double2* fw = reinterpret_cast<double2*>(diag + (size_t)npanel * QR_NB);   // forward substitution: f, then y
  hipLaunchKernelGGL(k_set_int, dim3(1), dim3(64), 0, s, bad, 0);
  if (tiled) {
    hipLaunchKernelGGL(k_frame_tiles, dim3((unsigned)(nrb * nct)), dim3(256), 0, s, p->fa_G.as<double>(), f, m, dim, N,
                       NM, over ? 1 : 0, nrb, npanel, A, fw);
    qr_factor(A, nrb, nct, npanel, diag, p->fa_T.as<double>(), over ? nullptr : fw, fw + npanel * QR_NB, s);
    if (over)
      qr_backsub_tiles(A, nrb, (int)c, diag, beta, bad, s);
    else
      qr_minnorm(A, nrb, (int)r, (int)c, diag, p->fa_T.as<double>(), fw + npanel * QR_NB, beta, bad, s);
  } else {
    hipLaunchKernelGGL(k_frame_assemble, dim3((unsigned)((m * NM + FR_BLOCK - 1) / FR_BLOCK)), dim3(FR_BLOCK), 0, s,
                       p->fa_G.as<double>(), f, m, dim, N, NM, A);
    for (int j = 0; j < c; ++j) {
      hipLaunchKernelGGL(k_house, dim3(1), dim3(FR_BLOCK), 0, s, A, r, j, diag);
      hipLaunchKernelGGL(k_reflect, dim3((unsigned)(c + 2 - j - 1)), dim3(FR_BLOCK), 0, s, A, r, j);
    }
    FTCG_HIP(hipGetLastError());
    qr_backsub_cols(A, r, (int)c, diag, beta, bad, s);
  }
  // A_fr at the pixels: inverse DFT of beta on the N^dim mode grid (G = N),
  // divided by w(x_p) = Phi(x_p / sigma) (the plan's deapodization factors)
  grid_to_image_raw(dim, N, N, true, s, p->fa_tw.p, p->deapod.as<double>(), p->fa_tmp.p, p->fa_beta.p, image);
  timing_end(p, STEP_FRAME);
  int* hb = reinterpret_cast<int*>(p->host_flags + 10);
  FTCG_HIP(hipMemcpyAsync(hb, bad, sizeof(int), hipMemcpyDeviceToHost, s));
  FTCG_HIP(hipStreamSynchronize(s));
  if (*hb) throw StatusError{FTCG_EINVAL};
}

}  // namespace ftcg
