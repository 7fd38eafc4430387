// Iterative density compensation (the iterative quadrature weights the paper
// cites in Sec. III-A), a comparator to the frame-theoretic weights of
// eq:difopt: starting from w = 1, each iteration spreads the weights onto the
// oversampled grid with the path's own kernel, interpolates the grid back at
// the samples with the same taps (d = Omega^T Omega w) and sets w <- w / d.
// The plan's spreading and interpolation kernels do the two products; the
// weights live in float64 (the plan's alpha) and reach the spread as the
// values (w, 0) in the plan's precision, in 2D as real values on a real
// grid with the update in the interpolation (25 instead of 44 us per
// iteration at 512^2, 2^17 samples; the weights are the same bit for bit). The
// result is scaled by
// (pi / (sigma beta))^dim, at which a uniform lattice of spacing h gets h^dim,
// as the frame weights do.
#include "ftcg_internal.h"

namespace ftcg {

constexpr int DEN_BLOCK = 256;

template <class T>
__global__ __launch_bounds__(DEN_BLOCK) void k_den_init(double* __restrict__ w, T* __restrict__ val, T one,
                                                       int64_t m) {
  const int64_t j = (int64_t)blockIdx.x * DEN_BLOCK + threadIdx.x;
  if (j >= m) return;
  w[j] = 1.0;
  val[j] = one;
}

// w <- w / Re(d); the next iteration's values, or (last) the scaled weights
template <class cx>
__global__ __launch_bounds__(DEN_BLOCK) void k_den_update(double* __restrict__ w, const cx* __restrict__ den,
                                                         cx* __restrict__ val, int64_t m, double scale, int last) {
  const int64_t j = (int64_t)blockIdx.x * DEN_BLOCK + threadIdx.x;
  if (j >= m) return;
  const double x = w[j] / (double)den[j].x;
  if (last) {
    w[j] = x * scale;
  } else {
    w[j] = x;
    cx v;
    v.x = (decltype(v.x))x;
    v.y = 0;
    val[j] = v;
  }
}

// the same on real values, which hold d
template <class real>
__global__ __launch_bounds__(DEN_BLOCK) void k_den_update_real(double* __restrict__ w, real* __restrict__ val,
                                                              int64_t m, double scale, int last) {
  const int64_t j = (int64_t)blockIdx.x * DEN_BLOCK + threadIdx.x;
  if (j >= m) return;
  const double x = w[j] / (double)val[j];
  w[j] = last ? x * scale : x;
  if (!last) val[j] = (real)x;
}

// Whether the update is a pass of its own, the interpolation leaving d in the values:
// in the interpolation it reads and writes the weight of each sample where the
// raster's order left it, which samples in random order pay for as soon as the taps
// are few and the weights outgrow the L2s. us a call, 20 iterations, float32, tile
// 32, in the interpolation and apart: W = 2, 2^20 random samples on 1024^2 1660 and
// 1102, a sector's 797 and 843; W = 3 1733 and 1192, 953 and 1022 (before the real
// form 1395 and 1139, 1590 and 1381); W = 4 in the interpolation 1937 (1957).
static bool update_apart(const ftcg_plan_s* p) { return p->W <= 3 && p->m >= (int64_t(1) << 19); }

template <class cx>
static void run_density_t(ftcg_plan p) {
  using real = decltype(cx::x);
  const int64_t m = p->m;
  const unsigned gb = (unsigned)((m + DEN_BLOCK - 1) / DEN_BLOCK);
  double* w = p->alpha.as<double>();
  double scale = 1.0;
  for (int a = 0; a < p->dim; ++a) scale *= WPI / (p->sigma * p->beta);
  if (density_real(p)) {
    real* val = p->den_val.as<real>();
    hipLaunchKernelGGL(k_den_init<real>, dim3(gb), dim3(DEN_BLOCK), 0, p->stream, w, val, (real)1, m);
    FTCG_HIP(hipGetLastError());
    for (int it = 0; it < p->den_iters; ++it) {
      spread_real(p, val, p->grid.p);
      const bool last = it + 1 == p->den_iters;
      if (!update_apart(p)) {
        interpolate_density(p, w, val, scale, last ? DEN_LAST : DEN_NEXT);
        continue;
      }
      interpolate_density(p, w, val, scale, DEN_SUM);
      hipLaunchKernelGGL(k_den_update_real<real>, dim3(gb), dim3(DEN_BLOCK), 0, p->stream, w, val, m, scale,
                         last ? 1 : 0);
      FTCG_HIP(hipGetLastError());
    }
    return;
  }
  cx* val = p->den_val.as<cx>();
  cx* den = p->den_d.as<cx>();
  cx one;
  one.x = 1;
  one.y = 0;
  hipLaunchKernelGGL(k_den_init<cx>, dim3(gb), dim3(DEN_BLOCK), 0, p->stream, w, val, one, m);
  for (int it = 0; it < p->den_iters; ++it) {
    spread(p, val, p->grid.p, false);
    interpolate_grid(p, den);
    hipLaunchKernelGGL(k_den_update<cx>, dim3(gb), dim3(DEN_BLOCK), 0, p->stream, w, den, val, m, scale,
                       it + 1 == p->den_iters ? 1 : 0);
  }
  FTCG_HIP(hipGetLastError());
}

void run_density_weights(ftcg_plan p) {
  const size_t csz = p->dtype == FTCG_F64 ? 16 : 8;
  p->den_val.ensure(csz * (size_t)p->m);
  if (!density_real(p)) p->den_d.ensure(csz * (size_t)p->m);
  timing_begin(p, STEP_DENSITY);
  if (p->dtype == FTCG_F64)
    run_density_t<double2>(p);
  else
    run_density_t<float2>(p);
  timing_end(p, STEP_DENSITY);
}

}  // namespace ftcg
