// Blocked Householder QR of a tall float64 matrix in 16 x 16 tiles and the
// triangular solves of the dense frame approximation (Sec. III-B eq:binv).
//
// Tiles lie column of tiles after column of tiles, 256 doubles each, columns
// within a tile contiguous, rows and columns padded with zeros: every load is a
// whole number of cache lines and no kernel checks an edge (with the matrix
// column-major, the strided 8-byte accesses of the update cost 18 us a panel
// against 12). Panels of 16 columns: k_qr_panel factors one panel in the registers
// of one workgroup and forms the panel's compact form H_0 ... H_15 =
// I - V T V^T (unit reflectors H_j = I - 2 v_j v_j^T); k_qr_update applies it to
// the later columns on the matrix cores (v_mfma_f64_16x16x4_f64), a
// workgroup per tile column. V stays in the matrix below the diagonal, R above
// it, R_jj apart.
//
// The serial chain of the columns bounds a factorization of this size (1024 x
// 900: 1.1 GFLOP of updates, 17 us at the measured 64 TFLOP/s). A column
// costs one block reduction: the 16 products of column j with every
// column of the panel (its own squared norm, the later columns' reflections
// and the Gram entries that T needs) are reduced together, before the
// reflector's scale is known, and scaled afterwards. Measured on 1024 x 900:
// 1740 us (11.7 an update, 17-20 a panel), against 6900 us for two launches per column.
#include <algorithm>

#include "ftcg_internal.h"
#include "qr.h"

namespace ftcg {

typedef double double4_t __attribute__((ext_vector_type(4)));

// A lane permutation of a double within rows of 16 lanes (DPP control CTRL)
template <int CTRL>
__device__ inline double dpp_f64(double v) {
  const long long b = __builtin_bit_cast(long long, v);
  const int lo = __builtin_amdgcn_mov_dpp((int)b, CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xf, 0xf, true);
  return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned)lo);
}
constexpr int DPP_XOR1 = 0xB1, DPP_XOR2 = 0x4E, DPP_HALF_MIRROR = 0x141, DPP_ROR8 = 0x128;

// Sum of two doubles over the pair of half wavefronts (32) or of neighbouring
// rows of 16 lanes (16): the lower half keeps a's sum, the upper b's.
template <int HALF>
__device__ inline double swap_sum(double a, double b) {
  const long long ia = __builtin_bit_cast(long long, a), ib = __builtin_bit_cast(long long, b);
  unsigned r[2][2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const unsigned x = (unsigned)(ia >> (32 * h)), y = (unsigned)(ib >> (32 * h));
    const auto s = HALF == 32 ? __builtin_amdgcn_permlane32_swap(x, y, false, false)
                              : __builtin_amdgcn_permlane16_swap(x, y, false, false);
    r[0][h] = s[0];
    r[1][h] = s[1];
  }
  const double u = __builtin_bit_cast(double, ((unsigned long long)r[0][1] << 32) | r[0][0]);
  const double v = __builtin_bit_cast(double, ((unsigned long long)r[1][1] << 32) | r[1][0]);
  return u + v;
}

// w[0..15] summed over the wavefront: lane l returns the sum of w[l / 4]
__device__ inline double wave_sum16(const double* w) {
  const int lane = __lane_id();
  double a[8], b[4], c[2];
#pragma unroll
  for (int p = 0; p < 8; ++p) a[p] = swap_sum<32>(w[p], w[p + 8]);
#pragma unroll
  for (int p = 0; p < 4; ++p) b[p] = swap_sum<16>(a[p], a[p + 4]);
  const bool h8 = lane & 8, h4 = lane & 4;
#pragma unroll
  for (int p = 0; p < 2; ++p) c[p] = (h8 ? b[p + 2] : b[p]) + dpp_f64<DPP_ROR8>(h8 ? b[p] : b[p + 2]);
  double s = (h4 ? c[1] : c[0]) + dpp_f64<DPP_HALF_MIRROR>(h4 ? c[0] : c[1]);
  s += dpp_f64<DPP_XOR1>(s);
  return s + dpp_f64<DPP_XOR2>(s);
}

__device__ inline double lane_f64(double v, int lane) {   // lane uniform
  const long long b = __builtin_bit_cast(long long, v);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)b, lane);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(b >> 32), lane);
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// base[i] where `on`, else 0, as one unconditional load (a conditional one
// becomes a branch, and a run of them waits for each in turn)
__device__ inline double ld0(const double* __restrict__ base, int64_t i, bool on) {
  const double v = base[on ? i : 0];
  return on ? v : 0.0;
}

// 1 / sqrt(x), x > 0: the hardware estimate and one third-order step
__device__ inline double rsqrt_f64(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double e = fma(-(x * y), y, 1.0);
  return fma(y * e, fma(e, 0.375, 0.5), y);
}

// y of R^T y = f for one diagonal tile (R_ki at col[i][k], k < i, diagonal
// apart; a padded unknown, with diagonal 0, gets 0): lane i & 15 returns y_i from
// its own f_i. Called by a whole wavefront.
__device__ inline double2 tri_lower(const double (*col)[QR_NB + 1], double d, double2 f, int i) {
  double r[QR_NB];
#pragma unroll
  for (int k = 0; k < QR_NB; ++k) r[k] = k < i ? col[i][k] : 0.0;
  const double id = d == 0.0 ? 0.0 : 1.0 / d;
#pragma unroll
  for (int k = 0; k < QR_NB; ++k) {
    const double br = lane_f64(f.x * id, k), bi = lane_f64(f.y * id, k);
    f.x = fma(-r[k], br, f.x);
    f.y = fma(-r[k], bi, f.y);
  }
  return make_double2(f.x * id, f.y * id);
}

// One panel: tile column p from tile row p on, `rows` rows (a multiple of 16, at most NT * RP);
// row q * NT + t is in registers P[q] of thread t. The columns rotate through
// the registers: at step j, position 0 holds column j, positions 1 .. 15 - j
// the later columns, and the last j positions the finished reflectors, so
// every step runs the same code with static register indices. With f (minimum
// norm) the second wavefront solves the panel's triangle of R^T y = f while the
// first forms T.
template <int NT, int RP>
__global__ __launch_bounds__(NT) void k_qr_panel(double* __restrict__ A, int nrb, int p, double* __restrict__ diag,
                                                 double* __restrict__ T, const double2* __restrict__ f,
                                                 double2* __restrict__ y) {
  constexpr int NW = NT / 64;
  __shared__ double part[2][NW][QR_NB];
  __shared__ double top[2][QR_NB];   // row j of every position
  __shared__ double gram[QR_NB][QR_NB];   // v_j . position p, written and read by the first wavefront
  __shared__ double sR[QR_NB][QR_NB + 1], sD[QR_NB];   // columns of the top tile above the diagonal, R_jj
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int rows = 16 * (nrb - p);
  double* base = A + ((int64_t)p * nrb + p) * 256 + (t >> 4) * 256 + (t & 15);
  double P[RP][QR_NB];
#pragma unroll
  for (int q = 0; q < RP; ++q)
#pragma unroll
    for (int k = 0; k < QR_NB; ++k) P[q][k] = 0.0;
#pragma unroll
  for (int q = 0; q < RP; ++q)
    if (q * NT + t < rows) {
#pragma unroll
      for (int k = 0; k < QR_NB; ++k) P[q][k] = base[q * NT * 16 + k * 16];
    }
#pragma unroll 1
  for (int j = 0; j < QR_NB; ++j) {
    const int buf = j & 1;
    double w[QR_NB];
    const double a0 = t > j ? P[0][0] : 0.0;   // rows below j only
#pragma unroll
    for (int k = 0; k < QR_NB; ++k) w[k] = a0 * P[0][k];
#pragma unroll
    for (int q = 1; q < RP; ++q)
#pragma unroll
      for (int k = 0; k < QR_NB; ++k) w[k] = fma(P[q][0], P[q][k], w[k]);
    const double s = wave_sum16(w);
    if ((lane & 3) == 0) part[buf][wave][lane >> 2] = s;
    if (t == j) {
#pragma unroll
      for (int k = 0; k < QR_NB; ++k) top[buf][k] = P[0][k];
    }
    __syncthreads();   // the other buffer is written next: one barrier per column
    double tot = part[buf][lane & 3][lane >> 2];
#pragma unroll
    for (int v = 4; v < NW; v += 4) tot += part[buf][v + (lane & 3)][lane >> 2];
    tot += dpp_f64<DPP_XOR1>(tot);
    tot += dpp_f64<DPP_XOR2>(tot);
    const double mine = top[buf][lane >> 2];
    const double s2 = lane_f64(tot, 0), alpha = lane_f64(mine, 0);
    const double n2 = fma(alpha, alpha, s2);
    const bool zero = n2 == 0.0;                      // a zero column: the reflector stays 0 (identity)
    const double nrm = zero ? 0.0 : n2 * rsqrt_f64(n2);
    const double rjj = alpha >= 0.0 ? -nrm : nrm;
    const double v0 = alpha - rjj;                    // |v0| = |alpha| + nrm: no cancellation
    const double inv = zero ? 0.0 : rsqrt_f64(2.0 * nrm * fabs(v0));   // v0^2 + s2 = 2 nrm |v0|
    const double dot = inv * fma(v0, mine, tot);      // v_j . (position lane / 4)
    if (wave == 0 && (lane & 3) == 0) gram[j][lane >> 2] = dot;
    const double later = (lane >> 2) < QR_NB - j ? -2.0 * dot : 0.0;   // finished reflectors stay
    double d[QR_NB];
#pragma unroll
    for (int k = 1; k < QR_NB; ++k) d[k] = lane_f64(later, 4 * k);
#pragma unroll
    for (int q = 0; q < RP; ++q) {
      const int i = q * NT + t;
      const double v = i > j ? P[q][0] * inv : (i == j ? v0 * inv : 0.0);
      if (i < rows) base[q * NT * 16 + j * 16] = i < j ? P[q][0] : v;   // R above the reflector
      if (q == 0 && t < QR_NB) sR[j][t] = P[0][0];
#pragma unroll
      for (int k = 1; k < QR_NB; ++k) P[q][k - 1] = fma(d[k], v, P[q][k]);
      P[q][QR_NB - 1] = v;
    }
    if (t == 0) {
      diag[p * QR_NB + j] = rjj;
      sD[j] = rjj;
    }
  }
  __syncthreads();
  if (f && wave == 1) {
    const int i = lane & 15;
    const double2 v = tri_lower(sR, sD[i], f[p * QR_NB + i], i);
    if (lane < QR_NB) y[p * QR_NB + i] = v;
  }
  // T by columns: T_jj = 2, T[0:j][j] = -2 T[0:j, 0:j] (V^T v_j), lane k holding
  // row k; v_l was at position 16 - j + l when column j was reduced
  if (wave == 0 && lane < QR_NB) {
    double Tr[QR_NB];
#pragma unroll
    for (int j = 0; j < QR_NB; ++j) {
      double tt = 0.0;
#pragma unroll
      for (int l = 0; l < j; ++l) tt = fma(Tr[l], gram[j][QR_NB - j + l], tt);
      Tr[j] = lane == j ? 2.0 : (lane < j ? -2.0 * tt : 0.0);
    }
#pragma unroll
    for (int k = 0; k < QR_NB; ++k) T[lane * QR_NB + k] = Tr[k];
  }
}

// Tile column p + 1 + block, tile rows p ..: A -= V (T^T (V^T A)), V the
// reflectors of panel p. Sixteen wavefronts take four tiles each at a time; up
// to 64 tile rows (ONE) there is one turn and the tiles stay in registers
// between the two products: k-step s of the first contracts rows 4g + s of
// lane group g, so a lane holds four consecutive rows of its column, which is
// where the second product's accumulators (logical row 4s + g) want them when
// its V operand takes the rows in the order 4 (i & 3) + (i >> 2).
//
// FWD (minimum norm) carries the forward substitution R^T y = f along: f holds
// the right-hand sides with the earlier panels taken out, and the new top
// tile R_p,ct takes y_p (k_qr_panel) out of f_ct. (As a pass of its own the
// substitution reads R across its columns, 8 bytes a line, and cost 0.5 ms.)
constexpr int UPD_NT = 1024, UPD_NW = UPD_NT / 64, UPD_RB = 4;
template <bool ONE, bool FWD>
__global__ __launch_bounds__(UPD_NT) void k_qr_update(double* __restrict__ A, int nrb, int p,
                                                      const double* __restrict__ T, double2* __restrict__ f,
                                                      const double2* __restrict__ yp) {
  __shared__ double sY[UPD_NW][256];
  __shared__ double sT[256], sZ[256];
  __shared__ double2 sF[QR_NB];
  const int tid = threadIdx.x, wave = tid >> 6, c = tid & 15, g = (tid >> 4) & 3;
  const int n = nrb - p;
  const double* V = A + ((int64_t)p * nrb + p) * 256;
  double* B = A + ((int64_t)(p + 1 + blockIdx.x) * nrb + p) * 256;
  if (tid < 256) sT[tid] = T[tid];
  if (FWD && tid < QR_NB) sF[tid] = yp[p * QR_NB + tid];
  const int e = c * 16 + 4 * g;            // a lane's four rows of column c
  const int pr = 4 * (c & 3) + (c >> 2);   // row of logical row c
  double4_t ba[UPD_RB];
  double vb[UPD_RB][4];
  const double4_t zero = {0.0, 0.0, 0.0, 0.0};
  auto load_b = [&](int t0) {
#pragma unroll
    for (int u = 0; u < UPD_RB; ++u) {
      const int t = t0 + u * UPD_NW;
      ba[u] = t < n ? *reinterpret_cast<const double4_t*>(B + (int64_t)t * 256 + e) : zero;
    }
  };
  auto load_v2 = [&](int t0) {
#pragma unroll
    for (int u = 0; u < UPD_RB; ++u) {
      const int t = t0 + u * UPD_NW;
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        vb[u][s] = t < n ? V[(int64_t)t * 256 + (4 * s + g) * 16 + pr] : 0.0;
        if (t == 0 && pr < 4 * s + g) vb[u][s] = 0.0;   // R above the reflectors
      }
    }
  };
  double4_t y = zero;
  for (int t0 = wave; ONE ? t0 == wave : t0 < n; t0 += UPD_RB * UPD_NW) {
    double4_t va[UPD_RB];
#pragma unroll
    for (int u = 0; u < UPD_RB; ++u) {
      const int t = t0 + u * UPD_NW;
      va[u] = t < n ? *reinterpret_cast<const double4_t*>(V + (int64_t)t * 256 + e) : zero;
    }
    load_b(t0);
    if (t0 == 0) {
#pragma unroll
      for (int s = 0; s < 4; ++s)
        if (4 * g + s < c) va[0][s] = 0.0;
    }
#pragma unroll
    for (int u = 0; u < UPD_RB; ++u)
#pragma unroll
      for (int s = 0; s < 4; ++s) y = __builtin_amdgcn_mfma_f64_16x16x4f64(va[u][s], ba[u][s], y, 0, 0, 0);
  }
  if (ONE) load_v2(wave);   // in flight during the sum over the wavefronts
#pragma unroll
  for (int q = 0; q < 4; ++q) sY[wave][(4 * q + g) * 16 + c] = y[q];   // rows: reflectors, columns: columns of A
  __syncthreads();
  if (tid < 256) {
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < UPD_NW; ++w) s += sY[w][tid];
    sY[0][tid] = s;
  }
  __syncthreads();
  if (tid < 256) {
    const int k = tid >> 4, col = tid & 15;
    double s = 0.0;
#pragma unroll
    for (int l = 0; l < 16; ++l) s = fma(sT[l * 16 + k], sY[0][l * 16 + col], s);
    sZ[tid] = -s;
  }
  __syncthreads();
  double z[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) z[s] = sZ[(4 * s + g) * 16 + c];
  for (int t0 = wave; ONE ? t0 == wave : t0 < n; t0 += UPD_RB * UPD_NW) {
    if (!ONE) {
      load_b(t0);
      load_v2(t0);
    }
#pragma unroll
    for (int u = 0; u < UPD_RB; ++u) {
      const int t = t0 + u * UPD_NW;
      double4_t a = ba[u];
#pragma unroll
      for (int s = 0; s < 4; ++s) a = __builtin_amdgcn_mfma_f64_16x16x4f64(vb[u][s], z[s], a, 0, 0, 0);
      if (t < n) *reinterpret_cast<double4_t*>(B + (int64_t)t * 256 + e) = a;
      if (FWD && t == 0) {   // the top tile is a tile of R: a lane has rows 4g .. of column c
        double fr = 0.0, fi = 0.0;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          fr = fma(a[s], sF[4 * g + s].x, fr);
          fi = fma(a[s], sF[4 * g + s].y, fi);
        }
        fr += __shfl_xor(fr, 16);
        fi += __shfl_xor(fi, 16);
        fr += __shfl_xor(fr, 32);
        fi += __shfl_xor(fi, 32);
        if (g == 0) {
          double2* fc = f + (p + 1 + (int)blockIdx.x) * QR_NB + c;
          *fc = make_double2(fc->x - fr, fc->y - fi);
        }
      }
    }
  }
}

void qr_factor(double* A, int nrb, int nct, int npanel, double* diag, double* T, double2* f, double2* y,
               hipStream_t s) {
  for (int p = 0; p < npanel; ++p) {
    const int rows = 16 * (nrb - p);
    double* Tp = T + (int64_t)p * QR_NB * QR_NB;
    // threads by rows: up to four rows per thread (128 registers of panel),
    // eight where the rows need more than 512 threads' worth
    if (rows <= 512)
      hipLaunchKernelGGL((k_qr_panel<256, 2>), dim3(1), dim3(256), 0, s, A, nrb, p, diag, Tp, f, y);
    else if (rows <= 1024)
      hipLaunchKernelGGL((k_qr_panel<256, 4>), dim3(1), dim3(256), 0, s, A, nrb, p, diag, Tp, f, y);
    else if (rows <= 2048)
      hipLaunchKernelGGL((k_qr_panel<512, 4>), dim3(1), dim3(512), 0, s, A, nrb, p, diag, Tp, f, y);
    else
      hipLaunchKernelGGL((k_qr_panel<512, 8>), dim3(1), dim3(512), 0, s, A, nrb, p, diag, Tp, f, y);
    if (nct > p + 1)
      hipLaunchKernelGGL(nrb - p <= UPD_RB * UPD_NW ? (f ? k_qr_update<true, true> : k_qr_update<true, false>)
                                                    : (f ? k_qr_update<false, true> : k_qr_update<false, false>),
                         dim3((unsigned)(nct - p - 1)), dim3(UPD_NT), 0, s, A, nrb, p, Tp, f, y);
  }
  FTCG_HIP(hipGetLastError());
}

// ---------------------------------------------------------------------------
// solves: one workgroup, the vector of the two right-hand sides (real and
// imaginary part) in LDS, blocks of 16 unknowns or reflectors. What bounds
// them is the latency of a block's entries (they come from the other XCDs'
// writes): every thread holds its part of the next block in registers before
// the current one is used.
// ---------------------------------------------------------------------------

constexpr int SOL_NT = 512, SOL_NW = SOL_NT / 64;
constexpr int SOL_RP = 2;   // vector entries per thread whose matrix entries are fetched a block ahead

// whether some |R_ii| is not above 1e-14 of the largest (the rank test)
__device__ inline bool small_pivot(const double* __restrict__ diag, int c, double* red) {
  double mx = 0.0;
  for (int k = threadIdx.x; k < c; k += SOL_NT) mx = fmax(mx, fabs(diag[k]));
  for (int off = 32; off > 0; off >>= 1) mx = fmax(mx, __shfl_xor(mx, off));
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = mx;
  __syncthreads();
  mx = 0.0;
  for (int w = 0; w < SOL_NW; ++w) mx = fmax(mx, red[w]);
  bool any = false;
  for (int k = threadIdx.x; k < c; k += SOL_NT) any |= !(fabs(diag[k]) > 1e-14 * mx);
  return __syncthreads_or(any);
}

// entry (i, k) of a tiled or a column-major matrix
struct Tiled {
  const double* A;
  int nrb;
  __device__ int64_t at(int i, int k) const {
    return ((int64_t)(k >> 4) * nrb + (i >> 4)) * 256 + (k & 15) * 16 + (i & 15);
  }
};
struct ColMajor {
  const double* A;
  int64_t r;
  __device__ int64_t at(int i, int k) const { return (int64_t)k * r + i; }
};

// x (c unknowns, in LDS) <- R^-1 x, R upper triangular above the diagonal of M,
// R_ii in diag. A block's triangle is solved by the first wavefront (lane i:
// unknown i of the block), then every thread takes the block out of its
// remaining entries.
template <class MAT>
__device__ void tri_solve(const MAT M, int c, const double* __restrict__ diag, double2* x) {
  const int tid = threadIdx.x;
  double tri[QR_NB], id = 0.0, e[SOL_RP][QR_NB];
  auto fetch = [&](int b) {
    const int nb = std::min(QR_NB, c - b);
    if (tid < 64) {
      const int i = tid < nb ? tid : 0;
      id = 1.0 / diag[b + i];
#pragma unroll
      for (int k = 0; k < QR_NB; ++k) tri[k] = ld0(M.A, M.at(b + i, b + k), k < nb && k > i);
    }
#pragma unroll
    for (int q = 0; q < SOL_RP; ++q) {
      const int i = tid + q * SOL_NT;
#pragma unroll
      for (int k = 0; k < QR_NB; ++k) e[q][k] = ld0(M.A, M.at(i, b + k), i < b && k < nb);
    }
  };
  fetch((c - 1) / QR_NB * QR_NB);
  for (int b = (c - 1) / QR_NB * QR_NB; b >= 0; b -= QR_NB) {
    const int nb = std::min(QR_NB, c - b);
    if (tid < 64) {
      const int i = tid < nb ? tid : 0;
      double2 v = x[b + i];
#pragma unroll
      for (int k = QR_NB - 1; k >= 0; --k) {
        if (k < nb) {
          const double br = lane_f64(v.x * id, k), bi = lane_f64(v.y * id, k);
          v.x = fma(-tri[k], br, v.x);
          v.y = fma(-tri[k], bi, v.y);
        }
      }
      if (tid < nb) x[b + i] = make_double2(v.x * id, v.y * id);
    }
    double cur[SOL_RP][QR_NB];
#pragma unroll
    for (int q = 0; q < SOL_RP; ++q)
#pragma unroll
      for (int k = 0; k < QR_NB; ++k) cur[q][k] = e[q][k];
    if (b > 0) fetch(b - QR_NB);
    __syncthreads();
#pragma unroll
    for (int q = 0; q < SOL_RP; ++q) {
      const int i = tid + q * SOL_NT;
      if (i < b) {
        double2 v = x[i];
#pragma unroll
        for (int k = 0; k < QR_NB; ++k) {
          const double2 y = x[b + (k < nb ? k : 0)];   // (entries past the block are 0)
          v.x = fma(-cur[q][k], y.x, v.x);
          v.y = fma(-cur[q][k], y.y, v.y);
        }
        x[i] = v;
      }
    }
    for (int i = tid + SOL_RP * SOL_NT; i < b; i += SOL_NT) {
      double2 v = x[i];
      for (int k = 0; k < nb; ++k) {
        const double a = M.A[M.at(i, b + k)];
        const double2 y = x[b + k];
        v.x = fma(-a, y.x, v.x);
        v.y = fma(-a, y.y, v.y);
      }
      x[i] = v;
    }
    __syncthreads();
  }
}

// least squares: R beta = (Q^T fhat)[0:c] (columns rhs and rhs + 1)
template <class MAT>
__global__ __launch_bounds__(SOL_NT) void k_qr_backsub(const MAT M, int c, int rhs, const double* __restrict__ diag,
                                                       double2* __restrict__ beta, int* __restrict__ bad) {
  extern __shared__ __align__(16) double2 x[];
  __shared__ double red[SOL_NW];
  const int tid = threadIdx.x;
  if (small_pivot(diag, c, red)) {
    if (tid == 0) *bad = 1;
    return;
  }
  for (int i = tid; i < c; i += SOL_NT) x[i] = make_double2(M.A[M.at(i, rhs)], M.A[M.at(i, rhs + 1)]);
  __syncthreads();
  tri_solve(M, c, diag, x);
  for (int i = tid; i < c; i += SOL_NT) beta[i] = x[i];
}

// minimum norm (A = Psi^T, r = modes, c = samples): beta = H_0 ... H_{c-1} [y; 0],
// panel by panel from the last: x -= V (T (V^T x))
__global__ __launch_bounds__(SOL_NT) void k_qr_minnorm(const double* __restrict__ A, int nrb, int r, int c,
                                                       const double* __restrict__ diag, const double* __restrict__ T,
                                                       const double2* __restrict__ y, double2* __restrict__ beta,
                                                       int* __restrict__ bad) {
  extern __shared__ __align__(16) double2 x[];
  __shared__ double red[SOL_NW];
  __shared__ double part[2][SOL_NW][QR_NB];
  __shared__ double2 sz[QR_NB];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (small_pivot(diag, c, red)) {
    if (tid == 0) *bad = 1;
    return;
  }
  const int last = (c - 1) / QR_NB, rp = 16 * nrb;
  for (int i = tid; i < rp; i += SOL_NT) x[i] = i < c ? y[i] : make_double2(0.0, 0.0);
  double v[SOL_RP][QR_NB], tk[QR_NB];
  const int t0 = (tid >> 4) * 256 + (tid & 15);   // row tid of a tile column
  auto fetch = [&](int p) {
    const double* V = A + ((int64_t)p * nrb + p) * 256 + t0;
#pragma unroll
    for (int q = 0; q < SOL_RP; ++q) {
#pragma unroll
      for (int k = 0; k < QR_NB; ++k) v[q][k] = 0.0;
      if (tid + q * SOL_NT < 16 * (nrb - p)) {
#pragma unroll
        for (int k = 0; k < QR_NB; ++k) v[q][k] = V[q * SOL_NT * 16 + k * 16];
      }
    }
    if (wave == 0) {   // row lane & 15 of the panel's T
#pragma unroll
      for (int k = 0; k < QR_NB; ++k) tk[k] = T[(int64_t)p * QR_NB * QR_NB + (lane & 15) * QR_NB + k];
    }
  };
  fetch(last);
  __syncthreads();
  for (int p = last; p >= 0; --p) {
    const int b = p * QR_NB, rows = 16 * (nrb - p);
    const double* V = A + ((int64_t)p * nrb + p) * 256;
    if (tid < QR_NB) {   // R above the reflectors
#pragma unroll
      for (int k = 0; k < QR_NB; ++k)
        if (tid < k) v[0][k] = 0.0;
    }
    double sr[QR_NB], si[QR_NB];
#pragma unroll
    for (int k = 0; k < QR_NB; ++k) sr[k] = si[k] = 0.0;
#pragma unroll
    for (int q = 0; q < SOL_RP; ++q) {
      const int i = tid + q * SOL_NT;
      const double2 u = i < rows ? x[b + i] : make_double2(0.0, 0.0);
#pragma unroll
      for (int k = 0; k < QR_NB; ++k) {
        sr[k] = fma(v[q][k], u.x, sr[k]);
        si[k] = fma(v[q][k], u.y, si[k]);
      }
    }
    for (int i = tid + SOL_RP * SOL_NT; i < rows; i += SOL_NT) {
      const double2 u = x[b + i];
#pragma unroll
      for (int k = 0; k < QR_NB; ++k) {
        const double a = V[(i >> 4) * 256 + k * 16 + (i & 15)];
        sr[k] = fma(a, u.x, sr[k]);
        si[k] = fma(a, u.y, si[k]);
      }
    }
    const double wr = wave_sum16(sr), wi = wave_sum16(si);
    if ((lane & 3) == 0) {
      part[0][wave][lane >> 2] = wr;
      part[1][wave][lane >> 2] = wi;
    }
    __syncthreads();
    if (wave == 0) {   // z = T (V^T x): lanes 0 .. 15 real, 16 .. 31 imaginary parts
      const int h = (lane >> 4) & 1;
      double s = 0.0, z = 0.0;
#pragma unroll
      for (int w = 0; w < SOL_NW; ++w) s += part[h][w][lane & 15];
#pragma unroll
      for (int l = 0; l < QR_NB; ++l) z = fma(tk[l], __shfl(s, 16 * h + l), z);
      if (lane < 32) reinterpret_cast<double*>(sz)[2 * (lane & 15) + h] = z;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < SOL_RP; ++q) {
      const int i = tid + q * SOL_NT;
      if (i < rows) {
        double2 u = x[b + i];
#pragma unroll
        for (int k = 0; k < QR_NB; ++k) {
          u.x = fma(-v[q][k], sz[k].x, u.x);
          u.y = fma(-v[q][k], sz[k].y, u.y);
        }
        x[b + i] = u;
      }
    }
    for (int i = tid + SOL_RP * SOL_NT; i < rows; i += SOL_NT) {
      double2 u = x[b + i];
#pragma unroll
      for (int k = 0; k < QR_NB; ++k) {
        const double a = V[(i >> 4) * 256 + k * 16 + (i & 15)];
        u.x = fma(-a, sz[k].x, u.x);
        u.y = fma(-a, sz[k].y, u.y);
      }
      x[b + i] = u;
    }
    if (p > 0) fetch(p - 1);
    __syncthreads();
  }
  for (int i = tid; i < r; i += SOL_NT) beta[i] = x[i];
}

template <class MAT>
static void launch_backsub(const MAT M, int c, int rhs, const double* diag, double2* beta, int* bad, hipStream_t s) {
  FTCG_HIP(hipFuncSetAttribute((const void*)k_qr_backsub<MAT>, hipFuncAttributeMaxDynamicSharedMemorySize, 96 * 1024));
  hipLaunchKernelGGL(k_qr_backsub<MAT>, dim3(1), dim3(SOL_NT), sizeof(double2) * (size_t)c, s, M, c, rhs, diag, beta,
                     bad);
  FTCG_HIP(hipGetLastError());
}

void qr_backsub_tiles(const double* A, int nrb, int c, const double* diag, double2* beta, int* bad, hipStream_t s) {
  launch_backsub(Tiled{A, nrb}, c, QR_NB * (int)qr_panels(c), diag, beta, bad, s);
}

void qr_backsub_cols(const double* A, int64_t r, int c, const double* diag, double2* beta, int* bad, hipStream_t s) {
  launch_backsub(ColMajor{A, r}, c, c, diag, beta, bad, s);
}

void qr_minnorm(const double* A, int nrb, int r, int c, const double* diag, const double* T, const double2* y,
                double2* beta, int* bad, hipStream_t s) {
  FTCG_HIP(hipFuncSetAttribute((const void*)k_qr_minnorm, hipFuncAttributeMaxDynamicSharedMemorySize, 96 * 1024));
  hipLaunchKernelGGL(k_qr_minnorm, dim3(1), dim3(SOL_NT), sizeof(double2) * 16 * (size_t)nrb, s, A, nrb, r, c, diag,
                     T, y, beta, bad);
  FTCG_HIP(hipGetLastError());
}

}  // namespace ftcg
