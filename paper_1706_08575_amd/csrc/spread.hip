// Weighting + spreading (the products D fhat and Omega (D fhat) of eq:cgmatrix /
// eq:twodcgmatrix): H[g] = sum_j alpha_j fhat_j prod_a exp(-beta (g_a - u_ja)^2).
//
// One workgroup owns one T x T tile of the oversampled grid. It reads the
// records binned to its tile (samples whose footprint reaches the tile),
// accumulates their taps into the tile held in LDS, and writes the tile to
// HBM once with plain, coalesced stores; tiles with no records are written as
// zeros, so the grid needs no separate clearing pass and no global atomics.
//
// Lane layout (2D): a wavefront takes 64 / (2W) records at a time (5 for
// W = 6); within a record, lane i owns footprint column i and walks the 2W
// rows. The row kernel values follow the recursion
//   e^{-beta (d+1)^2} = e^{-beta d^2} * q,  q_{next} = q * e^{-2 beta}.
//
// Two accumulations:
//   * float32 plans (k_spread2d_fx, the default): exact fixed-point integers,
//     one 64-bit LDS integer add per complex tap (see the block comment of
//     that kernel); on gfx950 the float32 LDS atomic add retires about 0.33
//     lanes per clock per CU and the 64-bit integer one about 9.9 (measured);
//   * float64 plans, and float32 plans that ask for it: matrix products in
//     float64 (k_spread2d_mm, one partial tile of 32 or 64 cells, larger W), else
//     float64 LDS words with ds_add_f64 (k_spread2d, k_spread1d); with
//     lds_copies > 1 wave w accumulates into partial tile w % copies and the
//     partial tiles are combined at the flush with compensated (TwoSum) addition.
#include <cmath>
#include <type_traits>

#include "ftcg_internal.h"

namespace ftcg {

constexpr int SPREAD_BLOCK = 256;

template <class real>
struct Cx;
template <>
struct Cx<float> { using t = float2; };
template <>
struct Cx<double> { using t = double2; };

__device__ inline float kexp(float x) { return __expf(x); }
__device__ inline double kexp(double x) { return exp(x); }

__device__ inline void lds_add(double* p, double v) {
  __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// compensated sum of the partial tiles at one LDS offset
template <class real>
__device__ inline real sum_copies(const real* base, int copy_stride, int copies) {
  real s = base[0];
  if (copies == 1) return s;
  real comp = (real)0;
  for (int c = 1; c < copies; ++c) {
    const real x = base[c * copy_stride];
    const real t = s + x;
    // TwoSum: exact error of s + x
    const real bp = t - s;
    const real e = (s - (t - bp)) + (x - bp);
    comp += e;
    s = t;
  }
  return s + comp;
}

// Where the 2D kernels take values and weights from: FX_RECS, record r has weight
// alpha_s[r]; FX_SUMS, the records carry no weights yet, and record r of sample
// j takes alpha_j = pi^2 pi^2 / wsum[inv[j]] (bin-order sums of the symmetric
// weight kernel, the same float64 division its finish does, rounded to the
// records' type); FX_REAL, weight 1, real values and a real grid (the density
// iterations).
enum FxSrc { FX_RECS = 0, FX_SUMS = 1, FX_REAL = 2 };

// ---------------------------------------------------------------------------
// float64 tile accumulation as a matrix product (one partial tile)
//
// A record's taps are an outer product of its 2W row factors and its 2W column
// factors times the value, so the tile is R C with R (rows x records) and C
// (records x columns, complex). One wavefront owns 16 x 16 cells (or several
// such blocks at tile 64) and runs v_mfma_f64_16x16x4 over the records whose
// footprint meets its block, four at a time: lane l supplies the row factor
// of cell row l % 16 and the column factor of cell column l % 16 of record
// l / 16, 0 outside the footprint. The factors of a chunk of MM_CH records
// are formed once, one record per lane and half an axis per wavefront (so a
// recursion runs over at most W of them), and stored record-minor with an odd
// pitch: conflict-free to write, and the 16 cells of a record read from 16
// different banks. With ds_add_f64 instead (k_spread2d) the LDS atomics bound
// the kernel, at about 10 cycles per 64 lanes of which 44 % were masked by the
// tile's edges, 72 cycles a record and CU. 611 x 1237 samples on 1000^2, G =
// 2048, W = 6, tile 32: 110 us against 185; 2^21 on 1024^2, spread and FFT: 329
// against 507 (tile 64: 402 against 645). Now the matrix unit (a third of the
// time), the factors' exponentials (as much) and the loads' latency share it.
// With the accumulators in the accumulation registers (the compiler's choice
// without the launch bound) 139 us.
//
// Non-finite values stay out of the products (0 times infinity would reach
// the whole block) and are added cell by cell.
// ---------------------------------------------------------------------------
constexpr int MM_CH = 64;
typedef double mm_acc __attribute__((ext_vector_type(4)));

template <int T>
struct MmTile {
  static constexpr int NB = T / 16;            // blocks per axis
  static constexpr int NW = 4;                 // wavefronts
  static constexpr int BPW = NB * NB / NW;     // blocks per wavefront
};

template <class real, int SRC>
using MmValue = std::conditional_t<SRC == FX_REAL, real, typename Cx<real>::t>;

template <class real, int W, int T, int SRC>
__global__ __launch_bounds__(64 * MmTile<T>::NW, T == 64 ? 3 : 6) void k_spread2d_mm(
    const Rec<real>* __restrict__ recs, const real* __restrict__ alpha_s, const double* __restrict__ wsum,
    const int32_t* __restrict__ inv, const int32_t* __restrict__ tile_off, const MmValue<real, SRC>* __restrict__ fhat,
    MmValue<real, SRC>* __restrict__ grid, int64_t G, int nt, real beta, real e2b) {
  constexpr bool REAL = SRC == FX_REAL;
  using cx = std::conditional_t<REAL, real, typename Cx<real>::t>;
  using fac = std::conditional_t<REAL, double, double2>;
  constexpr int L = 2 * W;
  constexpr int BPW = MmTile<T>::BPW, NB = MmTile<T>::NB;
  constexpr int PITCH = MM_CH + 1;
  constexpr int NC = REAL ? 1 : 2;
  __shared__ double frow[L * PITCH];
  __shared__ fac fcol[L * PITCH];
  __shared__ int first[MM_CH];    // first row | first column << 16 (signed, tile cells)
  __shared__ int finite[MM_CH];
  const int tile = blockIdx.x;
  const int t0 = tile / nt, t1 = tile - (tile / nt) * nt;
  const int beg = tile_off[tile], end = tile_off[tile + 1];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int l16 = lane & 15, l4 = lane >> 4;
  mm_acc acc[BPW][NC] = {};
  Rec<real> next = {};   // read one chunk ahead
  if (beg < end) next = recs[beg + min(lane, end - beg - 1)];
  for (int cb = beg; cb < end; cb += MM_CH) {
    const int cn = min(end - cb, MM_CH);
    __syncthreads();   // every wavefront has left the previous chunk
    {
      const int r = cb + min(lane, cn - 1);
      const Rec<real> rec = next;
      next = recs[min(cb + MM_CH + lane, end - 1)];
      {
        // rows, columns: two halves each, from the sample's cell (factor W - 1)
        // outward: the large taps carry the exponential's error at a small argument
        const int part = wave;
        const bool up = part & 1;        // factors W, W + 1, .. 2W - 1; else W - 1, .. 0
        const int j0 = up ? W : W - 1, step = up ? PITCH : -PITCH;
        const real d = (up ? (real)1 : (real)0) - (part < 2 ? rec.f0 : rec.f1);
        real e = kexp(-beta * d * d), q = kexp(up ? -beta * (2 * d + 1) : -beta * (1 - 2 * d));
        if (part < 2) {
          double* to = frow + j0 * PITCH + lane;
#pragma unroll
          for (int j = 0; j < W; ++j) {
            to[j * step] = (double)e;
            e *= q;
            q *= e2b;
          }
          if (part == 0) {
            const int c0 = (int)(int16_t)(rec.c01 & 0xffff) - W + 1, c1 = (rec.c01 >> 16) - W + 1;
            first[lane] = (int)(((uint32_t)c0 & 0xffffu) | ((uint32_t)c1 << 16));
          }
        } else {
          cx v = fhat[rec.src];
          bool fin;
          if constexpr (REAL) {
            fin = isfinite(v);
          } else {
            real a;
            if constexpr (SRC == FX_SUMS)
              a = (real)(wscale<2>() / wsum[inv[rec.src]]);
            else
              a = alpha_s[r];
            v.x *= a;
            v.y *= a;
            fin = isfinite(v.x) && isfinite(v.y);
          }
          if (part == 2) finite[lane] = fin ? 1 : 0;
          fac* to = fcol + j0 * PITCH + lane;
#pragma unroll
          for (int j = 0; j < W; ++j) {
            if constexpr (REAL)
              to[j * step] = (double)e * (double)v;
            else
              to[j * step] = make_double2((double)e * (double)v.x, (double)e * (double)v.y);
            e *= q;
            q *= e2b;
          }
        }
      }
    }
    __syncthreads();
    const int own = first[lane];
    const int own0 = (int)(int16_t)(own & 0xffff), own1 = own >> 16;
    const bool ok = finite[lane] != 0;
#pragma unroll
    for (int b = 0; b < BPW; ++b) {
      const int blk = wave * BPW + b;
      const int row0 = (blk / NB) * 16, col0 = (blk % NB) * 16;
      const bool meets = lane < cn && own0 < row0 + 16 && own0 + L > row0 && own1 < col0 + 16 && own1 + L > col0;
      const unsigned long long take = __ballot(meets && ok);
      unsigned long long odd = __ballot(meets && !ok);
      // records to take, in lanes 0 .. n - 1 (the others behind them: a permutation)
      const unsigned long long below = (1ull << lane) - 1ull;
      const int n = __popcll(take);
      const int to = (take >> lane) & 1 ? __popcll(take & below) : n + __popcll(~take & below);
      const int list = __builtin_amdgcn_ds_permute(to * 4, lane | ((own0 + 64) << 8) | ((own1 + 64) << 16));
      for (int g = 0; g < n; g += 4) {
        const int e = __shfl(list, g + l4);
        const bool live = g + l4 < n;
        const int rec = e & 0xff;
        const int j0 = row0 + l16 - (((e >> 8) & 0xff) - 64), j1 = col0 + l16 - ((e >> 16) - 64);
        const double fr = frow[min(max(j0, 0), L - 1) * PITCH + rec];
        const fac fc = fcol[min(max(j1, 0), L - 1) * PITCH + rec];
        const bool in0 = live && (unsigned)j0 < (unsigned)L, in1 = live && (unsigned)j1 < (unsigned)L;
        const double ra = in0 ? fr : 0.0;
        if constexpr (REAL) {
          acc[b][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(ra, in1 ? fc : 0.0, acc[b][0], 0, 0, 0);
        } else {
          acc[b][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(ra, in1 ? fc.x : 0.0, acc[b][0], 0, 0, 0);
          acc[b][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(ra, in1 ? fc.y : 0.0, acc[b][1], 0, 0, 0);
        }
      }
      while (odd) {
        const int rec = __ffsll(odd) - 1;
        odd &= odd - 1;
        const int o = first[rec];
        const int j1 = col0 + l16 - (o >> 16);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int j0 = row0 + 4 * v + l4 - (int)(int16_t)(o & 0xffff);
          if ((unsigned)j0 < (unsigned)L && (unsigned)j1 < (unsigned)L) {
            const double fr = frow[j0 * PITCH + rec];
            const fac fc = fcol[j1 * PITCH + rec];
            if constexpr (REAL) {
              acc[b][0][v] += fr * fc;
            } else {
              acc[b][0][v] += fr * fc.x;
              acc[b][1][v] += fr * fc.y;
            }
          }
        }
      }
    }
  }
  cx* out = grid + (int64_t)t0 * T * G + (int64_t)t1 * T;
#pragma unroll
  for (int b = 0; b < BPW; ++b) {
    const int blk = wave * BPW + b;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int row = (blk / NB) * 16 + 4 * v + l4, col = (blk % NB) * 16 + l16;
      cx o;
      if constexpr (REAL) {
        o = (real)acc[b][0][v];
      } else {
        o.x = (real)acc[b][0][v];
        o.y = (real)acc[b][1][v];
      }
      out[(int64_t)row * G + col] = o;
    }
  }
}

// Plans whose float64 accumulation runs through the kernel above: one partial tile
// of 32 or 64 cells and a half-width W that fills the 16 x 16 blocks. A block
// costs the same whatever part of it a footprint covers, so at small W the
// LDS-atomic kernel is faster (2^17 .. 2^20 samples, products and atomics, us:
// float64 tile 32 W = 2 71 and 39, W = 3 80 and 65, W = 4 24 and 24 to 92 and 94,
// with 20 density iterations 631 and 663 to 2596 and 2806; tile 64 W = 2 161 and
// 86, W = 4 50 and 40, W = 5 225 and 290). With float32 factors, which cost the
// lanes of the atomics less, W = 4 is the atomics' too (16 and 15 to 82 and 80), and
// so would be W = 5 of a dense raster in few tiles of 64 (2^19 samples on 256^2: 959
// and 770; on 1024^2 98 and 152). At tile 16 a block is the whole tile: one
// wavefront per workgroup and 19 KiB of LDS leave too few of them.
constexpr int MM_MIN_W = 4;
static bool spreads_by_products(const ftcg_plan_s* p) {
  if (p->dim != 2 || p->lds_copies != 1 || (p->tile != 32 && p->tile != 64)) return false;
  return p->W >= (p->tile == 32 && p->dtype == FTCG_F64 ? MM_MIN_W : MM_MIN_W + 1);
}

template <class real, int W, int SRC, class Val>
static void launch_mm(ftcg_plan p, const Val* val, Val* grid) {
  if constexpr (W >= MM_MIN_W + (sizeof(real) == 4 ? 1 : 0)) {
    auto go = [&](auto kernel, int nw) {
      hipLaunchKernelGGL(kernel, dim3((unsigned)p->ntiles), dim3(64 * nw), 0, p->stream, p->recs.as<Rec<real>>(),
                         p->alpha_s.as<real>(), p->ws_sum.as<double>(), p->ws_inv.as<int32_t>(),
                         p->tile_off.as<int32_t>(), val, grid, p->G, (int)p->nt, (real)p->beta,
                         (real)std::exp(-2 * p->beta));
    };
    if (p->tile == 32)
      go(k_spread2d_mm<real, W, 32, SRC>, MmTile<32>::NW);
    else
      go(k_spread2d_mm<real, W, 64, SRC>, MmTile<64>::NW);
    FTCG_HIP(hipGetLastError());
  }
}

// REAL: weight 1, real values and a real grid (the density iterations): one
// plane, half the atomics
template <class real, int W, bool REAL>
__global__ __launch_bounds__(SPREAD_BLOCK) void k_spread2d(const Rec<real>* __restrict__ recs,
                                                           const real* __restrict__ alpha_s,
                                                           const int32_t* __restrict__ tile_off,
                                                           const std::conditional_t<REAL, real, typename Cx<real>::t>* __restrict__ fhat,
                                                           std::conditional_t<REAL, real, typename Cx<real>::t>* __restrict__ grid,
                                                           int64_t G, int nt, int T, int copies, real beta) {
  using cx = std::conditional_t<REAL, real, typename Cx<real>::t>;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  double* lds = reinterpret_cast<double*>(smem_raw);
  const int tile = blockIdx.x;
  const int t0 = tile / nt, t1 = tile - (tile / nt) * nt;
  const int beg = tile_off[tile], end = tile_off[tile + 1];
  cx* out = grid + (int64_t)t0 * T * G + (int64_t)t1 * T;
  const int tid = threadIdx.x;
  if (beg == end) {
    const cx z = {};
    for (int idx = tid; idx < T * T; idx += SPREAD_BLOCK) out[(int64_t)(idx / T) * G + (idx % T)] = z;
    return;
  }
  const int TP = T + 1;                 // padded row pitch
  const int plane = T * TP;             // one real plane
  const int copy_stride = REAL ? plane : 2 * plane;    // re plane + im plane
  for (int idx = tid; idx < copies * copy_stride; idx += SPREAD_BLOCK) lds[idx] = 0.0;
  __syncthreads();

  constexpr int L = 2 * W;              // lanes per record
  constexpr int RPW = 64 / L;           // records per wavefront pass
  const int wave = tid >> 6, lane = tid & 63;
  const int s = lane / L, i = lane - (lane / L) * L;
  double* mine = lds + (wave % copies) * copy_stride;
  const real e2b = kexp(-2 * beta);
  constexpr int NWAVES = SPREAD_BLOCK / 64;
  for (int base = beg + wave * RPW; base < end; base += NWAVES * RPW) {
    const int r = base + s;
    if (s < RPW && r < end) {
      const Rec<real> rec = recs[r];
      const cx v = fhat[rec.src];
      const int c0 = (int)(int16_t)(rec.c01 & 0xffff);
      const int c1 = rec.c01 >> 16;
      const int col = c1 - W + 1 + i;
      if (col >= 0 && col < T) {
        const real d1 = (real)(i - W + 1) - rec.f1;
        const real w1 = REAL ? kexp(-beta * d1 * d1) : kexp(-beta * d1 * d1) * alpha_s[r];
        double* pre = mine + (c0 - W + 1) * TP + col;
        // rows j0, j0 + dir, .. (n of them), the first at distance d from the sample
        // and the others farther (or, dir 1 and d < 0, through it)
        auto walk = [&](int j0, int dir, auto n, real d) {
          real e = w1 * kexp(-beta * d * d), q = kexp(-beta * (2 * d + 1));
          real pr, pi = 0;
          if constexpr (REAL) {
            pr = v * e;
          } else {
            pr = v.x * e;
            pi = v.y * e;
          }
#pragma unroll
          for (int i = 0; i < decltype(n)::value; ++i) {
            const int j = j0 + dir * i, row = c0 - W + 1 + j;
            if (row >= 0 && row < T) {
              lds_add(pre + j * TP, (double)pr);
              if constexpr (!REAL) lds_add(pre + plane + j * TP, (double)pi);
            }
            pr *= q;
            if constexpr (!REAL) pi *= q;
            q *= e2b;
          }
        };
        // float32 taps from the sample's cell outward: from the footprint's edge on
        // every row would carry the exponential's error at beta W^2
        if constexpr (std::is_same<real, float>::value) {
          walk(W - 1, -1, std::integral_constant<int, W>{}, rec.f0);
          walk(W, 1, std::integral_constant<int, W>{}, 1 - rec.f0);
        } else {
          walk(0, 1, std::integral_constant<int, L>{}, (real)(1 - W) - rec.f0);
        }
      }
    }
  }
  __syncthreads();
  for (int idx = tid; idx < T * T; idx += SPREAD_BLOCK) {
    const int row = idx / T, col = idx - (idx / T) * T;
    const int o = row * TP + col;
    cx val;
    if constexpr (REAL) {
      val = (real)sum_copies(lds + o, copy_stride, copies);
    } else {
      val.x = (real)sum_copies(lds + o, copy_stride, copies);
      val.y = (real)sum_copies(lds + plane + o, copy_stride, copies);
    }
    out[(int64_t)row * G + col] = val;
  }
}

// ---------------------------------------------------------------------------
// float32 plans, fixed-point tile accumulation (the default for FTCG_F32)
//
// Each tap value x (complex) is scaled by s = (2^31 - 2^24) / B_t, where B_t >=
// sum over the tile's records of max(|Re c_r|, |Im c_r|) bounds every cell of
// the tile (kernel values never exceed 1; B_t is formed from order-independent
// reductions, so it is the same for any record order), rounded to the nearest
// int32 per component (fx_pack), and both components are added with ONE
// 64-bit LDS integer atomic: the pair (re, im) is packed as im * 2^32 + re in
// two's complement, and integer addition of packed pairs adds both components
// exactly as long as neither sum leaves int32, which the bound guarantees (its
// 2^24 quanta of headroom also cover the half quantum each rounding may add).
// The accumulation is therefore exact and independent of record order
// (bitwise reproducible), and its only error is the rounding of each tap to
// the quantum 2^-31 B_t: unbiased, at most half a quantum per tap.
//
// The LDS tile carries 2W - 1 halo rows above and below, so the 2W rows of a
// record's footprint never need a bounds check (halo rows are dropped at the
// flush); columns outside the tile are skipped per lane.
// ---------------------------------------------------------------------------

// FX_REAL: the cells are the low words of the
// packed ones, added with 32-bit LDS atomics (14.5 instead of 9.9 lanes per
// clock, and no packing), the sums bit for bit the real parts of the complex form.
// 512^2 raster, 2^17 samples: 15.2 against 20.9 us.
template <int SRC>
struct FxTypes {
  using val = float2;
  using cell = unsigned long long;
};
template <>
struct FxTypes<FX_REAL> {
  using val = float;
  using cell = unsigned;
};
template <int W, int T, int SRC>
__global__ __launch_bounds__(SPREAD_BLOCK) void k_spread2d_fx(const Rec<float>* __restrict__ recs,
                                                              const float* __restrict__ alpha_s,
                                                              const double* __restrict__ wsum,
                                                              const int32_t* __restrict__ inv,
                                                              const int32_t* __restrict__ tile_off,
                                                              const typename FxTypes<SRC>::val* __restrict__ fhat,
                                                              typename FxTypes<SRC>::val* __restrict__ grid, int64_t G,
                                                              int nt, float beta) {
  using val_t = typename FxTypes<SRC>::val;
  using cell_t = typename FxTypes<SRC>::cell;
  constexpr bool REAL = SRC == FX_REAL;
  auto weight = [&](int r, int src) -> float {
    if constexpr (SRC == FX_SUMS)
      return (float)(wscale<2>() / wsum[inv[src]]);
    else if constexpr (REAL)
      return 1.f;
    else
      return alpha_s[r];
  };
  // a record's weighted value
  auto value = [&](int r, int src) -> val_t {
    const val_t v = fhat[src];
    const float a = weight(r, src);
    if constexpr (REAL)
      return v * a;
    else
      return make_float2(v.x * a, v.y * a);
  };
  // its larger |component|; NaN and infinities give infinity. (& and not &&: behind
  // a branch the second component was loaded after the first had been tested, two
  // trips to memory a record in both passes below. 2^22 random samples on 1024^2:
  // 414 and 376 us at W = 6, 270 and 230 at W = 2.)
  auto size_of = [](val_t v) -> float {
    float m, t;
    if constexpr (REAL) {
      m = t = fabsf(v);
    } else {
      m = fabsf(v.x);
      t = fabsf(v.y);
    }
    return ((int)isfinite(m) & (int)isfinite(t)) ? fmaxf(m, t) : __builtin_inff();
  };
  auto geometry = [&](const Rec<float>& rec) -> float4 {
    const float d0 = (float)(1 - W) - rec.f0;
    return make_float4(rec.f1, fx_row0(d0, beta), fx_ratio(d0, beta), __int_as_float(rec.c01));
  };
  constexpr int L = 2 * W;              // lanes per record / taps per axis
  constexpr int PAD = 2 * W - 1;        // halo rows each side
  constexpr int TP = T + 1;             // row pitch (64-bit words)
  constexpr int ROWS = T + 2 * PAD;
  // stage only while the tile and the stage fit 64 KiB of LDS together
  constexpr bool STAGED = ROWS * TP * 8 + FX_STAGE * 24 <= 64 * 1024;
  constexpr int STG = STAGED ? FX_STAGE : 1;
  constexpr bool HALF = fx_halves(W, T);
  __shared__ cell_t acc[ROWS * TP];
  __shared__ float4 sgeo[STG];          // f1, first row's kernel value, ratio of the rows, c01 (bits)
  __shared__ val_t sval[STG];           // alpha * fhat[src]
  __shared__ int ncount[2];             // staged records: whole ones (from the front), halves (from the back)
  __shared__ float red[SPREAD_BLOCK / 64];
  __shared__ long long red2[SPREAD_BLOCK / 64];

  const int tile = blockIdx.x;
  const int t0 = tile / nt, t1 = tile - (tile / nt) * nt;
  const int beg = tile_off[tile], end = tile_off[tile + 1];
  val_t* out = grid + (int64_t)t0 * T * G + (int64_t)t1 * T;
  const int tid = threadIdx.x;
  const int wave = tid >> 6, lane = tid & 63;
  if (beg == end) {
    const val_t z = {};
    for (int idx = tid; idx < T * T; idx += SPREAD_BLOCK) out[(int64_t)(idx / T) * G + (idx % T)] = z;
    return;
  }
  // Bound of every cell of the tile, computed so that it does not depend on
  // the order of the records: first the largest |component| of alpha * fhat,
  // then the integer sum of each record's component bound rounded up in
  // units of 2^-20 of that maximum. The first pass stages the first chunk.
  const int first = STAGED ? min(end - beg, STG) : 0;
  float mx = 0.f;
  val_t mine = {};   // of the staged record of this thread
  if constexpr (STAGED) {
    static_assert(FX_STAGE == SPREAD_BLOCK, "one staged record per thread");
    if constexpr (HALF) {
      if (tid < 2) ncount[tid] = 0;
      __syncthreads();
    }
    const bool live = tid < first;
    const int r = beg + (live ? tid : 0);
    const Rec<float> rec = recs[r];
    mine = value(r, rec.src);
    fx_put<W, HALF>(sgeo, sval, ncount, live, rec, mine, T, beta);
    if (live) mx = size_of(mine);
  }
  for (int r = beg + first + tid; r < end; r += SPREAD_BLOCK) mx = fmaxf(mx, size_of(value(r, recs[r].src)));
  for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
  if (lane == 0) red[wave] = mx;
  for (int idx = tid; idx < ROWS * TP; idx += SPREAD_BLOCK) acc[idx] = 0;
  __syncthreads();
  mx = 0.f;
#pragma unroll
  for (int w = 0; w < SPREAD_BLOCK / 64; ++w) mx = fmaxf(mx, red[w]);
  if (!(mx > 0.f) || !isfinite(mx)) {
    // all-zero tile, or non-finite values: propagate as the float path would
    const float fill = mx == 0.f ? 0.f : __builtin_nanf("");
    val_t z;
    if constexpr (REAL)
      z = fill;
    else
      z = make_float2(fill, fill);
    for (int idx = tid; idx < T * T; idx += SPREAD_BLOCK) out[(int64_t)(idx / T) * G + (idx % T)] = z;
    return;
  }
  const float qs = 1048576.f / mx;
  long long qsum = 0;
  if (tid < first) qsum += (long long)ceilf(size_of(mine) * qs) + 1;
  for (int r = beg + first + tid; r < end; r += SPREAD_BLOCK)
    qsum += (long long)ceilf(size_of(value(r, recs[r].src)) * qs) + 1;
  for (int off = 32; off > 0; off >>= 1) qsum += __shfl_xor(qsum, off);
  __syncthreads();
  if (lane == 0) reinterpret_cast<long long*>(red2)[wave] = qsum;
  __syncthreads();
  qsum = 0;
#pragma unroll
  for (int w = 0; w < SPREAD_BLOCK / 64; ++w) qsum += reinterpret_cast<long long*>(red2)[w];
  const float bound = (float)((double)qsum * (double)mx * (1.0 / 1048576.0) * (1.0 + 1e-6));
  const float scale = (2147483648.f - 16777216.f) / bound;

  constexpr int RPW = 64 / L;
  const int s = lane / L, i = lane - (lane / L) * L;
  const float e2b = __expf(-2.f * beta);
  constexpr int NWAVES = SPREAD_BLOCK / 64;
  // one record's 2W (or, half, W) rows of 2W taps: lane i takes footprint column i
  auto splat = [&](float4 geo, val_t v, auto half) {
    constexpr int N = decltype(half)::value ? W : L;
    const int c01 = __float_as_int(geo.w);
    const int col = (c01 >> 16) - W + 1 + i;
    if (col < 0 || col >= T) return;
    const int c0 = (int)(int16_t)(c01 & 0xffff);
    const float w = fx_first((float)(i - W + 1) - geo.x, beta, geo.y, scale);
    cell_t* dst = acc + (c0 - W + 1 + PAD) * TP + col;
    if constexpr (REAL)
      fx_column<N>(dst, TP, v * w, geo.z, e2b);
    else
      fx_column<N>(dst, TP, v.x * w, v.y * w, geo.z, e2b);
  };
  if constexpr (STAGED) {
    for (int cb = beg; cb < end; cb += FX_STAGE) {
      if (cb != beg) {   // later chunks: restage once every wavefront has left the previous one
        __syncthreads();
        if constexpr (HALF) {
          if (tid < 2) ncount[tid] = 0;
          __syncthreads();
        }
        const bool live = cb + tid < end;
        const int r = live ? cb + tid : cb;
        const Rec<float> rec = recs[r];
        fx_put<W, HALF>(sgeo, sval, ncount, live, rec, value(r, rec.src), T, beta);
        __syncthreads();
      }
      fx_chunk<RPW, NWAVES, HALF>(sgeo, sval, ncount, min(end - cb, FX_STAGE), wave, s, splat);
    }
  } else {
    for (int base = beg + wave * RPW; base < end; base += NWAVES * RPW) {
      const int r = base + s;
      if (s < RPW && r < end) {
        const Rec<float> rec = recs[r];
        splat(geometry(rec), value(r, rec.src), std::false_type{});
      }
    }
  }
  __syncthreads();
  const float unscale = bound / (2147483648.f - 16777216.f);
  for (int idx = tid; idx < T * T; idx += SPREAD_BLOCK) {
    const int row = idx / T, col = idx - (idx / T) * T;
    const cell_t vv = acc[(row + PAD) * TP + col];
    if constexpr (REAL) {
      out[(int64_t)row * G + col] = (float)(int)vv * unscale;
    } else {
      const int re = (int)(unsigned)(vv & 0xffffffffull);
      const int im = (int)((long long)(vv - (unsigned long long)(long long)re) >> 32);
      float2 o;
      o.x = (float)re * unscale;
      o.y = (float)im * unscale;
      out[(int64_t)row * G + col] = o;
    }
  }
}

// ---------------------------------------------------------------------------
// Segmented float32 spread for large grids (the same exact fixed-point taps).
//
// The tile binning gives every tile the records of all samples whose
// footprint reaches it, so a sample near a tile edge has records in up to
// four tiles, and each walks all (2W)^2 taps (1.81 records per sample on the
// 4096^2 SAS raster at tile 32). Here one workgroup owns a segment of
// SEG_CW = 2 tile columns (64 cells) by K tile rows and walks its tile rows
// top to bottom, one step per tile row, taking the records of that row's two
// tiles. A record is used only in the tile where its sample is at home along
// the directions the segment covers: along rows, a record from the tile
// above or below is skipped (its home copy is taken in its own step) except
// in the segment's first and last step, where the home copy belongs to the
// next segment; along columns, a record of the left tile whose sample is at
// home in the right tile is skipped, and the other way round. So every
// sample is used once per segment it reaches (1.22 records per sample at
// K = 8 on the same raster).
//
// The step's LDS tile spans tile rows -(W-1) .. 32+W-1 (32 + 2W - 1 rows),
// which holds every tap of the step's home records. After the step, rows
// -(W-1) .. 31-(W-1) receive nothing more and are written out; the 2W - 1
// rows below them still receive taps from the next step's records, so they
// are carried in float (their fixed-point value times the step's quantum)
// and added to the next step's first 2W - 1 rows. Each step has its own
// bound B (the fixed-point kernel's rule over the step's records), so the
// carry is the sum of two exactly accumulated terms in a fixed order:
// deterministic, with one float rounding more than the tile kernel. Records
// from the neighbouring segments above and below (first and last step) have
// rows outside the LDS tile: they take a loop clipped to it.
// ---------------------------------------------------------------------------
constexpr int SEG_BLOCK = 512;
constexpr int SEG_CW = 2;               // tile columns per segment
constexpr int SEG_T = 32;               // tile edge
constexpr int SEG_COLS = SEG_CW * SEG_T;

template <int W, bool SUMS>
__global__ __launch_bounds__(SEG_BLOCK) void k_spread2d_seg(const Rec<float>* __restrict__ recs,
                                                            const float* __restrict__ alpha_s,
                                                            const double* __restrict__ wsum,
                                                            const int32_t* __restrict__ inv,
                                                            const int32_t* __restrict__ tile_off,
                                                            const float2* __restrict__ fhat,
                                                            float2* __restrict__ grid, int64_t G, int nt, int K,
                                                            float beta) {
  constexpr int L = 2 * W;
  constexpr int CROWS = 2 * W - 1;      // carried rows
  constexpr int ROWS = SEG_T + CROWS;   // LDS tile rows: tile rows -(W-1) .. SEG_T + W - 1
  constexpr int TP = SEG_COLS + 1;      // row pitch (64-bit words)
  __shared__ unsigned long long acc[ROWS * TP];
  __shared__ float2 carry[CROWS * SEG_COLS];
  __shared__ float4 sgeo[SEG_BLOCK];    // f1, first kept row's kernel value, ratio of the rows, and (bits)
                                        // LDS row | LDS column << 16 of the record's first tap
  __shared__ float2 sv[SEG_BLOCK];      // alpha * fhat
  __shared__ float red[SEG_BLOCK / 64];
  __shared__ long long red2[SEG_BLOCK / 64];
  __shared__ int ncount[2];             // staged home records (from the front), clipped ones (from the back)

  auto weight = [&](int r, int src) -> float {
    if constexpr (SUMS)
      return (float)(wscale<2>() / wsum[inv[src]]);
    else
      return alpha_s[r];
  };
  const int ncs = nt / SEG_CW;
  const int seg = blockIdx.x / ncs, cs = blockIdx.x - (blockIdx.x / ncs) * ncs;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int col_cell0 = cs * SEG_COLS;

  for (int idx = tid; idx < ROWS * TP; idx += SEG_BLOCK) acc[idx] = 0ull;
  for (int idx = tid; idx < CROWS * SEG_COLS; idx += SEG_BLOCK) carry[idx] = make_float2(0.f, 0.f);

  // record r of the step's two tiles [rb, rm) [rm, re): kept?, clipped?, and
  // the LDS position of its first tap
  struct Kept {
    bool keep, clip;
    int packed;
  };
  auto classify = [&](int r, int rm, int t, int c01) -> Kept {
    const int cc = r >= rm ? 1 : 0;
    const int l0 = (int)(int16_t)(c01 & 0xffff);
    const int l1 = c01 >> 16;
    const bool home0 = l0 >= 0 && l0 < SEG_T;
    const bool vk = home0 || (t == 0 && l0 < 0) || (t == K - 1 && l0 >= SEG_T);
    const bool hk = cc ? (l1 >= 0) : (l1 < SEG_T);
    Kept k;
    k.keep = vk && hk;
    k.clip = !home0;
    // LDS row of the first tap: tile row l0 - W + 1, LDS row 0 = tile row -(W-1)
    const int row0 = l0;
    const int col0 = l1 + cc * SEG_T - W + 1;
    k.packed = (int)(((uint32_t)row0 & 0xffffu) | ((uint32_t)col0 << 16));
    return k;
  };
  // stage one record (compacted: home records from the front, clipped ones
  // from the back of the stage)
  auto stage = [&](bool keep, bool clip, float f0, float f1, int packed, float2 c) {
    const unsigned long long bh = __ballot(keep && !clip), bc = __ballot(keep && clip);
    int baseh = 0, basec = 0;
    if (lane == 0) {
      if (bh) baseh = atomicAdd(&ncount[0], __popcll(bh));
      if (bc) basec = atomicAdd(&ncount[1], __popcll(bc));
    }
    baseh = __shfl(baseh, 0);
    basec = __shfl(basec, 0);
    if (keep) {
      const unsigned long long mine = clip ? bc : bh;
      const int rank = __popcll(mine & ((1ull << lane) - 1ull));
      const int slot = clip ? SEG_BLOCK - 1 - (basec + rank) : baseh + rank;
      const int j0 = max(0, -(int)(int16_t)(packed & 0xffff));   // 0 but for a clipped record
      const float d0 = (float)(1 - W + j0) - f0;
      sgeo[slot] = make_float4(f1, fx_row0(d0, beta), fx_ratio(d0, beta), __int_as_float(packed));
      sv[slot] = c;
    }
  };

  const float e2b = __expf(-2.f * beta);
  constexpr int RPW = 64 / L;
  const int s = lane / L, i = lane - (lane / L) * L;
  constexpr int NWAVES = SEG_BLOCK / 64;

  for (int t = 0; t < K; ++t) {
    const int trow = seg * K + t;
    const int key = trow * nt + cs * SEG_CW;
    const int rb = tile_off[key], rm = tile_off[key + 1], re = tile_off[key + 2];
    if (tid < 2) ncount[tid] = 0;
    __syncthreads();
    // pass 1: largest |component| of alpha * fhat over the kept records; the
    // first chunk of SEG_BLOCK records is staged
    float mx = 0.f;
    for (int cb = rb; cb < re; cb += SEG_BLOCK) {
      const int r = cb + tid;
      bool keep = false, clip = false;
      float2 c = make_float2(0.f, 0.f);
      float f0 = 0.f, f1 = 0.f;
      int packed = 0;
      if (r < re) {
        const Rec<float> rec = recs[r];
        const Kept k = classify(r, rm, t, rec.c01);
        keep = k.keep;
        clip = k.clip;
        packed = k.packed;
        if (keep) {
          const float a = weight(r, rec.src);
          const float2 v = fhat[rec.src];
          c = make_float2(v.x * a, v.y * a);
          f0 = rec.f0;
          f1 = rec.f1;
          mx = (isfinite(c.x) && isfinite(c.y)) ? fmaxf(mx, fmaxf(fabsf(c.x), fabsf(c.y))) : __builtin_inff();
        }
      }
      if (cb == rb) stage(keep, clip, f0, f1, packed, c);
    }
    for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
    if (lane == 0) red[wave] = mx;
    __syncthreads();
    mx = 0.f;
#pragma unroll
    for (int w = 0; w < NWAVES; ++w) mx = fmaxf(mx, red[w]);
    const bool bad = !isfinite(mx);
    float scale = 0.f, unscale = 0.f;
    if (mx > 0.f && !bad) {
      // pass 2: integer sum of each kept record's bound in units of 2^-20 mx
      const float qs = 1048576.f / mx;
      const int nh = ncount[0], ncl = ncount[1];
      long long qsum = 0;
      for (int q = tid; q < nh; q += SEG_BLOCK) {
        const float2 c = sv[q];
        qsum += (long long)ceilf(fmaxf(fabsf(c.x), fabsf(c.y)) * qs) + 1;
      }
      for (int q = tid; q < ncl; q += SEG_BLOCK) {
        const float2 c = sv[SEG_BLOCK - 1 - q];
        qsum += (long long)ceilf(fmaxf(fabsf(c.x), fabsf(c.y)) * qs) + 1;
      }
      for (int cb = rb + SEG_BLOCK; cb < re; cb += SEG_BLOCK) {
        const int r = cb + tid;
        if (r < re) {
          const Rec<float> rec = recs[r];
          if (classify(r, rm, t, rec.c01).keep) {
            const float a = weight(r, rec.src);
            const float2 v = fhat[rec.src];
            qsum += (long long)ceilf(fmaxf(fabsf(v.x * a), fabsf(v.y * a)) * qs) + 1;
          }
        }
      }
      for (int off = 32; off > 0; off >>= 1) qsum += __shfl_xor(qsum, off);
      __syncthreads();
      if (lane == 0) red2[wave] = qsum;
      __syncthreads();
      qsum = 0;
#pragma unroll
      for (int w = 0; w < NWAVES; ++w) qsum += red2[w];
      const float bound = (float)((double)qsum * (double)mx * (1.0 / 1048576.0) * (1.0 + 1e-6));
      scale = (2147483648.f - 16777216.f) / bound;
      unscale = bound / (2147483648.f - 16777216.f);

      // one record's taps: lane i takes LDS column col0 + i, rows row0 .. row0
      // + 2W - 1 (clipped to the LDS tile when clip)
      auto splat = [&](float4 geo, float2 c, bool clip) {
        const int packed = __float_as_int(geo.w);
        const int col = (packed >> 16) + i;
        if (col < 0 || col >= SEG_COLS) return;
        const int row0 = (int)(int16_t)(packed & 0xffff);
        const float w = fx_first((float)(i - W + 1) - geo.x, beta, geo.y, scale);
        float pr = c.x * w, pi = c.y * w;
        if (!clip) {
          fx_column<L>(acc + row0 * TP + col, TP, pr, pi, geo.z, e2b);
        } else {
          const int j1 = min(row0 + L, ROWS);
          float q = geo.z;
          for (int j = max(row0, 0); j < j1; ++j) {
            __hip_atomic_fetch_add(acc + j * TP + col, fx_pack(pr, pi), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_WORKGROUP);
            pr *= q;
            pi *= q;
            q *= e2b;
          }
        }
      };
      // taps of the staged records: home ones, then clipped ones
      auto taps = [&]() {
        const int nh = ncount[0], ncl = ncount[1];
        fx_pass<RPW, NWAVES>(sgeo, sv, nh, wave, s, [&](float4 g, float2 v) { splat(g, v, false); });
        const int npc = (ncl + RPW - 1) / RPW;
        for (int pass = wave; pass < npc; pass += NWAVES) {
          const int r = s * npc + pass;
          if (s < RPW && r < ncl) {
            const int q = SEG_BLOCK - 1 - r;
            splat(sgeo[q], sv[q], true);
          }
        }
      };
      taps();
      for (int cb = rb + SEG_BLOCK; cb < re; cb += SEG_BLOCK) {
        __syncthreads();   // every wavefront has left the previous chunk
        if (tid < 2) ncount[tid] = 0;
        __syncthreads();
        const int r = cb + tid;
        bool keep = false, clip = false;
        float2 c = make_float2(0.f, 0.f);
        float f0 = 0.f, f1 = 0.f;
        int packed = 0;
        if (r < re) {
          const Rec<float> rec = recs[r];
          const Kept k = classify(r, rm, t, rec.c01);
          keep = k.keep;
          clip = k.clip;
          packed = k.packed;
          if (keep) {
            const float a = weight(r, rec.src);
            const float2 v = fhat[rec.src];
            c = make_float2(v.x * a, v.y * a);
            f0 = rec.f0;
            f1 = rec.f1;
          }
        }
        stage(keep, clip, f0, f1, packed, c);
        __syncthreads();
        taps();
      }
    }
    __syncthreads();
    // write the rows that are final, carry the 2W - 1 rows below them
    const int bmin = t == 0 ? W - 1 : 0;
    const int bmax = t == K - 1 ? SEG_T + W - 1 : SEG_T;
    const int64_t row_cell0 = (int64_t)trow * SEG_T - (W - 1);
    const float fill = bad ? __builtin_nanf("") : 0.f;
    for (int idx = tid; idx < bmax * SEG_COLS; idx += SEG_BLOCK) {
      const int b = idx / SEG_COLS, col = idx - (idx / SEG_COLS) * SEG_COLS;
      float2 o;
      {
        const unsigned long long vv = acc[b * TP + col];
        const int re_ = (int)(unsigned)(vv & 0xffffffffull);
        const int im_ = (int)((long long)(vv - (unsigned long long)(long long)re_) >> 32);
        o.x = bad ? fill : (float)re_ * unscale;
        o.y = bad ? fill : (float)im_ * unscale;
      }
      if (b < CROWS) {
        const float2 cy = carry[b * SEG_COLS + col];
        o.x += cy.x;
        o.y += cy.y;
        if (t < K - 1) {
          const unsigned long long vv = acc[(SEG_T + b) * TP + col];
          const int re_ = (int)(unsigned)(vv & 0xffffffffull);
          const int im_ = (int)((long long)(vv - (unsigned long long)(long long)re_) >> 32);
          float2 nc;
          nc.x = bad ? fill : (float)re_ * unscale;
          nc.y = bad ? fill : (float)im_ * unscale;
          carry[b * SEG_COLS + col] = nc;
        }
      }
      if (b >= bmin) grid[(row_cell0 + b) * G + col_cell0 + col] = o;
    }
    __syncthreads();
    if (t + 1 < K)
      for (int idx = tid; idx < ROWS * TP; idx += SEG_BLOCK) acc[idx] = 0ull;
  }
}

// 1D: one thread per record walks its 2W taps; weights in record order, or
// (alpha given) in caller order
template <class real, int W>
__global__ __launch_bounds__(SPREAD_BLOCK) void k_spread1d(const Rec<real>* __restrict__ recs,
                                                           const real* __restrict__ alpha_s,
                                                           const double* __restrict__ alpha,
                                                           const int32_t* __restrict__ tile_off,
                                                           const typename Cx<real>::t* __restrict__ fhat,
                                                           typename Cx<real>::t* __restrict__ grid, int T, int copies,
                                                           real beta) {
  using cx = typename Cx<real>::t;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  double* lds = reinterpret_cast<double*>(smem_raw);
  const int tile = blockIdx.x;
  const int beg = tile_off[tile], end = tile_off[tile + 1];
  cx* out = grid + (int64_t)tile * T;
  const int tid = threadIdx.x;
  const int copy_stride = 2 * T;
  for (int idx = tid; idx < copies * copy_stride; idx += SPREAD_BLOCK) lds[idx] = 0.0;
  __syncthreads();
  double* mine = lds + ((tid >> 6) % copies) * copy_stride;
  const real e2b = kexp(-2 * beta);
  for (int r = beg + tid; r < end; r += SPREAD_BLOCK) {
    const Rec<real> rec = recs[r];
    const real a = alpha ? (real)alpha[rec.src] : alpha_s[r];
    const cx v = fhat[rec.src];
    const int c0 = (int)(int16_t)(rec.c01 & 0xffff);
    const real d0 = (real)(1 - W) - rec.f0;
    real q = kexp(-beta * (2 * d0 + 1));
    const real w0 = kexp(-beta * d0 * d0) * a;
    real pr = v.x * w0, pi = v.y * w0;
    const int cell0 = c0 - W + 1;
#pragma unroll
    for (int j = 0; j < 2 * W; ++j) {
      const int cell = cell0 + j;
      if (cell >= 0 && cell < T) {
        lds_add(mine + cell, (double)pr);
        lds_add(mine + T + cell, (double)pi);
      }
      pr *= q;
      pi *= q;
      q *= e2b;
    }
  }
  __syncthreads();
  for (int idx = tid; idx < T; idx += SPREAD_BLOCK) {
    cx val;
    val.x = (real)sum_copies(lds + idx, copy_stride, copies);
    val.y = (real)sum_copies(lds + T + idx, copy_stride, copies);
    out[idx] = val;
  }
}

template <int W, int T>
static void launch_fx(ftcg_plan p, const void* fhat, void* grid, bool sums) {
  if (sums)
    hipLaunchKernelGGL((k_spread2d_fx<W, T, FX_SUMS>), dim3((unsigned)p->ntiles), dim3(SPREAD_BLOCK), 0, p->stream,
                       p->recs.as<Rec<float>>(), p->alpha_s.as<float>(), p->ws_sum.as<double>(),
                       p->ws_inv.as<int32_t>(), p->tile_off.as<int32_t>(), static_cast<const float2*>(fhat),
                       static_cast<float2*>(grid), p->G, (int)p->nt, (float)p->beta);
  else
    hipLaunchKernelGGL((k_spread2d_fx<W, T, FX_RECS>), dim3((unsigned)p->ntiles), dim3(SPREAD_BLOCK), 0, p->stream,
                       p->recs.as<Rec<float>>(), p->alpha_s.as<float>(), nullptr, nullptr,
                       p->tile_off.as<int32_t>(), static_cast<const float2*>(fhat), static_cast<float2*>(grid),
                       p->G, (int)p->nt, (float)p->beta);
}

// segments of K tile rows for the segmented kernel on grids with enough of
// them to fill the chip (at least 2048 workgroups), else 0 (the tile kernel)
static int spread_segment_rows(const ftcg_plan_s* p) {
  if (p->dim != 2 || p->dtype != FTCG_F32 || p->accum != ACCUM_FIXED || p->tile != SEG_T) return 0;
  const int64_t nt = p->nt;
  if (nt % SEG_CW != 0) return 0;
  for (int K : {8, 4})
    if (nt % K == 0 && (nt / SEG_CW) * (nt / K) >= 2048) return K;
  return 0;
}

template <int W>
static void launch_seg(ftcg_plan p, const void* fhat, void* grid, int K, bool sums) {
  const unsigned nb = (unsigned)((p->nt / SEG_CW) * (p->nt / K));
  if (sums)
    hipLaunchKernelGGL((k_spread2d_seg<W, true>), dim3(nb), dim3(SEG_BLOCK), 0, p->stream, p->recs.as<Rec<float>>(),
                       p->alpha_s.as<float>(), p->ws_sum.as<double>(), p->ws_inv.as<int32_t>(),
                       p->tile_off.as<int32_t>(), static_cast<const float2*>(fhat), static_cast<float2*>(grid), p->G,
                       (int)p->nt, K, (float)p->beta);
  else
    hipLaunchKernelGGL((k_spread2d_seg<W, false>), dim3(nb), dim3(SEG_BLOCK), 0, p->stream,
                       p->recs.as<Rec<float>>(), p->alpha_s.as<float>(), nullptr, nullptr, p->tile_off.as<int32_t>(),
                       static_cast<const float2*>(fhat), static_cast<float2*>(grid), p->G, (int)p->nt, K,
                       (float)p->beta);
}

template <int W>
static void launch_fx_t(ftcg_plan p, const void* fhat, void* grid, bool sums) {
  if (p->spread_segments) {
    const int K = spread_segment_rows(p);
    if (K > 0) {
      launch_seg<W>(p, fhat, grid, K, sums);
      FTCG_HIP(hipGetLastError());
      return;
    }
  }
  switch (p->tile) {
    case 16: launch_fx<W, 16>(p, fhat, grid, sums); break;
    case 32: launch_fx<W, 32>(p, fhat, grid, sums); break;
    case 64: launch_fx<W, 64>(p, fhat, grid, sums); break;
    case 128: launch_fx<W, 128>(p, fhat, grid, sums); break;
    default: throw StatusError{FTCG_EUNSUPPORTED};
  }
  FTCG_HIP(hipGetLastError());
}

// Spreads that form the weights themselves (about 8 % of a call: two gathers
// and a division a record) before the finish is worth its launch: points that
// serve one spread never need it, points that serve many spread from the
// records' weights. The finish costs about two such spreads' extra (1M samples
// on 1024^2: 18 us against 8 a spread, 128 and 120 us a call; 756k in float64
// 18 against 10, 160 and 150), so the third takes it. A call being captured
// always forms them: points set before a replay refresh the sums, and not the
// records' weights.
constexpr int DEFERRED_SPREADS = 2;
bool ready_weights(ftcg_plan p) {
  if (!p->sums_ready) return false;
  const bool forms = p->dim == 2 && (p->accum == ACCUM_FIXED || spreads_by_products(p));
  if (forms) {
    if (p->weights_deferred && p->deferred_spreads < DEFERRED_SPREADS) {
      ++p->deferred_spreads;
      return true;
    }
    if (being_captured(p)) return true;
  }
  finish_deferred_weights(p);
  return false;
}

template <class real, int W>
static void launch_spread_w(ftcg_plan p, const void* fhat, void* grid, bool sums) {
  using cx = typename Cx<real>::t;
  const int T = p->tile;
  if (std::is_same<real, float>::value && p->dim == 2 && p->accum == ACCUM_FIXED) {
    launch_fx_t<W>(p, fhat, grid, sums);
    return;
  }
  const real beta = (real)p->beta;
  const int copies = p->lds_copies;
  if (p->dim == 2) {
    if (spreads_by_products(p)) {
      if (sums)
        launch_mm<real, W, FX_SUMS>(p, static_cast<const cx*>(fhat), static_cast<cx*>(grid));
      else
        launch_mm<real, W, FX_RECS>(p, static_cast<const cx*>(fhat), static_cast<cx*>(grid));
      return;
    }
    const size_t lds = (size_t)copies * 2 * T * (T + 1) * sizeof(double);
    static bool attr_done = false;
    if (!attr_done) {
      FTCG_HIP(hipFuncSetAttribute((const void*)k_spread2d<real, W, false>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                   160 * 1024));
      attr_done = true;
    }
    hipLaunchKernelGGL((k_spread2d<real, W, false>), dim3((unsigned)p->ntiles), dim3(SPREAD_BLOCK), lds, p->stream,
                       p->recs.as<Rec<real>>(), p->alpha_s.as<real>(), p->tile_off.as<int32_t>(),
                       static_cast<const cx*>(fhat), static_cast<cx*>(grid), p->G, (int)p->nt, T, copies, beta);
  } else {
    const size_t lds = (size_t)copies * 2 * T * sizeof(double);
    // a captured call takes the caller-order weights, which every path of
    // set_points writes, so that a replay finds those of whichever it was
    const bool by_src = p->alpha_by_src || (p->wmode == FTCG_W_PLAIN && being_captured(p));
    hipLaunchKernelGGL((k_spread1d<real, W>), dim3((unsigned)p->ntiles), dim3(SPREAD_BLOCK), lds, p->stream,
                       p->recs.as<Rec<real>>(), p->alpha_s.as<real>(),
                       by_src ? p->alpha.as<double>() : nullptr, p->tile_off.as<int32_t>(),
                       static_cast<const cx*>(fhat), static_cast<cx*>(grid), T, copies, beta);
  }
  FTCG_HIP(hipGetLastError());
}

// the real form of a 2D plan's spread (values and grid real, weight 1)
template <class real, int W>
static void launch_spread_real(ftcg_plan p, const void* val, void* grid) {
  const int T = p->tile;
  if constexpr (std::is_same<real, float>::value) {
    if (p->accum == ACCUM_FIXED) {
      auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)p->ntiles), dim3(SPREAD_BLOCK), 0, p->stream,
                           p->recs.as<Rec<float>>(), nullptr, nullptr, nullptr, p->tile_off.as<int32_t>(),
                           static_cast<const float*>(val), static_cast<float*>(grid), p->G, (int)p->nt,
                           (float)p->beta);
      };
      if (T == 16)
        go(k_spread2d_fx<W, 16, FX_REAL>);
      else if (T == 32)
        go(k_spread2d_fx<W, 32, FX_REAL>);
      else if (T == 64)
        go(k_spread2d_fx<W, 64, FX_REAL>);
      else
        throw StatusError{FTCG_EUNSUPPORTED};
      FTCG_HIP(hipGetLastError());
      return;
    }
  }
  if (spreads_by_products(p)) {
    launch_mm<real, W, FX_REAL>(p, static_cast<const real*>(val), static_cast<real*>(grid));
    return;
  }
  const int copies = p->lds_copies;
  const size_t lds = (size_t)copies * T * (T + 1) * sizeof(double);
  if (lds > 60 * 1024)
    FTCG_HIP(hipFuncSetAttribute((const void*)k_spread2d<real, W, true>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                 160 * 1024));
  hipLaunchKernelGGL((k_spread2d<real, W, true>), dim3((unsigned)p->ntiles), dim3(SPREAD_BLOCK), lds, p->stream,
                     p->recs.as<Rec<real>>(), nullptr, p->tile_off.as<int32_t>(), static_cast<const real*>(val),
                     static_cast<real*>(grid), p->G, (int)p->nt, T, copies, (real)p->beta);
  FTCG_HIP(hipGetLastError());
}

// plans whose density iterations run real (spread_real, interpolate_density):
// 2D with a square interpolation, except the grids whose complex spread takes
// segments (each sample is used once per segment there, not once per tile)
bool density_real(const ftcg_plan_s* p) {
  if (p->dim != 2 || !interp_in_squares(p)) return false;
  return !(p->spread_segments && spread_segment_rows(p) > 0);
}

void spread_real(ftcg_plan p, const void* val, void* grid) {
  auto go = [&](auto real_tag) {
    using real = decltype(real_tag);
    switch (p->W) {
      case 2: launch_spread_real<real, 2>(p, val, grid); break;
      case 3: launch_spread_real<real, 3>(p, val, grid); break;
      case 4: launch_spread_real<real, 4>(p, val, grid); break;
      case 5: launch_spread_real<real, 5>(p, val, grid); break;
      case 6: launch_spread_real<real, 6>(p, val, grid); break;
      case 7: launch_spread_real<real, 7>(p, val, grid); break;
      case 8: launch_spread_real<real, 8>(p, val, grid); break;
      default: throw StatusError{FTCG_EUNSUPPORTED};
    }
  };
  if (p->dtype == FTCG_F64)
    go(double{});
  else
    go(float{});
}

template <class real>
static void launch_spread_t(ftcg_plan p, const void* fhat, void* grid, bool sums) {
  switch (p->W) {
    case 2: launch_spread_w<real, 2>(p, fhat, grid, sums); break;
    case 3: launch_spread_w<real, 3>(p, fhat, grid, sums); break;
    case 4: launch_spread_w<real, 4>(p, fhat, grid, sums); break;
    case 5: launch_spread_w<real, 5>(p, fhat, grid, sums); break;
    case 6: launch_spread_w<real, 6>(p, fhat, grid, sums); break;
    case 7: launch_spread_w<real, 7>(p, fhat, grid, sums); break;
    case 8: launch_spread_w<real, 8>(p, fhat, grid, sums); break;
    default: throw StatusError{FTCG_EUNSUPPORTED};
  }
}

void spread(ftcg_plan p, const void* fhat, void* grid, bool sums) {
  if (p->dtype == FTCG_F64)
    launch_spread_t<double>(p, fhat, grid, sums);
  else
    launch_spread_t<float>(p, fhat, grid, sums);
}

}  // namespace ftcg
