// Forward (type-2) transform: image on the n^d pixel grid -> values at the
// raster, fhat_j ~ sum_p I[p] exp(-2 pi i k_j . x_p). It is the adjoint of
// the reconstruction of eq:cgmatrix (Omega^T after the forward DFT of the
// deapodized, zero-padded image), the operator that the frame approximation's
// Psi and the iterative weights of the cited density compensation apply.
//
// Steps:
//   1. forward FFT passes (fft.hip): columns of the image times the
//      deapodization factors, zero-padded to G, transformed, each written as
//      a contiguous row; in 2D the second pass transforms the G columns of
//      that intermediate into H (G x G, the grid's own layout);
//   2. interpolation: fhat_j = sum over the 2W x 2W taps of H[g]
//      prod_a exp(-beta (g_a - u_ja)^2), the taps of the spread. One
//      workgroup per square of ST x ST cells (S x S tiles of the spread's
//      binning, ST = 32, or 64 for tiles of 64 in float32) stages that square's
//      window of H (its ST + 2W - 1 rows and columns, indices modulo G) in
//      LDS with coalesced loads and takes each sample's home record (the record in the
//      tile that holds its cell floor(u), so every sample is computed once), where
//      it pays listed in an order without LDS bank conflicts, one per lane: the
//      lane forms the 2W column factors once, and for each row adds
//      the row's taps against them (two fused multiply-adds and one LDS read
//      per tap) before scaling the row sum by the row factor (rows by the
//      centre of each axis outward). Squares wider than LDS allows (tile 128, or
//      tile 64 in float64) use one workgroup per tile and 16 lanes per
//      record instead (lane i = footprint column i < 2W, the lanes' partial
//      sums added by shuffles), walking the tile's records and skipping the
//      ones that are not home.
#include "ftcg_internal.h"

namespace ftcg {

constexpr int FWD_BLOCK = 256;

template <class real>
struct CxI;
template <>
struct CxI<float> { using t = float2; };
template <>
struct CxI<double> { using t = double2; };

__device__ inline float iexp(float x) { return __expf(x); }
__device__ inline double iexp(double x) { return exp(x); }

template <class real, int W>
__global__ __launch_bounds__(FWD_BLOCK) void k_interp2d(const Rec<real>* __restrict__ recs,
                                                       const int32_t* __restrict__ tile_off,
                                                       const typename CxI<real>::t* __restrict__ grid, int64_t G,
                                                       int nt, int T, real beta,
                                                       typename CxI<real>::t* __restrict__ fhat) {
  using cx = typename CxI<real>::t;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  cx* win = reinterpret_cast<cx*>(smem_raw);
  const int tile = blockIdx.x;
  const int beg = tile_off[tile], end = tile_off[tile + 1];
  if (beg == end) return;
  const int t0 = tile / nt, t1 = tile - (tile / nt) * nt;
  const int WS = T + 2 * W - 1;                 // window edge
  const int64_t g0 = (int64_t)t0 * T - (W - 1), g1 = (int64_t)t1 * T - (W - 1);
  for (int idx = threadIdx.x; idx < WS * WS; idx += FWD_BLOCK) {
    const int r = idx / WS, c = idx - (idx / WS) * WS;
    int64_t gr = g0 + r, gc = g1 + c;
    gr = gr < 0 ? gr + G : (gr >= G ? gr - G : gr);
    gc = gc < 0 ? gc + G : (gc >= G ? gc - G : gc);
    win[idx] = grid[gr * G + gc];
  }
  __syncthreads();
  constexpr int L = 2 * W;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int s = lane >> 4, i = lane & 15;
  const real e2b = iexp((real)-2 * beta);
  for (int base = beg + wave * 4; base < end; base += (FWD_BLOCK / 64) * 4) {
    const int r = base + s;
    real ar = 0, ai = 0;
    bool home = false;
    Rec<real> rec;
    if (r < end) {
      rec = recs[r];
      const int c0 = (int)(int16_t)(rec.c01 & 0xffff), c1 = rec.c01 >> 16;
      home = c0 >= 0 && c0 < T && c1 >= 0 && c1 < T;
      if (home && i < L) {
        const real d1 = (real)(i - W + 1) - rec.f1;
        const real d0 = (real)(1 - W) - rec.f0;
        real w = iexp(-beta * (d0 * d0 + d1 * d1));
        real q = iexp(-beta * ((real)2 * d0 + (real)1));
        const cx* p = win + c0 * WS + c1 + i;
#pragma unroll
        for (int j = 0; j < L; ++j) {
          const cx v = p[j * WS];
          ar += w * v.x;
          ai += w * v.y;
          w *= q;
          q *= e2b;
        }
      }
    }
#pragma unroll
    for (int off = 8; off > 0; off >>= 1) {
      ar += __shfl_xor(ar, off, 64);
      ai += __shfl_xor(ai, off, 64);
    }
    if (home && i == 0) {
      cx o;
      o.x = ar;
      o.y = ai;
      fhat[rec.src] = o;
    }
  }
}


// the 2W kernel values exp(-beta (c - W + 1 - f)^2), c < 2W, of one axis
// (f the fractional position): the largest, at c = W - 1, from an exponent
// of at most beta in size, then outward by the ratio recursion in both
// directions, so the large taps carry the exponential's error at a small
// argument (an exponential at the footprint's edge, argument near -W^2 beta,
// would put |argument| x 2^-24 of relative error on every tap of the sample)
template <class real, int W>
__device__ inline void gauss_taps(real f, real beta, real e2b, real (&out)[2 * W]) {
  out[W - 1] = iexp(-beta * f * f);
  real qu = iexp(-beta * ((real)1 - (real)2 * f)), qd = iexp(-beta * ((real)1 + (real)2 * f));
#pragma unroll
  for (int c = W; c < 2 * W; ++c) {
    out[c] = out[c - 1] * qu;
    qu *= e2b;
  }
#pragma unroll
  for (int c = W - 2; c >= 0; --c) {
    out[c] = out[c + 1] * qd;
    qd *= e2b;
  }
}


// What a square's kernel does with a sample's sum: the forward transform
// stores it (FwdOut); a density iteration, whose grid is real, divides the
// sample's weight by it, or (DEN_SUM) leaves it in the values for a pass of its
// own (DenOut).
template <class real>
struct FwdOut {
  using elem = typename CxI<real>::t;   // grid cells
  static constexpr bool REAL = false;
  elem* fhat;
  __device__ void put(int src, real re, real im) const {
    elem o;
    o.x = re;
    o.y = im;
    fhat[src] = o;
  }
};
template <class real>
struct DenOut {
  using elem = real;
  static constexpr bool REAL = true;
  double* w;
  real* val;
  double scale;
  DenStep step;
  __device__ void put(int src, real re, real) const {
    if (step == DEN_SUM) {
      val[src] = re;
      return;
    }
    const double x = w[src] / (double)re;
    w[src] = step == DEN_LAST ? x * scale : x;
    if (step == DEN_NEXT) val[src] = (real)x;
  }
};

// A square's window of the grid in LDS: ST + 2W - 1 rows, and columns from a multiple
// of 16 bytes on, so that it is read in 16-byte pieces (none straddles the
// grid's edge). Its rows are an odd number of pieces apart, so that one column's
// cells fall on many banks: the samples of a pulse run down a column, and with the
// plain width, a multiple of 8 or 16 cells at W = 4 and 8, the listed kernel found
// only 4 or 2 slots there (float32, 2^20 samples on 512^2: W = 8 240 and 125 us, W =
// 4 71 and 59, W = 6 97 and 88). ODD: an odd number of cells apart, written cell by cell.
template <class elem, int W, int ST, bool ODD>
struct Window {
  static constexpr int EP = 16 / (int)sizeof(elem);
  static constexpr int LP = (W - 1 + EP - 1) / EP * EP;           // cells left of the square
  static constexpr int WR = ST + 2 * W - 1, WS = (LP + ST + W + EP - 1) / EP * EP;
  static constexpr int PITCH = ODD ? WS | 1 : WS + (WS / EP % 2 == 0 ? EP : 0);
  struct alignas(16) Piece {
    elem e[EP];
  };
  // square (sr, sc) of the G x G grid; indices modulo G
  __device__ static void load(elem* win, const elem* __restrict__ grid, int G, int sr, int sc) {
    constexpr int PPR = WS / EP, NP = WR * PPR;   // pieces per row, in all
    const int g0 = sr * ST - (W - 1), g1 = sc * ST - LP;
#pragma unroll 4
    for (int idx = threadIdx.x; idx < NP; idx += FWD_BLOCK) {
      const int r = idx / PPR, c = (idx - r * PPR) * EP;
      int gr = g0 + r, gc = g1 + c;
      gr = gr < 0 ? gr + G : (gr >= G ? gr - G : gr);
      gc = gc < 0 ? gc + G : (gc >= G ? gc - G : gc);
      const Piece v = *reinterpret_cast<const Piece*>(grid + (int64_t)gr * G + gc);
      if constexpr (PITCH % EP == 0) {
        *reinterpret_cast<Piece*>(win + r * PITCH + c) = v;
      } else {
#pragma unroll
        for (int i = 0; i < EP; ++i) win[r * PITCH + c + i] = v.e[i];
      }
    }
  }
  // first tap of a record whose cell is (c0, c1) of the square
  __device__ static int cell(int c0, int c1) { return c0 * PITCH + c1 + (LP - (W - 1)); }
};

// whether the S x S tiles of square (sr, sc) hold any record
template <int S>
__device__ inline bool square_has_records(const int32_t* __restrict__ tile_off, int nt, int sr, int sc) {
  int any = 0;
  for (int k = 0; k < S; ++k) any |= tile_off[(sr * S + k) * nt + sc * S] != tile_off[(sr * S + k) * nt + sc * S + S];
  return any != 0;
}

// Order of a square's records. Every lane of a wavefront reads its taps at the
// same offsets from its own first cell, so two lanes meet on an LDS bank in
// all of their taps or in none, by their first cells modulo the banks' cells
// (SLOTS). The home records of a chunk are listed round by round, a round taking
// one record of every slot that has one left, in slot order: lanes that
// are served together are on different banks, and no lane idles on another tile's
// record. Positions come from each record's rank within its slot (an LDS
// counter) and one ballot per round (records past SQ_ROUNDS of one slot
// follow in any order); a sample's value does not depend on its
// position. With records in binning order the kernel was bound by its LDS
// reads, half of them conflicts, with 45 % of the lanes idle: 4096^2
// raster, 2^23 samples, 605 against 530 us (437 with the window copied in 16-byte
// pieces, a row of reads in flight instead of two, and squares without records left out).
constexpr int SQ_CHUNK = 512;   // records listed at a time: two per thread
constexpr int SQ_ROUNDS = 32;

template <class real, int W, int T, int ST, class OUT>
__global__ __launch_bounds__(FWD_BLOCK) void k_interp2d_sq(const Rec<real>* __restrict__ recs,
                                                           const int32_t* __restrict__ tile_off,
                                                           const typename OUT::elem* __restrict__ grid,
                                                           int64_t G, int nt, real beta, const OUT out) {
  using elem = typename OUT::elem;
  constexpr int S = ST / T;             // tiles per edge of the square
  constexpr int L = 2 * W;
  using Win = Window<elem, W, ST, false>;
  constexpr int WS = Win::PITCH;
  constexpr int SLOTS = 256 / (int)sizeof(elem);   // cells across the 64 banks
  constexpr int PER = SQ_CHUNK / FWD_BLOCK;
  struct Item {
    real f0, f1;
    int cell, src;
  };
  __shared__ __align__(16) elem win[Win::WR * WS];
  __shared__ Item list[SQ_CHUNK];
  __shared__ unsigned long long round_mask[SQ_ROUNDS];   // slots with a record in round q
  __shared__ int round_base[SQ_ROUNDS];
  __shared__ int cnt[SLOTS];
  __shared__ int rest, total;           // first position past the rounds, records listed
  const int tid = threadIdx.x;
  const int nsq = nt / S;
  const int sq = (int)xcd_block(blockIdx.x, gridDim.x);
  const int sr = sq / nsq, sc = sq - (sq / nsq) * nsq;
  if (!square_has_records<S>(tile_off, nt, sr, sc)) return;   // 30 % of the 4096^2 raster's lie outside its sector
  Win::load(win, grid, (int)G, sr, sc);
  const real e2b = iexp((real)-2 * beta);
  for (int k = 0; k < S; ++k) {
    // the S tiles of this row of the square hold one contiguous record range
    const int id0 = (sr * S + k) * nt + sc * S;
    const int rbeg = tile_off[id0], rend = tile_off[id0 + S];
    int bnd[S > 1 ? S - 1 : 1];
#pragma unroll
    for (int q = 1; q < S; ++q) bnd[q - 1] = tile_off[id0 + q];
    for (int base = rbeg; base < rend; base += SQ_CHUNK) {
      if (tid < SLOTS) cnt[tid] = 0;
      __syncthreads();
      Item it[PER];
      int slot[PER], rank[PER];
#pragma unroll
      for (int u = 0; u < PER; ++u) {
        const int r = base + u * FWD_BLOCK + tid;
        slot[u] = -1;
        rank[u] = 0;
        if (r >= rend) continue;
        const Rec<real> rec = recs[r];
        const int c0 = (int)(int16_t)(rec.c01 & 0xffff), c1 = rec.c01 >> 16;
        if (c0 < 0 || c0 >= T || c1 < 0 || c1 >= T) continue;   // not the sample's home record
        int q = 0;
#pragma unroll
        for (int m = 1; m < S; ++m) q += r >= bnd[m - 1];
        it[u].f0 = rec.f0;
        it[u].f1 = rec.f1;
        it[u].src = rec.src;
        it[u].cell = Win::cell(c0 + k * T, c1 + q * T);
        slot[u] = it[u].cell % SLOTS;
        rank[u] = atomicAdd(&cnt[slot[u]], 1);
      }
      __syncthreads();
      if (tid < 64) {   // one wavefront: the rounds' slots and first positions
        const int n = tid < SLOTS ? cnt[tid] : 0;
        int at = 0, over = max(n - SQ_ROUNDS, 0);
        for (int q = 0; q < SQ_ROUNDS; ++q) {
          const unsigned long long mask = __ballot(n > q);
          if (!mask) break;
          if (tid == 0) {
            round_base[q] = at;
            round_mask[q] = mask;
          }
          at += __popcll(mask);
        }
        if (__any(over > 0)) {
          for (int o = 32; o > 0; o >>= 1) over += __shfl_xor(over, o);
        }
        if (tid == 0) {
          rest = at;
          total = at + over;
        }
      }
      __syncthreads();
#pragma unroll
      for (int u = 0; u < PER; ++u)
        if (slot[u] >= 0) {
          const int q = rank[u];
          const int at = q < SQ_ROUNDS ? round_base[q] + __popcll(round_mask[q] & ((1ull << slot[u]) - 1ull))
                                       : atomicAdd(&rest, 1);
          list[at] = it[u];
        }
      const int n = total;
      __syncthreads();
      for (int r = tid; r < n; r += FWD_BLOCK) {
        const Item rec = list[r];
        real a[L], b[L];
        gauss_taps<real, W>(rec.f0, beta, e2b, a);
        gauss_taps<real, W>(rec.f1, beta, e2b, b);
        const elem* p = win + rec.cell;
        real ar = 0, ai = 0;
#pragma unroll
        for (int j = 0; j < L; ++j) {
          if (j > 0) __builtin_amdgcn_sched_barrier(0);   // a row of reads in flight: the other wavefronts hide its latency
          real sr_ = 0, si_ = 0;
#pragma unroll
          for (int c = 0; c < L; ++c) {
            const elem v = p[j * WS + c];
            if constexpr (OUT::REAL) {
              sr_ += b[c] * v;
            } else {
              sr_ += b[c] * v.x;
              si_ += b[c] * v.y;
            }
          }
          ar += a[j] * sr_;
          if constexpr (!OUT::REAL) ai += a[j] * si_;
        }
        out.put(rec.src, ar, ai);
      }
    }
  }
}

// The same without the lists: every thread takes the records in binning order,
// skips those not at home, and has two rows of reads in flight, with no barrier in
// the loop (which of the two runs: launch_interp_sq).
template <class real, int W, int T, int ST, class OUT>
__global__ __launch_bounds__(FWD_BLOCK) void k_interp2d_direct(const Rec<real>* __restrict__ recs,
                                                               const int32_t* __restrict__ tile_off,
                                                               const typename OUT::elem* __restrict__ grid,
                                                               int64_t G, int nt, real beta, const OUT out) {
  using elem = typename OUT::elem;
  using Win = Window<elem, W, ST, true>;
  constexpr int S = ST / T;             // tiles per edge of the square
  constexpr int L = 2 * W;
  __shared__ __align__(16) elem win[Win::WR * Win::PITCH];
  const int nsq = nt / S;
  const int sq = (int)xcd_block(blockIdx.x, gridDim.x);
  const int sr = sq / nsq, sc = sq - (sq / nsq) * nsq;
  if (!square_has_records<S>(tile_off, nt, sr, sc)) return;
  Win::load(win, grid, (int)G, sr, sc);
  __syncthreads();
  const real e2b = iexp((real)-2 * beta);
  for (int k = 0; k < S; ++k) {
    const int id0 = (sr * S + k) * nt + sc * S;
    const int rbeg = tile_off[id0], rend = tile_off[id0 + S];
    int bnd[S > 1 ? S - 1 : 1];
#pragma unroll
    for (int q = 1; q < S; ++q) bnd[q - 1] = tile_off[id0 + q];
    for (int r = rbeg + (int)threadIdx.x; r < rend; r += FWD_BLOCK) {
      const Rec<real> rec = recs[r];
      const int c0 = (int)(int16_t)(rec.c01 & 0xffff), c1 = rec.c01 >> 16;
      if (c0 < 0 || c0 >= T || c1 < 0 || c1 >= T) continue;   // not the sample's home record
      int q = 0;
#pragma unroll
      for (int m = 1; m < S; ++m) q += r >= bnd[m - 1];
      real a[L], b[L];
      gauss_taps<real, W>(rec.f0, beta, e2b, a);
      gauss_taps<real, W>(rec.f1, beta, e2b, b);
      const elem* p = win + Win::cell(c0 + k * T, c1 + q * T);
      real ar = 0, ai = 0;
#pragma unroll 2   // two rows of reads in flight (all 2W rows would hold them all in registers)
      for (int j = 0; j < L; ++j) {
        real sr_ = 0, si_ = 0;
#pragma unroll
        for (int c = 0; c < L; ++c) {
          const elem v = p[j * Win::PITCH + c];
          if constexpr (OUT::REAL) {
            sr_ += b[c] * v;
          } else {
            sr_ += b[c] * v.x;
            si_ += b[c] * v.y;
          }
        }
        ar += a[j] * sr_;
        if constexpr (!OUT::REAL) ai += a[j] * si_;
      }
      out.put(rec.src, ar, ai);
    }
  }
}

// 1D: one workgroup per tile, one thread per home record, 2W taps from global memory
template <class real, int W>
__global__ __launch_bounds__(FWD_BLOCK) void k_interp1d_tiles(const Rec<real>* __restrict__ recs,
                                                             const int32_t* __restrict__ tile_off,
                                                             const typename CxI<real>::t* __restrict__ grid,
                                                             int64_t G, int T, real beta,
                                                             typename CxI<real>::t* __restrict__ fhat) {
  using cx = typename CxI<real>::t;
  const int tile = blockIdx.x;
  const int beg = tile_off[tile], end = tile_off[tile + 1];
  const real e2b = iexp((real)-2 * beta);
  for (int r = beg + (int)threadIdx.x; r < end; r += FWD_BLOCK) {
    const Rec<real> rec = recs[r];
    const int c0 = (int)(int16_t)(rec.c01 & 0xffff);
    if (c0 < 0 || c0 >= T) continue;   // not the home record
    const real d0 = (real)(1 - W) - rec.f0;
    real w = iexp(-beta * d0 * d0);
    real q = iexp(-beta * ((real)2 * d0 + (real)1));
    real ar = 0, ai = 0;
    int64_t g = (int64_t)tile * T + c0 - W + 1;
    g = g < 0 ? g + G : g;
#pragma unroll
    for (int j = 0; j < 2 * W; ++j) {
      const cx v = grid[g];
      ar += w * v.x;
      ai += w * v.y;
      w *= q;
      q *= e2b;
      g = g + 1 == G ? 0 : g + 1;
    }
    cx o;
    o.x = ar;
    o.y = ai;
    fhat[rec.src] = o;
  }
}

// Which plans list their squares' records. Lists pay for their barriers with the
// other workgroups of a compute unit, and by the taps of a record: with no more
// squares than compute units, and up to W = 3, the direct kernel is faster
// (float32 W = 6, lists and direct: half a million samples on 256^2, 256 squares,
// 101 and 74 us, 40 000 there 29 and 26; 2^20 on 512^2, 1024 squares, 68 and 92,
// W = 4 52 and 56, W = 3 45 and 44, W = 2 43 and 39; float64 W = 4 58 and 58). The
// direct kernel's 16 x 16 taps in float64 are twice as slow at any size (2^19 on
// 256^2 151 and 274).
constexpr int SQ_MIN = 256;   // squares: one per compute unit
template <class real, int W, class OUT>
struct Lists {
  static constexpr bool ALWAYS = sizeof(real) == 8 && W == 8 && !OUT::REAL, NEVER = W <= 3;
};

template <class real, int W, int ST, class OUT>
static void launch_interp_sq(ftcg_plan p, const OUT out) {
  using L = Lists<real, W, OUT>;
  const int64_t nsq = (p->G / ST) * (p->G / ST);
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)nsq), dim3(FWD_BLOCK), 0, p->stream, p->recs.as<Rec<real>>(),
                       p->tile_off.as<int32_t>(), p->grid.as<typename OUT::elem>(), p->G, (int)p->nt, (real)p->beta,
                       out);
    FTCG_HIP(hipGetLastError());
  };
  auto tiles = [&](auto tile) {
    constexpr int T = decltype(tile)::value;
    if constexpr (!L::NEVER) {
      if (L::ALWAYS || nsq > SQ_MIN) {
        go(k_interp2d_sq<real, W, T, ST, OUT>);
        return;
      }
    }
    if constexpr (!L::ALWAYS) go(k_interp2d_direct<real, W, T, ST, OUT>);
  };
  switch (p->tile) {
    case 16: tiles(std::integral_constant<int, 16>{}); break;
    case 32: tiles(std::integral_constant<int, 32>{}); break;
    default:
      if constexpr (ST == 64) {
        tiles(std::integral_constant<int, 64>{});
        break;
      }
      throw StatusError{FTCG_EUNSUPPORTED};
  }
}

// edge of the squares of a 2D plan's interpolation, 0 where its tiles are too
// wide: 32 x 32 cells (64 for tile 64 in float32). Squares of 64 re-read fewer
// window cells (1.37 instead of 1.81 per cell) but their 45 KiB windows leave
// three workgroups per compute unit, and measured slower (4096^2 raster: 0.645
// against 0.576 ms, before the records were listed)
static int square_edge(const ftcg_plan_s* p) {
  if (p->dtype == FTCG_F32 && p->tile == 64 && p->G % 64 == 0) return 64;
  return p->tile <= 32 && p->G % 32 == 0 ? 32 : 0;
}
bool interp_in_squares(const ftcg_plan_s* p) { return p->dim == 2 && square_edge(p) > 0; }

template <class real, int W, class OUT>
static void launch_interp_squares(ftcg_plan p, const OUT out) {
  if constexpr (sizeof(real) == 4) {
    if (square_edge(p) == 64) {
      launch_interp_sq<real, W, 64>(p, out);
      return;
    }
  }
  launch_interp_sq<real, W, 32>(p, out);
}

template <class real, int W>
static void launch_interp(ftcg_plan p, void* fhat) {
  using cx = typename CxI<real>::t;
  const real beta = (real)p->beta;
  if (p->dim == 1) {
    hipLaunchKernelGGL((k_interp1d_tiles<real, W>), dim3((unsigned)p->ntiles), dim3(FWD_BLOCK), 0, p->stream,
                       p->recs.as<Rec<real>>(), p->tile_off.as<int32_t>(), p->grid.as<cx>(), p->G, p->tile, beta,
                       static_cast<cx*>(fhat));
  } else {
    if (interp_in_squares(p)) {
      launch_interp_squares<real, W>(p, FwdOut<real>{static_cast<cx*>(fhat)});
      return;
    }
    // tiles of 128, or of 64 in float64: one workgroup per tile
    const int WS = p->tile + 2 * W - 1;
    const size_t lds = (size_t)WS * WS * sizeof(cx);
    if (lds > 160 * 1024) throw StatusError{FTCG_EUNSUPPORTED};   // tile 128 in float64
    static bool attr_done = false;
    if (!attr_done) {
      FTCG_HIP(hipFuncSetAttribute((const void*)k_interp2d<real, W>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                   160 * 1024));
      attr_done = true;
    }
    hipLaunchKernelGGL((k_interp2d<real, W>), dim3((unsigned)p->ntiles), dim3(FWD_BLOCK), lds, p->stream,
                       p->recs.as<Rec<real>>(), p->tile_off.as<int32_t>(), p->grid.as<cx>(), p->G, (int)p->nt,
                       p->tile, beta, static_cast<cx*>(fhat));
  }
  FTCG_HIP(hipGetLastError());
}

template <class real>
static void launch_interp_w(ftcg_plan p, void* fhat) {
  switch (p->W) {
    case 2: launch_interp<real, 2>(p, fhat); break;
    case 3: launch_interp<real, 3>(p, fhat); break;
    case 4: launch_interp<real, 4>(p, fhat); break;
    case 5: launch_interp<real, 5>(p, fhat); break;
    case 6: launch_interp<real, 6>(p, fhat); break;
    case 7: launch_interp<real, 7>(p, fhat); break;
    case 8: launch_interp<real, 8>(p, fhat); break;
    default: throw StatusError{FTCG_EUNSUPPORTED};
  }
}

void interpolate_grid(ftcg_plan p, void* out) {
  if (p->dtype == FTCG_F64)
    launch_interp_w<double>(p, out);
  else
    launch_interp_w<float>(p, out);
}

template <class real, int W>
static void launch_interp_density(ftcg_plan p, double* w, void* val, double scale, DenStep step) {
  launch_interp_squares<real, W>(p, DenOut<real>{w, static_cast<real*>(val), scale, step});
}

void interpolate_density(ftcg_plan p, double* w, void* val, double scale, DenStep step) {
  auto go = [&](auto real_tag) {
    using real = decltype(real_tag);
    switch (p->W) {
      case 2: launch_interp_density<real, 2>(p, w, val, scale, step); break;
      case 3: launch_interp_density<real, 3>(p, w, val, scale, step); break;
      case 4: launch_interp_density<real, 4>(p, w, val, scale, step); break;
      case 5: launch_interp_density<real, 5>(p, w, val, scale, step); break;
      case 6: launch_interp_density<real, 6>(p, w, val, scale, step); break;
      case 7: launch_interp_density<real, 7>(p, w, val, scale, step); break;
      case 8: launch_interp_density<real, 8>(p, w, val, scale, step); break;
      default: throw StatusError{FTCG_EUNSUPPORTED};
    }
  };
  if (p->dtype == FTCG_F64)
    go(double{});
  else
    go(float{});
}

void forward_transform(ftcg_plan p, const void* image, void* fhat) {
  const bool f64 = p->dtype == FTCG_F64;
  const int64_t n = p->n, G = p->G;
  const double* d = p->deapod.as<double>();
  timing_begin(p, STEP_FWD_FFT);
  if (p->dim == 1) {
    fft_cols_forward(f64, image, 1, p->grid.p, G, G, n, 1, d, nullptr, p->twiddle.p, p->stream);
  } else {
    // columns p1 of the image (positions p0) -> T[p1][g0] (n x G);
    // columns g0 of T (positions p1) -> H[g0][g1]
    fft_cols_forward(f64, image, n, p->fft_tmp.p, G, G, n, (int)n, d, d, p->twiddle.p, p->stream);
    fft_cols_forward(f64, p->fft_tmp.p, G, p->grid.p, G, G, n, (int)G, nullptr, nullptr, p->twiddle.p, p->stream);
  }
  timing_end(p, STEP_FWD_FFT);
  timing_begin(p, STEP_FWD_INTERP);
  if (f64)
    launch_interp_w<double>(p, fhat);
  else
    launch_interp_w<float>(p, fhat);
  timing_end(p, STEP_FWD_INTERP);
}

}  // namespace ftcg
