// FFT tiles of the multi-pass scheme (shared by the per-pass kernels and the
// persistent batched search); see fft.hip for the scheme.
#pragma once

#include "fchi2_internal.h"
#include "launch.h"
#include "es_kernel.h"

namespace fchi2 {

namespace {

constexpr double kC16[16] = {
    1.0, 0.92387953251128674, 0.70710678118654752, 0.38268343236508978,
    0.0, -0.38268343236508978, -0.70710678118654752, -0.92387953251128674,
    -1.0, -0.92387953251128674, -0.70710678118654752, -0.38268343236508978,
    0.0, 0.38268343236508978, 0.70710678118654752, 0.92387953251128674};
constexpr double kS16[16] = {
    0.0, 0.38268343236508978, 0.70710678118654752, 0.92387953251128674,
    1.0, 0.92387953251128674, 0.70710678118654752, 0.38268343236508978,
    0.0, -0.38268343236508978, -0.70710678118654752, -0.92387953251128674,
    -1.0, -0.92387953251128674, -0.70710678118654752, -0.38268343236508978};

// Products are written with their rounding spelled out (which of the two terms
// of a complex product's part is rounded before the fused multiply-add).  Left
// to the compiler, the choice depends on the code around a butterfly, and the
// variants of a pass (pruned, spreading fused in, persistent) would agree to
// rounding only; FP64 plans would show it in nearly singular bins.
//
// a b: re = fma(a.x, b.x, -(a.y b.y)), im = fma(a.y, b.x, a.x b.y).
__device__ __forceinline__ cplx<double> cmul_r(cplx<double> a, cplx<double> b) {
  return cmk<double>(__builtin_fma(a.x, b.x, -(a.y * b.y)), __builtin_fma(a.y, b.x, a.x * b.y));
}

// v * exp(+2 pi i E / N) for compile-time E, N <= 16.  The y terms are rounded
// first; X8: the x terms, for the eighth root E / N = 1/8.
template <int N, int E, bool X8>
__device__ __forceinline__ cplx<double> mul_root(cplx<double> v) {
  constexpr int e = E % N;
  if constexpr (e == 0) {
    return v;
  } else if constexpr (4 * e == N) {
    return cmk<double>(-v.y, v.x);
  } else if constexpr (2 * e == N) {
    return cmk<double>(-v.x, -v.y);
  } else if constexpr (4 * e == 3 * N) {
    return cmk<double>(v.y, -v.x);
  } else {
    constexpr int k = e * (16 / N);
    const double c = kC16[k];
    const double s = kS16[k];
    if constexpr (X8 && 8 * e == N) {
      const double t = v.x * c;
      return cmk<double>(__builtin_fma(-v.y, s, t), __builtin_fma(v.y, c, t));
    }
    return cmk<double>(__builtin_fma(v.x, c, -(v.y * s)), __builtin_fma(v.x, s, v.y * c));
  }
}

using C = cplx<double>;

template <int N, int I>
constexpr int bitrev() {
  int r = 0, x = I;
  for (int b = 1; b < N; b <<= 1) {
    r = (r << 1) | (x & 1);
    x >>= 1;
  }
  return r;
}

template <typename R, int N, int I>
__device__ __forceinline__ void bitrev_perm(cplx<R>* v) {
  if constexpr (I < N) {
    constexpr int J = bitrev<N, I>();
    if constexpr (I < J) {
      cplx<R> t = v[I];
      v[I] = v[J];
      v[J] = t;
    }
    bitrev_perm<R, N, I + 1>(v);
  }
}

// RND: where the eighth roots round their x terms first (mul_root's X8).
enum DftRound : int { RND_Y = 0, RND_X_LAST = 1, RND_X = 2 };

template <int N, int S, int K, int J, int RND>
__device__ __forceinline__ void bfly_j(C* v) {
  if constexpr (J < S) {
    constexpr int e = J * (N / (2 * S));
    constexpr bool x8 = RND == RND_X || (RND == RND_X_LAST && 2 * S == N);
    C t = mul_root<N, e, x8>(v[K + J + S]);
    C u = v[K + J];
    v[K + J] = cadd(u, t);
    v[K + J + S] = csub(u, t);
    bfly_j<N, S, K, J + 1, RND>(v);
  }
}
template <int N, int S, int K, int RND>
__device__ __forceinline__ void bfly_k(C* v) {
  if constexpr (K < N) {
    bfly_j<N, S, K, 0, RND>(v);
    bfly_k<N, S, K + 2 * S, RND>(v);
  }
}
template <int N, int S, int RND>
__device__ __forceinline__ void dit_stages(C* v) {
  if constexpr (S < N) {
    bfly_k<N, S, 0, RND>(v);
    dit_stages<N, 2 * S, RND>(v);
  }
}

// In-register N-point DFT (N <= 16), natural order in and out, sign +i.
template <int N, int RND>
__device__ __forceinline__ void dft_reg(C* v) {
  bitrev_perm<double, N, 0>(v);
  dit_stages<N, 1, RND>(v);
}

// A tile holds 2^12 complex elements, or 2^13 with FP32 grids (the same LDS
// bytes as an FP64 tile of 2^12; twice the columns, so runs twice as long):
// the plan chooses per pass.  Every thread holds kEPT elements, so a
// workgroup has 256 or 512 threads.
constexpr int kEPT = 16;  // elements per thread
template <typename S>
constexpr int tile_log_max() {
  return sizeof(S) == 4 ? 13 : 12;
}

// Grid data each pass touches once: element `off` bytes past a base that is
// the same for the whole workgroup, so that a lane's address is one 32-bit
// register (a pair's grid is at most 2^30 bytes).  Runs of at least 128 bytes
// (NT) are loaded and stored non-temporally (streaming); shorter runs measured
// slower that way and use ordinary accesses.
template <typename S, int W>
using vecS = S __attribute__((ext_vector_type(W)));
template <bool NT, typename S>
__device__ __forceinline__ cplx<S> ntl(const char* base, uint32_t off) {
  const vecS<S, 2>* p = (const vecS<S, 2>*)(base + off);
  vecS<S, 2> r;
  if constexpr (NT)
    r = __builtin_nontemporal_load(p);
  else
    r = *p;
  return cmk<S>(r.x, r.y);
}
template <bool NT, typename S>
__device__ __forceinline__ void nts(char* base, uint32_t off, cplx<S> v) {
  vecS<S, 2>* p = (vecS<S, 2>*)(base + off);
  vecS<S, 2> r = {v.x, v.y};
  if constexpr (NT)
    __builtin_nontemporal_store(r, p);
  else
    *p = r;
}
template <typename S>
__device__ __forceinline__ C widen(cplx<S> v) {
  return cmk<double>((double)v.x, (double)v.y);
}
template <typename S>
__device__ __forceinline__ cplx<S> narrow(C v) {
  return cmk<S>((S)v.x, (S)v.y);
}

// Stockham stage geometry over a tile of N rows x T columns, NT = N T / kEPT
// threads.  Butterfly bi of thread tid (slot it) is bi = tid + it * NT:
// column c = bi % T, butterfly
// b = bi / T; its element i is input row b + i N / RAD and output row
// (b / NS) NS RAD + b % NS + i NS.  Every thread holds kEPT elements.
template <int LOGN, int LOGT, int LOGNS>
struct Stage {
  static constexpr int N = 1 << LOGN;
  static constexpr int T = 1 << LOGT;
  static constexpr int NT = (N * T) / kEPT;
  static constexpr int LOGRAD = (LOGN - LOGNS) >= 4 ? 4 : (LOGN - LOGNS);
  static constexpr int RAD = 1 << LOGRAD;
  static constexpr int NS = 1 << LOGNS;
  static constexpr int PER = kEPT / RAD;
  static constexpr bool LAST = (LOGNS + LOGRAD) == LOGN;
  static_assert(PER * RAD == kEPT, "radix must divide the per-thread elements");
  __device__ static int col(int tid, int it) { return (tid + it * NT) & (T - 1); }
  __device__ static int bfly(int tid, int it) { return (tid + it * NT) >> LOGT; }
  __device__ static int in_row(int b, int i) { return b + i * (N / RAD); }
  __device__ static int out_row(int b, int i) {
    return ((b >> LOGNS) << (LOGNS + LOGRAD)) + (b & (NS - 1)) + i * NS;
  }
};

// Stage twiddles of a tile kept in LDS (FP32 grids, tiles of more than one
// column): the second stage's omega_{16 RAD}^{j i}, row i - 1, column j < 16,
// and for tiles of 2^9 rows the third stage's omega_512^j, j < 256.  Read from
// the global table every thread would gather 15 to 23 entries of 16 bytes per
// tile through the L1 beside the tile's own 16 loads.  FP64 tiles fill the LDS
// with data and single-column tiles have longer tables: both read the global
// table.
template <typename S, int LOGN, int LOGT>
struct StageTw {
  static constexpr bool kLds = sizeof(S) == 4 && LOGT > 0 && LOGN > 4;
  static constexpr int LR2 = LOGN - 4 >= 4 ? 4 : (LOGN > 4 ? LOGN - 4 : 0);
  static constexpr int N2 = kLds ? ((1 << LR2) - 1) * 16 : 0;
  static constexpr int N3 = kLds && LOGN > 8 ? 256 : 0;
  static_assert(!kLds || LOGN <= 9, "third stage of radix 2 at most");
  static constexpr int SIZE = N2 + N3 > 0 ? N2 + N3 : 1;
  __device__ static void fill(C* t, const C* __restrict__ tw, int tid, int nt) {
    if constexpr (kLds) {
      for (int e = tid; e < N2; e += nt)
        t[e] = tw[((e & 15) * ((e >> 4) + 1)) << (kStageLog - 4 - LR2)];
      for (int e = tid; e < N3; e += nt) t[N2 + e] = tw[e << (kStageLog - 9)];
    }
  }
};

// Butterflies of one stage on the registers (FP64): stage twiddles (LDS, or
// the omega_{2^13} table), then the in-register RAD-point DFT.
template <typename S, int LOGN, int LOGT, int LOGNS>
__device__ __forceinline__ void stage_compute(C* v, const C* __restrict__ tw, const C* tl,
                                              int tid) {
  using St = Stage<LOGN, LOGT, LOGNS>;
  using Tw = StageTw<S, LOGN, LOGT>;
  constexpr int TWS = kStageLog - LOGNS - St::LOGRAD;
  static_assert(TWS >= 0, "stage twiddle table too small");
#pragma unroll
  for (int it = 0; it < St::PER; ++it) {
    C* u = v + it * St::RAD;
    if constexpr (St::NS > 1) {
      const int j = St::bfly(tid, it) & (St::NS - 1);
#pragma unroll
      for (int i = 1; i < St::RAD; ++i) {
        if constexpr (Tw::kLds)
          u[i] = cmul_r(u[i], tl[LOGNS == 4 ? (i - 1) * 16 + j : Tw::N2 + j]);
        else
          u[i] = cmul_r(u[i], tw[(j * i) << TWS]);
      }
    }
    // First stage of 2^6 and 2^7 rows, of other tiles, later stages.
    constexpr int RND = LOGNS > 0 ? RND_X : (LOGN == 6 || LOGN == 7 ? RND_Y : RND_X_LAST);
    dft_reg<St::RAD, RND>(u);
  }
}

// Row pitch of a tile in LDS and the place of column c in row r.  A row of 16
// or more FP32 elements is 128 bytes or more, so sixteen lanes of an exchange
// between stages cover all banks without padding; where columns are read
// (tile_col: the first pass's transposition) the columns of a row are permuted
// by its low bits instead.  Shorter rows, and FP64 rows, have a padding column.
template <typename S, int LOGT>
constexpr bool tile_swizzled() {
  return sizeof(S) == 4 && LOGT >= 4;
}
template <typename S, int LOGT>
constexpr int tile_pitch() {
  return LOGT == 0 || tile_swizzled<S, LOGT>() ? (1 << LOGT) : (1 << LOGT) + 1;
}
template <typename S, int LOGT>
__device__ __forceinline__ int tile_col(int r, int c) {
  return r * tile_pitch<S, LOGT>() + (tile_swizzled<S, LOGT>() ? c ^ (r & 15) : c);
}

// Run the stages from LOGNS on; between stages the registers go through the
// LDS tile (type S, row pitch PT) in Stockham order.  On return v holds the
// last stage's outputs: element i of slot it is row out_row(b, i) of column
// col(tid, it).  FENCE: other threads may still be reading the tile when the
// first exchange writes it.
template <typename S, int LOGN, int LOGT, int LOGNS, int PT, bool FENCE>
__device__ __forceinline__ void run_stages(C* v, cplx<S>* sm, const C* __restrict__ tw,
                                           const C* tl, int tid) {
  using St = Stage<LOGN, LOGT, LOGNS>;
  stage_compute<S, LOGN, LOGT, LOGNS>(v, tw, tl, tid);
  if constexpr (!St::LAST) {
    using Nx = Stage<LOGN, LOGT, LOGNS + St::LOGRAD>;
    if constexpr (FENCE || LOGNS > 0) __syncthreads();  // previous readers of sm are done
#pragma unroll
    for (int it = 0; it < St::PER; ++it) {
      const int c = St::col(tid, it), b = St::bfly(tid, it);
#pragma unroll
      for (int i = 0; i < St::RAD; ++i)
        sm[St::out_row(b, i) * PT + c] = narrow<S>(v[it * St::RAD + i]);
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < Nx::PER; ++it) {
      const int c = Nx::col(tid, it), b = Nx::bfly(tid, it);
#pragma unroll
      for (int i = 0; i < Nx::RAD; ++i)
        v[it * Nx::RAD + i] = widen(sm[Nx::in_row(b, i) * PT + c]);
    }
    run_stages<S, LOGN, LOGT, LOGNS + St::LOGRAD, PT, FENCE>(v, sm, tw, tl, tid);
  }
}

// LOGNS of the last stage: stages advance by radix 16 until the remainder.
constexpr int last_logns(int logn) {
  int ns = 0;
  while (ns + ((logn - ns) >= 4 ? 4 : (logn - ns)) < logn) ns += 4;
  return ns;
}

// exp(+2 pi i e / 2^logM) for 0 <= e < 2^logM (exact argument reduction).
__device__ __forceinline__ C root(int64_t e, int logM) {
  double s, c;
  sincospi(ldexp((double)e, 1 - logM), &s, &c);
  return cmk<double>(c, s);
}

// Cells of a first-pass tile (pair p, columns g0 + cc, rows r of stride
// Sd = L / N; rows r >= r_lim are beyond the pair's extent and stay zero)
// spread from the curve's points straight into the LDS tile sm, as S values in
// the tile layout (row r, column cc at r * PT + cc).  A thread owns kEPT
// cells, as one segment of a row (T >= kEPT) or whole rows.  The points that
// can reach a segment are a contiguous index range (positions grow with t):
// the fine tile table of the spreading (first point at or past each tile of
// 2^tb_log cells, minus the kernel's reach) gives it with two loads, and the
// thread reads those points, forms their cell coordinate on the component's
// harmonic grid and strength as the spreading kernel does, and adds
// phi(cell - pos) times the strength point by point in index order:
// component 0 of the pair into the real part (and the imaginary part when
// both components are the same harmonic), component 1 into the imaginary
// part.  FLR: floor gridding (kernel width 1).
template <typename S, int LOGN, int LOGT, bool FLR>
__device__ __forceinline__ void spread_into_tile(const FftPassArgs& a, const Moments& mo,
                                                 const Geom& g, int p, int cw, int64_t g0,
                                                 int64_t r_lim, cplx<S>* sm, int tid) {
  constexpr int N = 1 << LOGN;
  constexpr int T = 1 << LOGT;
  constexpr int NTH = (N * T) / kEPT;
  constexpr int CPR = T >= kEPT ? kEPT : T;  // cells per owned row segment
  constexpr int RPT = kEPT / CPR;            // row segments per thread
  constexpr int TPR = T >= kEPT ? T / kEPT : 1;  // threads per row
  constexpr bool EXACT = sizeof(S) == 8;
  const int64_t Sd = g.L >> LOGN;
  double ar[RPT][CPR], ai[RPT][CPR];
#pragma unroll
  for (int j = 0; j < RPT; ++j)
#pragma unroll
    for (int u = 0; u < CPR; ++u) {
      ar[j][u] = 0.0;
      ai[j][u] = 0.0;
    }
  const int m0 = g.comp_m[p][0], m1 = g.comp_m[p][1];
  const bool both = m1 == m0;
  const int kd0 = g.comp_kind[p][0], kd1 = g.comp_kind[p][1];
  const double Ld = (double)g.L, coff = (double)g.c_off;
  const double two_over_w = 2.0 / (double)g.w;
  const double beta = g.beta;
  const double* __restrict__ t = a.t;
  const double* __restrict__ x = a.x;
  const double* __restrict__ sg = a.sigma;
  const int64_t pa = mo.start;
  const double t_last = t[pa + mo.n - 1];
  const int tbl = a.tb_log;
#pragma unroll
  for (int comp = 0; comp < 2; ++comp) {
    const int m = comp ? m1 : m0;
    if (m == 0 || (comp == 1 && both)) continue;
    const int kd = comp ? kd1 : kd0;
    const int32_t* row_tb = a.tb + ((int64_t)cw * (2 * g.H) + (m - 1)) * a.ntb;
    // Last table entry written for harmonic m (see the spreading kernel).
    const double last = cell_of((t_last - mo.T0) * g.df, m, Ld, coff, FLR);
    const int64_t lim = (int64_t)floor((last + (double)(g.w / 2 + 2)) / (double)((int64_t)1 << tbl)) + 3;
#pragma unroll
    for (int j = 0; j < RPT; ++j) {
      int row, c0;
      if constexpr (TPR > 1) {
        row = tid / TPR;
        c0 = (tid % TPR) * kEPT;
      } else {
        row = tid + j * NTH;
        c0 = 0;
      }
      if (row >= r_lim) continue;
      const int64_t cell0 = g0 + c0 + Sd * (int64_t)row;
      // The grid is periodic: the segment gathers its points lap after lap
      // (positions on the unwrapped axis, table over g.laps periods).
     for (int lap = 0; lap < g.laps; ++lap) {
      const int64_t ucell = cell0 + (int64_t)lap * g.L;
      const int64_t ta = ucell >> tbl, tb2 = ((ucell + CPR - 1) >> tbl) + 2;
      if (ta > lim - 2) break;  // no point of harmonic m reaches this far
      const int64_t lo = pa + row_tb[ta];
      const int64_t hi = tb2 <= lim ? pa + row_tb[tb2] : pa + mo.n;
      const double c0d = (double)ucell;
      const double reach = (double)(g.w / 2 + 1);
      for (int64_t i = lo; i < hi; ++i) {
        const double pos = cell_at(t[i], mo.T0, g.df, m, Ld, coff, FLR);
        // Only points within the kernel's reach of the segment add a nonzero
        // tap (the others add exact zeros): skip those before it, stop after.
        if (pos < c0d - reach) continue;
        if (pos > c0d + (double)(CPR - 1) + reach) break;
        const double si = sg[i];
        const double w = 1.0 / (si * si);
        const double wy = w * (x[i + mo.xshift] - mo.xbar);
        const double va = kd == 0 ? w : wy;
        const double vb = both ? (kd1 == 0 ? w : wy) : 0.0;
#pragma unroll
        for (int u = 0; u < CPR; ++u) {
          const double phi = es_kernel<EXACT>(((c0d + (double)u) - pos) * two_over_w, beta);
          if (comp == 0) {
            ar[j][u] += phi * va;
            if (both) ai[j][u] += phi * vb;
          } else {
            ai[j][u] += phi * va;
          }
        }
      }
     }
    }
  }
#pragma unroll
  for (int j = 0; j < RPT; ++j) {
    const int row = (TPR > 1) ? tid / TPR : tid + j * NTH;
    const int c0 = (TPR > 1) ? (tid % TPR) * kEPT : 0;
#pragma unroll
    for (int u = 0; u < CPR; ++u)
      sm[tile_col<S, LOGT>(row, c0 + u)] = cmk<S>((S)ar[j][u], (S)ai[j][u]);
  }
  __syncthreads();
}

// The variants of a pass: the first (TILE_FIRST2: of two passes), middle and
// single passes, the last forward pass of an ordinary plan (TILE_LAST: the half
// of the outputs that no bin needs is known at compile time) and any other last
// pass (TILE_LAST_ANY: band plans and the adjoint).
enum TileKind : int {
  TILE_FIRST = 0,
  TILE_MID = 1,
  TILE_LAST = 2,
  TILE_LAST_ANY = 3,
  TILE_SINGLE = 4,
  TILE_FIRST2 = 5
};
constexpr bool kind_first(int kind) { return kind == TILE_FIRST || kind == TILE_FIRST2; }

// One pass.  Twiddles between passes, for output row k of tile column cc:
//   PASS_FIRST, np >= 3: w_M^{jd k}        (jd fixed for the tile)   = r[k]
//   PASS_FIRST, np == 2: w_L^{c k}, c = g0 + cc = G + h  = w_L^{G k} * w_L^{h k}
//                        (h < TB, G a multiple of TB = 2^12 / N)
//   PASS_MID:            w_M^{jd (K0+cc+Tail k)}                     = c[cc] r[k]
// with r, c built per workgroup in FP64 from exactly reduced exponents; the two
// factors of the two-pass form are the plan's (Pass2Tw), so that a tile neither
// evaluates N sines and cosines nor gathers w_L^{h k} in scattered order.
//
// LDS of one tile: the data tile, the stage twiddles (FP32), the row and
// column twiddles and, in the first pass, the output offset of each tile
// column.  FP64 tiles keep the row twiddles in the padding column of the data
// tile (one 16-byte slot per row that no data access touches), which brings
// the 2^9 x 8 tile from 82 to 74 KB: two workgroups per CU instead of one.
// The two-pass first pass of FP32 grids puts its row factors where the stage
// twiddles were.  The FP32 tile of 2^9 x 16 takes the 80 KB that two workgroups
// per CU allow.
//
// Twiddle factors of the first of two passes with 2^LOGN rows: row[(G / TB) N +
// k] = w_L^{G k} and col[k TB + h] = w_L^{h k}, in FP64.  The columns of a tile
// of T = TB or 2 TB columns form G groups, so both tile sizes multiply the same
// factors.
template <int LOGN, int LOGT>
struct Pass2Tw {
  static constexpr int TB = LOGN < 12 ? 1 << (12 - LOGN) : 1;
  static constexpr int G = (1 << LOGT) / TB > 0 ? (1 << LOGT) / TB : 1;
  static constexpr int ROWS = G << LOGN;
};

template <typename S, int LOGN, int LOGT, int KIND>
struct FftSmem {
  static constexpr int N = 1 << LOGN;
  static constexpr int T = 1 << LOGT;
  static constexpr int PT = tile_pitch<S, LOGT>();
  static constexpr bool kTrInPad = sizeof(cplx<S>) == sizeof(C) && T > 1;
  static constexpr bool kTw = KIND == TILE_FIRST || KIND == TILE_MID;
  static constexpr int kSt = StageTw<S, LOGN, LOGT>::SIZE;
  static constexpr int kRows = KIND == TILE_FIRST2 && !kTrInPad ? Pass2Tw<LOGN, LOGT>::ROWS : 0;
  __align__(16) cplx<S> sm[N * PT];
  C st[kSt > kRows ? kSt : kRows];
  C tr[kTw && !kTrInPad ? N : 0];
  // middle pass: column twiddles; first pass: output byte offset of each column
  C aux[KIND == TILE_MID ? T : (KIND == TILE_FIRST ? (T + 3) / 4 : 0)];
  __device__ __forceinline__ C* tc() { return aux; }
  __device__ __forceinline__ uint32_t* s_rev() { return reinterpret_cast<uint32_t*>(aux); }
  __device__ __forceinline__ C& row_tw(int k) {
    if constexpr (kTrInPad)
      return *reinterpret_cast<C*>(&sm[k * PT + T]);
    else
      return tr[k];
  }
};

// One tile of one pass: columns [bx T, bx T + T) of packed grid p of wave slot
// cw, whose grid is at in + grid_off (input) and out + grid_off (output) and
// whose pruned spectra (last forward pass) start at zpair.  Every thread of
// the workgroup calls it (it synchronises the workgroup).
//
// What bounds it: HBM, once the work per element is small enough to hide.  The
// rows a thread loads and stores are b0 + (N/16) j of one column, so every
// address is one per-thread 32-bit offset past a uniform base.
template <typename S, int LOGN, int LOGT, bool FUSED, int KIND>
__device__ __forceinline__ void fft_pass_tile(const FftPassArgs& a, const cplx<S>* in,
                                              cplx<S>* out, const Moments* __restrict__ mom,
                                              const Geom& g, const C* __restrict__ tw_stage,
                                              int bx, int p, int cw, int64_t grid_off, cplx<S>* zpair,
                                              FftSmem<S, LOGN, LOGT, KIND>& sh,
                                              int tid) {
  constexpr int N = 1 << LOGN;
  constexpr int T = 1 << LOGT;
  constexpr bool FIRST = kind_first(KIND);
  constexpr int PT = tile_pitch<S, LOGT>();
  constexpr int kNT = (N * T) / kEPT;  // threads of this tile
  constexpr int R16 = N / kEPT;        // row step of a thread's elements
  constexpr uint32_t ES = sizeof(cplx<S>);
  static_assert(N * T == 4096 || (N * T == 8192 && sizeof(S) == 4), "tile size");
  static_assert(!FUSED || FIRST, "the spreading is fused into the first pass");
  constexpr bool NT = T * sizeof(cplx<S>) >= 128;
  using S0 = Stage<LOGN, LOGT, 0>;
  using SL = Stage<LOGN, LOGT, last_logns(LOGN)>;
  using Tw = StageTw<S, LOGN, LOGT>;
  cplx<S>* sm = sh.sm;

  const Moments& mo = mom[a.curve0 + cw];
  if (mo.flags & kCurveFatal) return;

  const int logL = a.logL;
  const uint32_t L = 1u << logL;
  const char* src = (const char*)(in + grid_off);
  char* dst = (char*)(out + grid_off);
  const uint32_t g0 = (uint32_t)bx << LOGT;  // first column of this tile

  int low_bits = 0;  // sum of log2 N over digits below q
  if constexpr (KIND == TILE_MID)
    for (int d = 1; d < a.q; ++d) low_bits += a.logn[d];
  // Column c = g0 + cc of the tile: its rows are 2^logS elements apart, from
  // element `first` + cc on (PASS_MID: column (pre, K0 + cc) of the digit-
  // reversed layout, the others' rows span the whole grid).
  const int logS = logL - low_bits - LOGN;
  uint32_t pre = 0, K0 = g0, first = g0;
  if constexpr (KIND == TILE_MID) {
    pre = g0 >> logS;
    K0 = g0 - (pre << logS);
    first = (pre << (LOGN + logS)) + K0;
  }
  // Thread: column cc, rows b0 + R16 j.
  const uint32_t cc0 = (uint32_t)tid & (T - 1), b0 = (uint32_t)tid >> LOGT;
  const uint32_t voff = ((b0 << logS) + cc0) * ES;
  const uint64_t rstep = (uint64_t)(R16 * ES) << logS;  // bytes between its rows
  const char* rb = src + (uint64_t)first * ES;

  Tw::fill(sh.st, tw_stage, tid, kNT);

  C v[kEPT];
  using P2 = Pass2Tw<LOGN, LOGT>;
  constexpr bool F64 = sizeof(S) == 8;
  static_assert(KIND != TILE_FIRST2 || P2::ROWS <= 2 * kNT, "row factors per thread");
  // TILE_FIRST2, FP32: row factors on their way to LDS (scalars: a struct copied
  // from memory to LDS would stay in memory between).
  double rax = 0.0, ray = 0.0, rbx = 0.0, rby = 0.0;
  // Stage-0 inputs straight from HBM: element i is row b0 + R16 i.
  static_assert(S0::PER == 1, "one radix-16 butterfly per thread in the first stage");
  if constexpr (FIRST || KIND == TILE_SINGLE) {
    uint32_t z_lo, z_hi;  // rows in [z_lo, z_hi) are zero
    if (a.mode == MODE_FWD) {
      const int64_t E = pair_extent(mo, g, p);
      z_lo = (uint32_t)((E + ((int64_t)1 << logS) - 1) >> logS);
      z_hi = N;
    } else {
      z_lo = (uint32_t)(g.n_freq >> logS);
      z_hi = (uint32_t)((g.L - g.n_freq) >> logS);
    }
    if constexpr (FUSED) {
      // Forward first pass only (the launcher guarantees it).
      if (g.w == 1)
        spread_into_tile<S, LOGN, LOGT, true>(a, mo, g, p, cw, g0, z_lo, sm, tid);
      else
        spread_into_tile<S, LOGN, LOGT, false>(a, mo, g, p, cw, g0, z_lo, sm, tid);
#pragma unroll
      for (int i = 0; i < kEPT; ++i) v[i] = widen(sm[tile_col<S, LOGT>(b0 + i * R16, cc0)]);
    } else {
      // Loads first, conversions after (the empty asm keeps the compiler from
      // moving them up): a conversion inside its row's branch would wait for
      // that one load, sixteen memory latencies in turn.
      cplx<S> raw[kEPT];
#pragma unroll
      for (int i = 0; i < kEPT; ++i) {
        const uint32_t r = b0 + i * R16;
        raw[i] = cmk<S>((S)0, (S)0);
        if (r < z_lo || r >= z_hi) raw[i] = ntl<NT, S>(rb + i * rstep, voff);
      }
#pragma unroll
      for (int i = 0; i < kEPT; ++i) {
        asm("" : "+v"(raw[i].x), "+v"(raw[i].y));
        v[i] = widen(raw[i]);
      }
    }
  } else {
#pragma unroll
    for (int i = 0; i < kEPT; ++i) v[i] = widen(ntl<NT, S>(rb + i * rstep, voff));
  }

  if constexpr (KIND == TILE_FIRST) {
    const int np = a.np;
    const int logM = a.logn[np - 1] + LOGN;
    int bits_below = 0;
    for (int d = 1; d < np - 1; ++d) bits_below += a.logn[d];
    const int64_t jd = (int64_t)(g0 >> bits_below);
    const int64_t Mmask = ((int64_t)1 << logM) - 1;
    for (int k = tid; k < N; k += kNT) sh.row_tw(k) = root((jd * k) & Mmask, logM);
  } else if constexpr (KIND == TILE_FIRST2) {
    const C* rt = (const C*)a.tw_row + ((uint64_t)(g0 / P2::TB) << LOGN);
    if constexpr (F64) {
      for (int k = tid; k < N; k += kNT) sh.row_tw(k) = rt[k];
    } else {
      rax = rt[tid < P2::ROWS ? tid : 0].x;
      ray = rt[tid < P2::ROWS ? tid : 0].y;
      if constexpr (P2::ROWS > kNT) {
        rbx = rt[tid + kNT].x;
        rby = rt[tid + kNT].y;
      }
    }
  } else if constexpr (KIND == TILE_MID) {
    const int lg = a.logn[a.q - 1];
    const int64_t jd = pre & ((1u << lg) - 1u);
    const int logM = lg + LOGN + logS;
    const int64_t Mmask = ((int64_t)1 << logM) - 1;
    for (int k = tid; k < N; k += kNT) sh.row_tw(k) = root(((jd << logS) * k) & Mmask, logM);
    for (int cc = tid; cc < T; cc += kNT) sh.tc()[cc] = root((jd * (K0 + cc)) & Mmask, logM);
  }

  // The LDS twiddles become visible at the barriers inside run_stages, or below.
  run_stages<S, LOGN, LOGT, 0, PT, FUSED>(v, sm, tw_stage, sh.st, tid);
  if constexpr (last_logns(LOGN) == 0) __syncthreads();  // single-stage tile

  // Output row b0 + R16 j is element j / PER of butterfly slot j % PER.
  auto at = [&](int j) -> C& { return v[(j % SL::PER) * SL::RAD + j / SL::PER]; };
  if constexpr (KIND == TILE_FIRST) {
#pragma unroll
    for (int j = 0; j < kEPT; ++j) at(j) = cmul_r(at(j), sh.row_tw(b0 + R16 * j));
  } else if constexpr (KIND == TILE_FIRST2) {
    // Entries read ahead: enough to cover the L2's latency, and no more than
    // the registers of two workgroups per CU allow.
    constexpr int kAhead = LOGN == 5 || LOGN == 7 ? 2 : 4;
    const C* tt = (const C*)a.tw_col + (b0 * P2::TB + (cc0 & (P2::TB - 1)));
    C nx[kAhead];
#pragma unroll
    for (int j = 0; j < kAhead; ++j) nx[j] = tt[j * (R16 * P2::TB)];
    const C* rw = sh.st + ((cc0 / P2::TB) << LOGN);
    if constexpr (!F64) {
      __syncthreads();  // the stage twiddles have been read
      if (tid < P2::ROWS) sh.st[tid] = cmk<double>(rax, ray);
      if constexpr (P2::ROWS > kNT) sh.st[tid + kNT] = cmk<double>(rbx, rby);
      __syncthreads();
    }
#pragma unroll
    for (int j = 0; j < kEPT; ++j) {
      const C t = nx[j % kAhead];
      if (j + kAhead < kEPT) nx[j % kAhead] = tt[(j + kAhead) * (R16 * P2::TB)];
      C r;
      if constexpr (F64)
        r = sh.row_tw(b0 + R16 * j);
      else
        r = rw[b0 + R16 * j];
      at(j) = cmul_r(at(j), cmul_r(r, t));
      __builtin_amdgcn_sched_barrier(0);
    }
  } else if constexpr (KIND == TILE_MID) {
    const C fc = sh.tc()[cc0];
#pragma unroll
    for (int j = 0; j < kEPT; ++j)
      at(j) = cmul_r(at(j), cmul_r(fc, sh.row_tw(b0 + R16 * j)));
  }

  if constexpr (FIRST) {
    // Transpose through LDS so that each column's N outputs leave as one
    // contiguous run at row rev(c) of the output.
    if constexpr (KIND == TILE_FIRST || F64) __syncthreads();
#pragma unroll
    for (int j = 0; j < kEPT; ++j) sm[tile_col<S, LOGT>(b0 + R16 * j, cc0)] = narrow<S>(at(j));
    if constexpr (KIND == TILE_FIRST) {
      // Mixed-radix reversal of each of the tile's T columns, once per tile:
      // rev = ((j_1 N_2 + j_2) N_3 + j_3) ... + j_{np-1} for column c = g0 + cc.
      for (int cc = tid; cc < T; cc += kNT) {
        uint32_t rev = 0, rest = g0 + cc;
        for (int d = 1; d < a.np; ++d) {
          const uint32_t dig = rest & ((1u << a.logn[d]) - 1u);
          rest >>= a.logn[d];
          rev = (rev << a.logn[d]) | dig;
        }
        sh.s_rev()[cc] = rev * (N * ES);
      }
    }
    __syncthreads();
#pragma unroll 4
    for (int it = 0; it < kEPT; ++it) {
      const int e = tid + it * kNT;
      const int k = e & (N - 1);
      const int cc = e >> LOGN;
      // of two passes: rev(c) = c
      const uint32_t ro = KIND == TILE_FIRST ? sh.s_rev()[cc] : (g0 + cc) * (N * ES);
      nts<NT, S>(dst, ro + k * ES, sm[tile_col<S, LOGT>(k, cc)]);
    }
  } else if constexpr (KIND == TILE_MID) {
    char* wb = dst + (uint64_t)first * ES;
#pragma unroll
    for (int j = 0; j < kEPT; ++j) nts<NT, S>(wb + j * rstep, voff, narrow<S>(at(j)));
  } else if constexpr (KIND == TILE_LAST) {
    // X = g0 + cc + Tail k: bins X < n_freq = L / 4 (rows j < 4) to the direct
    // half and bins L - X (rows j >= 12) to the mirror half, where bin k is
    // element k - 1: a run of columns X, aligned to its length, is then as
    // aligned in reverse (from element k on, every run of 128 bytes would
    // leave as a part of two lines).  Row 12's X = L - n_freq fills the mirror
    // half's unused last element.
    char* z0 = (char*)zpair + (uint64_t)g0 * ES;
#pragma unroll
    for (int j = 0; j < 4; ++j) nts<false, S>(z0 + j * rstep, voff, narrow<S>(at(j)));
    // Element L - X - 1, counted from the tile's row 16 (j + 1) back.
    char* z1 = (char*)(zpair + (L >> 2)) - ((int64_t)g0 + 1) * (int64_t)ES;
    const uint32_t moff = (uint32_t)rstep - voff;
#pragma unroll
    for (int j = 12; j < kEPT; ++j)
      nts<false, S>(z1 + (15 - j) * (int64_t)rstep, moff, narrow<S>(at(j)));
  } else {
    // PASS_LAST / PASS_SINGLE: X index = K + Tail * k, natural order.
    if (a.mode == MODE_FWD) {
      const uint32_t nf = (uint32_t)g.n_freq;
      cplx<S>* z0 = zpair;
      cplx<S>* z1 = z0 + nf;
#pragma unroll
      for (int j = 0; j < kEPT; ++j) {
        const uint32_t X = g0 + cc0 + ((b0 + R16 * j) << logS);
        const cplx<S> val = narrow<S>(at(j));
        if (X < nf) z0[X] = val;
        const uint32_t m1 = L - X - 1;  // mirror bin L - X is element L - X - 1
        if (m1 < nf) z1[m1] = val;
      }
    } else {
      const uint32_t E = (uint32_t)pair_extent(mo, g, p);
      cplx<S>* go = (cplx<S>*)a.grid_out + grid_off;
#pragma unroll
      for (int j = 0; j < kEPT; ++j) {
        const uint32_t X = g0 + cc0 + ((b0 + R16 * j) << logS);
        if (X < E) go[X] = narrow<S>(at(j));
      }
    }
  }
}

// Waves per SIMD a pass kernel is compiled for.  FP32 tiles of 8192
// elements are workgroups of eight waves with 68-80 KB of LDS, two per CU,
// which needs four waves per SIMD (at most 128 registers): without the bound an
// earlier form of the 2^9-row tiles took 130 registers and the CU one workgroup
// (a curve of 1e6 points, H = 8, 2^24 bins: FFT 9.3 -> 8.1 ms).  The fused
// first pass (spreading inside the tile) keeps its own allocation: at 128
// registers it spills.
template <typename S, bool FUSED>
constexpr int fft_pass_waves() {
  return (sizeof(S) == 4 && !FUSED) ? 4 : 1;
}

// The factors of Pass2Tw for rows of 2^logn: col from small[e] = w_L^e, e < 2^12,
// row from exactly reduced exponents.
__global__ void k_pass2_tw(const C* __restrict__ small, int logn, int logL, C* __restrict__ col,
                           C* __restrict__ row) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int logb = 12 - logn;
  if (e < 1 << 12) col[e] = small[(e & ((1 << logb) - 1)) * (e >> logb)];
  if (e < ((int64_t)1 << (logL - logb))) {
    const int64_t G = (e >> logn) << logb, k = e & ((1 << logn) - 1);
    row[e] = root((G * k) & (((int64_t)1 << logL) - 1), logL);
  }
}

// The pass over a wave of curves: grid (column tiles, pairs, curves).
template <typename S, int LOGN, int LOGT, bool FUSED, int KIND>
__global__ __launch_bounds__(((1 << LOGN) << LOGT) / kEPT, (fft_pass_waves<S, FUSED>())) void k_fft_pass(
    FftPassArgs a, const cplx<S>* in, cplx<S>* out, const Moments* __restrict__ mom, Geom g,
    const C* __restrict__ tw_stage) {
  __shared__ FftSmem<S, LOGN, LOGT, KIND> sh;
  const int p = blockIdx.y;
  const int cw = blockIdx.z;
  const int64_t grid_off = ((int64_t)cw * g.P + p) * g.L;
  cplx<S>* zpair = a.zc ? (cplx<S>*)a.zc + ((int64_t)cw * g.P + p) * 2 * g.n_freq : nullptr;
  fft_pass_tile<S, LOGN, LOGT, FUSED, KIND>(a, in, out, mom, g, tw_stage, blockIdx.x, p, cw,
                                            grid_off, zpair, sh, threadIdx.x);
}

}  // namespace

}  // namespace fchi2
