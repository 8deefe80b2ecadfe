// The spreading of one wave and its tile -> point-range table (shared by the
// spreading kernels and the persistent batched search); see spread.hip.
#pragma once

#include <cmath>
#include <type_traits>

#include "fchi2_internal.h"
#include "es_kernel.h"

namespace fchi2 {

namespace {

constexpr int kNT = 256;

// Tile -> point-range table.  For harmonic m and tile t of B cells, the
// points a tile may need are those with position in
// [x_t, x_{t+2}), x_t = t B - w/2 - 2 (a superset of the kernel footprint).
// tb[t] = first point index i (relative to the curve) with pos_i >= x_t.  The
// intervals (pos_{i-1}, pos_i] partition the line, so thread i writes exactly
// the entries whose x_t falls in its interval: one scatter, no searches.
// Last table entry written for harmonic m: the tile after the one holding the
// last point's footprint, plus the two-tile lookahead of the spreading.  (The
// last point's time is T0 + span: mo.span is t_last - T0 as the positions form
// it.)
__device__ __forceinline__ int64_t tile_limit_of(const Moments& mo, const Geom& g, int m,
                                                 int log_tile) {
  const double last = cell_of(mo.span * g.df, m, (double)g.L, (double)g.c_off, g.w == 1);
  return (int64_t)floor((last + (double)(g.w / 2 + 2)) / (double)((int64_t)1 << log_tile)) + 3;
}

// The table entries owned by point il (0..n; n: past the last point) of
// harmonic m for the curve mo in table slot cw.  Every lane of a wave calls it.
//
// A lane stores the entries of its own point one after another; an observing
// gap leaves one point most of a grid's entries, so an interval of more than
// kOwn is stored by the whole wave, a run of 64 at a time.  Table and spreading
// with a third of the span empty, one lane storing the gap and the wave: 1e5
// points on 2^22 bins, H = 5, 1118 and 167 us (without the gap 167); 300 points on 2^24
// bins, H = 3, 4575 and 347 (300).  kOwn of 4, 8, 32 and 64 measure the same.
__device__ __forceinline__ void tile_bounds_point(const double* __restrict__ t,
                                                  const Moments& mo, const Geom& g, int cw,
                                                  int m, int64_t il, int log_tile, int ntb,
                                                  int32_t* __restrict__ tb) {
  constexpr int kOwn = 16;
  const double Ld = (double)g.L, coff = (double)g.c_off;
  const double B = (double)((int64_t)1 << log_tile);
  const double shift = (double)(g.w / 2 + 2);
  int64_t t_min = 0, t_max = -1;
  if (il <= mo.n) {
    if (il > 0) {
      const double lo = cell_at(t[mo.start + il - 1], mo.T0, g.df, m, Ld, coff, g.w == 1);
      t_min = (int64_t)floor((lo + shift) / B) + 1;
    }
    if (il == mo.n) {
      t_max = tile_limit_of(mo, g, m, log_tile);
    } else {
      const double hi = cell_at(t[mo.start + il], mo.T0, g.df, m, Ld, coff, g.w == 1);
      t_max = (int64_t)floor((hi + shift) / B);
    }
    if (t_min < 0) t_min = 0;
    if (t_min > ntb) t_min = ntb;
    if (t_max > ntb - 1) t_max = ntb - 1;
  }
  const int a = (int)t_min, e = (int)t_max;
  int32_t* row = tb + ((int64_t)cw * (2 * g.H) + (m - 1)) * ntb;
  const bool own = e - a < kOwn;
  if (own)
    for (int q = a; q <= e; ++q) row[q] = (int32_t)il;
  const int lane = (int)(threadIdx.x & 63);
  for (uint64_t left = __ballot(!own); left; left &= left - 1) {
    const int src = __ffsll((unsigned long long)left) - 1;
    const int a1 = __builtin_amdgcn_readlane(a, src), e1 = __builtin_amdgcn_readlane(e, src);
    const int v = __builtin_amdgcn_readlane((int)il, src);
    for (int q = a1 + lane; q <= e1; q += 64) row[q] = v;
  }
}

// The spreading of one wave: four groups of 16 lanes, each summing one
// component of a strip of 2^LS consecutive cells of a packed grid: two strips'
// real and imaginary parts, or (band plans: one complex component) four
// strips.  LS is the granularity of the spreading's tile table: 7, or 5 where
// the grids are too small to fill the device with strips of 128 cells.
constexpr int kStripLogMax = 7, kStripLogMin = 5;
constexpr int spread_strips_per_wave(bool band) { return band ? 4 : 2; }

// The points of one component of a dense wave, up to kCellPoints at a time: the
// cell coordinate relative to the wave's first cell and the strength, with room
// for the sentinels that end them.  384 points are 24 KB a workgroup, which
// leaves the five workgroups per CU that the registers allow (FP64: four; the
// complex strengths of band plans: 36 KB, four, FP64 three); with
// both components staged at once, at half the points, several long curves on
// small grids (100 of 5000 points, H = 8, 2^11 bins) took a fifth longer.
constexpr int kCellPoints = 384, kTapUnroll = 4;
template <bool BAND>
struct CellPoints {
  double2 q[kCellPoints + kTapUnroll];
};
template <>
struct CellPoints<true> {
  double2 q[kCellPoints + kTapUnroll];
  double im[kCellPoints + kTapUnroll];
};
struct NoPoints {};

// What one wave of the spreading holds: the cells of its strips, in FP64 until
// they are written, or (DENSE) points.
template <int LS, bool BAND, bool DENSE>
union SpreadSmem {
  static constexpr int kCells = spread_strips_per_wave(BAND) << LS;
  struct {
    double re[kCells], im[kCells];
  } cell;
  typename std::conditional<DENSE, CellPoints<BAND>, NoPoints>::type pts;
};

// Sixteen points of a strip, one per lane of its group: the cell coordinate
// relative to the strip's first cell (exact: a multiple of the coordinate's
// ulp, smaller than it) and the strength (im: band plans only).
struct PointLane {
  double rel, re, im;
};

template <bool BAND>
__device__ __forceinline__ PointLane load_point(const double* __restrict__ t,
                                                const double* __restrict__ x,
                                                const double* __restrict__ sigma,
                                                const Moments& mo, const Geom& g, int m, int kind,
                                                int64_t i, double base) {
  PointLane q;
  const double ti = t[i], si = sigma[i], xi = x[i + mo.xshift];
  // floor gridding: the coordinate is an integer and the kernel is exp(0) = 1
  // at d = 0 and 0 at |d| >= 1 (w = 1)
  q.rel = cell_at(ti, mo.T0, g.df, m, (double)g.L, (double)g.c_off, g.w == 1) - base;
  const double w = 1.0 / (si * si);
  const double sa = kind == 0 ? w : w * (xi - mo.xbar);
  if constexpr (BAND) {
    // Band plan: strength times exp(+2 pi i kc m u), kc = k0 + n_freq/2 the
    // band's middle bin, so that grid bin j (j - L for j >= L/2) is bin
    // kc + j of the search.  The phase kc m u in cycles is reduced modulo 1
    // from the FP64 product and its exact rounding residual.
    const double km = (double)((g.k0 + g.n_freq / 2) * (int64_t)m);
    const double u = (ti - mo.T0) * g.df;
    const double ph = km * u;
    const double r = fma(km, u, -ph);
    double fr = (ph - floor(ph)) + r;
    fr -= floor(fr);
    double sn, cs;
    sincospi(2.0 * fr, &sn, &cs);
    q.re = sa * cs;
    q.im = sa * sn;
  } else {
    q.re = sa;
    q.im = 0.0;
  }
  return q;
}

// Whether a wave's strips are spread with a lane per cell, from the points of each
// lane's group (n).  Fewer than 48 points: a group's sixteen take them in a round
// or two.  Many in few cells: every cell sees most points, so a lane's own
// sequence is as long as a strip's, and the two components (band plans: the two
// runs of 64 cells) follow each other (640 points, 2^10 bins, H = 4, 18 points a
// cell in the first pair: FP32 54 us of spreading against 92 with the strips, FP64
// 146 against 134; 20 bands of 3000 points, 2^11 bins, H = 2, 30 a cell, the whole
// search by cells throughout 336 against 291 us, FP64 853 against 460).
template <bool EXACT, bool BAND>
__device__ __forceinline__ bool cells_pay(int n) {
  const int a = __builtin_amdgcn_readlane(n, 0) + __builtin_amdgcn_readlane(n, 16);
  const int b = __builtin_amdgcn_readlane(n, 32) + __builtin_amdgcn_readlane(n, 48);
  if constexpr (BAND) return a + b >= 48 && a + b <= (EXACT ? 2000 : 3000);
  return a + b >= 48 && (a > b ? a : b) <= (EXACT ? 1000 : 1500);
}

// The wave's strips of packed grid p from `strip` on, a lane per cell (band plans:
// two, 64 cells apart), where they hold many points: from points staged in LDS a
// lane adds to its cell the taps within the kernel's reach, in index order, four
// at a time (the first found by binary search).  Every tap it evaluates is of use,
// where a group's sixteen lanes share the ten or fourteen of a point, and a point
// is loaded once for the wave instead of once for every strip of 32 that it reaches.
// Each cell adds the same terms in the same order as in spread_strips.
//
// What bounds it: FP64 arithmetic where many curves fill the device, the longest
// sequence of taps elsewhere.  Spreading of equal curves, H = 4, in us, the
// harmonics over 7, 20 and 70 % of the grid, three figures each: by a workgroup
// per tile of 1024 cells (the form before the strips); by strips alone; with this:
//   400 of 640 points, 2^10 bins:  201, 130, 172;  357, 274, 207;  220, 127, 145
//   150 of 5120 points, 2^13 bins: 568, 434, 411;  570, 493, 502;  404, 249, 339
//   one of 640 points, 2^10 bins:   72,  38,  37;   92,  58,  24;   54,  23,  16
// Band plans, one sincospi a point and wave instead of one for every strip, the
// whole search, H = 5, over 10 and 80 %:
//   300 of 3000 points, 2^13 bins: 1271, 1360;  1717, 1109;  1157, 990
//   20 of 50000 points, 2^16 bins: 4200, 1138;  1840, 974;   1105, 763
template <typename S, int LS, bool BAND>
__device__ __forceinline__ void spread_cells(const double* __restrict__ t,
                                             const double* __restrict__ x,
                                             const double* __restrict__ sigma,
                                             const Moments& mo, const Geom& g,
                                             const int32_t* __restrict__ rows, int ntb, int p,
                                             int strip, cplx<S>* __restrict__ out,
                                             CellPoints<BAND>& sh, int lane) {
  constexpr int kStrips = spread_strips_per_wave(BAND), kRuns = kStrips / 2;
  static_assert(kStrips << LS == 64 * kRuns, "a lane per cell of two strips");
  static_assert(kCellPoints < 512, "the search's first step");
  constexpr bool EXACT = sizeof(S) == 8;
  const double two_over_w = 2.0 / (double)g.w;
  const double beta = g.beta;
  const double half = 0.5 * (double)g.w;
  const int nstrip = (int)(g.L >> LS);
  double acc[2], acc_i[2];  // of components, or (BAND) of the wave's two runs of 64 cells
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // the points take the cells' place
  // one body for both components: unrolled, its registers cost waves
#pragma unroll 1
  for (int c = 0; c < (BAND ? 1 : 2); ++c) {
    const int m = g.comp_m[p][c], kind = g.comp_kind[p][c];
    const int32_t* row = rows + (int64_t)(m - 1) * ntb;
    const int lim = m ? (int)tile_limit_of(mo, g, m, LS) : 0;
    double a[kRuns], ai[kRuns];
#pragma unroll
    for (int h = 0; h < kRuns; ++h) a[h] = ai[h] = 0.0;
    for (int lap = 0; lap < g.laps; ++lap) {
      const int ut = strip + lap * nstrip;
      if (ut + 2 > lim) break;  // no point reaches this far
      const double base = (double)((int64_t)ut << LS);
      const int end = ut + kStrips + 1;
      int lo = __builtin_amdgcn_readfirstlane(row[ut]);
      const int hi = __builtin_amdgcn_readfirstlane(row[end <= lim ? end : lim]);
      while (lo < hi) {
        const int n = hi - lo < kCellPoints ? hi - lo : kCellPoints;
        for (int i = lane; i < n; i += 64) {
          const PointLane pt =
              load_point<BAND>(t, x, sigma, mo, g, m, kind, mo.start + lo + i, base);
          sh.q[i] = make_double2(pt.rel, pt.re);
          if constexpr (BAND) sh.im[i] = pt.im;
        }
        if (lane < kTapUnroll) {
          sh.q[n + lane] = make_double2(1e300, 0.0);
          if constexpr (BAND) sh.im[n + lane] = 0.0;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        const double2* q = sh.q;
#pragma unroll 1
        for (int h = 0; h < kRuns; ++h) {
          const double cl = (double)(lane + 64 * h);
          double s = h ? a[kRuns - 1] : a[0], si = h ? ai[kRuns - 1] : ai[0];
          int k = 0;
#pragma unroll
          for (int step = 256; step > 0; step >>= 1)
            if (k + step <= n && q[k + step - 1].x < cl - half) k += step;
          while (q[k].x <= cl + half) {
            double phi[kTapUnroll], v[kTapUnroll], vi[kTapUnroll];
#pragma unroll
            for (int u = 0; u < kTapUnroll; ++u) {
              phi[u] = es_kernel<EXACT>((cl - q[k + u].x) * two_over_w, beta);
              v[u] = q[k + u].y;
              if constexpr (BAND) vi[u] = sh.im[k + u];
            }
#pragma unroll
            for (int u = 0; u < kTapUnroll; ++u) {
              s = fma(phi[u], v[u], s);
              if constexpr (BAND) si = fma(phi[u], vi[u], si);
            }
            k = k + kTapUnroll < n ? k + kTapUnroll : n;
          }
          (h ? a[kRuns - 1] : a[0]) = s;
          (h ? ai[kRuns - 1] : ai[0]) = si;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        lo += n;
      }
    }
    if constexpr (BAND) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        acc[h] = a[h];
        acc_i[h] = ai[h];
      }
    } else {
      (c ? acc[1] : acc[0]) = a[0];
    }
  }
  if constexpr (BAND) {
    out[lane] = cmk<S>((S)acc[0], (S)acc_i[0]);
    out[lane + 64] = cmk<S>((S)acc[1], (S)acc_i[1]);
  } else {
    out[lane] = cmk<S>((S)acc[0], (S)acc[1]);
  }
}

// The wave's strips from `strip` on, of packed grid p of the curve mo (its table
// rows at `rows`, ntb entries per harmonic), written to out.  One wave calls
// it; sh is the wave's own.
//
// Lane r of a group owns the cells j = r (mod 16) of its strip.  A point's
// nonzero taps (at most 16 = the largest kernel width) are 16 consecutive
// cells, one per lane, and points come in time order, so a lane meets its
// cells in ascending order: it adds phi(cell - point) times the strength to a
// running sum and stores the sum when the next point's window has moved past
// the cell.  Every cell adds its points in index order, as one thread per cell
// would: deterministic, no atomics, and work per tap instead of per cell (a
// curve of 1000 points touches a few per cent of its grid's cells).
//
// What bounds it: the exponentials of the taps and, on sparse grids, the
// latency of table and point loads, covered by twenty independent waves per CU
// (no workgroup barrier).  The points of a group go round its lanes by row
// broadcasts, a DPP row being a group, with no LDS permute on the chain of one
// point's tap (150 curves of 5120 points, H = 4, 2^13 bins: 571 us with the
// permutes, 496 now; 20 curves of 1280 points on 2^11 bins: 92 and 75).
template <typename S, int LS, bool BAND, bool DENSE = false>
__device__ __forceinline__ void spread_strips(const double* __restrict__ t,
                                              const double* __restrict__ x,
                                              const double* __restrict__ sigma,
                                              const Moments& mo, const Geom& g,
                                              const int32_t* __restrict__ rows, int ntb, int p,
                                              int strip, cplx<S>* __restrict__ out,
                                              SpreadSmem<LS, BAND, DENSE>& smem, int lane) {
  constexpr bool EXACT = sizeof(S) == 8;
  constexpr int kStrip = 1 << LS;
  constexpr int kWaveCells = SpreadSmem<LS, BAND, DENSE>::kCells;
  auto& sh = smem.cell;
  const int grp = lane >> 4, r = lane & 15;
  const double two_over_w = 2.0 / (double)g.w;
  const double beta = g.beta;
  const double reach = (double)(kStrip + g.w / 2 + 1);
  const int nstrip = (int)(g.L >> LS);
  const int comp = BAND ? 0 : grp >> 1;
  const int sub = BAND ? grp : grp & 1;
  const int m = g.comp_m[p][comp];
  const int kind = g.comp_kind[p][comp];
  const int32_t* row = rows + (int64_t)(m - 1) * ntb;
  const int lim = m ? (int)tile_limit_of(mo, g, m, LS) : 0;
  double* cells = (comp ? sh.im : sh.re) + sub * kStrip;
  double* cim = sh.im + sub * kStrip;
#pragma unroll
  for (int u = 0; u < kWaveCells / 64; ++u) {
    sh.re[lane + 64 * u] = 0.0;
    sh.im[lane + 64 * u] = 0.0;
  }
  __builtin_amdgcn_wave_barrier();
  // The grid is periodic: positions are kept unwrapped (the phase m u of a long
  // curve may span several periods), and the strips gather their points lap
  // after lap, in index order (positions grow with t).
  for (int lap = 0; lap < g.laps; ++lap) {
    const int ut = strip + sub + lap * nstrip;
    const bool any = ut + 2 <= lim;  // else no point reaches this far
    if (!__any(any)) break;
    int64_t lo = 0, hi = 0;
    if (any) {
      lo = mo.start + row[ut];
      hi = mo.start + row[ut + 2];
    }
    if constexpr (DENSE) {
      if (lap == 0 && cells_pay<EXACT, BAND>((int)(hi - lo))) {
        spread_cells<S, LS, BAND>(t, x, sigma, mo, g, rows, ntb, p, strip, out, smem.pts, lane);
        return;
      }
    }
    const double base = (double)((int64_t)ut << LS);
    int cur = -1;  // the lane's cell in hand
    double acc = 0.0, acc_i = 0.0;
    auto flush = [&]() {
      if (cur >= 0 && cur < kStrip) {
        cells[cur] = acc;
        if constexpr (BAND) cim[cur] = acc_i;
      }
    };
    for (int64_t b = lo; __any(b < hi); b += 16) {
      PointLane q;
      q.rel = 1e300;
      q.re = q.im = 0.0;
      if (b + r < hi) q = load_point<BAND>(t, x, sigma, mo, g, m, kind, b + r, base);
      // Points past the strip's reach add nothing, nor do those after them.
      const uint64_t near = __ballot(q.rel < reach);
      const int cnt = __popc((uint32_t)(near >> (16 * grp)) & 0xffffu);
      if (cnt < 16) hi = b;  // the group's last sixteen
      // Four points at a time: their taps do not depend on each other, only
      // the sums do.
      constexpr int kU = 4;
      for (int k = 0; __any(k < cnt); k += kU) {
        double phi[kU], vr[kU], vi[kU];
        int j[kU];
        static_for<0, kU>([&](auto uc) {
          constexpr int u = decltype(uc)::value;
          const double rel = row_bcast<u>(q.rel);
          vr[u] = row_bcast<u>(q.re);
          vi[u] = BAND ? row_bcast<u>(q.im) : 0.0;
          const int f = (int)floor(k + u < cnt ? rel : 0.0) - 7;
          j[u] = f + ((r - f) & 15);
          phi[u] = es_kernel<EXACT>(((double)j[u] - rel) * two_over_w, beta);
        });
#pragma unroll
        for (int u = 0; u < kU; ++u) {
          if (k + u < cnt) {
            if (j[u] != cur) {
              flush();
              cur = j[u];
              acc = acc_i = 0.0;
              if (lap > 0 && cur >= 0 && cur < kStrip) {  // a later lap continues the sum
                acc = cells[cur];
                if constexpr (BAND) acc_i = cim[cur];
              }
            }
            acc = fma(phi[u], vr[u], acc);
            if constexpr (BAND) acc_i = fma(phi[u], vi[u], acc_i);
          }
        }
        // the next four to the row's first lanes (row_ror 12: from lane r + 4)
        q.rel = row_move<0x12C>(q.rel);
        q.re = row_move<0x12C>(q.re);
        if constexpr (BAND) q.im = row_move<0x12C>(q.im);
      }
    }
    flush();
    __builtin_amdgcn_wave_barrier();
  }
#pragma unroll
  for (int u = 0; u < kWaveCells / 64; ++u) {
    const int c = lane + 64 * u;
    out[c] = cmk<S>((S)sh.re[c], (S)sh.im[c]);
  }
  __builtin_amdgcn_wave_barrier();
}

}  // namespace

}  // namespace fchi2
