// Per-frequency Delta chi2 for 9..16 harmonics (and, on request, for fewer):
// sixteen lanes per bin.
#include <cmath>
#include <type_traits>

#include "fchi2_internal.h"
#include "launch.h"
#include "solve_bin.h"

namespace fchi2 {

namespace {

constexpr int kNT = 256;

using namespace solve_detail;

// Wide solve for 9 <= H <= 16 (d = 2H + 1 <= 33 basis functions): the
// register solver's triangular factor would need d (d + 1) / 2 FP64 values per
// thread, so here sixteen lanes solve one bin, lane r holding rows r, r + 16
// and r + 32 of alpha.  Assembly (product-to-sum, Section 2), the pivot guard
// and the prefix sums are those of the register solver; the factorisation runs
// right-looking: at step j the pivot comes from row j's lane, every row below
// scales its entry L_ij and updates its columns with the L_kj of the rows
// above it, and the forward substitution z = L^-1 beta advances in the same
// step, so Delta chi2(H') = sum_{j <= 2H'} z_j^2 for every H' at once.
// Coefficients (COEF) by back substitution L^T A = z, one reduction over the
// bin's lanes per unknown.
//
// Sixteen lanes are a DPP row, and row_newbcast hands one lane's value to its
// row in one vector instruction, so no step goes through LDS (a whole wave per
// bin fetched every L_kj with two LDS permutes and left half its lanes idle:
// the whole search of three curves of 2^15 bins at H = 12 with coefficients
// took 1536 us, with this 230).  FP64 arithmetic bounds it, at two (H > 14) to
// four waves per SIMD.  A workgroup takes sixteen consecutive bins, so spectra
// and rows move in runs of sixteen.  DM: rows a build is unrolled for (d <= DM).
constexpr int kWideBins = kNT / 16;

template <bool COEF, int DM>
__global__ __launch_bounds__(kNT) void k_solve_wide(const void* __restrict__ zc,
                                                    const cplx<double>* __restrict__ D,
                                                    const Moments* __restrict__ mom, Geom g,
                                                    int curve0, double eps, bool fp64,
                                                    void* __restrict__ out,
                                                    uint8_t* __restrict__ flags,
                                                    void* __restrict__ coef) {
  constexpr int NQ = (DM + 15) / 16;  // rows per lane
  constexpr int HM = DM / 2;          // most harmonics
  constexpr int CP = 3 * HM + 3 - HM % 2;  // odd pitch of a bin's Q_m, -HM <= m <= 2 HM
  constexpr int PP = HM + 3 - HM % 2;      // and of its P_m, 0 <= m <= HM
  __shared__ double s_c[kWideBins][CP], s_s[kWideBins][CP];
  __shared__ double s_pr[kWideBins][PP], s_pi[kWideBins][PP];
  const int H = g.H;
  const int dd = 2 * H + 1;
  const int P = g.P;
  const int64_t nf = g.n_freq;
  const int tid = threadIdx.x;
  const int64_t kb = (int64_t)blockIdx.x * kWideBins;  // the block's first bin
  const int cw = blockIdx.y;
  const int c = curve0 + cw;
  const Moments& mo = mom[c];
  const int wb = tid & (kWideBins - 1), wr = tid / kWideBins;  // bin, row of a store
  const int64_t o = (int64_t)c * H * nf + kb + wb;
  const int64_t oc = (int64_t)c * dd * nf + kb + wb;
  uint8_t* of = flags ? flags + (int64_t)c * nf + kb : nullptr;
  // Spectra and results are FP64 or FP32 as the plan is; one branch here, not
  // a kernel for each.
  auto store = [&](void* p, int64_t i, double v) {
    if (fp64)
      ((double*)p)[i] = v;
    else
      ((float*)p)[i] = (float)v;
  };
  if (mo.flags & kCurveFatal) {  // whole block: uniform per curve
    if (wr < H) store(out, o + wr * nf, nan_of<double>());
    if constexpr (COEF)
      for (int j = wr; j < dd; j += 16) store(coef, oc + j * nf, nan_of<double>());
    if (of && tid < kWideBins) of[tid] = (uint8_t)(mo.flags & 0xF8u);
    return;
  }
  // Q_m = Q(m f_k) = C'_m + i S'_m, |m| <= 2H (C' even, S' odd, Q_0 = W), and
  // P_m, m <= H, unpacked from
  // the pair spectra and deconvolved as in the register solver.  (Bin 0's rows
  // are not the solve's: it goes through as bin 1.)
  auto unpack = [&](auto zt) {
    const auto* z = (const decltype(zt)*)zc;
    for (int pair = wr; pair < P; pair += 16) {
      const int64_t k = kb + wb > 0 ? kb + wb : 1;
      const auto z0 = z[(((int64_t)cw * P + pair) * 2 + 0) * nf + k];
      const auto z1 = z[(((int64_t)cw * P + pair) * 2 + 1) * nf + k - 1];
      const cplx<double> Dk = D[k];
      const double ax = 0.5 * ((double)z0.x + (double)z1.x);
      const double ay = 0.5 * ((double)z0.y - (double)z1.y);
      const double bx = 0.5 * ((double)z0.y + (double)z1.y);
      const double by = -0.5 * ((double)z0.x - (double)z1.x);
      const double ar = fma(ax, Dk.x, -(ay * Dk.y)), ai = fma(ax, Dk.y, ay * Dk.x);
      const double br = fma(bx, Dk.x, -(by * Dk.y)), bi = fma(bx, Dk.y, by * Dk.x);
      if (pair < H) {
        double* cc = s_c[wb] + HM;
        double* ss = s_s[wb] + HM;
        const int m = 2 * pair + 1;
        cc[m] = ar;
        ss[m] = ai;
        cc[m + 1] = br;
        ss[m + 1] = bi;
        if (m <= H) {
          cc[-m] = ar;
          ss[-m] = -ai;
        }
        if (m + 1 <= H) {
          cc[-m - 1] = br;
          ss[-m - 1] = -bi;
        }
      } else {
        const int m = 2 * (pair - H) + 1;
        s_pr[wb][m] = ar;
        s_pi[wb][m] = ai;
        if (m < H) {
          s_pr[wb][m + 1] = br;
          s_pi[wb][m + 1] = bi;
        }
      }
    }
  };
  if (fp64)
    unpack(cplx<double>{});
  else
    unpack(cplx<float>{});
  if (tid < kWideBins) {
    s_c[tid][HM] = mo.W;
    s_s[tid][HM] = 0.0;
    s_pr[tid][0] = 0.0;
  }
  __syncthreads();
  const int bin = tid >> 4, r = tid & 15;
  // Rows i = r + 16 q of alpha (entries j <= i; those above the diagonal are
  // computed along and never read), their diagonals and beta.  Row i = 2h - 1
  // is sin h, i = 2h is cos h, and with h' of column j:
  //   sin sin 0.5 (C'(h - h') - C'(h + h')), cos cos 0.5 (C'(h - h') + C'(h + h')),
  //   sin cos 0.5 (S'(h + h') + S'(h - h')), cos sin 0.5 (S'(h + h') - S'(h - h')).
  double a[NQ][DM], diag[NQ], b[NQ];
  static_for<0, NQ>([&](auto qc) {
    constexpr int q = decltype(qc)::value;
    const int i = r + 16 * q;
    const bool pad = i >= dd;
    const int h = pad ? 0 : (i + 1) >> 1;
    const bool si = i & 1;
    const double* xs = (si ? s_c[bin] : s_s[bin]) + HM + h;  // columns sin h'
    const double* xc = (si ? s_s[bin] : s_c[bin]) + HM + h;  // columns cos h'
    const double sg = si ? 0.5 : -0.5;
    diag[q] = 0.0;
    b[q] = pad ? 0.0 : (si ? s_pi[bin][h] : s_pr[bin][h]);
    static_for<0, (16 * q + 16 < DM ? 16 * q + 16 : DM)>([&](auto jc) {
      constexpr int j = decltype(jc)::value;
      constexpr int hj = (j + 1) >> 1;
      double v;
      if constexpr (j == 0)
        v = xc[0];
      else if constexpr (j % 2)
        v = sg * (xs[-hj] - xs[hj]);
      else
        v = 0.5 * (xc[-hj] + xc[hj]);
      if (pad) v = i == j ? 1.0 : 0.0;
      a[q][j] = v;
      if (i == j) diag[q] = v;
      if constexpr (j % 4 == 3) __builtin_amdgcn_sched_barrier(0);
    });
  });
  // Right-looking factorisation with the forward substitution alongside.  Rows
  // past d are those of the identity: they change nothing and need no branch.
  uint8_t fl = 0;
  double inv_own[NQ], z_own[NQ], acc = 0.0, dout = 0.0;
  static_for<0, NQ>([&](auto qc) { inv_own[decltype(qc)::value] = z_own[decltype(qc)::value] = 0.0; });
  static_for<0, DM>([&](auto jc) {
    constexpr int j = decltype(jc)::value;
    constexpr int qj = j / 16;
    const double piv = row_bcast<j % 16>(a[qj][j]);
    const double ajj = row_bcast<j % 16>(diag[qj]);
    const bool ok = piv > eps * ajj && piv > 0.0;
    double inv = rsqrt(piv);
    asm("" : "+v"(inv));  // no branch around it
    inv = ok ? inv : 0.0;
    if (!ok && j < dd) fl |= BF_PIVOT;
    const double zj = row_bcast<j % 16>(b[qj]) * inv;
    double l[NQ];
    static_for<qj, NQ>([&](auto qc) {
      constexpr int q = decltype(qc)::value;
      const int i = r + 16 * q;
      l[q] = i > j ? a[q][j] * inv : (i == j ? piv * inv : 0.0);
      if constexpr (COEF) a[q][j] = l[q];
      if (i > j) b[q] = fma(-l[q], zj, b[q]);
    });
    if constexpr (COEF) {
      if (r == j % 16) {
        inv_own[qj] = inv;
        z_own[qj] = zj;
      }
      // one register each, not every step's value kept to the end
      asm("" : "+v"(inv_own[qj]), "+v"(z_own[qj]));
    }
    acc = fma(zj, zj, acc);
    if constexpr (j >= 2 && j % 2 == 0)
      if (r == j / 2 - 1) dout = acc;
    static_for<j + 1, DM>([&](auto kc) {
      constexpr int k = decltype(kc)::value;
      const double lkj = row_bcast<k % 16>(l[k / 16]);
      static_for<k / 16, NQ>([&](auto qc) {
        constexpr int q = decltype(qc)::value;
        a[q][k] = fma(-l[q], lkj, a[q][k]);
      });
      if constexpr (k % 4 == 3) __builtin_amdgcn_sched_barrier(0);
    });
    __builtin_amdgcn_sched_barrier(0);
  });
  __syncthreads();  // the spectra have been read: the results take their place
  if (r < H) s_pr[bin][r] = dout;
  const int64_t kg = kb + bin;
  if (r == 0) {
    if (mo.span > 0.0 && (double)kg * g.df * mo.span < 1.0) fl |= BF_LOW_F;
    if (kg == 0) fl = (uint8_t)((fl & ~BF_PIVOT) | BF_DC);
    s_pi[bin][0] = (double)fl;
  }
  if constexpr (COEF) {
    // L^T A = z: A_j = (z_j - sum_{l > j} L_lj A_l) / L_jj, row l holds L_lj;
    // the sum over 64 row slots by a butterfly (32, 16, ..., 1).
#pragma clang fp contract(off)
    double A[NQ];
    static_for<0, NQ>([&](auto qc) { A[decltype(qc)::value] = 0.0; });
    static_for<0, DM>([&](auto jc) {
      constexpr int j = DM - 1 - decltype(jc)::value;
      double p[4] = {0.0, 0.0, 0.0, 0.0};
      static_for<j / 16, NQ>([&](auto qc) {
        constexpr int q = decltype(qc)::value;
        p[q] = r + 16 * q > j ? a[q][j] * A[q] : 0.0;
      });
      double sum = (p[0] + p[2]) + (p[1] + p[3]);
      sum += row_move<0x128>(sum);  // lane ^ 8 (row_ror 8)
      sum += row_move<0x124>(sum);  // lane ^ 4 (row_ror 4: lanes l and l ^ 8 are equal)
      sum += row_move<0x4E>(sum);   // lane ^ 2 (quad_perm)
      sum += row_move<0xB1>(sum);   // lane ^ 1
      if (r == j % 16) A[j / 16] = (z_own[j / 16] - sum) * inv_own[j / 16];
      __builtin_amdgcn_sched_barrier(0);
    });
    static_for<0, NQ>([&](auto qc) {
      constexpr int q = decltype(qc)::value;
      const int i = r + 16 * q;
      double v = A[q];
      if (i == 0) v = v + mo.xbar;
      if (kg == 0) v = i == 0 ? mo.xbar : 0.0;
      if (i < dd) s_c[bin][i] = v;
    });
  }
  __syncthreads();
  if (wr < H) store(out, o + wr * nf, kb + wb == 0 ? 0.0 : s_pr[wb][wr]);
  if (of && tid < kWideBins) of[tid] = (uint8_t)s_pi[tid][0];
  if constexpr (COEF)
    for (int j = wr; j < dd; j += 16) store(coef, oc + j * nf, s_c[wb][j]);
}

}  // namespace

hipError_t launch_solve_wide(bool fp64, const void* zc, const void* D, const Moments* mom,
                             const Geom& g, int curve0, int n_curves, double eps, void* out,
                             uint8_t* flags, void* coef, hipStream_t st) {
  if (g.H > kHWide || g.band || g.n_freq % kWideBins) return hipErrorInvalidValue;
  dim3 gr((unsigned)(g.n_freq / kWideBins), (unsigned)n_curves);
  auto launch = [&](auto rows, auto cf) {
    constexpr int DM = decltype(rows)::value;
    constexpr bool CF = decltype(cf)::value;
    hipLaunchKernelGGL((k_solve_wide<CF, DM>), gr, dim3(kNT), 0, st, zc,
                       (const cplx<double>*)D, mom, g, curve0, eps, fp64, out, flags, coef);
  };
  auto by_coef = [&](auto rows) {
    if (coef)
      launch(rows, std::true_type{});
    else
      launch(rows, std::false_type{});
  };
  // Rows unrolled in steps of two harmonics.
  if (g.H <= 10)
    by_coef(std::integral_constant<int, 21>{});
  else if (g.H <= 12)
    by_coef(std::integral_constant<int, 25>{});
  else if (g.H <= 14)
    by_coef(std::integral_constant<int, 29>{});
  else
    by_coef(std::integral_constant<int, 33>{});
  return hipGetLastError();
}

}  // namespace fchi2
