// Far field of the profile pass.  Away from a line its profile is smooth on
// the scale of a grid tile, so tiles at least one tile's width away take it
// through its values at P Chebyshev nodes of the tile instead of at each of
// the tile's points; tiles double in size with distance (far_geometry.h), so
// a window of 5000 points costs a line 20 to 26 tile visits of P nodes, plus the
// leaves next to its centre, which k_near takes point by point.  The
// interpolation error is below 3.4e-14 of the line's value for P = 20 (FP64
// form) and 2.2e-8 for P = 12 (FP32 form), reached for an undamped 1/x^2 tail
// on the nearest admissible tile (the Bernstein ellipse of a tile three
// half-widths from a pole has rho = 3 + sqrt(8)).
//
// What bounds a pass is the number of profile evaluations; measured on the
// whole call, point by point and with expansions: 1e7 lines, 2e6 points, window
// 5000 points, FP32 form 14.65 and 2.70 ms (near leaves 1.3, tiles 0.32, window
// ends and sigma 0.18); 1e6 lines, FP64 form 3.33 and 1.10 ms; 48 conditions of
// 1e6 lines, 2e5 points, FP32 form 113.2 and 7.1 ms.
//
// k_far_leaves, k_far_moments, k_far_cells: the tiles whose lines' moments serve
//   (below); k_far: the others, and short lists.
// k_far: one wave (up to four for wider tiles, then slices of their lines)
//   takes 64 lines at a time, one per lane, evaluates each at the tile's nodes
//   into P registers of the lane, and adds the lanes once at the end, so a
//   visit costs neither LDS traffic nor cross-lane sums per line.  The sums
//   become Chebyshev coefficients (one row of P per tile and slice).
// k_far_finish: the lines whose windows end inside a tile, then
//   sigma_k += sum over the levels of the expansion of k's tile.
#include <algorithm>

#include "far_tables.h"
#include "k_voigt.h"

namespace xs {

struct FarArgs {
  ModelDev m;
  const CondDev* cond;
  const double* sb;
  const int32_t* off;
  const double* rnu;
  const float* rgref;
  const float* rnexp;
  const double* rgpre;
  const void* rS;
  const int32_t* rkc;
  const float* rdel;
  const int32_t* rwin;
  int64_t max_lines;
  const int32_t* counter;
  double* rows;       // [conditions of the launch][cond_rows][P]
  int64_t cond_rows;  // rows per condition
  double* sigma;
  double* mom;        // [conditions of the launch][mom_cells][PM] moments, or null
  int64_t mom_cells;  // cells of all levels, those beyond the grid with them
  int32_t c0;         // first condition of the launch
  int32_t blocks;     // of k_far's levels
};

// The nodes' rational functions N/D, four over one reciprocal:
// acc[q] += N(x_q) / D(x_q).
template <int P, typename F>
__device__ __forceinline__ void far_rational(double xc, double ah, double (&acc)[P], F nd) {
#pragma unroll
  for (int q = 0; q < P; q += 4) {
    double N[4], D[4];
#pragma unroll
    for (int h = 0; h < 4; ++h) nd(fma(FarNodes<P>::x[q + h], ah, xc), N[h], D[h]);
    const double p01 = D[0] * D[1], p23 = D[2] * D[3];
    const double r = rcp64(p01 * p23);
    const double r01 = p23 * r, r23 = p01 * r;
    acc[q] = fma(N[0], D[1] * r01, acc[q]);
    acc[q + 1] = fma(N[1], D[0] * r01, acc[q + 1]);
    acc[q + 2] = fma(N[2], D[3] * r23, acc[q + 2]);
    acc[q + 3] = fma(N[3], D[2] * r23, acc[q + 3]);
  }
}

// Bin means of NP node pairs (or the Lorentzian, NP = 0) at a tile's nodes.
// The tile is at least 64 bins away, so each arctangent's argument is below
// h / |x| <= 1/64 and its odd series holds (four terms; two where the wave's
// largest argument allows: the same bounds as the gather's rows).
template <int PROF, int NP, int P, typename R>
__device__ __forceinline__ void far_bins(R xc, R ah, R h, R y, R c0, bool two, R (&acc)[P]) {
  const R hh = (R)0.5 * h, y2 = y * y, yh = y * h;
  if constexpr (NP == 0) {
    const R cl = fma(-hh, hh, (R)1);
#pragma unroll
    for (int q = 0; q < P; ++q) {
      const R x = fma((R)FarNodes<P>::x[q], ah, xc);
      acc[q] = fma(c0, atan_series<R>(h * rcp_r<R>(fma(x, x, cl))), acc[q]);
    }
  } else {
    if (two) {
#pragma unroll
      for (int q = 0; q < P; ++q)
        acc[q] = fma(c0, vpairs_bin_two<NP, R>(fma((R)FarNodes<P>::x[q], ah, xc), hh, yh, y2), acc[q]);
    } else {
#pragma unroll
      for (int q = 0; q < P; ++q) {
        const R x = fma((R)FarNodes<P>::x[q], ah, xc);
        acc[q] = fma(c0, vpairs_bin<NP, true, R>(x - hh, x + hh, yh, y2), acc[q]);
      }
    }
  }
}

// One line at the nodes of one tile: xc = x at the tile's centre, ah = half
// its width in x, so node q is at x = xc + x_q ah.  rho: the smallest |z|^2 on
// the tile; the choice of rule is the wave's.
template <int PROF, int P>
__device__ __forceinline__ void far_line_f32(float xc, float ah, float a, float y, float c0, bool live,
                                             float (&acc)[P]) {
  if constexpr (PROF == XS_LORENTZ) {
#pragma unroll
    for (int q = 0; q < P; ++q) {
      const float x = fmaf((float)FarNodes<P>::x[q], ah, xc);
      acc[q] = fmaf(c0, rcp32(fmaf(x, x, 1.0f)), acc[q]);
    }
  } else if constexpr (PROF == XS_BIN_LORENTZ) {
    far_bins<PROF, 0, P, float>(xc, ah, a, y, c0, false, acc);
  } else {
    const float xn = fabsf(xc) - ah, rho = fmaf(xn, xn, y * y);
    if (__ballot(live && !(fabsf(xc) + ah <= 1.0e9f && y <= 1.0e9f))) {
      // |x| or y beyond FP32's safe range: the FP64 evaluator
#pragma unroll 1
      for (int q = 0; q < P; ++q) {
        const double x = fma(FarNodes<P>::x[q], (double)ah, (double)xc);
        double v;
        if constexpr (PROF == XS_VOIGT) v = re_w_f64(x, (double)y);
        else v = voigt_bin_f64(x, (double)y, 0.5 * (double)a);
        const float t = live ? (float)((double)c0 * v) : 0.0f;
#pragma unroll
        for (int k = 0; k < P; ++k) acc[k] += k == q ? t : 0.0f;
      }
      return;
    }
    const bool one = __ballot(live && !(rho >= 1601.6f)) == 0;
    if constexpr (PROF == XS_BIN_VOIGT) {
      const bool two = __ballot(live && !(y * a <= 0.01f * rho)) == 0;
      if (one) far_bins<PROF, 1, P, float>(xc, ah, a, y, c0, two, acc);
      else far_bins<PROF, 2, P, float>(xc, ah, a, y, c0, two, acc);
    } else {
      const float y2 = y * y, k = c0 * (float)(2.0 / kPI) * y;
      auto term = [&](double tau, double W, float x) {
        const float s = fmaf(x, x, y2 - (float)tau), cw = k * (float)W;
        return fmaf(cw, s, cw * (float)(2.0 * tau)) * rcp32(fmaf(s, s, 4.0f * y2 * (float)tau));
      };
      if (one) {
        const float h = y2 - (float)GH::t2[0], cw = k * (float)GH::w2[0], cwt = cw * (float)(2.0 * GH::t2[0]);
        const float c = 4.0f * y2 * (float)GH::t2[0];
#pragma unroll
        for (int q = 0; q < P; ++q) {
          const float x = fmaf((float)FarNodes<P>::x[q], ah, xc), s = fmaf(x, x, h);
          acc[q] = fmaf(fmaf(cw, s, cwt), rcp32(fmaf(s, s, c)), acc[q]);
        }
      } else {
#pragma unroll
        for (int q = 0; q < P; ++q) {
          const float x = fmaf((float)FarNodes<P>::x[q], ah, xc);
          acc[q] += term(GH::t4[0], GH::w4[0], x) + term(GH::t4[1], GH::w4[1], x);
        }
      }
    }
  }
}

template <int PROF, int P>
__device__ __forceinline__ void far_line_f64(double xc, double ah, double a, double y, double c0, bool live,
                                             double (&acc)[P]) {
  if constexpr (PROF == XS_LORENTZ) {
    // the product of four denominators stays finite for |x| <= 1e35
    if (__ballot(live && !(fabs(xc) + ah <= 1.0e35))) {
#pragma unroll 1
      for (int q = 0; q < P; ++q) {
        const double x = fma(FarNodes<P>::x[q], ah, xc);
        const double t = live ? c0 * rcp64(fma(x, x, 1.0)) : 0.0;
#pragma unroll
        for (int k = 0; k < P; ++k) acc[k] += k == q ? t : 0.0;
      }
      return;
    }
    far_rational<P>(xc, ah, acc, [&](double x, double& N, double& D) {
      N = c0;
      D = fma(x, x, 1.0);
    });
  } else if constexpr (PROF == XS_BIN_LORENTZ) {
    far_bins<PROF, 0, P, double>(xc, ah, a, y, c0, false, acc);
  } else {
    const double xn = fabs(xc) - ah, y2 = y * y, rho = fma(xn, xn, y2);
    if (__ballot(live && !(fabs(xc) + ah <= 1.0e9 && y <= 1.0e9))) {
#pragma unroll 1
      for (int q = 0; q < P; ++q) {
        const double x = fma(FarNodes<P>::x[q], ah, xc);
        double v;
        if constexpr (PROF == XS_VOIGT) v = re_w_f64(x, y);
        else v = voigt_bin_f64(x, y, 0.5 * a);
        const double t = live ? c0 * v : 0.0;
#pragma unroll
        for (int k = 0; k < P; ++k) acc[k] += k == q ? t : 0.0;
      }
      return;
    }
    auto all = [&](double bound) { return __ballot(live && !(rho >= bound)) == 0; };
    if constexpr (PROF == XS_BIN_VOIGT) {
      const bool two = __ballot(live && !(y * a <= 1.25e-4 * rho)) == 0;
      if (all(9.0e6 * 1.001)) far_bins<PROF, 1, P, double>(xc, ah, a, y, c0, two, acc);
      else if (all(6400.0 * 1.001)) far_bins<PROF, 2, P, double>(xc, ah, a, y, c0, two, acc);
      else if (all(400.0 * 1.001)) far_bins<PROF, 3, P, double>(xc, ah, a, y, c0, two, acc);
      else if (all(144.0 * 1.001)) far_bins<PROF, 4, P, double>(xc, ah, a, y, c0, two, acc);
      else far_bins<PROF, 6, P, double>(xc, ah, a, y, c0, two, acc);
    } else {
      if (all(9.0e6 * 1.001)) {
        const Pair<double> A = make_pair<double>(c0, y, GH::t2[0], GH::w2[0]);
        far_rational<P>(xc, ah, acc, [&](double x, double& N, double& D) {
          const double s = fma(x, x, A.h);
          N = fma(A.cw, s, A.cwt);
          D = fma(s, s, A.c);
        });
      } else if (all(4.5e4 * 1.001)) {
        const Poly3 C = make_poly3(c0, y);
        far_rational<P>(xc, ah, acc, [&](double x, double& N, double& D) { poly3_nd(C, x, N, D); });
      } else if (all(4000.0 * 1.001)) {
        const Poly2 B = make_poly2(c0, y);
        far_rational<P>(xc, ah, acc, [&](double x, double& N, double& D) { poly2_nd(B, x, N, D); });
      } else {
        const double k = c0 * (y * (2.0 / kPI)), y4 = 4.0 * y2;
        // two nodes over one reciprocal (three and four pairs: the products stay finite
        // for |x|, y <= 1e9; six: for y <= 1e6)
        auto pairs = [&](auto np) {
#pragma unroll
          for (int q = 0; q < P; q += 2) {
            const double x0 = fma(FarNodes<P>::x[q], ah, xc), x1 = fma(FarNodes<P>::x[q + 1], ah, xc);
            double N0, D0, N1, D1;
            gh_nd<decltype(np)::value>(x0 * x0, y2, y4, N0, D0);
            gh_nd<decltype(np)::value>(x1 * x1, y2, y4, N1, D1);
            const double r = k * rcp64(D0 * D1);
            acc[q] = fma(N0 * D1, r, acc[q]);
            acc[q + 1] = fma(N1 * D0, r, acc[q + 1]);
          }
        };
        if (all(400.0 * 1.001)) pairs(std::integral_constant<int, 3>());
        else if (all(144.0 * 1.001)) pairs(std::integral_constant<int, 4>());
        else if (__ballot(live && !(y <= 1.0e6)) == 0) pairs(std::integral_constant<int, 6>());
        else
          // (a far wider line in the wave: its twelve factors of up to y^4 would overflow)
#pragma unroll 1
          for (int q = 0; q < P; ++q) {
            const double x = fma(FarNodes<P>::x[q], ah, xc);
            double N, D;
            gh_nd<6>(x * x, y2, y4, N, D);
            const double t = live ? k * N * rcp64(D) : 0.0;
#pragma unroll
            for (int h = 0; h < P; ++h) acc[h] += h == q ? t : 0.0;
          }
      }
    }
  }
}

// The profile is defined at the rounded grid points fl(nu0 + k dnu); the nodes
// lie on the exact grid.  exact - rounded at point k (FP64 form: up to an ulp
// of nu_k, which moves a value at distance d by a relative 2 ulp / d).
__device__ __forceinline__ double far_grid_residue(double nu0, double dnu, int64_t k) {
#pragma clang fp contract(off)
  const double kd = (double)k, p = kd * dnu, s = nu0 + p, b = s - nu0;
  const double es = (nu0 - (s - b)) + (p - b);
  return es + __builtin_fma(kd, dnu, -p);
}

// The lane's line and its constants for the tile that begins at point ts and
// has its centre mid points further on: step a and centre xc in the profile's
// unit x, width y, factor c0.  A lane without a line (in = false, or S = 0)
// holds another line's with c0 = 0.
template <typename Real>
struct FarLine {
  Real a, xc, y, c0;
  bool live;
};
template <typename Real>
struct FarIn {
  int kc;
  Real S;
  float gr, ne, del;
  double gp, nu;
};
template <typename Real>
__device__ __forceinline__ FarIn<Real> far_load(const FarArgs& g, const CondDev& cd, uint32_t p) {
  FarIn<Real> in;
  in.kc = g.rkc[p];
  in.S = ((const Real*)g.rS)[(int64_t)cd.slot * g.max_lines + p];
  in.gr = g.rgref[p];
  in.ne = g.rnexp[p];
  in.gp = g.rgpre ? g.rgpre[p] : 0.0;
  in.nu = g.rnu[p];
  in.del = sizeof(Real) == 4 ? g.rdel[p] : 0.0f;
  return in;
}
template <typename Real, int PROF>
__device__ __forceinline__ FarLine<Real> far_line(const FarArgs& g, const CondDev& cd, const FarIn<Real>& v, bool in,
                                                  int ts, Real mid) {
  const ModelDev& m = g.m;
  const int kc = v.kc;
  const Real S = v.S;
  const float gr = v.gr, ne = v.ne;
  const double gp = v.gp, nu = v.nu;
  FarLine<Real> L;
  L.live = in && S != (Real)0;
  L.y = 0;
  Real inv, del;
  if constexpr (sizeof(Real) == 4) {
    del = v.del;
    const float gamma = fmaf(gr * __builtin_amdgcn_exp2f(ne * (float)(cd.lnTr / kLN2)), (float)cd.pfac, (float)gp);
    if constexpr (PROF == XS_LORENTZ || PROF == XS_BIN_LORENTZ) {
      inv = rcp32(gamma);
      L.c0 = PROF == XS_LORENTZ ? S * (float)(1.0 / kPI) * inv : S * (float)(1.0 / (kPI * m.dnu));
    } else {
      inv = (float)0.83255461115769776 * rcp32((float)nu * (float)cd.dop);  // sqrt(ln2)/alpha
      L.y = gamma * inv;
      // 1/(sg sqrt(2 pi)); bin means: 1/(sqrt(pi) dnu)
      L.c0 = PROF == XS_VOIGT ? S * (float)0.56418958354775628 * inv : S * (float)(0.56418958354775628 / m.dnu);
    }
  } else {
    // from the exact grid point of the home bin
    del = (nu - nu_of_bin(m.nu0, m.dnu, kc)) - far_grid_residue(m.nu0, m.dnu, kc);
    const double gamma = (double)gr * exp((double)ne * cd.lnTr) * cd.pfac + gp;
    if constexpr (PROF == XS_LORENTZ || PROF == XS_BIN_LORENTZ) {
      inv = 1.0 / gamma;
      L.c0 = PROF == XS_LORENTZ ? S * inv * (1.0 / kPI) : S * (1.0 / (kPI * m.dnu));
    } else {
      inv = sqrt(kLN2) * rcp64(nu * cd.dop);
      L.y = gamma * inv;
      L.c0 = PROF == XS_VOIGT ? S * inv * (1.0 / sqrt(kPI)) : S * (1.0 / (sqrt(kPI) * m.dnu));
    }
  }
  if (!L.live) {  // (no width makes a Lorentzian's x infinite)
    L.c0 = 0;
    L.y = 0;
    if constexpr (PROF == XS_LORENTZ || PROF == XS_BIN_LORENTZ) inv = 1;
  }
  L.a = (Real)m.dnu * inv;
  L.xc = fma((Real)(ts - kc) + mid, L.a, -(del * inv));
  return L;
}

// The lane's value moved by a data-parallel-primitive control word (within its
// row of 16 lanes; 0 where no lane of the row is the source).
template <int CTRL>
__device__ __forceinline__ double far_dpp(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xf, 0xf, true);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
constexpr int kDppXor1 = 0xb1, kDppXor2 = 0x4e, kDppHalfMirror = 0x141, kDppMirror = 0x140;
constexpr int kDppShl = 0x100, kDppShr = 0x110;  // + n: from n lanes further on, further back

// Sum of v[0..P) over the wave's lanes: halves of the values are exchanged at
// the first two steps (35 adds for P = 20 instead of 120), the rows of 16
// lanes add up without the LDS.  Afterwards the lane holds P / 4 sums, those
// of the values far_slot(lane) + i.
template <int P>
__device__ __forceinline__ void far_fold(double (&v)[P], int lane) {
  static_assert(P % 4 == 0, "folded in quarters");
  const bool u1 = lane & 32, u2 = lane & 16;
#pragma unroll
  for (int i = 0; i < P / 2; ++i) {
    const double send = u1 ? v[i] : v[P / 2 + i], keep = u1 ? v[P / 2 + i] : v[i];
    v[i] = keep + __shfl_xor(send, 32, 64);
  }
#pragma unroll
  for (int i = 0; i < P / 4; ++i) {
    const double send = u2 ? v[i] : v[P / 4 + i], keep = u2 ? v[P / 4 + i] : v[i];
    v[i] = keep + __shfl_xor(send, 16, 64);
  }
#pragma unroll
  for (int i = 0; i < P / 4; ++i) {
    v[i] += far_dpp<kDppXor1>(v[i]);
    v[i] += far_dpp<kDppXor2>(v[i]);
    v[i] += far_dpp<kDppHalfMirror>(v[i]);
    v[i] += far_dpp<kDppMirror>(v[i]);
  }
}
template <int P>
__device__ __forceinline__ int far_slot(int lane) {
  return ((lane >> 5) & 1) * (P / 2) + ((lane >> 4) & 1) * (P / 4);
}

// ---------------------------------------------------------------------------
// Moments.  A Voigt profile in the far field is a Gaussian average of poles,
//   S / pi Im E[1 / (nu - nu0 - i gamma - sigma t)],  t normal,
// so about the centre c of a cell of lines its values are
//   sum_n M_n / (nu - c)^(n+1),  M_n = S / pi Im E[(nu0 - c + i gamma + sigma t)^n],
// and the M_n of all the cell's lines add up: a tile takes a cell, not each of its
// lines, at PM operations a node.  The averages obey u_(n+1) = s u_n + n sigma^2
// u_(n-1), s = nu0 - c + i gamma.  A wider cell's moments are those of its halves
// moved to its centre (binomially), so a line is entered once, in its leaf,
// instead of in the 20 tiles of its window.  Bin means average over the bin as
// well, which is done to the moments of the leaf.
//
// With gamma <= half a cell a line lies within 0.71 cells of c and the nodes 1.5
// away or more (of a narrower cell: within half the distance): the series ends
// at 0.5^PM, 4e-9 for PM = 28 (FP32 form) and 4e-15 for 48.  The Gaussian's
// part lies within 4.5 sigma at these orders, the nodes beyond 11 sigma.  Levels
// whose cells are too small for the widest line (far_mom_level) or for the widest
// Gaussian's powers (far_sigma_level) take lines one by one.
//
// The tiles of 1e7 lines FP32 (2e6 points) took 1.08 ms line by line, 0.32 by moments
// (leaves 0.18, wider cells 0.04, tiles 0.10), 1e6 lines FP64 0.60 and 0.22, 48
// conditions x 1e6 lines (of which 16 have lines too wide for most levels) 5.8
// and 3.7.  The leaves are bound by the recurrence, seven operations a moment
// (VALU issue at its peak rate in the FP32 form, 0.8 of it in FP64).
// ---------------------------------------------------------------------------
constexpr int kMoments32 = 28, kMoments64 = 48, kMomentsMax = 48;
constexpr int kMomLeaves = 64, kMomLevels = 6;  // cells of a block of k_far_moments, levels it builds from them

struct BinomTable {
  double c[kMomentsMax + 1][kMomentsMax + 1];
  constexpr BinomTable() : c() {
    for (int n = 0; n <= kMomentsMax; ++n) {
      c[n][0] = 1.0;
      for (int k = 1; k <= n; ++k) c[n][k] = c[n - 1][k - 1] + (k < n ? c[n - 1][k] : 0.0);
    }
  }
};
static __device__ const BinomTable kBinom = BinomTable();

// the lowest level of the condition that uses moments
__device__ __forceinline__ int far_cond_mom_level(const FarArgs& g, const CondDev& cd) {
  const float* e = (const float*)g.counter;
  const double n = fmax((double)e[kNexpMin] * cd.lnTr, (double)e[kNexpMax] * cd.lnTr);
  return max(cd.far.mom, far_mom_level(cd.far.sh, (double)e[kGammaMax] * exp(n) * cd.pfac * 1.00001 / g.m.dnu));
}

// Moments of the leaves, a wave to a leaf and a line to a lane.
template <typename Real, int PROF, int PM>
__global__ __launch_bounds__(256, sizeof(Real) == 4 ? 4 : 2) void k_far_leaves(FarArgs g) {
  constexpr bool F32 = sizeof(Real) == 4, LOR = PROF == XS_LORENTZ || PROF == XS_BIN_LORENTZ;
  constexpr bool BIN = PROF == XS_BIN_LORENTZ || PROF == XS_BIN_VOIGT;
  __shared__ double ma[4 * PM];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const CondDev& cd = g.cond[g.c0 + blockIdx.y];
  const FarCond& fc = cd.far;
  if (!fc.on || g.counter[kFarOff]) return;
  const int lm = far_cond_mom_level(g, cd);
  if (lm > fc.lmax) return;
  const ModelDev& m = g.m;
  const int nk = fine_keys(m), key = long_block() * 4 + wave, f = key - m.fine_v;
  if (key >= nk) return;
  // in cells of the first level that uses them, so that the powers stay small
  const double hp = (double)(1 << (fc.sh + lm)), ih = 1.0 / hp;
  // (the outermost cells' lines go point by point)
  const bool any = key > 0 && key < nk - 1;
  const uint32_t p0 = any ? g.off[f] : 0, p1 = any ? g.off[f + 1] : 0;
  double acc64[PM];
  Real acc[PM];
#pragma unroll
  for (int k = 0; k < PM; ++k) {
    acc[k] = (Real)0;
    if (F32) acc64[k] = 0.0;
  }
  const double centre = (double)(far_shl(f, fc.sh) + (1 << fc.sh) / 2) - 0.5;
  int since = 0;
  for (uint32_t q0 = p0; q0 < p1; q0 += 64) {
    const FarIn<Real> v = far_load<Real>(g, cd, min(q0 + lane, p1 - 1));
    const Real S = q0 + lane < p1 ? v.S : (Real)0;
    Real sr, si, sg2 = 0;
    if constexpr (F32) {
      const float gamma = fmaf(v.gr * __builtin_amdgcn_exp2f(v.ne * (float)(cd.lnTr / kLN2)), (float)cd.pfac, (float)v.gp);
      const float pt = (float)(ih / m.dnu);
      sr = fmaf(v.del, pt, (float)((v.kc - centre) * ih));
      si = gamma * pt;
      if constexpr (!LOR) {
        const float sg = (float)v.nu * ((float)cd.dop * (float)0.84932180028801907 * pt);  // alpha / sqrt(2 ln 2)
        sg2 = sg * sg;
      }
    } else {
      const double del = (v.nu - nu_of_bin(m.nu0, m.dnu, v.kc)) - far_grid_residue(m.nu0, m.dnu, v.kc);
      const double gamma = (double)v.gr * exp((double)v.ne * cd.lnTr) * cd.pfac + v.gp;
      const double pt = ih / m.dnu;
      sr = fma(del, pt, (v.kc - centre) * ih);
      si = gamma * pt;
      if constexpr (!LOR) {
        const double sg = v.nu * (cd.dop * 0.84932180028801907 * pt);
        sg2 = sg * sg;
      }
    }
    Real pr = 1, pi = 0, ur = sr, ui = si;  // u_(n-1), u_n
#pragma unroll
    for (int n = 1; n <= PM; ++n) {
      acc[n - 1] = fma(S, ui, acc[n - 1]);
      if (n < PM) {
        Real nr, ni;
        if constexpr (LOR) {
          nr = fma(sr, ur, -si * ui);
          ni = fma(sr, ui, si * ur);
        } else {
          const Real e = (Real)n * sg2;
          nr = fma(sr, ur, fma(-si, ui, e * pr));
          ni = fma(sr, ui, fma(si, ur, e * pi));
        }
        pr = ur;
        pi = ui;
        ur = nr;
        ui = ni;
      }
    }
    if constexpr (F32) {
      if (++since == 32) {
        since = 0;
#pragma unroll
        for (int k = 0; k < PM; ++k) {
          acc64[k] += (double)acc[k];
          acc[k] = (Real)0;
        }
      }
    }
  }
#pragma unroll
  for (int k = 0; k < PM; ++k) acc64[k] = F32 ? acc64[k] + (double)acc[k] : (double)acc[k];
  far_fold<PM>(acc64, lane);
  double* row = ma + wave * PM;
  if ((lane & 15) == 0) {
    const double f0 = ih / (kPI * m.dnu);
    const int s0 = far_slot<PM>(lane);
#pragma unroll
    for (int i = 0; i < PM / 4; ++i) row[s0 + i] = acc64[i] * f0;
  }
  if constexpr (BIN) {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    // E[(s + b t)^n], t uniform: sum over k of C(n, 2k) b^(2k) / (2k + 1) M_(n-2k); b <= 1/32
    const int n = lane + 1;
    double v = 0.0, e = 1.0;
    const double b2 = 0.25 * ih * ih;
    if (n <= PM)
      for (int k = 0; 2 * k < n && k <= 8; ++k) {
        v = fma(kBinom.c[n][2 * k] * e / (double)(2 * k + 1), row[n - 2 * k - 1], v);
        e *= b2;
      }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (n <= PM) row[n - 1] = v;
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  if (lane < PM) g.mom[((int64_t)blockIdx.y * g.mom_cells + key) * PM + lane] = row[lane];
}

// Moments of the kMomLevels levels above level `base`: a block has kMomLeaves of
// its cells, a thread a moment of a wider cell.
template <int PM>
__global__ __launch_bounds__(256) void k_far_moments(FarArgs g, int base) {
  __shared__ double ma[kMomLeaves * PM], mb[kMomLeaves / 2 * PM];
  __shared__ double wt[PM][PM];  // [k - 1][n - 1]: what M_k of a half gives to M_n
  const int tid = threadIdx.x;
  const CondDev& cd = g.cond[g.c0 + blockIdx.y];
  const FarCond& fc = cd.far;
  if (!fc.on || g.counter[kFarOff] || base >= fc.lmax) return;
  const int lm = far_cond_mom_level(g, cd);
  if (lm > fc.lmax) return;
  const int nf = fine_keys(g.m), i0 = blockIdx.x * kMomLeaves;  // cells from the first beyond the grid on
  double* const rows = g.mom + (int64_t)blockIdx.y * g.mom_cells * PM;
  const int nc = min(kMomLeaves, far_tiles(nf, base) - i0);
  const double* from = rows + (far_cells_before(nf, base) + i0) * PM;
  for (int i = tid; i < kMomLeaves * PM; i += 256) ma[i] = i < nc * PM ? from[i] : 0.0;
  __syncthreads();
  for (int l = base; l < min(base + kMomLevels, fc.lmax); ++l) {
    const double* src = (l - base) & 1 ? mb : ma;
    double* dst = (l - base) & 1 ? ma : mb;
    const int np = kMomLeaves / 2 >> (l - base);
    // halves half a half's width from the centre, d = 2^-ed of the parent's
    // unit, whose unit is 2^-er of it
    const int hpar = max(l + 1, lm), ed = hpar - (l - 1), er = hpar - max(l, lm);
    if (l == base || l <= lm) {  // (from the first level that uses them on always 2 and 1)
      for (int i = tid; i < PM * PM; i += 256) {
        const int k = i / PM + 1, n = i - (k - 1) * PM + 1;
        wt[k - 1][n - 1] = n >= k ? ldexp(kBinom.c[n][k], -(ed * (n - k) + er * k)) : 0.0;
      }
      __syncthreads();
    }
    const int first = i0 >> (l + 1 - base), nt = far_tiles(nf, l + 1);
    double* out = rows + (far_cells_before(nf, l + 1) + first) * PM;
    for (int i = tid; i < np * PM; i += 256) {
      const int c = i / PM, n = i - c * PM + 1;
      const double *L = src + 2 * c * PM, *R = L + PM;
      double v = 0.0, u = 0.0;
      const int o = n & 1;
#pragma unroll 4
      for (int k = 0; k < PM; k += 2) {  // M_(k + 1), M_(k + 2)
        const double w0 = wt[k][n - 1], w1 = wt[k + 1][n - 1];
        v = fma(w0, o ? R[k] + L[k] : R[k] - L[k], v);
        u = fma(w1, o ? R[k + 1] - L[k + 1] : R[k + 1] + L[k + 1], u);
      }
      v += u;
      dst[i] = v;
      if (first + c < nt) out[i] = v;
    }
    __syncthreads();
  }
}

// The tiles of the levels that take their cells through moments: P lanes to a
// tile, each one node.  A tile has three cells at the lower levels and up to a
// dozen where windows end.  (A wave to a tile spent most of its time on the ranges:
// 48 conditions x 25000 tiles 3.16 ms with the levels line by line, 2.66 so.)
template <int P, int PM>
__global__ __launch_bounds__(256) void k_far_cells(FarArgs g) {
  constexpr int G = 64 / P;
  __shared__ double sv[4][64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const CondDev& cd = g.cond[g.c0 + blockIdx.y];
  const FarCond& fc = cd.far;
  if (!fc.on || g.counter[kFarOff]) return;
  const int lm = far_cond_mom_level(g, cd), nf = g.m.n_fine;
  if (lm > fc.lmax) return;
  const int gi = lane / P, q = lane - gi * P;
  int t = (blockIdx.x * 4 + wave) * G + gi, l = lm;
  while (l <= fc.lmax && t >= far_tiles(nf, l)) t -= far_tiles(nf, l++);
  const bool live = gi < G && l <= fc.lmax;
  double v = 0.0;
  if (live) {
    CellRange r[4];
    far_tile_ranges(fc, l, t, r);
    const double half = (double)(1 << (l + fc.sh)) * 0.5;
    const double node = (double)(t << (l + fc.sh)) + (half - 0.5) + half * far_x<double, P>()[q];
    const double* const rows = g.mom + (int64_t)blockIdx.y * g.mom_cells * PM;
    for (int left = 4; left > 0;) {
      if (r[0].lo > r[0].hi) {
        r[0] = r[1];
        r[1] = r[2];
        r[2] = r[3];
        --left;
        continue;
      }
      const int lv = far_widest(r[0].lo, r[0].hi, l), cell = r[0].lo >> lv;
      r[0].lo += 1 << lv;
      const double2* mo = (const double2*)(rows + (far_cells_before(fine_keys(g.m), lv) + cell + (g.m.fine_v >> lv)) * PM);
      const double w = (double)(1 << (lv + fc.sh));
      const double c = (double)cell * w + (w * 0.5 - 0.5);
      const double inv = (double)(1 << (max(lv, lm) + fc.sh)) / (node - c);
      double h = 0.0;
#pragma unroll
      for (int k = PM / 2 - 1; k >= 0; --k) {
        const double2 a = mo[k];
        h = fma(fma(h, inv, a.y), inv, a.x);
      }
      // (in cells' widths; the row holds the factor of the first level's)
      v = fma(h * inv, ldexp(inv, -(max(lv, lm) - lm)), v);
    }
  }
  sv[wave][lane] = v;
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  if (live) {
    const double* D = far_dct<P>();
    double o = 0.0;
#pragma unroll
    for (int i = 0; i < P; ++i) o = fma(D[i * P + q], sv[wave][gi * P + i], o);
    const int64_t row = far_rows_before(nf, fc.sh, l) + (int64_t)t * far_slices(fc.sh, l);
    g.rows[((int64_t)blockIdx.y * g.cond_rows + row) * P + q] = o;
  }
}

template <typename Real, int PROF, int P>
__global__ __launch_bounds__(256, sizeof(Real) == 4 ? 4 : 3) void k_far(FarArgs g) {
  constexpr bool F32 = sizeof(Real) == 4;
  __shared__ double sv[4][P], st[4][P];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c = g.c0 + blockIdx.y;
  const CondDev& cd = g.cond[c];
  const FarCond& fc = cd.far;
  if (!fc.on || g.counter[kFarOff]) return;
  const ModelDev& m = g.m;
  const int nf = m.n_fine;
  const int ltop = min(fc.lmax, (g.mom ? far_cond_mom_level(g, cd) : kFarLevels) - 1);
  for (int item = blockIdx.x; item < g.blocks; item += gridDim.x) {
    // the block's level: the widest tiles, which have the most lines, first (above
    // them k_far_cells)
    int b = item, l = ltop;
    for (; l >= 0; --l) {
      const int nb = far_blocks(nf, fc.sh, l);
      if (b < nb) break;
      b -= nb;
    }
    if (l < 0) return;
    const int lw = min(far_wide(fc.sh, l), 2), nw = 1 << lw, sl = far_slices(fc.sh, l);
    const int t = lw < 2 ? (b << (2 - lw)) + (wave >> lw) : b / sl;
    const int slice = lw < 2 ? 0 : b % sl;
    // positions of the tile's lines: up to four ranges of sorted lines
    CellRange r[4];
    far_tile_ranges(fc, l, t, r);
    uint32_t cum[4], beg[4], total = 0;
    const bool live_tile = t < far_tiles(nf, l);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const bool ok = live_tile && r[k].lo <= r[k].hi;
      const uint32_t p0 = ok ? g.off[r[k].lo] : 0, p1 = ok ? g.off[r[k].hi + 1] : 0;
      beg[k] = p0 - total;  // position q of the tile is line q + beg of its range
      total += p1 - p0;
      cum[k] = total;
    }
    double acc64[P];
    Real acc[P];
#pragma unroll
    for (int q = 0; q < P; ++q) {
      acc[q] = (Real)0;
      if (F32) acc64[q] = 0.0;
    }
    const int ts = t << (l + fc.sh);  // the tile's first point
    const Real half = (Real)(1 << (l + fc.sh)) * (Real)0.5, mid = half - (Real)0.5;
    const uint32_t stride = (uint32_t)(nw * sl) * 64u;
    int since = 0;
    auto at = [&](uint32_t q0) {
      const uint32_t q = min(q0 + lane, total - 1);
      return q + (q < cum[0] ? beg[0] : q < cum[1] ? beg[1] : q < cum[2] ? beg[2] : beg[3]);
    };
    uint32_t q0 = (uint32_t)((wave & (nw - 1)) + slice * nw) * 64u;
    FarIn<Real> next;
    if (q0 < total) next = far_load<Real>(g, cd, at(q0));
    for (; q0 < total; q0 += stride) {
      const FarIn<Real> cur = next;
      if (q0 + stride < total) next = far_load<Real>(g, cd, at(q0 + stride));  // a batch ahead of its use
      const FarLine<Real> L = far_line<Real, PROF>(g, cd, cur, q0 + lane < total, ts, mid);
      if constexpr (F32) {
        far_line_f32<PROF, P>(L.xc, half * L.a, L.a, L.y, L.c0, L.live, acc);
        if (++since == 32) {
          since = 0;
#pragma unroll
          for (int k = 0; k < P; ++k) {
            acc64[k] += (double)acc[k];
            acc[k] = (Real)0;
          }
        }
      } else {
        far_line_f64<PROF, P>(L.xc, half * L.a, L.a, L.y, L.c0, L.live, acc);
      }
    }
    if constexpr (F32) {
#pragma unroll
      for (int k = 0; k < P; ++k) acc64[k] += (double)acc[k];
    } else {
#pragma unroll
      for (int k = 0; k < P; ++k) acc64[k] = acc[k];
    }
    far_fold<P>(acc64, lane);
    if ((lane & 15) == 0) {
      const int s0 = far_slot<P>(lane);
#pragma unroll
      for (int i = 0; i < P / 4; ++i) sv[wave][s0 + i] = acc64[i];
    }
    __syncthreads();
    // the tile's waves, then node values to coefficients
    const int tid = threadIdx.x, tiles = 4 >> lw;
    if (tid < tiles * P) {
      const int tg = tid / P, q = tid - tg * P;
      double v = 0.0;
      for (int w = 0; w < nw; ++w) v += sv[tg * nw + w][q];
      st[tg][q] = v;
    }
    __syncthreads();
    if (tid < tiles * P) {
      const int tg = tid / P, k = tid - tg * P;
      const int tt = lw < 2 ? (b << (2 - lw)) + tg : t;
      if (tt < far_tiles(nf, l)) {
        const double* D = far_dct<P>();
        double v = 0.0;
#pragma unroll
        for (int q = 0; q < P; ++q) v = fma(D[q * P + k], st[tg][q], v);
        const int64_t row = far_rows_before(nf, fc.sh, l) + (int64_t)tt * sl + slice;
        g.rows[((int64_t)blockIdx.y * g.cond_rows + row) * P + k] = v;
      }
    }
    __syncthreads();
  }
}

// The tiles that window ends cut, and sigma.  One block of four waves per tile
// of level `end` and condition.  A line whose window ends inside the tile adds
// its values at PE nodes to the LDS row of its last (first) point; the sum of
// the rows of all points from k upwards (downwards) is then, at point k, the
// nodes' values of exactly the lines that reach k, so a cut costs a line PE
// evaluations instead of one per point.  (PE = 12, FP64 form, and 6: the tile
// is at least 17 half-widths away, where these keep 1.3e-14 and 1e-8.)  One
// wave takes the upper ends and one the lower ends, each with rows of its own
// and its lanes adding in a fixed order; then every thread has a point, sums
// the rows (16 points at a time in registers, then the groups) and adds the
// expansions of the tiles of every level (Clenshaw's recurrence), and sigma is
// updated once.  (On one wave its chains of sums are exposed: 0.30 ms against 0.20 on 1e6
// lines FP64, 2e6 points; 0.79 against 0.27 on 1e7 lines FP32.)
template <int P>
__device__ __forceinline__ double far_clenshaw(const double (&co)[P], double x) {
  const double x2 = 2.0 * x;
  double b1 = 0.0, b2 = 0.0;
#pragma unroll
  for (int q = P - 1; q >= 1; --q) {
    const double b = fma(x2, b1, co[q] - b2);
    b2 = b1;
    b1 = b;
  }
  return fma(x, b1, co[0] - b2);
}

// the derivative of the same sum
template <int P>
__device__ __forceinline__ double far_clenshaw_slope(const double (&co)[P], double x) {
  // sum c_m T_m' = sum m c_m U_(m-1)
  const double x2 = 2.0 * x;
  double b1 = 0.0, b2 = 0.0;
#pragma unroll
  for (int q = P - 1; q >= 1; --q) {
    const double b = fma(x2, b1, fma((double)q, co[q], -b2));
    b2 = b1;
    b1 = b;
  }
  return b1;
}

template <typename Real, int PROF, int P, int PE>
__global__ __launch_bounds__(256) void k_far_finish(FarArgs g) {
  constexpr bool F32 = sizeof(Real) == 4;
  // FP64 rows in both forms: FP32 adds to LDS are several times slower
  __shared__ double row[2][PE * kFarEndBins];
  __shared__ double tot[2][kFarEndBins / 16][PE];
  const int tid = threadIdx.x, lane = tid & 63, c = g.c0 + blockIdx.y, t = long_block();
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const CondDev& cd = g.cond[c];
  const FarCond& fc = cd.far;
  if (!fc.on || g.counter[kFarOff]) return;
  const ModelDev& m = g.m;
  const int nf = m.n_fine, e = fc.end, n = 1 << (e + fc.sh);
  if (t >= far_tiles(nf, e)) return;
  const int ts = t * n;
  const Real half = (Real)n * (Real)0.5, mid = half - (Real)0.5;
  CellRange cut[2];
  far_cut(fc, t, cut);
  int64_t p0[2], p1[2];
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const bool any = cut[s].lo <= cut[s].hi;
    p0[s] = any ? g.off[cut[s].lo] : 0;
    p1[s] = any ? g.off[cut[s].hi + 1] : 0;
    if (p0[s] < p1[s])
      for (int i = tid; i < PE * n; i += 256) row[s][i] = 0.0;
  }
  __syncthreads();
  if (wave < 2) {
    const int side = wave;
    double* rw = row[side];
    const int64_t a0 = side == 0 ? p0[0] : p0[1], a1 = side == 0 ? p1[0] : p1[1];
    FarIn<Real> next;
    int2 nwin = {0, -1};
    auto fetch = [&](int64_t q0) {
      const int64_t p = min(q0 + lane, a1 - 1);
      nwin = ((const int2*)g.rwin)[(int64_t)cd.cclass * g.max_lines + p];
      next = far_load<Real>(g, cd, (uint32_t)p);
    };
    if (a0 < a1) fetch(a0);
    for (int64_t q0 = a0; q0 < a1; q0 += 64) {
      const FarIn<Real> cur = next;
      const int2 win = nwin;
      if (q0 + 64 < a1) fetch(q0 + 64);
      // the last (side 0) or first (side 1) point of the window in the tile
      const int j = side == 0 ? min(win.y - ts, n - 1) : max(win.x - ts, 0);
      const bool in = q0 + lane < a1 && win.x <= win.y && (side == 0 ? j >= 0 : j < n);
      const FarLine<Real> L = far_line<Real, PROF>(g, cd, cur, in, ts, mid);
      Real acc[PE];
#pragma unroll
      for (int q = 0; q < PE; ++q) acc[q] = (Real)0;
      if constexpr (F32) far_line_f32<PROF, PE>(L.xc, half * L.a, L.a, L.y, L.c0, L.live, acc);
      else far_line_f64<PROF, PE>(L.xc, half * L.a, L.a, L.y, L.c0, L.live, acc);
      if (L.live)
#pragma unroll
        for (int q = 0; q < PE; ++q) atomicAdd(&rw[q * n + j], (double)acc[q]);
    }
  }
  __syncthreads();
  const bool own = tid < n;  // whole waves: n is 64, 128 or 256
  double sum = 0.0;
#pragma unroll
  for (int side = 0; side < 2; ++side) {
    if (p0[side] >= p1[side]) continue;  // the block's
    double s[PE];
    if (own) {
#pragma unroll
      for (int q = 0; q < PE; ++q) {
        double v = row[side][q * n + tid];
        if (side == 0) {
          v += far_dpp<kDppShl + 1>(v);
          v += far_dpp<kDppShl + 2>(v);
          v += far_dpp<kDppShl + 4>(v);
          v += far_dpp<kDppShl + 8>(v);
        } else {
          v += far_dpp<kDppShr + 1>(v);
          v += far_dpp<kDppShr + 2>(v);
          v += far_dpp<kDppShr + 4>(v);
          v += far_dpp<kDppShr + 8>(v);
        }
        s[q] = v;
        if ((tid & 15) == (side == 0 ? 0 : 15)) tot[side][tid >> 4][q] = v;
      }
    }
    __syncthreads();
    if (tid < PE) {  // groups beyond (before) each group
      double run = 0.0;
      for (int h = 0; h < n / 16; ++h) {
        const int gr = side == 0 ? n / 16 - 1 - h : h;
        const double v = tot[side][gr][tid];
        tot[side][gr][tid] = run;
        run += v;
      }
    }
    __syncthreads();
    if (own) {
      const double* D = far_dct<PE>();
      double co[PE];
#pragma unroll
      for (int k = 0; k < PE; ++k) co[k] = 0.0;
#pragma unroll
      for (int q = 0; q < PE; ++q) {
        const double v = s[q] + tot[side][tid >> 4][q];
#pragma unroll
        for (int k = 0; k < PE; ++k) co[k] = fma(D[q * PE + k], v, co[k]);
      }
      sum += far_clenshaw<PE>(co, ((double)tid - ((double)half - 0.5)) / (double)half);
    }
  }
  if (!own) return;
  const int k = ts + tid;
  if (k - lane >= m.n_bins) return;
  double slope = 0.0;  // FP64 form: in units of 1 / dnu
  const int lm = g.mom ? far_cond_mom_level(g, cd) : kFarLevels;  // (k_far_cells has one row per tile)
  int64_t before = 0;
  for (int l = 0; l <= fc.lmax; ++l) {
    // tiles of 64 points or more hold all of the wave's points: their
    // coefficients are the wave's (scalar loads)
    const int lg = l + fc.sh, sl = far_slices(fc.sh, l);
    const int tl = lg >= 6 ? __builtin_amdgcn_readfirstlane(k >> lg) : min(k >> lg, far_tiles(nf, l) - 1);
    const double* r = g.rows + ((int64_t)blockIdx.y * g.cond_rows + before + (int64_t)tl * sl) * P;
    before += (int64_t)far_tiles(nf, l) * sl;
    double co[P];
#pragma unroll
    for (int q = 0; q < P; ++q) co[q] = r[q];
    for (int s = 1; s < (l < lm ? sl : 1); ++s)
#pragma unroll
      for (int q = 0; q < P; ++q) co[q] += r[s * P + q];
    // the point in the tile's variable: (k - centre) / half width
    const double hw = 0.5 * (double)(1 << lg);
    const double x = ((double)(k - (tl << lg)) - (hw - 0.5)) / hw;
    sum += far_clenshaw<P>(co, x);
    if constexpr (!F32) slope = fma(far_clenshaw_slope<P>(co, x), 1.0 / hw, slope);
  }
  // from the exact grid point to the rounded one
  if constexpr (!F32) sum = fma(slope, -far_grid_residue(m.nu0, m.dnu, k) / m.dnu, sum);
  if (k < m.n_bins) {
    const double scale = F32 ? exp(g.sb[cd.slot]) : 1.0;
    g.sigma[(int64_t)c * m.n_bins + k] += scale * sum;
  }
}

// Moments cost three kernels that short grids leave idle (45 us) and then go by
// cells, line by line costs go by lines: moments from so many cells on, or from so
// many lines to a leaf (whatever the other conditions: a condition has the same
// values by itself and in a table).  Measured, tiles line by one / by moments: FP32 form,
// 1.25e5 leaves, 4, 12, 80 lines each 395 / 300, 454 / 304, 1084 / 350 us; 1.25e4
// leaves, 2 and 16 lines 41 / 66, 52 / 66; FP64 form, 31250 leaves, 16 and 32 lines
// 648 / 209, 598 / 216, 3125 leaves, 19 lines 76 / 60.
constexpr int64_t kMomCells32 = 32768, kMomCells64 = 2048;
constexpr int kMomLines = 24;

int far_nodes(int prec) { return prec == XS_FP32 ? 12 : 20; }
int far_moments(int prec) { return prec == XS_FP32 ? kMoments32 : kMoments64; }

void launch_far(const ModelDev& m, const Work& w, int far_lmax, int end_min, int64_t n_lines, double* sigma,
                hipStream_t s) {
  FarArgs a;
  a.m = m;
  a.cond = w.cond;
  a.sb = w.sb;
  a.off = w.off + m.fine_v;
  a.rnu = w.rnu;
  a.rgref = w.rgref;
  a.rnexp = w.rnexp;
  a.rgpre = w.rgpre;
  a.rS = w.rS;
  a.rkc = w.rkc;
  a.rdel = w.rdel;
  a.rwin = w.rwin;
  a.max_lines = w.max_lines;
  a.counter = w.counter;
  a.cond_rows = far_rows_before(m.n_fine, m.fine_sh, far_lmax + 1);
  a.sigma = sigma;
  int64_t blocks = 0;
  for (int l = 0; l <= far_lmax; ++l) blocks += far_blocks(m.n_fine, m.fine_sh, l);
  a.blocks = (int32_t)blocks;
  // rows and moments lie in the partial rows, which the near leaves have done with; as
  // many conditions at a time as fit (lifetimes, whose widths have no bound
  // here, go line by line)
  a.mom_cells = far_cells_before(fine_keys(m), far_lmax + 1);
  const int64_t rows = a.cond_rows * far_nodes(m.prec), moments = a.mom_cells * far_moments(m.prec);
  const bool many = m.n_fine >= (m.prec == XS_FP32 ? kMomCells32 : kMomCells64) ||
                    n_lines >= kMomLines * (int64_t)m.n_fine;
  const bool mom = many && moments <= part_doubles(w) && !w.rgpre;
  const int at_once =
      w.far_extra ? 1 : (int)std::min<int64_t>(part_doubles(w) / (rows + (mom ? moments : 0)), m.n_cond);
  a.rows = w.far_extra ? w.far_extra : w.part;
  a.mom = !mom ? nullptr : w.far_extra ? w.part : w.part + at_once * rows;
  const int per_block = 4 * (64 / far_nodes(m.prec));  // tiles of a block of k_far_cells
  auto run = [&](auto leaves, auto moments, auto cells, auto far, auto finish) {
    for (a.c0 = 0; a.c0 < m.n_cond; a.c0 += at_once) {
      const int nc = std::min(at_once, m.n_cond - a.c0);
      const auto go = [&](auto k, int64_t bl) { hipLaunchKernelGGL(k, long_grid(bl, nc), dim3(256), 0, s, a); };
      if (a.mom) {
        go(leaves, (fine_keys(m) + 3) / 4);
        for (int b = 0; b < far_lmax; b += kMomLevels)
          hipLaunchKernelGGL(moments, dim3((far_tiles(fine_keys(m), b) + kMomLeaves - 1) / kMomLeaves, nc), dim3(256), 0, s,
                             a, b);
        go(cells, (far_cells_before(m.n_fine, far_lmax + 1) + per_block - 1) / per_block);
      }
      // (with moments most conditions have nothing left for it)
      go(far, std::min<int64_t>(blocks, a.mom ? 4096 : 1 << 22));
      go(finish, far_tiles(m.n_fine, end_min));
    }
  };
#define XS_F(PR)                                                                                                   \
  if (m.profile == PR && m.prec == XS_FP32)                                                                        \
    run(k_far_leaves<float, PR, kMoments32>, k_far_moments<kMoments32>, k_far_cells<12, kMoments32>,               \
        k_far<float, PR, 12>, k_far_finish<float, PR, 12, 6>);                                                     \
  else if (m.profile == PR)                                                                                        \
    run(k_far_leaves<double, PR, kMoments64>, k_far_moments<kMoments64>, k_far_cells<20, kMoments64>,              \
        k_far<double, PR, 20>, k_far_finish<double, PR, 20, 12>);
  XS_F(XS_VOIGT) XS_F(XS_LORENTZ) XS_F(XS_BIN_VOIGT) XS_F(XS_BIN_LORENTZ)
#undef XS_F
}

}  // namespace xs
