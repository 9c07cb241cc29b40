// Per-line constants of the profiles and the far-region evaluators of the
// Voigt profile, shared by the point-by-point gather and the tile expansions.
#pragma once
#include "k_common.h"

namespace xs {

struct LineParams {
  double inv, y, c0;
};

template <int PROF>
__device__ __forceinline__ LineParams line_params(const ModelDev& m, const CondDev& cd, double nu,
                                                  double gref, double nexp, double gpre, double S) {
  LineParams lp;
  double alpha = (PROF == XS_GAUSSIAN) ? cd.hwhm : nu * cd.dop;
  double gamma = gref * exp(nexp * cd.lnTr) * cd.pfac + gpre;
  if (PROF == XS_DOPPLER || PROF == XS_GAUSSIAN) {
    lp.inv = 1.0 / alpha;
    lp.y = 0.0;
    lp.c0 = S * sqrt(kLN2 / kPI) / alpha;
  } else if (PROF == XS_LORENTZ) {
    lp.inv = 1.0 / gamma;
    lp.y = 0.0;
    lp.c0 = S / (kPI * gamma);
  } else {
    lp.inv = sqrt(kLN2) / alpha;
    lp.y = gamma * lp.inv;
    lp.c0 = S * sqrt(kLN2) / (alpha * sqrt(kPI));
  }
  return lp;
}

// Far-region constants of node pair (tau, W) in the shifted variable
// s = x^2 + h, h = y^2 - tau: the pair's term is cW (s + 2 tau)/(s^2 + c),
// c = 4 y^2 tau (the same fraction as cW (u + p)/(u^2 + q u + p^2) with
// u = x^2, p = y^2 + tau, q = 2 y^2 - 2 tau, one operation fewer).
template <typename R>
struct Pair {
  R cw, cwt, h, c;  // cW, cW 2 tau, y^2 - tau, 4 y^2 tau
};
template <typename R>
__device__ __forceinline__ Pair<R> make_pair(double c0, double y, double tau, double W) {
  const double y2 = y * y;
  const double cw = c0 * (y * (2.0 / kPI)) * W;
  Pair<R> r;
  r.cw = (R)cw;
  r.cwt = (R)(cw * (2.0 * tau));
  r.h = (R)(y2 - tau);
  r.c = (R)(4.0 * y2 * tau);
  return r;
}

// FP64 two node pairs (tau_1, W_1), (tau_2, W_2) of the four-point rule as
// one fraction N(s)/D(s) in s = x^2 + y^2 - tau_1 = |z|^2 - tau_1.  With
// d = tau_1 - tau_2, c_j = 4 y^2 tau_j and cw_j = c0 (2 y/pi) W_j the pairs
// are cw_1 (s + e_1)/(s^2 + c_1) + cw_2 (s + e_2)/((s + d)^2 + c_2),
// e_1 = 2 tau_1, e_2 = tau_1 + tau_2, so
//   N = cw_1 (s + e_1)(s^2 + 2 d s + q) + cw_2 (s + e_2)(s^2 + c_1),
//   D = (s^2 + c_1)(s^2 + 2 d s + q),  q = d^2 + c_2,
// expanded into a cubic and a monic quartic.  Where the rule is used,
// s >= 4000 - tau_1 and c_j <= 4 tau_j (s + tau_1), so every lower term of
// either polynomial is below 3e-3 of the leading one: Horner's rule keeps the
// relative error at a few units of rounding, with one FMA per degree.
struct Poly2 {
  double h, n3, n2, n1, n0, d3, d2, d1, d0;  // h = y^2 - tau_1
};
__device__ __forceinline__ Poly2 make_poly2(double c0, double y) {
  const double t1 = GH::t4[0], t2 = GH::t4[1];
  const double y2 = y * y, k = c0 * (y * (2.0 / kPI));
  const double cw1 = k * GH::w4[0], cw2 = k * GH::w4[1];
  const double d = t1 - t2, c1 = 4.0 * y2 * t1, q = d * d + 4.0 * y2 * t2;
  const double e1 = 2.0 * t1, e2 = t1 + t2;
  Poly2 B;
  B.h = y2 - t1;
  B.n3 = cw1 + cw2;
  B.n2 = cw1 * (2.0 * d + e1) + cw2 * e2;
  B.n1 = cw1 * (q + 2.0 * d * e1) + cw2 * c1;
  B.n0 = cw1 * e1 * q + cw2 * e2 * c1;
  B.d3 = 2.0 * d;
  B.d2 = q + c1;
  B.d1 = 2.0 * d * c1;
  B.d0 = c1 * q;
  return B;
}
__device__ __forceinline__ void poly2_nd(const Poly2& B, double x, double& N, double& D) {
  const double s = fma(x, x, B.h);
  N = fma(fma(fma(B.n3, s, B.n2), s, B.n1), s, B.n0);
  D = fma(fma(fma(s + B.d3, s, B.d2), s, B.d1), s, B.d0);
}

// FP64 three-point rule (nodes 0 and +-t, tau = t^2 = 3/2) as one fraction
// in s = |z|^2 - tau.  The pair is cw (s + 2 tau)/(s^2 + c), c = 4 y^2 tau,
// cw = c0 (2 y/pi) W; the node at 0 adds e/(x^2 + y^2) = e/(s + tau) with
// e = c0 (y/pi) W_0.  Together
//   N = (cw + e) s^2 + 3 cw tau s + (2 cw tau^2 + e c),
//   D = (s^2 + c)(s + tau) = s^3 + tau s^2 + c s + c tau:
// two FMAs for N and an add and two FMAs for D, against three and four for
// the four-point fraction.  Where it is used, s >= 4.5e4 - tau, so the lower
// terms are below 1e-4 of the leading ones.
struct Poly3 {
  double h, tau, n2, n1, n0, c, ct;  // h = y^2 - tau; ct = c tau
};
__device__ __forceinline__ Poly3 make_poly3(double c0, double y) {
  const double tau = GH::t3[0];
  const double y2 = y * y, k = c0 * (y * (2.0 / kPI));
  const double cw = k * GH::w3[0], e = 0.5 * k * GH::w3c, c = 4.0 * y2 * tau;
  Poly3 C;
  C.h = y2 - tau;
  C.tau = tau;
  C.n2 = cw + e;
  C.n1 = 3.0 * cw * tau;
  C.n0 = 2.0 * cw * tau * tau + e * c;
  C.c = c;
  C.ct = c * tau;
  return C;
}
__device__ __forceinline__ void poly3_nd(const Poly3& C, double x, double& N, double& D) {
  const double s = fma(x, x, C.h);
  N = fma(fma(C.n2, s, C.n1), s, C.n0);
  D = fma(fma(s + C.tau, s, C.c), s, C.ct);
}

__device__ __forceinline__ float rcp32(float d) { return __builtin_amdgcn_rcpf(d); }

// The hardware FP64 reciprocal has a relative error below 5e-8 on gfx950
// (measured over 1e6 arguments spanning 1e-30..1e30); one Newton step
// squares it, to below 3e-15.
__device__ __forceinline__ double rcp64(double d) {
  const double r = __builtin_amdgcn_rcp(d);
  return fma(r, fma(-d, r, 1.0), r);
}

template <typename R>
__device__ __forceinline__ R pair_term(const Pair<R>& P, R x) {
  const R s = fma(x, x, P.h);
  const R n = fma(P.cw, s, P.cwt);
  const R d = fma(s, s, P.c);
  if constexpr (sizeof(R) == 4) return n * rcp32(d);
  else return n * rcp64(d);
}
// two pairs as one fraction (FP64 only: the product of the d_j stays finite)
__device__ __forceinline__ double pair2_term(const Pair<double>& P, const Pair<double>& Q, double x) {
  const double s1 = fma(x, x, P.h), s2 = fma(x, x, Q.h);
  const double n1 = fma(P.cw, s1, P.cwt), d1 = fma(s1, s1, P.c);
  const double n2 = fma(Q.cw, s2, Q.cwt), d2 = fma(s2, s2, Q.c);
  return fma(n1, d2, n2 * d1) * rcp64(d1 * d2);
}
__device__ __forceinline__ double poly2_term(const Poly2& B, double x) {
  double N, D;
  poly2_nd(B, x, N, D);
  return N * rcp64(D);
}

// NP node pairs of Re w without the factor 2 y / pi, as one fraction N/D
// (FP64: D is a product of NP terms below ~1e37 for |x|, y <= 1e9).
template <int NP>
__device__ __forceinline__ void gh_nd(double u, double y2, double y4, double& N, double& D) {
  const double* tau = gh_tau<NP>();
  const double* W = gh_w<NP>();
#pragma unroll
  for (int j = 0; j + 1 < NP; j += 2) {
    const double s1 = u + (y2 - tau[j]), s2 = u + (y2 - tau[j + 1]);
    const double d1 = fma(s1, s1, y4 * tau[j]), d2 = fma(s2, s2, y4 * tau[j + 1]);
    const double n1 = fma(W[j], s1, 2.0 * tau[j] * W[j]), n2 = fma(W[j + 1], s2, 2.0 * tau[j + 1] * W[j + 1]);
    const double n = fma(n1, d2, n2 * d1), d = d1 * d2;
    N = j ? fma(N, d, n * D) : n;
    D = j ? D * d : d;
  }
  if constexpr (NP & 1) {
    constexpr int j = NP - 1;
    const double s1 = u + (y2 - tau[j]);
    const double d = fma(s1, s1, y4 * tau[j]), n = fma(W[j], s1, 2.0 * tau[j] * W[j]);
    N = j ? fma(N, d, n * D) : n;
    D = j ? D * d : d;
  }
}
// the same, FP32, a reciprocal per pair
template <int NP>
__device__ __forceinline__ float gh_f32(float u, float y2, float y4) {
  const double* tau = gh_tau<NP>();
  const double* W = gh_w<NP>();
  float t = 0.0f;
#pragma unroll
  for (int j = 0; j < NP; ++j) {
    const float s = u + (y2 - (float)tau[j]);
    t = fmaf(fmaf((float)W[j], s, (float)(2.0 * tau[j] * W[j])), rcp32(fmaf(s, s, y4 * (float)tau[j])), t);
  }
  return t;
}

// Bin mean of NP node pairs (in the convention of vpairs_bin) with two terms
// of the arctangents' series: a pair +-s takes one reciprocal, den-+ =
// P -+ 2 s x with P = x^2 + (y^2 + s^2 - hh^2), D = den- den+ = P^2 - 4 s^2 x^2,
// t+ + t- = 2 y h P / D, t+ t- = (y h)^2 / D and
// atan(t+) + atan(t-) = (t+ + t-)(1 - (t+ + t-)^2/3 + t+ t-) + O(t^5):
// relative error below 1e-16 for t <= 2.5e-4, 3e-8 for t <= 0.02.
template <int NP, typename R>
__device__ __forceinline__ R vpairs_bin_two(R x, R hh, R yh, R y2) {
  const double* tau = gh_tau<NP>();
  const R u = x * x;
  R t = (R)0;
#pragma unroll
  for (int j = 0; j < NP; ++j) {
    const R P = u + (y2 + ((R)tau[j] - hh * hh));
    const R iD = rcp_r<R>(fma(P, P, u * (R)(-4.0 * tau[j])));
    const R A = yh * iD, e1 = (R)2 * P * A;
    t = fma((R)(gh_w<NP>()[j] / kPI), P * iD * fma(e1 * e1, (R)(-1.0 / 3.0), (R)1 + yh * A), t);
  }
  return ((R)2 * yh) * t;
}

}  // namespace xs
