// Near leaves of the profile pass (far_geometry.h): the points within a few
// cells of a line, where its profile has structure on the grid's scale, and
// the whole windows of the outermost cells' lines.  The tiles further out are
// k_far's.  Gaussians, which are zero a few widths away, go point by point as a whole.
//
// A block of four waves owns 256 grid points of one condition and takes the
// lines whose near leaves meet them, 64 at a time and one per lane (2^ks lanes
// where there are few).  A lane
// walks its own line's points region by region -- the core first, where the
// rational approximation of w is needed, then the rings where six, four,
// three, two or one node pairs serve -- and adds each value to the wave's row
// of FP64 sums in LDS.  So every lane of a step evaluates the same formula at
// a point that needs it (a wave across 64 neighbouring points would run the
// formula of the worst one on all), no line's constants are passed between
// lanes, and no point outside a window is evaluated.  Lanes begin at
// different places of their ranges, so that few of a step's adds meet in one
// point or bank.  The four rows are added in order, and a tile of many lines
// is split into parts whose rows k_reduce adds in order, so the sums do not
// depend on scheduling.  Bound by VALU issue: of one instruction a SIMD every four
// cycles, on 1e7 lines, 0.90 (FP32 Voigt; waits on LDS are 3% of the wave cycles), 0.79 to
// 0.87 (FP64), bin means 0.96 and 0.75 (FP64, two waves a SIMD).  Measured against the
// gather's rows clipped to the near leaves
// (64 points): 1e7 lines FP32 4.07 -> 1.3 ms with leaves of 16 points, 1e6 lines
// FP64 1.30 -> 0.61 ms, 48 conditions x 1e6 lines FP32 9.39 -> 2.64 ms.
#include <algorithm>

#include "k_voigt.h"

namespace xs {

constexpr int kNearBins = 256;

struct NearArgs {
  ModelDev m;
  const CondDev* cond;
  const double* sb;
  const int32_t* off;
  const double* rnu;
  float* rgref;
  float* rnexp;
  const double* rgpre;
  void* rS;
  const int32_t* rkc;
  const float* rdel;
  const int32_t* rwin;
  OddLines odd;             // (no positions: Gaussians)
  int64_t max_lines;
  int32_t* counter;         // [2..3] candidate total; [4..5] lines per part; [6] parts beyond the first
  int32_t* parts;           // [n_ct] parts of each (tile, condition), 0: the gather's
  int32_t* base;            // [n_ct] first row of a split one
  int32_t* extra;           // [kNearExtra][2] (tile, condition) and part of the parts beyond the first
  double* rows;             // partial rows of split tiles
  double* sigma;
  int32_t accumulate;
  int32_t n_ct;             // tiles * n_cond; ct = tile * n_cond + condition
  int32_t extra_blocks;     // the first blocks of k_near's grid, which take the parts beyond the first
  int32_t rest;             // the conditions without tile expansions are the gather's
};

// Lines of tile t: segments of sorted lines, then (all: with them) the odd ones, which
// have no intensity in the segments.
struct NearSegs {
  int64_t beg[kSegs], cum[kSegs], all;
};
__device__ __forceinline__ NearSegs near_segments(const NearArgs& g, const CondDev& cd, int t) {
  const int sh = g.m.fine_sh;
  const int a = t * (kNearBins >> sh), b = a + (kNearBins >> sh) - 1;
  const int reach = (cd.wbins >> sh) + 2;
  const int clo = max(a - reach, -g.m.fine_v), chi = min(b + reach, g.m.n_fine - 1 + g.m.fine_v);
  CellRange s[kSegs];
  if (cd.far.on && !g.counter[kFarOff]) {
    far_segments(cd.far, a, b, clo, chi, s);
  } else {
    s[0] = CellRange{0, -1};
    s[1] = CellRange{clo, chi};
    s[2] = CellRange{0, -1};
  }
  NearSegs r;
  int64_t total = 0;
#pragma unroll
  for (int k = 0; k < kSegs; ++k) {
    const bool ok = s[k].lo <= s[k].hi;
    const int64_t p0 = ok ? g.off[s[k].lo] : 0, p1 = ok ? g.off[s[k].hi + 1] : 0;
    r.beg[k] = p0 - total;
    total += p1 - p0;
    r.cum[k] = total;
  }
  r.all = total + (g.odd.pos && !g.counter[kFarOff] ? g.counter[kOddCount] : 0);
  return r;
}

// The lines of a tile, or -1 where the condition's points are the gather's.
__device__ __forceinline__ int64_t near_lines(const NearArgs& g, int c, int t) {
  return g.rest && !g.cond[c].far.on ? -1 : near_segments(g, g.cond[c], t).all;
}

// Planning: candidates in all, then the parts of each tile.  A part holds at
// least kNearChunk lines, and so many that the parts beyond the first stay
// under kNearExtra: an even list is not split, and a list whose lines crowd
// into a few tiles is spread over the chip.
// The parts beyond the first run before the tiles, since a grid that ends with
// its largest blocks leaves compute units waiting for them (parts of 4096 lines
// at the end of the grid: a third of the CU cycles of 1e7 lines idle, 2.22 -> 1.51 ms).
constexpr int64_t kNearChunk = 1024;
constexpr int kNearExtra = 8192;

__global__ __launch_bounds__(256) void k_near_count(NearArgs g) {
  unsigned long long local = 0;
  for (int64_t ct = (int64_t)blockIdx.x * 256 + threadIdx.x; ct < g.n_ct; ct += (int64_t)gridDim.x * 256) {
    const int c = (int)(ct % g.m.n_cond), t = (int)(ct / g.m.n_cond);
    const int64_t n = near_lines(g, c, t);
    g.parts[ct] = (int32_t)n;
    local += (unsigned long long)max<int64_t>(n, 0);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) local += __shfl_xor(local, o, 64);
  if ((threadIdx.x & 63) == 0 && local) atomicAdd((unsigned long long*)(g.counter + 2), local);
}

// Odd lines (OddLines), by one block: the list, filled in any order, is sorted, and
// their records get no intensity and a width of one.
__device__ __forceinline__ void near_hide_odd(const NearArgs& g) {
  __shared__ int32_t pos[kOddMax];
  const int n = g.odd.pos ? g.counter[kOddCount] : 0;
  if (n == 0 || g.counter[kOddHidden] || g.counter[kFarOff]) return;
  for (int i = threadIdx.x; i < n; i += blockDim.x) pos[i] = g.odd.pos[i];
  __syncthreads();
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    const int32_t p = pos[i];
    int j = 0;
    for (int k = 0; k < n; ++k) j += pos[k] < p;
    g.odd.pos[j] = p;
    g.odd.gref[j] = g.rgref[p];
    g.odd.nexp[j] = g.rnexp[p];
    g.rgref[p] = 1.0f;
    g.rnexp[p] = 0.0f;
    for (int q = 0; q < g.m.n_slots; ++q) {
      const int64_t at = (int64_t)q * g.max_lines + p;
      double& S = g.odd.S[(int64_t)j * g.m.n_slots + q];
      if (g.m.prec == XS_FP32) {
        S = ((const float*)g.rS)[at];
        ((float*)g.rS)[at] = 0.0f;
      } else {
        S = ((const double*)g.rS)[at];
        ((double*)g.rS)[at] = 0.0;
      }
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) g.counter[kOddHidden] = 1;
}

__device__ __forceinline__ void near_plan_tiles(const NearArgs& g, int64_t total, int64_t first, int64_t step) {
  int64_t chunk = (total + kNearExtra - 1) / kNearExtra;
  chunk = max(kNearChunk, (chunk + 63) / 64 * 64);
  if (first == 0) *(int64_t*)(g.counter + 4) = chunk;
  for (int64_t ct = first; ct < g.n_ct; ct += step) {
    const int64_t n = g.parts[ct];
    const int np = n < 0 ? 0 : n <= chunk ? 1 : (int)((n + chunk - 1) / chunk);
    g.parts[ct] = np;
    g.base[ct] = 0;
    if (np > 1) {
      // sum of (np - 1) <= sum of n / chunk <= kNearExtra
      const int e = atomicAdd(g.counter + 6, np - 1);
      g.base[ct] = e;
      for (int k = 1; k < np; ++k) {
        g.extra[2 * (e + k - 1)] = (int32_t)ct;
        g.extra[2 * (e + k - 1) + 1] = k;
      }
    }
  }
}

__global__ __launch_bounds__(256) void k_near_plan(NearArgs g) {
  if (blockIdx.x == 0) near_hide_odd(g);
  near_plan_tiles(g, (int64_t) * (const unsigned long long*)(g.counter + 2), (int64_t)blockIdx.x * 256 + threadIdx.x,
                  (int64_t)gridDim.x * 256);
}

// Both in one block, for short grids: a launch less (118 tiles 89 -> 81 us the whole
// call; with 3907 tiles 61 -> 64).
constexpr int kNearOnce = 1024;
__global__ __launch_bounds__(1024) void k_near_plan_once(NearArgs g) {
  __shared__ unsigned long long sum;
  near_hide_odd(g);
  if (threadIdx.x == 0) sum = 0;
  __syncthreads();
  unsigned long long local = 0;
  for (int ct = threadIdx.x; ct < g.n_ct; ct += 1024) {
    const int64_t n = near_lines(g, ct % g.m.n_cond, ct / g.m.n_cond);
    g.parts[ct] = (int32_t)n;  // (read by the same thread)
    local += (unsigned long long)max<int64_t>(n, 0);
  }
  if (local) atomicAdd(&sum, local);
  __syncthreads();
  near_plan_tiles(g, (int64_t)sum, threadIdx.x, 1024);
}

// Place of a tile's point in a wave's LDS row: the points of equal remainder
// modulo four are neighbours, since a step of near_sweep4 adds to every fourth
// point; 16 words between the four parts keep a step over neighbouring points
// on different banks as well.
constexpr int kNearPart = kNearBins / 4 + 16;
constexpr int kNearRow = 4 * kNearPart;
__device__ __forceinline__ int near_place(int o) { return (o & 3) * kNearPart + (o >> 2); }

// The lanes of a line: 2^ks of them, this one the sub-th of the slot-th line of
// the wave.  Lane sub takes every 2^ks-th point, from its own place on.
struct NearLane {
  int slot, sub, ks;
};
// The place of a wave's line in the order of beginnings.  The FP32 form reverses
// its bits, so that neighbouring lanes, whose adds the LDS takes together, begin
// far apart: over a ring of three points 64 lanes in order are 16 adds to one
// address at a time, reversed 6 (48 conditions x 1e6 lines 4.79 -> 2.73 ms, 1e7 lines
// 1.56 -> 1.32).  The FP64 form is not bound by the adds (0.68 ms at 1e6 lines either
// way, bin means 1.30 and 1.34).
template <typename Real>
__device__ __forceinline__ int near_slot(int v, int ks) {
  return sizeof(Real) == 4 ? (int)(__builtin_bitreverse32((unsigned)v) >> 1 >> (25 + ks)) : v;
}
__device__ __forceinline__ int near_count(const NearLane& ln, int n) {
  return n > ln.sub ? (n - ln.sub + (1 << ln.ks) - 1) >> ln.ks : 0;
}
__device__ __forceinline__ int near_first(const NearLane& ln, int cnt) { return (ln.slot * cnt << ln.ks) >> 6; }

// k in [lo, hi] but not in [slo, shi]: the lane's points.
struct Ring {
  int lo, hi, slo, shi;
};
// (PLAIN: points in order in the row, for profiles that never go by groups: four
// operations less a point, two temperatures x 4 x 1e7 Doppler lines 634 -> 532 us)
template <bool PLAIN = false, typename F>
__device__ __forceinline__ void near_sweep(const Ring& r, const NearLane& ln, double* row, int tlo, F value) {
  const int skip = max(0, r.shi - r.slo + 1);
  const int n = near_count(ln, r.hi - r.lo + 1 - skip);
  int i = near_first(ln, n);
  for (int it = 0; it < n; ++it) {
    int k = r.lo + (i << ln.ks) + ln.sub;
    if (skip && k >= r.slo) k += skip;
    atomicAdd(&row[PLAIN ? k - tlo : near_place(k - tlo)], value(k));
    i = i + 1 == n ? 0 : i + 1;
  }
}

// Points of [klo, khi] within X of the line (|x| < X); empty ranges are lo > hi
// with lo - 1 = hi.  X has a part in a thousand to spare, so rounding leaves no
// point to a rule that does not hold; a whole point to spare on either side gave
// the core's rule, which costs most, up to four more (bin means of 3.9e5 lines 1.30
// ms, without 1.08) and its error where Re w is least (9e-5, the gather's and this
// now 7.5e-5, at 1e-4 bar).
template <typename R>
__device__ __forceinline__ void near_range(R X, R a, R b, int kc, int klo, int khi, int& lo, int& hi) {
  lo = klo;
  hi = klo - 1;
  if (!(X > (R)0)) return;
  const R l = fmin(fmax(ceil((b - X) / a), (R)-1.0e9), (R)1.0e9);
  const R h = fmin(fmax(floor((b + X) / a), (R)-1.0e9), (R)1.0e9);
  const int kl = max((int)l + kc, klo), kh = min((int)h + kc, khi);
  if (kl <= kh) {
    lo = kl;
    hi = kh;
  }
}

// As near_sweep over groups of four points k0..k0+3 (k0 a multiple of four):
// every ring edge lies between groups.  value4 fills the four values.
template <typename F>
__device__ __forceinline__ void near_sweep4(const Ring& r, const NearLane& ln, double* row, int tlo, F value4) {
  const int glo = (r.lo - tlo) >> 2, skip = max(0, r.shi - r.slo + 1) >> 2, gs = (r.slo - tlo) >> 2;
  const int n = near_count(ln, ((r.hi - r.lo + 1) >> 2) - skip);
  int i = near_first(ln, n);
  for (int it = 0; it < n; ++it) {
    int gr = glo + (i << ln.ks) + ln.sub;
    if (skip && gr >= gs) gr += skip;
    double v[4];
    value4(tlo + 4 * gr, v);
#pragma unroll
    for (int j = 0; j < 4; ++j) atomicAdd(&row[j * kNearPart + gr], v[j]);
    i = i + 1 == n ? 0 : i + 1;
  }
}

// Widens [lo, hi] (inside [klo, khi], whose edges lie between groups) to whole
// groups of four points.  A rule of more node pairs serves the points further
// out as well, so the widened ring keeps its accuracy.
__device__ __forceinline__ void near_align(int& lo, int& hi) {
  if (lo > hi) return;
  lo &= ~3;
  hi |= 3;
}

// 2^t, t <= 0, to an ulp, in half of the library's operations.
__device__ __forceinline__ double near_exp2(double t) {
  t = fmax(t, -2000.0);
  const double k = rint(t), r = t - k;
  return ldexp(fma(r, exp2m1_over(r), 1.0), (int)k);
}

// A Gaussian's points: those where it is not zero in the working precision
// (2^-160, 2^-1100; erfc(10.1), erfc(27.3)).
template <typename Real, int PROF>
__device__ __forceinline__ void near_gauss(const ModelDev& m, const CondDev& cd, const NearLane& lane, int kc, int klo,
                                           int khi, float del, double nu, Real S, double* row, int tlo) {
  constexpr bool BIN = PROF == XS_BIN_DOPPLER || PROF == XS_BIN_GAUSSIAN;
  constexpr bool FIXED = PROF == XS_GAUSSIAN || PROF == XS_BIN_GAUSSIAN;
  Ring r = {0, 0, 0, -1};
  if constexpr (sizeof(Real) == 4) {
    const float ia = rcp32(FIXED ? (float)cd.hwhm : (float)nu * (float)cd.dop);
    const float inv = BIN ? (float)0.83255461115769776 * ia : ia;
    const float a = (float)m.dnu * inv, b = del * inv, hh = 0.5f * a;
    const float c0 = BIN ? S * (float)(0.5 / m.dnu) : S * (float)0.46971863934982566 * inv;  // sqrt(ln2/pi)/alpha
    near_range<float>(BIN ? 10.1f + hh : 12.649110640673518f, a, b, kc, klo, khi, r.lo, r.hi);
    near_sweep<true>(r, lane, row, tlo, [&](int k) -> double {
      const float x = fmaf((float)(k - kc), a, -b);
      if constexpr (BIN) return (double)(c0 * erf_bin<float>(x, hh));
      else return (double)(c0 * __builtin_amdgcn_exp2f(-(x * x)));
    });
  } else {
    const double alpha = FIXED ? cd.hwhm : nu * cd.dop;
    const double inv = (BIN ? sqrt(kLN2) : 1.0) / alpha;
    const double a = m.dnu * inv, hh = 0.5 * a, c0 = BIN ? S * (0.5 / m.dnu) : S * (sqrt(kLN2 / kPI) * inv);
    const double b = (nu - nu_of_bin(m.nu0, m.dnu, kc)) * inv;
    near_range<double>(BIN ? 27.3 + hh : sqrt(1100.0), a, b, kc, klo, khi, r.lo, r.hi);
    near_sweep<true>(r, lane, row, tlo, [&](int k) -> double {
      double x;
      {
#pragma clang fp contract(off)
        x = (nu_of_bin(m.nu0, m.dnu, k) - nu) * inv;
      }
      if constexpr (BIN) return c0 * erf_bin<double>(x, hh);
      else return c0 * near_exp2(-(x * x));
    });
  }
}

// One lane's line over its points [klo, khi] of the tile.
template <int PROF>
__device__ __forceinline__ void near_line_f32(const ModelDev& m, const CondDev& cd, const NearLane& lane, int kc, int klo, int khi,
                                              float del, float nu, float S, float gref, float nexp, float gpre,
                                              double* row, int tlo) {
  const float gamma = fmaf(gref * __builtin_amdgcn_exp2f(nexp * (float)(cd.lnTr / kLN2)), (float)cd.pfac, gpre);
  const Ring all = {klo, khi, 0, -1};
  if constexpr (PROF == XS_LORENTZ || PROF == XS_BIN_LORENTZ) {
    const float inv = rcp32(gamma), a = (float)m.dnu * inv, nb = -(del * inv), hh = 0.5f * a;
    const float c0 = PROF == XS_LORENTZ ? S * (float)(1.0 / kPI) * inv : S * (float)(1.0 / (kPI * m.dnu));
    near_sweep(all, lane, row, tlo, [&](int k) -> double {
      const float x = fmaf((float)(k - kc), a, nb);
      if constexpr (PROF == XS_LORENTZ) return (double)(c0 * rcp32(fmaf(x, x, 1.0f)));
      else return (double)(c0 * lor_bin<float>(x, hh, a));
    });
  } else {
    constexpr bool BIN = PROF == XS_BIN_VOIGT;
    const float inv = (float)0.83255461115769776 * rcp32(nu * (float)cd.dop);  // sqrt(ln2)/alpha
    const float y = gamma * inv, y2 = y * y, a = (float)m.dnu * inv, b = del * inv, hh = BIN ? 0.5f * a : 0.0f;
    // 1/(sg sqrt(2 pi)); bin means: 1/(sqrt(pi) dnu)
    const float c0 = BIN ? S * (float)(0.56418958354775628 / m.dnu) : S * (float)0.56418958354775628 * inv;
    const float xmax = fmaxf(fabsf((float)(klo - kc) * a - b), fabsf((float)(khi - kc) * a - b)) + hh;
    // |x| or y beyond FP32's safe range (nu of a few 1e-3 cm^-1 or less): FP64
    const bool wide = !(xmax <= 1.0e9f) || !(y <= 1.0e9f);
    Ring w = all;
    if (!wide) w.hi = w.lo - 1;
    near_sweep(w, lane, row, tlo, [&](int k) -> double {
      const double x = (double)(k - kc) * (double)a - (double)b;
      if constexpr (BIN) return (double)(float)((double)c0 * voigt_bin_f64(x, (double)y, 0.5 * (double)a));
      else return (double)(float)((double)c0 * re_w_f64(x, (double)y));
    });
    if (wide) khi = klo - 1;
    // rings by |z|^2 at the point (bin means: at the bin's nearest point).  Three
    // pairs to 100, two to 1600: a wave over a row of points took the nearest one's
    // rule for all, and with a line to a lane from 64 and 900 on the error of 1 bar
    // spectra was 3.1e-6, before 1.4e-6
    auto X = [&](float rho) { return rho > y2 ? sqrtf(rho - y2) + hh : 0.0f; };
    int l0, h0, l1, h1, l2, h2;
    near_range<float>(X(1601.6f), a, b, kc, klo, khi, l2, h2);
    near_range<float>(X(100.1f), a, b, kc, l2, h2, l1, h1);
    near_range<float>(X(36.036f), a, b, kc, l1, h1, l0, h0);
    const bool groups = !BIN && __ballot((klo & 3) != 0 || (khi & 3) != 3) == 0;
    if (groups) {
      near_align(l2, h2);
      near_align(l1, h1);
    }
    auto xof = [&](int k) { return fmaf((float)(k - kc), a, -b); };
    const float cy = c0 * (float)(2.0 / kPI) * y, yh = y * a, y4 = 4.0f * y2;
    // the core
    near_sweep(Ring{l0, h0, 0, -1}, lane, row, tlo, [&](int k) -> double {
      const float x = xof(k);
      if constexpr (BIN) return (double)(c0 * (float)voigt_bin_core<24>((double)x, (double)y, 0.5 * (double)a));
      double wr, wi;
      w_weideman<24>((double)x, (double)y, wr, wi);
      return (double)(float)((double)c0 * wr);
    });
    auto ring = [&](auto np, float rho, int lo, int hi, int slo, int shi) {
      constexpr int NP = decltype(np)::value;
      if constexpr (BIN) {
        // largest argument of the ring's arctangents: y h / (y^2 + (|x| - s)^2)
        const float xn = fmaxf(sqrtf(fmaxf(rho - y2, 0.0f)) - (float)gh_node<NP>()[NP - 1], 0.0f);
        const bool two = __ballot(lo <= hi && !(yh <= 0.02f * fmaf(xn, xn, y2))) == 0;
        if (two) {
          near_sweep(Ring{lo, hi, slo, shi}, lane, row, tlo, [&](int k) -> double {
            return (double)(c0 * vpairs_bin_two<NP, float>(xof(k), hh, yh, y2));
          });
        } else {
          near_sweep(Ring{lo, hi, slo, shi}, lane, row, tlo, [&](int k) -> double {
            const float x = xof(k);
            return (double)(c0 * vpairs_bin<NP, false, float>(x - hh, x + hh, yh, y2));
          });
        }
      } else {
        near_sweep(Ring{lo, hi, slo, shi}, lane, row, tlo, [&](int k) -> double {
          const float x = xof(k);
          return (double)(cy * gh_f32<NP>(x * x, y2, y4));
        });
      }
    };
    ring(std::integral_constant<int, 3>(), 36.0f, l1, h1, l0, h0);
    if (groups) {
      auto ring4 = [&](auto np, int lo, int hi, int slo, int shi) {
        constexpr int NP = decltype(np)::value;
        near_sweep4(Ring{lo, hi, slo, shi}, lane, row, tlo, [&](int k, double (&v)[4]) {
          const float r0 = (float)(k - kc);
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const float x = fmaf(r0 + (float)j, a, -b);
            v[j] = (double)(cy * gh_f32<NP>(x * x, y2, y4));
          }
        });
      };
      ring4(std::integral_constant<int, 2>(), l2, h2, l1, h1);
      ring4(std::integral_constant<int, 1>(), klo, khi, l2, h2);
    } else {
      ring(std::integral_constant<int, 2>(), 100.0f, l2, h2, l1, h1);
      ring(std::integral_constant<int, 1>(), 1600.0f, klo, khi, l2, h2);
    }
  }
}

template <int PROF>
__device__ __forceinline__ void near_line_f64(const ModelDev& m, const CondDev& cd, const NearLane& lane, int kc, int klo, int khi,
                                              double nu, double S, double gref, double nexp, double gpre,
                                              double* row, int tlo) {
  const double gamma = gref * exp(nexp * cd.lnTr) * cd.pfac + gpre;
  // x from the rounded grid point, as the profile is defined
  const double inv = (PROF == XS_LORENTZ || PROF == XS_BIN_LORENTZ) ? 1.0 / gamma : sqrt(kLN2) / (nu * cd.dop);
  auto xof = [&](int k) {
#pragma clang fp contract(off)
    return (nu_of_bin(m.nu0, m.dnu, k) - nu) * inv;
  };
  const double a = m.dnu * inv;
  const Ring all = {klo, khi, 0, -1};
  if constexpr (PROF == XS_LORENTZ || PROF == XS_BIN_LORENTZ) {
    const double hh = 0.5 * a, c0 = PROF == XS_LORENTZ ? S / (kPI * gamma) : S / (kPI * m.dnu);
    near_sweep(all, lane, row, tlo, [&](int k) -> double {
      const double x = xof(k);
      if constexpr (PROF == XS_LORENTZ) return c0 * rcp64(fma(x, x, 1.0));
      else return c0 * lor_bin<double>(x, hh, a);
    });
  } else {
    constexpr bool BIN = PROF == XS_BIN_VOIGT;
    const double y = gamma * inv, y2 = y * y, hh = BIN ? 0.5 * a : 0.0;
    const double c0 = BIN ? S / (sqrt(kPI) * m.dnu) : S * sqrt(kLN2) / (nu * cd.dop * sqrt(kPI));
    const double b = (nu - nu_of_bin(m.nu0, m.dnu, kc)) * inv;
    const double xmax = fmax(fabs((double)(klo - kc) * a - b), fabs((double)(khi - kc) * a - b));
    // the rings' shared reciprocals keep finite for |x|, y <= 1e9
    const bool wide = !BIN && (!(xmax <= 1.0e9) || !(y <= 1.0e9));
    Ring w = all;
    if (!wide) w.hi = w.lo - 1;
    if constexpr (!BIN) near_sweep(w, lane, row, tlo, [&](int k) -> double { return c0 * re_w_f64(xof(k), y); });
    if (wide) khi = klo - 1;
    // the ranges only pick formulas; FP32 suffices
    const float af = (float)a, bf = (float)b;
    auto X = [&](double rho) { return rho > y2 ? sqrtf((float)(rho - y2)) + (float)hh : 0.0f; };
    int l1, h1, l2, h2, l3, h3, l4, h4, l5, h5;
    constexpr double kTwo = BIN ? 6400.0 : 4000.0;
    near_range<float>(X(9.0e6 * 1.001), af, bf, kc, klo, khi, l5, h5);
    near_range<float>(X(kTwo * 1.001), af, bf, kc, l5, h5, l4, h4);
    near_range<float>(X(400.0 * 1.001), af, bf, kc, l4, h4, l3, h3);
    near_range<float>(X(144.0 * 1.001), af, bf, kc, l3, h3, l2, h2);
    near_range<float>(X(64.0 * 1.001), af, bf, kc, l2, h2, l1, h1);
    const bool groups = !BIN && __ballot((klo & 3) != 0 || (khi & 3) != 3) == 0;
    if (groups) {
      near_align(l5, h5);
      near_align(l4, h4);
      near_align(l3, h3);
      near_align(l2, h2);
    }
    const double cy = c0 * (y * (2.0 / kPI)), yh = y * a, y4 = 4.0 * y2;
    auto pairs = [&](auto np, double x) {
      double N, D;
      gh_nd<decltype(np)::value>(x * x, y2, y4, N, D);
      return cy * N * rcp64(D);
    };
    using P6 = std::integral_constant<int, 6>;
    // the core; a point of its margin has |z| >= 8 and takes six pairs, where
    // the approximation's error against a small Re w grows
    near_sweep(Ring{l1, h1, 0, -1}, lane, row, tlo, [&](int k) -> double {
      const double x = xof(k);
      if constexpr (BIN) {
        const double xn = fmax(fabs(x) - hh, 0.0);
        if (fma(xn, xn, y2) >= 64.0) return c0 * vpairs_bin<6, false, double>(x - hh, x + hh, yh, y2);
        return c0 * voigt_bin_core<40>(x, y, hh);
      } else {
        if (fma(x, x, y2) >= 64.0) return pairs(P6(), x);
        double wr, wi;
        w_weideman<40>(x, y, wr, wi);
        return c0 * wr;
      }
    });
    auto ring = [&](auto np, double rho, int lo, int hi, int slo, int shi) {
      constexpr int NP = decltype(np)::value;
      if constexpr (BIN) {
        // largest argument of the ring's arctangents: y h / (y^2 + (|x| - s)^2)
        const double xn = fmax(sqrt(fmax(rho - y2, 0.0)) - gh_node<NP>()[NP - 1], 0.0);
        const bool two = __ballot(lo <= hi && !(yh <= 2.5e-4 * fma(xn, xn, y2))) == 0;
        if (two) {
          near_sweep(Ring{lo, hi, slo, shi}, lane, row, tlo,
                     [&](int k) -> double { return c0 * vpairs_bin_two<NP, double>(xof(k), hh, yh, y2); });
        } else {
          near_sweep(Ring{lo, hi, slo, shi}, lane, row, tlo, [&](int k) -> double {
            const double x = xof(k);
            return c0 * vpairs_bin<NP, false, double>(x - hh, x + hh, yh, y2);
          });
        }
      } else if (groups && NP != 6) {
        near_sweep4(Ring{lo, hi, slo, shi}, lane, row, tlo, [&](int k, double (&v)[4]) {
#pragma unroll
          for (int j = 0; j < 4; j += 2) {
            const double x0 = xof(k + j), x1 = xof(k + j + 1);
            double N0, D0, N1, D1;
            gh_nd<NP>(x0 * x0, y2, y4, N0, D0);
            gh_nd<NP>(x1 * x1, y2, y4, N1, D1);
            // two points over one reciprocal (the products stay below 1e295)
            const double r = cy * rcp64(D0 * D1);
            v[j] = N0 * D1 * r;
            v[j + 1] = N1 * D0 * r;
          }
        });
      } else {
        near_sweep(Ring{lo, hi, slo, shi}, lane, row, tlo, [&](int k) -> double { return pairs(np, xof(k)); });
      }
    };
    ring(P6(), 64.0, l2, h2, l1, h1);
    ring(std::integral_constant<int, 4>(), 144.0, l3, h3, l2, h2);
    ring(std::integral_constant<int, 3>(), 400.0, l4, h4, l3, h3);
    ring(std::integral_constant<int, 2>(), kTwo, l5, h5, l4, h4);
    ring(std::integral_constant<int, 1>(), 9.0e6, klo, khi, l5, h5);
  }
}

template <typename Real, int PROF>
__global__ __launch_bounds__(256) void k_near(NearArgs g) {
  constexpr bool GAUSS = base_profile(PROF) == XS_DOPPLER || base_profile(PROF) == XS_GAUSSIAN;
  __shared__ double rows[4][kNearRow];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const ModelDev& m = g.m;
  double* row = rows[wave];
  // the grid's first blocks take the parts beyond tiles' first, the others one
  // tile each
  const int block = long_block();
  const bool extras = block < g.extra_blocks;
  const int items = extras ? g.counter[6] : min(block + 1, g.n_ct + g.extra_blocks);
  for (int item = block; item < items; item += extras ? g.extra_blocks : 1) {
    int ct = item - g.extra_blocks, part = 0;
    if (extras) {
      ct = g.extra[2 * item];
      part = g.extra[2 * item + 1];
    } else {
      // each tile begins with another condition: blocks go to the eight dies in
      // turn, and with a multiple of eight conditions a die had the same ones
      const int t = ct / m.n_cond;
      ct = t * m.n_cond + (ct + t) % m.n_cond;
    }
    const int np = g.parts[ct];
    if (!GAUSS && np == 0) continue;  // the gather's
    const int c = ct % m.n_cond, t = ct / m.n_cond;
    const CondDev& cd = g.cond[c];
    const NearSegs sg = near_segments(g, cd, t);
    const int gap = cd.far.on ? far_gap(cd.far, 0, t * (kNearBins >> m.fine_sh)) : 0;
    const int tlo = t * kNearBins, thi = (int)min<int64_t>((int64_t)tlo + kNearBins, m.n_bins) - 1;
    const int64_t chunk = *(const int64_t*)(g.counter + 4);
    const int64_t q0 = np > 1 ? part * chunk : 0;
    const int64_t all = GAUSS ? sg.cum[kSegs - 1] : sg.all;  // (Gaussians: neither odd lines nor the gather's)
    const int64_t q1 = np > 1 ? min(all, q0 + chunk) : all;
#pragma unroll
    for (int j = 0; j < kNearRow / 64; ++j) row[lane + 64 * j] = 0.0;
    __syncthreads();
    // few lines are spread over the block's lanes, up to a wave to a line
    int ks = 0;
    while (ks < 6 && ((q1 - q0) << (ks + 1)) <= 256) ++ks;
    const NearLane ln = {near_slot<Real>(lane >> ks, ks), lane & ((1 << ks) - 1), ks};
    for (int64_t b0 = q0; b0 < q1; b0 += 256 >> ks) {
      const int64_t q = b0 + (tid >> ks);
      if (q < q1) {
        const bool near = q < sg.cum[0];
        int64_t p = q + (near ? sg.beg[0] : q < sg.cum[1] ? sg.beg[1] : sg.beg[2]);
        if (!GAUSS && __builtin_expect(q >= sg.cum[kSegs - 1], 0)) p = g.odd.pos[q - sg.cum[kSegs - 1]];
        const int2 win = ((const int2*)g.rwin)[(int64_t)cd.cclass * g.max_lines + p];
        const int kc = g.rkc[p];
        Real S = ((const Real*)g.rS)[(int64_t)cd.slot * g.max_lines + p];
        const double nu = g.rnu[p];
        float gref = g.rgref[p], nexp = g.rnexp[p];
        if (!GAUSS && __builtin_expect(q >= sg.cum[kSegs - 1], 0)) {
          const int64_t j = q - sg.cum[kSegs - 1];
          S = (Real)g.odd.S[j * m.n_slots + cd.slot];
          gref = g.odd.gref[j];
          nexp = g.odd.nexp[j];
        }
        const double gpre = g.rgpre ? g.rgpre[p] : 0.0;
        int klo = max(win.x, tlo), khi = min(win.y, thi);
        if (near) {
          const int f = kc >> m.fine_sh;
          klo = max(klo, far_shl(f - gap, m.fine_sh));
          khi = min(khi, far_shl(f + gap + 1, m.fine_sh) - 1);
        }
        if (win.x <= win.y && klo <= khi && S != (Real)0) {
          if constexpr (GAUSS)
            near_gauss<Real, PROF>(m, cd, ln, kc, klo, khi, g.rdel[p], nu, S, row, tlo);
          else if constexpr (sizeof(Real) == 4)
            near_line_f32<PROF>(m, cd, ln, kc, klo, khi, g.rdel[p], (float)nu, S, gref, nexp, (float)gpre, row, tlo);
          else
            near_line_f64<PROF>(m, cd, ln, kc, klo, khi, nu, S, (double)gref, (double)nexp, gpre, row, tlo);
        }
      }
    }
    __syncthreads();
    const int o = GAUSS ? tid : near_place(tid);
    const double v = ((rows[0][o] + rows[1][o]) + rows[2][o]) + rows[3][o];
    if (np == 1) {
      const int64_t k = (int64_t)tlo + tid;
      if (k <= thi) {
        double* out = g.sigma + (int64_t)c * m.n_bins + k;
        const double s = (sizeof(Real) == 4 ? exp(g.sb[cd.slot]) : 1.0) * v;
        *out = g.accumulate ? *out + s : s;
      }
    } else {
      // rows of a split tile: part 0's after the extra parts' rows
      const int64_t r = part == 0 ? (int64_t)kNearExtra + g.base[ct] : (int64_t)g.base[ct] + part - 1;
      g.rows[r * kNearBins + tid] = v;
    }
    __syncthreads();  // (the rows are the next part's)
  }
}

// Sum of the rows of split tiles, in the order of their parts; and the queue's
// counters are cleared for the next pass, as they are by the preparation.
__global__ __launch_bounds__(256) void k_near_reduce(NearArgs g) {
  if (blockIdx.x == 0 && threadIdx.x < kFarOff) g.counter[threadIdx.x] = 0;
  for (int ct = blockIdx.x; ct < g.n_ct; ct += gridDim.x) {
    const int np = g.parts[ct];
    if (np <= 1) continue;
    const int c = ct % g.m.n_cond, t = ct / g.m.n_cond;
    const int64_t k = (int64_t)t * kNearBins + threadIdx.x;
    if (k >= g.m.n_bins) continue;
    const double* r = g.rows + (int64_t)g.base[ct] * kNearBins + threadIdx.x;
    double s = r[(int64_t)kNearExtra * kNearBins];
    for (int j = 1; j < np; ++j) s += r[(int64_t)(j - 1) * kNearBins];
    s *= g.m.prec == XS_FP32 ? exp(g.sb[g.cond[c].slot]) : 1.0;
    double* out = g.sigma + (int64_t)c * g.m.n_bins + k;
    *out = g.accumulate ? *out + s : s;
  }
}

size_t near_row_doubles() { return (size_t)2 * kNearExtra * kNearBins + kNearExtra; }

void launch_near(const ModelDev& m, const Work& w, double* sigma, int accumulate, bool rest, int64_t n_lines,
                 hipStream_t s) {
  NearArgs a;
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
  a.odd = w.odd;
  a.rest = rest;
  a.max_lines = w.max_lines;
  a.counter = w.counter;
  a.parts = w.item_cnt;
  a.base = w.item_base;
  a.rows = w.part;
  a.extra = (int32_t*)(w.part + (size_t)2 * kNearExtra * kNearBins);
  a.sigma = sigma;
  a.accumulate = accumulate;
  a.n_ct = (int)((m.n_bins + kNearBins - 1) / kNearBins) * m.n_cond;
  const int cb = (int)std::min<int64_t>(1024, (a.n_ct + 255) / 256);
  if (a.n_ct <= kNearOnce) {
    hipLaunchKernelGGL(k_near_plan_once, dim3(1), dim3(1024), 0, s, a);
  } else {
    hipLaunchKernelGGL(k_near_count, dim3(cb), dim3(256), 0, s, a);
    hipLaunchKernelGGL(k_near_plan, dim3(cb), dim3(256), 0, s, a);
  }
  // about as many as there are parts (a line meets a tile or two); fewer take turns
  a.extra_blocks = (int)std::min<int64_t>(kNearExtra, 8 + n_lines * m.n_cond / kNearChunk);
  const dim3 grid = long_grid((int64_t)a.n_ct + a.extra_blocks);
#define XS_N(PR)                                                                                        \
  if (m.profile == PR && m.prec == XS_FP32) hipLaunchKernelGGL((k_near<float, PR>), grid, dim3(256), 0, s, a); \
  else if (m.profile == PR) hipLaunchKernelGGL((k_near<double, PR>), grid, dim3(256), 0, s, a);
  XS_N(XS_VOIGT) XS_N(XS_LORENTZ) XS_N(XS_BIN_VOIGT) XS_N(XS_BIN_LORENTZ)
  XS_N(XS_DOPPLER) XS_N(XS_GAUSSIAN) XS_N(XS_BIN_DOPPLER) XS_N(XS_BIN_GAUSSIAN)
#undef XS_N
  hipLaunchKernelGGL(k_near_reduce, dim3((unsigned)std::min(a.n_ct, 4096)), dim3(256), 0, s, a);
}

}  // namespace xs
