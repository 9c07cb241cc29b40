// Geometry of the far field of the profile pass: which grid tiles take a
// line's profile through Chebyshev expansions and which take it point by
// point.  Plain integer functions, shared by the kernels, the host runtime
// and the host tests.
//
// The grid is cut into leaves of 2^sh points (the sort's cells); a tile of level
// l is 2^l leaves.  Tile t of level l is apart from cell f (the lines whose
// home bin is in leaf f) when at least one tile and at least `gap` cells lie
// between them: |(f >> l) - t| >= far_apart.  gap grows with wavenumber, as the
// lines' widths do, and is the same for all tiles inside one tile of the top
// level (and of 256 points).  Cells within gap of a leaf are near it and reach it point by point.
// Of the other leaves
//   - a tile of a level above `end` is admissible when it is apart and the
//     window of every line of the cell covers it;
//   - a tile of level l <= end when it is apart and the window of some line of
//     the cell can touch its ancestor of level `end`.
// A (tile, cell) pair belongs to the highest level at which it is admissible,
// so every leaf beyond the near ones that a window can touch takes a line
// through exactly one tile.  Only tiles of level `end` can be cut by a window
// end: their cells whose windows may end inside are set apart (far_cut), and
// their lines are added up to the window's end only.
// Lines beyond the grid lie in cells -v .. -1 and n_fine .. n_fine + v - 1, which
// differ from the others only in that no leaf belongs to them; v is a multiple of
// the widest tile (far_virtual).  The outermost cells, -v and n_fine - 1 + v, which
// also hold the lines further out, go point by point over their whole windows.
#pragma once
#include <stdint.h>

#ifdef __HIPCC__
#define XS_HD __host__ __device__ __forceinline__
#else
#define XS_HD static inline
#endif

namespace xs {

constexpr int kFarLevels = 16;
constexpr int kFarEndBins = 256;  // widest tile a window end may cut; the narrowest has 64 points

// Far field of one condition (part of the uploaded condition record).
struct FarCond {
  int32_t on;      // 0: every line goes point by point
  int32_t lmax;    // levels 0..lmax
  int32_t end;     // level of the tiles that window ends cut
  int32_t sh;      // a leaf has 2^sh points
  int32_t n_fine;  // cells of the grid
  // cells whose windows all cover a tile [a, b) of leaves: b - cL <= f <= a + cR;
  // cells whose windows can touch it: a - xL <= f <= b + xR
  int32_t cR, cL, xR, xL;
  int32_t gap_max;
  int32_t glev;    // level of the tiles that share a gap: lmax, and at least 256 points
  int32_t v;       // cells of lines beyond either end of the grid
  int32_t span;    // cells between a wave's lines up to which the adjoint's far part pays
  int32_t mom;     // lowest level whose cells may take moments of the lines' Gaussians
  // gap of the tiles up to cell e: (gap0 + e gap1) / 2^32, at least one
  int64_t gap0, gap1;
};

struct CellRange {
  int32_t lo, hi;  // lo > hi: empty
};

XS_HD int32_t far_min(int32_t a, int32_t b) { return a < b ? a : b; }
XS_HD int32_t far_max(int32_t a, int32_t b) { return a > b ? a : b; }
XS_HD int32_t far_shl(int32_t a, int l) { return a * (1 << l); }  // a may be negative

XS_HD int32_t far_tiles(int32_t n_fine, int l) { return (n_fine + (1 << l) - 1) >> l; }

XS_HD int32_t far_gap(const FarCond& c, int l, int32_t t) {
  const int64_t e = (int64_t)((t >> (c.glev - l)) + 1) * ((int64_t)1 << c.glev);  // (t may be negative)
  const int64_t g = (c.gap0 + e * c.gap1) >> 32;
  return g < 1 ? 1 : g > c.gap_max ? c.gap_max : (int32_t)g;
}
XS_HD int32_t far_apart(int32_t gap, int l) { return 1 + ((gap + (1 << l) - 1) >> l); }

// Cells that tile t of level l admits on its left and on its right.
XS_HD CellRange far_left(const FarCond& c, int32_t gap, int l, int32_t t) {
  const int32_t hi = far_shl(t - far_apart(gap, l) + 1, l) - 1;
  const int32_t lo = l > c.end ? ((t + 1) << l) - c.cL : ((t >> (c.end - l)) << c.end) - c.xL;
  return CellRange{far_max(1 - c.v, lo), hi};
}
XS_HD CellRange far_right(const FarCond& c, int32_t gap, int l, int32_t t) {
  const int32_t lo = far_shl(t + far_apart(gap, l), l);
  const int32_t hi = l > c.end ? (t << l) + c.cR : (((t >> (c.end - l)) + 1) << c.end) + c.xR;
  return CellRange{lo, far_min(c.n_fine - 2 + c.v, hi)};
}

// The leaves near cell f, n0..n1 (gap grows by at most one from a tile of level
// glev to the next, so they are one range).
XS_HD void far_near(const FarCond& c, int32_t f, int32_t& n0, int32_t& n1) {
  const int32_t gap = far_gap(c, 0, f);
  n0 = f - gap;
  n1 = f + gap;
  while (n0 < f && n0 >= 0 && f - n0 > far_gap(c, 0, n0)) ++n0;
  while (n1 + 1 - f <= far_gap(c, 0, n1 + 1)) ++n1;
}

// a minus b as up to two ranges
XS_HD void far_subtract(CellRange a, CellRange b, CellRange& r0, CellRange& r1) {
  r0 = a;
  r1 = CellRange{0, -1};
  if (a.lo > a.hi || b.lo > b.hi || b.hi < a.lo || b.lo > a.hi) return;
  r0.hi = far_min(a.hi, b.lo - 1);
  r1 = CellRange{far_max(a.lo, b.hi + 1), a.hi};
}

// Cells of tile t of level `end` whose windows may end inside it (or before
// it): those on the left ([0]: the windows' upper ends) and on the right ([1]).
XS_HD void far_cut(const FarCond& c, int32_t t, CellRange r[2]) {
  const int32_t gap = far_gap(c, c.end, t);
  const CellRange a = far_left(c, gap, c.end, t), b = far_right(c, gap, c.end, t);
  r[0] = CellRange{a.lo, far_min(a.hi, ((t + 1) << c.end) - c.cL - 1)};
  r[1] = CellRange{far_max(b.lo, (t << c.end) + c.cR + 1), b.hi};
}

// The cells whose lines tile t of level l takes whole: admissible here, not
// for the parent, and not cut.  Up to four ranges (empty ones have lo > hi).
XS_HD void far_tile_ranges(const FarCond& c, int l, int32_t t, CellRange r[4]) {
  const CellRange none = {0, -1};
  const bool top = l >= c.lmax;
  const int32_t gap = far_gap(c, l, t);
  CellRange a = far_left(c, gap, l, t), b = far_right(c, gap, l, t);
  if (l == c.end) {
    a.lo = far_max(a.lo, ((t + 1) << l) - c.cL);
    b.hi = far_min(b.hi, (t << l) + c.cR);
  }
  far_subtract(a, top ? none : far_left(c, gap, l + 1, t >> 1), r[0], r[1]);
  far_subtract(b, top ? none : far_right(c, gap, l + 1, t >> 1), r[2], r[3]);
}

// Tiles of level l that may take lines of the cells [f0, f1] whole (a
// superset: far_tile_ranges decides), and those of level `end` that their
// windows may cut on the right ([0]) and on the left ([1]).
XS_HD CellRange far_candidates(const FarCond& c, int l, int32_t f0, int32_t f1) {
  int32_t lo, hi;
  if (l < c.end) {  // beside the parents that are not apart
    const int32_t k = 2 * far_apart(c.gap_max, l + 1) + 1;
    lo = (f0 >> l) - k;
    hi = (f1 >> l) + k;
  } else {
    lo = (f0 - c.cR) >> l;
    hi = (f1 + c.cL) >> l;
  }
  return CellRange{far_max(lo, 0), far_min(hi, far_tiles(c.n_fine, l) - 1)};
}
XS_HD void far_cut_candidates(const FarCond& c, int32_t f0, int32_t f1, CellRange r[2]) {
  const int32_t last = far_tiles(c.n_fine, c.end) - 1;
  r[0] = CellRange{far_max((f0 + c.cL) >> c.end, 0), far_min((f1 + c.xL) >> c.end, last)};
  r[1] = CellRange{far_max(((f0 - c.xR) >> c.end) - 1, 0), far_min((f1 - c.cR - 1) >> c.end, last)};
}

// Candidate cells of the leaves [a, b] (inside one tile of 256 points) for
// the point-by-point part, among the cells [clo, chi] whose windows can reach
// them: the cells near them, and the outermost ones.  Of the lines of segment 0,
// cell f's take the leaves within gap of f.
constexpr int kSegs = 3;
XS_HD void far_segments(const FarCond& c, int32_t a, int32_t b, int32_t clo, int32_t chi, CellRange s[kSegs]) {
  const int32_t first = -c.v, last = c.n_fine - 1 + c.v, gap = far_gap(c, 0, a);
  s[0] = CellRange{far_max(far_max(a - gap, clo), first + 1), far_min(far_min(b + gap, chi), last - 1)};
  s[1] = clo == first ? CellRange{first, first} : CellRange{0, -1};
  s[2] = chi == last ? CellRange{last, last} : CellRange{0, -1};
}

// Waves and rows.  A tile of 64 points or fewer is one wave's, one of 128 takes
// two, wider ones a block's four; above 512 points the tile's lines are cut
// into slices, a block and a row of coefficients each, so that no wave takes
// more than four times another's share.  (Blocks of four waves: one of eight
// fits a compute unit only once at three waves per SIMD.)
XS_HD int far_wide(int sh, int l) { return far_max(0, l + sh - 6); }  // log2 of points / 64, at least 0
XS_HD int32_t far_slices(int sh, int l) { return far_wide(sh, l) > 3 ? 1 << (far_wide(sh, l) - 3) : 1; }
XS_HD int64_t far_rows_before(int32_t n_fine, int sh, int l) {
  int64_t r = 0;
  for (int k = 0; k < l; ++k) r += (int64_t)far_tiles(n_fine, k) * far_slices(sh, k);
  return r;
}
// most levels a grid of n_fine cells can use (a tile two away must exist)
XS_HD int far_levels_of_grid(int32_t n_fine) {
  int l = 0;
  while (l < kFarLevels && (n_fine >> l) >= 3) ++l;
  return l;
}
// Cells beyond either end of a grid for windows that reach Wx points: all that they
// can touch, in whole tiles of level lmax, up to kFarVirtual (which bounds the
// table of cells: at 16 points to a cell windows of a million points).
// Measured, whole calls of Voigt spectra whose lines lie up to a cut-off of 25 cm^-1 beyond
// a grid of 50 cm^-1 (5001 points), gather / these lines point by point / cells of
// their own: 2e4 lines FP32 272 / 547 / 131 us, FP64 348 / 795 / 181; 1e6 lines FP32 2067 /
// 1616 / 530, FP64 2970 / 3356 / 1123; bin means of 2e5 lines FP32 1557 / 2094 / 343.
constexpr int32_t kFarVirtual = 1 << 16;
XS_HD int32_t far_virtual(int sh, int lmax, int64_t Wx) {
  const int64_t n = (Wx >> sh) + 2;
  const int64_t v = ((n >> lmax) + 1) << lmax;
  return v >= kFarVirtual ? kFarVirtual : (int32_t)v;
}
// Adjoint: a wave's lines go through tiles together, every tile of any of them, so its
// cost grows with the cells between its first and its last line; point by point it grows with
// the window alone.  The most cells that pay, for windows of W points.  Measured, the whole
// adjoint point by point / through tiles (Voigt, even lists, 2e5 points): FP32, window 1000, lines of a
// wave over 2, 4, 8, 16 cells 477 / 348, 330 / 267, 220 / 251, 215 / 290 us; window 2500, 16, 32, 48 cells
// 368 / 259, 381 / 328, 394 / 394; window 12500, 48 cells 1382 / 398; FP64 (cells of 64
// points), window 1000, 1, 2, 4 cells 551 / 417, 328 / 303, 244 / 290; window 2500, 4, 7, on 2e6
// points 8 cells 384 / 263, 353 / 286, 2604 / 1652.  A list of 3e5 lines in 100 cm^-1 and 100 over the other 19900,
// whose last waves see every tile of the grid: 1.1 / 23.5 ms.
XS_HD int32_t far_adj_span(int64_t W, bool f32) {
  const int64_t n = W < 800 ? 0 : (W - 800) / (f32 ? 36 : 170);
  return n > (1 << 30) ? 1 << 30 : (int32_t)n;
}
// Moments: one row per cell of every level, level after level; and the cells of
// level `l` or less that make up the leaves [lo, hi], one after the other: the
// widest that begins at lo.
XS_HD int64_t far_cells_before(int32_t n_fine, int l) {
  int64_t r = 0;
  for (int k = 0; k < l; ++k) r += far_tiles(n_fine, k);
  return r;
}
XS_HD int far_widest(int32_t lo, int32_t hi, int l) {
  int v = 0;
  while (v < l && (lo & ((2 << v) - 1)) == 0 && hi - lo >= (2 << v) - 1) ++v;
  return v;
}
// The lowest level whose tiles may take lines of half-widths up to gamma (in
// points) through moments: half a cell of it.
XS_HD int far_mom_level(int sh, double gamma) {
  int l = 0;
  while (l < kFarLevels && !(gamma <= 0.5 * (double)(1 << (sh + l)))) ++l;
  return l;
}
// The lowest level of whose cells a Gaussian's standard deviation sigma (in points) is at
// most `cells`: moments are held in these cells' widths, where the n-th of a
// Gaussian alone is sigma^n (n - 1)!!.  With 4 cells the 28 of the FP32 form stay
// below 2e31 a line (6 cells 1.5e36, 8 past FP32's range), with 2^16 the 48 of the
// FP64 form below 1e262.
constexpr double kMomSigma32 = 4.0, kMomSigma64 = 65536.0;
XS_HD int far_sigma_level(int sh, double sigma, double cells) {
  int l = 0;
  while (l < kFarLevels && !(sigma <= cells * (double)(1 << (sh + l)))) ++l;
  return l;
}
// blocks of a level: 4 >> far_wide tiles each, or one slice of one tile
XS_HD int32_t far_blocks(int32_t n_fine, int sh, int l) {
  const int w = far_wide(sh, l);
  return w < 2 ? (far_tiles(n_fine, l) + (4 >> w) - 1) / (4 >> w) : far_tiles(n_fine, l) * far_slices(sh, l);
}

// The far field of one condition: windows surely reach W points to each side
// of the home bin and at most Wx; a line at cell e (as a real number) is
// smooth from g0 + g1 e cells on.  `end` is the widest level (64 to
// kFarEndBins points) whose tiles a window end finds at least 18 half-widths
// away, with everything closer than far_apart covered: there few nodes serve
// (k_far.hip).  Off where no level does.
inline FarCond far_make(int64_t W, int64_t Wx, int32_t n_fine, int sh, double g0, double g1) {
  FarCond c = {};
  const int levels = far_levels_of_grid(n_fine);
  const int64_t leaf = (int64_t)1 << sh;
  // a tile's lines lie up to a window beyond the tile
  const double reach = (double)Wx / (double)leaf + 1.0;
  const double most = g0 + g1 * ((double)n_fine + reach);
  if (W < leaf || levels < 1 || !(most >= 0.0) || !(most + 1.0 <= (double)W / (double)leaf)) return c;
  // gap grows by at most one from a tile of level glev to the next
  if (!(g1 * (double)(256 >> sh) < 1.0)) return c;
  c.n_fine = n_fine;
  c.sh = sh;
  c.gap_max = (int32_t)most + 1;
  c.gap1 = (int64_t)(g1 * 4294967296.0) + 1;
  c.gap0 = (int64_t)((g0 + g1 * reach + 1.0) * 4294967296.0);
  c.cR = (int32_t)((W - leaf + 1) >> sh);
  c.cL = (int32_t)((W + 1) >> sh);
  c.xR = (int32_t)((Wx - 1) >> sh);
  c.xL = (int32_t)((Wx + leaf - 1) >> sh);
  int e = -1;
  for (int l = 0; (leaf << l) <= kFarEndBins && l < levels; ++l)
    if ((leaf << l) >= 64 && W >= 9 * (leaf << l) && W >= leaf * (int64_t)(far_apart(c.gap_max, l) << l)) e = l;
  if (e < 0) return c;
  c.end = e;
  c.lmax = e;
  while (c.lmax + 1 < levels && g1 * (double)(2 << c.lmax) < 1.0 && (far_apart(c.gap_max, c.lmax + 1) << (c.lmax + 1)) <= c.cR)
    ++c.lmax;
  c.glev = far_max(c.lmax, 8 - sh);
  c.on = 1;
  return c;
}

}  // namespace xs
