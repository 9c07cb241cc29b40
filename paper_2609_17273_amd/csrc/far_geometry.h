// Geometry of the far field of the profile pass: which grid tiles take a
// line's profile through Chebyshev expansions and which take it point by
// point.  Plain integer functions, shared by the kernels, the host runtime
// and the host tests.
//
// The grid is cut into leaves of 64 points (the sort's cells); a tile of level
// l is 2^l leaves.  Tile t of level l is apart from cell f (the lines with
// home bin / 64 = f) when at least one tile and at least `gap` cells lie
// between them: |(f >> l) - t| >= far_apart(l).  Leaves within `gap` cells of f
// are f's near leaves and take its lines point by point.  Of the others
//   - a tile of a level above `end` is admissible when it is apart and the
//     window of every line of the cell covers it;
//   - a tile of level l <= end when it is apart and the window of some line of
//     the cell can touch its ancestor of level `end`.
// A (tile, cell) pair belongs to the highest level at which it is admissible,
// so every leaf beyond the near ones that a window can touch takes a line
// through exactly one tile.  Only tiles of level `end` can be cut by a window
// end: their cells whose windows may end inside are set apart (far_cut), and
// their lines are added up to the window's end only.
// Cells 0 and n_fine - 1, which also hold the lines beyond the grid, go point
// by point over their whole windows.
#pragma once
#include <stdint.h>

#ifdef __HIPCC__
#define XS_HD __host__ __device__ __forceinline__
#else
#define XS_HD static inline
#endif

namespace xs {

constexpr int kFarLevels = 16;
constexpr int kLeafBins = 64;
constexpr int kFarEndMax = 2;  // widest tile a window end may cut: 256 points

// Far field of one condition (part of the uploaded condition record).
struct FarCond {
  int32_t on;      // 0: every line goes point by point
  int32_t lmax;    // levels 0..lmax
  int32_t end;     // level of the tiles that window ends cut
  int32_t gap;     // near leaves: |leaf - f| <= gap
  int32_t n_fine;  // cells of the grid
  // cells whose windows all cover a tile [a, b) of leaves: b - cL <= f <= a + cR;
  // cells whose windows can touch it: a - xL <= f <= b + xR
  int32_t cR, cL, xR, xL;
  int32_t pad;
};

struct CellRange {
  int32_t lo, hi;  // lo > hi: empty
};

XS_HD int32_t far_min(int32_t a, int32_t b) { return a < b ? a : b; }
XS_HD int32_t far_max(int32_t a, int32_t b) { return a > b ? a : b; }
XS_HD int32_t far_shl(int32_t a, int l) { return a * (1 << l); }  // a may be negative

XS_HD int32_t far_apart(const FarCond& c, int l) { return 1 + ((c.gap + (1 << l) - 1) >> l); }

// Cells that tile t of level l admits on its left and on its right.
XS_HD CellRange far_left(const FarCond& c, int l, int32_t t) {
  const int32_t hi = far_shl(t - far_apart(c, l) + 1, l) - 1;
  const int32_t lo = l > c.end ? ((t + 1) << l) - c.cL : ((t >> (c.end - l)) << c.end) - c.xL;
  return CellRange{far_max(1, lo), hi};
}
XS_HD CellRange far_right(const FarCond& c, int l, int32_t t) {
  const int32_t lo = far_shl(t + far_apart(c, l), l);
  const int32_t hi = l > c.end ? (t << l) + c.cR : (((t >> (c.end - l)) + 1) << c.end) + c.xR;
  return CellRange{lo, far_min(c.n_fine - 2, hi)};
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
  const CellRange a = far_left(c, c.end, t), b = far_right(c, c.end, t);
  r[0] = CellRange{a.lo, far_min(a.hi, ((t + 1) << c.end) - c.cL - 1)};
  r[1] = CellRange{far_max(b.lo, (t << c.end) + c.cR + 1), b.hi};
}

// The cells whose lines tile t of level l takes whole: admissible here, not
// for the parent, and not cut.  Up to four ranges (empty ones have lo > hi).
XS_HD void far_tile_ranges(const FarCond& c, int l, int32_t t, CellRange r[4]) {
  const CellRange none = {0, -1};
  const bool top = l >= c.lmax;
  CellRange a = far_left(c, l, t), b = far_right(c, l, t);
  if (l == c.end) {
    a.lo = far_max(a.lo, ((t + 1) << l) - c.cL);
    b.hi = far_min(b.hi, (t << l) + c.cR);
  }
  far_subtract(a, top ? none : far_left(c, l + 1, t >> 1), r[0], r[1]);
  far_subtract(b, top ? none : far_right(c, l + 1, t >> 1), r[2], r[3]);
}

// Candidate cells of the leaves [a, b] for the point-by-point part, among the
// cells [clo, chi] whose windows can reach them: the cells that have near
// leaves there, and the edge cells.
constexpr int kSegs = 3;
XS_HD void far_segments(const FarCond& c, int32_t a, int32_t b, int32_t clo, int32_t chi, CellRange s[kSegs]) {
  const int32_t last = c.n_fine - 1;
  s[0] = CellRange{far_max(far_max(a - c.gap, clo), 1), far_min(far_min(b + c.gap, chi), last - 1)};
  s[1] = clo == 0 ? CellRange{0, 0} : CellRange{0, -1};
  s[2] = chi == last ? CellRange{last, last} : CellRange{0, -1};
}

// Rows of expansion coefficients: level l has one row per tile and slice,
// slices = 2^(l - 3) above level 3 (a tile's lines are split so that no block
// takes more than eight waves' share).
XS_HD int32_t far_tiles(int32_t n_fine, int l) { return (n_fine + (1 << l) - 1) >> l; }
XS_HD int32_t far_slices(int l) { return l > 3 ? 1 << (l - 3) : 1; }
XS_HD int64_t far_rows_before(int32_t n_fine, int l) {
  int64_t r = 0;
  for (int k = 0; k < l; ++k) r += (int64_t)far_tiles(n_fine, k) * far_slices(k);
  return r;
}
// most levels a grid of n_fine cells can use (a tile two away must exist)
XS_HD int far_levels_of_grid(int32_t n_fine) {
  int l = 0;
  while (l < kFarLevels && (n_fine >> l) >= 3) ++l;
  return l;
}

// Blocks of eight waves: a block takes 8 >> l tiles of level l < 3, else one
// slice of one tile.
XS_HD int32_t far_blocks(int32_t n_fine, int l) {
  return l < 3 ? (far_tiles(n_fine, l) + (8 >> l) - 1) / (8 >> l) : far_tiles(n_fine, l) * far_slices(l);
}

// The far field of one condition: windows surely reach W points to each side
// of the home bin and at most Wx; the profile is smooth over a tile `gap`
// cells away.  `end` is the widest level (up to kFarEndMax) whose tiles a
// window end finds at least 18 half-widths away, with everything closer than
// far_apart covered: there few nodes serve (k_far.hip).  Off where no level
// does.
inline FarCond far_make(int64_t W, int64_t Wx, int32_t n_fine, int64_t gap) {
  FarCond c = {};
  const int levels = far_levels_of_grid(n_fine);
  if (W < kLeafBins || levels < 1 || gap < 1 || gap > W / kLeafBins) return c;
  c.n_fine = n_fine;
  c.gap = (int32_t)gap;
  c.cR = (int32_t)((W - 63) / 64);
  c.cL = (int32_t)((W + 1) / 64);
  c.xR = (int32_t)((Wx - 1) / 64);
  c.xL = (int32_t)((Wx + 63) / 64);
  int e = -1;
  for (int l = 0; l <= kFarEndMax && l < levels; ++l)
    if (W >= (int64_t)18 * (32 << l) && W >= (int64_t)64 * (far_apart(c, l) << l)) e = l;
  if (e < 0) return c;
  c.end = e;
  c.lmax = e;
  while (c.lmax + 1 < levels && (far_apart(c, c.lmax + 1) << (c.lmax + 1)) <= c.cR) ++c.lmax;
  c.on = 1;
  return c;
}

}  // namespace xs
