// Host wrappers of far_geometry.h for the tests.
#include "../paper_2609_17273_amd/csrc/far_geometry.h"
using namespace xs;
extern "C" {
// how often cell f's lines reach each leaf of [0, n_fine): whole, through a
// tile (far[leaf]); through a tile that the window may cut (cut[leaf]); point
// by point through the segments of the rows of row_leaves leaves
// (direct[leaf]).  gap[leaf]: cells that are near the leaf; info: on, points of
// a cut tile, the near leaves of the cell, tiles missing from the candidates of
// the cells [f, f + 2].
int far_count(int64_t W, int64_t Wx, int32_t n_fine, int32_t sh, double g0, double g1, int32_t row_leaves, int32_t f,
              int32_t reach, int32_t* far, int32_t* cut, int32_t* direct, int32_t* gap, int32_t* info) {
  const FarCond c = far_make(W, Wx, n_fine, sh, g0, g1);
  for (int i = 0; i < n_fine; ++i) {
    far[i] = cut[i] = direct[i] = 0;
    gap[i] = c.on ? far_gap(c, 0, i) : 0;
  }
  info[0] = c.on;
  info[1] = c.on ? 1 << (c.sh + c.end) : 0;
  info[2] = info[3] = info[4] = 0;
  if (c.on) far_near(c, f, info[2], info[3]);
  if (c.on)
    for (int l = 0; l <= c.lmax; ++l)
      for (int t = 0; t < far_tiles(n_fine, l); ++t) {
        CellRange r[4], e[2];
        far_tile_ranges(c, l, t, r);
        const CellRange cand = far_candidates(c, l, f, f + 2);
        for (auto& q : r)
          if (q.lo <= q.hi && q.lo <= f + 2 && q.hi >= f && (t < cand.lo || t > cand.hi)) info[4]++;
        for (auto& q : r)
          if (q.lo <= f && f <= q.hi)
            for (int leaf = t << l; leaf < ((t + 1) << l) && leaf < n_fine; ++leaf) far[leaf]++;
        if (l != c.end) continue;
        far_cut(c, t, e);
        CellRange cc[2];
        far_cut_candidates(c, f, f + 2, cc);
        for (int k = 0; k < 2; ++k)
          if (e[k].lo <= e[k].hi && e[k].lo <= f + 2 && e[k].hi >= f && (t < cc[k].lo || t > cc[k].hi)) info[4]++;
        for (auto& q : e)
          if (q.lo <= f && f <= q.hi)
            for (int leaf = t << l; leaf < ((t + 1) << l) && leaf < n_fine; ++leaf) cut[leaf]++;
      }
  for (int a = 0; a < n_fine; a += row_leaves) {
    const int b = a + row_leaves - 1;
    int clo = a - reach, chi = b + reach;
    if (clo < 0) clo = 0;
    if (chi > n_fine - 1) chi = n_fine - 1;
    CellRange s[kSegs] = {{clo, chi}, {0, -1}, {0, -1}};
    if (c.on) far_segments(c, a, b, clo, chi, s);
    const int g = c.on ? far_gap(c, 0, a) : 0;
    for (int k = 0; k < kSegs; ++k) {
      if (f < s[k].lo || f > s[k].hi) continue;
      const bool near = c.on && k == 0;
      for (int leaf = a; leaf <= b && leaf < n_fine; ++leaf)
        if (!near || (leaf >= f - g && leaf <= f + g)) direct[leaf]++;
    }
  }
  return c.on;
}
}
