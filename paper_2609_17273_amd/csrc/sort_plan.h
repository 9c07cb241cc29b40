// Shape of the radix sort of the line keys and where its digit table lies:
// plain integer arithmetic, shared by the host runtime and the host tests.
#pragma once
#include <stdint.h>

namespace xs {

constexpr int kSortItems = 16;    // keys per thread in the radix sort (4096 per block)
constexpr int kSortBlock = 256 * kSortItems;
constexpr int kSortFew = 1 << 20;  // lines up to which 1024 keys make a block
constexpr int kColBlocks = 64;  // up to here a block adds the columns in less than the three scan kernels take
constexpr int kQBlocks = 256;     // partial sums per slot in the partition-function reduction

// Spaces of the workspace that may hold the table (int32 entries).
constexpr int64_t sort_hist_room(int64_t max_lines) { return 256 * ((max_lines + kSortBlock - 1) / kSortBlock); }
constexpr int64_t sort_rnu_room(int64_t max_lines) { return 2 * max_lines; }      // the records' nu, 8 bytes a line
constexpr int64_t sort_qpart_room(int64_t n_slots) { return 4 * n_slots * kQBlocks; }  // doubles [n_slots][2][kQBlocks]

enum { kSortInHist = 0, kSortInRnu = 1, kSortInQpart = 2, kSortNowhere = 3 };

struct SortPlan {
  int passes, rb;  // passes of rb bits
  bool few;        // 1024 keys a block (else kSortBlock)
  int nblk;
  int col;         // the scatter's blocks add up the digits' columns themselves: no scan, no scan sums
  int64_t entries; // digit table
  int place;       // where it lies
};

// The table's own space serves 8-bit digits of 4096 keys a block.  More entries
// lie where the records' nu are written after the sort, with the sums of the
// scan behind them if there is one (more than kColBlocks blocks); a single block
// of few lines, which that does not hold either, in the partition function's partial sums,
// which are read before the sort.  (Two blocks of 1024 digits, 2048 entries, always
// lie in nu: more than 1024 lines are 2050 entries or more.)
inline SortPlan sort_plan(int64_t n, int64_t max_key, int64_t max_lines, int64_t n_slots) {
  SortPlan p = {};
  int bits = 1;
  while ((1ll << bits) <= (long long)max_key) ++bits;
  p.passes = (bits + 9) / 10;
  p.rb = (bits + p.passes - 1) / p.passes;
  if (p.rb < 8) p.rb = 8;
  p.few = n <= kSortFew;
  const int64_t keys = p.few ? 1024 : kSortBlock;
  p.nblk = (int)((n + keys - 1) / keys);
  p.col = p.nblk <= kColBlocks;
  p.entries = (int64_t)p.nblk << p.rb;
  const int64_t sums = p.col ? 0 : p.entries / 1024 + 2;
  p.place = p.entries <= sort_hist_room(max_lines)          ? kSortInHist
            : p.entries + sums <= sort_rnu_room(max_lines) ? kSortInRnu
            : p.entries + sums <= sort_qpart_room(n_slots) ? kSortInQpart
                                                           : kSortNowhere;
  return p;
}

}  // namespace xs
