// Internal interface between the host runtime (xsec_api.cpp) and the HIP
// kernels (k_*.hip): device-side parameter blocks and launch wrappers.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/xsec.h"
#include "far_geometry.h"
#include "sort_plan.h"

namespace xs {

// CODATA 2018 exact SI values in CGS; c2 = h c / k_B (second radiation
// constant, symbol table of the paper).
constexpr double kH = 6.62607015e-27;      // erg s
constexpr double kC = 2.99792458e10;       // cm / s
constexpr double kKB = 1.380649e-16;       // erg / K
constexpr double kAMU = 1.66053906660e-24; // g
constexpr double kC2 = kH * kC / kKB;      // cm K
constexpr double kPI = 3.14159265358979323846;
constexpr double kLN2 = 0.69314718055994530942;

constexpr int kMaxCond = 256;
// The kind whose widths a profile uses: XS_BIN_x -> XS_x; pseudo-Voigts -> XS_VOIGT.
constexpr int base_profile(int profile) {
  return profile < 4 ? profile : (profile < 8 ? profile - 4 : 3);
}
constexpr int kItemsPerCU = 256;  // gather work items aimed at per compute unit when tiles are split
constexpr int kAdjBlocks = 16384;    // blocks of the adjoint's grid in a new plan
constexpr int kAdjBlocksMax = 32768;  // the most the configuration allows (sizes the partial sums)
// Device counters (int32): [0] gather work queue, [2..3] candidate total,
// [4..5] lines per item or part, [6] parts beyond
// tiles' first, [kFarOff] set by the
// record pass where more than kOddMax lines have values that are not finite (they then all go
// point by point), [kGammaMax..kNexpMax] largest
// |gamma_ref|, smallest and largest n_exp of the kept lines (floats), [kOddCount] how many such lines,
// [kOddHidden] whether their records are changed (OddLines).
constexpr int kCounterInts = 64;
constexpr int kFarOff = 9, kGammaMax = 10, kNexpMin = 11, kNexpMax = 12, kOddCount = 13, kOddHidden = 14;
// Lines are sorted by home bin >> sh: 64 points per key (the smallest bucket
// size), or the leaves of the tile expansions.
constexpr int kFineSh = 6;
// Leaves of 16 points (FP32 form) and 64 (FP64): smaller leaves leave fewer
// points to the near kernel and give the tiles a level more.  Measured near +
// tile kernels with 16 / 32 / 64 points, the tiles line by line: 1e7 lines FP32 3.45 / 3.90 / 4.02 ms,
// 48 conditions x 1e6 lines FP32 11.1 / 11.2 / 12.4; 1e6 lines FP64 2.28 /
// 1.79 / 1.61, 3.9e5 FP64 bin means 2.17 / 1.89 / 2.07 (20 nodes to a tile).
constexpr int kLeafSh32 = 4, kLeafSh64 = 6;

// Per-condition scalars, uploaded with the workspace.
struct CondDev {
  double T, P, Tv, Tr, cut;
  double Tk;      // kinetic temperature of the widths (T, or T_rot for two temperatures)
  double dop;     // Doppler HWHM per unit wavenumber: alpha = nu * dop (0 for fixed Gaussian)
  double hwhm;    // fixed Gaussian HWHM
  double lnTr;    // ln(T_ref / Tk)
  double pfac;    // P / P_ref
  int32_t slot;   // intensity slot (distinct T or (T_vib, T_rot))
  int32_t wbins;  // bound on |k - k_c| of a nonzero term: ceil(cut / dnu) + 2, less for a narrow Gaussian
  int32_t cclass; // cut-off class (index of the distinct cut-off)
  int32_t pad;
  FarCond far;    // tile expansions (Lorentzian and Voigt forms)
};

// Per intensity slot: the temperatures of the populations.
struct SlotDev {
  double T, Tv, Tr;
};

// Model and grid scalars shared by the kernels.
struct ModelDev {
  int32_t profile, mode, pop, prec;
  double nu0, dnu;
  int64_t n_bins;
  double T_ref, P_ref, hwhm_fixed, mass_amu;
  int32_t n_cond, n_slots;
  int32_t bucket_bins, n_buckets;  // lines bucketed by k_c / bucket_bins
  // Lines are sorted by the finer key k_c >> fine_sh (key n_fine = dropped),
  // whatever the bucket size, so that neighbouring sorted lines have nearly
  // equal home bins; a bucket is fine_per_bucket consecutive fine keys.  (With
  // tile expansions the keys begin fine_v cells before the grid and end as many
  // after it: see fine_v.)
  int32_t n_fine, fine_per_bucket, fine_sh;
  int32_t fine_v;                  // cells of lines beyond either end of the grid: keys (k_c >> fine_sh) + fine_v
  int32_t n_cut_classes;           // distinct cut-offs (window statistics)
  double max_cut;
};

constexpr int fine_keys(const ModelDev& m) { return m.n_fine + 2 * m.fine_v; }  // the key of dropped lines

// Views of the caller's inputs.
struct StatesView {
  int64_t n;
  const double* E;
  const double* g;
  const int32_t* v;
  const double* ev;
  int32_t n_v;
  const double* nv;  // vibronic densities (custom-density populations)
  const double* tau; // state lifetimes (s) for predissociation broadening, or null
};
struct LinesView {
  int64_t n;
  const int32_t* up;
  const int32_t* lo;
  const float* A;
  const float* gref;
  const float* nexp;
  const float* lscale;
  double gref_scalar, nexp_scalar;
};

// What the record pass takes of one line, packed by the first line pass in
// input order: that pass visits the lines in wavenumber order and so fetches one
// block per line instead of a cache line from each input array and state table.
// The factors are those of LineFac (k_common.h); ev, er, xv, xr only where the
// populations are not LTE's.
struct __attribute__((aligned(32))) LinePackLTE {
  double P, er, nu;
  float gref, nexp;
};
struct __attribute__((aligned(64))) LinePack {
  double P, ev, er, xv, xr, nu;
  float gref, nexp;
};

// With tile expansions: the kept lines whose values may be other than finite (no finite
// intensity in some slot, parameters of the width that are not, a Lorentzian of no width).
// Expansions would spread them over whole tiles, moments over a cell's lines, so a pass with
// expansions first gives their records no intensity and an ordinary width (saved here) and adds
// them point by point itself (k_near.hip); whatever else reads the records puts them back first.
constexpr int kOddMax = 1024;
struct OddLines {
  int32_t* pos;          // [kOddMax] sorted positions; null: a workspace without expansions
  float *gref, *nexp;    // [kOddMax]
  double* S;             // [kOddMax][n_slots]
};

// Workspace pointers (carved by the host runtime from the caller's buffer).
struct Work {
  CondDev* cond;            // [n_cond]
  SlotDev* slot;            // [n_slots]
  ModelDev* model;          // [1]
  double* qpart;            // [n_slots][2][kQBlocks]
  double* Q;                // [n_slots]
  double* dQ;               // [n_slots]
  unsigned long long* smax; // [n_slots] ordered keys of max ln|S|
  double* sb;               // [n_slots] log scale s_b (FP32 form)
  int32_t* key;             // [max_lines] bucket key per line
  int32_t* keyA;            // sort ping-pong
  int32_t* keyB;
  int32_t* valA;
  int32_t* valB;
  int32_t* hist;            // [sort_hist_room] digit table of the sort (sort_plan.h)
  int32_t* hsum;            // scan block sums
  int32_t* off;             // [fine_keys + 1] offsets of the cells (2^fine_sh grid points) into the sorted records
  double* rnu;              // sorted records: nu
  float* rgref;             //                 gamma_ref
  float* rnexp;             //                 n_exp
  double* rgpre;            //                 lifetime HWHM of the upper state, 1/(4 pi c tau) or 0
                            //                 (kernels get null when the states carry no lifetimes)
  int32_t* ridx;            //                 original line index
  double* rEs;              //                 energy of the state whose population enters S
                            //                 (lower: absorption, upper: emission; LTE adjoint)
  LinePack* lpack;          // [max_lines] line inputs in input order (first pass -> record pass)
  int32_t* rkc;             //                 home bin k_c = rint((nu - nu0)/dnu)
  float* rdel;              //                 nu - nu_{k_c}
  int32_t* rwin;            //                 [n_cut_classes][max_lines][2] window (klo, khi), klo > khi if empty
  void* rS;                 //                 S (f64) or S~ (f32), [n_slots][max_lines]
  int32_t* counter;         // [kCounterInts] work queues, candidate total, lines per item
  int32_t* item_cnt;        // [n_ct_max] candidate lines of each (tile, condition)
  int32_t* item_base;       // [n_ct_max + 1] work items of each (tile, condition), scanned
  int32_t* part_base;       // [n_ct_max + 1] partial rows of split tiles, scanned
  int32_t* item_sums;       // scan block sums
  double* part;             // [2 item_target][1024] partial rows
  int64_t item_target;      // work items aimed at when tiles are split
  int64_t far_cond_rows;    // rows of a condition's tile expansions at the most levels, 0: none.  The rows (and
                            // the adjoint's moments of the cotangent) lie in `part`, which the passes before them
                            // have done with, for as many conditions at a time as fit
  double* far_extra;        // or for one condition here, where the grid is too long for that (else null)
  OddLines odd;
  unsigned long long* stats;// [8]
  double* own;              // [4][n_slots] Q, dQ, sb and smax of partition functions and stick spectra
  double* adjpart;          // [n_cond][2][2 kAdjBlocksMax]: the near and the far part's blocks
  unsigned long long* gmax; // [n_cond] max |dL/dsigma| per condition (bits; FP32 adjoint's scale)
  double* cut_class;        // [n_cut_classes] distinct cut-offs
  int32_t* cut_mult;        // [n_cut_classes] conditions sharing each cut-off
  int64_t max_lines;
};

struct Tiling {
  int32_t tile_bins;   // bins per gather tile: 64 lanes x tile_bins / 64 bins each
  int32_t persistent;
  int32_t grid_blocks; // persistent grid size (one wave per block)
  int64_t chunk_lines; // requested candidate lines per work item (0: automatic)
  int32_t adj_blocks;  // persistent blocks of the adjoint
};

// Grids of many blocks: HIP takes less than 2^32 threads along x, so beyond 2^22 blocks
// the rest goes along z (up to 255 too many blocks, which find no work).
inline dim3 long_grid(int64_t blocks, int y = 1) {
  const int64_t x = blocks < 1 ? 1 : blocks < (1 << 22) ? blocks : (1 << 22);
  return dim3((unsigned)x, (unsigned)y, (unsigned)((blocks + x - 1) / x < 1 ? 1 : (blocks + x - 1) / x));
}
#ifdef __HIPCC__
__device__ __forceinline__ int long_block() { return (int)(blockIdx.z * gridDim.x + blockIdx.x); }
#endif

// ---- launch wrappers (k_lines.hip) ----
// clear > 0: also clears the first `clear` counters and the statistics, and packs
// the states for the line passes (kCounterInts: a preparation; kFarOff: a stick
// spectrum, which leaves the records of the last preparation and what belongs to them)
void launch_partition(const ModelDev& m, const Work& w, const StatesView& st, int clear, hipStream_t s);
void launch_lines_pass1(const ModelDev& m, const Work& w, const StatesView& st,
                        const LinesView& ln, hipStream_t s);
// Stable sort of the int32 keys w.key[0..n) (values 0..max_key) with their
// positions; returns the sorted keys and positions (ping-pong buffers), or false
// if the workspace has no room for the digit table (nothing enqueued).
bool launch_radix_sort(const ModelDev& m, const Work& w, int64_t n, int64_t max_key, hipStream_t s,
                       int32_t** sorted_keys, int32_t** sorted_vals);
void launch_offsets_records(const ModelDev& m, const Work& w, const StatesView& st,
                            const LinesView& ln, const int32_t* skeys, const int32_t* svals, hipStream_t s);
void launch_intensity_out(const ModelDev& m, const Work& w, const StatesView& st,
                          const LinesView& ln, void* S, double* log_scale, hipStream_t s);
void launch_q_out(const ModelDev& m, const Work& w, double* Q, double* dQ, hipStream_t s);
void launch_reset_queue(const Work& w, hipStream_t s);
void launch_scan_i32(int32_t* a, int64_t n, int32_t* sums, hipStream_t s);  // exclusive, in place

// ---- profile pass (k_profile.hip) ----
// (some: only the conditions without tile expansions)
void launch_gather(const ModelDev& m, const Work& w, const Tiling& t, double* sigma,
                   int accumulate, bool some, hipStream_t s);
void launch_scatter(const ModelDev& m, const Work& w, double* sigma, int accumulate,
                    int64_t n_lines, hipStream_t s);

// ---- near leaves (k_near.hip) ----
inline int64_t part_doubles(const Work& w) { return 2 * w.item_target * 1024; }  // of Work::part
size_t near_row_doubles();  // what it takes of Work::part
// sigma = (or +=) the points near each line, for the conditions with tile
// expansions, and every point of the others (rest: which are the gather's)
void launch_near(const ModelDev& m, const Work& w, double* sigma, int accumulate, bool rest, int64_t n_lines,
                 hipStream_t s);

// ---- tile expansions (k_far.hip) ----
int far_nodes(int prec);  // nodes per tile
int far_moments(int prec);  // moments per cell
// sigma += the expansions of the lines' far tiles (levels up to far_lmax, the
// conditions' largest)
// (end_min: the conditions' lowest level of cut tiles)
void launch_far(const ModelDev& m, const Work& w, int far_lmax, int end_min, int64_t n_lines, double* sigma,
                hipStream_t s);

// ---- cooling function (k_cooling.hip) ----
// doubles of Work::part the temperatures and partial sums take
int64_t cooling_doubles(int32_t nT);
// false: no room for the sort (as launch_radix_sort)
bool launch_cooling(const ModelDev& m, const Work& w, const StatesView& st, const LinesView& ln,
                    const double* T_dev, int32_t nT, double* W, double* Q, hipStream_t s);

// ---- adjoint (k_adjoint.hip) ----
// far_lmax, end_min: as launch_far's; far_lmax < 0: every window point by point
constexpr int kCutRowBins = 16;  // grid points per row of moments of the parts of cut tiles
// doubles of Work::part (or Work::far_extra) that one condition takes, of rows tile rows;
// kAdjTail doubles at the end of Work::part are left to the caller
constexpr int kAdjTail = 2 * kMaxCond;
int64_t adj_far_doubles(const ModelDev& m, int64_t rows);
void launch_adjoint(const ModelDev& m, const Work& w, const StatesView& st, const LinesView& ln,
                    const double* g, double* dT, double* dP, double* dgref, double* dnexp,
                    double* dls, int64_t n_lines, int adj_blocks, int far_lmax, int end_min, hipStream_t s);

}  // namespace xs
