// Line-side kernels: partition functions, the intensity pass, bucketing of
// lines by home bin (stable LSD radix sort) and the sorted line records.
#include <algorithm>

#include "k_common.h"

namespace xs {

// ---------------------------------------------------------------------------
// Partition functions, Eq. (pf): Q(T) = sum_n g_n exp(-c2 E_n / T) and
// dQ/dT = sum_n g_n (c2 E_n / T^2) exp(-c2 E_n / T); two temperatures,
// Eq. (Q nlte 2T), with E_rot = E - E_vib(v).  FP64, deterministic two-stage
// tree reduction (per-block partials, then one block per slot).
// ---------------------------------------------------------------------------
__device__ __forceinline__ double block_sum256(double v, double* sh) {
  const int tid = threadIdx.x;
  sh[tid] = v;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (tid < s) sh[tid] += sh[tid + s];
    __syncthreads();
  }
  double r = sh[0];
  __syncthreads();
  return r;
}

// Per-state record for the first line pass: one random load per state of a
// line instead of one per table (energies, degeneracies, manifold index and
// energy).  Built once per prepare into the sort's second ping-pong buffers,
// which are free until the sort's last pass; lists with more states than that
// space holds read the tables directly.
struct __attribute__((aligned(16))) StatePackLTE {
  double E, g;
};
struct __attribute__((aligned(32))) StatePackNLTE {
  double E, g, ev;  // ev: E_vib of the state's manifold
  int64_t vi;       // manifold index, or -1 when outside the table
};

// With pack or clear set it also writes the state records and clears the
// per-call counters, so that preparing lines starts with one kernel, not three
// (a kernel of a few microseconds each where lists are short).
__global__ __launch_bounds__(256) void k_partition(ModelDev m, const SlotDev* slots, StatesView st, double* qpart,
                                                   void* pack, int clear, int32_t* counter,
                                                   unsigned long long* stats) {
  __shared__ double sh[256];
  const int slot = blockIdx.y;
  const SlotDev sd = slots[slot];
  if (slot != 0) pack = nullptr;
  if (clear && slot == 0 && blockIdx.x == 0) {
    for (int q = threadIdx.x; q < clear; q += 256) counter[q] = 0;
    if (threadIdx.x < 8) stats[threadIdx.x] = 0ull;
  }
  double q = 0.0, dq = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < st.n; i += (int64_t)gridDim.x * 256) {
    const double E = st.E[i], g = st.g[i];
    if (m.pop == XS_LTE) {
      if (pack) ((StatePackLTE*)pack)[i] = StatePackLTE{E, g};
      const double b = g * exp(-kC2 * E / sd.T);
      q += b;
      dq += b * (kC2 * E / (sd.T * sd.T));
    } else {
      const int32_t vi = st.v[i];
      const bool ok = (uint32_t)vi < (uint32_t)st.n_v;
      const double ev = ok ? st.ev[vi] : 0.0;
      if (pack) ((StatePackNLTE*)pack)[i] = StatePackNLTE{E, g, ev, ok ? (int64_t)vi : -1};
      if (ok) {  // states with an invalid manifold index are skipped
        if (m.pop == XS_NLTE_2T) {
          q += g * exp(-kC2 * ev / sd.Tv - kC2 * (E - ev) / sd.Tr);
        } else {  // custom vibronic densities, Eq. (Q nlte Nvib)
          const double w = st.nv[vi];
          if (w > 0.0) q += g * w * exp(-kC2 * (E - ev) / sd.Tr);
        }
      }
    }
  }
  q = block_sum256(q, sh);
  dq = block_sum256(dq, sh);
  if (threadIdx.x == 0) {
    qpart[(slot * 2 + 0) * kQBlocks + blockIdx.x] = q;
    qpart[(slot * 2 + 1) * kQBlocks + blockIdx.x] = dq;
  }
}

__global__ __launch_bounds__(256) void k_partition_final(ModelDev m, const double* qpart,
                                                         double* Q, double* dQ,
                                                         unsigned long long* smax) {
  __shared__ double sh[256];
  const int slot = blockIdx.x;
  double q = block_sum256(qpart[(slot * 2 + 0) * kQBlocks + threadIdx.x], sh);
  double dq = block_sum256(qpart[(slot * 2 + 1) * kQBlocks + threadIdx.x], sh);
  if (threadIdx.x == 0) {
    Q[slot] = q;
    dQ[slot] = (m.pop == XS_LTE) ? dq : __longlong_as_double(0x7ff8000000000000ll);
    smax[slot] = 0ull;  // reset the running max of ln|S| for the intensity pass
  }
}

// Where the packed state table goes: the sort's second ping-pong buffers (keyB,
// valB: adjacent), or nowhere when it does not fit there.
static void* state_pack(const ModelDev& m, const Work& w, const StatesView& st) {
  const size_t rec = (m.pop == XS_LTE) ? sizeof(StatePackLTE) : sizeof(StatePackNLTE);
  const size_t room = (size_t)((const char*)w.valB - (const char*)w.keyB) + 4 * (size_t)w.max_lines;
  return (size_t)st.n * rec <= room && ((uintptr_t)w.keyB % 32) == 0 ? (void*)w.keyB : nullptr;
}

void launch_partition(const ModelDev& m, const Work& w, const StatesView& st, int clear, hipStream_t s) {
  hipLaunchKernelGGL(k_partition, dim3(kQBlocks, m.n_slots), dim3(256), 0, s, m, w.slot, st, w.qpart,
                     clear ? state_pack(m, w, st) : (void*)nullptr, clear, w.counter, w.stats);
  hipLaunchKernelGGL(k_partition_final, dim3(m.n_slots), dim3(256), 0, s, m, w.qpart, w.Q, w.dQ,
                     w.smax);
}

__global__ void k_q_out(ModelDev m, const CondDev* cond, const double* Q, const double* dQ,
                        double* Qo, double* dQo) {
  const int c = threadIdx.x;
  if (c < m.n_cond) {
    Qo[c] = Q[cond[c].slot];
    if (dQo) dQo[c] = dQ[cond[c].slot];
  }
}

void launch_q_out(const ModelDev& m, const Work& w, double* Q, double* dQ, hipStream_t s) {
  hipLaunchKernelGGL(k_q_out, dim3(1), dim3(256), 0, s, m, w.cond, w.Q, w.dQ, Q, dQ);
}

// ---------------------------------------------------------------------------
// Intensity pass 1: nu_i = E_u - E_l; keep lines with nu > 0 whose window
// (widest cut-off) reaches the grid; key = k_c >> fine_sh for the home bin
// k_c = rint((nu - nu0)/dnu), clamped to the grid (lines past either end
// keep their wings, section "Spectral synthesis") and the fine_v cells beyond it; dropped
// lines get key fine_keys.  FP32 form: running max of ln|S| per slot.  Counters:
// kept lines and window pairs (exact windows per distinct cut-off).
// ---------------------------------------------------------------------------
// The states of one line, read once: from the packed table, or from the
// caller's tables.  ok: both indices (and, non-LTE, both manifolds) inside
// the tables.
template <int MODE, bool LTE>
__device__ __forceinline__ bool gather_line_states(const ModelDev& m, const StatesView& st, const void* pack,
                                                   int32_t u, int32_t l, LineState& ls) {
  int32_t vu = 0, vl = 0;
  if ((uint32_t)u >= (uint64_t)st.n || (uint32_t)l >= (uint64_t)st.n) return false;
  if (LTE) {
    if (MODE) {
      const StatePackLTE a = ((const StatePackLTE*)pack)[u], b = ((const StatePackLTE*)pack)[l];
      ls.Eu = a.E;
      ls.gu = a.g;
      ls.El = b.E;
    } else {
      ls.Eu = st.E[u];
      ls.gu = st.g[u];
      ls.El = st.E[l];
    }
    ls.evu = ls.evl = 0.0;
  } else {
    if (MODE) {
      const StatePackNLTE a = ((const StatePackNLTE*)pack)[u], b = ((const StatePackNLTE*)pack)[l];
      if (a.vi < 0 || b.vi < 0) return false;
      ls.Eu = a.E;
      ls.gu = a.g;
      ls.evu = a.ev;
      ls.El = b.E;
      ls.evl = b.ev;
      vu = (int32_t)a.vi;
      vl = (int32_t)b.vi;
    } else {
      vu = st.v[u];
      vl = st.v[l];
      if ((uint32_t)vu >= (uint32_t)st.n_v || (uint32_t)vl >= (uint32_t)st.n_v) return false;
      ls.Eu = st.E[u];
      ls.gu = st.g[u];
      ls.El = st.E[l];
      ls.evu = st.ev[vu];
      ls.evl = st.ev[vl];
    }
  }
  if (!LTE && m.pop == XS_NLTE_DENSITY) {
    ls.nvu = st.nv[vu];
    ls.nvl = st.nv[vl];
  } else {
    ls.nvu = ls.nvl = 1.0;
  }
  return true;
}

// Totals over the lines: kept lines, window pairs, lines with bad indices.
// Every block writes its own to part[value][block] and k_line_totals adds them: an
// atomic per block on one address costs 12 ns whoever waits, and 8192 blocks with
// 3 counters each bound shorter lists (1.1e6 lines 206 -> 65 us without them).
constexpr int kPass1Blocks = 2048;

struct Totals {
  unsigned long long kept = 0, pairs = 0, bad = 0;
};
__device__ __forceinline__ unsigned long long wave_sum(unsigned long long v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
// sh: [12]
__device__ __forceinline__ void block_totals(const Totals& t, unsigned long long* sh, unsigned long long* part) {
  const unsigned long long a = wave_sum(t.kept), b = wave_sum(t.pairs), c = wave_sum(t.bad);
  if ((threadIdx.x & 63) == 0) {
    sh[threadIdx.x >> 6] = a;
    sh[4 + (threadIdx.x >> 6)] = b;
    sh[8 + (threadIdx.x >> 6)] = c;
  }
  __syncthreads();
  if (threadIdx.x < 3) {
    const unsigned long long* r = sh + 4 * threadIdx.x;
    part[(int64_t)threadIdx.x * gridDim.x + blockIdx.x] = r[0] + r[1] + r[2] + r[3];
  }
}

// The exact windows of a kept line, over the conditions; [a, b]: its window at
// the widest cut-off.
__device__ __forceinline__ unsigned long long window_pairs(const ModelDev& m, const double* cutc, const int32_t* cutm,
                                                           double nu, int64_t a, int64_t b) {
  if (m.n_cut_classes == 1 && cutc[0] == m.max_cut)
    return (unsigned long long)(b - a + 1) * (unsigned long long)cutm[0];
  unsigned long long pairs = 0;
#pragma unroll 1
  for (int q = 0; q < m.n_cut_classes; ++q)
    if (line_window(nu, cutc[q], m.nu0, m.dnu, m.n_bins, a, b))
      pairs += (unsigned long long)(b - a + 1) * (unsigned long long)cutm[q];
  return pairs;
}

__device__ __forceinline__ void put_pack(LinePackLTE* p, const LineFac& f, double nu, float gref, float nexp) {
  *p = LinePackLTE{f.P, f.er, nu, gref, nexp};
}
__device__ __forceinline__ void put_pack(LinePack* p, const LineFac& f, double nu, float gref, float nexp) {
  *p = LinePack{f.P, f.ev, f.er, f.xv, f.xr, nu, gref, nexp};
}
__device__ __forceinline__ LineFac pack_fac(const LinePackLTE& p) { return LineFac{p.P, 0.0, p.er, 0.0, p.nu}; }
__device__ __forceinline__ LineFac pack_fac(const LinePack& p) { return LineFac{p.P, p.ev, p.er, p.xv, p.xr}; }
template <bool LTE>
struct PackOf {
  using type = LinePack;
};
template <>
struct PackOf<true> {
  using type = LinePackLTE;
};

// MODE 1: states from the packed table; 0: from the caller's tables.  REC: write
// the sort keys and line packs (a stick spectrum in the FP32 form needs only
// the totals).  Bound by memory: a line's two random state loads miss the L2 where
// the table is larger (64 bytes each), and its pack is written and read once
// more (1e7 lines, 3e5 states: 1.2 GB fetched, 397 us; 588 with logarithms and
// packs of 64 bytes, the record pass 307, before 435).
template <int MODE, bool REC, bool LTE>
__global__ __launch_bounds__(256) void k_lines_pass1(ModelDev m, const SlotDev* slots,
                                                     const double* Q, const double* cutc,
                                                     const int32_t* cutm, StatesView st, const void* spack,
                                                     LinesView ln, int32_t* key,
                                                     void* lpack,
                                                     unsigned long long* smax,
                                                     unsigned long long* part) {
  __shared__ SlotFac sf[kMaxCond];
  __shared__ unsigned long long bmax[kMaxCond];  // the block's largest ln|S| of every slot (FP32 form)
  __shared__ unsigned long long scnt[12];
  const bool f32 = m.prec == XS_FP32;
  if (f32)
    for (int q = threadIdx.x; q < m.n_slots; q += 256) {
      sf[q] = slot_fac(slots[q], m.pop, Q[q], 0.0);
      bmax[q] = 0ull;
    }
  __syncthreads();
  Totals tot;
  float gmax = 0.0f, nlo = INFINITY, nhi = -INFINITY;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < ln.n; i += (int64_t)gridDim.x * 256) {
    const int32_t u = ln.up[i], l = ln.lo[i];
    int32_t kk = fine_keys(m);
    LineState ls;
    if (!gather_line_states<MODE, LTE>(m, st, spack, u, l, ls)) {
      ++tot.bad;
      if (REC) key[i] = kk;
      continue;
    }
    const double nu = ls.Eu - ls.El;
    int64_t a, b;
    if (nu > 0.0 && line_window(nu, m.max_cut, m.nu0, m.dnu, m.n_bins, a, b)) {
      ++tot.kept;
      const LineFac f = line_fac(m.mode, LTE ? XS_LTE : m.pop, ls, (double)ln.A[i], nu);
      if (REC) {
        int64_t kc = home_bin(nu, m.nu0, m.dnu);
        const int64_t fk = (kc >> m.fine_sh) + m.fine_v;
        kk = (int32_t)(fk < 0 ? 0 : fk < fine_keys(m) - 1 ? fk : fine_keys(m) - 1);
        const float gref = ln.gref ? ln.gref[i] : (float)ln.gref_scalar;
        const float nexp = ln.nexp ? ln.nexp[i] : (float)ln.nexp_scalar;
        if (isfinite(gref) && isfinite(nexp)) {  // (others: OddLines)
          gmax = fmaxf(gmax, fabsf(gref));
          nlo = fminf(nlo, nexp);
          nhi = fmaxf(nhi, nexp);
        }
        put_pack((typename PackOf<LTE>::type*)lpack + i, f, nu, gref, nexp);
      }
      tot.pairs += window_pairs(m, cutc, cutm, nu, a, b);
      if (f32) {
        const double sc = ln.lscale ? (double)ln.lscale[i] : 0.0;
#pragma unroll 1
        for (int q = 0; q < m.n_slots; ++q) {
          const double lS = intensity_log(intensity<LTE>(m.mode, m.pop, f, sf[q]), sf[q], sc);
          // (a stale maximum only costs an atomic that changes nothing)
          if (lS > -INFINITY && dbl_key(lS) > bmax[q]) atomicMax(&bmax[q], dbl_key(lS));
        }
      }
    }
    if (REC) key[i] = kk;
  }
  block_totals(tot, scnt, part);  // (and a barrier)
  if (REC) {
    __shared__ float sext[4][3];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      gmax = fmaxf(gmax, __shfl_xor(gmax, o, 64));
      nlo = fminf(nlo, __shfl_xor(nlo, o, 64));
      nhi = fmaxf(nhi, __shfl_xor(nhi, o, 64));
    }
    if ((threadIdx.x & 63) == 0) {
      float* e = sext[threadIdx.x >> 6];
      e[0] = gmax;
      e[1] = nlo;
      e[2] = nhi;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
      float r = sext[0][threadIdx.x];
      for (int v = 1; v < 4; ++v) {
        const float x = sext[v][threadIdx.x];
        r = threadIdx.x == 1 ? fminf(r, x) : fmaxf(r, x);
      }
      ((float*)(part + 3 * (int64_t)gridDim.x))[(int64_t)threadIdx.x * gridDim.x + blockIdx.x] = r;
    }
  }
  if (f32)
    for (int q = threadIdx.x; q < m.n_slots; q += 256)
      if (bmax[q] > __hip_atomic_load(smax + q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(smax + q, bmax[q]);
}

// Adds the blocks' totals, and sets the FP32 form's scale of every slot.
// (rec: and the extremes of the lines' widths)
__global__ __launch_bounds__(512) void k_line_totals(ModelDev m, const unsigned long long* part, int blocks, int rec,
                                                     const unsigned long long* smax, double* sb,
                                                     unsigned long long* stats, int32_t* counter) {
  const int v = threadIdx.x >> 6, lane = threadIdx.x & 63;  // a wave per value
  if (rec && v >= 4 && v < 7) {
    const float* e = (const float*)(part + 3 * (int64_t)blocks) + (int64_t)(v - 4) * blocks;
    float r = v == 5 ? INFINITY : -INFINITY;
#pragma unroll 8
    for (int b = lane; b < blocks; b += 64) r = v == 5 ? fminf(r, e[b]) : fmaxf(r, e[b]);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      const float x = __shfl_xor(r, o, 64);
      r = v == 5 ? fminf(r, x) : fmaxf(r, x);
    }
    if (lane == 0) ((float*)counter)[kGammaMax + v - 4] = r;
  }
  if (v < 3) {
    unsigned long long r = 0;
#pragma unroll 8
    for (int b = lane; b < blocks; b += 64) r += part[(int64_t)v * blocks + b];
    r = wave_sum(r);
    if (lane == 0) stats[1 + v] = r;
  }
  if (threadIdx.x < m.n_slots) sb[threadIdx.x] = smax[threadIdx.x] ? key_dbl(smax[threadIdx.x]) : 0.0;
}

static int line_blocks(int64_t n) { return (int)std::max<int64_t>(1, std::min<int64_t>(kPass1Blocks, (n + 255) / 256)); }

// The blocks' totals go to keyA, free until the sort's first pass: 36 bytes a
// block, which has 256 lines (the last fewer; the carve is at least 256 bytes).
static unsigned long long* totals_part(const Work& w) { return reinterpret_cast<unsigned long long*>(w.keyA); }
static void line_totals(const ModelDev& m, const Work& w, int64_t n, bool rec, hipStream_t s) {
  hipLaunchKernelGGL(k_line_totals, dim3(1), dim3(512), 0, s, m, totals_part(w), line_blocks(n), (int)rec, w.smax,
                     w.sb, w.stats, w.counter);
}

template <bool REC>
static void pass1(const ModelDev& m, const Work& w, const StatesView& st, const LinesView& ln, hipStream_t s) {
  const void* pack = state_pack(m, w, st);
  const bool lte = m.pop == XS_LTE;
  auto* const k = pack ? (lte ? k_lines_pass1<1, REC, true> : k_lines_pass1<1, REC, false>)
                       : (lte ? k_lines_pass1<0, REC, true> : k_lines_pass1<0, REC, false>);
  hipLaunchKernelGGL(k, dim3(line_blocks(ln.n)), dim3(256), 0, s, m, w.slot, w.Q, w.cut_class, w.cut_mult, st, pack,
                     ln, w.key, (void*)w.lpack, w.smax, totals_part(w));
}

void launch_lines_pass1(const ModelDev& m, const Work& w, const StatesView& st,
                        const LinesView& ln, hipStream_t s) {
  pass1<true>(m, w, st, ln, s);
  line_totals(m, w, ln.n, true, s);
}

// ---------------------------------------------------------------------------
// Stable LSD radix sort of the bucket keys, RB = 8, 9 or 10 bits per pass: as
// few passes as 10 bits allow, the bits shared out evenly (17-bit keys of 1e7
// lines: 3 passes of 8 bits 370 us, 2 of 9 225).  Each block owns
// 256 ITEMS consecutive keys: 4096, or 1024 where that leaves compute units idle.
// Pass: (1) per-block digit histogram; (2) exclusive scan of the digit-major
// [digits][blocks] table, or with few blocks none (COL: block-major table, every
// scatter block adds up its digits' columns itself); (3) stable scatter.
// Stability makes the sorted order, and so every later summation order,
// deterministic.
// ---------------------------------------------------------------------------
template <int RB, int ITEMS>
__global__ __launch_bounds__(256) void k_sort_hist(const int32_t* keys, int64_t n, int shift,
                                                   int32_t* hist, int nblk, int col) {
  constexpr int ND = 1 << RB;
  __shared__ int h[ND];
  for (int d = threadIdx.x; d < ND; d += 256) h[d] = 0;
  __syncthreads();
  const int64_t base = (int64_t)blockIdx.x * (256 * ITEMS);
  int k[ITEMS];
#pragma unroll
  for (int s = 0; s < ITEMS; ++s) {
    const int64_t i = base + s * 256 + threadIdx.x;
    k[s] = i < n ? keys[i] : 0;
  }
#pragma unroll
  for (int s = 0; s < ITEMS; ++s)
    if (base + s * 256 + threadIdx.x < n) atomicAdd(&h[(k[s] >> shift) & (ND - 1)], 1);
  __syncthreads();
  for (int d = threadIdx.x; d < ND; d += 256)
    hist[col ? (int64_t)blockIdx.x * ND + d : (int64_t)d * nblk + blockIdx.x] = h[d];
}

// Exclusive scan of int32 arrays: per-block scan of 1024 elements, block sums
// scanned by one block, then added back.
// sh: [4]
__device__ __forceinline__ int block_excl_scan256(int v, int* sh, int& total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int incl = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int t = __shfl_up(incl, o, 64);
    if (lane >= o) incl += t;
  }
  if (lane == 63) sh[wave] = incl;
  __syncthreads();
  const int s0 = sh[0], s1 = sh[1], s2 = sh[2], s3 = sh[3];
  total = s0 + s1 + s2 + s3;
  __syncthreads();
  return incl - v + (wave > 0 ? s0 : 0) + (wave > 1 ? s1 : 0) + (wave > 2 ? s2 : 0);
}

__global__ __launch_bounds__(256) void k_scan_blocks(int32_t* a, int64_t n, int32_t* sums) {
  __shared__ int sh[4];
  const int64_t base = (int64_t)blockIdx.x * 1024 + threadIdx.x * 4;
  int v[4], s = 0;
  for (int j = 0; j < 4; ++j) {
    v[j] = (base + j < n) ? a[base + j] : 0;
    s += v[j];
  }
  int total;
  int ex = block_excl_scan256(s, sh, total);
  for (int j = 0; j < 4; ++j) {
    if (base + j < n) a[base + j] = ex;
    ex += v[j];
  }
  if (threadIdx.x == 0) sums[blockIdx.x] = total;
}

__global__ __launch_bounds__(256) void k_scan_sums(int32_t* sums, int64_t n) {
  __shared__ int sh[4];
  int carry = 0;
  for (int64_t b0 = 0; b0 < n; b0 += 256) {
    const int64_t i = b0 + threadIdx.x;
    int v = i < n ? sums[i] : 0;
    int total;
    int ex = block_excl_scan256(v, sh, total);
    if (i < n) sums[i] = ex + carry;
    carry += total;
  }
}

__global__ __launch_bounds__(256) void k_scan_add(int32_t* a, int64_t n, const int32_t* sums) {
  const int64_t base = (int64_t)blockIdx.x * 1024 + threadIdx.x * 4;
  const int add = sums[blockIdx.x];
  for (int j = 0; j < 4; ++j)
    if (base + j < n) a[base + j] += add;
}

// Stable scatter of one pass, staged through LDS: the block places its keys
// in digit order in LDS, then writes each digit's run to its global place, so
// neighbouring threads write neighbouring addresses.  Every wave owns 64 ITEMS
// consecutive keys and ranks them by itself, against its own counts: the rank
// of a key among its wave's equal digits is the count so far + the number of
// earlier lanes with the same digit (RB ballots); no step waits for another
// wave (one block of 4096 keys: 15.5 us with three barriers a step, now
// 5.3 with 1024 a block).  offs: the scanned table, or with col the counts.
template <int RB, int ITEMS>
__global__ __launch_bounds__(256) void k_sort_scatter(const int32_t* keys, const int32_t* vals,
                                                      int64_t n, int shift, const int32_t* offs,
                                                      int nblk, int col, int32_t* okeys, int32_t* ovals) {
  constexpr int ND = 1 << RB, PT = ND / 256;  // PT: digits per thread
  __shared__ int wc[4][ND];     // the waves' counts, then the positions of their first keys
  __shared__ int lstart[ND];    // first LDS position of each digit
  __shared__ int goff[ND];      // global position of the block's first key of each digit
  __shared__ int sk[256 * ITEMS], sv[256 * ITEMS];
  __shared__ int sh[4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t base = (int64_t)blockIdx.x * (256 * ITEMS);
  const int64_t wbase = base + wave * (64 * ITEMS) + lane;
  int k[ITEMS], rank[ITEMS];
#pragma unroll
  for (int it = 0; it < ITEMS; ++it) k[it] = wbase + it * 64 < n ? keys[wbase + it * 64] : 0;
  for (int d = lane; d < ND; d += 64) wc[wave][d] = 0;
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  const unsigned long long lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
#pragma unroll
  for (int it = 0; it < ITEMS; ++it) {
    const bool act = wbase + it * 64 < n;
    const int d = (k[it] >> shift) & (ND - 1);
    unsigned long long same = __ballot(act);
#pragma unroll
    for (int bt = 0; bt < RB; ++bt) {
      const unsigned long long bb = __ballot((d >> bt) & 1);
      same &= ((d >> bt) & 1) ? bb : ~bb;
    }
    const int r = __popcll(same & lt);
    const int c = wc[wave][d];
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (act && r == 0) wc[wave][d] = c + __popcll(same);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    rank[it] = c + r;
  }
  __syncthreads();
  int sum = 0, all = 0, before[PT], tot[PT];
  for (int e = 0; e < PT; ++e) {
    const int d = tid * PT + e;
    int c = 0;
    for (int w2 = 0; w2 < 4; ++w2) {
      const int t = wc[w2][d];
      wc[w2][d] = c;
      c += t;
    }
    lstart[d] = c;
    sum += c;
    before[e] = tot[e] = 0;
  }
  int total;
  int ex = block_excl_scan256(sum, sh, total);
  for (int e = 0; e < PT; ++e) {
    const int c = lstart[tid * PT + e];
    lstart[tid * PT + e] = ex;
    ex += c;
  }
  if (col) {
#pragma unroll 4
    for (int b = 0; b < nblk; ++b)
      for (int e = 0; e < PT; ++e) {
        const int c = offs[b * ND + tid * PT + e];
        tot[e] += c;
        if (b < (int)blockIdx.x) before[e] += c;
      }
    for (int e = 0; e < PT; ++e) all += tot[e];
    int g = block_excl_scan256(all, sh, total);
    for (int e = 0; e < PT; ++e) {
      goff[tid * PT + e] = g + before[e];
      g += tot[e];
    }
  } else {
    for (int e = 0; e < PT; ++e) goff[tid * PT + e] = offs[(int64_t)(tid * PT + e) * nblk + blockIdx.x];
  }
  __syncthreads();
#pragma unroll
  for (int it = 0; it < ITEMS; ++it) {
    const int64_t i = wbase + it * 64;
    if (i < n) {
      const int d = (k[it] >> shift) & (ND - 1);
      const int pos = lstart[d] + wc[wave][d] + rank[it];
      sk[pos] = k[it];
      sv[pos] = vals ? vals[i] : (int32_t)i;
    }
  }
  __syncthreads();
  const int cnt = (int)min<int64_t>(256 * ITEMS, n - base);
  for (int p = tid; p < cnt; p += 256) {
    const int kp = sk[p];
    const int d = (kp >> shift) & (ND - 1);
    const int64_t g = (int64_t)goff[d] + (p - lstart[d]);
    okeys[g] = kp;
    ovals[g] = sv[p];
  }
}

static void scan_excl(int32_t* a, int64_t n, int32_t* sums, hipStream_t s) {
  const int64_t nb = (n + 1023) / 1024;
  hipLaunchKernelGGL(k_scan_blocks, dim3((unsigned)nb), dim3(256), 0, s, a, n, sums);
  hipLaunchKernelGGL(k_scan_sums, dim3(1), dim3(256), 0, s, sums, nb);
  hipLaunchKernelGGL(k_scan_add, dim3((unsigned)nb), dim3(256), 0, s, a, n, sums);
}

template <int RB, int ITEMS>
static void sort_pass(const int32_t* ik, const int32_t* iv, int64_t n, int shift, int32_t* hist, int32_t* sums,
                      int nblk, int32_t* ok, int32_t* ov, hipStream_t s) {
  const int col = nblk <= kColBlocks;
  hipLaunchKernelGGL((k_sort_hist<RB, ITEMS>), dim3(nblk), dim3(256), 0, s, ik, n, shift, hist, nblk, col);
  if (!col) scan_excl(hist, (int64_t)nblk << RB, sums, s);
  hipLaunchKernelGGL((k_sort_scatter<RB, ITEMS>), dim3(nblk), dim3(256), 0, s, ik, iv, n, shift, hist, nblk, col, ok,
                     ov);
}

bool launch_radix_sort(const ModelDev& m, const Work& w, int64_t n, int64_t max_key, hipStream_t s,
                       int32_t** sorted_keys, int32_t** sorted_vals) {
  const SortPlan sp = sort_plan(n, max_key, w.max_lines, m.n_slots);
  if (sp.place == kSortNowhere) return false;
  const int passes = sp.passes, rb = sp.rb, nblk = sp.nblk;
  const bool few = sp.few;
  int32_t* const hist = sp.place == kSortInHist  ? w.hist
                        : sp.place == kSortInRnu ? reinterpret_cast<int32_t*>(w.rnu)
                                                 : reinterpret_cast<int32_t*>(w.qpart);
  int32_t* const sums = sp.place == kSortInHist ? w.hsum : hist + sp.entries;
  const int32_t* ik = w.key;
  const int32_t* iv = nullptr;
  int32_t* ok = w.keyA;
  int32_t* ov = w.valA;
  for (int p = 0; p < passes; ++p) {
    if (nblk > 0) {
      auto* const pass = rb == 8 ? (few ? sort_pass<8, 4> : sort_pass<8, kSortItems>)
                      : rb == 9 ? (few ? sort_pass<9, 4> : sort_pass<9, kSortItems>)
                                : (few ? sort_pass<10, 4> : sort_pass<10, kSortItems>);
      pass(ik, iv, n, rb * p, hist, sums, nblk, ok, ov, s);
    }
    ik = ok;
    iv = ov;
    ok = (ok == w.keyA) ? w.keyB : w.keyA;
    ov = (ov == w.valA) ? w.valB : w.valA;
  }
  *sorted_keys = const_cast<int32_t*>(ik);
  *sorted_vals = const_cast<int32_t*>(iv);
  return true;
}

// ---------------------------------------------------------------------------
// Cell offsets from the sorted keys (the dropped key is n = fine_keys, and the position
// after the last line acts as n + 1, so every cell 0..n gets its start; off[n] = kept lines),
// and, in the same pass, the sorted line records: nu, gamma_ref, n_exp, original index, and the
// intensity of every slot, S (FP64) or S~ = sign exp(ln|S| - s_b) (FP32).
// ---------------------------------------------------------------------------
template <bool LTE>
__global__ __launch_bounds__(256) void k_records(ModelDev m, const SlotDev* slots, const double* Q,
                                                 const double* sb, StatesView st, LinesView ln,
                                                 const void* lpack,
                                                 const int32_t* skeys, const int32_t* svals,
                                                 const unsigned long long* stats, int32_t* off, int far,
                                                 int64_t max_lines, double* rnu, float* rgref,
                                                 float* rnexp, double* rgpre, int32_t* ridx, double* rEs,
                                                 void* rS, int32_t* oddl,
                                                 const double* cut_class, int32_t* rkc, float* rdel,
                                                 int32_t* rwin, int32_t* counter) {
  __shared__ SlotFac sf[kMaxCond];
  for (int q = threadIdx.x; q < m.n_slots; q += 256)
    sf[q] = slot_fac(slots[q], m.pop, Q[q], m.prec == XS_FP32 ? sb[q] : 0.0);
  __syncthreads();
  const int64_t n = ln.n, nk = (int64_t)stats[1];
  for (int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x; p <= n; p += (int64_t)gridDim.x * 256) {
    {
      const int k = min((p < n) ? skeys[p] : fine_keys(m) + 1, fine_keys(m));
      const int kp = (p > 0) ? skeys[p - 1] : -1;
      // empty cells, those beyond the grid's ends above all: many at a time are the wave's (one
      // lane's stores of 200 in turn took 4 us)
      constexpr int kFew = 8;
      const unsigned long long here = __ballot(1);
      const int rank = __builtin_amdgcn_mbcnt_hi((unsigned)(here >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)here, 0u));
      for (unsigned long long many = __ballot(k - kp > kFew); many; many &= many - 1) {
        const int s = __builtin_ctzll(many);
        const int lo = __builtin_amdgcn_readlane(kp, s) + 1, hi = __builtin_amdgcn_readlane(k, s);
        const int at = __builtin_amdgcn_readlane((int)p, s);
        for (int b = lo + rank; b <= hi; b += __popcll(here)) off[b] = at;
      }
      if (k - kp <= kFew)
        for (int b = kp + 1; b <= k; ++b) off[b] = (int32_t)p;
    }
    if (p >= nk) continue;
    const int32_t i = svals[p];
    const auto lp = ((const typename PackOf<LTE>::type*)lpack)[i];
    const double nu = lp.nu;
    rnu[p] = nu;
    rgref[p] = lp.gref;
    rnexp[p] = lp.nexp;
    double gpre = 0.0;
    if (rgpre) {
      // natural width of a predissociating upper state: HWHM 1/(4 pi c tau)
      const double tau = st.tau[ln.up[i]];
      rgpre[p] = gpre = (tau > 0.0 && tau < INFINITY) ? 1.0 / (4.0 * kPI * kC * tau) : 0.0;
    }
    ridx[p] = i;
    if (LTE) rEs[p] = lp.er;
    // home bin, offset from it, and the exact window of every cut-off class
    const int64_t kc = home_bin(nu, m.nu0, m.dnu);
    rkc[p] = (int32_t)kc;
    rdel[p] = (float)(nu - nu_of_bin(m.nu0, m.dnu, kc));
    for (int q = 0; q < m.n_cut_classes; ++q) {
      int64_t klo, khi;
      if (!line_window(nu, cut_class[q], m.nu0, m.dnu, m.n_bins, klo, khi)) {
        klo = 1;
        khi = 0;
      }
      ((int2*)rwin)[(int64_t)q * max_lines + p] = make_int2((int)klo, (int)khi);
    }
    const LineFac f = pack_fac(lp);
    const double sc = ln.lscale ? (double)ln.lscale[i] : 0.0;
    bool odd = false;
    for (int q = 0; q < m.n_slots; ++q) {
      const double S = intensity_value(intensity<LTE>(m.mode, m.pop, f, sf[q]), sf[q], sc);
      if (m.prec == XS_FP32)
        ((float*)rS)[(int64_t)q * max_lines + p] = (float)S;
      else
        ((double*)rS)[(int64_t)q * max_lines + p] = S;
      if (far) odd |= m.prec == XS_FP32 ? !isfinite((float)S) : !isfinite(S);
    }
    // (far: with tile expansions) lines that are not finite, in a list (OddLines; k_near puts it in order)
    const bool lor = m.profile == XS_LORENTZ || m.profile == XS_BIN_LORENTZ;
    if (far && (odd || !isfinite(lp.gref) || !isfinite(lp.nexp) || (lor && lp.gref == 0.0f && gpre == 0.0)) &&
        __hip_atomic_load(counter + kOddCount, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) <= kOddMax) {
      const int at = atomicAdd(counter + kOddCount, 1);
      if (at < kOddMax) oddl[at] = (int32_t)p;
      else counter[kFarOff] = 1;
    }
  }
}

void launch_offsets_records(const ModelDev& m, const Work& w, const StatesView& st,
                            const LinesView& ln, const int32_t* skeys, const int32_t* svals, hipStream_t s) {
  int64_t blocks = (ln.n + 256) / 256;
  if (blocks > 8192) blocks = 8192;
  hipLaunchKernelGGL((m.pop == XS_LTE ? k_records<true> : k_records<false>), dim3((unsigned)blocks), dim3(256), 0, s,
                     m, w.slot, w.Q, w.sb, st, ln, (const void*)w.lpack, skeys, svals, w.stats, w.off,
                     w.far_cond_rows > 0, w.max_lines, w.rnu, w.rgref, w.rnexp, w.rgpre, w.ridx, w.rEs, w.rS, w.odd.pos,
                     w.cut_class, w.rkc, w.rdel, w.rwin, w.counter);
}

// ---------------------------------------------------------------------------
// Stick spectrum output: S of every line for every condition, original order.
// ---------------------------------------------------------------------------
// The FP64 form needs no scale, so its totals are counted here, without a pass
// before it (5e6 lines: 403 + 218 us in two passes with logarithms, 155 in one); ln Q is
// taken once per block and the states from the packed table (MODE, as above).
template <int MODE, bool COUNT, bool LTE>
__global__ __launch_bounds__(256) void k_intensity_out(ModelDev m, const CondDev* cond,
                                                       const SlotDev* slots, const double* Q,
                                                       const double* sb, const double* cutc, const int32_t* cutm,
                                                       StatesView st, const void* spack,
                                                       LinesView ln, void* S, double* lsc, unsigned long long* part) {
  __shared__ SlotFac sf[kMaxCond];
  __shared__ unsigned long long scnt[12];
  for (int q = threadIdx.x; q < m.n_slots; q += 256) sf[q] = slot_fac(slots[q], m.pop, Q[q], COUNT ? 0.0 : sb[q]);
  __syncthreads();
  Totals tot;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < ln.n;
       i += (int64_t)gridDim.x * 256) {
    const int32_t u = ln.up[i], l = ln.lo[i];
    LineState ls{0, 0, 0, 0, 0, 0, 0};
    const bool ok = gather_line_states<MODE, LTE>(m, st, spack, u, l, ls);
    const double nu = ok ? ls.Eu - ls.El : 0.0;
    if (COUNT) {
      int64_t a, b;
      if (!ok) {
        ++tot.bad;
      } else if (nu > 0.0 && line_window(nu, m.max_cut, m.nu0, m.dnu, m.n_bins, a, b)) {
        ++tot.kept;
        tot.pairs += window_pairs(m, cutc, cutm, nu, a, b);
      }
    }
    const double sc = ln.lscale ? (double)ln.lscale[i] : 0.0;
    const LineFac f = line_fac(m.mode, LTE ? XS_LTE : m.pop, ls, (double)ln.A[i], nu);
    for (int c = 0; c < m.n_cond; ++c) {
      const SlotFac& q = sf[cond[c].slot];
      const double v = nu > 0.0 ? intensity_value(intensity<LTE>(m.mode, m.pop, f, q), q, sc) : 0.0;
      if (m.prec == XS_FP32)
        ((float*)S)[(int64_t)c * ln.n + i] = (float)v;
      else
        ((double*)S)[(int64_t)c * ln.n + i] = v;
    }
  }
  if (COUNT) block_totals(tot, scnt, part);
  if (lsc && ln.n > 0 && blockIdx.x == 0 && threadIdx.x < m.n_cond)
    lsc[threadIdx.x] = COUNT ? 0.0 : sb[cond[threadIdx.x].slot];
}

template <bool COUNT>
static void intensity_out(const ModelDev& m, const Work& w, const StatesView& st, const LinesView& ln, void* S,
                          double* log_scale, hipStream_t s) {
  const void* pack = state_pack(m, w, st);
  const bool lte = m.pop == XS_LTE;
  auto* const k = pack ? (lte ? k_intensity_out<1, COUNT, true> : k_intensity_out<1, COUNT, false>)
                       : (lte ? k_intensity_out<0, COUNT, true> : k_intensity_out<0, COUNT, false>);
  hipLaunchKernelGGL(k, dim3(line_blocks(ln.n)), dim3(256), 0, s, m, w.cond, w.slot, w.Q, w.sb, w.cut_class,
                     w.cut_mult, st, pack, ln, S, log_scale, totals_part(w));
}

// After launch_partition with clear set.
void launch_intensity_out(const ModelDev& m, const Work& w, const StatesView& st,
                          const LinesView& ln, void* S, double* log_scale, hipStream_t s) {
  if (m.prec == XS_FP32) {
    pass1<false>(m, w, st, ln, s);
    line_totals(m, w, ln.n, false, s);
    if (ln.n > 0) intensity_out<false>(m, w, st, ln, S, log_scale, s);
  } else {
    intensity_out<true>(m, w, st, ln, S, log_scale, s);
    line_totals(m, w, ln.n, false, s);
  }
}

// Clear the work queue (a kernel, not a memset, so the step can be captured in a
// graph); the counters of xs_prepare, kFarOff and on, are kept.
__global__ void k_reset_queue(int32_t* counter) {
  if (threadIdx.x < kFarOff) counter[threadIdx.x] = 0;
}

void launch_scan_i32(int32_t* a, int64_t n, int32_t* sums, hipStream_t s) { scan_excl(a, n, sums, s); }

void launch_reset_queue(const Work& w, hipStream_t s) {
  hipLaunchKernelGGL(k_reset_queue, dim3(1), dim3(64), 0, s, w.counter);
}

}  // namespace xs
