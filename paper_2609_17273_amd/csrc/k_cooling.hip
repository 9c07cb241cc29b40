// Cooling function, Eq. (cf):
//   W(T) = h c / (4 pi Q(T)) sum_u g_u exp(-c2 E_u / T) sum_{lines from u} A nu,
// with Q(T) of Eq. (pf).  The lines are grouped by upper state first (stable
// radix sort of the upper index, then one ordered sum of A nu per run of equal
// keys), so the temperature loop runs over the states, not over the lines, and
// W and Q share every state's exponential: two sums
//   sum_i g_i exp(-c2 E_i / T) (1, sum_{lines from i} A nu),
// evaluated per (chunk of states, temperature) and added in chunk order, so the
// result does not depend on scheduling.
#include "k_common.h"

namespace xs {

// Key of every line: its upper state if the line counts (valid indices,
// nu > 0), else n_states (sorts after every state); and its A nu.  The blocks' counts of kept
// lines and of lines with an index outside the states go to part[2][blocks] and
// are added by k_cf_final (an atomic per wave on one address: 381 us at 2e6
// lines; now 25 with the terms).
constexpr int kKeyBlocks = 2048;
__global__ __launch_bounds__(256) void k_cf_keys(StatesView st, LinesView ln, int32_t* key, double* term, int32_t* counter,
                                                 unsigned long long* stats, uint32_t* part) {
  __shared__ uint32_t sh[2];
  if (threadIdx.x < 2) sh[threadIdx.x] = 0;
  if (blockIdx.x == 0) {  // the per-call counters
    for (int q = threadIdx.x; q < kCounterInts; q += 256) counter[q] = 0;
    if (threadIdx.x < 8) stats[threadIdx.x] = 0ull;
  }
  __syncthreads();
  uint32_t kept = 0, bad = 0;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < ln.n; i += (int64_t)gridDim.x * 256) {
    const int32_t u = ln.up[i], l = ln.lo[i];
    int32_t k = (int32_t)st.n;
    if ((uint32_t)u < (uint64_t)st.n && (uint32_t)l < (uint64_t)st.n) {
      const double nu = st.E[u] - st.E[l];
      if (nu > 0.0) {
        k = u;
        term[i] = (double)ln.A[i] * nu;
        ++kept;
      }
    } else {
      ++bad;
    }
    key[i] = k;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    kept += __shfl_xor(kept, o, 64);
    bad += __shfl_xor(bad, o, 64);
  }
  if ((threadIdx.x & 63) == 0) {
    atomicAdd(&sh[0], kept);
    atomicAdd(&sh[1], bad);
  }
  __syncthreads();
  if (threadIdx.x < 2) part[threadIdx.x * gridDim.x + blockIdx.x] = sh[threadIdx.x];
}

// A nu of every line in sorted order, so that the sums below read them one
// after the other (chasing line, state and energy inside each sum: 97 us at 2e6
// lines; now 33 and 22); and zero weights for the states [0, nzero).
__global__ __launch_bounds__(256) void k_cf_terms(const int32_t* sk, const int32_t* sv, int64_t n, int32_t nst,
                                                  const double* term, double* sorted, double* gw, int64_t nzero) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x, step = (int64_t)gridDim.x * 256;
  for (int64_t i = t; i < nzero; i += step) gw[i] = 0.0;
  for (int64_t p = t; p < n; p += step)
    if (sk[p] < nst) sorted[p] = term[sv[p]];
}

// gw[u - s0] = g_u sum A nu for the upper states u of [s0, s0 + ns), the sum in
// sorted order (the lines' original order, the sort being stable).
__global__ __launch_bounds__(256) void k_cf_runs(const int32_t* sk, const double* term, int64_t n, StatesView st,
                                                 int64_t s0, int64_t ns, double* gw) {
  for (int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x; p < n; p += (int64_t)gridDim.x * 256) {
    const int32_t u = sk[p];
    if (u < s0 || u >= s0 + ns || (p > 0 && sk[p - 1] == u)) continue;
    double s = 0.0;
    int64_t q = p;
    // four at a time: their loads do not wait for the keys before them
    while (q + 4 <= n && sk[q + 3] == u) {
      const double a = term[q], b = term[q + 1], c = term[q + 2], d = term[q + 3];
      s += a;
      s += b;
      s += c;
      s += d;
      q += 4;
    }
    for (; q < n && sk[q] == u; ++q) s += term[q];
    gw[u - s0] = st.g[u] * s;
  }
}

// 2^t; t is finite or a NaN.
__device__ __forceinline__ double exp2_poly(double t) {
  const double k = rint(t), r = t - k;
  return ldexp(fma(r, exp2m1_over(r), 1.0), (int)k);
}

// part[c][0..1][j] (+)= sums over chunk c of the states: g_i exp(-c2 E_i / T_j), and
// the same with gw_i.  One thread per temperature; the block stages 256 states
// at a time in LDS (-c2 E_i / ln 2 and the weights, read by every lane at the
// same address).  Bound by the FP64 units: an exponential is 16 operations here
// (1000 temperatures x 3e5 states: two sums with the library's, 250 us each; now
// both in 197 us).
__global__ __launch_bounds__(256) void k_cf_sum(const double* E, const double* g, const double* gw, int64_t n,
                                                const double* T, int32_t nT, int accumulate, double* part) {
  __shared__ double sE[256], sG[256], sW[256];
  const int chunks = gridDim.x, c = blockIdx.x;
  const int64_t per = (n + chunks - 1) / chunks;
  const int64_t i0 = min<int64_t>(n, (int64_t)c * per), i1 = min<int64_t>(n, i0 + per);
  const int j = blockIdx.y * 256 + threadIdx.x;
  // kept finite, so that only a NaN makes one: beyond either bound every
  // exponential is 0 or infinite all the same
  const double invT = j < nT ? fmin(1.0 / T[j], 1e200) : 0.0;
  double q = 0.0, w = 0.0;
  for (int64_t b = i0; b < i1; b += 256) {
    const int64_t i = b + threadIdx.x;
    __syncthreads();
    double e = i < i1 ? (-kC2 / kLN2) * E[i] : 0.0;
    e = e > 1e100 ? 1e100 : (e < -1e100 ? -1e100 : e);
    sE[threadIdx.x] = e;
    sG[threadIdx.x] = i < i1 ? g[i] : 0.0;
    sW[threadIdx.x] = i < i1 ? gw[i] : 0.0;
    __syncthreads();
    const int m = (int)min<int64_t>(256, i1 - b);
#pragma unroll 4
    for (int k = 0; k < m; ++k) {
      const double x = exp2_poly(sE[k] * invT);
      q = fma(sG[k], x, q);
      w = fma(sW[k], x, w);
    }
  }
  if (j < nT) {
    double* o = part + (int64_t)c * 2 * nT + j;
    o[0] = accumulate ? o[0] + q : q;
    o[nT] = accumulate ? o[nT] + w : w;
  }
}

// Adds the chunks: 16 temperatures a block, 16 threads to each (one thread per
// temperature waited for 1024 loads in turn: 136 us, now 13).  The first block
// also adds the key pass's counts.
__global__ __launch_bounds__(256) void k_cf_final(const double* part, int chunks, int32_t nT, double* W, double* Q,
                                                  const uint32_t* cnt, int blocks, unsigned long long* stats) {
  __shared__ double sq[16][16], sw[16][16];
  const int tj = threadIdx.x & 15, tc = threadIdx.x >> 4;
  const int j = blockIdx.x * 16 + tj;
  double q = 0.0, w = 0.0;
  if (j < nT)
#pragma unroll 8
    for (int c = tc; c < chunks; c += 16) {
      q += part[(int64_t)c * 2 * nT + j];
      w += part[(int64_t)c * 2 * nT + nT + j];
    }
  sq[tc][tj] = q;
  sw[tc][tj] = w;
  __syncthreads();
  if (tc == 0 && j < nT) {
    q = w = 0.0;
    for (int c = 0; c < 16; ++c) {
      q += sq[c][tj];
      w += sw[c][tj];
    }
    W[j] = (kH * kC / (4.0 * kPI)) * w / q;
    if (Q) Q[j] = q;
  }
  if (blockIdx.x == 0 && threadIdx.x < 128) {  // a wave per count
    const int v = threadIdx.x >> 6;
    unsigned long long r = 0;
    for (int b = threadIdx.x & 63; b < blocks; b += 64) r += cnt[v * blocks + b];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) r += __shfl_xor(r, o, 64);
    if ((threadIdx.x & 63) == 0) stats[v ? 3 : 1] = r;
  }
}

// Blocks enough to fill the chip, but no chunk shorter than it takes to stage.
static int cooling_chunks(int32_t nT) {
  const int tb = (nT + 255) / 256;
  return std::max(1, std::min(1024, (2048 + tb - 1) / tb));
}
int64_t cooling_doubles(int32_t nT) {
  return ((int64_t)nT + 31) / 32 * 32 + 2 * (int64_t)cooling_chunks(nT) * nT;
}

bool launch_cooling(const ModelDev& m, const Work& w, const StatesView& st, const LinesView& ln,
                    const double* T_dev, int32_t nT, double* W, double* Q, hipStream_t s) {
  const int64_t n = ln.n;
  const int bl = (int)std::max<int64_t>(1, std::min<int64_t>(kKeyBlocks, (n + 255) / 256));
  // the line packs' space (64 bytes a line, none here): the terms in either
  // order, then the blocks' counts
  double* term = reinterpret_cast<double*>(w.lpack);
  double* sorted = term + w.max_lines;
  uint32_t* cnt = reinterpret_cast<uint32_t*>(sorted + w.max_lines);
  hipLaunchKernelGGL(k_cf_keys, dim3(bl), dim3(256), 0, s, st, ln, w.key, term, w.counter, w.stats,
                     cnt);
  int32_t *sk = w.key, *sv = nullptr;
  if (!launch_radix_sort(m, w, n, st.n, s, &sk, &sv)) return false;
  const int chunks = cooling_chunks(nT);
  double* part = w.part + ((int64_t)nT + 31) / 32 * 32;
  // the states' weights: what is left of the partial rows, or (no room for 1024
  // there) the records' nu; more states than that take several turns
  double* gw = w.part + cooling_doubles(nT);
  int64_t room = 2 * w.item_target * 1024 - cooling_doubles(nT);
  if (room < 1024 && w.max_lines > room) {
    gw = w.rnu;
    room = w.max_lines;
  }
  for (int64_t s0 = 0; s0 < st.n; s0 += room) {
    const int64_t ns = std::min(room, st.n - s0);
    const int bz = (int)std::max<int64_t>(bl, std::min<int64_t>(kKeyBlocks, (ns + 255) / 256));
    hipLaunchKernelGGL(k_cf_terms, dim3(bz), dim3(256), 0, s, sk, sv, s0 ? 0 : n, (int32_t)st.n, term,
                       sorted, gw, ns);
    if (n > 0) hipLaunchKernelGGL(k_cf_runs, dim3(bl), dim3(256), 0, s, sk, sorted, n, st, s0, ns, gw);
    hipLaunchKernelGGL(k_cf_sum, dim3(chunks, (nT + 255) / 256), dim3(256), 0, s, st.E + s0, st.g + s0, gw, ns,
                       T_dev, nT, s0 > 0, part);
  }
  hipLaunchKernelGGL(k_cf_final, dim3((nT + 15) / 16), dim3(256), 0, s, part, chunks, nT, W, Q, cnt, bl, w.stats);
  return true;
}

}  // namespace xs
