// Level determination and image weighting, on the device.
//
// k-means levels (Section 2.6; the positive/negative split of Section 4.2):
// exact one-dimensional k-means of the positive eigenvalues, i.e. the cut of
// the sorted values into k contiguous runs with the least total within-run sum
// of squared deviations, found by dynamic programming over the last cut:
// bitonic sort, the cost of every run (thread j extends a
// Welford mean / sum of squares from v[j] down to v[0], so every run's cost is
// formed directly from its values), k DP sweeps over them, back-tracking,
// interval bounds at the gap midpoints and the level id of every eigenvalue.
//
// Uniform weighting (Section 3.5): every visibility V_pq is divided by the
// number of ordered antenna pairs whose baseline falls in the same uv cell,
// cells 1/FoV wide.  Cells are counted in an open-addressing hash table
// (64-bit keys, linear probing, global atomics) at least twice as large as the
// number of pairs, so that every probe sequence ends.

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "bb_internal.h"

namespace bb {

// ---------------------------------------------------------------------------
// k-means levels

constexpr int kKmThreads = 1024;  // = kMaxEig: one value per thread

// One Welford step: the run starting at v, its count now c (rc = 1 / c rounded).
// delta / c is formed from rc with one residual correction, which gives the
// correctly rounded quotient (Markstein) at a fraction of a division's latency.
__device__ __forceinline__ void welford(double v, double c, double rc, double& mean, double& m2) {
  const double delta = v - mean;
  const double q = delta * rc;
  mean += fma(fma(-q, c, delta), rc, q);
  m2 += delta * (v - mean);
}

struct KmArgs {
  const double* lam;
  int n, k, negative_level, n_levels;
  double* intervals;
  int* level_of;
  int* err;
};

// What the sort leaves for the other parts.
struct KmSorted {
  double v[kKmThreads];  // positive eigenvalues ascending
  double maxneg;         // largest non-positive one
  int np, nneg;
};

// Sorts the positive values into S (LDS or memory of the workgroup; scratch:
// kKmThreads doubles of LDS).  Too few of them: NaN intervals, ids -1, the error bit.
__device__ bool km_sort(const KmArgs& K, KmSorted& S, double* scratch) {
  const int t = threadIdx.x;
  const double x = t < K.n ? K.lam[t] : 0.0;
  const bool pos = t < K.n && x > 0.0;
  scratch[t] = pos ? x : INFINITY;
  const int np = __syncthreads_count(pos);
  // largest non-positive eigenvalue
  double mn = (t < K.n && !pos) ? x : -INFINITY;
  for (int o = 32; o > 0; o >>= 1) mn = fmax(mn, __shfl_xor(mn, o));
  __shared__ double s_mn[kKmThreads / 64];
  if ((t & 63) == 0) s_mn[t >> 6] = mn;
  __syncthreads();
  if (t == 0) {
    for (int w = 1; w < kKmThreads / 64; ++w) mn = fmax(mn, s_mn[w]);
    S.maxneg = mn;
    S.np = np;
    S.nneg = K.n - np;
  }
  // bitonic sort, ascending, of the values' next power of two
  int padded = 64;
  while (padded < K.n) padded <<= 1;
  for (int size = 2; size <= padded; size <<= 1) {
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      const int partner = t ^ stride;
      if (partner > t && t < padded) {
        const bool up = (t & size) == 0;
        const double a = scratch[t], b = scratch[partner];
        if ((a > b) == up) {
          scratch[t] = b;
          scratch[partner] = a;
        }
      }
      __syncthreads();
    }
  }
  S.v[t] = scratch[t];
  __syncthreads();
  if (np >= K.k) return true;
  if (t == 0) atomicOr(K.err, kErrKmeansTooFew);
  if (t < K.n_levels) {
    K.intervals[t] = NAN;
    K.intervals[K.n_levels + t] = NAN;
  }
  if (t < K.n) K.level_of[t] = -1;
  return false;
}

// Intervals and level ids from the last runs' starts cut[m][j].
__device__ void km_finish(const KmArgs& K, const KmSorted& S, const int16_t (*cut)[kKmThreads]) {
  __shared__ double s_lo[kMaxLevels], s_hi[kMaxLevels];
  const int t = threadIdx.x, k = K.k;
  if (t == 0) {
    int starts[kMaxLevels];
    int j = S.np - 1;
    for (int m = k - 1; m > 0; --m) {
      starts[m] = cut[m][j];
      j = starts[m] - 1;
    }
    starts[0] = 0;
    const double low = 0.5 * (S.v[0] + (S.nneg > 0 ? S.maxneg : 0.0));
    // run g (ascending) -> level k - 1 - g
    for (int g = 0; g < k; ++g) {
      const double lo = g == 0 ? low : 0.5 * (S.v[starts[g] - 1] + S.v[starts[g]]);
      const double hi = g + 1 < k ? 0.5 * (S.v[starts[g + 1] - 1] + S.v[starts[g + 1]]) : INFINITY;
      s_lo[k - 1 - g] = lo;
      s_hi[k - 1 - g] = hi;
    }
    if (K.negative_level) {
      s_lo[k] = -INFINITY;
      s_hi[k] = nextafter(low, -INFINITY);
    }
  }
  __syncthreads();
  if (t < K.n_levels) {
    K.intervals[t] = s_lo[t];
    K.intervals[K.n_levels + t] = s_hi[t];
  }
  if (t < K.n) {
    const double x = K.lam[t];
    int lev = -1;
    for (int l = 0; l < K.n_levels; ++l) {
      if (s_lo[l] <= x && x <= s_hi[l]) {
        lev = l;
        break;
      }
    }
    K.level_of[t] = lev;
  }
}

// All in one workgroup and its LDS: for at most a wave of positive values, whose
// runs' costs LDS holds (64 values into 8 + 1 levels: 66 us when every sweep
// formed them again with a division a step, 24 us now), and for calls without room
// for the costs in memory; there every sweep still forms them.
constexpr int kKmLds = 64;

__global__ __launch_bounds__(kKmThreads) void kmeans_levels_kernel(KmArgs K) {
  __shared__ KmSorted S;
  __shared__ double s_prev[kKmThreads];     // best cost of v[0..j] in m runs
  __shared__ double s_cur[kKmThreads];      // ... in m + 1 runs
  __shared__ double s_rc[kKmThreads];       // 1 / (t + 1)
  __shared__ double s_cost[kKmLds][kKmLds];  // [start][end]
  __shared__ int16_t s_cut[kMaxLevels][kKmThreads];  // start of the last run
  const int t = threadIdx.x;
  s_rc[t] = 1.0 / (double)(t + 1);
  if (!km_sort(K, S, s_cur)) return;
  const bool held = S.np <= kKmLds;
  // dynamic programme: s_cur[j] = min over i of s_prev[i - 1] + cost(v[i..j])
  for (int m = 0; m < K.k; ++m) {
    if (t >= m && t < S.np) {
      double mean = 0.0, m2 = 0.0, best = INFINITY;
      int arg = m;
      if (held && m > 0) {
#pragma unroll 8
        for (int i = t; i >= m; --i) {
          const double cand = s_prev[i - 1] + s_cost[i][t];
          if (cand <= best) {
            best = cand;
            arg = i;
          }
        }
      } else {
        for (int i = t; i >= m; --i) {  // run start i >= m (m runs before it need m values)
          welford(S.v[i], (double)(t - i + 1), s_rc[t - i], mean, m2);
          if (held) s_cost[i][t] = m2;
          const double cand = m == 0 ? m2 : s_prev[i - 1] + m2;
          if (m == 0 ? i == 0 : cand <= best) {  // going down in i: ties keep the smallest start
            best = cand;
            arg = i;
          }
        }
      }
      s_cur[t] = best;
      s_cut[m][t] = (int16_t)arg;
    }
    __syncthreads();
    if (t < S.np) s_prev[t] = s_cur[t];
    __syncthreads();
  }
  km_finish(K, S, s_cut);
}

// The same over the chip, with the runs' costs in memory.  512 eigenvalues (342
// positive) into 8 + 1 levels: one workgroup took 375 us (a division a step,
// every sweep forming its costs again) and 156 us with the costs kept, bound by
// the latency of one CU's loads; a launch per sweep spreads them (110 us).
struct KmScratch {
  KmSorted S;
  double prev[2][kKmThreads];
  int16_t cut[kMaxLevels][kKmThreads];
  int ok;
  double cost[1];  // n x n, [start][end]
};

__global__ __launch_bounds__(kKmThreads) void km_sort_kernel(KmArgs K, KmScratch* M) {
  __shared__ double s[kKmThreads];
  const bool ok = km_sort(K, M->S, s);
  if (threadIdx.x == 0) M->ok = ok;
}

// Thread j: the costs of all runs that end at j; the programme's first row.
__global__ __launch_bounds__(64) void km_cost_kernel(int n, KmScratch* M) {
  __shared__ double s_v[kKmThreads], s_rc[kKmThreads];
  const int np = M->S.np;
  const int t = blockIdx.x * 64 + threadIdx.x, top = min(np, (int)blockIdx.x * 64 + 64);
  if (!M->ok) return;
  for (int i = threadIdx.x; i < top; i += 64) {
    s_v[i] = M->S.v[i];
    s_rc[i] = 1.0 / (double)(i + 1);
  }
  __syncthreads();
  if (t >= np) return;
  double mean = 0.0, m2 = 0.0;
  for (int i0 = t; i0 >= 0; i0 -= 8) {  // eight values read ahead of the chain
    double v[8], rc[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      v[u] = s_v[max(i0 - u, 0)];
      rc[u] = s_rc[min(t - i0 + u, t)];
    }
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (i0 - u >= 0) {
        welford(v[u], (double)(t - i0 + u + 1), rc[u], mean, m2);
        M->cost[(int64_t)(i0 - u) * n + t] = m2;
      }
  }
  M->prev[0][t] = m2;
}

// Sweep m >= 1: 64 ends per workgroup, 16 segments of starts each.
__global__ __launch_bounds__(1024) void km_sweep_kernel(int n, int m, KmScratch* M) {
  __shared__ double s_best[16][64];
  __shared__ int s_arg[16][64];
  if (!M->ok) return;
  const int np = M->S.np, jj = threadIdx.x & 63, seg = threadIdx.x >> 6;
  const int j = blockIdx.x * 64 + jj;
  const int top = min(np, (int)blockIdx.x * 64 + 64);  // starts reach at most the block's last end
  const int len = (top - m + 15) / 16;
  const double* const prev = M->prev[(m - 1) & 1];
  double best = INFINITY;
  int arg = m;
  if (j < np) {
    const int lo = m + seg * len, hi = min(j, lo + len - 1);
    for (int i0 = hi; i0 >= lo; i0 -= 16) {
      double c[16], pv[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        const int i = max(i0 - u, lo);
        c[u] = M->cost[(int64_t)i * n + j];
        pv[u] = prev[i - 1];
      }
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        const double cand = pv[u] + c[u];
        const bool take = i0 - u >= lo && cand <= best;  // going down in i: ties keep the smallest start
        best = take ? cand : best;
        arg = take ? i0 - u : arg;
      }
    }
  }
  s_best[seg][jj] = best;
  s_arg[seg][jj] = arg;
  __syncthreads();
  if (seg != 0 || j >= np) return;
  for (int q = 1; q < 16; ++q)  // segments upwards: an equal cost does not replace a smaller start
    if (s_best[q][jj] < best) {
      best = s_best[q][jj];
      arg = s_arg[q][jj];
    }
  M->prev[m & 1][j] = best;
  M->cut[m][j] = (int16_t)arg;
}

__global__ __launch_bounds__(kKmThreads) void km_finish_kernel(KmArgs K, const KmScratch* M) {
  if (M->ok) km_finish(K, M->S, M->cut);
}

size_t kmeans_scratch_bytes(int n) { return sizeof(KmScratch) + (size_t)n * n * sizeof(double); }

hipError_t launch_kmeans_levels(const double* lam, int n, int k, int negative_level, double* intervals,
                                int* level_of, int* err, void* scratch, size_t scratch_bytes, hipStream_t s) {
  if (n < 1 || n > kKmThreads || k < 1 || k + (negative_level ? 1 : 0) > kMaxLevels) return hipErrorInvalidValue;
  const KmArgs K{lam, n, k, negative_level, k + (negative_level ? 1 : 0), intervals, level_of, err};
  // below a wave of values, or with a single run, one workgroup is done before the launches are
  if (n <= 64 || k < 2 || kmeans_scratch_bytes(n) > scratch_bytes) {
    hipLaunchKernelGGL(kmeans_levels_kernel, dim3(1), dim3(kKmThreads), 0, s, K);
    return hipGetLastError();
  }
  KmScratch* const M = static_cast<KmScratch*>(scratch);
  const dim3 ends((n + 63) / 64);
  hipLaunchKernelGGL(km_sort_kernel, dim3(1), dim3(kKmThreads), 0, s, K, M);
  hipLaunchKernelGGL(km_cost_kernel, ends, dim3(64), 0, s, n, M);
  for (int m = 1; m < k; ++m) hipLaunchKernelGGL(km_sweep_kernel, ends, dim3(1024), 0, s, n, m, M);
  hipLaunchKernelGGL(km_finish_kernel, dim3(1), dim3(kKmThreads), 0, s, K, M);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Uniform weighting

constexpr uint64_t kEmptyKey = 0x8000000080000000ull;  // cell (INT_MIN, INT_MIN): never a real cell
constexpr double kMaxCell = 1073741824.0;              // |cell| < 2^30

__device__ __forceinline__ uint64_t mix64(uint64_t z) {  // splitmix64 finaliser
  z ^= z >> 30;
  z *= 0xbf58476d1ce4e5b9ull;
  z ^= z >> 27;
  z *= 0x94d049bb133111ebull;
  z ^= z >> 31;
  return z;
}

// uv cell of the ordered pair (p, q); false when it is out of range.  The
// operation order is part of the definition (a coordinate on a cell edge is
// decided by it), so no multiply-add is fused here.
__device__ bool uv_cell_key(const double* __restrict__ ant, int64_t ld, int p, int q, const UvFrame& f,
                            uint64_t& key) {
#pragma clang fp contract(off)
  const double d0 = ant[p] - ant[q];
  const double d1 = ant[p + ld] - ant[q + ld];
  const double d2 = ant[p + 2 * ld] - ant[q + 2 * ld];
  const double au = ((d0 * f.eu[0] + d1 * f.eu[1]) + d2 * f.eu[2]) * f.scale;
  const double av = ((d0 * f.ev[0] + d1 * f.ev[1]) + d2 * f.ev[2]) * f.scale;
  const double cu = round(au), cv = round(av);  // halves away from zero
  if (!(fabs(cu) < kMaxCell) || !(fabs(cv) < kMaxCell)) return false;
  key = ((uint64_t)(uint32_t)(int32_t)cu << 32) | (uint64_t)(uint32_t)(int32_t)cv;
  return true;
}

__global__ __launch_bounds__(256) void uv_clear_kernel(uint64_t* __restrict__ keys, uint32_t* __restrict__ counts,
                                                       int64_t slots) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= slots) return;
  keys[i] = kEmptyKey;
  counts[i] = 0u;
}

// Pairs (p, q) and (q, p) fall in mirrored cells, so both passes take the pairs
// p <= q once, under the smaller key of the two cells: a cell other than the
// origin holds one ordered pair for each of them, the origin two, or one for an
// autocorrelation.  (Atomics and table reads are what bounds the passes: 512
// antennas took 29 and 10 us with every ordered pair on its own, now 18 and 8.)
struct UvCell {
  uint64_t key;  // of the pair p < q's cell or its mirror, whichever is smaller
  bool origin;
};
__device__ __forceinline__ bool uv_pair_cell(const double* __restrict__ ant, int64_t ld, int p, int q,
                                             const UvFrame& f, UvCell& c) {
  uint64_t key;
  if (!uv_cell_key(ant, ld, p, q, f, key)) return false;
  const uint32_t u = (uint32_t)(key >> 32), v = (uint32_t)key;
  const uint64_t mirror = (uint64_t)(0u - u) << 32 | (0u - v);
  c.key = key < mirror ? key : mirror;
  c.origin = key == 0;
  return true;
}

// Pair p <= q of a thread, in tiles of 16 x 16 pairs: both V_pq and V_qp are then
// reached in pieces of at least 64 bytes.
__device__ __forceinline__ bool uv_pair(int L, int& p, int& q) {
  p = blockIdx.x * 16 + (threadIdx.x & 15);
  q = blockIdx.y * 16 + (threadIdx.x >> 4);
  return p <= q && q < L;
}

__global__ __launch_bounds__(256) void uv_count_kernel(const double* __restrict__ ant, int64_t ld, int L, UvFrame f,
                                                       uint64_t* __restrict__ keys, uint32_t* __restrict__ counts,
                                                       int64_t slots, int* __restrict__ err) {
  int p, q;
  if (!uv_pair(L, p, q)) return;
  UvCell cell;
  if (!uv_pair_cell(ant, ld, p, q, f, cell)) {
    atomicOr(err, kErrUvRange);
    return;
  }
  const uint64_t mask = (uint64_t)slots - 1;
  uint64_t h = mix64(cell.key) & mask;
  for (int64_t probe = 0; probe < slots; ++probe) {
    const unsigned long long prev =
        atomicCAS((unsigned long long*)&keys[h], (unsigned long long)kEmptyKey, (unsigned long long)cell.key);
    if (prev == kEmptyKey || prev == cell.key) {
      atomicAdd(&counts[h], cell.origin && p != q ? 2u : 1u);
      return;
    }
    h = (h + 1) & mask;
  }
}

__global__ __launch_bounds__(256) void uv_apply_kernel(const double* __restrict__ ant, int64_t ld, int L, UvFrame f,
                                                       const uint64_t* __restrict__ keys,
                                                       const uint32_t* __restrict__ counts, int64_t slots,
                                                       double* __restrict__ vis) {
  int p, q;
  if (!uv_pair(L, p, q)) return;
  UvCell cell;
  if (!uv_pair_cell(ant, ld, p, q, f, cell)) return;  // flagged by the count pass
  const uint64_t mask = (uint64_t)slots - 1;
  uint64_t h = mix64(cell.key) & mask;
  uint32_t pairs = 1;
  for (int64_t probe = 0; probe < slots; ++probe) {
    const uint64_t kk = keys[h];
    if (kk == cell.key) {
      pairs = counts[h];
      break;
    }
    h = (h + 1) & mask;
  }
  const double c = (double)pairs;
  double* v = vis + 2 * ((int64_t)q * L + p);
  v[0] = v[0] / c;
  v[1] = v[1] / c;
  if (p == q) return;
  v = vis + 2 * ((int64_t)p * L + q);
  v[0] = v[0] / c;
  v[1] = v[1] / c;
}

int64_t uv_table_slots(int L) {
  int64_t slots = 1;
  while (slots < 2 * (int64_t)L * L) slots <<= 1;
  return slots;
}

hipError_t launch_uniform_weighting(const double* ant, int64_t ld, int L, const UvFrame& f, void* table,
                                    double* vis, int* err, hipStream_t s) {
  const int64_t slots = uv_table_slots(L);
  uint64_t* keys = (uint64_t*)table;
  uint32_t* counts = (uint32_t*)(keys + slots);
  const dim3 pairs((unsigned)((L + 15) / 16), (unsigned)((L + 15) / 16));
  hipLaunchKernelGGL(uv_clear_kernel, dim3((unsigned)((slots + 255) / 256)), dim3(256), 0, s, keys, counts, slots);
  hipLaunchKernelGGL(uv_count_kernel, pairs, dim3(256), 0, s, ant, ld, L, f, keys, counts, slots, err);
  hipLaunchKernelGGL(uv_apply_kernel, pairs, dim3(256), 0, s, ant, ld, L, f, keys, counts, slots, vis);
  return hipGetLastError();
}

// Byte fill with 0xFF: the workspace poison of the BB_DEBUG_FILL debug mode.
__global__ void fill_poison_kernel(unsigned char* p, size_t n) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
    p[i] = 0xFF;
}

hipError_t launch_fill_poison(void* p, size_t n, hipStream_t s) {
  if (n == 0) return hipSuccess;
  size_t blocks = (n + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(fill_poison_kernel, dim3((unsigned)blocks), dim3(256), 0, s, (unsigned char*)p, n);
  return hipGetLastError();
}

}  // namespace bb
