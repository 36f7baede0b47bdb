// Output-driven spreading of the NUFFT (gfx950) for grids of at most 64 points
// along axis 2.
//
// The spread is the same sum as in nufft.hip (every baseline adds its value
// times the tensor-product kernel on the w^3 grid points nearest to it), but
// taken from the side of the grid: each wave owns a block of columns (x, y) and
// adds, for every level at once, the baselines whose kernel reaches it.
//
//   1. baselines are sorted by their first grid point on axes 0 and 1
//      (counting sort over N0 x N1 bins);
//   2. one record per sorted baseline: its three kernel rows, its first points
//      on axes 1 and 2, and V'_l[r, q] exp(2 pi i <b, D>) for every level;
//   3. the baselines that reach a block of PX x 2 columns lie in PX + w - 1 runs
//      of the sorted list, one per bin row x' (two where the row wraps).  For a
//      column they are one matrix product over the run,
//        G[level, re/im][z] += sum_p V[level, re/im][p] (k0 k1 k2)[p][z],
//      taken 4 baselines a step by v_mfma_f32_16x16x4f32: both operands have
//      row or column l % 16 and baseline l / 16 in lane l, so a lane forms the
//      weight of its own (baseline, z) and loads one value of the baseline's
//      levels, and nothing is broadcast.  k1 k2 is formed once for the block's
//      columns x, and a bin row is multiplied into the columns it reaches only.
//      Eight levels fill a tile's 16 rows; up to three more are added by vector
//      multiply-adds, which costs less than a second product (2 x 4 cycles per
//      level and column against 32), beyond that there is a second product.
// Blocks near the centre of the uv plane see up to ~1e5 baselines, so a block is
// split into parts, each an equal share of every run; a block of one part stores
// its points if the grid was clear, and all others are added with atomics (a read
// and a sum would wait for every read).
//
// 50 x 512 antennas (6.5 M baselines) on 1600 x 1620 x 12 points, 9 levels, w = 6:
// 2.9 ms; 14.8 ms with a thread per point that broadcast each value along a row
// of lanes (2 instructions per multiply-add, one baseline in flight).  Products
// (4 x 32 cycles per baseline and SIMD) and vector instructions would take about
// 1 ms and 1.4 ms; the rest is the latency of short runs (17 baselines on average).

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "bb_internal.h"
#include "nufft_device.h"

namespace bb {

namespace {

constexpr int kPartLoad = 1024;  // target baselines per block and part
constexpr int kPartsMax = 1024;  // parts per block
constexpr int kXcds = 8;         // XCDs of the device (workgroups are dealt to them round-robin)
constexpr int kRun = 64;         // consecutive parts an XCD takes at a time

typedef float f32x4_t __attribute__((ext_vector_type(4)));

// f(integral_constant<int, I>) for I = B .. E - 1
template <int B, int E, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    static_for<B + 1, E>(f);
  }
}

// Word N (0..15) of each row of 16 lanes, to every lane of that row.  The
// empty asm keeps the broadcast a v_mov_b32_dpp of its own.  Left alone, the
// compiler folds the broadcast into its consumer as a DPP operand, among
// others into v_subrev_u32_dpp for the integer grid index; on gfx950 that
// opcode applies the DPP lane control to src1 instead of src0 (measured with
// one-wave checks: v_subrev_u32_dpp with row_newbcast or row_shr selects the
// lanes of src1, while v_sub_u32_dpp, v_sub_f32_dpp, v_subrev_f32_dpp and
// v_mul_f32_dpp select those of src0), so the folded code read the wrong
// lanes.  A plain v_mov_b32_dpp behaves as documented.
template <int N>
__device__ __forceinline__ int row_bcast(int v) {
  int r = __builtin_amdgcn_mov_dpp(v, 0x150 + N, 0xF, 0xF, true);
  asm volatile("" : "+v"(r));
  return r;
}

__device__ __forceinline__ float as_float(int v) { return __builtin_bit_cast(float, v); }

struct SrcRec {  // one sorted baseline: two rows of 16 words
  float k2[8], k1[8];  // zero from w on
  float k0[8];
  int pad0[4];
  int f1, f2;  // 4 x the first points on axes 1 and 2 (a byte offset of a kernel row's word)
  int pad1[2];
};
static_assert(sizeof(SrcRec) == kGatherRecBytes, "record size");

// Columns of a block: PX along axis 0, 2 along axis 1, times ZT tiles of 16
// points (64 accumulators per product).  A bin row costs nothing in the columns
// x that it does not reach, a baseline a product in each of the columns y: hence
// the block's longer side along x (before the other steps 4 x 4 columns took 4.3 ms, 8 x 2 3.8).
template <int ZT>
constexpr int kBlockX = 8 / ZT;
constexpr int kBlockY = 2;
// Groups of four baselines per step: 2 in flight hide the memory's latency better
// than 1 (3.7 ms); with 3 or 4 the registers leave fewer waves (3.0 ms).
constexpr int kGroups = 2;

// Run i of a block at (x0, y0): the sorted baselines whose first bins are row
// x' = x0 - (w - 1) + i / 2 and, of the w + 1 bins along axis 1 that reach the
// block's columns, those before (i odd) or after the wrap.  [beg, end).
struct Run {
  int beg, end;
};
__device__ __forceinline__ Run block_run(const NufftGeom& g, const int* __restrict__ offset, int px, int x0, int y0,
                                         int i) {
  const int N0 = g.N[0], N1 = g.N[1], w = g.w;
  int xb = x0 - (w - 1) + (i >> 1);
  if ((i >> 1) >= px + w - 1 || xb >= N0) return {0, 0};
  if (xb < 0) xb += N0;
  const int lo = y0 - (w - 1), hi = min(y0 + kBlockY, N1);  // bins lo .. hi - 1
  if ((i & 1) && lo >= 0) return {0, 0};
  const int first = (i & 1) ? lo + N1 : max(lo, 0), last = (i & 1) ? N1 : hi;
  const int64_t row = (int64_t)xb * N1;
  return {offset[row + first], offset[row + last]};
}

// Baseline t of an instance: antennas q < r, t = r (r - 1) / 2 + q.
__device__ __forceinline__ void baseline_of(int64_t t, int& q, int& r) {
  r = (int)((1.0f + sqrtf(1.0f + 8.0f * (float)t)) * 0.5f);
  while ((int64_t)r * (r - 1) / 2 > t) --r;
  while ((int64_t)r * (r + 1) / 2 <= t) ++r;
  q = (int)(t - (int64_t)r * (r - 1) / 2);
}

// The sort: each baseline's bin and its rank there, in the order of the counters'
// increments (bin -1: not transformed), then, at the bin's offset plus the rank,
// its record, which a wave writes from LDS with whole lines (1.4 ms with a record
// per lane).  50 x 512 antennas, 9 levels: 0.65 and 0.64 ms, bound by the scattered
// atomics and lines; 3.1 ms with a second counting pass that listed the sorted
// baselines, whose records then gathered their V' (a line of memory per value).
struct Place {
  int bin, rank;
};

__global__ __launch_bounds__(256) void nufft_rank_kernel(NufftGeom g, const NufftInst* __restrict__ insts,
                                                         const double* __restrict__ ant, int64_t ld,
                                                         int* __restrict__ count, Place* __restrict__ place,
                                                         int* __restrict__ err) {
  const NufftInst I = insts[blockIdx.y];
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (int64_t)I.n_ant * (I.n_ant - 1) / 2) return;
  int q, r;
  baseline_of(t, q, r);
  double xi[3], td;
  const int where = source_coords(g, I, ant, ld, q, r, xi, td);
  Place P = {-1, 0};
  if (where == 0) {
    P.bin = first_cell(xi[0], g.w, g.N[0]) * g.N[1] + first_cell(xi[1], g.w, g.N[1]);
    P.rank = atomicAdd(&count[P.bin], 1);
  } else if (where == 1) {  // beyond the extent; 2 is another uvw cell's
    atomicOr(err, kErrNufftExtent);
  }
  place[I.pair_off + t] = P;
}

template <int W>
__global__ __launch_bounds__(256) void nufft_records_kernel(NufftGeom g, const NufftInst* __restrict__ insts,
                                                            const double* __restrict__ ant, int64_t ld,
                                                            const float2* __restrict__ vp,
                                                            const Place* __restrict__ place,
                                                            const int* __restrict__ offset, int n_levels,
                                                            int cv_stride, SrcRec* __restrict__ rec,
                                                            float2* __restrict__ cv) {
  __shared__ alignas(16) float s_out[4][64][36];  // a wave's records, then level values; rows 16-byte aligned
  const NufftInst I = insts[blockIdx.y];
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int lane = threadIdx.x & 63;
  float(*const row)[36] = s_out[threadIdx.x >> 6];
  Place P = {-1, 0};
  if (t < (int64_t)I.n_ant * (I.n_ant - 1) / 2) P = place[I.pair_off + t];
  const int p = P.bin >= 0 ? offset[P.bin] + P.rank : -1;
  int q = 0, r = 0;
  double td = 0.0;
  if (p >= 0) {
    baseline_of(t, q, r);
    double xi[3];
    source_coords(g, I, ant, ld, q, r, xi, td);
    float k0[W], k1[W], k2[W];
    int j0[W], j1[W], j2[W];
    kernel_row<W>(xi[0], g.N[0], g.beta, k0, j0);
    kernel_row<W>(xi[1], g.N[1], g.beta, k1, j1);
    kernel_row<W>(xi[2], g.N[2], g.beta, k2, j2);
    SrcRec R = {};
#pragma unroll
    for (int i = 0; i < W; ++i) {
      R.k0[i] = k0[i];
      R.k1[i] = k1[i];
      R.k2[i] = k2[i];
    }
    R.f1 = 4 * j1[0];
    R.f2 = 4 * j2[0];
    *reinterpret_cast<SrcRec*>(row[lane]) = R;
  }
  __builtin_amdgcn_wave_barrier();
  // pieces of 16 bytes, a record's in neighbouring lanes
  float4* const rec4 = reinterpret_cast<float4*>(rec);
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int src = 8 * i + (lane >> 3), to = __shfl(p, src);
    if (to >= 0) rec4[(int64_t)to * 8 + (lane & 7)] = *reinterpret_cast<const float4*>(&row[src][4 * (lane & 7)]);
  }
  __builtin_amdgcn_wave_barrier();
  const float f = (float)(td - rint(td));
  const float pc = __builtin_amdgcn_cosf(f), ps = __builtin_amdgcn_sinf(f);
  const int L = I.n_ant;
  if (p >= 0)
    for (int lv = 0; lv < cv_stride; ++lv) {
      float2 v = make_float2(0.0f, 0.0f);
      if (lv < n_levels) v = vp[I.vp_off + (int64_t)lv * L * L + q + (int64_t)r * L];
      row[lane][2 * lv] = v.x * pc - v.y * ps;
      row[lane][2 * lv + 1] = v.x * ps + v.y * pc;
    }
  __builtin_amdgcn_wave_barrier();
  const int n4 = cv_stride / 2;  // pieces of a baseline's values
  float4* const cv4 = reinterpret_cast<float4*>(cv);
  for (int i = 0; i < n4; ++i) {
    const int e = 64 * i + lane, src = e / n4, part = e - src * n4;
    const int to = __shfl(p, src);
    if (to >= 0) cv4[(int64_t)to * n4 + part] = *reinterpret_cast<const float4*>(&row[src][4 * part]);
  }
}

// Parts of each block: ceil(its baselines / kPartLoad), none for an empty one.
__global__ __launch_bounds__(256) void nufft_block_parts_kernel(NufftGeom g, const int* __restrict__ offset, int px,
                                                                int nbx, int nby, int* __restrict__ nparts) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= nbx * nby) return;
  const int bx = b / nby, by = b - bx * nby;
  int load = 0;
  for (int i = 0; i < 2 * (px + g.w - 1); ++i) {
    const Run r = block_run(g, offset, px, bx * px, by * kBlockY, i);
    load += r.end - r.beg;
  }
  nparts[b] = min((load + kPartLoad - 1) / kPartLoad, kPartsMax);
}

// A wave per part of a block (part k of block b for part_off[b] <= k <
// part_off[b + 1]); see the file comment.  MF products of 8
// levels each and NL levels on vector units.
template <int ZT, int MF, int NL>
__global__ __launch_bounds__(256, MF == 1 && NL < 2 ? 3 : 2) void nufft_gather_spread_kernel(NufftGeom g, const int* __restrict__ offset,
                                                                  const SrcRec* __restrict__ rec,
                                                                  const float2* __restrict__ cv, int n_levels,
                                                                  int cv_stride, const int* __restrict__ part_off,
                                                                  int nbx, int nby, int fresh,
                                                                  float* __restrict__ grid, int64_t n_cell) {
  constexpr int PX = kBlockX<ZT>, PY = kBlockY;
  const int lane = threadIdx.x & 63, t = lane & 15, kk = lane >> 4;
  const int n_blocks = nbx * nby;
  const int n_parts = part_off[n_blocks];
  const int N0 = g.N[0], N1 = g.N[1], N2 = g.N[2], W = g.w;
  const int* const recw = reinterpret_cast<const int*>(rec);
  const float* const cvf = reinterpret_cast<const float*>(cv);
  int vi[MF];  // this lane's value of a baseline's levels (rows past the levels repeat the last and are not stored)
#pragma unroll
  for (int m = 0; m < MF; ++m) vi[m] = min(16 * m + t, 2 * n_levels - 1);
  const int li = 16 * MF + min(t, max(2 * NL - 1, 0));
  // Workgroups are dealt to the 8 XCDs round-robin (XCD = blockIdx.x mod 8);
  // each XCD takes runs of kRun consecutive parts (neighbouring column
  // blocks, which read many of the same records through its L2), the runs
  // dealt round-robin too so that the busy centre of the uv plane is shared.
  const int u = (blockIdx.x / kXcds) * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int part = ((u / kRun) * kXcds + blockIdx.x % kXcds) * kRun + u % kRun;
  if (part >= n_parts) return;
  // block of the part: last b with part_off[b] <= part, 64 candidates a step
  int b = 0;
  for (int hi = n_blocks; hi - b > 1;) {
    const int step = (hi - b + 63) / 64;
    const int n = __popcll(__ballot(part_off[min(b + lane * step, hi)] <= part));
    hi = min(b + n * step, hi);
    b += (n - 1) * step;
  }
  const int k = part - part_off[b], K = part_off[b + 1] - part_off[b];
  const int x0 = b / nby * PX, y0 = b % nby * PY;
  const int n_run = 2 * (PX + W - 1);
  Run mine = block_run(g, offset, PX, x0, y0, lane);
  {
    const int64_t n = mine.end - mine.beg;
    mine.end = mine.beg + (int)(n * (k + 1) / K);
    mine.beg += (int)(n * k / K);
  }
  f32x4_t acc[PX][PY][ZT][MF];
  float2 accl[PX][PY][ZT][NL ? NL : 1];
#pragma unroll
  for (int jx = 0; jx < PX; ++jx)
#pragma unroll
    for (int j = 0; j < PY; ++j)
#pragma unroll
      for (int zt = 0; zt < ZT; ++zt) {
#pragma unroll
        for (int m = 0; m < MF; ++m) acc[jx][j][zt][m] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int l = 0; l < NL; ++l) accl[jx][j][zt][l] = make_float2(0.0f, 0.0f);
      }
  // S groups of four baselines each, from p0 on, of run `run` that ends before
  // `end`; the next ones' words are requested before these are used.  Lane t of a
  // row holds words t and 16 + t of the row's baseline, and its values t, 16 MF + t.
  constexpr int S = kGroups;
  struct Group {
    int w0, w1, l;
    float v[MF];
  };
  int run = -1, p0 = 0, end = 0;
  auto advance = [&]() -> bool {
    p0 += 4 * S;
    while (p0 >= end) {
      if (++run >= n_run) return false;
      p0 = __builtin_amdgcn_readlane(mine.beg, run);
      end = __builtin_amdgcn_readlane(mine.end, run);
    }
    return true;
  };
  auto fetch = [&](Group (&G)[S]) {
    const int* const r = recw + (int64_t)p0 * 32;
    const float* const c = cvf + (int64_t)p0 * (2 * cv_stride);
#pragma unroll
    for (int g = 0; g < S; ++g) {
      if (g > 0 && p0 + 4 * g >= end) break;
      const unsigned q = min(kk + 4 * g, end - 1 - p0);
      G[g].w0 = r[q * 32 + t];
      G[g].w1 = r[q * 32 + 16 + t];
      const unsigned qc = q * (2 * cv_stride);
#pragma unroll
      for (int m = 0; m < MF; ++m) G[g].v[m] = c[qc + vi[m]];
      if (NL) G[g].l = __builtin_bit_cast(int, c[qc + li]);
    }
  };
  // rows of the kernel are read from the row's lanes by 4 x the point
  const int row_k2 = (lane & ~15) * 4, row_k1 = row_k2 + 32;
  bool more = advance();
  Group cur[S], nxt[S];
  if (more) fetch(nxt);
  while (more) {
#pragma unroll
    for (int g = 0; g < S; ++g) cur[g] = nxt[g];
    const int a = W - 1 - (run >> 1);  // kernel point of the block's first column on axis 0
    const int left = end - p0;
    more = advance();
    if (more) fetch(nxt);
#pragma unroll
    for (int g = 0; g < S; ++g) {
      if (g > 0 && 4 * g >= left) break;
      const bool live = kk + 4 * g < left;
      // lane jx of a row: k0[a + jx] where that is a kernel point
      const int k0s = __builtin_amdgcn_ds_bpermute((4 * (t + a) & 60) | row_k2, cur[g].w1);
      // points of the block's columns on axis 1 and of this lane on axis 2,
      // wrapped by the unsigned minimum: a negative number is the larger one
      const unsigned e1 = 4 * (y0 + PY - 1) - row_bcast<12>(cur[g].w1);
      const int d1 = (int)min(e1, e1 + 4 * N1) - 4 * (PY - 1);
      float k1[PY];
#pragma unroll
      for (int j = 0; j < PY; ++j) {
        const int c = d1 + 4 * j;
        const float v = as_float(__builtin_amdgcn_ds_bpermute((c & 28) | row_k1, cur[g].w0));
        k1[j] = (unsigned)c < 32u ? v : 0.0f;
    }
      const int f2 = row_bcast<13>(cur[g].w1);
      float k12[PY][ZT];
#pragma unroll
      for (int zt = 0; zt < ZT; ++zt) {
        const unsigned e2 = 4 * t + 64 * zt - f2, d = min(e2, e2 + 4 * N2);
        const float v = as_float(__builtin_amdgcn_ds_bpermute((d & 28) | row_k2, cur[g].w0));
        const float k2 = d < 32u && live ? v : 0.0f;
#pragma unroll
        for (int j = 0; j < PY; ++j) k12[j][zt] = k1[j] * k2;
    }
      float2 lv[NL ? NL : 1];
      static_for<0, NL>([&](auto l) {
        lv[l] = make_float2(as_float(row_bcast<2 * l>(cur[g].l)), as_float(row_bcast<2 * l + 1>(cur[g].l)));
      });
      static_for<0, PX>([&](auto jx) {
        if ((unsigned)(a + jx) >= (unsigned)W) return;  // the same for the wave
        const float k0 = as_float(row_bcast<jx>(k0s));
#pragma unroll
        for (int j = 0; j < PY; ++j)
#pragma unroll
          for (int zt = 0; zt < ZT; ++zt) {
            const float wgt = k0 * k12[j][zt];
#pragma unroll
            for (int m = 0; m < MF; ++m)
              acc[jx][j][zt][m] = __builtin_amdgcn_mfma_f32_16x16x4f32(cur[g].v[m], wgt, acc[jx][j][zt][m], 0, 0, 0);
#pragma unroll
            for (int l = 0; l < NL; ++l) {
              accl[jx][j][zt][l].x += wgt * lv[l].x;
              accl[jx][j][zt][l].y += wgt * lv[l].y;
            }
          }
      });
    }
  }
  // whole sums of a grid that was clear are stored, others are added
  const bool store = fresh && K == 1;
  auto add = [&](int lv, int x, int y, int z, float re, float im) {
    if (lv >= n_levels || y >= N1 || z >= N2 || (re == 0.0f && im == 0.0f)) return;
    float* const G = grid + 2 * ((int64_t)lv * n_cell + ((int64_t)x * N1 + y) * N2 + z);
    if (store) {
      *reinterpret_cast<float2*>(G) = make_float2(re, im);
    } else {
      unsafeAtomicAdd(G, re);
      unsafeAtomicAdd(G + 1, im);
    }
  };
#pragma unroll
  for (int jx = 0; jx < PX; ++jx) {
    if (x0 + jx >= N0) break;
#pragma unroll
    for (int zt = 0; zt < ZT; ++zt) {
#pragma unroll
      for (int j = 0; j < PY; ++j)
#pragma unroll
        for (int m = 0; m < MF; ++m) {  // registers 2 h, 2 h + 1: level 8 m + 2 kk + h
          const f32x4_t& d = acc[jx][j][zt][m];
          add(8 * m + 2 * kk, x0 + jx, y0 + j, 16 * zt + t, d[0], d[1]);
          add(8 * m + 2 * kk + 1, x0 + jx, y0 + j, 16 * zt + t, d[2], d[3]);
        }
#pragma unroll
      for (int l = 0; l < NL; ++l) {  // four baselines' shares; lane quarter kk < PY stores column y0 + kk
        float re = 0.0f, im = 0.0f;
#pragma unroll
        for (int j = 0; j < PY; ++j) {
          float2 v = accl[jx][j][zt][l];
          v.x += __shfl_xor(v.x, 16);
          v.y += __shfl_xor(v.y, 16);
          v.x += __shfl_xor(v.x, 32);
          v.y += __shfl_xor(v.y, 32);
          if (kk == j) re = v.x, im = v.y;
        }
        if (kk < PY) add(8 * MF + l, x0 + jx, y0 + kk, 16 * zt + t, re, im);
      }
    }
  }
}

// Blocks of `px` points of a periodic axis of n points that w consecutive points
// (w <= n / 2) reach at most.  Across the wrap the last block may be a remainder
// of r = n mod px points, one block more: with a points before the wrap and w - a
// behind it, 1 + ceil((a - r) / px) + ceil((w - a) / px) blocks.
int64_t axis_reach(int n, int px, int w) { return (w - 1 + px - 1) / px + 1 + (n % px ? 1 : 0); }

}  // namespace

int nufft_gather_z(const NufftGeom& g) {
  for (int z : {16, 32, 64})
    if (g.N[2] <= z) return z;
  return 0;
}

void nufft_gather_blocks(const NufftGeom& g, int& nbx, int& nby) {
  const int px = 128 / nufft_gather_z(g);
  nbx = (g.N[0] + px - 1) / px;
  nby = (g.N[1] + kBlockY - 1) / kBlockY;
}

hipError_t launch_nufft_spread_gather(const NufftGeom& g, const NufftInst* insts, int n_inst, int max_ant,
                                      int64_t max_src, const double* ant, int64_t ld, const void* vp, int* count,
                                      int* offset, void* place, int n_levels, void* rec, void* cv, int* nparts,
                                      int* part_off, int* scan_tmp, bool fresh, float* grid, int64_t n_cell, int* err,
                                      hipStream_t s) {
  const int Zc = nufft_gather_z(g);
  if (Zc == 0) return hipErrorInvalidValue;
  int nbx, nby;
  nufft_gather_blocks(g, nbx, nby);
  const int n_blocks = nbx * nby, n_bins = g.N[0] * g.N[1];
  const int cv_stride = (n_levels + 1) & ~1;
  const dim3 pairs((unsigned)(((int64_t)max_ant * (max_ant - 1) / 2 + 255) / 256), (unsigned)n_inst);
  hipError_t e = launch_fill_zero(reinterpret_cast<float*>(count), n_bins, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(nufft_rank_kernel, pairs, dim3(256), 0, s, g, insts, ant, ld, count, static_cast<Place*>(place),
                     err);
  e = launch_scan_i32(count, n_bins, offset, nullptr, scan_tmp, s);
  if (e != hipSuccess) return e;
  e = with_width(g.w, [&](auto wc) -> hipError_t {
    constexpr int KW = decltype(wc)::value;
    hipLaunchKernelGGL(nufft_records_kernel<KW>, pairs, dim3(256), 0, s, g, insts, ant, ld,
                       static_cast<const float2*>(vp), static_cast<const Place*>(place), offset, n_levels, cv_stride,
                       static_cast<SrcRec*>(rec), static_cast<float2*>(cv));
    return hipGetLastError();
  });
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(nufft_block_parts_kernel, dim3((unsigned)((n_blocks + 255) / 256)), dim3(256), 0, s, g, offset,
                     128 / Zc, nbx, nby, nparts);
  e = launch_scan_i32(nparts, n_blocks, part_off, nullptr, scan_tmp, s);
  if (e != hipSuccess) return e;
  // a wave takes one part: sum over blocks of ceil(load / kPartLoad) of them at most
  const int64_t reach = axis_reach(g.N[0], 128 / Zc, g.w) * axis_reach(g.N[1], kBlockY, g.w);
  const int64_t parts = n_blocks + reach * max_src / kPartLoad;
  const int64_t per = 4 * kXcds * (kRun / 4);  // whole runs for every XCD
  const unsigned wgs = (unsigned)((parts + per - 1) / per * (kRun / 4) * kXcds);
  auto run = [&](auto zc, auto mc, auto lc) -> hipError_t {
    hipLaunchKernelGGL((nufft_gather_spread_kernel<decltype(zc)::value, decltype(mc)::value, decltype(lc)::value>),
                       dim3(wgs), dim3(256), 0, s, g, offset, static_cast<const SrcRec*>(rec),
                       static_cast<const float2*>(cv), n_levels, cv_stride, part_off, nbx, nby, fresh ? 1 : 0, grid,
                       n_cell);
    return hipGetLastError();
  };
  auto by_levels = [&](auto zc) -> hipError_t {
    using std::integral_constant;
    if (n_levels <= 8) return run(zc, integral_constant<int, 1>{}, integral_constant<int, 0>{});
    if (n_levels == 9) return run(zc, integral_constant<int, 1>{}, integral_constant<int, 1>{});
    if (n_levels == 10) return run(zc, integral_constant<int, 1>{}, integral_constant<int, 2>{});
    if (n_levels == 11) return run(zc, integral_constant<int, 1>{}, integral_constant<int, 3>{});
    return run(zc, integral_constant<int, 2>{}, integral_constant<int, 0>{});
  };
  if (Zc == 16) return by_levels(std::integral_constant<int, 1>{});
  if (Zc == 32) return by_levels(std::integral_constant<int, 2>{});
  return by_levels(std::integral_constant<int, 4>{});
}

}  // namespace bb
