// Staging and fused standard-synthesis kernels for gfx950 (CDNA4).
//
// Per (time step, channel) instance the image of each energy level is
//     I_l(p) += sum_{k in l} d_k |E_kp|^2,   E = W^H B,   B_lp = exp(+j 2 pi <x_l, p> / lambda_w)
// (standard synthesis, Section 2.4; levels and filters, Section 2.6 and
// Algorithm 1).
//
// The contraction runs on 16-bit MFMAs with FP32 accumulators: every operand
// value is the sum of two 16-bit words, hi + lo, and a product is hi hi + hi lo
// + lo hi.  With fp16 words (the FP32 modes; the columns of W scaled by powers
// of two, the phases in [-sqrt 2, sqrt 2]) hi + lo holds 22 bits, the dropped
// lo lo is below 2^-24 of the product, and one MFMA adds 32 products to an
// accumulator where an FP32 one adds 2 or 4, so that fewer roundings meet the
// running sum: against 64 bits the images are closer than with FP32 MFMAs
// (relative error of all levels, measured: 512 antennas x 512 eigenpairs
// 1.0e-7 against 1.2e-7 in the three-product form and 3.2e-7 against 5.0e-7 in
// the four-product form at 65 km; 64 x 64 1.2e-7 against 1.7e-7; with fewer than
// 12 antennas there is little to save, and the three-product form is 3 to 18 %
// farther, 1.2e-7 to 1.5e-7), at 2.7 times the products per second of the FP32
// matrix rate.  With bf16 words (the BF16
// modes) hi + lo holds 16 bits.
//
// The complex product takes four real products (planes Wr, Wi and Br, Bi) or,
// with Gauss, three: conj(w) b = (k1 - k3) + j (k1 + k2), k1 = (wr - wi) br,
// k2 = wr (bi - br), k3 = -wi (br + bi).
//
// Kernel structure (one workgroup = one pixel tile of one image slot):
//   for each instance of the slot (its scaled positions copied to LDS once),
//   for each K pass, for each 32-antenna chunk:
//     MFMA (16x16x32): W^H operand from L2 in operand order, B operand from LDS,
//       both read ahead of their use
//     phase generation of the next chunk, a slice per MFMA step: FP64 <x_l, p>
//       in turns modulo 1, hardware FP32 sin/cos in turns, the hi / lo split ->
//       the other B buffer in LDS (double-buffered)
//   epilogue of a pass: d_k (Er^2 + Ei^2) reduced over k in-lane, across the
//     four row groups, and into per-level partial sums in LDS
//   end of the tile: sum over waves in a fixed order, one read-modify-write of
//     the images (one writer per pixel and launch: deterministic, no atomics).
// Neither B (L x N_pix) nor E (K x N_pix) is ever written to HBM.
//
// What bounds it: the card's power.  16-bit MFMAs on random data hold 2.4 GHz
// only while the matrix pipes are partly idle: a loop of nothing but
// 16x16x32 fp16 MFMAs reaches 1.75 PFLOP/s (32x32x16: 1.5, hence the smaller
// MFMA), and 1.39 with the W loads, LDS reads and phase instructions of this
// kernel beside them; a large fp16 matrix product of the vendor library
// reaches 1.12.  512 antennas x 512 eigenpairs x 1024^2 pixels x 16 epochs:
// 64.7 ms in the three-product form (1.22 PFLOP/s, 6.8e13 products/s; 67.0 on
// another card) against 197.6 ms on FP32 MFMAs (85 % of their peak).

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "bb_internal.h"
#include "split.h"

namespace bb {

constexpr size_t kMaxLds = 160 * 1024;  // LDS of a gfx950 compute unit

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));

// ---------------------------------------------------------------------------
// Pointers read out of an instance descriptor are generic to the compiler, and
// generic (flat) loads count against the LDS wait counter too, so every wait
// for an LDS read would also wait for the prefetched W operand.  Casting them
// to the global address space makes those loads vector-memory loads only.
#define BB_GLOBAL __attribute__((address_space(1)))
#define BB_LDS __attribute__((address_space(3)))
template <class T>
__device__ __forceinline__ const BB_GLOBAL T* as_global(const void* p) {
  return (const BB_GLOBAL T*)p;
}

// Phase of one (antenna, pixel) pair: xs = position / wavelength, so the phase
// in turns is t = <xs, p>, needed modulo 1; gfx950's transcendental unit takes
// its sine and cosine argument in turns (sin(2 pi f)), with an absolute error
// near 1.3e-7 on [-1/2, 1/2].
//
// FAST: the FP64 multiply-adds start from kPhaseBias = 1.5 * 2^20, where FP64
// has a spacing of 2^-32, so the low word of the sum is t modulo 1 in units of
// 2^-32 (two's complement, so f in [-1/2, 1/2)), within three roundings of
// 2^-33 turns, far below the 2^-26 of the conversion to FP32 that follows
// either way.  It needs |t| < 2^19.  Otherwise t - rint(t), exact in FP64.
constexpr double kPhaseBias = 0x1.8p20;
constexpr double kPhaseFastMax = 0x1p19;  // largest sum of |xs| components for the fast form
template <bool FAST>
__device__ __forceinline__ void phase_pair(double x, double y, double z, double px, double py, double pz, double bias,
                                           float& c, float& s) {
  float f;
  if (FAST) {
    const double t = fma(z, pz, fma(y, py, fma(x, px, bias)));
    f = (float)(int)(uint32_t)__builtin_bit_cast(uint64_t, t) * 0x1p-32f;
  } else {
    const double t = fma(z, pz, fma(y, py, x * px));
    f = (float)(t - rint(t));
  }
  s = __builtin_amdgcn_sinf(f);
  c = __builtin_amdgcn_cosf(f);
}

// ---------------------------------------------------------------------------
// Staging, part 1 (one workgroup per instance): sort eigenpairs by level
// (stable, dropping level -1), scaled positions, level ranges of 16-blocks.
__global__ __launch_bounds__(256) void stage_meta_kernel(const InstDesc* __restrict__ descs,
                                                         InstDyn* __restrict__ dyn, int n_levels, bool relative,
                                                         int* __restrict__ err) {
  const InstDesc D = descs[blockIdx.x];
  __shared__ int s_lev[kMaxEig];
  __shared__ int s_cnt[kMaxLevels + 1];
  __shared__ int s_base[kMaxLevels + 1];
  const int tid = threadIdx.x;
  if (tid <= kMaxLevels) s_cnt[tid] = 0;
  __syncthreads();
  for (int k = tid; k < D.K; k += blockDim.x) {
    int lv = D.lev_in[k];
    if (lv < -1 || lv >= n_levels) {
      atomicOr(err, kErrLevelId);
      lv = -1;
    }
    s_lev[k] = lv;
    if (lv >= 0) atomicAdd(&s_cnt[lv], 1);
  }
  __syncthreads();
  if (tid == 0) {
    int acc = 0;
    for (int l = 0; l < n_levels; ++l) {
      s_base[l] = acc;
      acc += s_cnt[l];
    }
    s_base[n_levels] = acc;
    dyn[blockIdx.x].K_eff = acc;
    dyn[blockIdx.x].K_pad = round_up(acc, 32);
  }
  __syncthreads();
  const int K_eff = s_base[n_levels];
  for (int k = tid; k < D.K; k += blockDim.x) {
    const int lv = s_lev[k];
    if (lv < 0) continue;
    int r = 0;
    for (int j = 0; j < k; ++j) r += (s_lev[j] == lv);
    const int pos = s_base[lv] + r;
    D.perm[pos] = k;
    D.wts[pos] = D.d[k];
    D.levs[pos] = lv;
  }
  for (int pos = K_eff + tid; pos < D.K_alloc; pos += blockDim.x) {
    D.perm[pos] = -1;
    D.wts[pos] = 0.0f;
    D.levs[pos] = -1;
  }
  __syncthreads();
  // level range of each 16-block of sorted positions (levels are
  // non-decreasing; (1, 0) for a block with no kept eigenpair)
  for (int i = tid; i < D.K_alloc / 16; i += blockDim.x) {
    const int p0 = i * 16;
    int lo = 1, hi = 0;
    if (p0 < K_eff) {
      const int p1 = min(p0 + 15, K_eff - 1);
      // sorted positions: find their levels through the base offsets
      int l0 = 0, l1 = 0;
      for (int l = 0; l < n_levels; ++l) {
        if (s_base[l] <= p0 && p0 < s_base[l + 1]) l0 = l;
        if (s_base[l] <= p1 && p1 < s_base[l + 1]) l1 = l;
      }
      lo = l0;
      hi = l1;
    }
    D.kbr[i] = make_int2(lo, hi);
  }
  // positions relative to the first antenna (a common shift multiplies every
  // E_kp of a pixel by one phase factor, which |E|^2 does not see)
  double r0 = 0.0, r1 = 0.0, r2 = 0.0;
  if (relative) {
    r0 = D.ant[0];
    r1 = D.ant[D.ant_ld];
    r2 = D.ant[2 * D.ant_ld];
  }
  bool near = true;
  for (int l = tid; l < D.L_pad; l += blockDim.x) {
    double v0 = 0.0, v1 = 0.0, v2 = 0.0;
    if (l < D.L) {
      v0 = (D.ant[l] - r0) * D.scale;
      v1 = (D.ant[l + D.ant_ld] - r1) * D.scale;
      v2 = (D.ant[l + 2 * D.ant_ld] - r2) * D.scale;
    }
    D.xs[4 * l + 0] = v0;
    D.xs[4 * l + 1] = v1;
    D.xs[4 * l + 2] = v2;
    D.xs[4 * l + 3] = 0.0;
    near = near && fabs(v0) + fabs(v1) + fabs(v2) < 0.999 * kPhaseFastMax;  // false for NaN
  }
  near = __syncthreads_and(near);
  if (tid == 0) dyn[blockIdx.x].fast_phase = near;
}

// f over the wave's four rows of 16 lanes: row q gets that of v[q], as
// f(f(row 0, row 1), f(row 2, row 3)).
template <class F>
__device__ __forceinline__ float over_rows(const float (&v)[4], F f) {
  auto swapped = [&](auto x) {
    const unsigned a = x[0], b = x[1];  // a bit cast of a vector's element would take its first
    return f(__builtin_bit_cast(float, a), __builtin_bit_cast(float, b));
  };
  float t[2];
#pragma unroll
  for (int i = 0; i < 2; ++i)  // rows 0, 2 take the even value, rows 1, 3 the odd one
    t[i] = swapped(__builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, v[2 * i]),
                                                    __builtin_bit_cast(unsigned, v[2 * i + 1]), false, false));
  return swapped(__builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, t[0]),
                                                  __builtin_bit_cast(unsigned, t[1]), false, false));
}

// Component l of a column of W; T: its real type.
template <class T>
__device__ __forceinline__ void load_w(const InstDesc& D, int l, int col, float& wr, float& wi) {
  const BB_GLOBAL T* const w = as_global<T>(D.W) + 2 * ((int64_t)col * D.W_ld + l);
  wr = (float)w[0];
  wi = (float)w[1];
}

// Staging, part 2 (workgroup = 32 eigenpairs of an instance, every gridDim.z-th
// group of 128 antennas): the W^H operand in MFMA order, each value split into two
// 16-bit words hi + lo.
//
// An eigenpair's column is first scaled by a power of two of its own: its
// largest component lands in [2^13, 2^14), so that hi and lo of every value
// down to 2^-27 of the largest hold 22 bits (fp16 has 11, and the split rounds
// to nearest twice), and smaller ones are within 2^-39 of the largest.  The
// scaling is exact and undone in the epilogue (D.wexp).  BF16 words have
// FP32's range and take no scale (exponent 0).
//
// Planes: NPL = 2 (four real products): Wr, Wi; NPL = 3 (Gauss, conj(w) b =
// (k1 - k3) + j (k1 + k2)): Wr - Wi, Wr, -Wi.  Vectors of 8 antennas, ordered
// (16-eigenpair block, 32-antenna step, plane, hi / lo, lane): lane = row +
// 16 kk holds antennas 32 step + 8 kk + e, the operand of one 16x16x32 MFMA.
template <class H, int NPL, class T>
__device__ __forceinline__ void stage_pack(const InstDesc& D, int* s_ex) {
  typedef H h8 __attribute__((ext_vector_type(8)));
  constexpr bool kScaled = std::is_same<H, _Float16>::value;
  const int tid = threadIdx.x, lane = tid & 63, steps = D.L_pad / 32;
  auto column = [&](int k) {
    const int src = D.perm[k];
    return src < 0 ? -1 : (D.wcol ? D.wcol[src] : src);
  };
  // wave = (16 eigenpairs, step); the eigenpair's row in its 16-block in the low four bits of the lane
  const int col32 = (tid & 15) + 16 * (tid >> 8);
  const int k = blockIdx.x * 32 + col32;
  const int col = column(k);
  float wr[8], wi[8];
  auto load = [&](int st) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int l = 32 * st + 8 * (lane >> 4) + e;
      wr[e] = wi[e] = 0.0f;
      if (col >= 0 && l < D.L) load_w<T>(D, l, col, wr[e], wi[e]);
    }
  };
  int st = 4 * blockIdx.z + ((tid >> 6) & 3);
  load(st);  // in flight beside the reads of the scales
  if (kScaled) {  // the columns' largest finite components, four of them a wave
    const int c0 = (tid >> 6) * 4;
    int col4[4];
    float m[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      col4[c] = column(blockIdx.x * 32 + c0 + c);
      m[c] = 0.0f;
    }
    auto turn = [&](auto n_c, int l0) {  // 64 n antennas, all reads in flight at once; past the end the last antenna again
      constexpr int N = decltype(n_c)::value;
      float a[N][4];
#pragma unroll
      for (int u = 0; u < N; ++u)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          float x, y;
          load_w<T>(D, min(l0 + 64 * u + lane, D.L - 1), max(col4[c], 0), x, y);
          a[u][c] = fmaxf(fabsf(x), fabsf(y));
        }
#pragma unroll
      for (int u = 0; u < N; ++u)
#pragma unroll
        for (int c = 0; c < 4; ++c) m[c] = a[u][c] <= 3.4028235e38f ? fmaxf(m[c], a[u][c]) : m[c];
    };
    if (D.L <= 64)
      turn(std::integral_constant<int, 1>{}, 0);
    else
      for (int l0 = 0; l0 < D.L; l0 += 256) turn(std::integral_constant<int, 4>{}, l0);
#pragma unroll
    for (int c = 0; c < 4; ++c) m[c] = col4[c] >= 0 ? m[c] : 0.0f;
    float top = over_rows(m, [](float x, float y) { return fmaxf(x, y); });  // of column c0 + lane / 16
    for (int o = 8; o > 0; o >>= 1) top = fmaxf(top, __shfl_xor(top, o));
    int ex = 0;
    if (top > 0.0f) {
      (void)frexpf(top, &ex);  // top < 2^ex
      ex = 14 - ex;
    }
    if ((lane & 15) == 0) s_ex[c0 + (lane >> 4)] = ex;
    __syncthreads();
  }
  const int ex = kScaled ? s_ex[col32] : 0;
  if (blockIdx.z == 0 && (tid & 0xf0) == 0) D.wexp[k] = -ex;
  h8* const out = (h8*)D.apack + (int64_t)(k >> 4) * steps * NPL * 128;
  while (st < steps) {
    h8 hi[NPL], lo[NPL];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float r = kScaled ? ldexpf(wr[e], ex) : wr[e], i = kScaled ? ldexpf(wi[e], ex) : wi[e];
#pragma unroll
      for (int q = 0; q < NPL; ++q) {
        const float v = NPL == 2 ? (q == 0 ? r : i) : (q == 0 ? r - i : (q == 1 ? r : -i));
        // an infinite component is a low word alone: its products are infinite, not NaN
        const H vh = kScaled && fabsf(v) == INFINITY ? (H)0.0f : (H)v;
        hi[q][e] = vh;
        lo[q][e] = (H)(v - (float)vh);
      }
    }
#pragma unroll
    for (int q = 0; q < NPL; ++q) {
      out[(st * NPL + q) * 128 + lane] = hi[q];
      out[(st * NPL + q) * 128 + 64 + lane] = lo[q];
    }
    st += 4 * gridDim.z;
    load(st);
  }
}

template <class H, int NPL>
__global__ __launch_bounds__(512) void stage_pack_kernel(const InstDesc* __restrict__ descs) {
  __shared__ int s_ex[32];
  const InstDesc D = descs[blockIdx.y];
  if ((int)blockIdx.x * 32 >= D.K_alloc || (int)blockIdx.z * 128 >= D.L_pad) return;
  if (D.W_c128)
    stage_pack<H, NPL, double>(D, s_ex);
  else
    stage_pack<H, NPL, float>(D, s_ex);
}

hipError_t launch_stage_meta(const InstDesc* d_descs, InstDyn* d_dyn, int n_inst, int n_levels, bool relative,
                             int* d_err, hipStream_t s) {
  if (n_inst <= 0) return hipSuccess;
  hipLaunchKernelGGL(stage_meta_kernel, dim3(n_inst), dim3(256), 0, s, d_descs, d_dyn, n_levels, relative, d_err);
  return hipGetLastError();
}

hipError_t launch_stage(const InstDesc* d_descs, InstDyn* d_dyn, int n_inst, int max_K_alloc, int max_L_pad,
                        int n_levels, int precision, int* d_err, hipStream_t s) {
  if (n_inst <= 0) return hipSuccess;
  const hipError_t e = launch_stage_meta(d_descs, d_dyn, n_inst, n_levels, true, d_err, s);
  if (e != hipSuccess) return e;
  // antennas over workgroups until those are about two a compute unit: a single
  // instance is otherwise the latency of a loop over its antennas (900 antennas, 24
  // eigenpairs: 4.3 us in bf16, 12.2 in one workgroup), while each finds its columns'
  // scales itself
  const int64_t cols = (int64_t)(max_K_alloc / 32) * n_inst, parts = (max_L_pad + 127) / 128;
  const dim3 grid(max_K_alloc / 32, n_inst, (unsigned)std::max<int64_t>(1, std::min(parts, 512 / cols))), block(512);
  switch (precision) {
    case 1: hipLaunchKernelGGL((stage_pack_kernel<__bf16, 2>), grid, block, 0, s, d_descs); break;
    case 2: hipLaunchKernelGGL((stage_pack_kernel<_Float16, 3>), grid, block, 0, s, d_descs); break;
    case 3: hipLaunchKernelGGL((stage_pack_kernel<__bf16, 3>), grid, block, 0, s, d_descs); break;
    default: hipLaunchKernelGGL((stage_pack_kernel<_Float16, 2>), grid, block, 0, s, d_descs); break;
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Synthesis kernel.
//   H, NPL: 16-bit type of the split operands and planes of the complex product
//           (2: four real products, accumulators Er, Ei; 3: Gauss, k1, k2, k3)
//   MR x NP: 16x16 output blocks per wave (eigenpair blocks x pixel blocks);
//   WK x WN: waves along eigenpairs and along pixels.
template <int MR_, int NP_, int WK_, int WN_, int OCC_ = 2>
struct Tile {
  static constexpr int MR = MR_, NP = NP_, WK = WK_, WN = WN_;
  static constexpr int OCC = OCC_;             // waves per SIMD the register budget allows (512 / OCC registers each)
  static constexpr int WAVES = WK * WN;
  static constexpr int THREADS = 64 * WAVES;
  static constexpr int KC = 16 * MR * WK;      // eigenpairs per pass
  static constexpr int NT = 16 * NP * WN;      // pixels per tile
  static constexpr int NPB = NT / 16;          // 16-pixel blocks per tile
  static constexpr int LCH = 32;               // antennas per LDS chunk: one MFMA step
  static constexpr int JT = NT * 8 / THREADS;  // (pixel, 4-antenna) phase tasks per thread and chunk
  static_assert(THREADS % NT == 0, "a thread keeps one pixel");
  static_assert(NT % 64 == 0, "a wave keeps one antenna group per task");
  static_assert(JT >= 1 && NT * 8 % THREADS == 0, "whole tasks per thread");
  static_assert(kAntChunk % LCH == 0, "antenna padding covers the chunk");
  // LDS of a workgroup: two phase chunks, the positions of the largest instance
  // and each k-wave's level partials, sized by the launch so that small problems
  // leave room for a second workgroup on the CU.
  static constexpr size_t buf_bytes(int npl) { return (size_t)npl * NPB * 256 * sizeof(uint2); }
  static constexpr size_t lds_bytes(int npl, int max_L_pad, int n_part_levels) {
    return 2 * buf_bytes(npl) + (size_t)max_L_pad * 32 + (size_t)WK * n_part_levels * NT * sizeof(float);
  }
};

template <class H>
struct Mma;
template <>
struct Mma<_Float16> {
  typedef _Float16 h8 __attribute__((ext_vector_type(8)));
  static __device__ __forceinline__ f32x4 op(h8 a, h8 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
  }
};
template <>
struct Mma<__bf16> {
  typedef __bf16 h8 __attribute__((ext_vector_type(8)));
  static __device__ __forceinline__ f32x4 op(h8 a, h8 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
  }
};

// Task j of a thread: its pixel and the antennas 4 Q .. 4 Q + 3 of the chunk
// (Q wave-uniform: a wave's 64 lanes share one group).
template <class C>
__device__ __forceinline__ int gen_group(int tid, int j) {
  return __builtin_amdgcn_readfirstlane((tid + j * C::THREADS) / C::NT);
}

// A thread's phases of one chunk: P pairs (pair q = antenna q % 4 of task q / 4),
// the positions read from LDS ahead of each pair's arithmetic.
template <class C>
struct Phases {
  static constexpr int P = 4 * C::JT;
  float cr[P], ci[P];
  double x[P][3];
  __device__ __forceinline__ void read(const BB_LDS double* __restrict__ xs_chunk, int tid, int q) {
    const BB_LDS double* const at = xs_chunk + 4 * (4 * gen_group<C>(tid, q >> 2) + (q & 3));
#pragma unroll
    for (int a = 0; a < 3; ++a) x[q][a] = at[a];
  }
  template <bool FAST>
  __device__ __forceinline__ void pair(double px, double py, double pz, double bias, int q) {
    phase_pair<FAST>(x[q][0], x[q][1], x[q][2], px, py, pz, bias, cr[q], ci[q]);
  }
  template <bool FAST>
  __device__ __forceinline__ void all(const BB_LDS double* __restrict__ xs_chunk, double px, double py, double pz,
                                      double bias, int tid) {
#pragma unroll
    for (int q = 0; q < P; ++q) {
      read(xs_chunk, tid, q);
      pair<FAST>(px, py, pz, bias, q);
    }
  }
};

// Plane q of the thread's tasks into the chunk buffer: Br, Bi (NPL = 2) or Br,
// Bi - Br, Br + Bi (NPL = 3).  An MFMA operand is 16 bytes a lane (8 antennas,
// lane = pixel + 16 kk), kept as two 8-byte halves of 4 antennas, ordered
// (plane, pixel block, hi / lo, half, lane): a task writes one half, and
// consecutive lanes write consecutive 8 bytes, without bank conflicts.
template <class C, class H, int NPL>
__device__ __forceinline__ void gen_store(uint2* __restrict__ buf, const Phases<C>& ph, int tid, int q) {
#pragma unroll
  for (int j = 0; j < C::JT; ++j) {
    const int pl = tid % C::NT;
    const int Q = gen_group<C>(tid, j);
    const int at = ((q * C::NPB + (pl >> 4)) * 4 + (Q & 1)) * 64 + (Q >> 1) * 16 + (pl & 15);
    uint2 hi, lo;
    float v[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float r = ph.cr[4 * j + e], i = ph.ci[4 * j + e];
      v[e] = NPL == 2 ? (q == 0 ? r : i) : (q == 0 ? r : (q == 1 ? i - r : r + i));
    }
    split2<H>(v[0], v[1], hi.x, lo.x);
    split2<H>(v[2], v[3], hi.y, lo.y);
    buf[at] = hi;
    buf[at + 128] = lo;
  }
}

// One plane of the W^H operand of a step: hi and lo words of the wave's NV blocks.
template <class H, int NV>
struct AFrag {
  typename Mma<H>::h8 v[NV][2];
};
template <class H, int NV>
__device__ __forceinline__ void load_a(AFrag<H, NV>& a, const BB_GLOBAL typename Mma<H>::h8* A, int64_t m_step,
                                       int unit, int lane) {
#pragma unroll
  for (int m = 0; m < NV; ++m) {
    const BB_GLOBAL typename Mma<H>::h8* const blk = A + (m * m_step + (int64_t)unit * 128);  // wave-uniform
#pragma unroll
    for (int t = 0; t < 2; ++t) a.v[m][t] = blk[lane + t * 64];
  }
}

// x with every 16-bit word negated.
template <class V>
__device__ __forceinline__ V negated(V x) {
  typedef unsigned u4 __attribute__((ext_vector_type(4)));
  return __builtin_bit_cast(V, __builtin_bit_cast(u4, x) ^ (u4)0x80008000u);
}

// B operand of one step (pixel block n of the wave, plane u of the W operand):
// hi and lo words of plane u of the phases, with NPL = 2 of both planes.
template <class H, int NPL>
struct BFrag {
  typename Mma<H>::h8 v[NPL == 2 ? 2 : 1][2];
};
template <class C, class H, int NPL>
__device__ __forceinline__ void load_b(BFrag<H, NPL>& b, const uint2* __restrict__ buf, int u, int pb, int lane) {
#pragma unroll
  for (int i = 0; i < (NPL == 2 ? 2 : 1); ++i) {
    const uint2* const at = buf + ((NPL == 2 ? i : u) * C::NPB + pb) * 256 + lane;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      typedef unsigned u4 __attribute__((ext_vector_type(4)));
      const uint2 x = at[t * 128], y = at[t * 128 + 64];
      b.v[i][t] = __builtin_bit_cast(typename Mma<H>::h8, u4{x.x, x.y, y.x, y.y});
    }
  }
}

// acc[m][n] += a b (or -a b) of the split operands: lo hi + hi lo + hi hi.
template <class H, int NV, int MR, int NP, bool NEG>
__device__ __forceinline__ void mma3(f32x4 (&acc)[MR][NP], int n, const AFrag<H, NV>& a,
                                     const typename Mma<H>::h8 (&b)[2]) {
#pragma unroll
  for (int t = 0; t < 3; ++t)
#pragma unroll
    for (int m = 0; m < NV; ++m) {
      const typename Mma<H>::h8 av = a.v[m][t == 0 ? 1 : 0];
      acc[m][n] = Mma<H>::op(NEG ? negated(av) : av, b[t == 1 ? 1 : 0], acc[m][n]);
    }
}

// MFMAs of one step.  NPL = 3: accumulators k1, k2, k3; NPL = 2: Er = Wr Br + Wi Bi, Ei = Wr Bi - Wi Br.
template <class C, class H, int NPL, int NV>
__device__ __forceinline__ void mma_step(f32x4 (&acc)[NPL][C::MR][C::NP], const AFrag<H, NV>& a,
                                         const BFrag<H, NPL>& b, int u, int n) {
  if constexpr (NPL == 3) {
    mma3<H, NV, C::MR, C::NP, false>(acc[u], n, a, b.v[0]);
  } else if (u == 0) {
    mma3<H, NV, C::MR, C::NP, false>(acc[0], n, a, b.v[0]);
    mma3<H, NV, C::MR, C::NP, false>(acc[1], n, a, b.v[1]);
  } else {
    mma3<H, NV, C::MR, C::NP, false>(acc[0], n, a, b.v[1]);
    mma3<H, NV, C::MR, C::NP, true>(acc[1], n, a, b.v[0]);
  }
}

template <class C, class H, int NPL>
__global__ __launch_bounds__(C::THREADS, C::OCC) void synth_fwd_kernel(const FwdParams P) {
  typedef typename Mma<H>::h8 h8;
  constexpr int MR = C::MR, NP = C::NP, WK = C::WK, WN = C::WN;
  extern __shared__ __align__(16) char s_mem[];
  constexpr int kBuf = NPL * C::NPB * 256;
  uint2* const s_buf = (uint2*)s_mem;  // two chunk buffers
  // scaled positions of the current instance, (x, y, z, 0) per antenna: every
  // phase chunk reads them from here (a broadcast LDS read per antenna) rather
  // than through L2, whose latency would otherwise open each chunk
  double* const s_xs = (double*)(s_mem + 2 * C::buf_bytes(NPL));
  const BB_LDS double* const xs = (const BB_LDS double*)s_xs;
  float* const s_part = (float*)(s_xs + 4 * P.max_L_pad);  // [WK][n_levels][NT]
  auto part = [&](int q, int l, int pl) -> float& { return s_part[(q * P.n_levels + l) * C::NT + pl]; };

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  // Block m of a wave in pass p is block p MR WK + m WK + wk, wk = wave / WN: the
  // blocks that exist at a given K fall evenly on the waves of each SIMD.
  const int wk = __builtin_amdgcn_readfirstlane(wave / WN);
  const int pb0 = __builtin_amdgcn_readfirstlane((wave % WN) * NP);
  const int n_levels = P.n_levels;

  // the fast phase form needs pixels of at most unit length (up to rounding):
  // checked once, over every pixel this wave will generate phases for
  bool unit_pixels = true;
  for (int64_t tile = blockIdx.x; tile < P.n_tiles; tile += gridDim.x) {
    int64_t pg = tile * C::NT + (tid % C::NT);
    if (pg >= P.n_pix) pg = P.n_pix - 1;
    for (int a = 0; a < 3; ++a) unit_pixels = unit_pixels && fabs(P.pix[pg + a * P.pix_ld]) <= 1.001;
  }
  unit_pixels = __all(unit_pixels);

  // Persistent grid: workgroup b owns pixel tiles b, b + gridDim.x, ...; every
  // workgroup walks the groups (slots) and their instances in the same order,
  // so the workgroups running at one time stream the same instance's W operand
  // through L2.  Each image tile has exactly one writer (its owner).
  for (int grp = 0; grp < P.n_groups; ++grp) {
    const int slot = __builtin_amdgcn_readfirstlane(P.group_slot[grp]);
    for (int ii = P.group_begin[grp]; ii < P.group_begin[grp + 1]; ++ii) {
      // Instance fields are copied into (wave-uniform) locals once: read
      // through the descriptor pointer they would be reloaded after every LDS
      // store, which the compiler cannot prove does not alias them.
      const int inst = __builtin_amdgcn_readfirstlane(P.inst_list[ii]);
      const InstDesc& Dg = P.descs[inst];
      const BB_GLOBAL h8* const apack = as_global<h8>(Dg.apack);
      const BB_GLOBAL double* const xs_g = as_global<double>(Dg.xs);
      const BB_GLOBAL float* const wts = as_global<float>(Dg.wts);
      const BB_GLOBAL int* const wexp = as_global<int>(Dg.wexp);
      const BB_GLOBAL int* const levs = as_global<int>(Dg.levs);
      const BB_GLOBAL int* const kbr = as_global<int>(Dg.kbr);
      const int nkb = __builtin_amdgcn_readfirstlane(P.dyn[inst].K_eff + 15) / 16;
      const int L_pad = __builtin_amdgcn_readfirstlane(Dg.L_pad);
      const int n_chunks = L_pad / C::LCH;
      const int n_pass = (nkb * 16 + C::KC - 1) / C::KC;
      const int64_t kb_vec = (int64_t)n_chunks * NPL * 128;  // 16-byte vectors per 16-eigenpair block
      const bool near = __builtin_amdgcn_readfirstlane(P.dyn[inst].fast_phase) != 0;
      if (blockIdx.x >= P.n_tiles || n_pass == 0) continue;  // workgroup-uniform
      __syncthreads();  // the previous instance's phases are done with s_xs
      for (int i = tid; i < 2 * L_pad; i += C::THREADS) ((f64x2*)s_xs)[i] = ((const BB_GLOBAL f64x2*)xs_g)[i];
      for (int i = tid; i < WK * n_levels * C::NT; i += C::THREADS) s_part[i] = 0.0f;
      __syncthreads();

      // this thread's pixel (phase generation); clamp the ragged tail
      double px, py, pz;
      auto load_pixel = [&](int64_t tile) {
        int64_t pg = tile * C::NT + (tid % C::NT);
        if (pg >= P.n_pix) pg = P.n_pix - 1;
        px = P.pix[pg];
        py = P.pix[pg + P.pix_ld];
        pz = P.pix[pg + 2 * P.pix_ld];
      };
      double bias = kPhaseBias;
      asm("" : "+v"(bias));  // kept in registers: the multiply-add then takes it as an operand
      load_pixel(blockIdx.x);
      const bool fast = near && unit_pixels;  // wave-uniform
      int par = 0;  // chunk buffer holding the current chunk
      {
        Phases<C> ph;
        if (fast)
          ph.template all<true>(xs, px, py, pz, bias, tid);
        else
          ph.template all<false>(xs, px, py, pz, bias, tid);
#pragma unroll
        for (int q = 0; q < NPL; ++q) gen_store<C, H, NPL>(s_buf, ph, tid, q);
      }
      __syncthreads();
      for (int64_t tile = blockIdx.x; tile < P.n_tiles; tile += gridDim.x) {
        const int64_t p0 = tile * C::NT;
        // Where the registers allow it, the images are read before the last pass's
        // epilogue: with a chunk or two per instance the latency of these reads is a
        // tile's longest wait (29 antennas, 10 levels, 512^2 pixels: 70 us against 74).
        constexpr bool kEarly = MR == 1 && C::OCC == 2;
        constexpr int RP = kMaxLevels * C::NT / C::THREADS;
        float was[RP];
        for (int pass = 0; pass < n_pass; ++pass) {
          const int b0 = pass * MR * WK + wk;  // this wave's first block; block m is b0 + m WK
          int nv = nkb > b0 ? (nkb - b0 + WK - 1) / WK : 0;
          nv = __builtin_amdgcn_readfirstlane(nv < MR ? nv : MR);
          f32x4 acc[NPL][MR][NP];
#pragma unroll
          for (int t = 0; t < NPL; ++t)
#pragma unroll
            for (int m = 0; m < MR; ++m)
#pragma unroll
              for (int n = 0; n < NP; ++n) acc[t][m][n] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

          // The chunks of this pass, for NV existing blocks of this wave (NV = 0:
          // phases only).  A chunk is S steps (plane u, pixel block n) of 3 NV MFMAs
          // (6 NV with two planes); each step reads the next one's B operand, and the
          // first of a plane the next plane's A operand, so that neither is waited
          // for.  Beside the MFMAs the steps generate and store the phases of the
          // next chunk, in slices, since a burst of them would leave the matrix pipe
          // idle; the last chunk of a pass prepares the first chunk of the next pass
          // or of the workgroup's next tile.  The chunk's one barrier comes before
          // its last step: by then every wave has stored its phases and read its last
          // B operand of this chunk, and the last step can read the next chunk's first.
          auto chunks = [&](auto nv_c, auto fast_c) {
            constexpr int NV = decltype(nv_c)::value;
            constexpr int NVA = NV > 0 ? NV : 1;
            constexpr bool FAST = decltype(fast_c)::value;
            constexpr int S = NPL * NP;
            constexpr int PH = Phases<C>::P;
            constexpr int PS = S - 1 - NPL;  // the pairs go to the first PS steps, the stores to the next NPL
            static_assert(S % 2 == 0 && PS >= 1, "double-buffered B operand; steps for phases and stores");
            const BB_GLOBAL h8* const A = apack + (int64_t)b0 * kb_vec;
            const int64_t m_step = (int64_t)WK * kb_vec;
            AFrag<H, NVA> a_cur, a_nxt;
            BFrag<H, NPL> b[2];
            if constexpr (NV > 0) {
              load_a<H, NVA>(a_cur, A, m_step, 0, lane);
              load_b<C, H, NPL>(b[0], s_buf + par * kBuf, 0, pb0, lane);
            }
            for (int c = 0; c < n_chunks; ++c) {
              const bool last = c == n_chunks - 1;
              if (last && pass == n_pass - 1) load_pixel(tile + gridDim.x);
              const BB_LDS double* const xs_next = xs + (last ? 0 : 4 * (c + 1) * C::LCH);
              Phases<C> ph;
              if constexpr (NV > 0) {
#pragma unroll
                for (int st = 0; st < S; ++st) {
                  const int u = st / NP, n = st % NP;
                  if (n == 0)  // next plane's operand (past the pass's end: its first again)
                    load_a<H, NVA>(a_nxt, A, m_step, u + 1 < NPL ? c * NPL + u + 1 : (last ? 0 : (c + 1) * NPL), lane);
                  if (st + 1 < S)
                    load_b<C, H, NPL>(b[(st + 1) & 1], s_buf + par * kBuf, (st + 1) / NP, pb0 + (st + 1) % NP, lane);
                  else
                    load_b<C, H, NPL>(b[0], s_buf + (par ^ 1) * kBuf, 0, pb0, lane);
#pragma unroll
                  for (int q = 0; q < PH; ++q) {
                    const int at = q * PS / PH + (PS >= 2 * PH ? 1 : 0);  // step of pair q; its position is read a step before
                    if ((at > 0 ? at - 1 : 0) == st) ph.read(xs_next, tid, q);
                  }
                  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                  for (int q = 0; q < PH; ++q)
                    if (q * PS / PH + (PS >= 2 * PH ? 1 : 0) == st) ph.template pair<FAST>(px, py, pz, bias, q);
                  if (st >= PS && st < PS + NPL) gen_store<C, H, NPL>(s_buf + (par ^ 1) * kBuf, ph, tid, st - PS);
                  mma_step<C, H, NPL, NVA>(acc, a_cur, b[st & 1], u, n);
                  if (n == NP - 1) a_cur = a_nxt;
                  if (st == S - 2) __syncthreads();
                  __builtin_amdgcn_sched_barrier(0);
                }
              } else {
                ph.template all<FAST>(xs_next, px, py, pz, bias, tid);
#pragma unroll
                for (int q = 0; q < NPL; ++q) gen_store<C, H, NPL>(s_buf + (par ^ 1) * kBuf, ph, tid, q);
                __syncthreads();
              }
              par ^= 1;
            }
          };
          auto by_form = [&](auto nv_c) {
            if (fast)
              chunks(nv_c, std::true_type{});
            else
              chunks(nv_c, std::false_type{});
          };
          if (nv == MR)
            by_form(std::integral_constant<int, MR>{});
          else if (MR > 1 && nv == 1)
            by_form(std::integral_constant<int, 1>{});
          else
            by_form(std::integral_constant<int, 0>{});
          static_assert(MR <= 2, "block counts covered above");

          if (kEarly && pass == n_pass - 1) {
#pragma unroll
            for (int r = 0; r < RP; ++r) {
              const int i = tid + r * C::THREADS, l = i / C::NT, pl = i % C::NT;
              if (l < n_levels && p0 + pl < P.n_pix) was[r] = P.img[((int64_t)slot * n_levels + l) * P.img_ld + p0 + pl];
            }
          }
#pragma unroll
          for (int m = 0; m < MR; ++m) {
            if (m >= nv) continue;
            const int kb = b0 + m * WK;
            const int lev_lo = kbr[2 * kb], lev_hi = kbr[2 * kb + 1];
            if (lev_lo > lev_hi) continue;  // no kept eigenpair in this block
            float w[4];
            int lv[4], ex[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const int k = kb * 16 + 4 * (lane >> 4) + r;
              w[r] = wts[k];
              lv[r] = levs[k];
              ex[r] = wexp[k];
            }
            // G pixel blocks together: weighted |E|^2 by level, a lane's rows summed in
            // place, the four row groups of G NL sums by halving
            constexpr int G = NP >= 4 ? 4 : 2, NL = 4 / G;
#pragma unroll
            for (int n0 = 0; n0 < NP; n0 += G) {
              float e2[G][4];
#pragma unroll
              for (int g = 0; g < G; ++g)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                  const int n = n0 + g;
                  // fields (Er, Ei) of the accumulators, the columns' power-of-two scale undone
                  float er = NPL == 3 ? acc[0][m][n][r] - acc[NPL - 1][m][n][r] : acc[0][m][n][r];
                  float ei = NPL == 3 ? acc[0][m][n][r] + acc[1][m][n][r] : acc[1][m][n][r];
                  if (std::is_same<H, _Float16>::value) {
                    er = ldexpf(er, ex[r]);
                    ei = ldexpf(ei, ex[r]);
                  }
                  e2[g][r] = w[r] * fmaf(er, er, ei * ei);
                }
              for (int l = lev_lo; l <= lev_hi; l += NL) {
                float sum[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                  sum[q] = 0.0f;
#pragma unroll
                  for (int r = 0; r < 4; ++r) sum[q] += (lv[r] == l + q / G) ? e2[q % G][r] : 0.0f;
                }
                const float t = over_rows(sum, [](float x, float y) { return x + y; });
                const int q = lane >> 4;  // this lane's sum: pixel block q % G, level l + q / G
                if (NL == 1 || l + q / G <= lev_hi) part(wk, l + q / G, (pb0 + n0 + q % G) * 16 + (lane & 15)) += t;
              }
            }
          }
        }
        // sum over the waves in a fixed order; the partials are cleared for the next tile
        __syncthreads();
        auto finish = [&](int i, float& was_i) {
          const int l = i / C::NT, pl = i % C::NT;
          float sum = 0.0f;
#pragma unroll
          for (int q = 0; q < WK; ++q) {
            float& x = part(q, l, pl);
            sum += x;
            x = 0.0f;
          }
          if (p0 + pl < P.n_pix) {
            float* const dst = P.img + ((int64_t)slot * n_levels + l) * P.img_ld + p0 + pl;
            *dst = (kEarly ? was_i : *dst) + sum;
          }
        };
        if constexpr (kEarly) {
#pragma unroll
          for (int r = 0; r < RP; ++r)
            if (tid + r * C::THREADS < n_levels * C::NT) finish(tid + r * C::THREADS, was[r]);
        } else {
          for (int i = tid; i < n_levels * C::NT; i += C::THREADS) finish(i, was[0]);
        }
      }
    }
  }
}

// Compute units of the current device (one device type per process).
static int compute_units() {
  static const int n = [] {
    int dev = 0, ncu = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    return ncu;
  }();
  return n;
}

int resident_blocks(const void* kernel, int threads) {
  int per_cu = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, 0) != hipSuccess || per_cu < 1) per_cu = 1;
  const int n = compute_units();
  return (n > 0 ? n : 256) * per_cu;
}

template <class C, class H, int NPL>
static hipError_t launch_cfg(const FwdParams& p, hipStream_t s) {
  if (p.n_tiles <= 0 || p.n_groups <= 0) return hipSuccess;
  auto kern = synth_fwd_kernel<C, H, NPL>;
  const size_t lds = C::lds_bytes(NPL, p.max_L_pad, p.n_levels);
  static const hipError_t attr =
      hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLds);
  if (attr != hipSuccess) return attr;
  if (lds > kMaxLds) return hipErrorInvalidValue;
  // persistent grid: as many workgroups as are resident (registers and LDS)
  const int by_regs = 4 * C::OCC / C::WAVES > 0 ? 4 * C::OCC / C::WAVES : 1;
  const int by_lds = (int)(kMaxLds / lds);
  int64_t grid = (int64_t)compute_units() * (by_regs < by_lds ? by_regs : by_lds);
  if (grid <= 0) grid = 256;
  if (grid > p.n_tiles) grid = p.n_tiles;
  hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(C::THREADS), lds, s, p);
  return hipGetLastError();
}

// Contraction of a precision: the words of its split operands and its planes.
template <int PREC>
struct Form {
  using H = typename std::conditional<PREC == 1 || PREC == 3, __bf16, _Float16>::type;
  static constexpr int NPL = PREC >= 2 ? 3 : 2;
};

// ---------------------------------------------------------------------------
// Tile candidates.  Each precision has a list of tile shapes (kernel
// instantiations); a launch names one by its index in the list.  Instances
// fall in K classes by their kept eigenpairs rounded up to 32: at most 32, 64,
// 128, or more.  Each class has a default shape (the measured best on this
// GPU) and may use every shape of the list whose eigenpairs per pass do not
// exceed the class's largest K (so that no wave of a tile is idle at that K).
// Register budget: 512 / OCC VGPRs a wave at OCC waves per SIMD.  Three waves suit
// the 32 x 64 tile (four spill 60 registers: 20 antennas, 20 eigenpairs, 1500^2
// pixels 269 us against 327), and in the four-product form four waves of 2 x 4
// blocks the 64 x 128 one (50 antennas, 40 eigenpairs, 2048^2 pixels: 656 us
// against 732 in sixteen waves of 1 x 2).
template <class... T>
struct TileList {};

template <int PREC>
struct Cands;
template <>
struct Cands<0> {  // 4 products: Er / Ei accumulators, half as many as three planes need, so twice the pixels a wave
  using L = TileList<Tile<2, 8, 8, 1>,      // 0: 256 x 128
                     Tile<2, 4, 4, 2>,      // 1: 128 x 128
                     Tile<2, 4, 2, 2>,      // 2: 64 x 128, 4 waves
                     Tile<1, 2, 2, 2, 3>,   // 3: 32 x 64, 4 waves
                     Tile<2, 4, 4, 1>>;     // 4: 128 x 64, 4 waves
  static constexpr int dflt[4] = {3, 2, 1, 0};
};
template <>
struct Cands<1> {
  using L = TileList<Tile<2, 8, 8, 1>,      // 0: 256 x 128
                     Tile<2, 4, 4, 2>,      // 1: 128 x 128
                     Tile<2, 4, 2, 2>,      // 2: 64 x 128, 4 waves
                     Tile<1, 2, 2, 2, 3>,   // 3: 32 x 64, 4 waves
                     Tile<2, 4, 4, 1>,      // 4: 128 x 64, 4 waves
                     Tile<2, 4, 8, 1>>;     // 5: 256 x 64
  static constexpr int dflt[4] = {3, 2, 1, 0};
};
template <>
struct Cands<2> {  // 3 products: k1, k2, k3 accumulators
  using L = TileList<Tile<2, 4, 8, 1>,      // 0: 256 x 64
                     Tile<2, 4, 4, 1>,      // 1: 128 x 64, 4 waves
                     Tile<2, 2, 2, 4>,      // 2: 64 x 128
                     Tile<1, 2, 2, 2, 3>,   // 3: 32 x 64, 4 waves, three workgroups a CU
                     Tile<2, 2, 4, 2>,      // 4: 128 x 64
                     Tile<1, 4, 4, 2>,      // 5: 64 x 128
                     Tile<1, 4, 8, 2, 4>,   // 6: 128 x 128, 16 waves
                     Tile<2, 2, 2, 2>,      // 7: 64 x 64, 4 waves
                     Tile<1, 2, 2, 4, 4>,   // 8: 32 x 128
                     Tile<1, 2, 4, 4, 4>,   // 9: 64 x 128, 16 waves
                     Tile<1, 2, 4, 2, 4>,   // 10: 64 x 64
                     Tile<2, 4, 4, 2>>;     // 11: 128 x 128
  static constexpr int dflt[4] = {3, 9, 11, 0};
};
template <>
struct Cands<3> {
  using L = TileList<Tile<2, 4, 8, 1>,      // 0: 256 x 64
                     Tile<2, 4, 4, 2>,      // 1: 128 x 128
                     Tile<1, 2, 4, 4, 4>,   // 2: 64 x 128, 16 waves
                     Tile<1, 2, 2, 2, 3>,   // 3: 32 x 64, 4 waves
                     Tile<2, 4, 4, 1>>;     // 4: 128 x 64, 4 waves
  static constexpr int dflt[4] = {3, 2, 1, 0};
};

// The shape of half the pixels and the same eigenpairs per pass that takes a
// tile's place where the image leaves the last round of tiles nearly empty, or has
// fewer of them than compute units (launch_shape).
template <class C>
struct Narrow {
  using T = C;
};
template <>
struct Narrow<Tile<2, 8, 8, 1>> {
  using T = Tile<2, 4, 8, 1>;
};
template <>
struct Narrow<Tile<2, 4, 4, 2>> {
  using T = Tile<2, 4, 4, 1>;
};
template <>
struct Narrow<Tile<2, 4, 2, 2>> {
  using T = Tile<2, 2, 2, 2>;
};
template <>
struct Narrow<Tile<1, 2, 4, 4, 4>> {
  using T = Tile<1, 2, 4, 2, 4>;
};

// The shape of the same rows and pixels that takes a tile's place where local
// memory (antenna positions, level partials) leaves a CU fewer workgroups than the
// registers do: more waves a workgroup (391 antennas, 36 eigenpairs, 12 levels,
// 1680^2 pixels, 3 epochs in bf16: 5.3 ms against 7.3), or more registers a wave
// (29 antennas, 18 eigenpairs, 10 levels: 236 us against 243; 900 antennas, 40
// eigenpairs, 314^2 pixels, 10 epochs in fp32_3m: 1.39 ms against 1.67).  The
// sixteen waves of 128 x 128 need more than a CU holds (512 antennas from 13
// levels, 1024 from 9).
template <class C>
struct Roomy {
  using T = C;
};
template <>
struct Roomy<Tile<2, 4, 2, 2>> {
  using T = Tile<2, 2, 2, 4>;
};
template <>
struct Roomy<Tile<1, 2, 2, 2, 3>> {
  using T = Tile<1, 2, 2, 2, 2>;
};
template <>
struct Roomy<Tile<1, 2, 4, 2, 4>> {
  using T = Tile<2, 2, 2, 2>;
};
template <>
struct Roomy<Tile<1, 4, 8, 2, 4>> {
  using T = Tile<2, 4, 4, 2>;
};

// Of those, the shape of twice the pixels in eight waves that is better still in
// the three-product form, whose chunks leave a CU eight waves of either: each row of
// W is read once per 128 pixels (900 antennas, 24 eigenpairs, 512^2 pixels in bf16:
// 323 us against 340), unless its tiles fill the rounds worse.
template <class C>
struct Wide {
  using T = C;
};
template <>
struct Wide<Tile<1, 2, 2, 2, 3>> {
  using T = Tile<1, 2, 2, 4>;
};

template <class C>
static int64_t tiles_of(int64_t n_pix) {
  return (n_pix + C::NT - 1) / C::NT;
}
// Pixels that the busiest compute unit takes.
template <class C>
static int64_t cu_pixels(int64_t n_pix) {
  const int64_t n = std::max(compute_units(), 1);
  return (tiles_of<C>(n_pix) + n - 1) / n * C::NT;
}
template <class C, int NPL>
static int by_lds(const FwdParams& p) {  // workgroups of a CU's local memory
  return (int)(kMaxLds / C::lds_bytes(NPL, p.max_L_pad, p.n_levels));
}
template <class C>
constexpr int kByRegs = std::max(1, 4 * C::OCC / C::WAVES);  // ... and of its registers

template <class C, class H, int NPL>
static hipError_t launch_fitting(FwdParams p, hipStream_t s) {
  using R = typename Roomy<C>::T;
  using W = typename Wide<C>::T;
  static_assert(R::NT == C::NT && R::KC == C::KC, "the same rows and pixels");
  static_assert(R::lds_bytes(NPL, kMaxAnt, kMaxLevels) <= kMaxLds, "a listed shape runs every instance");
  if constexpr (!std::is_same<R, C>::value) {
    // (fewer waves help only where a second workgroup has a tile)
    const int fit = by_lds<C, NPL>(p);
    if (fit < kByRegs<C> && (fit == 0 || R::WAVES >= C::WAVES || p.n_tiles > compute_units())) {
      if constexpr (NPL == 3 && !std::is_same<W, C>::value) {
        static_assert(W::lds_bytes(NPL, kMaxAnt, kMaxLevels) <= kMaxLds, "and so does its wide form");
        if (cu_pixels<W>(p.n_pix) <= cu_pixels<C>(p.n_pix)) {
          p.n_tiles = tiles_of<W>(p.n_pix);
          return launch_cfg<W, H, NPL>(p, s);
        }
      }
      return launch_cfg<R, H, NPL>(p, s);
    }
  }
  return launch_cfg<C, H, NPL>(p, s);
}

template <class C, class H, int NPL>
static hipError_t launch_shape(FwdParams p, hipStream_t s) {
  using N = typename Narrow<C>::T;
  if constexpr (!std::is_same<N, C>::value) {
    // Compute units work through their tiles at one rate, whether one workgroup at a
    // time or two, so that the launch takes what the busiest one does: 200^2 pixels are
    // 313 tiles of 128, two on some of 256 units, or 625 of 64, three (391 antennas, 100
    // eigenpairs in bf16: 81 us against 95).  A tenth is what the narrow form loses
    // where both are even, but with fewer tiles than units (300 antennas, 200
    // eigenpairs, 150^2 pixels in bf16: 78 us against 84).
    if (p.n_tiles < compute_units() || 10 * cu_pixels<N>(p.n_pix) <= 9 * cu_pixels<C>(p.n_pix)) {
      p.n_tiles = tiles_of<N>(p.n_pix);
      return launch_fitting<N, H, NPL>(p, s);
    }
  }
  return launch_fitting<C, H, NPL>(p, s);
}

template <int I, class F, class T0, class... Ts>
static hipError_t tile_at(int id, F&& f, TileList<T0, Ts...>) {
  if (id == I) return f(T0{});
  if constexpr (sizeof...(Ts) > 0)
    return tile_at<I + 1>(id, f, TileList<Ts...>{});
  else
    return hipErrorInvalidValue;
}

template <class... Ts>
static constexpr int list_len(TileList<Ts...>) {
  return (int)sizeof...(Ts);
}

// f(cfg) for tile `id` of `precision`; hipErrorInvalidValue for an unknown id.
template <class F>
static hipError_t with_tile(int precision, int id, F&& f) {
  switch (precision) {
    case 1: return tile_at<0>(id, f, Cands<1>::L{});
    case 2: return tile_at<0>(id, f, Cands<2>::L{});
    case 3: return tile_at<0>(id, f, Cands<3>::L{});
    default: return tile_at<0>(id, f, Cands<0>::L{});
  }
}

int synth_k_class(int K_alloc) { return K_alloc <= 32 ? 0 : (K_alloc <= 64 ? 1 : (K_alloc <= 128 ? 2 : 3)); }

int synth_n_tiles(int precision) {
  switch (precision) {
    case 1: return list_len(Cands<1>::L{});
    case 2: return list_len(Cands<2>::L{});
    case 3: return list_len(Cands<3>::L{});
    default: return list_len(Cands<0>::L{});
  }
}

int synth_default_tile(int precision, int k_class) {
  if (k_class < 0 || k_class > 3) return -1;
  switch (precision) {
    case 1: return Cands<1>::dflt[k_class];
    case 2: return Cands<2>::dflt[k_class];
    case 3: return Cands<3>::dflt[k_class];
    default: return Cands<0>::dflt[k_class];
  }
}

bool synth_tile_info(int precision, int id, int* kc, int* nt, int* waves) {
  int a = 0, b = 0, c = 0;
  const hipError_t e = with_tile(precision, id, [&](auto cfg) {
    using C = decltype(cfg);
    a = C::KC;
    b = C::NT;
    c = C::WAVES;
    return hipSuccess;
  });
  if (e != hipSuccess) return false;
  if (kc) *kc = a;
  if (nt) *nt = b;
  if (waves) *waves = c;
  return true;
}

bool synth_tile_allowed(int precision, int id, int k_class) {
  static const int kmax[4] = {32, 64, 128, kMaxEig};
  int kc = 0;
  if (k_class < 0 || k_class > 3 || !synth_tile_info(precision, id, &kc, nullptr, nullptr)) return false;
  return kc <= kmax[k_class];
}

template <int PREC>
static hipError_t launch_prec_tile(const FwdParams& p, int id, hipStream_t s) {
  using F = Form<PREC>;
  return tile_at<0>(id, [&](auto cfg) { return launch_shape<decltype(cfg), typename F::H, F::NPL>(p, s); },
                    typename Cands<PREC>::L{});
}

hipError_t launch_synth_tile(const FwdParams& p, int precision, int id, hipStream_t s) {
  switch (precision) {
    case 1: return launch_prec_tile<1>(p, id, s);
    case 2: return launch_prec_tile<2>(p, id, s);
    case 3: return launch_prec_tile<3>(p, id, s);
    default: return launch_prec_tile<0>(p, id, s);
  }
}

// Phase-generation throughput probe (measurement only): every thread takes one
// pixel and evaluates the phases of all antennas `reps` times with the
// synthesis kernel's own arithmetic (positions from LDS, FP64 argument and
// reduction, hardware sine and cosine), summing cos + sin so that nothing is
// dropped.  No MFMA work runs beside it: its rate is the device's peak for
// phase generation alone.
__global__ __launch_bounds__(256) void phase_probe_kernel(const double* __restrict__ ant, int n_ant, double inv_wl,
                                                          const double* __restrict__ pix, int64_t n_pix, int reps,
                                                          float* __restrict__ out) {
  __shared__ __align__(16) double s_xs[4 * kMaxAnt];
  for (int l = threadIdx.x; l < n_ant; l += blockDim.x) {
    s_xs[4 * l + 0] = ant[l] * inv_wl;
    s_xs[4 * l + 1] = ant[l + n_ant] * inv_wl;
    s_xs[4 * l + 2] = ant[l + 2 * n_ant] * inv_wl;
    s_xs[4 * l + 3] = 0.0;
  }
  __syncthreads();
  const BB_LDS double* const xs = (const BB_LDS double*)s_xs;
  bool near = true;
  for (int l = threadIdx.x; l < n_ant; l += blockDim.x)
    near = near && fabs(xs[4 * l]) + fabs(xs[4 * l + 1]) + fabs(xs[4 * l + 2]) < 0.999 * kPhaseFastMax;
  near = __syncthreads_and(near);
  double bias = kPhaseBias;
  asm("" : "+v"(bias));
  for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < n_pix; p += (int64_t)gridDim.x * blockDim.x) {
    const double px = pix[p], py = pix[p + n_pix], pz = pix[p + 2 * n_pix];
    float acc = 0.0f;
    auto all = [&](auto fast_c) {
      for (int r = 0; r < reps; ++r)
        for (int l = 0; l < n_ant; ++l) {
          float c, sn;
          phase_pair<decltype(fast_c)::value>(xs[4 * l], xs[4 * l + 1], xs[4 * l + 2], px, py, pz, bias, c, sn);
          acc += c + sn;
        }
    };
    if (near && fabs(px) <= 1.001 && fabs(py) <= 1.001 && fabs(pz) <= 1.001)
      all(std::true_type{});
    else
      all(std::false_type{});
    out[p] = acc;
  }
}

hipError_t launch_phase_probe(const double* ant, int n_ant, double inv_wl, const double* pix, int64_t n_pix, int reps,
                              float* out, hipStream_t s) {
  int64_t blocks = (n_pix + 255) / 256;
  if (blocks > 8192) blocks = 8192;
  hipLaunchKernelGGL(phase_probe_kernel, dim3((unsigned)blocks), dim3(256), 0, s, ant, n_ant, inv_wl, pix, n_pix, reps,
                     out);
  return hipGetLastError();
}

__global__ void fill_zero_kernel(float* p, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = 0.0f;
}

hipError_t launch_fill_zero(float* p, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  int64_t blocks = (n + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(fill_zero_kernel, dim3((unsigned)blocks), dim3(256), 0, s, p, n);
  return hipGetLastError();
}

}  // namespace bb
