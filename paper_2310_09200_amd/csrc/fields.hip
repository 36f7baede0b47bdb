// E = W^H B of one instance for the backward pass, on FP32 MFMA.
//
// The antenna-position gradient is a sum over pixels of H B p with H = conj(W) M
// and M = d c conj(E), returned in FP64: its pixels' terms cancel, so it keeps
// FP32 products throughout (the forward images take the split 16-bit products
// of synth_kernels.hip).  E is computed in the three-product form
//     conj(w) b = (k1 - k3) + j (k1 + k2),
//     k1 = (wr - wi) br, k2 = wr (bi - br), k3 = -wi (br + bi)
// on v_mfma_f32_32x32x2f32, two antennas per step, and written as two planes
// (re, im) of [K_alloc][n_pix].
//
// Bound: FP32 MFMA (6 flop per antenna x eigenpair x pixel).  One workgroup owns
// pixel tiles; per 32-antenna chunk (16 on the 256-pixel tiles) the phases go to
// LDS double-buffered, each wave's share computed between its own MFMA groups,
// and W^H streams from L2 one group ahead of its use.

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "bb_internal.h"

namespace bb {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));

#define BB_GLOBAL __attribute__((address_space(1)))
#define BB_LDS __attribute__((address_space(3)))

namespace {

__device__ __forceinline__ void phase_pair(const BB_LDS double* __restrict__ xs, double px, double py, double pz,
                                           float& c, float& s) {
  const double t = fma(xs[2], pz, fma(xs[1], py, xs[0] * px));
  const float f = (float)(t - rint(t));
  s = __builtin_amdgcn_sinf(f);
  c = __builtin_amdgcn_cosf(f);
}

// W^H operand: three planes (Wr - Wi, Wr, -Wi) of 32-eigenpair blocks in
// 32x32x2 order: lane = row + 32 * (antenna parity), float4 = 4 steps = 8
// antennas, vectors ordered (32-block, plane, 8-antenna group, lane).
__global__ __launch_bounds__(256) void fields_pack_kernel(const InstDesc* __restrict__ desc) {
  const InstDesc D = *desc;
  const int64_t total = (int64_t)D.K_alloc * 3 * D.L_pad / 4;
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= total) return;
  const int lane = (int)(idx % 64);
  int64_t rest = idx / 64;
  const int G8 = D.L_pad / 8;
  const int g = (int)(rest % G8);
  rest /= G8;
  const int q = (int)(rest % 3);
  const int kb = (int)(rest / 3);
  const int src = D.perm[kb * 32 + (lane & 31)];
  f32x4 out;
  for (int s = 0; s < 4; ++s) {
    const int l = 8 * g + 2 * s + (lane >> 5);
    float wr = 0.0f, wi = 0.0f;
    if (src >= 0 && l < D.L) {
      const float* w = (const float*)D.W + 2 * ((int64_t)src * D.W_ld + l);
      wr = w[0];
      wi = w[1];
    }
    out[s] = q == 0 ? wr - wi : (q == 1 ? wr : -wi);
  }
  ((f32x4*)D.apack)[idx] = out;
}

// NB 32-pixel blocks per wave; WK x WN waves along eigenpairs and along pixels.
template <int NB_, int WK_, int WN_>
struct Cfg {
  static constexpr int NB = NB_, WK = WK_, WN = WN_;
  static constexpr int THREADS = 64 * WK * WN;
  static constexpr int KC = 32 * WK;               // eigenpairs per pass
  static constexpr int NT = 32 * NB * WN;          // pixels per tile
  static constexpr int NCB = NT / 32;
  static constexpr int LCH = NT <= 128 ? 32 : 16;  // antennas per LDS chunk
  static constexpr int NG = LCH / 8;               // MFMA groups (8 antennas) per chunk
  static constexpr int JT = NT * (LCH / 4) / THREADS;  // (pixel, 4-antenna) phase tasks per thread
  static constexpr int PPG = 4 * JT / NG;          // phase pairs per MFMA group
  static_assert(THREADS % NT == 0 && NT % 64 == 0, "a thread keeps one pixel, a wave one antenna group per task");
  static_assert(JT >= 1 && NT * (LCH / 4) % THREADS == 0 && PPG * NG == 4 * JT, "whole tasks, split evenly");
  static_assert(kAntChunk % LCH == 0, "antenna padding covers the chunk");
};

template <class C>
__device__ __forceinline__ int task_group(int tid, int j) {
  return __builtin_amdgcn_readfirstlane((tid + j * C::THREADS) / C::NT);
}

template <class C>
__device__ __forceinline__ void gen_pairs(float (&cr)[4 * C::JT], float (&ci)[4 * C::JT],
                                          const BB_LDS double* __restrict__ xs_chunk, double px, double py, double pz,
                                          int tid, int first, int count) {
#pragma unroll
  for (int q = 0; q < 4 * C::JT; ++q)
    if (q >= first && q < first + count) {
      const int g4 = task_group<C>(tid, q >> 2);
      phase_pair(xs_chunk + 4 * (8 * (g4 >> 1) + 2 * (q & 3) + (g4 & 1)), px, py, pz, cr[q], ci[q]);
    }
}

// Planes Br, Bi - Br, Br + Bi of this thread's tasks.
template <class C>
__device__ __forceinline__ void gen_store(f32x4* __restrict__ buf, const float (&pr)[4 * C::JT],
                                          const float (&pi)[4 * C::JT], int tid) {
#pragma unroll
  for (int j = 0; j < C::JT; ++j) {
    const int pl = (tid + j * C::THREADS) % C::NT;
    const int g4 = task_group<C>(tid, j);
    const int g8 = g4 >> 1, h = g4 & 1;
    const float* cr = pr + 4 * j;
    const float* ci = pi + 4 * j;
    f32x4* const at = buf + (g8 * 3 * C::NCB + (pl >> 5)) * 64 + h * 32 + (pl & 31);
    at[0] = f32x4{cr[0], cr[1], cr[2], cr[3]};
    at[C::NCB * 64] = f32x4{ci[0] - cr[0], ci[1] - cr[1], ci[2] - cr[2], ci[3] - cr[3]};
    at[2 * C::NCB * 64] = f32x4{cr[0] + ci[0], cr[1] + ci[1], cr[2] + ci[2], cr[3] + ci[3]};
  }
}

struct AFrag {
  f32x4 v[3];
};

template <class C>
__global__ __launch_bounds__(C::THREADS) void fields_kernel(const FwdParams P) {
  constexpr int NB = C::NB;
  __shared__ f32x4 s_buf[2][C::NG * 3 * C::NCB * 64];
  __shared__ __align__(16) double s_xs[4 * kMaxAnt];
  const BB_LDS double* const xs = (const BB_LDS double*)s_xs;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wk = wave / C::WN;
  const int cb0 = (wave % C::WN) * NB;
  const InstDesc& Dg = *P.descs;
  const BB_GLOBAL f32x4* const A = (const BB_GLOBAL f32x4*)Dg.apack;
  const BB_GLOBAL double* const xs_g = (const BB_GLOBAL double*)Dg.xs;
  const int K_pad = __builtin_amdgcn_readfirstlane(P.dyn->K_pad);
  const int L_pad = __builtin_amdgcn_readfirstlane(Dg.L_pad);
  const int n_chunks = L_pad / C::LCH;
  const int n_pass = (K_pad + C::KC - 1) / C::KC;
  const int64_t a_stride = (int64_t)(L_pad / 8) * 64;  // vectors per plane
  for (int i = tid; i < 2 * L_pad; i += C::THREADS) ((f64x2*)s_xs)[i] = ((const BB_GLOBAL f64x2*)xs_g)[i];
  __syncthreads();
  for (int64_t tile = blockIdx.x; tile < P.n_tiles; tile += gridDim.x) {
    const int64_t p0 = tile * C::NT;
    int64_t pg = p0 + (tid % C::NT);
    if (pg >= P.n_pix) pg = P.n_pix - 1;
    const double px = P.pix[pg], py = P.pix[pg + P.pix_ld], pz = P.pix[pg + 2 * P.pix_ld];
    for (int pass = 0; pass < n_pass; ++pass) {
      const int kb = pass * (C::KC / 32) + wk;
      const bool active = kb < K_pad / 32;  // wave-uniform
      const int64_t a_base = (int64_t)kb * 3 * a_stride;
      auto load_a = [&](AFrag& a, int c, int g) {
        const int64_t o = a_base + (int64_t)(c * C::NG + g) * 64 + lane;
#pragma unroll
        for (int q = 0; q < 3; ++q) a.v[q] = A[o + q * a_stride];
      };
      f32x16 acc[3][NB];
#pragma unroll
      for (int t = 0; t < 3; ++t)
#pragma unroll
        for (int n = 0; n < NB; ++n)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[t][n][r] = 0.0f;
      AFrag a_cur;
      if (active) load_a(a_cur, 0, 0);
      float cr[4 * C::JT], ci[4 * C::JT];
      __syncthreads();  // previous users of s_buf are done
      gen_pairs<C>(cr, ci, xs, px, py, pz, tid, 0, 4 * C::JT);
      gen_store<C>(s_buf[0], cr, ci, tid);
      __syncthreads();
      for (int c = 0; c < n_chunks; ++c) {
        // the last chunk regenerates itself into the idle buffer, so that no branch splits the MFMA stream
        const int c_next = min(c + 1, n_chunks - 1);
        const BB_LDS double* const xs_next = xs + 4 * c_next * C::LCH;
        if (active) {
          // the second wave of each SIMD multiplies at a higher priority, which staggers the phase slices
          if (wave >= C::WK * C::WN / 2) __builtin_amdgcn_s_setprio(1);
          const f32x4* const buf = s_buf[c & 1];
#pragma unroll
          for (int g = 0; g < C::NG; ++g) {
            AFrag a_nxt;
            load_a(a_nxt, g + 1 < C::NG ? c : c_next, g + 1 < C::NG ? g + 1 : 0);
            gen_pairs<C>(cr, ci, xs_next, px, py, pz, tid, g * C::PPG, C::PPG);
            f32x4 b[3][NB];
#pragma unroll
            for (int q = 0; q < 3; ++q)
#pragma unroll
              for (int n = 0; n < NB; ++n) b[q][n] = buf[((g * 3 + q) * C::NCB + cb0 + n) * 64 + lane];
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
              for (int n = 0; n < NB; ++n)
#pragma unroll
                for (int q = 0; q < 3; ++q)
                  acc[q][n] = __builtin_amdgcn_mfma_f32_32x32x2f32(a_cur.v[q][s], b[q][n][s], acc[q][n], 0, 0, 0);
            a_cur = a_nxt;
            __builtin_amdgcn_sched_barrier(0);
          }
          if (wave >= C::WK * C::WN / 2) __builtin_amdgcn_s_setprio(0);
        } else {
          gen_pairs<C>(cr, ci, xs_next, px, py, pz, tid, 0, 4 * C::JT);
        }
        gen_store<C>(s_buf[(c + 1) & 1], cr, ci, tid);
        __syncthreads();
      }
      if (!active) continue;
#pragma unroll
      for (int n = 0; n < NB; ++n) {
        const int64_t p = p0 + (cb0 + n) * 32 + (lane & 31);
        if (p < P.n_pix) {
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int k = kb * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
            P.e_out[(int64_t)k * P.e_ld + p] = acc[0][n][r] - acc[2][n][r];
            P.e_out[(int64_t)(P.e_rows + k) * P.e_ld + p] = acc[0][n][r] + acc[1][n][r];
          }
        }
      }
    }
    __syncthreads();
  }
}

template <class C>
hipError_t launch(FwdParams p, hipStream_t s) {
  p.n_tiles = (p.n_pix + C::NT - 1) / C::NT;
  int64_t grid = resident_blocks((const void*)fields_kernel<C>, C::THREADS);
  if (grid > p.n_tiles) grid = p.n_tiles;
  hipLaunchKernelGGL(fields_kernel<C>, dim3((unsigned)grid), dim3(C::THREADS), 0, s, p);
  return hipGetLastError();
}

}  // namespace

// One shape per K class, so that no wave idles: K <= 32: 32 x 256, <= 64: 64 x 256,
// <= 128: 128 x 128, above: 256 x 64.
hipError_t launch_fields(const FwdParams& p, int K_alloc, int L_pad, hipStream_t s) {
  const int64_t vecs = (int64_t)K_alloc * 3 * L_pad / 4;
  hipLaunchKernelGGL(fields_pack_kernel, dim3((unsigned)((vecs + 255) / 256)), dim3(256), 0, s, p.descs);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  switch (synth_k_class(K_alloc)) {
    case 0: return launch<Cfg<1, 1, 8>>(p, s);
    case 1: return launch<Cfg<2, 2, 4>>(p, s);
    case 2: return launch<Cfg<2, 4, 2>>(p, s);
    default: return launch<Cfg<2, 8, 1>>(p, s);
  }
}

}  // namespace bb
