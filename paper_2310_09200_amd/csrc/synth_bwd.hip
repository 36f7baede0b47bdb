// Backward of the level images of one instance.
//
// Loss = sum_l sum_p g_lp I_lp with I_lp = sum_{k in l} d_k |E_kp|^2, E = W^H B,
// B_lp = exp(+j 2 pi <x_l, p> / lambda_w) (Sections 2.4 and 2.6).  With
// c_kp = g_{level(k), p}:
//   dd_k  = sum_p c_kp |E_kp|^2
//   M_kp  = d_k c_kp conj(E_kp)
//   dW_lk = 2 sum_p B_lp M_kp            (d/dRe W + j d/dIm W)
//   H_lp  = sum_k conj(W_lk) M_kp
//   dx_l  = -(4 pi / lambda_w) sum_p Im(H_lp B_lp) p
// E is recomputed on FP32 MFMA into HBM.  H runs on FP32 MFMA (32x32x2): dx is an
// FP64 result whose sums show every rounding of H.  dW, a complex64 result, runs on
// fp16 products of two-term splits.  The kernels work in level-sorted eigenpair order (the staging
// permutation) and
// the reduction writes results back in the caller's order.  Contractions over
// pixels are split into fixed pixel ranges whose FP64 partials are summed in a
// fixed order: the result is deterministic.

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "bb_internal.h"
#include "split.h"

namespace bb {

// Same phase evaluation as the forward kernels: xs = position / wavelength,
// exact FP64 reduction to [-1/2, 1/2] turns, hardware sine and cosine in turns.
__device__ __forceinline__ void phase_b(const double* __restrict__ xs, double px, double py, double pz, float& c,
                                        float& s) {
  const double t = fma(xs[2], pz, fma(xs[1], py, xs[0] * px));
  const float f = (float)(t - rint(t));
  s = __builtin_amdgcn_sinf(f);
  c = __builtin_amdgcn_cosf(f);
}

template <int N>
__device__ __forceinline__ double block_sum(double v, double* sh) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) sh[w] = v;
  __syncthreads();
  double t = 0.0;
  if (threadIdx.x == 0)
    for (int i = 0; i < N / 64; ++i) t += sh[i];
  __syncthreads();
  return t;
}

// M = d c conj(E) in place, dd partial sums, and the largest finite |Re M|, |Im M| of
// the split, negative (at least the smallest normal number) where some are infinite;
// grid (K_alloc, n_split), 256 threads.
__global__ __launch_bounds__(256) void bwd_m_kernel(const BwdParams P) {
  __shared__ double sh[4];
  __shared__ float shm[4];
  float top = 0.0f;
  bool wild = false;
  const int k = blockIdx.x;
  const int s = blockIdx.y;
  const InstDesc& D = *P.desc;
  const int lev = D.levs[k];
  const float w = D.wts[k];
  float* er = P.E + (int64_t)k * P.n_pix;
  float* ei = P.E + (int64_t)(P.K_alloc + k) * P.n_pix;
  const int64_t p0 = (int64_t)s * P.split_len;
  int64_t p1 = p0 + P.split_len;
  if (p1 > P.n_pix) p1 = P.n_pix;
  double acc = 0.0;
  if (lev < 0) {
    // padding / unused rows (the recompute leaves rows past K_pad unwritten)
    for (int64_t p = p0 + threadIdx.x; p < p1; p += blockDim.x) {
      er[p] = 0.0f;
      ei[p] = 0.0f;
    }
  } else {
    for (int64_t p = p0 + threadIdx.x; p < p1; p += blockDim.x) {
      const float c = P.gimg[(int64_t)lev * P.gimg_ld + p];
      const float a = er[p], b = ei[p];
      acc += (double)(c * fmaf(a, a, b * b));
      const float mr = w * c * a, mi = -w * c * b;
      er[p] = mr;
      ei[p] = mi;
      const float ar = fabsf(mr), ai = fabsf(mi);
      top = fmaxf(top, fmaxf(ar < INFINITY ? ar : 0.0f, ai < INFINITY ? ai : 0.0f));
      wild = wild || ar == INFINITY || ai == INFINITY;
    }
  }
  for (int o = 32; o > 0; o >>= 1) top = fmaxf(top, __shfl_xor(top, o));
  if ((threadIdx.x & 63) == 0) shm[threadIdx.x >> 6] = top;
  wild = __syncthreads_or(wild);
  const double t = block_sum<256>(acc, sh);
  if (threadIdx.x == 0) {
    P.dd_part[(int64_t)k * P.n_split + s] = t;
    top = fmaxf(fmaxf(shm[0], shm[1]), fmaxf(shm[2], shm[3]));
    P.m_top[(int64_t)k * P.n_split + s] = wild ? -fmaxf(top, 0x1p-126f) : top;
  }
}

typedef float bwd_f32x16 __attribute__((ext_vector_type(16)));

// One chunk's H block of a wave: H[l][p] += sum over 64 eigenpairs of
// conj(W)[l][k] M[k][p] for pixels 32 blk .. 32 blk + 31, real part (PART 0:
// Wr' Mr - Wi' Mi) or imaginary part (PART 1: Wr' Mi + Wi' Mr), W' = conj W.
// PART is a template argument and the loop is unrolled whole, so that it holds
// no branch: its LDS reads then run ahead of the MFMAs instead of each step
// waiting for its own.
// The real part takes -Wi' from the staged plane sWn (no negation per step).
template <int PART>
__device__ __forceinline__ void h_chunk(bwd_f32x16& h, const float2 (*sW)[65], const float (*sWn)[65],
                                        const float2 (*sM)[65], int blk, int lane) {
#pragma unroll
  for (int st = 0; st < 32; ++st) {
    const int kk = 2 * st + (lane >> 5);              // this lane's contraction row (eigenpair)
    const float2 w = sW[lane & 31][kk];               // A operand: row l = lane % 32
    const float2 m = sM[kk][32 * blk + (lane & 31)];  // B operand: column p = lane % 32 of the half
    if (PART == 0) {
      h = __builtin_amdgcn_mfma_f32_32x32x2f32(w.x, m.x, h, 0, 0, 0);
      h = __builtin_amdgcn_mfma_f32_32x32x2f32(sWn[lane & 31][kk], m.y, h, 0, 0, 0);
    } else {
      h = __builtin_amdgcn_mfma_f32_32x32x2f32(w.x, m.y, h, 0, 0, 0);
      h = __builtin_amdgcn_mfma_f32_32x32x2f32(w.y, m.x, h, 0, 0, 0);
    }
  }
}

// h_chunk over conj(W) staged once for every eigenpair of the instance (rows
// of WS, this slice's columns kc .. kc + 63); the real part negates Wi' per
// step.
template <int PART, int WS>
__device__ __forceinline__ void h_chunk_all(bwd_f32x16& h, const float2 (*sW)[WS], int kc, const float2 (*sM)[65],
                                            int blk, int lane) {
#pragma unroll
  for (int st = 0; st < 32; ++st) {
    const int kk = 2 * st + (lane >> 5);
    const float2 w = sW[lane & 31][kc + kk];
    const float2 m = sM[kk][32 * blk + (lane & 31)];
    if (PART == 0) {
      h = __builtin_amdgcn_mfma_f32_32x32x2f32(w.x, m.x, h, 0, 0, 0);
      h = __builtin_amdgcn_mfma_f32_32x32x2f32(-w.y, m.y, h, 0, 0, 0);
    } else {
      h = __builtin_amdgcn_mfma_f32_32x32x2f32(w.x, m.y, h, 0, 0, 0);
      h = __builtin_amdgcn_mfma_f32_32x32x2f32(w.y, m.x, h, 0, 0, 0);
    }
  }
}

// dW partial: sum over a split's pixels of B_lp M_kp for 128 antennas x 16 NKT
// eigenpairs.  512 threads: wave w takes antennas 32 (w / 2) .. + 31 of the block
// and pixels 32 (w % 2) .. + 31 of every 64-pixel chunk, on
// v_mfma_f32_16x16x32_f16 (A = phases, B = M; both operands hold 8 consecutive
// pixels per lane):
//   Re += Br Mr + Bi (-Mi),  Im += Br Mi + Bi Mr,
// each factor as hi + lo halves and three of the four half products.  A wave
// forms its phases where the matrix unit wants them, in registers; M is read
// once per 128 antennas, scaled by a power of two per eigenpair (its largest
// |M|, found when M was formed, becomes 2^14, so that a low half reaches 2^-38 of
// it), split and staged as planes [re hi, re lo, im hi, im lo][half][k][32 px],
// two chunks deep.
//   Three products at the fp16 rate (16 times FP32's) against one: 250 antennas,
// 121 eigenpairs, 500^2 pixels take 257 us against 693 on FP32 MFMA, and
// against 64 bits the result is closer (one rounding per 32 pixels in the split's
// sum: 5.5e-7 against 9.0e-7).
// A tile of 32 antennas x all eigenpairs keeps phases (a wave's 1200 cycles a
// chunk) below products (3072, NKT = 8).
typedef _Float16 bwd_f16x8 __attribute__((ext_vector_type(8)));
typedef float bwd_f32x4 __attribute__((ext_vector_type(4)));
typedef float bwd_f32x4u __attribute__((ext_vector_type(4), aligned(4)));

__device__ __forceinline__ bwd_f32x4 mfma_h(const uint4& a, const uint4& b, bwd_f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(bwd_f16x8, a), __builtin_bit_cast(bwd_f16x8, b), c,
                                                0, 0, 0);
}

template <int NKT>
__global__ __launch_bounds__(512, 2) void bwd_dw_kernel(const BwdParams P) {
  constexpr int K = 16 * NKT;       // eigenpairs of the block
  constexpr int PLANE = 2 * K * 4;  // 16-byte words of a plane: [half][k][4]
  constexpr int Q = NKT / 2;        // rows of M per thread and chunk, every 32nd
  extern __shared__ uint4 s_m[];    // [2][4][PLANE]; then the halves' exchange
  __shared__ double sP[2][3][64];
  __shared__ double sX[128][4];
  __shared__ int sE[K];  // exponent of each eigenpair's scale
  __shared__ int sWild[K];  // whether it has infinite values
  const InstDesc& D = *P.desc;
  const int l0 = blockIdx.x * 128, k0 = blockIdx.y * K, s = blockIdx.z;
  const int t = threadIdx.x, lane = t & 63, r16 = lane & 15, kq = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6), wl = wave >> 1, half = wave & 1;
  const bool live = l0 + 32 * wl < P.L_pad;  // the wave's antennas exist
  (&sX[0][0])[t] = l0 + (t >> 2) < P.L_pad ? D.xs[4 * l0 + t] : 0.0;
  {  // scales: 512 / K threads per eigenpair
    constexpr int TP = 512 / K;
    const int k = t / TP;
    float top = 0.0f;
    int wild = 0;
    if (k0 + k < P.K_alloc)
      for (int i = t % TP; i < P.n_split; i += TP) {
        const float m = P.m_top[(int64_t)(k0 + k) * P.n_split + i];
        top = fmaxf(top, fabsf(m));
        wild |= m < 0.0f;
      }
    for (int o = TP / 2; o > 0; o >>= 1) {
      top = fmaxf(top, __shfl_xor(top, o));
      wild |= __shfl_xor(wild, o);
    }
    // 2^-e top in [2^13, 2^14); within the range of a normal factor 2^-e
    const int e = top > 0.0f ? ilogbf(top) - 13 : 0;
    if (t % TP == 0) {
      sE[k] = max(-120, min(120, e));
      sWild[k] = wild;
    }
  }
  __syncthreads();
  const int64_t p0 = (int64_t)s * P.dw_len;
  const int64_t p1 = min(p0 + P.dw_len, P.n_pix);
  // M rows kr + 32 q, pixels 4 px .. + 3 of a chunk
  const int px = t & 15, kr = t >> 4;
  float scale[Q];
  unsigned wild = 0;  // bit q: row q has infinite values
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    scale[q] = __int_as_float((127 - sE[kr + 32 * q]) << 23);
    wild |= (unsigned)sWild[kr + 32 * q] << q;
  }
  // rows q0 .. q0 + Q / 2 - 1, real and imaginary parts, of the chunk at pc
  constexpr int QH = Q / 2;
  bwd_f32x4 next[2][QH];
  auto load = [&](int64_t pc, int q0) {
    const int64_t p = pc + 4 * px;
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int q = 0; q < QH; ++q) {
        const int k = k0 + kr + 32 * (q0 + q);
        const float* const row = P.E + ((int64_t)c * P.K_alloc + k) * P.n_pix;
        bwd_f32x4 v = {0.0f, 0.0f, 0.0f, 0.0f};
        if (k < P.K_alloc) {
          if (p + 4 <= p1) {
            v = *reinterpret_cast<const bwd_f32x4u*>(row + p);
          } else {
#pragma unroll
            for (int i = 0; i < 4; ++i)
              if (p + i < p1) v[i] = row[p + i];
          }
        }
        next[c][q] = v;
      }
  };
  auto store = [&](int buf, int q0) {
    uint2* const dst = reinterpret_cast<uint2*>(s_m + buf * 4 * PLANE);
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int q = 0; q < QH; ++q) {
        const bwd_f32x4 v = next[c][q] * scale[q0 + q];
        uint2 hi, lo;
        split2<_Float16>(v[0], v[1], hi.x, lo.x);
        split2<_Float16>(v[2], v[3], hi.y, lo.y);
        if (wild >> (q0 + q) & 1) {  // infinite values are low words alone: their products are infinite, not NaN
          uint16_t* const h = reinterpret_cast<uint16_t*>(&hi);
          uint16_t* const l = reinterpret_cast<uint16_t*>(&lo);
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (fabsf(v[i]) == INFINITY) l[i] = h[i], h[i] = 0;
        }
        // [half = px / 8][k][8 words of 8 bytes]
        const int at = ((px >> 3) * K + kr + 32 * (q0 + q)) * 8 + (px & 7);
        dst[2 * (2 * c) * PLANE + at] = hi;
        dst[2 * (2 * c + 1) * PLANE + at] = lo;
      }
  };
  double pnext = 0.0;
  auto load_pix = [&](int64_t pc) {
    const int64_t p = pc + (t & 63);
    if (t < 192) pnext = p < p1 ? P.pix[p + (t >> 6) * P.pix_ld] : 0.0;
  };
  load(p0, 0);
  store(0, 0);
  load(p0, QH);
  store(0, QH);
  load_pix(p0);
  if (t < 192) sP[0][t >> 6][t & 63] = pnext;
  bwd_f32x4 acc[2][NKT][2];  // [antennas][eigenpairs][re, im]
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < NKT; ++j) acc[i][j][0] = acc[i][j][1] = bwd_f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  int buf = 0;
  for (int64_t pc = p0; pc < p1; pc += 64, buf ^= 1) {
    const bool more = pc + 64 < p1;  // the same for the workgroup
    __syncthreads();
    if (more) {
      load(pc + 64, 0);
      load_pix(pc + 64);
    }
    uint4 bh[2][2], bl[2][2];  // phases [antennas][cos, sin], 8 pixels each
    if (live) {
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const double* const xs = sX[32 * wl + 16 * i + r16];
        const double x0 = xs[0], x1 = xs[1], x2 = xs[2];
        uint32_t* const ch = reinterpret_cast<uint32_t*>(&bh[i][0]);
        uint32_t* const cl = reinterpret_cast<uint32_t*>(&bl[i][0]);
        uint32_t* const sh = reinterpret_cast<uint32_t*>(&bh[i][1]);
        uint32_t* const sl = reinterpret_cast<uint32_t*>(&bl[i][1]);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          float c[2], sn[2];
#pragma unroll
          for (int v = 0; v < 2; ++v) {
            const int pp = 32 * half + 8 * kq + 2 * u + v;
            const double xsv[3] = {x0, x1, x2};
            phase_b(xsv, sP[buf][0][pp], sP[buf][1][pp], sP[buf][2][pp], c[v], sn[v]);
          }
          split2<_Float16>(c[0], c[1], ch[u], cl[u]);
          split2<_Float16>(sn[0], sn[1], sh[u], sl[u]);
        }
      }
    }
    const uint4* const m = s_m + buf * 4 * PLANE + half * K * 4 + r16 * 4 + kq;
    auto products = [&](int j) {
      const uint4 rh = m[j * 64], rl = m[PLANE + j * 64], ih = m[2 * PLANE + j * 64], il = m[3 * PLANE + j * 64];
      auto neg = [](uint4 v) {
        return make_uint4(v.x ^ 0x80008000u, v.y ^ 0x80008000u, v.z ^ 0x80008000u, v.w ^ 0x80008000u);
      };
      const uint4 nh = neg(ih), nl = neg(il);
      // the chunk's sum by itself, low products first, then one rounding in the
      // split's sum: [re, im] += cos x [Mr, Mi] + sin x [-Mi, Mr]
      bwd_f32x4 sum[2][2];
#pragma unroll
      for (int i = 0; i < 2; ++i) sum[i][0] = sum[i][1] = bwd_f32x4{0.0f, 0.0f, 0.0f, 0.0f};
      auto add = [&](const uint4(&b)[2][2], const uint4& mr, const uint4& mi, const uint4& mn) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          sum[i][0] = mfma_h(b[i][0], mr, sum[i][0]);
          sum[i][1] = mfma_h(b[i][0], mi, sum[i][1]);
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          sum[i][0] = mfma_h(b[i][1], mn, sum[i][0]);
          sum[i][1] = mfma_h(b[i][1], mr, sum[i][1]);
        }
      };
      add(bh, rl, il, nl);
      add(bl, rh, ih, nh);
      add(bh, rh, ih, nh);
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        acc[i][j][0] += sum[i][0];
        acc[i][j][1] += sum[i][1];
      }
    };
    if (live)
#pragma unroll
      for (int j = 0; j < NKT / 2; ++j) products(j);
    if (more) {
      store(buf ^ 1, 0);
      if (t < 192) sP[buf ^ 1][t >> 6][t & 63] = pnext;
      load(pc + 64, QH);
    }
    if (live)
#pragma unroll
      for (int j = NKT / 2; j < NKT; ++j) products(j);
    if (more) store(buf ^ 1, QH);
  }
  // the second halves' sums go through LDS to the first halves, real parts then imaginary
  float* const ex = reinterpret_cast<float*>(s_m) + wl * (2 * NKT * 4 * 64) + lane;
#pragma unroll
  for (int part = 0; part < 2; ++part) {
    __syncthreads();
    if (half == 1)
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < NKT; ++j)
#pragma unroll
          for (int r = 0; r < 4; ++r) ex[((i * NKT + j) * 4 + r) * 64] = acc[i][j][part][r];
    __syncthreads();
    if (half == 0 && live)
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < NKT; ++j) {
          const int k = 16 * j + r16;
          if (k0 + k >= P.K_alloc) continue;
          const double back = ldexp(1.0, sE[k]);
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int l = l0 + 32 * wl + 16 * i + 4 * kq + r;
            P.dW_part[(((int64_t)s * P.L_pad + l) * P.K_alloc + k0 + k) * 2 + part] =
                ((double)acc[i][j][part][r] + (double)ex[((i * NKT + j) * 4 + r) * 64]) * back;
          }
        }
  }
}

// dx partial: H_lp = sum_k conj(W_lk) M_kp on MFMA, then Im(H_lp B_lp) p
// summed over the split's pixels.  grid (L_pad/32, n_split), 256 threads.  The
// work runs in steps (64-pixel chunk, 64-eigenpair slice); each step stages
// conj(W) [32 l][64 k] and M [64 k][64 p] in LDS from registers loaded during
// the step before.  Wave w computes one real 32 x 32 block of H: pixel half
// w / 2, real part (w even: Wr Mr - Wi' Mi with W' = conj W) or imaginary part
// (w odd: Wr' Mi + Wi' Mr).  After a chunk's last slice the blocks go through
// LDS (pixel-major, rows padded to 33) to the threads that own (antenna t % 32,
// pixels t / 32 + 8 j), which evaluate the phases.  WONCE (K_alloc <= 128):
// conj(W) of all the instance's eigenpairs is staged once, and the steps
// stage only M.
template <int KONCE>
__global__ __launch_bounds__(256, KONCE == 64 ? 3 : 2) void bwd_dx_kernel(const BwdParams P) {
  __shared__ float2 sW[32][65];   // conj(W) for 32 antennas x 64 eigenpairs (+1 pad: column reads)
  __shared__ float sWn[32][65];   // its negated imaginary parts
  __shared__ float2 sM[64][65];   // M for 64 eigenpairs x 64 pixels; then H re / im [2][64 p][33] floats
  __shared__ double sP[3][64];    // the chunk's pixel coordinates
  __shared__ double sX[32][4];    // the tile's scaled antenna positions
  __shared__ int sOff[kMaxEig];   // staged eigenpair -> offset of its column of W (src * L), -1 if none
  constexpr bool WONCE = KONCE > 0;
  __shared__ float2 sWall[32][KONCE + 1];  // WONCE: conj(W) for 32 antennas x KONCE eigenpairs (+1 pad)
  const InstDesc& D = *P.desc;
  const int l0 = blockIdx.x * 32, s = blockIdx.y;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int tl = t & 31, tp = t >> 5;
  const int l = l0 + tl;
  if (t < 128) (&sX[0][0])[t] = D.xs[4 * l0 + t];  // rows l0 .. l0 + 31 < L_pad
  // this wave's H block: pixel half, re / im (wave-uniform, held in scalar registers)
  const int blk = __builtin_amdgcn_readfirstlane(wave >> 1), part = __builtin_amdgcn_readfirstlane(wave & 1);
  const int64_t p0 = (int64_t)s * P.split_len;
  int64_t p1 = p0 + P.split_len;
  if (p1 > P.n_pix) p1 = P.n_pix;
  const int K_pad = P.dyn->K_pad;
  const int n_kc = K_pad > 64 ? (K_pad + 63) / 64 : 1;  // slices per chunk (one of zeros if K_pad = 0)
  const float* Er = P.E;
  const float* Ei = P.E + (int64_t)P.K_alloc * P.n_pix;
  const float* Wf = (const float*)P.W;
  float* const sH = reinterpret_cast<float*>(&sM[0][0]);  // [2 parts][64 p][33]
  // The next step's M (16 values per thread: eigenpair 4 j + t / 64 of the
  // slice, pixel t % 64), conj(W) (8 per thread: antenna t % 32, eigenpair
  // t / 32 + 8 j of the slice, so that a wave reads 32 consecutive antennas
  // of a column of W) and, for a new chunk, pixel coordinates.  Lanes outside
  // the split, K_pad or the antennas load a valid address and keep zeros.
  float2 mnext[16], wnext[8];
  double pnext = 0.0;
  auto load_step = [&](int64_t pc, int kc) {
    const int64_t p = pc + (t & 63);
    const bool p_ok = p < p1;
    const int64_t pq = p_ok ? p : p1 - 1;
    const int64_t r0 = (int64_t)(kc + (t >> 6)) * P.n_pix + pq, st4 = 4 * P.n_pix;  // rows advance by 4 per j
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const int k = kc + 4 * j + (t >> 6);
      const int64_t e = k < K_pad ? r0 + j * st4 : pq;
      const float er = Er[e], ei = Ei[e];
      mnext[j] = (p_ok && k < K_pad) ? make_float2(er, ei) : make_float2(0.0f, 0.0f);
    }
    const bool l_ok = l0 + tl < P.L;
#pragma unroll
    for (int j = 0; j < 8 && !WONCE; ++j) {
      const int k = kc + tp + 8 * j;
      const int off = sOff[k];
      const bool ok = l_ok && off >= 0;
      const float* w = Wf + 2 * ((int64_t)(ok ? off : 0) + (l_ok ? l0 + tl : 0));
      float wr = w[0], wi = w[1];
      // keep the loads unconditional (a load the compiler moves under `ok`
      // becomes a branch per element)
      asm volatile("" : "+v"(wr), "+v"(wi));
      wnext[j] = ok ? make_float2(wr, -wi) : make_float2(0.0f, 0.0f);
    }
    if (kc == 0 && t < 192) pnext = p_ok ? P.pix[pq + (t >> 6) * P.pix_ld] : 0.0;
  };
  if constexpr (WONCE) {
    for (int i = t; i < 32 * KONCE; i += 256) {
      const int ll = i & 31, kk = i >> 5;  // a wave reads 32 consecutive antennas of two columns of W
      const int src = kk < K_pad ? D.perm[kk] : -1;
      float2 wv = make_float2(0.0f, 0.0f);
      if (l0 + ll < P.L && src >= 0) {
        const float* w = Wf + 2 * ((int64_t)src * P.L + l0 + ll);
        wv = make_float2(w[0], -w[1]);
      }
      sWall[ll][kk] = wv;
    }
  } else {
    for (int k = t; k < 64 * n_kc; k += 256) {  // 64 n_kc <= kMaxEig
      const int src = k < K_pad ? D.perm[k] : -1;
      sOff[k] = src >= 0 ? src * P.L : -1;
    }
  }
  __syncthreads();
  load_step(p0, 0);
  double gx = 0.0, gy = 0.0, gz = 0.0;
  for (int64_t pc = p0; pc < p1; pc += 64) {
    bwd_f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
    for (int kq = 0; kq < n_kc; ++kq) {
#pragma unroll
      for (int j = 0; j < 16; ++j) sM[4 * j + (t >> 6)][t & 63] = mnext[j];
      if constexpr (!WONCE) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          sW[tl][tp + 8 * j] = wnext[j];
          sWn[tl][tp + 8 * j] = -wnext[j].y;
        }
      }
      if (kq == 0 && t < 192) sP[t >> 6][t & 63] = pnext;
      __syncthreads();
      // the next step: the chunk's next slice, else the next chunk's first
      const bool last = kq + 1 == n_kc;
      const int64_t npc = last ? pc + 64 : pc;
      if (npc < p1) load_step(npc, last ? 0 : 64 * (kq + 1));  // workgroup-uniform
      if constexpr (WONCE) {
        if (part == 0)
          h_chunk_all<0, KONCE + 1>(acc, sWall, 64 * kq, sM, blk, lane);
        else
          h_chunk_all<1, KONCE + 1>(acc, sWall, 64 * kq, sM, blk, lane);
      } else {
        if (part == 0)
          h_chunk<0>(acc, sW, sWn, sM, blk, lane);
        else
          h_chunk<1>(acc, sW, sWn, sM, blk, lane);
      }
      __syncthreads();
    }
    // register r of lane q holds H at (l, p) = (8 (r / 4) + 4 (q / 32) + r % 4, 32 blk + q % 32)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int ll = 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
      sH[(part * 64 + 32 * blk + (lane & 31)) * 33 + ll] = acc[r];
    }
    __syncthreads();
    if (l < P.L) {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        // pixels past the split add exact zeros (their M and hence H, and
        // coordinates are 0)
        const int pp = tp + 8 * j;
        const double px = sP[0][pp], py = sP[1][pp], pz = sP[2][pp];
        float c, sn;
        phase_b(&sX[tl][0], px, py, pz, c, sn);
        const float hr = sH[pp * 33 + tl], hi = sH[(64 + pp) * 33 + tl];
        const double v = (double)fmaf(hr, sn, hi * c);  // Im(H B)
        gx += v * px;
        gy += v * py;
        gz += v * pz;
      }
    }
    __syncthreads();  // sH (in sM) and sP are restaged by the next chunk
  }
  double* const sh = reinterpret_cast<double*>(&sM[0][0]);  // [3][256]; sM is free after the loop
  sh[t] = gx;
  sh[256 + t] = gy;
  sh[512 + t] = gz;
  __syncthreads();
  if (tp == 0 && l < P.L_pad) {
    double a = 0, b = 0, c = 0;
    for (int j = 0; j < 8; ++j) {
      a += sh[t + 32 * j];
      b += sh[256 + t + 32 * j];
      c += sh[512 + t + 32 * j];
    }
    double* o = P.dx_part + ((int64_t)s * P.L_pad + l) * 3;
    o[0] = a;
    o[1] = b;
    o[2] = c;
  }
}

// dW and dd of eigenpairs outside every level are zero.
__global__ __launch_bounds__(256) void bwd_zero_kernel(int64_t n_w, int K, float* __restrict__ dW,
                                                       float* __restrict__ dd) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx < n_w) {
    dW[2 * idx] = 0.0f;
    dW[2 * idx + 1] = 0.0f;
  }
  if (idx < K) dd[idx] = 0.0f;
}

// Fixed-order sums over splits, scattered back to the caller's eigenpair order.
// Bound by reads in flight (67 MB for 256 antennas and 64 eigenpairs): one wave
// per workgroup spreads them over the chip.
__global__ __launch_bounds__(64) void bwd_reduce_kernel(const BwdParams P, float* __restrict__ dW,
                                                         float* __restrict__ dd, double* __restrict__ dx) {
  const InstDesc& D = *P.desc;
  const int K_pad = P.dyn->K_pad;
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx < (int64_t)P.L * K_pad) {
    // consecutive threads take consecutive eigenpairs: their partials are adjacent
    const int k = (int)(idx % K_pad), l = (int)(idx / K_pad);
    const int src = D.perm[k];
    if (src >= 0) {
      double re = 0.0, im = 0.0;
#pragma unroll 8
      for (int s = 0; s < P.n_dw; ++s) {
        const double* q = P.dW_part + (((int64_t)s * P.L_pad + l) * P.K_alloc + k) * 2;
        re += q[0];
        im += q[1];
      }
      dW[2 * ((int64_t)src * P.L + l)] = (float)(2.0 * re);
      dW[2 * ((int64_t)src * P.L + l) + 1] = (float)(2.0 * im);
      if (l == 0) {
        double a = 0.0;
#pragma unroll 8
        for (int s = 0; s < P.n_split; ++s) a += P.dd_part[(int64_t)k * P.n_split + s];
        dd[src] = (float)a;
      }
    }
  }
  if (idx < (int64_t)P.L * 3) {
    const int l = (int)(idx % P.L), c = (int)(idx / P.L);
    double a = 0.0;
#pragma unroll 8
    for (int s = 0; s < P.n_split; ++s) a += P.dx_part[((int64_t)s * P.L_pad + l) * 3 + c];
    dx[(int64_t)c * P.L + l] = P.scale_x * a;
  }
}

hipError_t launch_backward(const BwdParams& p, hipStream_t s) {
  hipLaunchKernelGGL(bwd_m_kernel, dim3(p.K_alloc, p.n_split), dim3(256), 0, s, p);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  auto dw = [&](auto* fn, int nkt) -> hipError_t {
    const size_t lds = (size_t)2 * 4 * (2 * 16 * nkt * 4) * sizeof(uint4);
    const hipError_t r = hipFuncSetAttribute(reinterpret_cast<const void*>(fn),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (r != hipSuccess) return r;
    hipLaunchKernelGGL(fn, dim3((p.L_pad + 127) / 128, (p.K_alloc + 16 * nkt - 1) / (16 * nkt), p.n_dw), dim3(512),
                       lds, s, p);
    return hipGetLastError();
  };
  e = p.K_alloc <= 64 ? dw(&bwd_dw_kernel<4>, 4) : dw(&bwd_dw_kernel<8>, 8);
  if (e != hipSuccess) return e;
  auto* const dx = p.K_alloc <= 64 ? &bwd_dx_kernel<64> : p.K_alloc <= 128 ? &bwd_dx_kernel<128> : &bwd_dx_kernel<0>;
  hipLaunchKernelGGL(dx, dim3(p.L_pad / 32, p.n_split), dim3(256), 0, s, p);
  return hipGetLastError();
}

hipError_t launch_backward_reduce(const BwdParams& p, void* dW, float* dd, double* dx, hipStream_t s) {
  const int64_t n_w = (int64_t)p.L * p.K;
  int64_t n = n_w > p.K ? n_w : p.K;
  hipLaunchKernelGGL(bwd_zero_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, n_w, p.K,
                     static_cast<float*>(dW), dd);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  n = (int64_t)p.L * p.K_alloc;
  if (n < (int64_t)p.L * 3) n = (int64_t)p.L * 3;
  hipLaunchKernelGGL(bwd_reduce_kernel, dim3((unsigned)((n + 63) / 64)), dim3(64), 0, s, p,
                     static_cast<float*>(dW), dd, dx);
  return hipGetLastError();
}

}  // namespace bb
