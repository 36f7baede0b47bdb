// Line FFTs of the NUFFT's pruned type-2 transform (gfx950): of a line's L = M
// points N <= M are stored (index i holds frequency i for i < N/2, else i - N;
// the others are zero), each is divided by the axis's kernel transform on load,
// and of the inverse DFT X[m] = sum_n x[n] exp(+2 pi i n m / M) (unnormalised)
// only the window (lo + w) mod M, w < len, is kept.  Three kernels:
//
//   line_reg_kernel   lengths that are products of two or three radices up to 20
//                     (most 2,3,5-smooth lengths up to 8000): a butterfly per
//                     thread and pass, in registers;
//   line_fft_kernel   any other 2,3,5-smooth length up to 16384, in place in LDS;
//   line_dft_kernel   at most 64 points (the thin axis of a grid): a direct
//                     pruned DFT on MFMA.
//
// line_fft_kernel:
// Each workgroup transforms one or more lines of L = M points held in LDS
// (L 2,3,5-smooth, at most 16384), in place by mixed-radix decimation in time (radix 8,
// 4, 2, 3, 5 in the order R_0, R_1, ...): pass s combines R_s transforms of
// length Ns = R_0 ... R_{s-1} that sit Ns apart into one of length P = Ns R_s,
// each butterfly reading and writing the same R_s points (twiddles
// exp(2 pi i k r / P)).  For that the load puts input n at the digit-reversed
// position sum_s r_s Ns_s, where n = r_{S-1} + R_{S-1} (r_{S-2} + R_{S-2} (...)),
// from a table made on the host.  One LDS buffer of L x 8 bytes per
// line.  Twiddles come from a table made in FP64 on the host: pass s keeps
// its Ns (R_s - 1) values exp(2 pi i k r / P), k < Ns, 1 <= r < R_s, at
// offset Ns - 1 (the earlier passes hold sum (P - Ns) = Ns - 1 of them), so
// a butterfly reads its R - 1 twiddles as one contiguous run.  Index
// quotients use an FP32 reciprocal: for j, d <= 16384, (j + 1/2) / d is at
// least 1/(2d) from an integer and the rounding error stays below that.

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>
#include <utility>

#include "bb_internal.h"

namespace bb {

namespace {

__device__ __forceinline__ float2 cmul(float2 a, float2 b) {
  return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ float2 mul_i(float2 a) { return make_float2(-a.y, a.x); }  // i a

// Inverse DFTs of size R in place: y[q] = sum_r v[r] exp(+2 pi i r q / R).
template <int R>
__device__ __forceinline__ void small_dft(float2 (&v)[R]);

template <>
__device__ __forceinline__ void small_dft<2>(float2 (&v)[2]) {
  const float2 a = v[0], b = v[1];
  v[0] = cadd(a, b);
  v[1] = csub(a, b);
}

template <>
__device__ __forceinline__ void small_dft<4>(float2 (&v)[4]) {
  const float2 s02 = cadd(v[0], v[2]), d02 = csub(v[0], v[2]);
  const float2 s13 = cadd(v[1], v[3]), d13 = mul_i(csub(v[1], v[3]));
  v[0] = cadd(s02, s13);
  v[1] = cadd(d02, d13);
  v[2] = csub(s02, s13);
  v[3] = csub(d02, d13);
}

template <>
__device__ __forceinline__ void small_dft<8>(float2 (&v)[8]) {
  float2 e[4] = {v[0], v[2], v[4], v[6]};
  float2 o[4] = {v[1], v[3], v[5], v[7]};
  small_dft<4>(e);
  small_dft<4>(o);
  constexpr float h = 0.70710678118654752440f;  // 1 / sqrt(2)
  const float2 o1 = make_float2(h * (o[1].x - o[1].y), h * (o[1].x + o[1].y));    // (1 + i)/sqrt2
  const float2 o2 = mul_i(o[2]);                                                   // i
  const float2 o3 = make_float2(-h * (o[3].x + o[3].y), h * (o[3].x - o[3].y));   // (-1 + i)/sqrt2
  v[0] = cadd(e[0], o[0]);
  v[4] = csub(e[0], o[0]);
  v[1] = cadd(e[1], o1);
  v[5] = csub(e[1], o1);
  v[2] = cadd(e[2], o2);
  v[6] = csub(e[2], o2);
  v[3] = cadd(e[3], o3);
  v[7] = csub(e[3], o3);
}

template <>
__device__ __forceinline__ void small_dft<3>(float2 (&v)[3]) {
  constexpr float s = 0.86602540378443864676f;  // sin(2 pi / 3)
  const float2 a = v[0], p = cadd(v[1], v[2]), m = csub(v[1], v[2]);
  const float2 t = make_float2(a.x - 0.5f * p.x, a.y - 0.5f * p.y);
  const float2 u = make_float2(-s * m.y, s * m.x);  // i s (b - c)
  v[0] = cadd(a, p);
  v[1] = cadd(t, u);
  v[2] = csub(t, u);
}

template <>
__device__ __forceinline__ void small_dft<5>(float2 (&v)[5]) {
  constexpr float c1 = 0.30901699437494742410f;   // cos(2 pi / 5)
  constexpr float c2 = -0.80901699437494742410f;  // cos(4 pi / 5)
  constexpr float s1 = 0.95105651629515357212f;   // sin(2 pi / 5)
  constexpr float s2 = 0.58778525229247312917f;   // sin(4 pi / 5)
  const float2 a = v[0];
  const float2 p14 = cadd(v[1], v[4]), m14 = csub(v[1], v[4]);
  const float2 p23 = cadd(v[2], v[3]), m23 = csub(v[2], v[3]);
  const float2 r1 = make_float2(a.x + c1 * p14.x + c2 * p23.x, a.y + c1 * p14.y + c2 * p23.y);
  const float2 r2 = make_float2(a.x + c2 * p14.x + c1 * p23.x, a.y + c2 * p14.y + c1 * p23.y);
  // i (s1 m14 + s2 m23) and i (s2 m14 - s1 m23)
  const float2 j1 = mul_i(make_float2(s1 * m14.x + s2 * m23.x, s1 * m14.y + s2 * m23.y));
  const float2 j2 = mul_i(make_float2(s2 * m14.x - s1 * m23.x, s2 * m14.y - s1 * m23.y));
  v[0] = make_float2(a.x + p14.x + p23.x, a.y + p14.y + p23.y);
  v[1] = cadd(r1, j1);
  v[4] = csub(r1, j1);
  v[2] = cadd(r2, j2);
  v[3] = csub(r2, j2);
}

// Composite sizes R = A B with A, B coprime (no twiddles): with inputs
// n = B n1 + A n2 and outputs k = k1 mod A = k2 mod B (both mod R),
// exp(2 pi i n k / R) = exp(2 pi i n1 k1 / A) exp(2 pi i n2 k2 / B).
template <int A, int B>
__device__ __forceinline__ void coprime_dft(float2 (&v)[A * B]) {
  constexpr int R = A * B;
  float2 y[A][B];
#pragma unroll
  for (int n2 = 0; n2 < B; ++n2) {
    float2 x[A];
#pragma unroll
    for (int n1 = 0; n1 < A; ++n1) x[n1] = v[(B * n1 + A * n2) % R];
    small_dft<A>(x);
#pragma unroll
    for (int k1 = 0; k1 < A; ++k1) y[k1][n2] = x[k1];
  }
#pragma unroll
  for (int k1 = 0; k1 < A; ++k1) {
    small_dft<B>(y[k1]);
#pragma unroll
    for (int k = 0; k < R; ++k)
      if (k % A == k1) v[k] = y[k1][k % B];
  }
}

template <>
__device__ __forceinline__ void small_dft<9>(float2 (&v)[9]) {
  // exp(2 pi i p / 9) for p = 1, 2, 4
  constexpr float2 w1 = {0.76604444311897803520f, 0.64278760968653932632f};
  constexpr float2 w2 = {0.17364817766693034885f, 0.98480775301220805937f};
  constexpr float2 w4 = {-0.93969262078590838405f, 0.34202014332566873304f};
  float2 y[3][3];  // [k1][n2]
#pragma unroll
  for (int n2 = 0; n2 < 3; ++n2) {
    float2 x[3] = {v[n2], v[3 + n2], v[6 + n2]};
    small_dft<3>(x);
#pragma unroll
    for (int k1 = 0; k1 < 3; ++k1) y[k1][n2] = x[k1];
  }
  y[1][1] = cmul(y[1][1], w1);
  y[2][1] = cmul(y[2][1], w2);
  y[1][2] = cmul(y[1][2], w2);
  y[2][2] = cmul(y[2][2], w4);
#pragma unroll
  for (int k1 = 0; k1 < 3; ++k1) {
    small_dft<3>(y[k1]);
#pragma unroll
    for (int k2 = 0; k2 < 3; ++k2) v[k1 + 3 * k2] = y[k1][k2];
  }
}

template <>
__device__ __forceinline__ void small_dft<16>(float2 (&v)[16]) {
  constexpr float c = 0.92387953251128675613f, s = 0.38268343236508977173f;  // cos, sin of pi / 8
  constexpr float h = 0.70710678118654752440f;
  constexpr float2 w[10] = {{1, 0}, {c, s}, {h, h}, {s, c}, {0, 1}, {-s, c}, {-h, h}, {-c, s}, {-1, 0}, {-c, -s}};
  float2 y[4][4];  // [k1][n2]
#pragma unroll
  for (int n2 = 0; n2 < 4; ++n2) {
    float2 x[4] = {v[n2], v[4 + n2], v[8 + n2], v[12 + n2]};
    small_dft<4>(x);
#pragma unroll
    for (int k1 = 0; k1 < 4; ++k1) y[k1][n2] = n2 * k1 == 0 ? x[k1] : n2 * k1 == 4 ? mul_i(x[k1]) : cmul(x[k1], w[n2 * k1]);
  }
#pragma unroll
  for (int k1 = 0; k1 < 4; ++k1) {
    small_dft<4>(y[k1]);
#pragma unroll
    for (int k2 = 0; k2 < 4; ++k2) v[k1 + 4 * k2] = y[k1][k2];
  }
}

template <>
__device__ __forceinline__ void small_dft<6>(float2 (&v)[6]) { coprime_dft<2, 3>(v); }
template <>
__device__ __forceinline__ void small_dft<10>(float2 (&v)[10]) { coprime_dft<2, 5>(v); }
template <>
__device__ __forceinline__ void small_dft<12>(float2 (&v)[12]) { coprime_dft<4, 3>(v); }
template <>
__device__ __forceinline__ void small_dft<15>(float2 (&v)[15]) { coprime_dft<3, 5>(v); }
template <>
__device__ __forceinline__ void small_dft<18>(float2 (&v)[18]) { coprime_dft<2, 9>(v); }
template <>
__device__ __forceinline__ void small_dft<20>(float2 (&v)[20]) { coprime_dft<4, 5>(v); }

// floor(j / d) for 0 <= j, 1 <= d <= 16384, given inv_d = 1 / d in FP32.
__device__ __forceinline__ int quot(int j, float inv_d) { return (int)(((float)j + 0.5f) * inv_d); }

// One in-place decimation-in-time pass of radix R over nl lines of L points
// (nl = 1 unless MULTI); tw holds this pass's twiddles, [k][r - 1].
// LDS position of point i of the lines: with PAD one spare point after every
// 32, which spreads the power-of-two strides of the early radix-8 passes of
// a line with many factors of 2 over the banks (one long line per workgroup).
template <bool PAD>
__device__ __forceinline__ int padi(int i) { return PAD ? i + (i >> 5) : i; }

template <int R, int T, bool MULTI, bool PAD>
__device__ __forceinline__ void dit_pass(float2* s, int L, int nl, int Ns, const float2* __restrict__ tw) {
  const int per_line = L / R;
  const int nb = nl * per_line;
  const int P = Ns * R;
  const float inv_pl = 1.0f / (float)per_line, inv_ns = 1.0f / (float)Ns;
  for (int j = threadIdx.x; j < nb; j += T) {
    const int line = MULTI ? quot(j, inv_pl) : 0, jj = j - line * per_line;
    const int g = quot(jj, inv_ns), k = jj - g * Ns;
    const int base = line * L + g * P + k;
    const float2* const w = tw + k * (R - 1);
    float2 v[R];
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = s[padi<PAD>(base + r * Ns)];
#pragma unroll
    for (int r = 1; r < R; ++r) v[r] = cmul(v[r], w[r - 1]);
    small_dft<R>(v);
#pragma unroll
    for (int r = 0; r < R; ++r) s[padi<PAD>(base + r * Ns)] = v[r];
  }
  __syncthreads();
}

// nl lines of L points per workgroup (nl = 1 unless MULTI), T threads.
template <int T, bool MULTI, bool PAD>
__global__ __launch_bounds__(T) void line_fft_kernel(LineFft p, const float2* __restrict__ in,
                                                     const float* __restrict__ inv_psi, const int* __restrict__ perm,
                                                     const float2* __restrict__ tw, float2* __restrict__ out) {
  extern __shared__ float2 s_line[];  // nl x L points
  const int L = p.L, nl = MULTI ? p.nl : 1;
  const int n_in = p.n_in, half = n_in / 2, gap = L - n_in;
  const int in_stride = (int)p.in_stride;
  const int tid = threadIdx.x;
  const float inv_nin = 1.0f / (float)n_in;
  for (int64_t l0 = (int64_t)blockIdx.x * nl; l0 < p.n_lines; l0 += (int64_t)gridDim.x * nl) {
    const int nh = MULTI ? (int)min<int64_t>(nl, p.n_lines - l0) : 1;
    // zero the lines (L is even), then place the stored inputs: input i of a
    // line holds the frequency at position m (i, or i + M - N for the
    // negative half), which the passes want at perm[m]
    float4* const z = reinterpret_cast<float4*>(s_line);
    for (int e = tid; e < (padi<PAD>(nl * L) + 1) / 2; e += T) z[e] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    __syncthreads();
    const float2* const src = in + l0 * p.in_stride;
#pragma unroll 4
    for (int e = tid; e < nh * n_in; e += T) {
      const int l = MULTI ? quot(e, inv_nin) : 0;
      const int i = e - l * n_in;
      const int m = i < half ? i : i + gap;
      const float2 x = src[l * in_stride + i];
      const float sc = inv_psi[i];
      s_line[padi<PAD>(l * L + perm[m])] = make_float2(x.x * sc, x.y * sc);
    }
    __syncthreads();
    int Ns = 1;
    for (int ps = 0; ps < p.n_pass; ++ps) {
      const int R = (int)((p.radix_codes >> (4 * ps)) & 15);
      switch (R) {
        case 8: dit_pass<8, T, MULTI, PAD>(s_line, L, nl, Ns, tw + (Ns - 1)); break;
        case 4: dit_pass<4, T, MULTI, PAD>(s_line, L, nl, Ns, tw + (Ns - 1)); break;
        case 2: dit_pass<2, T, MULTI, PAD>(s_line, L, nl, Ns, tw + (Ns - 1)); break;
        case 3: dit_pass<3, T, MULTI, PAD>(s_line, L, nl, Ns, tw + (Ns - 1)); break;
        default: dit_pass<5, T, MULTI, PAD>(s_line, L, nl, Ns, tw + (Ns - 1)); break;
      }
      Ns *= R;
    }
    const int wl = p.win_len, lo = p.win_lo;
    if (p.out_mode == 0) {  // out[line][w]
      float2* const dst = out + l0 * p.out_stride;
      const int os = (int)p.out_stride;
      const float inv_wl = 1.0f / (float)wl;
      for (int e = tid; e < nh * wl; e += T) {
        const int l = MULTI ? quot(e, inv_wl) : 0, w = e - l * wl;
        const int m = lo + w < L ? lo + w : lo + w - L;
        dst[l * os + w] = s_line[padi<PAD>(l * L + m)];
      }
    } else {  // lines are (outer, inner), inner < t_inner: out[outer][w][inner]
      const int64_t outer0 = l0 / p.t_inner;
      const int inner0 = (int)(l0 - outer0 * p.t_inner);
      const int ti = (int)p.t_inner;
      float2* const dst = out + outer0 * wl * p.t_inner + inner0;
      const float inv_nh = 1.0f / (float)nh, inv_ti = 1.0f / (float)ti;
      for (int e = tid; e < nh * wl; e += T) {
        const int w = quot(e, inv_nh), l = e - w * nh;
        const int q = quot(inner0 + l, inv_ti);  // (inner0 + l) / t_inner
        const int m = lo + w < L ? lo + w : lo + w - L;
        dst[(q * wl + w) * ti + l - q * ti] = s_line[padi<PAD>(l * L + m)];
      }
    }
    __syncthreads();  // the lines are reused by the next group
  }
}

// L = R1 R2 R3 (R2 = 1: two passes), self-sorting: the pass of radix R after
// passes of product Ns takes the points j + r L / R of butterfly j < L / R, times
// exp(2 pi i r (j mod Ns) / (Ns R)), and leaves output q at (j div Ns) Ns R +
// j mod Ns + q Ns.  The first pass reads the line from memory (a butterfly's
// points at a stride of L / R1: whole cache lines over the threads) and the last
// one writes the window to memory, so LDS sees each point once per pass between
// them and nothing is zeroed, placed or copied out.  There it is held in rows of
// R1 points P1 apart, and after the second pass of R1 R2 points P2 apart: P1 odd,
// and P2 = R1 modulo 32, which spreads the strided writes over the banks and
// leaves every read a constant stride.  A butterfly of every pass per thread; the
// last pass's twiddles are requested before the barrier that it waits at.  The
// radices are constants: with a switch over them addresses and windows took as
// many instructions as the butterflies (360 us).
//
// 32 k lines of 3200 or 3240 points, half of them stored and half kept (0.83 GB,
// 0.17 ms): 250 us, the vector units 70 to 74 % busy; 440 and 540 us in line_fft_kernel
// (six or seven passes through LDS with bank conflicts in the early ones).  A
// workgroup takes one set of lines: as a loop over lines with the twiddles kept
// (in LDS or registers) fewer workgroups fit a CU and it took 500 us.
template <int R1, int R2, int R3>
struct RegGeom {
  static constexpr int L = R1 * R2 * R3;
  static constexpr int S1 = L / R1, S2 = L / R2, S3 = R1 * R2;  // butterflies of the passes
  static constexpr int T = std::max(std::max(S1, S3), R2 > 1 ? S2 : 0);
  static constexpr int NL = std::max(1, 256 / T);  // lines per workgroup
  static constexpr int TPB = (NL * T + 63) / 64 * 64;
  // waves per SIMD: a radix above 16 needs more than the 96 registers of five
  static constexpr int WAVES = std::max(std::max(R1, R2), R3) > 16 ? 4 : 5;
  static constexpr int P1 = R1 | 1;
  static constexpr int P2 = R2 == 1 ? P1 : S3 + ((R1 - S3) % 32 + 32) % 32;
  static constexpr int POINTS = std::max(S1 * P1, R2 == 1 ? 0 : R3 * P2);  // of LDS per line
  static constexpr size_t LDS = ((size_t)NL * POINTS + (R2 > 1 ? S3 : 0)) * sizeof(float2);
};

template <int R1, int R2, int R3>
__global__ __launch_bounds__((RegGeom<R1, R2, R3>::TPB), (RegGeom<R1, R2, R3>::WAVES)) void line_reg_kernel(LineFft p,
                                                                                 const float2* __restrict__ in,
                                                                                 const float* __restrict__ inv_psi,
                                                                                 const float2* __restrict__ tw,
                                                                                 float2* __restrict__ out) {
  using G = RegGeom<R1, R2, R3>;
  constexpr int L = G::L, S1 = G::S1, S2 = G::S2, S3 = G::S3, P1 = G::P1, P2 = G::P2, NL = G::NL;
  extern __shared__ float2 s_line[];  // NL lines, then the second pass's twiddles
  float2* const s_tw = s_line + NL * G::POINTS;
  const int n_in = p.n_in, half = n_in / 2, gap = L - n_in, lo = p.win_lo;
  const unsigned wl = p.win_len;
  const int line_t = NL == 1 ? 0 : (int)threadIdx.x / G::T;
  const int j = threadIdx.x - line_t * G::T;
  float2* const s = s_line + line_t * G::POINTS;
  const unsigned in_off = line_t * (unsigned)p.in_stride, out_off = line_t * (unsigned)p.out_stride;
  if constexpr (R2 > 1) {
    for (int i = threadIdx.x; i < S3; i += G::TPB) s_tw[i] = tw[i];
    tw += S3;
  }
  const int64_t line0 = (int64_t)blockIdx.x * NL;
  const bool live = j < G::T && line_t < min((int64_t)NL, p.n_lines - line0);
  const float2* const src = in + line0 * p.in_stride;
  float2* const dst = out + line0 * p.out_stride;
  float* const dst_re = reinterpret_cast<float*>(out) + line0 * p.out_stride;
  {
    const bool act = live && j < S1;
    float2 v[R1];
    if (act) {
      float sc[R1];
#pragma unroll
      for (int r = 0; r < R1; ++r) {  // all requested before the first is used; input 0 where none is stored
        const int m = j + r * S1;
        const bool stored = m < half || m >= L - half;
        const unsigned i = !stored ? 0 : m < half ? m : m - gap;
        v[r] = src[in_off + i];
        sc[r] = inv_psi[i];
        if (!stored) sc[r] = 0.0f;
      }
#pragma unroll
      for (int r = 0; r < R1; ++r) v[r] = make_float2(v[r].x * sc[r], v[r].y * sc[r]);
      small_dft<R1>(v);
    }
    if (act)
#pragma unroll
      for (int q = 0; q < R1; ++q) s[j * P1 + q] = v[q];
  }
  if constexpr (R2 > 1) {
    __syncthreads();
    const bool act = live && j < S2;
    const int g = j / R1, k = j - g * R1;
    float2 v[R2];
    if (act) {
#pragma unroll
      for (int r = 0; r < R2; ++r) v[r] = s[g * P1 + k + r * (R3 * P1)];  // S2 = R1 R3 points: R3 rows
#pragma unroll
      for (int r = 1; r < R2; ++r) v[r] = cmul(v[r], s_tw[r * R1 + k]);
      small_dft<R2>(v);
    }
    __syncthreads();
    if (act)
#pragma unroll
      for (int q = 0; q < R2; ++q) s[g * P2 + k + q * R1] = v[q];
  }
  const bool act = live && j < S3;
  float2 t[R3], v[R3];
  if (act)
#pragma unroll
    for (int r = 1; r < R3; ++r) t[r] = tw[(unsigned)(r * S3 + j)];
  __syncthreads();
  if (act) {
#pragma unroll
    for (int r = 0; r < R3; ++r) v[r] = s[j + r * P2];
#pragma unroll
    for (int r = 1; r < R3; ++r) v[r] = cmul(v[r], t[r]);
    small_dft<R3>(v);
#pragma unroll
    for (int q = 0; q < R3; ++q) {
      const int m = j + q * S3 - lo;
      const unsigned w = min((unsigned)m, (unsigned)(m + L));  // m mod L
      if (w < wl) {
        if (p.real)
          dst_re[out_off + w] = v[q].x;
        else
          dst[out_off + w] = v[q];
      }
    }
  }
}

// The lengths' radices: two if possible, then the fewest threads per line (the
// largest count of butterflies of a pass) for the fewest idle ones, then an odd
// first radix (no padding).  Radices up to 20 keep a pass within 96 registers.
constexpr int kRegRadices[] = {4, 5, 6, 8, 9, 10, 12, 15, 16, 18, 20};
constexpr int kRegMax = 8000;  // = 20^3
struct RegPlan {
  int L, r1, r2, r3, t;
};
constexpr RegPlan reg_plan(int L) {
  RegPlan best{L, 0, 0, 0, 0};
  int rest = L;
  for (int f : {2, 3, 5})
    while (rest % f == 0) rest /= f;
  if (rest != 1) return best;
  for (int r1 : kRegRadices)
    for (int r3 : kRegRadices) {
      if (L % (r1 * r3)) continue;
      const int r2 = L / (r1 * r3);
      bool known = r2 == 1;
      for (int r : kRegRadices) known |= r2 == r;
      const int t = std::max(std::max(L / r1, L / r3), r2 > 1 ? L / r2 : 0);
      if (!known || t > 512) continue;
      const bool first = best.t == 0, fewer = best.r2 > 1 && r2 == 1, more = best.r2 == 1 && r2 > 1;
      if (first || fewer || (!more && (t < best.t || (t == best.t && r1 % 2 > best.r1 % 2))))
        best = {L, r1, r2, r3, t};
    }
  return best;
}
constexpr int reg_plan_count() {
  int n = 0;
  for (int L = 16; L <= kRegMax; L += 4) n += reg_plan(L).t > 0;  // an axis has 2 N points, N even
  return n;
}
constexpr int kRegPlanCount = reg_plan_count();
struct RegPlans {
  RegPlan p[kRegPlanCount];
};
constexpr RegPlans reg_plans() {
  RegPlans t{};
  int n = 0;
  for (int L = 16; L <= kRegMax; L += 4)
    if (const RegPlan q = reg_plan(L); q.t > 0) t.p[n++] = q;
  return t;
}
constexpr RegPlans kRegPlans = reg_plans();

int reg_find(int L) {
  for (int i = 0; i < kRegPlanCount; ++i)
    if (kRegPlans.p[i].L == L) return i;
  return -1;
}

template <size_t I>
hipError_t launch_reg(const LineFft& p, const float2* in, const float* inv_psi, const float2* tw, float2* out,
                      hipStream_t s) {
  constexpr RegPlan q = kRegPlans.p[I];
  using G = RegGeom<q.r1, q.r2, q.r3>;
  auto* const fn = &line_reg_kernel<q.r1, q.r2, q.r3>;
  if (G::LDS > 65536) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(fn),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)G::LDS);
    if (e != hipSuccess) return e;
  }
  const int64_t groups = (p.n_lines + G::NL - 1) / G::NL;
  hipLaunchKernelGGL(fn, dim3((unsigned)groups), dim3(G::TPB), G::LDS, s, p, in, inv_psi, tw, out);
  return hipGetLastError();
}
template <size_t... I>
hipError_t launch_reg_plan(int i, const LineFft& p, const float2* in, const float* inv_psi, const float2* tw, float2* out,
                      hipStream_t s, std::index_sequence<I...>) {
  static constexpr decltype(&launch_reg<0>) fn[] = {&launch_reg<I>...};
  return fn[i](p, in, inv_psi, tw, out, s);
}

// out[c][r] = in[r][c] for an rows x cols matrix of complex64, 32 x 32 tiles.
__global__ __launch_bounds__(256) void transpose_c64_kernel(const float2* __restrict__ in, int64_t rows, int64_t cols,
                                                            float2* __restrict__ out) {
  __shared__ float2 tile[32][33];
  in += (int64_t)blockIdx.z * rows * cols;
  out += (int64_t)blockIdx.z * rows * cols;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;  // 32 x 8
  const int64_t c0 = (int64_t)blockIdx.x * 32, r0 = (int64_t)blockIdx.y * 32;
#pragma unroll
  for (int k = 0; k < 32; k += 8) {
    const int64_t r = r0 + ty + k, c = c0 + tx;
    if (r < rows && c < cols) tile[ty + k][tx] = in[r * cols + c];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 32; k += 8) {
    const int64_t c = c0 + ty + k, r = r0 + tx;
    if (r < rows && c < cols) out[c * rows + r] = tile[tx][ty + k];
  }
}

// Lines of at most kLineDftMax points as a direct pruned DFT on MFMA: the
// kept outputs of a block of 16 lines are one small dense product,
//   D[n][line] = sum_k A[n][k] B[k][line],
// B the lines' stored inputs as floats (k <-> float f of the line: re / im of
// input f / 2), A the real form of the table T (complex64, n_in x win_len,
// exp(+2 pi i f_i m_w / L) / psi_i): row n = 2 w + c gives the real (c = 0) or
// imaginary (c = 1) part of output w, A[2w][2i] = Re T, A[2w][2i+1] = -Im T,
// A[2w+1][2i] = Im T, A[2w+1][2i+1] = Re T.  One wave per 16-line block on
// v_mfma_f32_16x16x4f32 (A lane l = row l % 16 of k = 4 s + l / 16; B lane l
// = line l % 16; D register r of lane l = row 4 (l / 16) + r); K index
// k = 4 s + q is float q STEPS + s of the line, so lane (line, q) reads STEPS
// consecutive floats of its line and the table fragments stay in registers
// for the whole kernel.  D registers r, r + 1 are the real and imaginary part
// of one output: each lane stores whole complex values, 16 consecutive lines
// at a time.  STEPS = 2 n_in / 4; at most 8 blocks of 16 output rows.
template <int STEPS, int NBMAX>
__global__ __launch_bounds__(256) void line_dft_kernel(LineFft p, const float2* __restrict__ in,
                                                       const float2* __restrict__ tab, float2* __restrict__ out) {
  typedef float f32x4_t __attribute__((ext_vector_type(4)));
  // blocks of 16 lines per wave and step: all their inputs are requested
  // before the first product, so that a wave keeps G x 2 KB of reads in flight
  constexpr int G = 4;
  const int lane = threadIdx.x & 63, q = lane >> 4, r16 = lane & 15;
  const int wl = p.win_len, n_in = p.n_in;
  const int nb = (2 * wl + 15) / 16;  // blocks of 16 output rows (wave-uniform, <= NBMAX)
  float a[NBMAX][STEPS];
#pragma unroll
  for (int b = 0; b < NBMAX; ++b)
#pragma unroll
    for (int s = 0; s < STEPS; ++s) {
      const int n = 16 * b + r16, w = n >> 1, cn = n & 1;
      const int f = q * STEPS + s, i = f >> 1, cf = f & 1;
      float v = 0.0f;
      if (b < nb && w < wl && i < n_in) {
        const float2 t = tab[i * wl + w];
        v = cn == 0 ? (cf == 0 ? t.x : -t.y) : (cf == 0 ? t.y : t.x);
      }
      a[b][s] = v;
    }
  const int64_t n_blocks = (p.n_lines + 15) / 16;
  const int64_t wave0 = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const int64_t n_waves = ((int64_t)gridDim.x * blockDim.x) >> 6;
  for (int64_t blk0 = wave0 * G; blk0 < n_blocks; blk0 += n_waves * G) {
    float x[G][STEPS];
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const int64_t line = (blk0 + g) * 16 + r16;
      const bool live = line < p.n_lines;
      const float* const src = reinterpret_cast<const float*>(in + (live ? line : 0) * p.in_stride) + q * STEPS;
      if constexpr (STEPS % 4 == 0) {  // 16-byte aligned runs: vector loads
#pragma unroll
        for (int s = 0; s < STEPS; s += 4) {
          const float4 v = live ? *reinterpret_cast<const float4*>(src + s) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
          x[g][s] = v.x;
          x[g][s + 1] = v.y;
          x[g][s + 2] = v.z;
          x[g][s + 3] = v.w;
        }
      } else {
#pragma unroll
        for (int s = 0; s < STEPS; ++s) x[g][s] = live ? src[s] : 0.0f;
      }
    }
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const int64_t line = (blk0 + g) * 16 + r16;
      f32x4_t d[NBMAX];
#pragma unroll
      for (int b = 0; b < NBMAX; ++b) {
        d[b] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
        if (b < nb)
#pragma unroll
          for (int s = 0; s < STEPS; ++s)
            d[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[b][s], x[g][s], d[b], 0, 0, 0);
      }
      if (line >= p.n_lines) continue;
      float2* dst;
      int64_t wstride;
      if (p.out_mode == 0) {
        dst = out + line * p.out_stride;
        wstride = 1;
      } else {  // line = outer * t_inner + inner, stored at [outer][w][inner]
        const int64_t outer = line / p.t_inner, inner = line - outer * p.t_inner;
        dst = out + outer * wl * p.t_inner + inner;
        wstride = p.t_inner;
      }
#pragma unroll
      for (int b = 0; b < NBMAX; ++b)
#pragma unroll
        for (int h = 0; h < 2; ++h) {  // registers 2 h, 2 h + 1: output w = 8 b + 2 q + h
          const int w = 8 * b + 2 * q + h;
          if (b < nb && w < wl) dst[w * wstride] = make_float2(d[b][2 * h], d[b][2 * h + 1]);
        }
    }
  }
}

}  // namespace

void line_dft_table(const LineFft& p, const float* inv_psi, float* tab) {
  const int half = p.n_in / 2;
  for (int i = 0; i < p.n_in; ++i) {
    const int f = i < half ? i : i - p.n_in;
    for (int w = 0; w < p.win_len; ++w) {
      const int m = (p.win_lo + w) % p.L;
      // the angle's numerator reduced mod L first: exact in integers
      const int64_t fm = (((int64_t)f * m) % p.L + p.L) % p.L;
      const double a = 2.0 * M_PI * (double)fm / p.L;
      tab[2 * ((size_t)i * p.win_len + w)] = (float)(std::cos(a) * inv_psi[i]);
      tab[2 * ((size_t)i * p.win_len + w) + 1] = (float)(std::sin(a) * inv_psi[i]);
    }
  }
}

bool line_dft_fits(const LineFft& p) {
  // 2 n_in floats per line in 4 lane groups (2 <= STEPS <= 16), at most 8 blocks of 16 output rows
  return p.L <= kLineDftMax && p.n_in % 2 == 0 && p.n_in >= 4 && p.n_in <= 32 && p.win_len >= 1 &&
         2 * p.win_len <= 128;
}

hipError_t launch_line_dft(const LineFft& p, const void* in, const float2* tab, void* out, hipStream_t s) {
  if (p.n_lines <= 0) return hipSuccess;
  if (!line_dft_fits(p)) return hipErrorInvalidValue;
  // the vector loads of runs of 4 floats need 16-byte aligned lines
  if ((p.n_in / 2) % 4 == 0 && ((p.in_stride * 8) % 16 != 0 || reinterpret_cast<uintptr_t>(in) % 16 != 0))
    return hipErrorInvalidValue;
  const int64_t waves = (p.n_lines + 63) / 64;  // four 16-line blocks per wave and step
  const unsigned grid = (unsigned)std::min<int64_t>((waves + 3) / 4, 1 << 16);
  const float2* const x = static_cast<const float2*>(in);
  float2* const y = static_cast<float2*>(out);
  const bool narrow = 2 * p.win_len <= 64;  // at most 4 blocks of 16 output rows
#define BB_DFT_CASE(S)                                                                                  \
  case S:                                                                                               \
    if (narrow)                                                                                         \
      hipLaunchKernelGGL((line_dft_kernel<S, 4>), dim3(grid), dim3(256), 0, s, p, x, tab, y);           \
    else                                                                                                \
      hipLaunchKernelGGL((line_dft_kernel<S, 8>), dim3(grid), dim3(256), 0, s, p, x, tab, y);           \
    break;
  switch (p.n_in / 2) {
    BB_DFT_CASE(2) BB_DFT_CASE(3) BB_DFT_CASE(4) BB_DFT_CASE(5) BB_DFT_CASE(6) BB_DFT_CASE(7) BB_DFT_CASE(8)
    BB_DFT_CASE(9) BB_DFT_CASE(10) BB_DFT_CASE(11) BB_DFT_CASE(12) BB_DFT_CASE(13) BB_DFT_CASE(14)
    BB_DFT_CASE(15) BB_DFT_CASE(16)
    default: return hipErrorInvalidValue;
  }
#undef BB_DFT_CASE
  return hipGetLastError();
}

int line_fft_plan(int L, LineFft& p) {
  if (L < 2 || L > kLineFftMax) return -1;
  int m = L, n2 = 0, n3 = 0, n5 = 0;
  while (m % 2 == 0) m /= 2, ++n2;
  while (m % 3 == 0) m /= 3, ++n3;
  while (m % 5 == 0) m /= 5, ++n5;
  if (m != 1) return -1;
  int rad[32], n = 0;
  while (n2 > 4 || n2 == 3) rad[n++] = 8, n2 -= 3;
  if (n2 == 4) rad[n++] = 4, rad[n++] = 4;
  if (n2 == 2) rad[n++] = 4;
  if (n2 == 1) rad[n++] = 2;
  for (int i = 0; i < n3; ++i) rad[n++] = 3;
  for (int i = 0; i < n5; ++i) rad[n++] = 5;
  if (n > 16) return -1;
  p.L = L;
  p.n_pass = n;
  p.radix_codes = 0;
  for (int i = 0; i < n; ++i) p.radix_codes |= (uint64_t)rad[i] << (4 * i);
  p.nl = std::max(1, 4096 / L);
  p.reg = reg_find(L);
  return 0;
}

// Padding pays for long lines with at least 2^6 in their length (4608: 0.92
// against 1.02 ms per call on the 1024^2 benchmark grid); for the others
// (4500 = 2^2 3^2 5^3) the extra index work outweighs it.
static bool fft_pad(const LineFft& p) { return p.nl == 1 && p.L % 64 == 0; }
size_t line_fft_lds_bytes(const LineFft& p) {
  const size_t n = (size_t)p.nl * p.L;
  return (fft_pad(p) ? n + (n >> 5) + 2 : n) * sizeof(float2);
}

// Whether line_reg_kernel transforms the planned lines.
static bool reg_fits(const LineFft& p) { return p.reg >= 0 && p.out_mode == 0; }

bool line_real_fits(const LineFft& p) { return reg_fits(p) && !p.direct; }

size_t line_fft_twiddle_points(int L) { return 2 * (size_t)L; }

void line_fft_twiddles(const LineFft& p, float* tw) {
  if (reg_fits(p)) {
    const RegPlan& q = kRegPlans.p[p.reg];
    const int r1 = q.r1, r2 = q.r2, r3 = q.r3;
    auto fill = [&](int ns, int R) {  // [r][k], k < ns: exp(2 pi i r k / (ns R))
      for (int r = 0; r < R; ++r)
        for (int k = 0; k < ns; ++k) {
          const double a = 2.0 * M_PI * (double)(r * k) / (ns * R);
          *tw++ = (float)std::cos(a);
          *tw++ = (float)std::sin(a);
        }
    };
    if (r2 > 1) fill(r1, r2);
    fill(r1 * r2, r3);
    return;
  }
  int ns = 1;
  for (int s = 0; s < p.n_pass; ++s) {
    const int R = (int)((p.radix_codes >> (4 * s)) & 15), P = ns * R;
    float* t = tw + 2 * (size_t)(ns - 1);
    for (int k = 0; k < ns; ++k)
      for (int r = 1; r < R; ++r) {
        const double a = 2.0 * M_PI * (double)(k * r) / P;
        t[2 * (k * (R - 1) + r - 1)] = (float)std::cos(a);
        t[2 * (k * (R - 1) + r - 1) + 1] = (float)std::sin(a);
      }
    ns = P;
  }
}

void line_fft_perm(const LineFft& p, int* perm) {
  int rad[16], span[16];
  int ns = 1;
  for (int s = 0; s < p.n_pass; ++s) {
    rad[s] = (int)((p.radix_codes >> (4 * s)) & 15);
    span[s] = ns;
    ns *= rad[s];
  }
  for (int n = 0; n < p.L; ++n) {
    int rem = n, pos = 0;
    for (int s = p.n_pass - 1; s >= 0; --s) {
      pos += (rem % rad[s]) * span[s];
      rem /= rad[s];
    }
    perm[n] = pos;
  }
}

hipError_t launch_line_fft(const LineFft& p, const void* in, const float* inv_psi, const int* perm, const float2* tw,
                           void* out, hipStream_t s) {
  if (p.n_lines <= 0) return hipSuccess;
  if (reg_fits(p))
    return launch_reg_plan(p.reg, p, static_cast<const float2*>(in), inv_psi, tw, static_cast<float2*>(out), s,
                      std::make_index_sequence<kRegPlanCount>{});
  const int64_t groups = (p.n_lines + p.nl - 1) / p.nl;
  const unsigned grid = (unsigned)std::min<int64_t>(groups, 1 << 16);
  const size_t lds = line_fft_lds_bytes(p);
  const bool pad = fft_pad(p);
  const void* const fn = p.nl > 1 ? reinterpret_cast<const void*>(&line_fft_kernel<512, true, false>)
                                  : (pad ? reinterpret_cast<const void*>(&line_fft_kernel<512, false, true>)
                                         : reinterpret_cast<const void*>(&line_fft_kernel<512, false, false>));
  if (lds > 65536) {
    const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  if (p.nl > 1)
    hipLaunchKernelGGL((line_fft_kernel<512, true, false>), dim3(grid), dim3(512), lds, s, p, static_cast<const float2*>(in),
                       inv_psi, perm, tw, static_cast<float2*>(out));
  else if (pad)
    hipLaunchKernelGGL((line_fft_kernel<512, false, true>), dim3(grid), dim3(512), lds, s, p,
                       static_cast<const float2*>(in), inv_psi, perm, tw, static_cast<float2*>(out));
  else
    hipLaunchKernelGGL((line_fft_kernel<512, false, false>), dim3(grid), dim3(512), lds, s, p,
                       static_cast<const float2*>(in), inv_psi, perm, tw, static_cast<float2*>(out));
  return hipGetLastError();
}

hipError_t launch_transpose_c64(const void* in, int64_t rows, int64_t cols, int n, void* out, hipStream_t s) {
  if (rows <= 0 || cols <= 0) return hipSuccess;
  const dim3 grid((unsigned)((cols + 31) / 32), (unsigned)((rows + 31) / 32), (unsigned)n);
  hipLaunchKernelGGL(transpose_c64_kernel, grid, dim3(256), 0, s, static_cast<const float2*>(in), rows, cols,
                     static_cast<float2*>(out));
  return hipGetLastError();
}

}  // namespace bb
