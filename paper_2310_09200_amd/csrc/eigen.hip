// The generalized eigenproblem V a = lambda G a of one instance in FP64
// (Section 2.3, Eq. eigenvaleq), G real symmetric positive definite (or I),
// n <= kEigMaxN antennas:
//   G = L L^T and its inverse factor Y = L^{-1}   (64-column panels)
//   C = Y V Y^T                                   (two products)
//   C = Q T Q^H, T real tridiagonal               (Householder)
//   T = Z diag(lambda) Z^T                        (rocSOLVER dstedc, host API)
//   a = Y^T (Q Z)                                 (reflectors, product)
//
// The library's one-call solver (zhegvd) spent 35 ms on n = 512 and 3.8 ms on
// n = 64, nearly all of it in chains of small dependent launches (a
// triangular solve, two axpys and a rank-2 update per column to reduce to
// standard form, and four to six launches per Householder column).  Here the
// reduction to standard form is products with the inverse factor, and the
// tridiagonalisation is one launch that keeps C in registers: 6.2 and 1.0 ms a
// call, of which n = 512 spends 2.7 ms in the tridiagonalisation (5.3 us a
// column), 2.4 in dstedc, 0.7 in the Cholesky panels and 0.4 in the reflectors.

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "bb_internal.h"

namespace bb {

namespace {

struct cd {
  double x, y;
};
__device__ __forceinline__ cd operator+(cd a, cd b) { return {a.x + b.x, a.y + b.y}; }
// a b, a conj(b), and accumulating forms
__device__ __forceinline__ cd mul(cd a, cd b) { return {a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x}; }
__device__ __forceinline__ void fma_c(cd& r, cd a, cd b) {
  r.x = fma(a.x, b.x, fma(-a.y, b.y, r.x));
  r.y = fma(a.x, b.y, fma(a.y, b.x, r.y));
}
__device__ __forceinline__ void fms_conj(cd& r, cd a, cd b) {  // r -= a conj(b)
  r.x = fma(-a.x, b.x, fma(-a.y, b.y, r.x));
  r.y = fma(a.x, b.y, fma(-a.y, b.x, r.y));
}

// 1 / sqrt(d) and 1 / d from the hardware estimates (relative error near 2^-23
// in FP64) by two Newton steps: 1 to 2 units in the last place, in a third of
// the dependent instructions of sqrt and divide.
__device__ __forceinline__ double rsqrt_newton(double d) {
  double y = __builtin_amdgcn_rsq(d);
  for (int i = 0; i < 2; ++i) y = fma(0.5 * y, fma(-d * y, y, 1.0), y);
  return y;
}
__device__ __forceinline__ double rcp_newton(double d) {
  double y = __builtin_amdgcn_rcp(d);
  for (int i = 0; i < 2; ++i) y = fma(y, fma(-d, y, 1.0), y);
  return y;
}
__device__ __forceinline__ double lane_of(double x, int lane) {  // wave-uniform lane
  const uint64_t u = __builtin_bit_cast(uint64_t, x);
  const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)u, lane);
  const uint32_t hi = __builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), lane);
  return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}

// ---- inputs -----------------------------------------------------------------
// A = V from its lower triangle (diagonal real), the real Gram matrix (unless
// G = I; `same` is set where two antennas are in one place), and per-workgroup sums of the Hermiticity check: part[2 b] of
// ||V - V^H||_F^2 and part[2 b + 1] of ||V||_F^2 (kHermParts workgroups; the
// host adds them in order).
__global__ __launch_bounds__(256) void eig_inputs_kernel(const double* __restrict__ ant, int n, double inv_wl,
                                                         int identity, const double* __restrict__ V,
                                                         double* __restrict__ A, double* __restrict__ G,
                                                         double* __restrict__ part, int* __restrict__ same) {
  __shared__ double s[2][4];
  double dsum = 0.0, nsum = 0.0;
  bool coincide = false;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < (int64_t)n * n; i += (int64_t)gridDim.x * 256) {
    const int p = (int)(i % n), q = (int)(i / n);
    const cd a = ((const cd*)V)[i];                          // V_pq
    const cd b = ((const cd*)V)[(int64_t)p * n + q];         // V_qp
    const double dr = a.x - b.x, di = a.y + b.y;             // V_pq - conj(V_qp)
    dsum += dr * dr + di * di;
    nsum += a.x * a.x + a.y * a.y;
    ((cd*)A)[i] = p > q ? a : (p < q ? cd{b.x, -b.y} : cd{a.x, 0.0});
    if (!identity) {
      const double dx = ant[p] - ant[q];
      const double dy = ant[p + n] - ant[q + n];
      const double dz = ant[p + 2 * n] - ant[q + 2 * n];
      const double u = 2.0 * sqrt(dx * dx + dy * dy + dz * dz) * inv_wl;
      G[i] = (u == 0.0) ? 1.0 : sinpi(u) / (M_PI * u);
      coincide = coincide || (u == 0.0 && p != q);
    }
  }
  if (coincide) atomicOr(same, 1);
  for (int o = 32; o > 0; o >>= 1) {
    dsum += __shfl_xor(dsum, o);
    nsum += __shfl_xor(nsum, o);
  }
  if ((threadIdx.x & 63) == 0) {
    s[0][threadIdx.x >> 6] = dsum;
    s[1][threadIdx.x >> 6] = nsum;
  }
  __syncthreads();
  if (threadIdx.x < 2) {
    double t = 0.0;
    for (int w = 0; w < 4; ++w) t += s[threadIdx.x][w];
    part[2 * blockIdx.x + threadIdx.x] = t;
  }
}

// ---- G = L L^T, Y = L^{-1} ----------------------------------------------------
// Panel k of 64 columns, three launches: the diagonal block with its inverse,
// the block column L_ik = G_ik D^T and block row Y_kj = D Y_kj (D the inverse of
// the diagonal factor), and the trailing updates G_ij -= L_ik L_jk^T (k < j <= i),
// Y_ij -= L_ik Y_kj (j <= k < i).  Rows and columns past n are those of I.
constexpr int kNB = 64;

// Elimination of [block | I], the factor's column c giving its place to the
// inverse's once it is used: thread (r, g) keeps row r of columns g + 8 m in
// registers.  A column's step publishes its multipliers and the pivot row, one
// barrier, and eight multiply-adds a thread; bound by its 64 dependent steps
// (0.2 us each).  info becomes c + 1 at a pivot c that is NaN and -(c + 1) at one
// of at most kPivotNoise: with the diagonal of G at 1 its sign is then rounding,
// which this elimination and the library's need not share, and the library
// decides (kPivotNoise is 8 n eps at n = 512).
constexpr double kPivotNoise = 0x1p-40;
__global__ __launch_bounds__(512) void chol_diag_kernel(const double* __restrict__ G, double* __restrict__ Y, int n,
                                                        int k, int* __restrict__ info) {
  __shared__ double s_l[2][kNB];        // multipliers L[r][c]
  __shared__ double s_f[2][8][10];      // [g][m]: L[g + 8 m][c] right of the pivot, the pivot row left of it
  __shared__ double s_inv[2];
  const int t = threadIdx.x, r = t & 63, g = t >> 6;
  const int r0 = k * kNB;
  double v[8];
#pragma unroll
  for (int m = 0; m < 8; ++m) {
    const int c = g + 8 * m;
    v[m] = r0 + r < n && r0 + c < n ? G[(int64_t)(r0 + c) * n + r0 + r] : (r == c ? 1.0 : 0.0);
  }
#pragma unroll
  for (int mc = 0; mc < 8; ++mc)
    for (int gc = 0; gc < 8; ++gc) {
      const int c = gc + 8 * mc, buf = c & 1;
      if (g == gc) {  // the wave that holds column c
        const double d = lane_of(v[mc], c);
        if (r == c && !(d > kPivotNoise) && r0 + c < n && *info == 0) *info = d != d ? r0 + c + 1 : -(r0 + c + 1);
        const double inv = rsqrt_newton(d), l = v[mc] * inv;
        s_l[buf][r] = l;
        if (r > c) s_f[buf][r & 7][r >> 3] = l;
        if (r == c) s_inv[buf] = inv;
      }
      if (r == c)
#pragma unroll
        for (int m = 0; m < 8; ++m)
          if (g + 8 * m < c) s_f[buf][g][m] = v[m];
      __syncthreads();
      const double inv = s_inv[buf], l = s_l[buf][r];
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        const int cc = g + 8 * m;
        const double f = cc > c ? s_f[buf][g][m] : (cc < c ? s_f[buf][g][m] * inv : inv);
        if (r > c)
          v[m] = cc == c ? -l * inv : fma(-l, f, v[m]);
        else if (r == c && cc <= c)
          v[m] = f;
      }
    }
#pragma unroll
  for (int m = 0; m < 8; ++m) {
    const int c = g + 8 * m;
    if (r0 + r < n && r0 + c < n) Y[(int64_t)(r0 + c) * n + r0 + r] = r >= c ? v[m] : 0.0;
  }
}

// 64 x 64 product of two LDS tiles: out[4][4] of this thread (256 threads).
struct Tile64 {
  double a[kNB][kNB + 1], b[kNB][kNB + 1];  // a[r][k], b[k][c]
};
__device__ __forceinline__ void tile_product(const Tile64& s, double (&o)[4][4], int tr, int tc) {
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) o[i][j] = 0.0;
#pragma unroll 8
  for (int k = 0; k < kNB; ++k) {
    double x[4], y[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) x[i] = s.a[tr + 16 * i][k];
#pragma unroll
    for (int j = 0; j < 4; ++j) y[j] = s.b[k][tc + 16 * j];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) o[i][j] = fma(x[i], y[j], o[i][j]);
  }
}

// Element (r, c) of block (i, j) of an n x n column-major matrix, 0 outside.
__device__ __forceinline__ double block_at(const double* __restrict__ M, int n, int i, int j, int r, int c) {
  const int R = i * kNB + r, C = j * kNB + c;
  return R < n && C < n ? M[(int64_t)C * n + R] : 0.0;
}

// blockIdx.x < nb - 1 - k: L_ik = G_ik D^T for i = k + 1 + blockIdx.x; then
// Y_kj = D Y_kj for j = blockIdx.x - (nb - 1 - k) < k.  D = Y_kk.
__global__ __launch_bounds__(256) void chol_panel_kernel(double* __restrict__ G, double* __restrict__ Y, int n,
                                                         int k) {
  __shared__ Tile64 s;
  const int nb = (n + kNB - 1) / kNB, below = nb - 1 - k;
  const int t = threadIdx.x, tr = t & 15, tc = t >> 4;
  const bool is_l = (int)blockIdx.x < below;
  const int o = is_l ? k + 1 + blockIdx.x : blockIdx.x - below;
  for (int i = t; i < kNB * kNB; i += 256) {
    const int r = i % kNB, c = i / kNB;
    const double d = block_at(Y, n, k, k, r, c);
    if (is_l) {
      s.a[r][c] = block_at(G, n, o, k, r, c);
      s.b[c][r] = d;
    } else {
      s.a[r][c] = d;
      s.b[r][c] = block_at(Y, n, k, o, r, c);
    }
  }
  __syncthreads();
  double out[4][4];
  tile_product(s, out, tr, tc);
  double* const M = is_l ? G : Y;
  const int bi = is_l ? o : k, bj = is_l ? k : o;
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int R = bi * kNB + tr + 16 * i, C = bj * kNB + tc + 16 * j;
      if (R < n && C < n) M[(int64_t)C * n + R] = out[i][j];
    }
}

// Trailing updates for block row i = k + 1 + blockIdx.x, block column j = blockIdx.y <= i.
__global__ __launch_bounds__(256) void chol_update_kernel(double* __restrict__ G, double* __restrict__ Y, int n,
                                                          int k) {
  __shared__ Tile64 s;
  const int bi = k + 1 + blockIdx.x, bj = blockIdx.y;
  if (bj > bi) return;
  const int t = threadIdx.x, tr = t & 15, tc = t >> 4;
  const bool is_g = bj > k;
  for (int i = t; i < kNB * kNB; i += 256) {
    const int r = i % kNB, c = i / kNB;
    s.a[r][c] = block_at(G, n, bi, k, r, c);
    if (is_g)
      s.b[c][r] = block_at(G, n, bj, k, r, c);
    else
      s.b[r][c] = block_at(Y, n, k, bj, r, c);
  }
  __syncthreads();
  double out[4][4];
  tile_product(s, out, tr, tc);
  double* const M = is_g ? G : Y;
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int R = bi * kNB + tr + 16 * i, C = bj * kNB + tc + 16 * j;
      if (R >= n || C >= n) continue;
      double* const m = M + (int64_t)C * n + R;
      *m = (bj == k ? 0.0 : *m) - out[i][j];  // Y_ik starts here
    }
}

// ---- products with the inverse factor -------------------------------------------
// out(i, j) = sum_k R(i, k) Z(k, j), R real triangular, Z complex, with
// R(i, k) = Y[i + k n] (lower, k <= i) or, TRANS, Y[k + i n] (k >= i);
// Z(k, j) = Z[k zk + j zj], out(i, j) = out[i oi + j oj] (complex elements).
// 32 x 32 outputs a workgroup, 32-deep chunks through LDS.
template <bool TRANS>
__global__ __launch_bounds__(256) void tri_product_kernel(const double* __restrict__ Y, const cd* __restrict__ Z,
                                                          int64_t zk, int64_t zj, cd* __restrict__ out, int64_t oi,
                                                          int64_t oj, int n) {
  __shared__ double s_r[32][33];
  __shared__ cd s_z[32][33];
  const int i0 = blockIdx.x * 32, j0 = blockIdx.y * 32;
  const int t = threadIdx.x, a = t & 31, b = t >> 5;  // loads: a along the contiguous axis
  const int ti = t & 15, tj = t >> 4;                 // outputs (ti + 16 p, tj + 16 q)
  cd o[2][2] = {};
  const int k_lo = TRANS ? i0 : 0, k_hi = TRANS ? n : (i0 + 32 < n ? i0 + 32 : n);
  double r_nx[4];
  cd z_nx[4];
  auto load = [&](int k0) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int u = a, v = b + 8 * q;
      const int i = i0 + (TRANS ? v : u), k = k0 + (TRANS ? u : v);
      const bool in = i < n && k < n && (TRANS ? k >= i : k <= i);
      r_nx[q] = in ? Y[TRANS ? (int64_t)i * n + k : (int64_t)k * n + i] : 0.0;
      const int kz = k0 + (zk == 1 ? u : v), jz = j0 + (zk == 1 ? v : u);
      z_nx[q] = kz < n && jz < n ? Z[kz * zk + jz * zj] : cd{0.0, 0.0};
    }
  };
  load(k_lo);
  for (int k0 = k_lo; k0 < k_hi; k0 += 32) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int u = a, v = b + 8 * q;
      s_r[TRANS ? u : v][TRANS ? v : u] = r_nx[q];  // [k][i]
      s_z[zk == 1 ? u : v][zk == 1 ? v : u] = z_nx[q];
    }
    __syncthreads();
    if (k0 + 32 < k_hi) load(k0 + 32);
#pragma unroll 8
    for (int k = 0; k < 32; ++k) {
      double r[2];
      cd z[2];
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        r[p] = s_r[k][ti + 16 * p];
        z[p] = s_z[k][tj + 16 * p];
      }
#pragma unroll
      for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          o[p][q].x = fma(r[p], z[q].x, o[p][q].x);
          o[p][q].y = fma(r[p], z[q].y, o[p][q].y);
        }
    }
    __syncthreads();
  }
#pragma unroll
  for (int p = 0; p < 2; ++p)
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int i = i0 + ti + 16 * p, j = j0 + tj + 16 * q;
      if (i < n && j < n) out[i * oi + j * oj] = o[p][q];
    }
}

// ---- tridiagonalisation -----------------------------------------------------------
// C = Q T Q^H, Q = H_0 H_1 ... H_{n-2}, H_j = I - tau_j v_j v_j^H (the lower
// variant of the one-column Householder reduction).  NW workgroups own the rows
// i = r NW + w and keep them in registers: thread (tr, tc) of TR x TC the rows
// tr + TR a and columns tc + TC b.  Every workgroup holds the vectors and repeats
// their short arithmetic, so a column needs one exchange: each row's owner
// publishes p_i = tau (C v)_i and y_i = C_{i,j+1}, from which all form
//   w = p - (tau / 2) (p^H v) v,  C -= v w^H + w v^H,  column j + 1 of C.
// The exchange goes through 64-bit words in memory, valid once they differ from a
// signalling NaN that arithmetic cannot produce, in three buffers by turns: a
// buffer is cleared by its rows' owners after the next column's exchange, when all
// have read it, and used again one column later.  Waits end after wait_ticks;
// then info says so, every workgroup returns, and D and E are zeros: the solver
// that is already queued behind must not iterate on half a matrix.  The same
// where the Cholesky factorisation failed (chol).
// Bound by its dependent steps: 2.1 us a column in one workgroup (n = 64), 5.3 us
// with 32 of them (n = 512).
constexpr uint64_t kEmpty = 0xFFF4DEADBEEF5A5AULL;

template <int NW, int TR, int RA, int CB>
struct TrdCfg {
  static constexpr int THREADS = 512;
  static constexpr int TC = THREADS / TR;
  static constexpr int R = TR * RA;    // rows per workgroup
  static constexpr int NMAX = TC * CB;
  static_assert(NMAX <= THREADS && R * NW >= NMAX, "one vector element per thread; rows cover the matrix");
  static constexpr int PARTS = TC / 16;  // groups of 16 lanes that share a row
  static_assert(RA == 2 || RA == 4 || RA == 8, "2 RA values halve over 16 lanes");
};

template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp(double x) {  // 0 where the pattern has no source
  const uint64_t u = __builtin_bit_cast(uint64_t, x);
  const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, ROWS, 0xf, true);
  const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, ROWS, 0xf, true);
  return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}

// Sum over the wave, in lane 63 (row shifts, then the rows' last lanes to the rows above).
__device__ __forceinline__ double wave_sum63(double x) {
  x += dpp<0x111, 0xf>(x);
  x += dpp<0x112, 0xf>(x);
  x += dpp<0x114, 0xf>(x);
  x += dpp<0x118, 0xf>(x);
  x += dpp<0x142, 0xa>(x);
  x += dpp<0x143, 0xc>(x);
  return x;
}

// Sum over the block; every thread gets it.  buf: 8 doubles, not reused before the next barrier.
__device__ __forceinline__ double block_sum(double a, double* buf) {
  a = wave_sum63(a);
  if ((threadIdx.x & 63) == 63) buf[threadIdx.x >> 6] = a;
  __syncthreads();
  a = 0.0;
#pragma unroll
  for (int w = 0; w < 8; ++w) a += buf[w];
  return a;
}

// One halving step of a sum over 16 lanes: of the 2 h values in s, lanes with
// `up` keep the upper half, the others the lower, each adding its partner's.
template <int CTRL, int N>
__device__ __forceinline__ void halve(double (&s)[N], int h, bool up) {
#pragma unroll
  for (int q = 0; q < N / 2; ++q)
    if (q < h) {
      const double send = up ? s[q] : s[q + h], keep = up ? s[q + h] : s[q];
      s[q] = keep + dpp<CTRL, 0xf>(send);
    }
}

template <class K, int NW, int TR, int RA, int CB>
__global__ __launch_bounds__(512) void hetrd_kernel(cd* __restrict__ A, int n, double* __restrict__ D,
                                                    double* __restrict__ E, cd* __restrict__ tau_out,
                                                    uint64_t* __restrict__ pub, uint64_t wait_ticks,
                                                    const int* __restrict__ chol, int* __restrict__ info) {
  constexpr int TC = K::TC, R = K::R;
  if (NW > 1 && blockIdx.x % 8 != 0) return;  // every eighth workgroup: neighbours in one L2, as it happens
  const int wg = NW > 1 ? blockIdx.x / 8 : 0;
  const int t = threadIdx.x, tc = t % TC, tr = t / TC, lane = t & 63;
  __shared__ cd s_x[512], s_v[512], s_w[512], s_p[512], s_y[512], s_own[NW == 1 ? 1 : R];
  __shared__ double s_sum[3][8];
  __shared__ double s_part[K::PARTS][R][2];
  auto no_matrix = [&]() {  // by one thread of the first workgroup
    for (int j = 0; j < n; ++j) {
      D[j] = 0.0;
      if (j < n - 1) E[j] = 0.0;
    }
  };
  if (*chol != 0) {  // the same for every workgroup
    if (wg == 0 && t == 0) no_matrix();
    return;
  }
  cd C[RA][CB];
#pragma unroll
  for (int a = 0; a < RA; ++a)
#pragma unroll
    for (int b = 0; b < CB; ++b) {
      const int i = (tr + TR * a) * NW + wg, c = tc + TC * b;
      cd v = {0.0, 0.0};
      if (i < n && c < n) {  // from the lower triangle
        v = i >= c ? A[(int64_t)c * n + i] : A[(int64_t)i * n + c];
        if (i < c) v.y = -v.y;
        if (i == c) v.y = 0.0;
      }
      C[a][b] = v;
    }
  s_x[t] = t < n ? A[t] : cd{0.0, 0.0};  // column 0
  bool finite = true;
  bool late = false;
  __syncthreads();
  // The matrix is in registers; its memory takes the reflectors (column j below
  // the diagonal), column 0 after the first exchange, when every workgroup has read it.
  for (int j = 0; j < n - 1; ++j) {
    // reflector of column j
    const cd x = s_x[t];
    const double xn = block_sum(t > j + 1 ? fma(x.x, x.x, x.y * x.y) : 0.0, s_sum[0]);
    const cd alpha = s_x[j + 1];
    cd tau = {0.0, 0.0}, scale = {0.0, 0.0};
    double beta = alpha.x;
    // nothing to reflect below 2^-480, where squares leave the range of normal numbers
    if (!(xn < 0x1p-960 && fabs(alpha.y) < 0x1p-480)) {
      const double s2 = fma(alpha.x, alpha.x, fma(alpha.y, alpha.y, xn)), rs = rsqrt_newton(s2), rt = s2 * rs;
      beta = -copysign(fma(fma(-rt, rt, s2), 0.5 * rs, rt), alpha.x);
      const double dx = alpha.x - beta, ib = -copysign(rs, alpha.x);
      const double inv = rcp_newton(fma(dx, dx, alpha.y * alpha.y));
      tau = {-dx * ib, -alpha.y * ib};
      scale = {dx * inv, -alpha.y * inv};
    }
    const cd v = t == j + 1 ? cd{1.0, 0.0} : (t > j + 1 && t < n ? mul(x, scale) : cd{0.0, 0.0});
    s_v[t] = v;
    const double dj = s_x[j].x;
    if (wg == 0 && t == 0) {
      finite = finite && isfinite(dj) && isfinite(beta);
      D[j] = dj;
      E[j] = beta;
      tau_out[j] = tau;
    }
    __syncthreads();
    // own rows of C v
    double s[2 * RA];
#pragma unroll
    for (int q = 0; q < 2 * RA; ++q) s[q] = 0.0;
#pragma unroll
    for (int b = 0; b < CB; ++b) {
      if (TC * (b + 1) <= j + 1) continue;  // v is zero there
      const cd vc = s_v[tc + TC * b];
#pragma unroll
      for (int a = 0; a < RA; ++a) {
        s[2 * a] = fma(C[a][b].x, vc.x, fma(-C[a][b].y, vc.y, s[2 * a]));
        s[2 * a + 1] = fma(C[a][b].x, vc.y, fma(C[a][b].y, vc.x, s[2 * a + 1]));
      }
    }
    // sum over groups of 16 lanes of a row, halving the values while there are two
    {
      int idx = 0;
      halve<0x128>(s, RA, lane & 8);  // rotated by 8
      idx += lane & 8 ? RA : 0;
      halve<0x141>(s, RA / 2, lane & 4);  // mirrored within 8
      idx += lane & 4 ? RA / 2 : 0;
      if constexpr (RA >= 4) {
        halve<0x4e>(s, RA / 4, lane & 2);  // lanes 2, 3, 0, 1 of four
        idx += lane & 2 ? RA / 4 : 0;
      } else {
        s[0] += dpp<0x4e, 0xf>(s[0]);
      }
      if constexpr (RA >= 8) {
        halve<0xb1>(s, RA / 8, lane & 1);  // lanes 1, 0, 3, 2 of four
        idx += lane & 1 ? RA / 8 : 0;
      } else {
        s[0] += dpp<0xb1, 0xf>(s[0]);
      }
      constexpr int kOwn = RA >= 8 ? 1 : 8 / RA;  // lanes that end with the same value
      if ((lane & (kOwn - 1)) == 0) s_part[tc / 16][tr + TR * (idx >> 1)][idx & 1] = s[0];
    }
    // and the next column's entries
    if (tc == (j + 1) % TC) {
#pragma unroll
      for (int b = 0; b < CB; ++b)
        if (b == (j + 1) / TC)
#pragma unroll
          for (int a = 0; a < RA; ++a) (NW == 1 ? s_y : s_own)[tr + TR * a] = C[a][b];
    }
    __syncthreads();
    auto row_p = [&](int r) {
      cd q = {0.0, 0.0};
#pragma unroll
      for (int w = 0; w < K::PARTS; ++w) q = q + cd{s_part[w][r][0], s_part[w][r][1]};
      return mul(tau, q);
    };
    cd p = {0.0, 0.0}, y = {0.0, 0.0};
    if constexpr (NW == 1) {
      if (t < n) {
        if (t > j) p = row_p(t);
        y = s_y[t];
      }
      s_p[t] = p;
    } else {
      // record of a workgroup: 4 R words, Re p, Im p, Re y, Im y of its rows
      constexpr int kRec = 4 * R;
      constexpr int kAll = NW * kRec;  // words of a buffer
      static_assert(kAll % 512 == 0 && kRec >= 64, "every thread takes the same number of words; a wave of one record");
      uint64_t* const cur = pub + (j % 3) * kAll;
      if (t < R) {
        const int i = t * NW + wg;
        const cd q = i > j && i < n ? row_p(t) : cd{0.0, 0.0};
        const cd yy = s_own[t];
        const double w4[4] = {q.x, q.y, yy.x, yy.y};
#pragma unroll
        for (int e = 0; e < 4; ++e)
          __hip_atomic_store(cur + wg * kRec + e * R + t, __builtin_bit_cast(uint64_t, w4[e]), __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
      }
      {
        uint64_t w4[kAll / 512] = {};
        uint64_t t0 = 0;
        late = wait_ticks == 0;
        for (int spin = 0; !late; ++spin) {
          bool ok = true;
#pragma unroll
          for (int e = 0; e < kAll / 512; ++e) {
            w4[e] = __hip_atomic_load(cur + t + 512 * e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            ok = ok && w4[e] != kEmpty;
          }
          if (ok) break;
          if ((spin & 63) == 0) {
            const uint64_t now = wall_clock64();
            if (spin == 0) t0 = now;
            late = now - t0 > wait_ticks;
          }
        }
#pragma unroll
        for (int e = 0; e < kAll / 512; ++e) {
          const int word = t + 512 * e, rec = word / kRec, in = word % kRec;
          const int i = (in % R) * NW + rec, part = in / R;
          double* const to = (double*)(part < 2 ? s_p : s_y) + 2 * i + (part & 1);
          *to = __builtin_bit_cast(double, w4[e]);
        }
      }
      if (__syncthreads_or(late)) {  // a row's owner did not come: give up, all of them will
        if (t == 0) atomicOr(info, kTrdLate);
        if (wg == 0 && t == 0) no_matrix();
        return;
      }
      if (t < n) {  // the records cover R NW rows, which may be fewer than the threads
        p = s_p[t];
        y = s_y[t];
      }
      if (t < 64 && t < kRec) {  // clear the buffer of the column before: every workgroup has published this one
        uint64_t* const old = pub + ((j + 2) % 3) * kAll + wg * kRec;
        for (int e = t; e < kRec; e += 64)
          __hip_atomic_store(old + e, kEmpty, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // cleared before this workgroup publishes again
      }
    }
    // w = p - (tau / 2) (p^H v) v
    double dr = wave_sum63(fma(p.x, v.x, p.y * v.y)), di = wave_sum63(fma(p.x, v.y, -p.y * v.x));  // conj(p) v
    if (lane == 63) {
      s_sum[1][t >> 6] = dr;
      s_sum[2][t >> 6] = di;
    }
    __syncthreads();  // orders s_p too
    dr = di = 0.0;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      dr += s_sum[1][q];
      di += s_sum[2][q];
    }
    const cd a2 = mul(cd{-0.5 * tau.x, -0.5 * tau.y}, cd{dr, di});
    cd w = p;
    fma_c(w, a2, v);
    s_w[t] = w;
    // column j + 1 after the update: y - v conj(w_{j+1}) - w conj(1)
    const cd w1 = s_p[j + 1] + a2;
    cd nx = {y.x - w.x, y.y - w.y};
    fms_conj(nx, v, w1);
    s_x[t] = t > j && t < n ? nx : cd{0.0, 0.0};
    // the reflector to memory: column j of the matrix, which every workgroup has read by now
    if (wg == 0 && t > j && t < n) A[(int64_t)j * n + t] = v;
    __syncthreads();
    cd vi[RA], wi[RA];
#pragma unroll
    for (int a = 0; a < RA; ++a) {
      const int i = (tr + TR * a) * NW + wg;
      vi[a] = i < 512 ? s_v[i] : cd{0.0, 0.0};
      wi[a] = i < 512 ? s_w[i] : cd{0.0, 0.0};
    }
#pragma unroll
    for (int b = 0; b < CB; ++b) {
      if (TC * (b + 1) <= j + 1) continue;
      const cd vc = s_v[tc + TC * b], wc = s_w[tc + TC * b];
#pragma unroll
      for (int a = 0; a < RA; ++a) {
        fms_conj(C[a][b], vi[a], wc);
        fms_conj(C[a][b], wi[a], vc);
      }
    }
  }
  if (wg == 0 && t == 0) {
    const double d = s_x[n - 1].x;
    finite = finite && isfinite(d);
    D[n - 1] = d;
    if (!finite) {  // nothing for the tridiagonal solver: zeros, and say so
      atomicOr(info, kTrdNotFinite);
      no_matrix();
    }
  }
}

__global__ __launch_bounds__(256) void eig_clear_kernel(uint64_t* __restrict__ pub, int* __restrict__ info,
                                                        int n_info) {
  const int i = blockIdx.x * 256 + threadIdx.x;  // a thread per word
  pub[i] = kEmpty;
  if (i < n_info) info[i] = 0;
}

// ---- eigenvectors of C ----------------------------------------------------------
// U = H_0 H_1 ... H_{n-2} Z, a column of U per wave in registers (element lane +
// 64 k in slot k), the reflectors read in order from L2, one ahead.  Bound by the
// n dependent reflectors, each a sum over the wave.
template <int NK>
__global__ __launch_bounds__(256) void reflect_kernel(const cd* __restrict__ V, const cd* __restrict__ tau, int n,
                                                      const double* __restrict__ Z, cd* __restrict__ U) {
  const int lane = threadIdx.x & 63;
  const int col = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (col >= n) return;
  cd z[NK], v[NK];
  auto load = [&](int j, cd (&r)[NK]) {
#pragma unroll
    for (int k = 0; k < NK; ++k) {
      const int i = lane + 64 * k;
      r[k] = i > j && i < n ? V[(int64_t)j * n + i] : cd{0.0, 0.0};
    }
  };
#pragma unroll
  for (int k = 0; k < NK; ++k) {
    const int i = lane + 64 * k;
    z[k] = {i < n ? Z[(int64_t)col * n + i] : 0.0, 0.0};
  }
  cd tj = {0.0, 0.0};
  if (n >= 2) {
    load(n - 2, v);
    tj = tau[n - 2];
  }
  for (int j = n - 2; j >= 0; --j) {
    cd nx[NK], tn = {0.0, 0.0};
    if (j > 0) {
      load(j - 1, nx);
      tn = tau[j - 1];
    }
    double a = 0.0, b = 0.0;  // v^H z
#pragma unroll
    for (int k = 0; k < NK; ++k) {
      a = fma(v[k].x, z[k].x, fma(v[k].y, z[k].y, a));
      b = fma(v[k].x, z[k].y, fma(-v[k].y, z[k].x, b));
    }
    a = wave_sum63(a);
    b = wave_sum63(b);
    a = lane_of(a, 63);
    b = lane_of(b, 63);
    const cd f = mul(tj, cd{-a, -b});
#pragma unroll
    for (int k = 0; k < NK; ++k) fma_c(z[k], f, v[k]);
#pragma unroll
    for (int k = 0; k < NK; ++k) v[k] = nx[k];
    tj = tn;
  }
#pragma unroll
  for (int k = 0; k < NK; ++k) {
    const int i = lane + 64 * k;
    if (i < n) U[(int64_t)col * n + i] = z[k];
  }
}

template <int NW, int TR, int RA, int CB>
void launch_trd(const EigBuffers& b, int n, uint64_t wait_ticks, hipStream_t s) {
  using K = TrdCfg<NW, TR, RA, CB>;
  hipLaunchKernelGGL((hetrd_kernel<K, NW, TR, RA, CB>), dim3(NW > 1 ? 8 * NW : 1), dim3(512), 0, s, (cd*)b.A, n, b.D,
                     b.E, (cd*)b.tau, b.pub, wait_ticks, &b.status->chol, &b.status->trd);
}

}  // namespace

// three buffers of 4 words for up to 512 rows, whatever n
constexpr int kPubWords = 3 * 4 * kEigMaxN;
size_t eig_pub_bytes() { return kPubWords * sizeof(uint64_t); }

hipError_t launch_eig_reduce(const EigBuffers& b, const double* ant, const double* vis, int n, double wl,
                             bool identity, uint64_t wait_ticks, hipStream_t s) {
  hipLaunchKernelGGL(eig_clear_kernel, dim3(kPubWords / 256), dim3(256), 0, s, b.pub, (int*)b.status,
                     (int)(offsetof(EigStatus, herm) / sizeof(int)));
  hipLaunchKernelGGL(eig_inputs_kernel, dim3(kHermParts), dim3(256), 0, s, ant, n, 1.0 / wl, identity ? 1 : 0, vis,
                     b.A, b.G, b.status->herm, &b.status->coincident);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (!identity) {
    const int nb = (n + kNB - 1) / kNB;
    for (int k = 0; k < nb; ++k) {
      hipLaunchKernelGGL(chol_diag_kernel, dim3(1), dim3(512), 0, s, b.G, b.Y, n, k, &b.status->chol);
      if (nb > 1) hipLaunchKernelGGL(chol_panel_kernel, dim3(nb - 1), dim3(256), 0, s, b.G, b.Y, n, k);
      if (k + 1 < nb)
        hipLaunchKernelGGL(chol_update_kernel, dim3(nb - 1 - k, nb), dim3(256), 0, s, b.G, b.Y, n, k);
    }
    const dim3 grid((n + 31) / 32, (n + 31) / 32);
    // X = Y V, then C^T(j, i) = sum_k Y(j, k) X(i, k)
    hipLaunchKernelGGL(tri_product_kernel<false>, grid, dim3(256), 0, s, b.Y, (const cd*)b.A, (int64_t)1, (int64_t)n,
                       (cd*)b.T, (int64_t)1, (int64_t)n, n);
    hipLaunchKernelGGL(tri_product_kernel<false>, grid, dim3(256), 0, s, b.Y, (const cd*)b.T, (int64_t)n, (int64_t)1,
                       (cd*)b.A, (int64_t)n, (int64_t)1, n);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  // rows over as few workgroups as hold them in registers; one needs no exchange
  if (n <= 64)
    launch_trd<1, 16, 4, 2>(b, n, wait_ticks, s);
  else if (n <= 128)
    launch_trd<1, 16, 8, 4>(b, n, wait_ticks, s);
  else if (n <= 256)
    launch_trd<16, 8, 2, 4>(b, n, wait_ticks, s);
  else
    launch_trd<32, 4, 4, 4>(b, n, wait_ticks, s);
  return hipGetLastError();
}

hipError_t launch_eig_vectors(const EigBuffers& b, int n, bool identity, hipStream_t s) {
  const dim3 grid((n + 3) / 4), block(256);
  const cd* V = (const cd*)b.A;
  const cd* tau = (const cd*)b.tau;
  cd* U = (cd*)b.U;
  const double* Z = b.T;
  if (n <= 64)
    hipLaunchKernelGGL(reflect_kernel<1>, grid, block, 0, s, V, tau, n, Z, U);
  else if (n <= 128)
    hipLaunchKernelGGL(reflect_kernel<2>, grid, block, 0, s, V, tau, n, Z, U);
  else if (n <= 256)
    hipLaunchKernelGGL(reflect_kernel<4>, grid, block, 0, s, V, tau, n, Z, U);
  else
    hipLaunchKernelGGL(reflect_kernel<8>, grid, block, 0, s, V, tau, n, Z, U);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (identity) return launch_copy_c128(b.U, n, b.A, n, s);
  hipLaunchKernelGGL(tri_product_kernel<true>, dim3((n + 31) / 32, (n + 31) / 32), dim3(256), 0, s, b.Y, (const cd*)b.U,
                     (int64_t)1, (int64_t)n, (cd*)b.A, (int64_t)1, (int64_t)n, n);
  return hipGetLastError();
}

}  // namespace bb
