// SparseGPT 2:4 pruning with a protected dense region, on the GPU (paper sec. 3.1.2,
// Eqs. (2)-(3); sec. 3.3.1: the dense columns are placed last so that they absorb the
// compensation of the 2:4 columns processed before them).
//
// Two offline steps:
//  1. The factor.  U upper triangular with Hd^{-1} = U^T U, Hd = H + lambda I (plus
//     H_jj = 1 for columns no input excites).  Row j of U scaled by U_jj is row j of the
//     inverse Hessian of the columns j..K-1, so U_jj^2 is the OBS denominator of Eq. (3)
//     for column j and U[j, j:] / U_jj its compensation direction.  With P the index
//     reversal, P Hd P = L L^T (lower Cholesky) gives Hd = (P L P)(P L P)^T with P L P
//     upper, hence U = (P L P)^{-1} = P L^{-1} P: one Cholesky factorisation and one
//     triangular inverse of the reversed matrix, then a reversal back.  Both are blocked
//     (64-wide diagonal blocks factored and inverted in LDS, everything else as fp32
//     matrix-core products).
//  2. The sweep, 64 columns at a time: four lanes per row keep the row's 64 weights of
//     the block in registers and process the columns in order (2:4 choice at each
//     group's first column by the OBS error w^2 / U_mm^2, then the compensation inside
//     the block); the block's scaled errors E then update every later column at once,
//     W[:, j0+64:] -= E U[j0:j0+64, j0+64:], on the matrix cores.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>
#include <utility>

#include "spense.h"
#include "spense_internal.h"

namespace spense {
namespace {

typedef float f4 __attribute__((ext_vector_type(4)));

constexpr int NB = 64;  // diagonal block of the factorisations, sweep block, GEMM tile

template <typename F, int... I>
__device__ __forceinline__ void unrolled_impl(F& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>()), ...);
}
// f(integral_constant<int, i>) for i = 0 .. N-1: every index a compile-time constant.
template <int N, typename F>
__device__ __forceinline__ void unrolled(F&& f) {
  unrolled_impl(f, std::make_integer_sequence<int, N>());
}

// ------------------------------------------------------------------ fp32 matrix-core GEMM
// C[i][j] = beta C[i][j] + alpha sum_k A[i][k] B(k, j) over an m x n output, row-major
// operands, B(k, j) = TB ? B[j][k] : B[k][j].
// LOWER: only output tiles on or below the diagonal (tile column <= tile row) are formed.
// TRI (bit mask) marks triangular operands whose other half is read as 0 (and holds
// anything in memory): 1 = A lower (A[i][k] = 0 for k > i), 2 = B(k, j) = 0 for k > j,
// 4 = B(k, j) = 0 for k < j; the k loop is cut to the range they leave.
// BT x BT output tile per workgroup of 4 waves (2 x 2; each BT/2 x BT/2 as TW x TW
// v_mfma_f32_16x16x4_f32 tiles), k staged through LDS 16 deep in two buffers, 16-byte
// loads when the operands allow.
// Operand lanes (measured): A lane l = A[l % 16][l / 16], B lane l = B[l / 16][l % 16],
// D lane l, element r = D[4 (l / 16) + r][l % 16].
struct GemmF32 {
  const float* A;
  int64_t lda;
  const float* B;
  int64_t ldb;
  float* C;
  int64_t ldc;
  int64_t m, n, k;
  float alpha, beta;
};

template <int BT, bool TB, bool LOWER, int TRI>
__global__ __launch_bounds__(256) void gemm_f32_kernel(GemmF32 g, int vec) {
  // LDS row pitch (floats): the four rows an operand read takes (k = 4 q + lane / 16) start
  // 16 banks apart.  Columns of row kk sit at column ^ 16 (kk / 4 % 4), so that the rows 4
  // apart that a transposing store writes do too.
  constexpr int P = BT + 16;
  constexpr int TW = BT / 32;      // MFMA tiles per wave and dimension
  constexpr int NQ = BT / 64;      // 16-byte pieces per thread and operand per step
  __shared__ float As[2][16][P];   // As[kk][i]
  __shared__ float Bs[2][16][P];   // Bs[kk][j]
  const int tr = blockIdx.y, tc = blockIdx.x;
  if (LOWER && tc > tr) return;
  const int64_t i0 = (int64_t)tr * BT, j0 = (int64_t)tc * BT;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int wi = (wave >> 1) * (BT / 2), wj = (wave & 1) * (BT / 2);
  int64_t klo = 0, khi = g.k;
  if (TRI & 1) khi = khi < i0 + BT ? khi : i0 + BT;
  if (TRI & 2) khi = khi < j0 + BT ? khi : j0 + BT;
  if (TRI & 4) klo = j0;
  const int s0 = (int)(klo / 16), s1 = (int)((khi + 15) / 16);

  float ra[NQ][4], rb[NQ][4];
  // four consecutive elements of a row-major operand at (row, k), zero outside
  // [klo, khi), past `rows` and where `keep(k)` says the triangular half is empty
  auto quad = [&](const float* base, int64_t ld, int64_t row, int64_t rows, int64_t kq, float* out, auto keep)
      __attribute__((always_inline)) {
    const bool full = vec && row < rows && kq >= klo && kq + 3 < khi;
    if (full) {
      const float4 v = *reinterpret_cast<const float4*>(base + row * ld + kq);
      out[0] = v.x;
      out[1] = v.y;
      out[2] = v.z;
      out[3] = v.w;
    } else {
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int64_t kk = kq + c;
        out[c] = (row < rows && kk >= klo && kk < khi) ? base[row * ld + kk] : 0.0f;
      }
    }
#pragma unroll
    for (int c = 0; c < 4; ++c)
      if (!keep(kq + c)) out[c] = 0.0f;
  };
  // Steps whose 16 columns lie inside every operand and off the triangular edges take plain
  // 16-byte loads from pointers that advance by a step; the bounds and masks of the others
  // cost more instructions than the step's 64 matrix instructions leave room for.
  const bool inside = vec && i0 + BT <= g.m && j0 + BT <= g.n;
  const float* pa[NQ];
  const float* pb[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int slot = t + 256 * q;
    pa[q] = g.A + (i0 + (slot >> 2)) * g.lda + (slot & 3) * 4;
    pb[q] = TB ? g.B + (j0 + (slot >> 2)) * g.ldb + (slot & 3) * 4
               : g.B + (int64_t)(slot / (BT / 4)) * g.ldb + j0 + (slot % (BT / 4)) * 4;
  }
  auto load = [&](int s) __attribute__((always_inline)) {
    const int64_t k0 = (int64_t)s * 16;
    if (inside && k0 >= klo && k0 + 16 <= khi && (!(TRI & 1) || k0 + 15 <= i0) && (!(TRI & 2) || k0 + 15 <= j0) &&
        (!(TRI & 4) || k0 >= j0 + BT - 1)) {
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        const float4 x = *reinterpret_cast<const float4*>(pa[q] + k0);
        const float4 y = *reinterpret_cast<const float4*>(pb[q] + (TB ? k0 : k0 * g.ldb));
        ra[q][0] = x.x, ra[q][1] = x.y, ra[q][2] = x.z, ra[q][3] = x.w;
        rb[q][0] = y.x, rb[q][1] = y.y, rb[q][2] = y.z, rb[q][3] = y.w;
      }
      return;
    }
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const int slot = t + 256 * q;
      const int64_t i = i0 + (slot >> 2), kq = k0 + (slot & 3) * 4;
      quad(g.A, g.lda, i, g.m, kq, ra[q], [&](int64_t kk) { return !(TRI & 1) || kk <= i; });
      if (TB) {
        const int64_t j = j0 + (slot >> 2);
        quad(g.B, g.ldb, j, g.n, kq, rb[q], [&](int64_t kk) {
          return (!(TRI & 2) || kk <= j) && (!(TRI & 4) || kk >= j);
        });
      } else {
        const int64_t kk = k0 + slot / (BT / 4), jq = j0 + (slot % (BT / 4)) * 4;
        const bool full = vec && kk >= klo && kk < khi && jq + 3 < g.n;
        if (full) {
          const float4 v = *reinterpret_cast<const float4*>(g.B + kk * g.ldb + jq);
          rb[q][0] = v.x;
          rb[q][1] = v.y;
          rb[q][2] = v.z;
          rb[q][3] = v.w;
        } else {
#pragma unroll
          for (int c = 0; c < 4; ++c)
            rb[q][c] = (kk >= klo && kk < khi && jq + c < g.n) ? g.B[kk * g.ldb + jq + c] : 0.0f;
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const int64_t j = jq + c;
          if (((TRI & 2) && kk > j) || ((TRI & 4) && kk < j)) rb[q][c] = 0.0f;
        }
      }
    }
  };
  auto store = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const int slot = t + 256 * q;
#pragma unroll
      for (int c = 0; c < 4; ++c) As[buf][(slot & 3) * 4 + c][(slot >> 2) ^ (16 * (slot & 3))] = ra[q][c];
      if (TB) {
#pragma unroll
        for (int c = 0; c < 4; ++c) Bs[buf][(slot & 3) * 4 + c][(slot >> 2) ^ (16 * (slot & 3))] = rb[q][c];
      } else {
        const int kr = slot / (BT / 4);
        *reinterpret_cast<float4*>(&Bs[buf][kr][((slot % (BT / 4)) * 4) ^ (16 * ((kr >> 2) & 3))]) =
            make_float4(rb[q][0], rb[q][1], rb[q][2], rb[q][3]);
      }
    }
  };

  f4 acc[TW][TW];
#pragma unroll
  for (int a = 0; a < TW; ++a)
#pragma unroll
    for (int b = 0; b < TW; ++b) acc[a][b] = f4{0.0f, 0.0f, 0.0f, 0.0f};

  if (s0 < s1) {
    load(s0);
    store(0);
  }
  __syncthreads();
  for (int s = s0; s < s1; ++s) {
    const int buf = (s - s0) & 1;
    if (s + 1 < s1) load(s + 1);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int kk = q * 4 + (lane >> 4);
      float av[TW], bv[TW];
#pragma unroll
      for (int a = 0; a < TW; ++a) av[a] = As[buf][kk][(wi + a * 16 + (lane & 15)) ^ (16 * q)];
#pragma unroll
      for (int b = 0; b < TW; ++b) bv[b] = Bs[buf][kk][(wj + b * 16 + (lane & 15)) ^ (16 * q)];
#pragma unroll
      for (int a = 0; a < TW; ++a)
#pragma unroll
        for (int b = 0; b < TW; ++b) acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[a], bv[b], acc[a][b], 0, 0, 0);
    }
    if (s + 1 < s1) store(buf ^ 1);
    __syncthreads();
  }
  // C is read ahead of the stores, a row of tiles at a time: read next to its store, each
  // element would wait for the store before it, which may alias (64 round trips a tile)
#pragma unroll
  for (int a = 0; a < TW; ++a) {
    float c[TW][4];
#pragma unroll
    for (int b = 0; b < TW; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t i = i0 + wi + a * 16 + 4 * (lane >> 4) + r, j = j0 + wj + b * 16 + (lane & 15);
        c[b][r] = g.beta != 0.0f && i < g.m && j < g.n ? g.C[i * g.ldc + j] : 0.0f;
      }
#pragma unroll
    for (int b = 0; b < TW; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t i = i0 + wi + a * 16 + 4 * (lane >> 4) + r, j = j0 + wj + b * 16 + (lane & 15);
        const float v = g.alpha * acc[a][b][r];
        if (i < g.m && j < g.n) g.C[i * g.ldc + j] = g.beta == 0.0f ? v : g.beta * c[b][r] + v;
      }
  }
}

// Output tiles of 128 from which they are used instead of 64: a workgroup takes ~0.9 us per
// 16 columns of k on a 128 tile and a quarter of that on a 64 one, so 64 is faster until both
// fill the CUs several times over (the factor at K = 5120: 128 tiles from 1 / 300 / 1024 on
// 11.0 / 7.1 / 6.6 ms); beyond, 128 reads its operands half as often.
constexpr int64_t kWideTiles = 1024;

template <bool TB, bool LOWER, int TRI>
hipError_t gemm_f32(const GemmF32& g, hipStream_t st) {
  if (g.m <= 0 || g.n <= 0) return hipSuccess;
  const int vec = (g.lda % 4 == 0) && (g.ldb % 4 == 0) && ((uintptr_t)g.A % 16 == 0) && ((uintptr_t)g.B % 16 == 0);
  if ((int64_t)((g.m + 127) / 128) * ((g.n + 127) / 128) >= kWideTiles) {
    const dim3 grid((unsigned)((g.n + 127) / 128), (unsigned)((g.m + 127) / 128));
    hipLaunchKernelGGL((gemm_f32_kernel<128, TB, LOWER, TRI>), grid, dim3(256), 0, st, g, vec);
  } else {
    const dim3 grid((unsigned)((g.n + 63) / 64), (unsigned)((g.m + 63) / 64));
    hipLaunchKernelGGL((gemm_f32_kernel<64, TB, LOWER, TRI>), grid, dim3(256), 0, st, g, vec);
  }
  return hipGetLastError();
}

// ------------------------------------------------------------------ the factor
// Damping: lambda = percdamp * mean(diag H) with H_jj = 0 read as 1 (and flagged dead).
// One workgroup; the sum runs in a fixed order.  st[0] = lambda.
__global__ __launch_bounds__(1024) void damp_kernel(const float* __restrict__ H, int64_t ldh, int64_t K,
                                                   float percdamp, uint8_t* __restrict__ dead,
                                                   float* __restrict__ st) {
  __shared__ float red[16];
  float acc = 0.0f;
  for (int64_t j = threadIdx.x; j < K; j += 1024) {
    const float h = H[j * ldh + j];
    dead[j] = h == 0.0f ? 1 : 0;
    acc += h == 0.0f ? 1.0f : h;
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) acc += __shfl_xor(acc, o, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    float s = 0.0f;
    for (int w = 0; w < 16; ++w) s += red[w];
    st[0] = percdamp * (s / (float)K);
  }
}

// A[a][b] = Hd[K-1-a][K-1-b] for a >= b, read from the lower triangle of H (the reversed
// pair (K-1-a, K-1-b) has its larger index first when swapped).  64 x 64 tiles.
__global__ __launch_bounds__(256) void reverse_damp_kernel(const float* __restrict__ H, int64_t ldh, int64_t K,
                                                           const uint8_t* __restrict__ dead,
                                                           const float* __restrict__ st, float* __restrict__ A,
                                                           int64_t lda) {
  const int64_t a0 = (int64_t)blockIdx.y * 64, b0 = (int64_t)blockIdx.x * 64;
  if (b0 > a0) return;
  const float lambda = st[0];
  for (int e = threadIdx.x; e < 64 * 64; e += 256) {
    const int64_t a = a0 + (e >> 6), b = b0 + (e & 63);
    if (a >= K || b > a) continue;
    const int64_t r = K - 1 - b, c = K - 1 - a;  // r >= c: the lower triangle of H
    float v = H[r * ldh + c];
    if (a == b) v = (dead[r] ? 1.0f : v) + lambda;
    A[a * lda + b] = v;
  }
}

__device__ __forceinline__ float lane_value(float v, int lane) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}

// A 64 x 64 lower Cholesky block and its inverse: L is factored and X = L^{-1} replaces it.
// A workgroup of 8 waves; wave w holds columns w, w + 8, ... of L and of the running
// right-hand side R of L X = I, lane t row t.  Step j: the column's owner takes the pivot
// L_jj, scales the column and passes it on through LDS (two buffers, one barrier a step);
// every lane below j then updates its row, and row j of X is R_j / L_jj.  A non-positive or
// NaN pivot sets *fail and continues with pivot 1 so that the rest stays finite.  Each
// element sees the operations of a one-wave elimination in the same order.  The chain of 64
// pivots (sqrt, division, broadcast) and the instructions of the updates bound it: one wave
// with all columns took 43 us, eight take 31.
// get(t, c) reads an element (identity past the block), put(i, t, c, x) takes X.
struct PotrfLds {
  float col[2][64];
  float inv[2];
};
template <typename Get, typename Put>
__device__ __forceinline__ void potrf64(PotrfLds& sh, int n, int* fail, Get get, Put put) {
  const int t = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  float L[8], R[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int c = w + 8 * i;
    L[i] = get(t, c);
    R[i] = t == c ? 1.0f : 0.0f;
  }
  bool bad = false;
  unrolled<8>([&](auto i_const) __attribute__((always_inline)) {
    constexpr int i8 = decltype(i_const)::value;
    for (int w8 = 0; w8 < 8; ++w8) {
      const int j = 8 * i8 + w8, buf = w8 & 1;
      if (w == w8) {
        float d = lane_value(L[i8], j);
        if (!(d > 0.0f)) {
          bad = bad || j < n;
          d = 1.0f;
        }
        const float s = sqrtf(d), inv = 1.0f / s;
        L[i8] = t == j ? s : (t > j ? L[i8] * inv : L[i8]);
        sh.col[buf][t] = L[i8];
        if (t == 0) sh.inv[buf] = inv;
      }
      __syncthreads();
      const float v = sh.col[buf][t], inv = sh.inv[buf];
      const float ltj = t > j ? v : 0.0f;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int c = w + 8 * i;
        if (c > j) {
          L[i] = __builtin_fmaf(-ltj, lane_value(v, c), L[i]);
        } else {
          if (t == j) R[i] *= inv;
          R[i] = __builtin_fmaf(-ltj, lane_value(R[i], j), R[i]);
        }
      }
    }
  });
  if (bad && t == 0) atomicOr(fail, 1);
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int c = w + 8 * i;
    put(t, c, c <= t ? R[i] : 0.0f);
  }
}

__global__ __launch_bounds__(512) void potrf_block_kernel(float* __restrict__ A, int64_t lda, int n,
                                                          int* __restrict__ fail) {
  __shared__ PotrfLds sh;
  potrf64(
      sh, n, fail,
      [&](int t, int c) { return t < n && c <= t && c < n ? A[t * lda + c] : (t == c ? 1.0f : 0.0f); },
      [&](int t, int c, float x) {
        if (t < n && c < n) A[t * lda + c] = x;
      });
}

// A block of 65 .. 128 in one workgroup: the recursion of chol_inv on two 64-wide halves
// (n2 = n - 64 rows in the second), whose products are 64 x 64 x 64 from LDS with the matrix
// instruction and the k order of gemm_f32_kernel.  Otherwise two leaves, four products and a copy,
// about 100 us of dependent launches; this takes 66.
__global__ __launch_bounds__(512) void chol_pair_kernel(float* __restrict__ A, int64_t lda, int n,
                                                        int* __restrict__ fail) {
  constexpr int P = 65;  // LDS row pitch
  __shared__ PotrfLds sh;
  __shared__ float Xa[64][P], Ld[64][P], Xb[64][P];  // X11; A21, then L21, then T; A22, then X22
  const int n2 = n - 64, tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ti = wave >> 1, tj = 2 * (wave & 1);  // the wave's two 16 x 16 tiles: (ti, tj), (ti, tj + 1)
  const int li = lane & 15, lq = lane >> 4;
  float* const A21 = A + 64 * lda;
  float* const A22 = A21 + 64;
  for (int e = tid; e < 64 * 64; e += 512) {
    const int r = e >> 6, c = e & 63;
    Ld[r][c] = r < n2 ? A21[r * lda + c] : 0.0f;
  }
  potrf64(
      sh, 64, fail, [&](int t, int c) { return c <= t ? A[t * lda + c] : 0.0f; },
      [&](int t, int c, float x) {
        Xa[t][c] = x;
        A[t * lda + c] = x;
      });
  __syncthreads();
  f4 acc[2];
  // acc = sum_k a(i, k) b(k, j) over the wave's tiles
  auto product = [&](auto a, auto b) __attribute__((always_inline)) {
    acc[0] = acc[1] = f4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int k = 4 * q + lq;
      const float av = a(16 * ti + li, k);
#pragma unroll
      for (int b2 = 0; b2 < 2; ++b2)
        acc[b2] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, b(k, 16 * (tj + b2) + li), acc[b2], 0, 0, 0);
    }
  };
  auto each = [&](auto f) __attribute__((always_inline)) {  // f(i, j, value) of the wave's tiles
#pragma unroll
    for (int b2 = 0; b2 < 2; ++b2)
#pragma unroll
      for (int r = 0; r < 4; ++r) f(16 * ti + 4 * lq + r, 16 * (tj + b2) + li, acc[b2][r]);
  };
  // L21 = A21 X11^T
  product([&](int i, int k) { return Ld[i][k]; }, [&](int k, int j) { return Xa[j][k]; });
  __syncthreads();
  each([&](int i, int j, float v) { Ld[i][j] = v; });
  __syncthreads();
  // A22 -= L21 L21^T
  product([&](int i, int k) { return Ld[i][k]; }, [&](int k, int j) { return Ld[j][k]; });
  each([&](int i, int j, float v) { Xb[i][j] = i < n2 && j <= i ? A22[i * lda + j] - v : (i == j ? 1.0f : 0.0f); });
  // T = L21 X11
  product([&](int i, int k) { return Ld[i][k]; }, [&](int k, int j) { return Xa[k][j]; });
  __syncthreads();
  each([&](int i, int j, float v) { Ld[i][j] = v; });
  potrf64(
      sh, n2, fail, [&](int t, int c) { return Xb[t][c]; }, [&](int t, int c, float x) { Xb[t][c] = x; });
  __syncthreads();
  for (int e = tid; e < 64 * 64; e += 512) {
    const int r = e >> 6, c = e & 63;
    if (r < n2 && c < n2) A22[r * lda + c] = Xb[r][c];
  }
  // X21 = -X22 T
  product([&](int i, int k) { return Xb[i][k]; }, [&](int k, int j) { return Ld[k][j]; });
  each([&](int i, int j, float v) {
    if (i < n2) A21[i * lda + j] = -v;
  });
}

// The reversal back: U[K-1-a][K-1-b] = X[a][b] for a > b (lower -> upper), and the
// diagonal reversed (pairs swapped).  Reads only the lower triangle, writes only the
// upper triangle and the diagonal pairs each thread owns.
__global__ __launch_bounds__(256) void reverse_out_kernel(float* __restrict__ A, int64_t lda, int64_t K) {
  const int64_t a0 = (int64_t)blockIdx.y * 64, b0 = (int64_t)blockIdx.x * 64;
  if (b0 > a0) return;
  for (int e = threadIdx.x; e < 64 * 64; e += 256) {
    const int64_t a = a0 + (e >> 6), b = b0 + (e & 63);
    if (a >= K || b > a) continue;
    if (a > b) {
      A[(K - 1 - a) * lda + (K - 1 - b)] = A[a * lda + b];
    } else if (a < K - 1 - a) {
      const int64_t z = K - 1 - a;
      const float x = A[a * lda + a], y = A[z * lda + z];
      A[a * lda + a] = y;
      A[z * lda + z] = x;
    }
  }
}

__global__ __launch_bounds__(256) void zero_lower_kernel(float* __restrict__ A, int64_t lda, int64_t K) {
  const int64_t a0 = (int64_t)blockIdx.y * 64, b0 = (int64_t)blockIdx.x * 64;
  if (b0 > a0) return;
  for (int e = threadIdx.x; e < 64 * 64; e += 256) {
    const int64_t a = a0 + (e >> 6), b = b0 + (e & 63);
    if (a < K && b < a) A[a * lda + b] = 0.0f;
  }
}

// ------------------------------------------------------------------ the sweep
// A thread per column: most columns are not dead and end here.
__global__ __launch_bounds__(256) void zero_dead_kernel(float* __restrict__ W, int64_t ldw, int64_t N, int64_t K,
                                                        const uint8_t* __restrict__ dead) {
  const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (j >= K || !dead[j]) return;
  for (int64_t n = blockIdx.y; n < N; n += gridDim.y) W[n * ldw + j] = 0.0f;
}

// Lane m's value for all four lanes of a quad.
template <int M>
__device__ __forceinline__ float quad_value(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), M * 0x55, 0xf, 0xf, true));
}

// One 64-column block [j0, j0 + 64) of the sweep; columns j0 .. j0+cnt-1 are 2:4 columns
// (cnt a multiple of 4), the rest of the block (dense columns, or past K) only take
// updates.  Four lanes per row, lane l the columns 4 i + l in registers (every index a
// compile-time constant), so that a group of four has one column per lane; U's block (upper;
// 1 on the diagonal past K) in LDS in the lanes' order, the rows, their errors and flags in
// and out through LDS as whole rows.  Writes the block back, the kept flags of the whole
// block (1 for the columns past the 2:4 ones) and E[n][c] = (w_c - q_c) / U_cc (0 where
// nothing changed).  Each weight takes the updates of a thread-per-row sweep in the same
// order.  What bounds it is the chain over the 64 columns (a division and a broadcast each);
// with a thread per row (75 workgroups at 19200 rows, every load and store of a lane in a
// line of its own) a block took 57 us, now 29.
__global__ __launch_bounds__(256) void sweep_block_kernel(float* __restrict__ W, int64_t ldw, int64_t N, int64_t K,
                                                          const float* __restrict__ U, int64_t ldu, int64_t j0, int cnt,
                                                          uint8_t* __restrict__ keep, int64_t ldk,
                                                          float* __restrict__ E, int64_t lde) {
  constexpr int P = 68;  // row pitch of the staged rows: the lanes of 16 rows in 64 banks
  __shared__ __attribute__((aligned(16))) float Ub[64][64];  // Ub[c][16 l + i] = U[c][4 i + l]
  __shared__ float Wt[64][P], Et[64][P];
  __shared__ uint8_t Kt[64][64];
  const int width = (int)(K - j0 < 64 ? K - j0 : 64);
  const int64_t n0 = (int64_t)blockIdx.x * 64;
  {
    // every load before the first use (addresses clamped into the block)
    const int c = threadIdx.x & 63, cc = c < width ? c : width - 1;
    float u[16], v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int r = (threadIdx.x >> 6) + 4 * i;
      u[i] = U[(j0 + (r < width ? r : width - 1)) * ldu + j0 + cc];
      v[i] = W[(n0 + r < N ? n0 + r : N - 1) * ldw + j0 + cc];
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int r = (threadIdx.x >> 6) + 4 * i;
      Ub[r][16 * (c & 3) + (c >> 2)] = r < width && c < width && c >= r ? u[i] : (r == c ? 1.0f : 0.0f);
      Wt[r][c] = n0 + r < N && c < width ? v[i] : 0.0f;
    }
  }
  __syncthreads();
  const int row = threadIdx.x >> 2, l = threadIdx.x & 3;
  float w[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) w[i] = Wt[row][4 * i + l];
  unrolled<16>([&](auto g_const) __attribute__((always_inline)) {
    constexpr int g = decltype(g_const)::value;
    // OBS error of each weight of the group (Eq. (3)); prune the two smallest, ties pruning
    // the lower index; only inside the 2:4 columns
    const float d = Ub[4 * g + l][16 * l + g];
    const float s = (w[g] * w[g]) / (d * d);
    int rank = 0;
    unrolled<4>([&](auto o_const) __attribute__((always_inline)) {
      constexpr int o = decltype(o_const)::value;
      const float so = quad_value<o>(s);
      rank += (so < s) || (so == s && o < l);
    });
    const bool k = !(4 * g < cnt && rank < 2);
    float em = 0.0f;  // this lane's error
    unrolled<4>([&](auto m_const) __attribute__((always_inline)) {
      constexpr int m = decltype(m_const)::value;
      const float q = k ? w[g] : 0.0f;
      float ec = (w[g] - q) / d;  // the group's column m: lane m's value
      if (l == m) {
        em = ec;
        w[g] = q;
      }
      ec = quad_value<m>(ec);
      const float* u = &Ub[4 * g + m][16 * l];
      if (l > m) w[g] = __builtin_fmaf(-ec, u[g], w[g]);
#pragma unroll
      for (int i = g + 1; i < 16; ++i) w[i] = __builtin_fmaf(-ec, u[i], w[i]);
    });
    Et[row][4 * g + l] = em;
    Kt[row][4 * g + l] = k ? 1 : 0;
  });
#pragma unroll
  for (int i = 0; i < 16; ++i) Wt[row][4 * i + l] = w[i];
  __syncthreads();
  for (int e = threadIdx.x; e < 64 * 64; e += 256) {
    const int r = e >> 6, c = e & 63;
    if (n0 + r >= N) continue;
    E[(n0 + r) * lde + c] = Et[r][c];
    if (c < width) {
      W[(n0 + r) * ldw + j0 + c] = Wt[r][c];
      keep[(n0 + r) * ldk + j0 + c] = Kt[r][c];
    }
  }
}

// keep = 1 on the columns [from, K) of every row.
__global__ __launch_bounds__(256) void keep_dense_kernel(uint8_t* __restrict__ keep, int64_t ldk, int64_t N,
                                                         int64_t from, int64_t K) {
  for (int64_t n = blockIdx.y; n < N; n += gridDim.y)
    for (int64_t j = from + (int64_t)blockIdx.x * 256 + threadIdx.x; j < K; j += (int64_t)gridDim.x * 256)
      keep[n * ldk + j] = 1;
}

__global__ __launch_bounds__(256) void copy_f32_kernel(const float* __restrict__ src, int64_t lds, float* __restrict__ dst,
                                                       int64_t ldd, int64_t rows, int64_t cols) {
  for (int64_t r = blockIdx.y; r < rows; r += gridDim.y) {
    const int64_t c = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (c < cols) dst[r * ldd + c] = src[r * lds + c];
  }
}

dim3 lower_tiles(int64_t K) {
  const unsigned t = (unsigned)((K + 63) / 64);
  return dim3(t, t);
}

// Recursive factor-and-invert of the lower part of A (n x n, in place): on return A holds
// X = L^{-1} with L L^T = A.  With A = [[A11, .], [A21, A22]] split at n1 (a multiple of
// 64): X11 = (L11)^{-1} recursively, L21 = A21 X11^T, A22 -= L21 L21^T, X22 recursively,
// X21 = -X22 (L21 X11).  Every product is a large, square-ish matrix-core GEMM.
// Workspace: L21 (n2 x n1) plus the second recursion's, behind it.
int64_t chol_inv_ws(int64_t n) {
  if (n <= NB) return 0;
  const int64_t n1 = (n / 2 + NB - 1) / NB * NB, n2 = n - n1;
  const int64_t a = chol_inv_ws(n1), b = n2 * n1 + chol_inv_ws(n2);
  return a > b ? a : b;
}

hipError_t chol_inv(float* A, int64_t lda, int64_t n, float* ws, int* fail, hipStream_t st) {
  if (n <= NB) {
    hipLaunchKernelGGL(potrf_block_kernel, dim3(1), dim3(512), 0, st, A, lda, (int)n, fail);
    return hipGetLastError();
  }
  if (n <= 2 * NB) {
    hipLaunchKernelGGL(chol_pair_kernel, dim3(1), dim3(512), 0, st, A, lda, (int)n, fail);
    return hipGetLastError();
  }
  const int64_t n1 = (n / 2 + NB - 1) / NB * NB, n2 = n - n1;
  float* A11 = A;
  float* A21 = A + n1 * lda;
  float* A22 = A21 + n1;
  float* L21 = ws;
  hipError_t e = chol_inv(A11, lda, n1, ws, fail, st);
  // L21 = A21 X11^T (X11 lower: B(k, j) = X11[j][k] vanishes for k > j)
  if (e == hipSuccess) e = gemm_f32<true, false, 2>(GemmF32{A21, lda, A11, lda, L21, n1, n2, n1, n1, 1.0f, 0.0f}, st);
  // A22 -= L21 L21^T, lower tiles
  if (e == hipSuccess) e = gemm_f32<true, true, 0>(GemmF32{L21, n1, L21, n1, A22, lda, n2, n2, n1, -1.0f, 1.0f}, st);
  if (e == hipSuccess) e = chol_inv(A22, lda, n2, ws + n2 * n1, fail, st);
  // T = L21 X11 into A21's place (X11 lower: B(k, j) = X11[k][j] vanishes for k < j)
  if (e == hipSuccess) e = gemm_f32<false, false, 4>(GemmF32{L21, n1, A11, lda, A21, lda, n2, n1, n1, 1.0f, 0.0f}, st);
  // X21 = -X22 T into the workspace (X22 lower), then back into A21's place
  if (e == hipSuccess) e = gemm_f32<false, false, 1>(GemmF32{A22, lda, A21, lda, L21, n1, n2, n1, n2, -1.0f, 0.0f}, st);
  if (e == hipSuccess) {
    hipLaunchKernelGGL(copy_f32_kernel, dim3((unsigned)((n1 + 255) / 256), (unsigned)(n2 < 65535 ? n2 : 65535)),
                       dim3(256), 0, st, L21, n1, A21, lda, n2, n1);
    e = hipGetLastError();
  }
  return e;
}

}  // namespace

// Workspace: lambda at float 0, the failure flag at float 16, the recursion's from
// float 64 on.
size_t obs_factor_workspace(int64_t K) { return (size_t)(64 + chol_inv_ws(K)) * sizeof(float); }

int* obs_factor_fail_flag(void* ws, int64_t) { return reinterpret_cast<int*>(static_cast<float*>(ws) + 16); }

hipError_t launch_obs_factor(const float* H, int64_t ldh, int64_t K, float percdamp, float* U, int64_t ldu,
                             uint8_t* dead, void* ws, hipStream_t st) {
  float* stat = static_cast<float*>(ws);  // lambda
  int* fail = obs_factor_fail_flag(ws, K);
  hipLaunchKernelGGL(damp_kernel, dim3(1), dim3(1024), 0, st, H, ldh, K, percdamp, dead, stat);
  hipLaunchKernelGGL(reverse_damp_kernel, lower_tiles(K), dim3(256), 0, st, H, ldh, K, dead, stat, U, ldu);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess) e = chol_inv(U, ldu, K, stat + 64, fail, st);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(reverse_out_kernel, lower_tiles(K), dim3(256), 0, st, U, ldu, K);
  hipLaunchKernelGGL(zero_lower_kernel, lower_tiles(K), dim3(256), 0, st, U, ldu, K);
  return hipGetLastError();
}

// The sweep in two levels: 64-column blocks inside 256-column outer blocks.  Inside an
// outer block each 64-block's errors update only the rest of the outer block (k = 64);
// at its end the outer block's errors update every later column at once (k = 256), so
// the trailing columns are read and written once per 256 columns instead of per 64.
constexpr int OB = 256;

size_t obs_prune_workspace(int64_t N) { return (size_t)N * OB * sizeof(float); }

hipError_t launch_obs_prune(float* W, int64_t ldw, int64_t N, int64_t K, const float* U, int64_t ldu,
                            const uint8_t* dead, int64_t dense_begin, uint8_t* keep, int64_t ldk, void* ws,
                            hipStream_t st) {
  float* E = static_cast<float*>(ws);  // N x OB: the outer block's scaled errors
  const unsigned rows_y = (unsigned)(N < 65535 ? N : 65535);
  if (dead)
    hipLaunchKernelGGL(zero_dead_kernel, dim3((unsigned)((K + 255) / 256), (unsigned)(N < 64 ? N : 64)), dim3(256), 0, st,
                       W, ldw, N, K, dead);
  hipError_t e = hipGetLastError();
  int64_t pe = 0;  // end of the processed 64-blocks
  for (int64_t o0 = 0; o0 < dense_begin && e == hipSuccess; o0 += OB) {
    const int64_t last = o0 + OB < dense_begin ? o0 + OB : dense_begin;  // 2:4 columns of this outer block end here
    pe = o0 + (last - o0 + NB - 1) / NB * NB;                             // processed blocks end here
    for (int64_t j0 = o0; j0 < last && e == hipSuccess; j0 += NB) {
      const int cnt = (int)(last - j0 < NB ? last - j0 : NB);
      hipLaunchKernelGGL(sweep_block_kernel, dim3((unsigned)((N + 63) / 64)), dim3(256), 0, st, W, ldw, N, K, U,
                         ldu, j0, cnt, keep, ldk, E + (j0 - o0), (int64_t)OB);
      e = hipGetLastError();
      const int64_t c0 = j0 + NB, c1 = pe < K ? pe : K;  // the rest of the processed blocks
      if (e == hipSuccess && c0 < c1)
        e = gemm_f32<false, false, 0>(GemmF32{E + (j0 - o0), OB, U + j0 * ldu + c0, ldu, W + c0, ldw, N, c1 - c0, NB,
                                              -1.0f, 1.0f}, st);
    }
    if (e == hipSuccess && pe < K)
      e = gemm_f32<false, false, 0>(GemmF32{E, OB, U + o0 * ldu + pe, ldu, W + pe, ldw, N, K - pe, pe - o0, -1.0f,
                                            1.0f}, st);
  }
  if (e != hipSuccess) return e;
  const int64_t from = pe < K ? pe : K;  // the sweep blocks wrote the flags of [0, pe)
  if (from < K)
    hipLaunchKernelGGL(keep_dense_kernel, dim3((unsigned)((K - from + 255) / 256 < 64 ? (K - from + 255) / 256 : 64), rows_y),
                       dim3(256), 0, st, keep, ldk, N, from, K);
  return hipGetLastError();
}

}  // namespace spense
