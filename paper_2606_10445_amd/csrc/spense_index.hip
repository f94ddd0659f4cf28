// SpenseGPT+ dense-index selection on the GPU (paper sec. 3.3.1, Eqs. (8)-(12)): each
// intermediate index i of a GLU MLP gets a Wanda-style priority from its row of Wgate and
// Wup and its column of Wdown,
//   s_gate[i] = mean_j |Wgate[i, j]| sqrt(h_in[j]),   s_up likewise,
//   s_down[i] = mean_n |Wdown[n, i]| sqrt(h_mid[i]),
// with h the diagonals of the input Hessians X^T X; each vector is divided by its mean
// (plus eps) and the three are summed.  The pN indices with the largest priority (ties:
// lower index first) are kept dense and permuted to the back, the others keep their
// order in front (Eq. (4): the MLP is unchanged when the rows of Wgate, Wup and the
// columns of Wdown move together).  Offline tooling next to spense_compress; every sum runs in a fixed
// order, so results are deterministic.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <mutex>
#include <type_traits>

#include "spense.h"
#include "spense_internal.h"

namespace spense {
namespace {

template <int TYPE>
__device__ __forceinline__ float wval(const uint8_t* row, int64_t j) {
  if constexpr (TYPE == SPENSE_BF16)
    return __uint_as_float((uint32_t)reinterpret_cast<const uint16_t*>(row)[j] << 16);
  else
    return reinterpret_cast<const float*>(row)[j];
}

template <int THREADS>
__device__ __forceinline__ float block_sum(float v, float* red) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
  const int w = threadIdx.x >> 6;
  __syncthreads();  // red may still be read by a previous call
  if ((threadIdx.x & 63) == 0) red[w] = v;
  __syncthreads();
  float r = 0.0f;
#pragma unroll
  for (int i = 0; i < THREADS / 64; ++i) r += red[i];
  return r;
}

// Row scores of Wgate and Wup, general form: one workgroup per row (blockIdx.y = 0 gate,
// 1 up), element loads.  Used when a row does not split into 16-byte pieces.
template <int TYPE>
__global__ __launch_bounds__(256) void row_scores_kernel(const uint8_t* __restrict__ wg, const uint8_t* __restrict__ wu,
                                                         int64_t ld_b, int64_t D, const float* __restrict__ h_in,
                                                         float* __restrict__ out, int64_t I) {
  __shared__ float red[4];
  const int64_t i = blockIdx.x;
  const uint8_t* row = (blockIdx.y == 0 ? wg : wu) + i * ld_b;
  float acc = 0.0f;
  for (int64_t j = threadIdx.x; j < D; j += 256) acc += fabsf(wval<TYPE>(row, j)) * sqrtf(h_in[j]);
  acc = block_sum<256>(acc, red);
  if (threadIdx.x == 0) out[blockIdx.y * I + i] = acc / (float)D;
}

// Row scores, streaming form: a wave per row (rows 0..I-1 of Wgate, then of Wup, shared
// out among the waves of the grid).  Lane l owns the 16-byte pieces l, l + 64, ... of
// every row (T of them, T <= TMAX) and keeps sqrt(h_in) of their elements in registers;
// the workgroup computes each square root once, in LDS (D <= 8192), so that a wave does
// not spend as long on its 8 T roots as on several rows.  A row's loads are issued before
// the previous row is summed.  Each lane sums its pieces in order, then the wave adds its
// lanes with a fixed butterfly.  HBM-bound: 25600 x 5120 bf16, gate and up, 158 us with
// the roots per wave and one row at a time, 122 now.
template <int TYPE, int TMAX>
__global__ __launch_bounds__(256) void row_scores_wave_kernel(const uint8_t* __restrict__ wg,
                                                              const uint8_t* __restrict__ wu, int64_t ld_b, int64_t D,
                                                              int T, const float* __restrict__ h_in,
                                                              float* __restrict__ out, int64_t I) {
  constexpr int EP = TYPE == SPENSE_BF16 ? 8 : 4;  // elements per 16-byte piece
  __shared__ float root[TMAX * 64 * EP];
  const int lane = threadIdx.x & 63;
  const int64_t wave = ((int64_t)blockIdx.x * 256 + threadIdx.x) >> 6;
  const int64_t nwaves = (int64_t)gridDim.x * 4;
  for (int j = threadIdx.x; j < TMAX * 64 * EP; j += 256) root[j] = j < D ? sqrtf(h_in[j]) : 0.0f;
  __syncthreads();
  float sh[TMAX][EP];
#pragma unroll
  for (int t = 0; t < TMAX; ++t)
#pragma unroll
    for (int e = 0; e < EP; ++e) sh[t][e] = root[(t * 64 + lane) * EP + e];
  auto load = [&](int4 (&v)[TMAX], int64_t r) __attribute__((always_inline)) {
    const uint8_t* row = (r < I ? wg + r * ld_b : wu + (r - I) * ld_b);
#pragma unroll
    for (int t = 0; t < TMAX; ++t) {
      const int64_t j = ((int64_t)t * 64 + lane) * EP;
      v[t] = (t < T && j < D) ? *reinterpret_cast<const int4*>(row + j * (16 / EP)) : make_int4(0, 0, 0, 0);
    }
  };
  int4 v[TMAX], nx[TMAX];
  if (wave < 2 * I) load(v, wave);
  for (int64_t r = wave; r < 2 * I; r += nwaves) {
    if (r + nwaves < 2 * I) load(nx, r + nwaves);
    float acc = 0.0f;
#pragma unroll
    for (int t = 0; t < TMAX; ++t) {
      const uint32_t w[4] = {(uint32_t)v[t].x, (uint32_t)v[t].y, (uint32_t)v[t].z, (uint32_t)v[t].w};
#pragma unroll
      for (int e = 0; e < EP; ++e) {
        float x;
        if constexpr (TYPE == SPENSE_BF16)
          x = __uint_as_float(e & 1 ? (w[e >> 1] & 0xffff0000u) : (w[e >> 1] << 16));
        else
          x = __uint_as_float(w[e]);
        acc += fabsf(x) * sh[t][e];
      }
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) acc += __shfl_xor(acc, o, 64);
    if (lane == 0) out[r] = acc / (float)D;
#pragma unroll
    for (int t = 0; t < TMAX; ++t) v[t] = nx[t];
  }
}

// Column scores of Wdown (D x I), general form: a workgroup covers 64 columns; its 4
// waves each sum a quarter of the rows of every column (rows n = wave, wave + 4, ...),
// then the four partial sums are added in wave order.
template <int TYPE>
__global__ __launch_bounds__(256) void col_scores_kernel(const uint8_t* __restrict__ wd, int64_t ld_b, int64_t D,
                                                         int64_t I, const float* __restrict__ h_mid,
                                                         float* __restrict__ out) {
  __shared__ float part[4][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t i = (int64_t)blockIdx.x * 64 + lane;
  float acc = 0.0f;
  if (i < I)
    for (int64_t n = wave; n < D; n += 4) acc += fabsf(wval<TYPE>(wd + n * ld_b, i));
  part[wave][lane] = acc;
  __syncthreads();
  if (wave == 0 && i < I) {
    const float s = ((part[0][lane] + part[1][lane]) + part[2][lane]) + part[3][lane];
    out[2 * I + i] = s / (float)D * sqrtf(h_mid[i]);
  }
}

// Column scores, streaming form: a workgroup of 16 waves covers 128 columns, lane l the
// columns 2l, 2l + 1 (one 4- or 8-byte load per row); wave w sums rows w, w + 16, ... (UNR
// rows' loads in flight at a time), then the 16 partial sums of each column are added in
// wave order.  Needs I % 4 == 0 and 4-element-aligned rows.  256 columns a workgroup
// left 100 workgroups at I = 25600 (69 us for 5120 rows of bf16; 200 workgroups 48).
template <int TYPE>
__global__ __launch_bounds__(1024) void col_scores_wide_kernel(const uint8_t* __restrict__ wd, int64_t ld_b,
                                                               int64_t D, int64_t I, const float* __restrict__ h_mid,
                                                               float* __restrict__ out) {
  constexpr int UNR = 16;
  typedef typename std::conditional<TYPE == SPENSE_BF16, uint32_t, uint2>::type V;
  __shared__ float part[16][128];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t c0 = (int64_t)blockIdx.x * 128 + lane * 2;
  const bool live = c0 < I;
  const uint8_t* base = wd + c0 * (TYPE == SPENSE_BF16 ? 2 : 4);
  float acc[2] = {0.0f, 0.0f};
  auto add = [&](const V& v) __attribute__((always_inline)) {
    if constexpr (TYPE == SPENSE_BF16) {
      acc[0] += fabsf(__uint_as_float(v << 16));
      acc[1] += fabsf(__uint_as_float(v & 0xffff0000u));
    } else {
      acc[0] += fabsf(__uint_as_float(v.x));
      acc[1] += fabsf(__uint_as_float(v.y));
    }
  };
  if (live) {
    int64_t n = wave;
    for (; n + 16 * (UNR - 1) < D; n += 16 * UNR) {
      V v[UNR];
#pragma unroll
      for (int u = 0; u < UNR; ++u) v[u] = *reinterpret_cast<const V*>(base + (n + 16 * u) * ld_b);
#pragma unroll
      for (int u = 0; u < UNR; ++u) add(v[u]);
    }
    for (; n < D; n += 16) add(*reinterpret_cast<const V*>(base + n * ld_b));
  }
#pragma unroll
  for (int k = 0; k < 2; ++k) part[wave][lane * 2 + k] = acc[k];
  __syncthreads();
  if (threadIdx.x < 128) {
    const int64_t i = (int64_t)blockIdx.x * 128 + threadIdx.x;
    if (i < I) {
      float s = 0.0f;
#pragma unroll
      for (int w = 0; w < 16; ++w) s += part[w][threadIdx.x];
      out[2 * I + i] = s / (float)D * sqrtf(h_mid[i]);
    }
  }
}

// total[i] = sum over the three vectors of raw[v][i] / (mean(raw[v]) + eps); one
// workgroup, means summed in a fixed order.
__global__ __launch_bounds__(1024) void normalize_kernel(const float* __restrict__ raw, int64_t I, float eps,
                                                         float* __restrict__ total) {
  __shared__ float red[16];
  float inv[3];
  for (int v = 0; v < 3; ++v) {
    float acc = 0.0f;
    // eight loads in flight; added in index order
    int64_t i = threadIdx.x;
    for (; i + 7 * 1024 < I; i += 8 * 1024) {
      float x[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) x[u] = raw[v * I + i + 1024 * u];
#pragma unroll
      for (int u = 0; u < 8; ++u) acc += x[u];
    }
    for (; i < I; i += 1024) acc += raw[v * I + i];
    const float mean = block_sum<1024>(acc, red) / (float)I;
    inv[v] = 1.0f / (mean + eps);
  }
  for (int64_t i = threadIdx.x; i < I; i += 1024)
    total[i] = (raw[i] * inv[0] + raw[I + i] * inv[1]) + raw[2 * I + i] * inv[2];
}

// Order-preserving 32-bit key of a priority: larger priority, larger key; -0 equals +0;
// every NaN gets key 0, below every number (-inf included).
__device__ __forceinline__ uint32_t order_key(float x) {
  if (x != x) return 0u;
  const uint32_t u = x == 0.0f ? 0u : __float_as_uint(x);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Exclusive prefix count of `pred` over the 1024 threads in thread order, and the total
// (ballot per wave, wave counts through LDS).
__device__ __forceinline__ uint32_t block_prefix(bool pred, uint32_t* wcnt, uint32_t* total) {
  const uint64_t m = __ballot(pred);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint32_t below = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
  __syncthreads();  // wcnt may still be read by a previous call
  if (lane == 0) wcnt[wave] = (uint32_t)__popcll(m);
  __syncthreads();
  uint32_t before = 0, all = 0;
#pragma unroll
  for (int w = 0; w < 16; ++w) {
    const uint32_t c = wcnt[w];
    before += w < wave ? c : 0u;
    all += c;
  }
  *total = all;
  return before + below;
}

// TopK and permutation in one workgroup of 1024 threads.
// 1. Radix select, 8 bits a pass from the top: the key T of the n_dense-th largest
//    priority and the number k of indices with key T that still belong to the TopK.
// 2. One pass over the indices in 1024-index blocks: flag = key > T, or key == T among
//    the first k such indices (ties: the lower index first); the flagged indices are
//    written to the back of perm and the others to the front, each in ascending order.
__global__ __launch_bounds__(1024) void select_kernel(const float* __restrict__ t, int64_t I, int64_t n_dense,
                                                     uint8_t* __restrict__ flag, int32_t* __restrict__ perm) {
  __shared__ uint32_t hist[256];
  __shared__ uint32_t wcnt[16];
  __shared__ uint32_t sel[2];  // chosen digit, remaining count
  uint32_t prefix = 0, mask = 0;
  uint32_t k = (uint32_t)n_dense;
  if (n_dense > 0) {
    for (int shift = 24; shift >= 0; shift -= 8) {
      if (threadIdx.x < 256) hist[threadIdx.x] = 0;
      __syncthreads();
      for (int64_t i = threadIdx.x; i < I; i += 1024) {
        const uint32_t key = order_key(t[i]);
        if ((key & mask) == prefix) atomicAdd(&hist[(key >> shift) & 255u], 1u);
      }
      __syncthreads();
      if (threadIdx.x < 64) {
        // lane l holds digits 4l..4l+3; above(d) = candidates with a larger digit
        const int l = threadIdx.x;
        const uint32_t h0 = hist[4 * l], h1 = hist[4 * l + 1], h2 = hist[4 * l + 2], h3 = hist[4 * l + 3];
        const uint32_t mine = h0 + h1 + h2 + h3;
        uint32_t suf = mine;  // inclusive sum over lanes >= l
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
          const uint32_t x = __shfl_down(suf, o, 64);
          suf += l + o < 64 ? x : 0u;
        }
        uint32_t above = suf - mine;
        const uint32_t hs[4] = {h3, h2, h1, h0};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          if (above < k && k <= above + hs[q]) {
            sel[0] = (uint32_t)(4 * l + 3 - q);
            sel[1] = k - above;
          }
          above += hs[q];
        }
      }
      __syncthreads();
      prefix |= sel[0] << shift;
      mask |= 255u << shift;
      k = sel[1];
      __syncthreads();  // sel and hist are rewritten by the next pass
    }
  }
  const bool any = n_dense > 0;
  uint32_t eq_before = 0;     // indices with key T in earlier blocks
  int64_t dense_before = 0;   // flagged indices in earlier blocks
  for (int64_t b = 0; b < I; b += 1024) {
    const int64_t i = b + threadIdx.x;
    const bool in = i < I;
    const uint32_t key = in ? order_key(t[i]) : 0u;
    const bool eq = any && in && key == prefix;
    uint32_t eq_all;
    const uint32_t eq_rank = eq_before + block_prefix(eq, wcnt, &eq_all);
    const bool f = any && in && (key > prefix || (eq && eq_rank < k));
    uint32_t f_all;
    const int64_t d = dense_before + block_prefix(f, wcnt, &f_all);  // flagged indices before i
    if (in) {
      flag[i] = f ? 1 : 0;
      const int64_t pos = f ? (I - n_dense) + d : i - d;
      if (pos >= 0 && pos < I) perm[pos] = (int32_t)i;
    }
    eq_before += eq_all;
    dense_before += f_all;
  }
}

// Sum of v over the wave, in every lane.
__device__ __forceinline__ uint32_t wave_sum(uint32_t v) {
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, true);  // row_shr:1
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, true);  // row_shr:2
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, true);  // row_shr:4
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, true);  // row_shr:8: lane 15 of a row has its sum
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 15) + (uint32_t)__builtin_amdgcn_readlane((int)v, 31) +
         (uint32_t)__builtin_amdgcn_readlane((int)v, 47) + (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// The same selection with the keys in registers (I <= 1024 KPT), thread t the indices
// t KPT .. t KPT + KPT - 1.  The key of the n_dense-th largest priority bit by bit from the
// top (a bit is set if at least n_dense keys are as large with it): counts by comparison,
// with no histogram that near-equal priorities all hit in one counter.  Then one prefix
// sum over the threads places both parts, through LDS (4 I bytes) so that perm leaves in
// order.  I = 25600: radix passes over memory 65 us, 50 here.
template <int KPT>
__global__ __launch_bounds__(1024) void select_reg_kernel(const float* __restrict__ t, int64_t I, int64_t n_dense,
                                                          uint8_t* __restrict__ flag, int32_t* __restrict__ perm, int vec) {
  extern __shared__ int32_t order[];
  __shared__ uint32_t cnt[2][16];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int i0 = (int)threadIdx.x * KPT, n = (int)I;
  const int mine = min(max(n - i0, 0), KPT);  // this thread's indices
  uint32_t key[KPT];  // 0 past I: no candidate threshold is 0, so these are never counted
#pragma unroll
  for (int u = 0; u < KPT; u += 4) {
    float4 x = make_float4(__builtin_nanf(""), __builtin_nanf(""), __builtin_nanf(""), __builtin_nanf(""));
    if (vec && u + 4 <= mine) {
      x = *reinterpret_cast<const float4*>(t + i0 + u);
    } else {
      if (u < mine) x.x = t[i0 + u];
      if (u + 1 < mine) x.y = t[i0 + u + 1];
      if (u + 2 < mine) x.z = t[i0 + u + 2];
      if (u + 3 < mine) x.w = t[i0 + u + 3];
    }
    key[u] = order_key(x.x), key[u + 1] = order_key(x.y), key[u + 2] = order_key(x.z), key[u + 3] = order_key(x.w);
  }
  // sum of v over the workgroup (buffers alternate: one barrier a call)
  auto total_of = [&](uint32_t v, int b) __attribute__((always_inline)) {
    v = wave_sum(v);
    if (lane == 0) cnt[b][wave] = v;
    __syncthreads();
    uint32_t s = 0;
#pragma unroll
    for (int w = 0; w < 16; ++w) s += cnt[b][w];
    return s;
  };
  uint32_t T = 0, k = 0;  // threshold key, indices with that key that belong to the set
  if (n_dense > 0) {
    for (int bit = 31; bit >= 0; --bit) {
      const uint32_t cand = T | (1u << bit);
      uint32_t c = 0;
#pragma unroll
      for (int u = 0; u < KPT; ++u) c += key[u] >= cand ? 1u : 0u;
      if (total_of(c, bit & 1) >= (uint32_t)n_dense) T = cand;
    }
    uint32_t c = 0;
#pragma unroll
    for (int u = 0; u < KPT; ++u) c += key[u] > T ? 1u : 0u;
    k = (uint32_t)n_dense - total_of(c, 1);
    __syncthreads();
  }
  // exclusive prefix of v over the threads, in thread order
  auto prefix_of = [&](uint32_t v, int b) __attribute__((always_inline)) {
    uint32_t inc = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t x = __shfl_up(inc, o, 64);
      inc += lane >= o ? x : 0u;
    }
    if (lane == 63) cnt[b][wave] = inc;
    __syncthreads();
    uint32_t before = 0;
#pragma unroll
    for (int w = 0; w < 16; ++w) before += w < wave ? cnt[b][w] : 0u;
    return before + inc - v;
  };
  uint32_t eq = 0;
#pragma unroll
  for (int u = 0; u < KPT; ++u) eq += n_dense > 0 && u < mine && key[u] == T ? 1u : 0u;
  uint32_t eq_rank = prefix_of(eq, 0), f = 0, set = 0;
#pragma unroll
  for (int u = 0; u < KPT; ++u) {
    const bool e = n_dense > 0 && u < mine && key[u] == T;
    const bool in = n_dense > 0 && u < mine && (key[u] > T || (e && eq_rank < k));
    eq_rank += e ? 1u : 0u;
    set |= in ? 1u << u : 0u;
    f += in ? 1u : 0u;
  }
  int d = (int)prefix_of(f, 1);  // flagged indices before this thread's
#pragma unroll
  for (int u = 0; u < KPT; ++u) {
    if (u < mine) {
      const bool in = (set >> u) & 1u;
      flag[i0 + u] = in ? 1 : 0;
      const int pos = in ? n - (int)n_dense + d : i0 + u - d;
      if (pos >= 0 && pos < n) order[pos] = i0 + u;
      d += in ? 1 : 0;
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < n; i += 1024) perm[i] = order[i];
}

// dst[r] = src[perm[r]] row by row (bytes per row `cols_b`; source rows = destination
// rows, indices clamped into range), a wave per row.  vec: 16-byte pieces, up to 8 of a
// row's loads in flight before their stores; else bytes.
__global__ __launch_bounds__(256) void gather_rows_kernel(const uint8_t* __restrict__ src, int64_t ld_src_b,
                                                          uint8_t* __restrict__ dst, int64_t ld_dst_b, int64_t rows,
                                                          int64_t cols_b, const int32_t* __restrict__ perm, int vec) {
  const int lane = threadIdx.x & 63;
  const int64_t nwaves = (int64_t)gridDim.x * 4;
  for (int64_t r = ((int64_t)blockIdx.x * 256 + threadIdx.x) >> 6; r < rows; r += nwaves) {
    const int64_t pr = min(max((int64_t)perm[r], (int64_t)0), rows - 1);
    const uint8_t* s = src + pr * ld_src_b;
    uint8_t* d = dst + r * ld_dst_b;
    if (vec) {
      for (int64_t c0 = 0; c0 < cols_b; c0 += 8 * 64 * 16) {
        int4 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int64_t c = c0 + ((int64_t)u * 64 + lane) * 16;
          v[u] = c < cols_b ? *reinterpret_cast<const int4*>(s + c) : make_int4(0, 0, 0, 0);
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int64_t c = c0 + ((int64_t)u * 64 + lane) * 16;
          if (c < cols_b) *reinterpret_cast<int4*>(d + c) = v[u];
        }
      }
    } else {
      for (int64_t c = lane; c < cols_b; c += 64) d[c] = s[c];
    }
  }
}

// dst[n][c] = src[n][perm[c]] (elements of ES bytes).  tpr threads of a workgroup (a power of
// two; all 256 on wide rows) share a row; each owns GCU 4-byte pieces of V = 4 / ES consecutive
// outputs, tpr pieces apart, and keeps their sources' indices over the rows n, n + step, ...;
// neighbouring lanes write neighbouring pieces and (ascending runs of perm) read neighbouring
// sources.  xcd: all workgroups of a row on one XCD (workgroups are dealt to the 8 XCDs
// round-robin), so that a scattered perm's lines are read into one L2 and not into eight.
// vec: 4-byte stores; else element stores.
// us, 5120 x 25600, perm of two ascending runs / random: a row per workgroup and perm read again
// for each 323 / 571 (bf16), 288 / 733 (fp32), 306 / 449 (bytes); indices kept, two rows in
// flight, a row's workgroups on all XCDs 150 / 663, 238 / 1450, 96 / 221; now 149 / 478, 203 / 673,
// 84 / 203.  Two rows in flight (ROWS) of fp32 push the rows out of L2 again: 227 / 779.
constexpr int GCU = 4;
constexpr int64_t kGatherGroups = 2048;  // eight workgroups per CU
template <int ES, bool WIDE>
__global__ __launch_bounds__(256) void gather_cols_kernel(const uint8_t* __restrict__ src, int64_t ld_src_b,
                                                          uint8_t* __restrict__ dst, int64_t ld_dst_b, int64_t rows,
                                                          int64_t cols, const int32_t* __restrict__ perm, int vec, int xcd,
                                                          int tpr_narrow) {
  typedef typename std::conditional<ES == 1, uint8_t, typename std::conditional<ES == 2, uint16_t, uint32_t>::type>::type T;
  constexpr int V = 4 / ES, ROWS = ES == 4 ? 1 : 2;
  const int tpr = WIDE ? 256 : tpr_narrow;
  int64_t n = blockIdx.y, cx = blockIdx.x;
  if (xcd) {
    const uint32_t g = blockIdx.y * gridDim.x + blockIdx.x, l = g / 8;
    n = l / gridDim.x * 8 + g % 8;
    cx = l % gridDim.x;
  }
  int64_t step = gridDim.y;
  if (!WIDE) {
    n = n * (256 / tpr) + threadIdx.x / tpr;
    step *= 256 / tpr;
  }
  const int64_t c0 = (cx * GCU * tpr + threadIdx.x % tpr) * V;
  int32_t p[GCU][V];
#pragma unroll
  for (int u = 0; u < GCU; ++u)
#pragma unroll
    for (int e = 0; e < V; ++e) {
      // every index at once (those past the row again the last one's)
      p[u][e] = min(max(perm[min(c0 + (int64_t)tpr * V * u + e, cols - 1)], 0), (int32_t)(cols - 1));
    }
  T v[ROWS][GCU][V];
  auto load = [&](int r) __attribute__((always_inline)) {
    const T* const sr = reinterpret_cast<const T*>(src + (n + r * step) * ld_src_b);
#pragma unroll
    for (int u = 0; u < GCU; ++u)
#pragma unroll
      for (int e = 0; e < V; ++e) v[r][u][e] = sr[p[u][e]];
  };
  auto store = [&](int r) __attribute__((always_inline)) {
    T* const dr = reinterpret_cast<T*>(dst + (n + r * step) * ld_dst_b);
#pragma unroll
    for (int u = 0; u < GCU; ++u) {
      const int64_t c = c0 + (int64_t)tpr * V * u;
      if (vec && c + V <= cols) {
        uint32_t o = 0;
#pragma unroll
        for (int e = 0; e < V; ++e) o |= (uint32_t)v[r][u][e] << (8 * ES * e % 32);
        *reinterpret_cast<uint32_t*>(dr + c) = o;
      } else {
#pragma unroll
        for (int e = 0; e < V; ++e)
          if (c + e < cols) dr[c + e] = v[r][u][e];
      }
    }
  };
  for (; n < rows; n += ROWS * step) {
    load(0);
    if (ROWS == 2 && n + step < rows) {
      load(1);
      store(0);
      store(1);
    } else {
      store(0);
    }
  }
}

}  // namespace

namespace {
int grid_for(int64_t waves) {  // workgroups of 4 waves, at most 8 per CU's worth
  const int64_t g = (waves + 3) / 4;
  return (int)(g < 2048 ? (g < 1 ? 1 : g) : 2048);
}

template <int TYPE>
void launch_row_scores(dim3 grid, hipStream_t st, const uint8_t* g, const uint8_t* u, int64_t ld_b, int64_t D, int T,
                       const float* h_in, float* raw, int64_t I) {
  if (T <= 4)
    hipLaunchKernelGGL((row_scores_wave_kernel<TYPE, 4>), grid, dim3(256), 0, st, g, u, ld_b, D, T, h_in, raw, I);
  else if (T <= 10)
    hipLaunchKernelGGL((row_scores_wave_kernel<TYPE, 10>), grid, dim3(256), 0, st, g, u, ld_b, D, T, h_in, raw, I);
  else
    hipLaunchKernelGGL((row_scores_wave_kernel<TYPE, 16>), grid, dim3(256), 0, st, g, u, ld_b, D, T, h_in, raw, I);
}
}  // namespace

hipError_t launch_index_scores(int type, const void* wg, const void* wu, int64_t ld_gu_b, int64_t I, int64_t D,
                               const void* wd, int64_t ld_d_b, const float* h_in, const float* h_mid, float eps,
                               float* raw, float* total, hipStream_t st) {
  const uint8_t* g = static_cast<const uint8_t*>(wg);
  const uint8_t* u = static_cast<const uint8_t*>(wu);
  const uint8_t* d = static_cast<const uint8_t*>(wd);
  const int64_t es = type == SPENSE_BF16 ? 2 : 4, ep = 16 / es;
  const int64_t T = (D + 64 * ep - 1) / (64 * ep);
  const bool row_vec = D % ep == 0 && ld_gu_b % 16 == 0 && (uintptr_t)g % 16 == 0 && (uintptr_t)u % 16 == 0 && T <= 16;
  const bool col_vec = I % 4 == 0 && ld_d_b % (4 * es) == 0 && (uintptr_t)d % (4 * es) == 0;
  const dim3 rg((unsigned)I, 2), cg((unsigned)((I + 63) / 64));
  const unsigned gw = (unsigned)grid_for(2 * I);
  const dim3 wg_grid(gw < 512 ? gw : 512);  // two workgroups per CU: the registers of two rows in flight
  const dim3 cwg((unsigned)((I + 127) / 128));
  if (type == SPENSE_BF16) {
    if (row_vec)
      launch_row_scores<SPENSE_BF16>(wg_grid, st, g, u, ld_gu_b, D, (int)T, h_in, raw, I);
    else
      hipLaunchKernelGGL(row_scores_kernel<SPENSE_BF16>, rg, dim3(256), 0, st, g, u, ld_gu_b, D, h_in, raw, I);
    if (col_vec)
      hipLaunchKernelGGL(col_scores_wide_kernel<SPENSE_BF16>, cwg, dim3(1024), 0, st, d, ld_d_b, D, I, h_mid, raw);
    else
      hipLaunchKernelGGL(col_scores_kernel<SPENSE_BF16>, cg, dim3(256), 0, st, d, ld_d_b, D, I, h_mid, raw);
  } else {
    if (row_vec)
      launch_row_scores<SPENSE_F32>(wg_grid, st, g, u, ld_gu_b, D, (int)T, h_in, raw, I);
    else
      hipLaunchKernelGGL(row_scores_kernel<SPENSE_F32>, rg, dim3(256), 0, st, g, u, ld_gu_b, D, h_in, raw, I);
    if (col_vec)
      hipLaunchKernelGGL(col_scores_wide_kernel<SPENSE_F32>, cwg, dim3(1024), 0, st, d, ld_d_b, D, I, h_mid, raw);
    else
      hipLaunchKernelGGL(col_scores_kernel<SPENSE_F32>, cg, dim3(256), 0, st, d, ld_d_b, D, I, h_mid, raw);
  }
  hipLaunchKernelGGL(normalize_kernel, dim3(1), dim3(1024), 0, st, raw, I, eps, total);
  return hipGetLastError();
}

namespace {
// select_reg_kernel of up to IMAX indices: 4 I bytes of LDS, above the default limit (64 KB, with
// the counters) by a per-device attribute that is set once.
template <int KPT, int IMAX>
hipError_t launch_select_reg(const float* total, int64_t I, int64_t n_dense, uint8_t* flag, int32_t* perm, hipStream_t st) {
  static_assert(IMAX <= 1024 * KPT, "keys of a workgroup");
  if (IMAX > 1024 * 15) {
    static std::once_flag once[64];
    static hipError_t rc[64];
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    std::call_once(once[dev], [&] {
      rc[dev] = hipFuncSetAttribute(reinterpret_cast<const void*>(select_reg_kernel<KPT>),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, IMAX * 4);
    });
    if (rc[dev] != hipSuccess) return rc[dev];
  }
  hipLaunchKernelGGL(select_reg_kernel<KPT>, dim3(1), dim3(1024), (size_t)I * 4, st, total, I, n_dense, flag, perm,
                     (uintptr_t)total % 16 == 0 ? 1 : 0);
  return hipGetLastError();
}
}  // namespace

hipError_t launch_dense_permutation(const float* total, int64_t I, int64_t n_dense, uint8_t* flag, int32_t* perm,
                                    hipStream_t st) {
  // In registers where that is faster for any distribution of the priorities; its 32 counts have a
  // barrier each, so the radix passes win on few indices and, like the counts of KPT keys a thread
  // where many are padding, cost more as I grows.  us, radix passes (priorities uniform in [0, 1) /
  // normal around 3 with deviation 0.3) and registers: I = 1024 6.5 / 7.0 and 23.5, 4096 12.3 /
  // 13.9 and 23.8, 8192 20.9 / 24.2 and 24.7, 10240 25.0 / 29.2 and 25.8, 12288 29.1 / 34.1 and
  // 26.6, 16384 37.0 / 43.7 and 32.2 (KPT 24; 41.4 with 32), 25600 55.1 / 65.4 and 48.9.
  if (I <= 10240 || I > 1024 * 32) {
    hipLaunchKernelGGL(select_kernel, dim3(1), dim3(1024), 0, st, total, I, n_dense, flag, perm);
    return hipGetLastError();
  }
  if (I <= 1024 * 15) return launch_select_reg<16, 1024 * 15>(total, I, n_dense, flag, perm, st);
  if (I <= 1024 * 24) return launch_select_reg<24, 1024 * 24>(total, I, n_dense, flag, perm, st);
  return launch_select_reg<32, 1024 * 32>(total, I, n_dense, flag, perm, st);
}

hipError_t launch_gather_rows(const void* src, int64_t ld_src_b, void* dst, int64_t ld_dst_b, int64_t rows,
                              int64_t cols_b, const int32_t* perm, hipStream_t st) {
  const int vec = ((uintptr_t)src % 16 == 0) && ((uintptr_t)dst % 16 == 0) && ld_src_b % 16 == 0 &&
                  ld_dst_b % 16 == 0 && cols_b % 16 == 0;
  hipLaunchKernelGGL(gather_rows_kernel, dim3((unsigned)grid_for(rows)), dim3(256), 0, st,
                     static_cast<const uint8_t*>(src), ld_src_b, static_cast<uint8_t*>(dst), ld_dst_b, rows, cols_b,
                     perm, vec);
  return hipGetLastError();
}

hipError_t launch_gather_cols(int es, const void* src, int64_t ld_src_b, void* dst, int64_t ld_dst_b, int64_t rows,
                              int64_t cols, const int32_t* perm, hipStream_t st) {
  const uint8_t* s = static_cast<const uint8_t*>(src);
  uint8_t* d = static_cast<uint8_t*>(dst);
  const int64_t pieces = (cols * es + 3) / 4;
  int tpr = 1;
  while (tpr < 256 && (int64_t)tpr * GCU < pieces) tpr *= 2;
  const int vec = (uintptr_t)d % 4 == 0 && ld_dst_b % 4 == 0;
  const int64_t gx = (pieces + tpr * GCU - 1) / (tpr * GCU), groups = (rows + 256 / tpr - 1) / (256 / tpr);
  // each workgroup keeps its indices over many rows
  int64_t gy = std::min(groups, std::max<int64_t>(1, kGatherGroups / gx));
  const int xcd = gx > 1 && gy >= 8;
  if (xcd) gy = gy / 8 * 8;
  const dim3 grid((unsigned)gx, (unsigned)gy);
  auto launch = [&](auto k) {
    hipLaunchKernelGGL(k, grid, dim3(256), 0, st, s, ld_src_b, d, ld_dst_b, rows, cols, perm, vec, xcd, tpr);
  };
  const bool wide = tpr == 256;
  if (es == 1)
    wide ? launch(gather_cols_kernel<1, true>) : launch(gather_cols_kernel<1, false>);
  else if (es == 2)
    wide ? launch(gather_cols_kernel<2, true>) : launch(gather_cols_kernel<2, false>);
  else
    wide ? launch(gather_cols_kernel<4, true>) : launch(gather_cols_kernel<4, false>);
  return hipGetLastError();
}

}  // namespace spense
