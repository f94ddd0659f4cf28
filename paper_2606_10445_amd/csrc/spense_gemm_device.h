// Device helpers shared by the GEMM translation units: buffer loads, matrix instructions,
// barriers, the epilogue.
#pragma once
#include <mutex>
#include <utility>

#include "spense_internal.h"

namespace spense {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef __bf16 v16bf __attribute__((ext_vector_type(16)));

constexpr uint32_t kOOB = 0x80000000u;  // any offset past every buffer extent
// Cache policy of the weight loads.  Measured on MI355X: for rows read as 16 x 64-byte
// segments per instruction the default policy streams ~15% faster than non-temporal;
// for the tiled layout (1 KB contiguous per instruction) non-temporal is 5-9% faster.
constexpr int kNT = 0;
constexpr int kTiledNT = 2;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes, 0x00020000);
}
// voffset: per-lane byte offset; soffset: wave-uniform byte offset (scalar register)
template <int AUX>
__device__ __forceinline__ v4i bl16(__amdgpu_buffer_rsrc_t r, uint32_t off, int soff = 0) {
  return __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, soff, AUX));
}
template <int AUX>
__device__ __forceinline__ int bl4(__amdgpu_buffer_rsrc_t r, uint32_t off, int soff = 0) {
  return (int)__builtin_amdgcn_raw_buffer_load_b32(r, (int)off, soff, AUX);
}
__device__ __forceinline__ v8i cat8(v4i a, v4i b) { return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7); }
__device__ __forceinline__ uint32_t sel(bool ok, uint32_t off) { return ok ? off : kOOB; }

// Matrix-core results are written several cycles after the instruction issues (up to
// about a dozen wait states for the 8-pass fp8 instruction), and the hardware does not
// interlock a later non-matrix read (or a matrix read of a different register) against
// that write.  Where such a read sits in another basic block than the producing matrix
// instruction (loop exits, the 2:4 -> dense switch, the epilogue), the compiler's own
// padding was measured to fall short on gfx950, so these points get 20 explicit wait
// states.  The scheduling barriers keep instructions from moving across them.
__device__ __forceinline__ void xdl_fence() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 3" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

template <int DT>
struct Traits;
template <>
struct Traits<kFP8> {
  static constexpr int KS = 128;  // logical K per sparse instruction
  static constexpr int KD = 128;  // K per dense instruction
  static constexpr int ES = 1;
};
template <>
struct Traits<kBF16> {
  static constexpr int KS = 64;
  static constexpr int KD = 32;
  static constexpr int ES = 2;
};

__device__ __forceinline__ v4f mma_sparse(v4i a, v8i b, v4f c, int idx, std::integral_constant<int, kFP8>) {
  return __builtin_amdgcn_smfmac_f32_16x16x128_fp8_fp8(a, b, c, idx, 0, 0);
}
__device__ __forceinline__ v4f mma_sparse(v4i a, v8i b, v4f c, int idx, std::integral_constant<int, kBF16>) {
  return __builtin_amdgcn_smfmac_f32_16x16x64_bf16(__builtin_bit_cast(v8bf, a), __builtin_bit_cast(v16bf, b), c,
                                                   idx, 0, 0);
}
__device__ __forceinline__ v4f mma_dense(v8i a, v8i b, v4f c, std::integral_constant<int, kFP8>) {
  // fp8 e4m3 for both operands (format selectors 0), no block scales
  return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a, b, c, 0, 0, 0, 0, 0, 0);
}
__device__ __forceinline__ v4f mma_dense(v8i a, v8i b, v4f c, std::integral_constant<int, kBF16>) {
  const v4i a4 = {a[0], a[1], a[2], a[3]}, b4 = {b[0], b[1], b[2], b[3]};
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, a4), __builtin_bit_cast(v8bf, b4), c, 0,
                                                 0, 0);
}

// ---------------------------------------------------------------- epilogue
__device__ __forceinline__ uint32_t bf16_bits(float v) {
  __bf16 h = (__bf16)v;  // round to nearest even
  return (uint32_t)__builtin_bit_cast(uint16_t, h);
}

// Epilogue of 4 consecutive output rows n0.. of token m: (acc * w_scale[n]) * x_scale[m],
// bf16 (round to nearest even) or fp32, one vector store where allowed.
// Y[m, n0 + r] = v[r] for r < 4 (rows before rowend), bf16 RNE or fp32 per a.out_f32.
__device__ __forceinline__ void put4(void* Y, int64_t ldy, int vec_store, const GemmArgs& a, const float (&v)[4], int m,
                                     int n0, int rowend) {
  if (a.out_f32) {
    float* yp = reinterpret_cast<float*>(Y) + (int64_t)m * ldy + n0;
    if (vec_store && n0 + 3 < rowend) {
      *reinterpret_cast<v4f*>(yp) = (v4f){v[0], v[1], v[2], v[3]};
    } else {
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (n0 + r < rowend) yp[r] = v[r];
    }
  } else {
    uint16_t* yp = reinterpret_cast<uint16_t*>(Y) + (int64_t)m * ldy + n0;
    const uint32_t b0 = bf16_bits(v[0]), b1 = bf16_bits(v[1]), b2 = bf16_bits(v[2]), b3 = bf16_bits(v[3]);
    if (vec_store && n0 + 3 < rowend) {
      typedef uint32_t u2 __attribute__((ext_vector_type(2)));
      *reinterpret_cast<u2*>(yp) = (u2){b0 | (b1 << 16), b2 | (b3 << 16)};
    } else {
      const uint32_t bb[4] = {b0, b1, b2, b3};
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (n0 + r < rowend) yp[r] = (uint16_t)bb[r];
    }
  }
}

// The epilogue of one output quad: Y[m, n0 + r] = (acc[r] * w_scale[n]) * x_scale[m]
// (each factor only where given), fp32, then put4.
__device__ __forceinline__ void store4(void* Y, int64_t ldy, const float* sw, int vec_store, const GemmArgs& a,
                                       v4f acc, int m, int n0, int rowend) {
  const float xs = a.sx ? a.sx[m] : 1.0f;
  float v[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int n = n0 + r < rowend ? n0 + r : rowend - 1;
    float y = acc[r];
    if (sw) y = y * sw[n];
    v[r] = y * xs;
  }
  put4(Y, ldy, vec_store, a, v, m, n0, rowend);
}

// The scales of one wave's RT x CT output quads (rows n0 + 16 t + [0, 4), token m0 +
// 16 c), loaded together before any output store: read next to each store, a scale load
// would follow stores that may alias it and wait for their acknowledgement, one memory
// round trip per quad.  Rows past the region and tokens past M read the last valid one
// (their stores are skipped); a missing scale reads as 1.
template <int RT, int CT>
struct EpiScales {
  float w[RT][4];
  float x[CT];
};

template <int RT, int CT>
__device__ __forceinline__ void epi_scales(EpiScales<RT, CT>& e, const float* sw, const float* sx, int M, int n0, int m0,
                                           int rowend) {
#pragma unroll
  for (int t = 0; t < RT; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) e.w[t][r] = sw ? sw[min(n0 + 16 * t + r, rowend - 1)] : 1.0f;
#pragma unroll
  for (int c = 0; c < CT; ++c) e.x[c] = sx ? sx[min(m0 + 16 * c, M - 1)] : 1.0f;
}

// store4 of quad (t, c) with its scales from epi_scales: the same arithmetic, bit for bit.
template <int RT, int CT>
__device__ __forceinline__ void store4e(void* Y, int64_t ldy, bool wscaled, int vec_store, const GemmArgs& a,
                                        const EpiScales<RT, CT>& e, int t, int c, v4f acc, int m, int n0, int rowend) {
  float v[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    float y = acc[r];
    if (wscaled) y = y * e.w[t][r];
    v[r] = y * e.x[c];
  }
  put4(Y, ldy, vec_store, a, v, m, n0, rowend);
}

__device__ __forceinline__ void store4(const GemmArgs& a, v4f acc, int m, int n0, int rowend) {
  store4(a.Y, a.ldy, a.sw, a.vec_store, a, acc, m, n0, rowend);
}

// A large-M workgroup's bf16 output tile through LDS, so that it leaves as whole token
// rows: stored straight from the accumulators, each instruction would write 16 token rows
// 32 bytes apiece, four times the write requests of whole rows (measured on the 256 x 256
// kernel: about 9 us of store issue per tile against 2).  Token row r of the tile (NB
// 16-byte blocks of eight outputs) sits at byte r * 16 NB, its block b stored at block
// b ^ (r % NB), so that neither the quad writes nor the row reads meet in a bank.
// out_tile_write: a wave's RT x CT quads (rows 16 (RT wr + t) + 4 lq + [0, 4) of the tile,
// token 16 (CT wc + c) + li), scaled and rounded as store4e does.
template <int RT, int CT, int NB>
__device__ __forceinline__ void out_tile_write(uint8_t* ot, const v4f (&acc)[RT][CT], const EpiScales<RT, CT>& es,
                                               bool wscaled, int wr, int wc, int li, int lq) {
  typedef uint32_t u2 __attribute__((ext_vector_type(2)));
#pragma unroll
  for (int t = 0; t < RT; ++t)
#pragma unroll
    for (int c = 0; c < CT; ++c) {
      float v[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float y = acc[t][c][r];
        if (wscaled) y = y * es.w[t][r];
        v[r] = y * es.x[c];
      }
      const int r = 16 * (CT * wc + c) + li, n = 16 * (RT * wr + t) + 4 * lq;
      *reinterpret_cast<u2*>(ot + r * (16 * NB) + (((n >> 3) ^ (r % NB)) << 4) + (n & 7) * 2) =
          (u2){bf16_bits(v[0]) | (bf16_bits(v[1]) << 16), bf16_bits(v[2]) | (bf16_bits(v[3]) << 16)};
    }
}

// out_tile_store: the tile's first ntok token rows to Y (tile row 0 = output row rblk,
// token 0 = m0), 16 bytes per thread; Y 16-byte aligned, ldy and rblk multiples of 8.
template <int NB, int NTHR>
__device__ __forceinline__ void out_tile_store(const uint8_t* ot, int ntok, int m0, int M, int rblk, int rowend, void* Y,
                                               int64_t ldy) {
  for (int q = threadIdx.x; q < ntok * NB; q += NTHR) {
    const int r = q / NB, b = q % NB;
    const int m = m0 + r, n = rblk + 8 * b;
    if (m >= M || n >= rowend) continue;
    const v4i d = *reinterpret_cast<const v4i*>(ot + r * (16 * NB) + ((b ^ (r % NB)) << 4));
    uint16_t* yp = reinterpret_cast<uint16_t*>(Y) + (int64_t)m * ldy + n;
    if (n + 8 <= rowend) {
      *reinterpret_cast<v4i*>(yp) = d;
    } else {
      for (int e = 0; e < rowend - n; ++e) yp[e] = (uint16_t)((uint32_t)d[e >> 1] >> (16 * (e & 1)));
    }
  }
}

// Workgroup barrier that first waits until at most N of this wave's vector-memory
// operations are outstanding (loads complete in issue order, so every older one is
// done).  The wait is the builtin, which the compiler's own wait insertion takes into
// account; the barrier's memory clobber keeps LDS accesses from moving across it.
template <int N>
__device__ __forceinline__ void barrier_vm() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  // s_waitcnt fields: vmcnt[3:0] and [15:14], expcnt [6:4] and lgkmcnt [11:8] left at max
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
  asm volatile("s_barrier" ::: "memory");
}

// Wait until at most N of this wave's vector-memory operations are outstanding.
template <int N>
__device__ __forceinline__ void wait_vm() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

// Workgroup barrier after this wave's LDS accesses; vector-memory operations stay in flight.
__device__ __forceinline__ void barrier_lgkm0() {
  __builtin_amdgcn_s_waitcnt(15 | (3 << 14) | (7 << 4) | (0 << 8));
  asm volatile("s_barrier" ::: "memory");
}

// As barrier_vm, and also wait for this wave's LDS accesses (lgkmcnt(0)).
template <int N>
__device__ __forceinline__ void barrier_vm_lgkm0() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (0 << 8));
  asm volatile("s_barrier" ::: "memory");
}

template <typename F, int... I>
__device__ __forceinline__ void static_for_impl(F& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>()), ...);
}
// f(integral_constant<int, i>) for i = 0 .. N-1, each index a compile-time constant.
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_impl(f, std::make_integer_sequence<int, N>());
}

template <int AUX>
__device__ __forceinline__ void lds_load4(__amdgpu_buffer_rsrc_t r, uint8_t* dst, uint32_t voff, int soff) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)dst, 4, voff, soff, 0, AUX);
}
template <int AUX>
__device__ __forceinline__ void lds_load16(__amdgpu_buffer_rsrc_t r, uint8_t* dst, uint32_t voff, int soff) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)dst, 16, voff, soff, 0, AUX);
}

// The large-M kernels' dynamic LDS above the default limit is a per-device function
// attribute: set once per (device, kernel instance), under std::call_once, so that host
// threads making their first large-M call together do not race.
constexpr int kMaxDevices = 64;
std::once_flag g_big_lds_once[kMaxDevices][2][5];  // [device][tiled][kernel instance]
hipError_t g_big_lds_rc[kMaxDevices][2][5];

template <typename KernelT>
hipError_t set_big_lds(KernelT k, int tiled, int which, int lds) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::call_once(g_big_lds_once[dev][tiled][which], [&] {
    g_big_lds_rc[dev][tiled][which] =
        hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  });
  return g_big_lds_rc[dev][tiled][which];
}

}  // namespace
}  // namespace spense
