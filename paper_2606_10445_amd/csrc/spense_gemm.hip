// Fused Spense GEMM for gfx950: Y = X W^T with W in the hybrid 2:4 / dense format
// (paper sec. 3.2), one kernel launch for both regions.
//
//   - 2:4 region: v_smfmac_f32_16x16x128_fp8_fp8 / v_smfmac_f32_16x16x64_bf16, the
//     compressed weight as the sparse A operand, one metadata word as the index register
//     (sec. 3.1.1: kept values + 2-bit positions);
//   - dense region: v_mfma_f32_16x16x128_f8f6f4 / v_mfma_f32_16x16x32_bf16;
//   - output-split: a workgroup lies in one region, so the regions write disjoint output
//     columns; input-split: a wave's fp32 accumulator runs over its 2:4 columns and then
//     its dense columns, with no rounding between the two partial products;
//   - epilogue: y = (acc * w_scale[n]) * x_scale[m], rounded to bf16 (or kept fp32).
//
// Operand layouts (measured on gfx950 with one-hot and random-integer probes):
//   A row = lane % 16 for all four instructions; D[lane][r] = (row 4*(lane/16) + r,
//   column lane % 16).  Dense: lane group q = lane/16 holds K [32q, 32q+32) (fp8) or
//   [8q, 8q+8) (bf16) of both A and B.  Any permutation of K applied to both operands
//   gives the same dot products, so the dense fp8 step feeds lane group q the K range
//   [16q, 16q+16) in bytes 0..15 and [64+16q, 64+16q+16) in bytes 16..31 (the sparse B
//   order): each 16-byte load instruction then covers 64 contiguous bytes of a row.  Sparse fp8: lane group q holds the 16 kept values
//   of logical K [32q, 32q+32) with their 2-bit positions in bits [2c, 2c+2) of the
//   index register, i.e. exactly one canonical metadata word; B holds K [16q, 16q+16) in
//   bytes 0..15 and [64+16q, 64+16q+16) in bytes 16..31.  Sparse bf16: lane group q
//   holds logical K [16q, 16q+16) (half a metadata word, chosen by shifting); B holds K
//   [8q, 8q+8) and [32+8q, 32+8q+8).
//
// Six GEMM kernels; the host planner picks one per call from M and the weight geometry:
//   - spense_gemm_rows_kernel (decode, HBM-bound): each wave owns 16 weight rows over all
//     of K; the waves of a workgroup share every chunk of activations through LDS (or
//     keep all of them resident) and keep two chunks of weights in flight; K slices, where
//     the weight has few rows, go through splitk_reduce_kernel;
//   - spense_gemm_rows2_kernel (tiled fp8, 65-768 tokens): the same with two 64-token halves
//     per workgroup, each weight chunk feeding both;
//   - spense_gemm_kernel: a workgroup owns 16*RT weight rows and its W waves split the K
//     range (cost-balanced on the host), U instruction steps per batch of loads; at the
//     end the waves add their accumulators in LDS in wave order (deterministic);
//   - spense_gemm_mid_kernel (spense_gemm_mid.hip; tiled fp8, row-major bf16): 128 x 128
//     workgroup tiles, optionally of a K slice, with waves that only copy;
//   - spense_gemm_big_kernel (fp8) / spense_gemm_big2_kernel (spense_gemm_big2.hip; tiled fp8,
//     row-major bf16): many tokens, 128 x 256 and 256 x 256 (192, 128) workgroup tiles.
// The last three copy both operands into LDS a few steps ahead, and their bf16 output tile
// leaves through LDS as whole token rows.
// All loads are range-checked buffer loads: a lane whose chunk lies past the end of its
// range gets an out-of-range offset and reads zeros, so the loops have no divergent
// branches.
#include "spense_gemm_device.h"

namespace spense {
namespace {

// ---------------------------------------------------------------- pipeline stages
// One stage = U instruction steps of one wave.  Offsets are byte offsets into the
// buffers; masked lanes use kOOB and read zeros.
template <int DT, int CT, int RT, int U>
struct SparseStage {
  v4i a[U][RT];
  int ix[U][RT];
  v8i b[U][CT];
};
template <int DT, int CT, int RT, int U>
struct DenseStage {
  v8i a[U][RT];
  v8i b[U][CT];
};

struct LaneCtx {
  __amdgpu_buffer_rsrc_t rx, rv, rm, rd;
  int lq;
};

// FULL: every step of the stage lies inside [k, kend): no per-lane masks, the step's K
// offset travels in the scalar offset.  Otherwise lanes past kend read zeros.
template <int DT, int CT, int RT, int U, bool WM, bool FULL>
__device__ __forceinline__ void load_sparse(SparseStage<DT, CT, RT, U>& st, const LaneCtx& L, const uint32_t (&vrow)[RT],
                                            const uint32_t (&mrow)[RT], const uint32_t (&xrow)[CT],
                                            const bool (&xok)[CT], int k, int kend) {
  const int lq = L.lq;
#pragma unroll
  for (int j = 0; j < U; ++j) {
    const int kk = k + j * Traits<DT>::KS;
    if constexpr (DT == kFP8 && FULL) {
#pragma unroll
      for (int t = 0; t < RT; ++t) {
        st.a[j][t] = bl16<kNT>(L.rv, vrow[t], kk >> 1);
        if constexpr (!WM) st.ix[j][t] = bl4<kNT>(L.rm, mrow[t], 4 * (kk >> 5));
      }
#pragma unroll
      for (int c = 0; c < CT; ++c) {
        const uint32_t o = xok[c] ? xrow[c] : kOOB;
        st.b[j][c] = cat8(bl16<0>(L.rx, o, kk), bl16<0>(L.rx, o, kk + 64));
      }
    } else if constexpr (DT == kFP8) {
      const bool oka = kk + 32 * lq < kend;  // this lane group's 32 logical K
#pragma unroll
      for (int t = 0; t < RT; ++t) {
        st.a[j][t] = bl16<kNT>(L.rv, sel(oka, vrow[t] + (kk >> 1)));
        if constexpr (!WM) st.ix[j][t] = bl4<kNT>(L.rm, sel(oka, mrow[t] + 4 * (kk >> 5)));
      }
      const bool ok0 = kk + 16 * lq < kend, ok1 = kk + 64 + 16 * lq < kend;
#pragma unroll
      for (int c = 0; c < CT; ++c) {
        const v4i p0 = bl16<0>(L.rx, sel(ok0 && xok[c], xrow[c] + kk));
        const v4i p1 = bl16<0>(L.rx, sel(ok1 && xok[c], xrow[c] + kk + 64));
        st.b[j][c] = cat8(p0, p1);
      }
    } else {
      const bool oka = kk + 16 * lq < kend;
#pragma unroll
      for (int t = 0; t < RT; ++t) {
        st.a[j][t] = bl16<kNT>(L.rv, sel(oka, vrow[t] + kk));
        st.ix[j][t] = (int)((uint32_t)bl4<kNT>(L.rm, sel(oka, mrow[t] + 4 * (kk >> 5))) >> (16 * (lq & 1)));
      }
      const bool ok0 = kk + 8 * lq < kend, ok1 = kk + 32 + 8 * lq < kend;
#pragma unroll
      for (int c = 0; c < CT; ++c) {
        const v4i p0 = bl16<0>(L.rx, sel(ok0 && xok[c], xrow[c] + 2 * kk));
        const v4i p1 = bl16<0>(L.rx, sel(ok1 && xok[c], xrow[c] + 2 * (kk + 32)));
        st.b[j][c] = cat8(p0, p1);
      }
    }
  }
  if constexpr (WM) {
    static_assert(DT == kFP8 && U % 4 == 0, "wide metadata loads cover four fp8 steps");
    // Metadata for four steps at once: lane group q loads the 16 bytes holding words
    // 4q..4q+3 of those steps' 16 words (one line segment per row), then a 4x4 transpose
    // across lane groups hands step j's word 4j+q to lane group q.  Words of steps past
    // kend only meet zeroed A and B operands.
#pragma unroll
    for (int j0 = 0; j0 < U; j0 += 4) {
      const int kk = k + j0 * Traits<DT>::KS;
#pragma unroll
      for (int t = 0; t < RT; ++t) {
        const v4i w = FULL ? bl16<kNT>(L.rm, mrow[t] + 12 * lq, 4 * (kk >> 5))
                           : bl16<kNT>(L.rm, sel(kk + 128 * lq < kend, mrow[t] + 4 * (kk >> 5) + 12 * lq));
        const auto s02 = __builtin_amdgcn_permlane32_swap((unsigned)w[0], (unsigned)w[2], false, false);
        const auto s13 = __builtin_amdgcn_permlane32_swap((unsigned)w[1], (unsigned)w[3], false, false);
        const auto s01 = __builtin_amdgcn_permlane16_swap(s02[0], s13[0], false, false);
        const auto s23 = __builtin_amdgcn_permlane16_swap(s02[1], s13[1], false, false);
        st.ix[j0 + 0][t] = (int)s01[0];
        st.ix[j0 + 1][t] = (int)s01[1];
        st.ix[j0 + 2][t] = (int)s23[0];
        st.ix[j0 + 3][t] = (int)s23[1];
      }
    }
  }
}

template <int DT, int CT, int RT, int U, bool FULL>
__device__ __forceinline__ void load_dense(DenseStage<DT, CT, RT, U>& st, const LaneCtx& L, const uint32_t (&drow)[RT],
                                           const uint32_t (&xrow)[CT], const bool (&xok)[CT], int k, int kend,
                                           int dco) {
  const int lq = L.lq;
  const v4i z = {0, 0, 0, 0};
#pragma unroll
  for (int j = 0; j < U; ++j) {
    const int kk = k + j * Traits<DT>::KD;
    if constexpr (DT == kFP8 && FULL) {
#pragma unroll
      for (int t = 0; t < RT; ++t) st.a[j][t] = cat8(bl16<kNT>(L.rd, drow[t], kk - dco), bl16<kNT>(L.rd, drow[t], kk - dco + 64));
#pragma unroll
      for (int c = 0; c < CT; ++c) {
        const uint32_t o = xok[c] ? xrow[c] : kOOB;
        st.b[j][c] = cat8(bl16<0>(L.rx, o, kk), bl16<0>(L.rx, o, kk + 64));
      }
    } else if constexpr (DT == kFP8) {
      const bool ok0 = kk + 16 * lq < kend, ok1 = kk + 64 + 16 * lq < kend;
#pragma unroll
      for (int t = 0; t < RT; ++t) {
        const uint32_t o = drow[t] + (uint32_t)(kk - dco);
        st.a[j][t] = cat8(bl16<kNT>(L.rd, sel(ok0, o)), bl16<kNT>(L.rd, sel(ok1, o + 64)));
      }
#pragma unroll
      for (int c = 0; c < CT; ++c) {
        const uint32_t o = xrow[c] + kk;
        st.b[j][c] = cat8(bl16<0>(L.rx, sel(ok0 && xok[c], o)), bl16<0>(L.rx, sel(ok1 && xok[c], o + 64)));
      }
    } else {
      const bool ok = kk + 8 * lq < kend;
#pragma unroll
      for (int t = 0; t < RT; ++t) st.a[j][t] = cat8(bl16<kNT>(L.rd, sel(ok, drow[t] + 2 * (uint32_t)(kk - dco))), z);
#pragma unroll
      for (int c = 0; c < CT; ++c) st.b[j][c] = cat8(bl16<0>(L.rx, sel(ok && xok[c], xrow[c] + 2 * kk)), z);
    }
  }
}

template <int DT, int CT, int RT, int U>
__device__ __forceinline__ void mma_stage(v4f (&acc)[RT][CT], const SparseStage<DT, CT, RT, U>& st) {
#pragma unroll
  for (int j = 0; j < U; ++j)
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int c = 0; c < CT; ++c)
        acc[t][c] = mma_sparse(st.a[j][t], st.b[j][c], acc[t][c], st.ix[j][t], std::integral_constant<int, DT>());
}
template <int DT, int CT, int RT, int U>
__device__ __forceinline__ void mma_stage(v4f (&acc)[RT][CT], const DenseStage<DT, CT, RT, U>& st) {
#pragma unroll
  for (int j = 0; j < U; ++j)
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int c = 0; c < CT; ++c)
        acc[t][c] = mma_dense(st.a[j][t], st.b[j][c], acc[t][c], std::integral_constant<int, DT>());
}

// One stage at a time: issue all loads of U steps, then feed the matrix cores.  Latency
// is hidden by the many resident waves rather than by register double buffering, which
// measured slower on MI355X for this access pattern.  Whole stages run unmasked with
// wave-uniform offsets; the last, partial stage masks lanes past kend.
template <typename Stage, typename LoadFull, typename LoadTail, int RT, int CT>
__device__ __forceinline__ void run_stages(v4f (&acc)[RT][CT], int k0, int kend, int step, LoadFull full,
                                           LoadTail tail) {
  int k = k0;
  for (; k + step <= kend; k += step) {
    Stage st;
    full(st, k);
    mma_stage(acc, st);
  }
  if (k < kend) {
    Stage st;
    tail(st, k);
    xdl_fence();
    mma_stage(acc, st);
  }
  xdl_fence();
}

// ---------------------------------------------------------------- kernel
template <int DT, int CT, int RT, int W, int U, bool WM>
__global__ __launch_bounds__(64 * W) void spense_gemm_kernel(GemmArgs a) {
  typedef Traits<DT> T;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int li = lane & 15, lq = lane >> 4;
  const int g = blockIdx.x, mb = blockIdx.y;
  const int ri = (a.nreg > 1 && g >= a.reg[1].wg0) ? 1 : 0;
  const Region& R = a.reg[ri];
  const int nbase = R.row0 + (g - R.wg0) * 16 * RT;
  const int rowend = R.row0 + R.rows;
  const int m0 = mb * 16 * CT;
  const int ka = R.cut[wave], kb = R.cut[wave + 1];
  const int ks_end = min(kb, R.kbound);  // 2:4 columns of this wave: [ka, ks_end)
  const int kd_beg = max(ka, R.kbound);  // dense columns of this wave: [kd_beg, kb)

  LaneCtx L;
  L.lq = lq;
  L.rx = rsrc(a.X, a.x_bytes);
  L.rv = rsrc(a.values, a.v_bytes);
  L.rm = rsrc(a.meta, a.m_bytes);
  L.rd = rsrc(a.dense, a.d_bytes);

  v4f acc[RT][CT];
#pragma unroll
  for (int t = 0; t < RT; ++t)
#pragma unroll
    for (int c = 0; c < CT; ++c) acc[t][c] = (v4f){0.f, 0.f, 0.f, 0.f};

  uint32_t xrow[CT];
  bool xok[CT];
#pragma unroll
  for (int c = 0; c < CT; ++c) {
    const int m = m0 + 16 * c + li;
    xok[c] = m < a.M;
    // the lane group's offset inside a step (16 bytes per group for every kind of step)
    // is added per region below
    xrow[c] = (uint32_t)((int64_t)(xok[c] ? m : 0) * a.ldx_b);
  }

  if (ka < ks_end) {
    uint32_t vrow[RT], mrow[RT];
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      const int n = min(nbase + 16 * t + li, rowend - 1);
      vrow[t] = (uint32_t)((int64_t)n * a.v_ld_b) + (DT == kFP8 ? 16u : 16u) * lq;
      mrow[t] = (uint32_t)((int64_t)n * a.m_ld_b) + (DT == kFP8 ? 4u * lq : 4u * (lq >> 1));
    }
    uint32_t xr[CT];
#pragma unroll
    for (int c = 0; c < CT; ++c) xr[c] = xrow[c] + (DT == kFP8 ? 16u * lq : 16u * lq);
    run_stages<SparseStage<DT, CT, RT, U>>(
        acc, ka, ks_end, U * T::KS,
        [&](SparseStage<DT, CT, RT, U>& st, int k) {
          load_sparse<DT, CT, RT, U, WM, true>(st, L, vrow, mrow, xr, xok, k, ks_end);
        },
        [&](SparseStage<DT, CT, RT, U>& st, int k) {
          load_sparse<DT, CT, RT, U, WM, false>(st, L, vrow, mrow, xr, xok, k, ks_end);
        });
  }
  if (kd_beg < kb) {
    uint32_t drow[RT];
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      const int n = min(nbase + 16 * t + li, rowend - 1);
      drow[t] = (uint32_t)((int64_t)(n - R.dense_row_off) * a.d_ld_b) + 16u * lq;
    }
    uint32_t xr[CT];
#pragma unroll
    for (int c = 0; c < CT; ++c) xr[c] = xrow[c] + 16u * lq;
    const int dco = R.dense_col_off;
    run_stages<DenseStage<DT, CT, RT, U>>(
        acc, kd_beg, kb, U * T::KD,
        [&](DenseStage<DT, CT, RT, U>& st, int k) { load_dense<DT, CT, RT, U, true>(st, L, drow, xr, xok, k, kb, dco); },
        [&](DenseStage<DT, CT, RT, U>& st, int k) {
          load_dense<DT, CT, RT, U, false>(st, L, drow, xr, xok, k, kb, dco);
        });
  }

  // ---- add the waves' partial sums in LDS (wave order), then the epilogue; one
  // activation tile at a time keeps the buffer at W * RT KB
  __shared__ v4f red[W * RT * 64];
#pragma unroll
  for (int c = 0; c < CT; ++c) {
    if (c) __syncthreads();  // the previous tile's reads are done
#pragma unroll
    for (int t = 0; t < RT; ++t) red[(wave * RT + t) * 64 + lane] = acc[t][c];
    __syncthreads();
    for (int e = threadIdx.x; e < RT * 64; e += 64 * W) {
      const int ln = e & 63, t = e >> 6;
      v4f s = red[e];
#pragma unroll
      for (int w = 1; w < W; ++w) s += red[w * RT * 64 + e];
      const int m = m0 + 16 * c + (ln & 15);
      const int n0 = nbase + 16 * t + 4 * (ln >> 4);
      if (m < a.M && n0 < rowend) store4(a, s, m, n0, rowend);
    }
  }
}

// ---------------------------------------------------------------- row-split kernel
// For several activation tiles the activations are the reused operand.  Here each of the
// first `wused` waves of a workgroup owns 16 weight rows and all of K; the waves walk K
// together in chunks of four instruction steps.  Each chunk of activations (16*CT rows)
// is copied once per workgroup from global memory straight into LDS (buffer loads with
// an LDS destination; 16-byte blocks XOR-swizzled by row so the fragment reads are
// conflict-free; two buffers), and every wave reads its B fragments from there.  The
// weights are requested D chunks ahead into registers; the barrier that publishes the
// next activation chunk waits only for the activation loads, so the weight loads stay
// in flight across it.  No wave splits K: the epilogue stores from the accumulators.
template <int DT, int CT>
struct XTile {
  static constexpr int KS = Traits<DT>::KS;
  static constexpr int CHUNK_K = 4 * KS;                  // logical K per chunk
  static constexpr int ROW_B = CHUNK_K * Traits<DT>::ES;  // bytes per activation row (512)
  static constexpr int ROWS = 16 * CT;
  static constexpr int BYTES = ROWS * ROW_B;
  // LDS byte address of 16-byte block b of row r
  __device__ static __forceinline__ int addr(int r, int b) { return r * ROW_B + ((b ^ (r & 31)) << 4); }
};

template <int DT, int CT>
__device__ __forceinline__ v4i xlds(const uint8_t* lds, int r, int byte) {
  return *reinterpret_cast<const v4i*>(lds + XTile<DT, CT>::addr(r, byte >> 4) + (byte & 15));
}

// B fragments of one step from the LDS tile (step_b: byte offset of the step in a row).
// 2:4 steps and dense fp8 steps read K [16q, 16q+16) and [64+16q, 64+16q+16) of the
// step; dense bf16 steps read K [8q, 8q+8).
template <int DT, int CT>
__device__ __forceinline__ void frag_pair(v8i (&b)[CT], const uint8_t* lds, int li, int lq, int step_b) {
#pragma unroll
  for (int c = 0; c < CT; ++c) {
    const int r = 16 * c + li;
    b[c] = cat8(xlds<DT, CT>(lds, r, step_b + 16 * lq), xlds<DT, CT>(lds, r, step_b + 64 + 16 * lq));
  }
}
template <int DT, int CT>
__device__ __forceinline__ void frag_one(v8i (&b)[CT], const uint8_t* lds, int li, int lq, int step_b) {
  const v4i z = {0, 0, 0, 0};
#pragma unroll
  for (int c = 0; c < CT; ++c) b[c] = cat8(xlds<DT, CT>(lds, 16 * c + li, step_b + 16 * lq), z);
}

// Copy activations [m0, m0+16CT) x [kc, kc+CHUNK_K) into an LDS tile: each wave fills XI
// consecutive 1 KB blocks (lane l writes bytes 16l..16l+15 of its block; the source
// address applies the swizzle).  Rows past M and columns past kend are written as zeros.
template <int DT, int CT, int XI>
__device__ __forceinline__ void x_to_lds(uint8_t* lds, const GemmArgs& a, __amdgpu_buffer_rsrc_t rx, int m0, int kc,
                                         int kend, int wave, int lane) {
  typedef XTile<DT, CT> XT;
#pragma unroll
  for (int i = 0; i < XI; ++i) {
    const int blk = wave * XI + i;                           // 1 KB block of the tile
    const int r = (blk * 1024 + 16 * lane) / XT::ROW_B;      // tile row
    const int pb = ((blk * 1024 + 16 * lane) % XT::ROW_B) >> 4;  // physical 16-byte slot
    const int b = pb ^ (r & 31);                             // logical block stored there
    const int kcol = kc + b * 16 / Traits<DT>::ES;
    const int m = m0 + r;
    const uint32_t off = sel(m < a.M && kcol < kend, (uint32_t)((int64_t)m * a.ldx_b + (int64_t)kcol * Traits<DT>::ES));
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (__attribute__((address_space(3))) void*)(lds + blk * 1024), 16, off,
                                             0, 0, 0);
  }
}

// Weights of one chunk in registers: eight 16-byte fragments and four metadata words.
// fp8 (both kinds of chunk have four 128-wide steps): w[j] is step j's 2:4 value fragment
// or the first half of its dense fragment, w[4+j] the dense second half.  bf16: w[j] is
// step j's value fragment (2:4, j < 4) or dense fragment (eight 32-wide steps).
struct WChunk {
  v4i w[8];
  int ix[4];
};

// Load instructions one chunk issues; the same for 2:4 and dense chunks (the unused ones
// get out-of-range offsets), so the loads need no branches and the compiler keeps the
// fragments in place while they are in flight.
template <bool WM>
struct ChunkLoads {
  static constexpr int N = 8 + (WM ? 1 : 4);
};

// ok = false masks every lane (past the last chunk, or a wave that owns no rows).
template <int DT, bool WM>
__device__ __forceinline__ void load_chunk(WChunk& W, bool sparse, bool ok, int kc, int ke, int lq, uint32_t vrow,
                                           uint32_t mrow, uint32_t drow, int dco, __amdgpu_buffer_rsrc_t rv,
                                           __amdgpu_buffer_rsrc_t rm, __amdgpu_buffer_rsrc_t rd) {
  const __amdgpu_buffer_rsrc_t rw = sparse ? rv : rd;
  if constexpr (DT == kFP8) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int kk = kc + 128 * j;
      // 2:4: 16 kept values of logical K [kk+32q, kk+32q+32); dense: K [kk+16q, +16) and
      // [kk+64+16q, +16)
      const bool oka = ok && kk + (sparse ? 32 : 16) * lq < ke;
      const bool okb = ok && !sparse && kk + 64 + 16 * lq < ke;
      const uint32_t oa = sparse ? vrow + (uint32_t)(kk >> 1) : drow + (uint32_t)(kk - dco);
      W.w[j] = bl16<kNT>(rw, sel(oka, oa));
      W.w[4 + j] = bl16<kNT>(rd, sel(okb, oa + 64));
    }
  } else {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int kk = kc + (sparse ? 64 : 32) * j;
      const bool okj = ok && (!sparse || j < 4) && kk + (sparse ? 16 : 8) * lq < ke;
      const uint32_t o = sparse ? vrow + (uint32_t)kk : drow + 2 * (uint32_t)(kk - dco);
      W.w[j] = bl16<kNT>(rw, sel(okj, o));
    }
  }
  if constexpr (WM) {
    // lane group q loads step q's four words (16 bytes of the row); they are transposed
    // when the chunk is consumed (meta_words), not here, so the load stays in flight
    const v4i w = bl16<kNT>(rm, sel(ok && sparse && kc + 128 * lq < ke, mrow + 4 * (kc >> 5) + 12 * lq));
#pragma unroll
    for (int j = 0; j < 4; ++j) W.ix[j] = w[j];
  } else {
    constexpr int KS = Traits<DT>::KS;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int kk = kc + j * KS;
      W.ix[j] = bl4<kNT>(rm, sel(ok && sparse && kk + (DT == kFP8 ? 32 : 16) * lq < ke, mrow + 4 * (kk >> 5)));
    }
  }
}

// Tiled layout (fp8): each fragment of the chunk is one contiguous kilobyte.  vt, mt, dt:
// this lane's byte offset in its tile's first 2:4 / metadata / dense chunk (16 * lane
// included); cs, cd >= 0: the chunk's index within the 2:4 / dense part.  The chunk part
// of the address travels in the scalar offset; ok = false masks every lane.
__device__ __forceinline__ void load_chunk_tiled(WChunk& W, bool sparse, bool ok, int cs, int cd, uint32_t vt,
                                                 uint32_t mt, uint32_t dt, __amdgpu_buffer_rsrc_t rv,
                                                 __amdgpu_buffer_rsrc_t rm, __amdgpu_buffer_rsrc_t rd) {
  const __amdgpu_buffer_rsrc_t rw = sparse ? rv : rd;
  const uint32_t base = sel(ok, sparse ? vt : dt);
  const uint32_t dbase = sel(ok && !sparse, dt);
  const int s0 = sparse ? cs * 4096 : cd * 8192, sj = sparse ? 1024 : 2048;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    W.w[j] = bl16<kTiledNT>(rw, base, s0 + sj * j);
    W.w[4 + j] = bl16<kTiledNT>(rd, dbase, cd * 8192 + 2048 * j + 1024);
  }
  const v4i w = bl16<kTiledNT>(rm, sel(ok && sparse, mt), cs * 1024);
#pragma unroll
  for (int j = 0; j < 4; ++j) W.ix[j] = w[j];
}

// The metadata word of each step for this lane group.  Wide loads: lane group q holds
// step q's four words; a 4x4 transpose across lane groups (two lane swaps) gives lane
// group q word 4j+q of every step j.
template <bool WM>
__device__ __forceinline__ void meta_words(int (&ix)[4], const WChunk& W) {
  if constexpr (WM) {
    const auto s02 = __builtin_amdgcn_permlane32_swap((unsigned)W.ix[0], (unsigned)W.ix[2], false, false);
    const auto s13 = __builtin_amdgcn_permlane32_swap((unsigned)W.ix[1], (unsigned)W.ix[3], false, false);
    const auto s01 = __builtin_amdgcn_permlane16_swap(s02[0], s13[0], false, false);
    const auto s23 = __builtin_amdgcn_permlane16_swap(s02[1], s13[1], false, false);
    ix[0] = (int)s01[0];
    ix[1] = (int)s01[1];
    ix[2] = (int)s23[0];
    ix[3] = (int)s23[1];
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) ix[j] = W.ix[j];
  }
}

// MMAs of one chunk.  The B fragments of P steps are read from LDS before their MMAs,
// so the LDS latency is paid once per group rather than once per step.
template <int DT, int CT, int RT, bool WM, int P>
__device__ __forceinline__ void mma_chunk(v4f (&acc)[RT][CT], const WChunk (&W)[RT], bool sparse, const uint8_t* lds,
                                          int li, int lq) {
  static_assert(P == 1 || P == 2 || P == 4, "fragment group size");
  // each B fragment read from LDS feeds the RT row tiles of this wave
  if (sparse) {
    int mw[RT][4];
#pragma unroll
    for (int t = 0; t < RT; ++t) meta_words<WM>(mw[t], W[t]);
#pragma unroll
    for (int j0 = 0; j0 < 4; j0 += P) {
      v8i b[P][CT];
#pragma unroll
      for (int j = 0; j < P; ++j) frag_pair<DT, CT>(b[j], lds, li, lq, (j0 + j) * 128);
      if constexpr (P > 1) __builtin_amdgcn_sched_barrier(0);  // all reads of the group before its MMAs
#pragma unroll
      for (int j = 0; j < P; ++j)
#pragma unroll
        for (int t = 0; t < RT; ++t) {
          const int ix = DT == kFP8 ? mw[t][j0 + j] : (int)((uint32_t)mw[t][j0 + j] >> (16 * (lq & 1)));
#pragma unroll
          for (int c = 0; c < CT; ++c)
            acc[t][c] = mma_sparse(W[t].w[j0 + j], b[j][c], acc[t][c], ix, std::integral_constant<int, DT>());
        }
    }
  } else if constexpr (DT == kFP8) {
#pragma unroll
    for (int j0 = 0; j0 < 4; j0 += P) {
      v8i b[P][CT];
#pragma unroll
      for (int j = 0; j < P; ++j) frag_pair<DT, CT>(b[j], lds, li, lq, (j0 + j) * 128);
      if constexpr (P > 1) __builtin_amdgcn_sched_barrier(0);  // all reads of the group before its MMAs
#pragma unroll
      for (int j = 0; j < P; ++j)
#pragma unroll
        for (int t = 0; t < RT; ++t) {
          const v8i av = cat8(W[t].w[j0 + j], W[t].w[4 + j0 + j]);
#pragma unroll
          for (int c = 0; c < CT; ++c) acc[t][c] = mma_dense(av, b[j][c], acc[t][c], std::integral_constant<int, DT>());
        }
    }
  } else {
    const v4i z = {0, 0, 0, 0};
#pragma unroll
    for (int j0 = 0; j0 < 8; j0 += 2 * P) {
      v8i b[2 * P][CT];
#pragma unroll
      for (int j = 0; j < 2 * P; ++j) frag_one<DT, CT>(b[j], lds, li, lq, (j0 + j) * 64);
      if constexpr (P > 1) __builtin_amdgcn_sched_barrier(0);  // all reads of the group before its MMAs
#pragma unroll
      for (int j = 0; j < 2 * P; ++j)
#pragma unroll
        for (int t = 0; t < RT; ++t) {
          const v8i av = cat8(W[t].w[j0 + j], z);
#pragma unroll
          for (int c = 0; c < CT; ++c) acc[t][c] = mma_dense(av, b[j][c], acc[t][c], std::integral_constant<int, DT>());
        }
    }
  }
}

// Pipeline with NS register slots and NS LDS buffers, D = NS-1 chunks ahead (per wave,
// in issue order within chunk step c): activations of chunk c+D -> LDS buffer
// (c+D) % NS, weights of chunk c+D -> register slot (c+D) % NS, MMAs of chunk c (buffer
// and slot c % NS), then a barrier that waits for the activations of chunk c+1 (issued
// in step c+1-D, before that step's weights), so D chunks of weights stay in flight
// across it.  The buffer being filled held chunk c-1, which every wave has finished.
//
// XR (one or two token tiles): the activations of every chunk of the workgroup's K range
// are copied into dynamic LDS once, behind one barrier, and each wave then streams its
// weights with no further barrier, as far ahead as its register slots allow.
template <int DT, int CT, int RT, int WR, bool WM, int NS, int P, bool TL, int GM, bool XR = false>
__global__ __launch_bounds__(64 * WR) void spense_gemm_rows_kernel(GemmArgs a) {
  constexpr bool GR = GM == 1;   // grouped launch
  constexpr bool GLU = GM == 2;  // gate and up paired, the GLU step in the epilogue
  static_assert(!GLU || (RT == 1 && WR == 8), "paired gate / up: four waves per weight");
  static_assert(NS == 3 || NS == 4, "three or four pipeline slots");
  static_assert(!TL || (DT == kFP8 && WM), "the tiled layout is fp8 with whole-chunk metadata loads");
  static_assert(!XR || (CT <= 2 && GM <= 1), "resident activations: one or two token tiles, plain or grouped launch");
  constexpr int D = NS - 1;
  typedef XTile<DT, CT> XT;
  constexpr int KC = XT::CHUNK_K;
  constexpr int XI = XT::BYTES / 1024 / WR;  // 1 KB activation blocks per wave per chunk
  static_assert(XI >= 1 && XI * 1024 * WR == XT::BYTES, "activation tile must split evenly");
  constexpr int NL = ChunkLoads<WM>::N;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int li = lane & 15, lq = lane >> 4;
  int g = blockIdx.x, mb = blockIdx.y;
  if (a.rorder == 2) {  // XCD x (= id % 8) runs the token blocks of row groups x, x + 8, ...
    const int x = (int)blockIdx.x & 7, l = (int)blockIdx.x >> 3;
    g = (l / a.mblk) * 8 + x;
    mb = l % a.mblk;
  } else if (a.rorder == 1) {
    g = (int)blockIdx.x / a.mblk;
    mb = (int)blockIdx.x % a.mblk;
  }
  // GR (grouped launch): up to kMaxRegions regions in workgroup order, each of one weight
  // (its buffers, output and scales in a.mat); otherwise one weight (GLU: two weights,
  // gate and up, of equal geometry), up to two regions, buffers in a or a.mat (GLU).
  int ri = 0;
  if constexpr (GR) {
    for (int i = 1; i < a.nreg; ++i)
      if (g >= a.reg[i].wg0) ri = i;
  } else {
    ri = (a.nreg > 1 && g >= a.reg[1].wg0) ? 1 : 0;
  }
  const Region& R = a.reg[ri];
  // GLU: waves 0-3 own gate tiles, waves 4-7 the up tiles of the same rows
  const int wsel = GLU ? (wave & 3) : wave;
  const MatDesc& MD = a.mat[GR ? R.mat : (GLU ? wave >> 2 : 0)];
  const int rowend = R.row0 + R.rows;
  // workgroups of a region: (row group, K slice), slices of one row group adjacent
  const int slice = (g - R.wg0) % R.ksplit, rgroup = (g - R.wg0) / R.ksplit;
  const int nbase = R.row0 + (rgroup * R.wused + wsel) * 16 * RT;  // first row of the wave's RT tiles
  const int m0 = mb * 16 * CT;
  const int K = R.kend;
  const int kbound = R.kbound;
  const bool active = wsel < R.wused && nbase < rowend;

  __shared__ __attribute__((aligned(1024))) uint8_t xbuf[NS][XT::BYTES];
  extern __shared__ __attribute__((aligned(1024))) uint8_t xres[];  // XR: chunk c at (c - c_lo) * XT::BYTES
  constexpr bool FROM_MAT = GR || GLU;
  const __amdgpu_buffer_rsrc_t rx = rsrc(a.X, a.x_bytes),
                               rv = FROM_MAT ? rsrc(MD.values, MD.v_bytes) : rsrc(a.values, a.v_bytes),
                               rm = FROM_MAT ? rsrc(MD.meta, MD.m_bytes) : rsrc(a.meta, a.m_bytes),
                               rd = FROM_MAT ? rsrc(MD.dense, MD.d_bytes) : rsrc(a.dense, a.d_bytes);

  v4f acc[RT][CT];
#pragma unroll
  for (int t = 0; t < RT; ++t)
#pragma unroll
    for (int c = 0; c < CT; ++c) acc[t][c] = (v4f){0.f, 0.f, 0.f, 0.f};

  bool tok[RT];  // tile t of this wave holds rows of the region
  uint32_t vrow[RT], mrow[RT], drow[RT];
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    tok[t] = nbase + 16 * t < rowend;
    const int n = min(nbase + 16 * t + li, rowend - 1);
    vrow[t] = (uint32_t)((int64_t)n * a.v_ld_b) + 16u * lq;
    mrow[t] = (uint32_t)((int64_t)n * a.m_ld_b) + (DT == kFP8 ? 4u * lq : 4u * (lq >> 1));
    drow[t] = (uint32_t)((int64_t)max(n - R.dense_row_off, 0) * a.d_ld_b) + 16u * lq;
  }

  // chunk list: 2:4 chunks start at 0 and cover [0, kbound); dense chunks start at kbound;
  // this workgroup's K slice is chunks [c_lo, c_hi)
  const int n_sp = (kbound + KC - 1) / KC;
  const int n_de = (K - kbound + KC - 1) / KC;
  const int c_lo = R.cut[slice], c_hi = R.cut[slice + 1];
  auto chunk_k = [&](int c) { return c < n_sp ? c * KC : kbound + (c - n_sp) * KC; };
  auto chunk_end = [&](int c) { return c < n_sp ? kbound : K; };
  // tiled layout: offsets of this lane in its tiles' first chunk of each part
  uint32_t vt[RT], mt[RT], dt[RT];
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    vt[t] = mt[t] = dt[t] = 0;
    if constexpr (TL) {
      const uint32_t ts = (uint32_t)(nbase / 16 + t), td = (uint32_t)((nbase - R.dense_row_off) / 16 + t);
      vt[t] = ts * (uint32_t)n_sp * 4096u + 16u * lane;
      mt[t] = ts * (uint32_t)n_sp * 1024u + 16u * lane;
      dt[t] = td * (uint32_t)n_de * 8192u + 16u * lane;
    }
  }
  auto load = [&](WChunk (&W)[RT], int c) {
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      if constexpr (TL)
        load_chunk_tiled(W[t], c < n_sp, tok[t] && c < c_hi, c, max(c - n_sp, 0), vt[t], mt[t], dt[t], rv, rm, rd);
      else
        load_chunk<DT, WM>(W[t], c < n_sp, tok[t] && c < c_hi, chunk_k(c), chunk_end(c), lq, vrow[t], mrow[t],
                           drow[t], R.dense_col_off, rv, rm, rd);
    }
  };
  auto xload = [&](int buf, int c) {
    x_to_lds<DT, CT, XI>(xbuf[buf], a, rx, m0, chunk_k(c), c < c_hi ? chunk_end(c) : -1, wave, lane);
  };
  auto xtile = [&](int s, int c) -> const uint8_t* {
    if constexpr (XR)
      return xres + (c - c_lo) * XT::BYTES;
    else
      return xbuf[s];
  };

  // A wave that owns rows loads weights and runs the MMAs; the others only stage
  // activations and take part in the barriers.  The two loops are separate so that no
  // path leaves a weight load pending where the compiler would have to wait for it.
  auto run = [&](auto act_const) {
    constexpr bool ACT = decltype(act_const)::value;
    // loads issued after the activations of chunk c+1, at the barrier of chunk c: that
    // step's weights, then D-1 further steps of activations and weights
    constexpr int AFTER = ACT ? RT * NL + (D - 1) * (XI + RT * NL) : (D - 1) * XI;
    WChunk slot[NS][RT];
    if constexpr (XR) {
      // every chunk's activations, then the first D chunks of weights; the barrier waits
      // for the activations only (loads complete in issue order)
      for (int c = c_lo; c < c_hi; ++c)
        x_to_lds<DT, CT, XI>(xres + (c - c_lo) * XT::BYTES, a, rx, m0, chunk_k(c), chunk_end(c), wave, lane);
      if constexpr (ACT) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
          __builtin_amdgcn_sched_barrier(0);  // each chunk's weights before the next chunk's
          load(slot[d], c_lo + d);
        }
      }
      barrier_vm<ACT ? D * RT * NL : 0>();
      if constexpr (!ACT) return;
    } else {
#pragma unroll
      for (int d = 0; d < D; ++d) {
        xload(d, c_lo + d);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (ACT) load(slot[d], c_lo + d);
        __builtin_amdgcn_sched_barrier(0);
      }
      // the first chunk's activations only: the loads issued after them (D chunks of
      // weights, D - 1 of activations, in this order: the scheduling barriers keep a
      // chunk's weight loads from sinking below the next chunk's) stay in flight while the
      // next ones are requested
      barrier_vm<AFTER>();
    }
    auto step = [&](auto s_const, int c) {
      constexpr int S = decltype(s_const)::value;
      constexpr int SD = (S + D) % NS;
      if constexpr (!XR) {
        xload(SD, c + D);
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (ACT) {
        load(slot[SD], c + D);
        __builtin_amdgcn_sched_barrier(0);
        mma_chunk<DT, CT, RT, WM, P>(acc, slot[S], c < n_sp, xtile(S, c), li, lq);
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (!XR) barrier_vm<AFTER>();
    };
    int c = c_lo;
    for (; c + NS <= c_hi; c += NS) {
      step(std::integral_constant<int, 0>(), c);
      step(std::integral_constant<int, 1>(), c + 1);
      step(std::integral_constant<int, 2>(), c + 2);
      if constexpr (NS == 4) step(std::integral_constant<int, 3 % NS>(), c + 3);
    }
    if (c < c_hi) step(std::integral_constant<int, 0>(), c);
    if (c + 1 < c_hi) step(std::integral_constant<int, 1>(), c + 1);
    if constexpr (NS == 4)
      if (c + 2 < c_hi) step(std::integral_constant<int, 2>(), c + 2);
  };
  // the epilogue's scales, requested before any weight or activation so that they have
  // long arrived when the stores begin (K slices write unscaled partials and need none)
  EpiScales<RT, CT> es, eu;  // GLU: gate scales and token scales in es, up scales in eu
  if constexpr (GLU) {
    if (wave >= 4 && active) {
      epi_scales(es, a.mat[0].sw, a.sx, a.M, nbase + 4 * lq, m0 + li, rowend);
      epi_scales(eu, a.mat[1].sw, nullptr, a.M, nbase + 4 * lq, m0 + li, rowend);
    }
  } else {
    if (active && R.ksplit == 1) epi_scales(es, MD.sw, a.sx, a.M, nbase + 4 * lq, m0 + li, rowend);
  }
  if (active)
    run(std::true_type());
  else
    run(std::false_type());

  if constexpr (GLU) {
    // h = glu(g, u) with g, u each scaled as the plain epilogue scales them: the gate waves
    // pass their accumulators through the (now idle) staging buffers to the up waves of
    // the same rows, which write H (fp32).  Every wave takes both barriers.
    xdl_fence();
    barrier_vm<0>();  // all staging loads of every wave have landed
    static_assert(XT::BYTES >= 4 * CT * 64 * 16, "gate accumulators fit one staging buffer");
    float* ex = reinterpret_cast<float*>(&xbuf[0][0]);
    if (wave < 4 && active) {
#pragma unroll
      for (int cc = 0; cc < CT; ++cc) *reinterpret_cast<v4f*>(ex + ((wsel * CT + cc) * 64 + lane) * 4) = acc[0][cc];
    }
    barrier_vm_lgkm0<63>();
    float tmax[CT];  // per token: the maximum of |h| over this lane's stored rows
#pragma unroll
    for (int cc = 0; cc < CT; ++cc) tmax[cc] = 0.0f;
    if (wave >= 4 && active) {
      const MatDesc& G = a.mat[0];
      const MatDesc& Up = a.mat[1];
#pragma unroll
      for (int cc = 0; cc < CT; ++cc) {
        const int m = m0 + 16 * cc + li;
        const int n0 = nbase + 4 * lq;
        if (m >= a.M || n0 >= rowend) continue;
        const v4f gv = *reinterpret_cast<const v4f*>(ex + ((wsel * CT + cc) * 64 + lane) * 4);
        const float xs = es.x[cc];
        float h[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          float gg = gv[r], uu = acc[0][cc][r];
          if (G.sw) gg = gg * es.w[0][r];
          if (Up.sw) uu = uu * eu.w[0][r];
          h[r] = glu_silu(gg * xs, uu * xs);
          if (n0 + r < rowend) tmax[cc] = fmaxf(tmax[cc], fabsf(h[r]));
        }
        float* hp = reinterpret_cast<float*>(G.Y) + (int64_t)m * G.ldy + n0;
        if (G.vec_store && n0 + 3 < rowend) {
          *reinterpret_cast<v4f*>(hp) = (v4f){h[0], h[1], h[2], h[3]};
        } else {
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (n0 + r < rowend) hp[r] = h[r];
        }
      }
    }
    if (a.hmax) {
      // per token, the maximum over the workgroup's rows: the four row groups of a lane
      // column (lanes li, li + 16, li + 32, li + 48), then the four up waves through LDS
      float* red = reinterpret_cast<float*>(&xbuf[1][0]);
      if (wave >= 4) {
#pragma unroll
        for (int cc = 0; cc < CT; ++cc) {
          float v = fmaxf(tmax[cc], __shfl_xor(tmax[cc], 16, 64));
          v = fmaxf(v, __shfl_xor(v, 32, 64));
          if (lq == 0) red[wsel * 16 * CT + 16 * cc + li] = v;
        }
      }
      barrier_vm_lgkm0<63>();
      if (wave == 4 && lane < 16 * CT) {
        const int m = m0 + lane;
        const float v = fmaxf(fmaxf(red[lane], red[16 * CT + lane]), fmaxf(red[32 * CT + lane], red[48 * CT + lane]));
        if (m < a.M) a.hmax[(int64_t)m * a.groups + g] = v;
      }
    }
    return;
  }
  if (!active) return;
  xdl_fence();
#pragma unroll
  for (int t = 0; t < RT; ++t)
#pragma unroll
    for (int cc = 0; cc < CT; ++cc) {
      const int m = m0 + 16 * cc + li;
      const int n0 = nbase + 16 * t + 4 * lq;
      if (m >= a.M || n0 >= rowend) continue;
      if (R.ksplit == 1) {
        store4e(MD.Y, MD.ldy, MD.sw != nullptr, MD.vec_store, a, es, t, cc, acc[t][cc], m, n0, rowend);
      } else {  // unscaled fp32 partial of this K slice, one 16-byte store where it can
        float* pp = a.part + ((int64_t)slice * a.M + m) * a.N + n0;
        if (n0 + 3 < rowend && a.part_vec) {
          *reinterpret_cast<v4f*>(pp) = acc[t][cc];
        } else {
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (n0 + r < rowend) pp[r] = acc[t][cc][r];
        }
      }
    }
}

// Row-split kernel for two 64-token halves per workgroup (65-128 tokens per block): each
// wave's weights of a chunk, in registers, feed the MMAs of both halves, so a weight row
// is streamed once for up to 128 tokens instead of once per 64.  The activations of a
// chunk (both halves, 64 KB) take two LDS buffers: chunk c + 1 is copied during step c
// into the buffer chunk c - 1 left (every wave finished with it at the previous barrier),
// and the barrier at the end of step c waits for it; the weights run NS - 1 chunks ahead
// in NS register slots.  Plain launches of tiled fp8 weights, one row tile and eight
// waves per workgroup; with K slices (workgroups (row group, slice), slices of a row
// group adjacent) each writes its unscaled fp32 partial sums for the reduction launch.
template <int WR, int NS>
__global__ __launch_bounds__(64 * WR) void spense_gemm_rows2_kernel(GemmArgs a) {
  constexpr int DT = kFP8, CT = 4, RT = 1, D = NS - 1;
  static_assert(NS == 2 || NS == 3, "two or three weight slots");
  typedef XTile<DT, CT> XT;  // one 64-token half
  constexpr int KC = XT::CHUNK_K;
  constexpr int XI = XT::BYTES / 1024 / WR;  // 1 KB activation blocks per wave per half
  static_assert(XI >= 1 && XI * 1024 * WR == XT::BYTES, "activation tile must split evenly");
  constexpr int NL = ChunkLoads<true>::N;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int li = lane & 15, lq = lane >> 4;
  const int g = blockIdx.x;
  const int ri = (a.nreg > 1 && g >= a.reg[1].wg0) ? 1 : 0;
  const Region& R = a.reg[ri];
  const MatDesc& MD = a.mat[0];
  const int rowend = R.row0 + R.rows;
  const int slice = (g - R.wg0) % R.ksplit, rgroup = (g - R.wg0) / R.ksplit;
  const int nbase = R.row0 + (rgroup * R.wused + wave) * 16;
  const int m0 = blockIdx.y * 32 * CT;
  const int K = R.kend, kbound = R.kbound;
  const bool active = wave < R.wused && nbase < rowend;

  __shared__ __attribute__((aligned(1024))) uint8_t xbuf[2][2 * XT::BYTES];
  const __amdgpu_buffer_rsrc_t rx = rsrc(a.X, a.x_bytes), rv = rsrc(a.values, a.v_bytes),
                               rm = rsrc(a.meta, a.m_bytes), rd = rsrc(a.dense, a.d_bytes);
  v4f acc0[RT][CT], acc1[RT][CT];
#pragma unroll
  for (int c = 0; c < CT; ++c) acc0[0][c] = acc1[0][c] = (v4f){0.f, 0.f, 0.f, 0.f};

  const int n_sp = (kbound + KC - 1) / KC, n_de = (K - kbound + KC - 1) / KC;
  const int c_lo = R.cut[slice], c_hi = R.cut[slice + 1];  // this workgroup's chunks
  auto chunk_k = [&](int c) { return c < n_sp ? c * KC : kbound + (c - n_sp) * KC; };
  auto chunk_end = [&](int c) { return c < n_sp ? kbound : K; };
  const bool tok = nbase < rowend;
  const uint32_t ts = (uint32_t)(nbase / 16), td = (uint32_t)((nbase - R.dense_row_off) / 16);
  const uint32_t vt = ts * (uint32_t)n_sp * 4096u + 16u * lane, mt = ts * (uint32_t)n_sp * 1024u + 16u * lane,
                 dt = td * (uint32_t)n_de * 8192u + 16u * lane;
  auto load = [&](WChunk& W, int c) {
    load_chunk_tiled(W, c < n_sp, tok && c < c_hi, c, max(c - n_sp, 0), vt, mt, dt, rv, rm, rd);
  };
  auto xload = [&](int c) {  // both halves of chunk c into buffer c % 2
    uint8_t* b = xbuf[c & 1];
    const int ke = c < c_hi ? chunk_end(c) : -1;
    x_to_lds<DT, CT, XI>(b, a, rx, m0, chunk_k(c), ke, wave, lane);
    x_to_lds<DT, CT, XI>(b + XT::BYTES, a, rx, m0 + 16 * CT, chunk_k(c), ke, wave, lane);
  };

  auto run = [&](auto act_const) {
    constexpr bool ACT = decltype(act_const)::value;
    WChunk slot[NS][RT];
    // the first chunk's activations, then D chunks of weights; the barrier waits for the
    // activations only (loads complete in issue order)
    xload(c_lo);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (ACT) {
#pragma unroll
      for (int d = 0; d < D; ++d) {
        load(slot[d][0], c_lo + d);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    barrier_vm<ACT ? D * NL : 0>();
    // step c: activations of chunk c + 1, weights of chunk c + 2, the MMAs of chunk c for
    // both halves, then a barrier that waits for chunk c + 1's activations (issued before
    // this step's weights, the only loads younger than them)
    auto step = [&](auto s_const, int c) {
      constexpr int S = decltype(s_const)::value;
      xload(c + 1);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (ACT) {
        load(slot[(S + D) % NS][0], c + D);
        __builtin_amdgcn_sched_barrier(0);
        const uint8_t* xb = xbuf[c & 1];
        mma_chunk<DT, CT, RT, true, 1>(acc0, slot[S], c < n_sp, xb, li, lq);
        mma_chunk<DT, CT, RT, true, 1>(acc1, slot[S], c < n_sp, xb + XT::BYTES, li, lq);
        __builtin_amdgcn_sched_barrier(0);
      }
      barrier_vm<ACT ? NL : 0>();
    };
    int c = c_lo;
    for (; c + NS <= c_hi; c += NS) {
      step(std::integral_constant<int, 0>(), c);
      step(std::integral_constant<int, 1>(), c + 1);
      if constexpr (NS == 3) step(std::integral_constant<int, 2 % NS>(), c + 2);
    }
    if (c < c_hi) step(std::integral_constant<int, 0>(), c);
    if constexpr (NS == 3)
      if (c + 1 < c_hi) step(std::integral_constant<int, 1>(), c + 1);
  };
  if (active)
    run(std::true_type());
  else
    run(std::false_type());
  if (!active) return;
  if (R.ksplit > 1) {  // unscaled fp32 partials of this K slice, one 16-byte store where it can
    xdl_fence();
#pragma unroll
    for (int c = 0; c < 2 * CT; ++c) {
      const int m = m0 + 16 * c + li;
      const int n0 = nbase + 4 * lq;
      if (m >= a.M || n0 >= rowend) continue;
      const v4f v = c < CT ? acc0[0][c] : acc1[0][c - CT];
      float* pp = a.part + ((int64_t)slice * a.M + m) * a.N + n0;
      if (n0 + 3 < rowend && a.part_vec) {
        *reinterpret_cast<v4f*>(pp) = v;
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (n0 + r < rowend) pp[r] = v[r];
      }
    }
    return;
  }
  // the epilogue's scales only now: held through the loop they would push the kernel
  // past the register file
  EpiScales<RT, 2 * CT> es;
  epi_scales(es, MD.sw, a.sx, a.M, nbase + 4 * lq, m0 + li, rowend);
  xdl_fence();
#pragma unroll
  for (int c = 0; c < 2 * CT; ++c) {
    const int m = m0 + 16 * c + li;
    const int n0 = nbase + 4 * lq;
    if (m >= a.M || n0 >= rowend) continue;
    store4e(MD.Y, MD.ldy, MD.sw != nullptr, MD.vec_store, a, es, 0, c, c < CT ? acc0[0][c] : acc1[0][c - CT], m, n0,
            rowend);
  }
}

// Y of a K-sliced GEMM (the planner slices every region of a weight alike, KS slices):
// the sum of the slices' fp32 partials in slice order, then the epilogue of store4
// ((sum * w_scale[n]) * x_scale[m], bf16 or fp32).  One thread per output element; its
// KS loads and the scales are issued before the first add, so their latencies overlap.
template <int KS>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(GemmArgs a) {
  const int64_t total = (int64_t)a.M * a.N;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const bool narrow = total < ((int64_t)1 << 31);
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += stride) {
    const int m = narrow ? (int)e / a.N : (int)(e / a.N);
    const int n = (int)(e - (int64_t)m * a.N);
    const float* pe = a.part + e;  // slice sl's partial of this element: pe[sl * M * N]
    float p[KS];
#pragma unroll
    for (int sl = 0; sl < KS; ++sl) p[sl] = pe[sl * total];
    const float sw = a.sw ? a.sw[n] : 1.0f, sx = a.sx ? a.sx[m] : 1.0f;
    float v = p[0];
#pragma unroll
    for (int sl = 1; sl < KS; ++sl) v += p[sl];
    if (a.sw) v = v * sw;
    v = v * sx;
    if (a.out_f32)
      reinterpret_cast<float*>(a.Y)[(int64_t)m * a.ldy + n] = v;
    else
      reinterpret_cast<uint16_t*>(a.Y)[(int64_t)m * a.ldy + n] = (uint16_t)bf16_bits(v);
  }
}

// Pipeline depth and fragment grouping per instance, chosen to stay within the register
// file: four slots and whole-chunk fragment groups for up to two activation tiles, three
// slots and two-step groups for four; fp8 without wide metadata loads (metadata rows not
// 16-byte aligned, four separately masked loads per chunk) one step lighter, and even so
// its four-tile, eight-wave instance spills a few registers.
// The resident-activation instances' dynamic LDS above the default limit: a per-device
// function attribute, set once per (device, instance) under std::call_once.
constexpr int kXresMaxBytes = 160 * 1024;

template <int DT, int CT, int RT, int WR, bool WM, bool TL, int GM = 0>
hipError_t launch_rows_wm(const dim3& grid, const dim3& block, const GemmArgs& a, hipStream_t s, int xres = 0) {
  constexpr bool light = DT == kFP8 && !WM;
  constexpr int NS = CT <= 2 && RT == 1 && !light ? 4 : 3;
  constexpr int P = CT == 1 && RT == 1 ? 4 : 1;
  if constexpr (DT == kFP8 && CT <= 2 && RT == 1 && WR == 8 && TL && GM <= 1) {
    if (xres > 0) {
      const int lds = xres * XTile<DT, CT>::BYTES;
      if (lds > kXresMaxBytes) return hipErrorInvalidValue;
      auto k = spense_gemm_rows_kernel<DT, CT, RT, WR, WM, NS, P, TL, GM, true>;
      int dev = 0;
      hipError_t e = hipGetDevice(&dev);
      if (e != hipSuccess) return e;
      if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
      static std::once_flag once[64];  // one set per instance of this function
      static hipError_t rc[64];
      std::call_once(once[dev], [&] {
        rc[dev] = hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize,
                                      kXresMaxBytes);
      });
      if (rc[dev] != hipSuccess) return rc[dev];
      hipLaunchKernelGGL(k, grid, block, lds, s, a);
      return hipGetLastError();
    }
  }
  if (xres > 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL((spense_gemm_rows_kernel<DT, CT, RT, WR, WM, NS, P, TL, GM>), grid, block, 0, s, a);
  return hipGetLastError();
}

template <int DT, int CT, int RT, int WR>
hipError_t launch_rows(const LaunchShape& ls, const GemmArgs& a, hipStream_t s) {
  dim3 grid = a.rorder ? dim3(a.groups * ls.mblocks) : dim3(a.groups, ls.mblocks), block(64 * WR);
  if constexpr (DT == kFP8) {
    if (a.tiled && (a.nmat > 1 || ls.glu)) {  // grouped or paired launch: tiled fp8, 8 waves
      if constexpr (RT == 1 && WR == 8) {
        if (ls.glu) return launch_rows_wm<DT, CT, RT, WR, true, true, 2>(grid, block, a, s);
        return launch_rows_wm<DT, CT, RT, WR, true, true, 1>(grid, block, a, s, ls.xres);
      }
      return hipErrorInvalidValue;
    }
    if (a.tiled) return launch_rows_wm<DT, CT, RT, WR, true, true>(grid, block, a, s, ls.xres);
    if (ls.xres) return hipErrorInvalidValue;
    if (a.m_ld_b % 16 == 0) return launch_rows_wm<DT, CT, RT, WR, true, false>(grid, block, a, s);
  }
  if (a.tiled || ls.xres) return hipErrorInvalidValue;
  return launch_rows_wm<DT, CT, RT, WR, false, false>(grid, block, a, s);
}

template <int DT, int CT, int RT, int W, int UMAX = 0>
hipError_t launch_t(const LaunchShape& ls, const GemmArgs& a, hipStream_t s) {
  // steps per pipeline stage: keep two stages of operands within the register budget
  constexpr int per_step = 8 * RT + 8 * CT;  // VGPRs of one dense step (the larger kind)
  constexpr int budget = W >= 16 ? 80 : (W >= 8 ? 100 : 128);
  constexpr int U0 = budget / per_step;
  constexpr int U = UMAX ? UMAX : (U0 < 1 ? 1 : (U0 > 4 ? 4 : U0));
  dim3 grid(a.groups, ls.mblocks), block(64 * W);
  // metadata rows 16-byte aligned -> one 16-byte load covers four steps of a row
  constexpr bool kWide = DT == kFP8 && U % 4 == 0;
  if (kWide && a.m_ld_b % 16 == 0)
    hipLaunchKernelGGL((spense_gemm_kernel<DT, CT, RT, W, U, kWide>), grid, block, 0, s, a);
  else
    hipLaunchKernelGGL((spense_gemm_kernel<DT, CT, RT, W, U, false>), grid, block, 0, s, a);
  return hipGetLastError();
}

template <int DT, int CT>
hipError_t launch_ct(const LaunchShape& ls, const GemmArgs& a, hipStream_t s) {
  // the LDS reduction buffer is W * RT KB
  switch (ls.rt * 100 + ls.waves + (ls.u8 && CT == 1 ? 10000 : 0)) {
    case 104: return launch_t<DT, CT, 1, 4>(ls, a, s);
    case 108: return launch_t<DT, CT, 1, 8>(ls, a, s);
    case 116: return launch_t<DT, CT, 1, 16>(ls, a, s);
    case 204: return launch_t<DT, CT, 2, 4>(ls, a, s);
    case 208: return launch_t<DT, CT, 2, 8>(ls, a, s);
    case 404: return launch_t<DT, CT, 4, 4>(ls, a, s);
    case 10104: return launch_t<DT, CT, 1, 4, 8>(ls, a, s);
    case 10108: return launch_t<DT, CT, 1, 8, 8>(ls, a, s);
    default: return hipErrorInvalidValue;
  }
}

template <int DT, int CT>
hipError_t launch_rows_ct(const LaunchShape& ls, const GemmArgs& a, hipStream_t s) {
  switch (ls.rt * 100 + ls.waves) {
    case 104: return launch_rows<DT, CT, 1, 4>(ls, a, s);
    case 108: return launch_rows<DT, CT, 1, 8>(ls, a, s);
    case 204: return launch_rows<DT, CT, 2, 4>(ls, a, s);
    default: return hipErrorInvalidValue;
  }
}

// ---------------------------------------------------------------- large-M kernel
// For many tokens the matrix cores become the bound, and every byte moved should feed
// many MMAs.  A workgroup computes 128 weight rows x 256 tokens; its waves form a grid of
// 2 row halves x 2 or 4 token parts, each wave 64 rows (4 row tiles) x 128 or 64 tokens
// (with 8 waves, two per SIMD, one wave's stalls are covered by the other's MMAs).  Both
// operands of a step (128 columns) are copied once into LDS by direct loads
// (activations 256 x 128 bytes, with 16-byte blocks swizzled so that the fragment reads
// of 16 rows are conflict-free; the weight fragments of the 8 row tiles in lane order),
// three stages deep, so that two steps of loads are in flight without holding
// registers.  Each B fragment read feeds 4 MMAs, each A fragment 4 or 8.  The barrier of
// a step sits before its last MMA group, and the fragments of the next step are read
// from LDS right after it, under that group, so that no wave starts a step waiting for
// LDS.  Workgroups of one row block are adjacent (token block fastest), so with 8 token
// blocks each XCD keeps one activation block in its L2.  fp8 only.
constexpr int kBigTokens = 256, kBigRowTiles = 8;

struct BigStage {
  static constexpr int X_B = kBigTokens * 128;       // activations: 256 tokens x 128 bytes
  static constexpr int W_B = kBigRowTiles * 2048;    // per row tile: 2:4 values or dense halves
  static constexpr int M_B = kBigRowTiles * 256;     // per row tile: metadata words
  static constexpr int BYTES = X_B + W_B + M_B;
  __device__ static __forceinline__ int xaddr(int r, int b) { return r * 128 + ((b ^ ((r >> 1) & 7)) << 4); }
};

// Where the loads of one step go and what they cover.
struct BigStepLd {
  uint8_t* st;                 // stage buffer
  int ks, ke, cs, js, cd, jd;  // first column, column end, tiled-layout chunk and step
  bool in, sparse;
};

// Step kinds for the fragment reads of the next step.
constexpr int kStepSparse = 0, kStepDense = 1, kStepNone = 2;

template <bool TL, int WV>
__global__ __launch_bounds__(64 * WV) void spense_gemm_big_kernel(GemmArgs a) {
  static_assert(WV == 4 || WV == 8, "4 or 8 waves");
  constexpr int RPW = 4, NT = kBigRowTiles;
  typedef BigStage St;
  constexpr int NS = 3, D = NS - 1;
  constexpr int TC = 32 / WV;                    // token tiles per wave
  constexpr int TU = NT / WV;                    // row tiles whose weights a wave copies
  constexpr int XI = St::X_B / 1024 / WV;        // 1 KB activation blocks per wave per step
  constexpr int NL = XI + 3 * TU;                // loads per wave per step
  constexpr int PER = (NL + TC - 1) / TC;        // loads issued after each MMA group
  constexpr int NL_AT_BAR = (TC - 1) * PER < NL ? (TC - 1) * PER : NL;  // issued before the barrier
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int li = lane & 15, lq = lane >> 4;
  const int wr = wave & 1, wc = wave >> 1;
  int g = blockIdx.x;
  if (a.xgt > 0 && g < a.xg1) {
    // XCD-aware order: XCD x (= id % 8) takes token group x % (T / GT) (GT blocks) and
    // the row blocks of class x / (T / GT) (every RC-th); a bijection on [0, xg1)
    const int T = a.tblocks, GT = a.xgt, RC = a.xrc, TGc = T / GT;
    const int x = g & 7, l = g >> 3, tg = x % TGc, rc = x / TGc;
    g = ((l / GT) * RC + rc) * T + tg * GT + l % GT;
  }
  const int ri = (a.nreg > 1 && g >= a.reg[1].wg0) ? 1 : 0;
  const Region& R = a.reg[ri];
  const int rowend = R.row0 + R.rows;
  const int rb = (g - R.wg0) / a.tblocks, tb = (g - R.wg0) % a.tblocks;
  const int rblk = R.row0 + rb * 16 * NT;  // first row of the workgroup
  const int m0 = tb * kBigTokens;
  const int K = R.kend, kbound = R.kbound;

  extern __shared__ __attribute__((aligned(1024))) uint8_t big_lds[];
  const __amdgpu_buffer_rsrc_t rx = rsrc(a.X, a.x_bytes), rv = rsrc(a.values, a.v_bytes),
                               rm = rsrc(a.meta, a.m_bytes), rd = rsrc(a.dense, a.d_bytes);
  v4f acc[RPW][TC];
#pragma unroll
  for (int t = 0; t < RPW; ++t)
#pragma unroll
    for (int c = 0; c < TC; ++c) acc[t][c] = (v4f){0.f, 0.f, 0.f, 0.f};

  // steps of 128 columns: 2:4 steps cover [0, kbound), dense steps start at kbound
  const int n_sp = (kbound + 127) / 128, n_de = (K - kbound + 127) / 128, nst = n_sp + n_de;
  const int nch_sp = (n_sp + 3) / 4, nch_de = (n_de + 3) / 4;  // tiled layout chunks
  auto step_k = [&](int s) __attribute__((always_inline)) { return s < n_sp ? 128 * s : kbound + 128 * (s - n_sp); };

  // This wave copies the weights of row tiles TU wave .. TU wave + TU - 1.
  bool tok[TU];
  uint32_t vb[TU], mb[TU], db[TU];
#pragma unroll
  for (int u = 0; u < TU; ++u) {
    const int r0 = rblk + 16 * (TU * wave + u);
    tok[u] = r0 < rowend;
    if constexpr (TL) {
      const uint32_t ts = (uint32_t)(r0 / 16), td = (uint32_t)((r0 - R.dense_row_off) / 16);
      vb[u] = ts * (uint32_t)nch_sp * 4096u + 16u * lane;
      mb[u] = ts * (uint32_t)nch_sp * 1024u + 16u * li + 4u * lq;
      db[u] = td * (uint32_t)nch_de * 8192u + 16u * lane;
    } else {
      const int n = min(r0 + li, rowend - 1);
      vb[u] = (uint32_t)((int64_t)n * a.v_ld_b) + 16u * lq;
      mb[u] = (uint32_t)((int64_t)n * a.m_ld_b) + 4u * lq;
      db[u] = (uint32_t)((int64_t)max(n - R.dense_row_off, 0) * a.d_ld_b) + 16u * lq;
    }
  }

  // Loads of step s into a stage buffer, numbered 0 .. NL-1: the activation blocks, then
  // for each of the wave's row tiles the value (or first dense) fragment, the second
  // dense fragment and the metadata word.  The ones a step does not use get out-of-range
  // offsets, so every step issues the same loads.
  auto prep = [&](int buf, int s) __attribute__((always_inline)) {
    BigStepLd p;
    p.st = big_lds + buf * St::BYTES;
    // wave-uniform (readfirstlane), so that the buffer resources chosen by them stay scalar
    p.in = __builtin_amdgcn_readfirstlane(s < nst ? 1 : 0) != 0;
    p.sparse = __builtin_amdgcn_readfirstlane(s < n_sp ? 1 : 0) != 0;
    p.ks = step_k(s);
    p.ke = !p.in ? -1 : (p.sparse ? kbound : K);
    const int sd = max(s - n_sp, 0);
    p.cs = s / 4;
    p.js = s & 3;
    p.cd = sd / 4;
    p.jd = sd & 3;
    return p;
  };
  auto load_one = [&](auto i_const, const BigStepLd& p) __attribute__((always_inline)) {
    constexpr int i = decltype(i_const)::value;
    if constexpr (i < XI) {
      const int blk = wave * XI + i;
      const int r = 8 * blk + (lane >> 3), pb = lane & 7, b = pb ^ ((r >> 1) & 7);
      const int m = m0 + r, kcol = p.ks + 16 * b;
      const uint32_t off = sel(m < a.M && kcol < p.ke, (uint32_t)((int64_t)m * a.ldx_b + kcol));
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (__attribute__((address_space(3))) void*)(p.st + blk * 1024), 16, off,
                                               0, 0, 0);
    } else {
      constexpr int u = (i - XI) / 3, kind = (i - XI) % 3;
      const int tile = TU * wave + u;
      const bool ok = p.in && tok[u];
      if constexpr (kind == 0) {
        uint32_t off;
        bool k;
        if constexpr (TL) {
          off = p.sparse ? vb[u] + (uint32_t)(p.cs * 4096 + 1024 * p.js) : db[u] + (uint32_t)(p.cd * 8192 + 2048 * p.jd);
          k = ok;
        } else {
          off = p.sparse ? vb[u] + (uint32_t)(p.ks >> 1) : db[u] + (uint32_t)(p.ks - R.dense_col_off);
          k = ok && p.ks + (p.sparse ? 32 : 16) * lq < p.ke;
        }
        __builtin_amdgcn_raw_ptr_buffer_load_lds(p.sparse ? rv : rd,
                                                 (__attribute__((address_space(3))) void*)(p.st + St::X_B + tile * 2048),
                                                 16, sel(k, off), 0, 0, TL ? kTiledNT : kNT);
      } else if constexpr (kind == 1) {
        uint32_t off;
        bool k;
        if constexpr (TL) {
          off = db[u] + (uint32_t)(p.cd * 8192 + 2048 * p.jd + 1024);
          k = ok;
        } else {
          off = db[u] + (uint32_t)(p.ks - R.dense_col_off) + 64;
          k = ok && p.ks + 64 + 16 * lq < p.ke;
        }
        __builtin_amdgcn_raw_ptr_buffer_load_lds(
            rd, (__attribute__((address_space(3))) void*)(p.st + St::X_B + tile * 2048 + 1024), 16,
            sel(k && !p.sparse, off), 0, 0, TL ? kTiledNT : kNT);
      } else {
        uint32_t off;
        bool k;
        if constexpr (TL) {
          off = mb[u] + (uint32_t)(p.cs * 1024 + 256 * p.js);
          k = ok;
        } else {
          off = mb[u] + 4u * (uint32_t)(p.ks >> 5);
          k = ok && p.ks + 32 * lq < p.ke;
        }
        __builtin_amdgcn_raw_ptr_buffer_load_lds(
            rm, (__attribute__((address_space(3))) void*)(p.st + St::X_B + St::W_B + tile * 256), 4,
            sel(k && p.sparse, off), 0, 0, TL ? kTiledNT : kNT);
      }
    }
  };

  // Fragments.  A of the wave's 4 row tiles (2:4: value fragment and metadata word; dense:
  // both halves) in two sets that alternate between steps (set P holds the current step's,
  // the other receives the next step's); B, one register per token tile (the next step's
  // first two land in registers the current step's last group no longer reads).
  static_assert(TC >= 3, "the last group must not use B registers 0 and 1");
  v4i alo[2][RPW], ahi[2][RPW];
  int aix[2][RPW];
  v8i bq[TC];
  auto bfrag = [&](const uint8_t* st, int c) __attribute__((always_inline)) {
    const int r = 16 * (TC * wc + c) + li;
    return cat8(*reinterpret_cast<const v4i*>(st + St::xaddr(r, lq)),
                *reinterpret_cast<const v4i*>(st + St::xaddr(r, 4 + lq)));
  };
  auto read_a = [&](auto kind_const, auto set_const, const uint8_t* st) __attribute__((always_inline)) {
    constexpr int KIND = decltype(kind_const)::value, Q = decltype(set_const)::value;
    const uint8_t* wl = st + St::X_B + (RPW * wr) * 2048 + 16 * lane;
    const int* ml = reinterpret_cast<const int*>(st + St::X_B + St::W_B + (RPW * wr) * 256) + lane;
#pragma unroll
    for (int t = 0; t < RPW; ++t) {
      alo[Q][t] = *reinterpret_cast<const v4i*>(wl + t * 2048);
      if constexpr (KIND == kStepSparse) aix[Q][t] = ml[t * 64];
      if constexpr (KIND == kStepDense) ahi[Q][t] = *reinterpret_cast<const v4i*>(wl + t * 2048 + 1024);
    }
    bq[0] = bfrag(st, 0);
    bq[1] = bfrag(st, 1);
  };

  // One step: MMA group c uses B fragment c; fragment c + 2 is read before it.  Before the
  // last group: wait for this wave's reads of the stage and for its loads of step s + 1
  // (the loads of step s + D issued so far are younger), meet the other waves, and read the
  // first fragments of step s + 1 into the other set, under the last group.  The loads of
  // step s + D into stage (s + D) % NS (it held step s - 1, which every wave had finished
  // reading at the previous barrier) follow the MMA groups, PER at a time.
  int s = 0, cur = 0;  // cur = s % NS
  auto step = [&](auto kind_const, auto next_const, auto set_const) __attribute__((always_inline)) {
    constexpr bool SPARSE = decltype(kind_const)::value == kStepSparse;
    constexpr int NEXT = decltype(next_const)::value, P = decltype(set_const)::value;
    const int nxt = cur == 0 ? D : cur - 1;  // (s + D) % NS
    const int nx1 = cur == NS - 1 ? 0 : cur + 1;
    const uint8_t* st = big_lds + cur * St::BYTES;
    const BigStepLd ld = prep(nxt, s + D);
    static_for<TC>([&](auto c_const) {
      constexpr int c = decltype(c_const)::value;
      if constexpr (c == TC - 1) {
        barrier_vm_lgkm0<NL_AT_BAR>();
        if constexpr (NEXT != kStepNone)
          read_a(std::integral_constant<int, NEXT>(), std::integral_constant<int, 1 - P>(), big_lds + nx1 * St::BYTES);
      } else if constexpr (c + 2 < TC) {
        bq[c + 2] = bfrag(st, c + 2);
      }
#pragma unroll
      for (int t = 0; t < RPW; ++t) {
        if constexpr (SPARSE)
          acc[t][c] = mma_sparse(alo[P][t], bq[c], acc[t][c], aix[P][t], std::integral_constant<int, kFP8>());
        else
          acc[t][c] = mma_dense(cat8(alo[P][t], ahi[P][t]), bq[c], acc[t][c], std::integral_constant<int, kFP8>());
      }
      static_for<PER>([&](auto j_const) {
        constexpr int i = c * PER + decltype(j_const)::value;
        if constexpr (i < NL) load_one(std::integral_constant<int, i>(), ld);
      });
      __builtin_amdgcn_sched_barrier(0);
    });
    ++s;
    cur = nx1;
  };
  const std::integral_constant<int, 0> S0;
  const std::integral_constant<int, 1> S1;
  // Steps [s, e) of one kind, entered with the current fragments in set 0 and left with
  // the next part's first fragments (kind NEXT) in set 0.
  auto part = [&](auto kind_const, auto next_const, int e) __attribute__((always_inline)) {
    while (s + 2 < e) {
      step(kind_const, kind_const, S0);
      step(kind_const, kind_const, S1);
    }
    if (s + 2 == e) {
      step(kind_const, kind_const, S0);
      step(kind_const, next_const, S1);
    } else {
      step(kind_const, next_const, S0);
      if constexpr (decltype(next_const)::value != kStepNone) {
#pragma unroll
        for (int t = 0; t < RPW; ++t) {
          alo[0][t] = alo[1][t];
          ahi[0][t] = ahi[1][t];
          aix[0][t] = aix[1][t];
        }
      }
    }
  };

  // Prologue: loads of steps 0 .. D-1, then the first fragments of step 0.
#pragma unroll
  for (int d = 0; d < D; ++d) {
    const BigStepLd p = prep(d, d);
    static_for<NL>([&](auto i_const) { load_one(i_const, p); });
  }
  barrier_vm<NL>();  // step 0 is in LDS (only step 1's loads may be outstanding)
  const std::integral_constant<int, kStepSparse> SP;
  const std::integral_constant<int, kStepDense> DE;
  const std::integral_constant<int, kStepNone> NO;
  if (n_sp > 0)
    read_a(SP, S0, big_lds);
  else
    read_a(DE, S0, big_lds);

  // 2:4 steps, then dense steps.
  if (n_sp > 0) {
    if (n_de > 0)
      part(SP, DE, n_sp);
    else
      part(SP, NO, n_sp);
  }
  if (n_de > 0) part(DE, NO, nst);

  xdl_fence();
  EpiScales<RPW, TC> es;
  epi_scales(es, a.sw, a.sx, a.M, rblk + 16 * RPW * wr + 4 * lq, m0 + 16 * TC * wc + li, rowend);
  if (!a.out_f32 && ((uintptr_t)a.Y % 16 == 0) && (a.ldy % 8 == 0) && (rblk % 8 == 0)) {
    // whole token rows through LDS (out_tile_write)
    static_assert(16 * NT * 2 * kBigTokens <= 3 * St::BYTES, "the output tile fits the stages");
    barrier_vm_lgkm0<0>();  // every wave's last operand reads and copies are done
    out_tile_write<RPW, TC, 2 * NT>(big_lds, acc, es, a.sw != nullptr, wr, wc, li, lq);
    barrier_vm_lgkm0<0>();
    out_tile_store<2 * NT, 64 * WV>(big_lds, kBigTokens, m0, a.M, rblk, rowend, a.Y, a.ldy);
    return;
  }
#pragma unroll
  for (int t = 0; t < RPW; ++t)
#pragma unroll
    for (int c = 0; c < TC; ++c) {
      const int m = m0 + 16 * (TC * wc + c) + li;
      const int n0 = rblk + 16 * (RPW * wr + t) + 4 * lq;
      if (m < a.M && n0 < rowend) store4e(a.Y, a.ldy, a.sw != nullptr, a.vec_store, a, es, t, c, acc[t][c], m, n0, rowend);
    }
}

template <int WV>
hipError_t launch_big_wv(const GemmArgs& a, hipStream_t s) {
  constexpr int lds = 3 * BigStage::BYTES;
  static_assert(lds <= 160 * 1024, "LDS of a CU");
  auto k = a.tiled ? spense_gemm_big_kernel<true, WV> : spense_gemm_big_kernel<false, WV>;
  hipError_t e = set_big_lds(k, a.tiled ? 1 : 0, WV == 8 ? 1 : 0, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k, dim3(a.groups), dim3(64 * WV), lds, s, a);
  return hipGetLastError();
}

hipError_t launch_big(const LaunchShape& ls, const GemmArgs& a, hipStream_t s) {
  return ls.waves == 4 ? launch_big_wv<4>(a, s) : launch_big_wv<8>(a, s);
}

template <int DT>
hipError_t launch_dt(const LaunchShape& ls, const GemmArgs& a, hipStream_t s) {
  if (ls.big == 3) return launch_mid(DT, a, s);
  if (ls.big == 2) return launch_big2(DT, a, s);
  if (ls.big) return DT == kFP8 ? launch_big(ls, a, s) : hipErrorInvalidValue;
  if (a.tiled && !ls.rows) return hipErrorInvalidValue;  // the K-split kernel reads the row-major layout only
  if (ls.rows == 2) {  // two 64-token halves per workgroup: tiled fp8, 8 waves, one row tile
    if constexpr (DT == kFP8) {
      if (!a.tiled || ls.rt != 1 || ls.waves != 8 || a.nmat != 1) return hipErrorInvalidValue;
      for (int i = 0; i < a.nreg; ++i)
        if (a.reg[i].ksplit > 1 && !a.part) return hipErrorInvalidValue;
      // two weight slots: with three the kernel spills past the register file
      hipLaunchKernelGGL((spense_gemm_rows2_kernel<8, 2>), dim3(a.groups, ls.mblocks), dim3(512), 0, s, a);
      return hipGetLastError();
    }
    return hipErrorInvalidValue;
  }
  if (ls.rows) {
    if (ls.ct == 1) return launch_rows_ct<DT, 1>(ls, a, s);
    if (ls.ct == 2) return launch_rows_ct<DT, 2>(ls, a, s);
    return launch_rows_ct<DT, 4>(ls, a, s);
  }
  if (ls.ct == 1) return launch_ct<DT, 1>(ls, a, s);
  if (ls.ct == 2) return launch_ct<DT, 2>(ls, a, s);
  return launch_ct<DT, 4>(ls, a, s);
}

}  // namespace

hipError_t launch_splitk_reduce(const GemmArgs& a, hipStream_t s) {
  const int64_t total = (int64_t)a.M * a.N;
  int64_t g = (total + 255) / 256;
  if (g > 4096) g = 4096;
  const dim3 grid((unsigned)(g < 1 ? 1 : g)), block(256);
  for (int i = 1; i < a.nreg; ++i)
    if (a.reg[i].ksplit != a.reg[0].ksplit) return hipErrorInvalidValue;  // one slice count per weight
  switch (a.reg[0].ksplit) {
    case 2: hipLaunchKernelGGL(splitk_reduce_kernel<2>, grid, block, 0, s, a); break;
    case 3: hipLaunchKernelGGL(splitk_reduce_kernel<3>, grid, block, 0, s, a); break;
    case 4: hipLaunchKernelGGL(splitk_reduce_kernel<4>, grid, block, 0, s, a); break;
    case 5: hipLaunchKernelGGL(splitk_reduce_kernel<5>, grid, block, 0, s, a); break;
    case 6: hipLaunchKernelGGL(splitk_reduce_kernel<6>, grid, block, 0, s, a); break;
    case 7: hipLaunchKernelGGL(splitk_reduce_kernel<7>, grid, block, 0, s, a); break;
    case 8: hipLaunchKernelGGL(splitk_reduce_kernel<8>, grid, block, 0, s, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_gemm(int dtype, const LaunchShape& ls, const GemmArgs& a, hipStream_t s) {
  return dtype == kFP8 ? launch_dt<kFP8>(ls, a, s) : launch_dt<kBF16>(ls, a, s);
}

}  // namespace spense
