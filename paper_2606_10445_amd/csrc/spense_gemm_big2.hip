// The 256 x 256 large-M kernel (spense_gemm.hip has the overview of all GEMM kernels).
#include "spense_gemm_device.h"

namespace spense {
namespace {

// ---------------------------------------------------------------- large-M kernel, 256 x 256 tiles
// Both operands through LDS as in spense_gemm_big_kernel, with twice the rows per
// workgroup and per wave: a workgroup computes 256 weight rows x 256 tokens, its 8 waves a
// grid of 2 row halves x 4 token quarters, each wave 128 rows (8 row tiles) x 64 tokens (4
// token tiles, 128 accumulators).  Each B fragment read from LDS feeds 8 MMAs, each A
// fragment 4.  Tiled weight layout only.
//
// The CU's load path moves about 57 bytes per clock from L2 with 16-byte-per-lane loads,
// into registers or straight into LDS alike, but a load instruction costs at least ~18
// clocks however few bytes it moves (a 4-byte-per-lane load moves 256 bytes in ~32; all
// measured on MI355X).  So every load here moves 1 KB: per 128-column step a wave issues 4
// activation blocks and, for its 2 row tiles, the 2:4 value blocks or both dense halves;
// a 2:4 step's metadata (256 bytes per row tile) takes 4 more loads, one on each of waves
// 0-3, each gathering the pieces of 4 row tiles.  6.5 loads per 2:4 step (52 KB per
// workgroup) against ~1.07k clocks of its 256 MMAs.
//
// Per-wave timelines showed every wave waiting at the barrier for the loads when they had
// one step to land in, so the 2:4 steps run three stages deep (loads two steps ahead; a
// stage is 52 KB: activations, values, metadata) and the dense steps, whose stage is 64 KB
// and whose MMAs take twice as long, two.  Within a step the loads go out early: the
// activation blocks before the first group of 4 MMAs, the weight blocks before the third.
// An input-split weight switches from the first layout to the second once, after a
// barrier.  The per-lane offsets are loop-invariant; the step's offset travels in the
// scalar offset.  The barrier at the start of a step waits for this wave's loads of the
// step and for its LDS reads of the previous step.
constexpr int kB2Rows = 256, kB2Tokens = 256, kB2RowTiles = 16;
constexpr int kB2XSlot = kB2Tokens * 128;                                      // activations of one step
constexpr int kB2SStage = kB2XSlot + kB2RowTiles * 1024 + kB2RowTiles * 256;  // + 2:4 values, metadata
constexpr int kB2DStage = kB2XSlot + kB2RowTiles * 2048;                       // + both dense halves
constexpr int kB2Lds = 3 * kB2SStage > 2 * kB2DStage ? 3 * kB2SStage : 2 * kB2DStage;

// GR: a grouped launch (several weights sharing X and K): up to kMaxRegions regions, each
// reading its weight's buffers, output and scales from a.mat[R.mat].
template <bool GR>
__global__ __launch_bounds__(512) void spense_gemm_big2_kernel(GemmArgs a) {
  constexpr int WV = 8, NT = kB2RowTiles, RPW = 8, TC = 4;
  constexpr int TU = NT / WV;                // row tiles whose weights a wave copies
  constexpr int XI = kB2XSlot / 1024 / WV;  // 1 KB activation blocks per wave per step
  constexpr int MW = NT * 256 / 1024;       // waves that copy a 2:4 step's metadata
  static_assert(XI + 2 * TU == RPW, "eight loads per dense step");
  static_assert(XI == 4 && TU == 2 && MW <= WV, "load schedule");
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int li = lane & 15, lq = lane >> 4;
  const int wr = wave & 1, wc = wave >> 1;
  // Workgroups [0, hg0): 256 x 256 tiles, in the XCD-aware order when it is on.  From
  // hg0 on (dispatched last, so that they fill the tail of the grid): the row blocks
  // hrb0 .. of the last region as 256 x 128 tiles, hper per row block; their waves of
  // token quarters 2 and 3 only copy and take part in the barriers.
  int g = blockIdx.x, ri, rb, m0;
  bool half = false;
  if (g < a.hg0) {
    if (a.xgt > 0 && g < a.xg1) {  // XCD-aware order, as in spense_gemm_big_kernel
      const int T = a.tblocks, GT = a.xgt, RC = a.xrc, TGc = T / GT;
      const int x = g & 7, l = g >> 3, tg = x % TGc, rc = x / TGc;
      g = ((l / GT) * RC + rc) * T + tg * GT + l % GT;
    }
    ri = 0;
    if constexpr (GR) {
      for (int i = 1; i < a.nreg; ++i)
        if (g >= a.reg[i].wg0) ri = i;
    } else {
      ri = (a.nreg > 1 && g >= a.reg[1].wg0) ? 1 : 0;
    }
    rb = (g - a.reg[ri].wg0) / a.tblocks;
    m0 = (g - a.reg[ri].wg0) % a.tblocks * (a.btok > 0 ? a.btok : kB2Tokens);
  } else {
    const int h = g - a.hg0;
    ri = a.nreg - 1;
    rb = a.hrb0 + h / a.hper;
    m0 = h % a.hper * (kB2Tokens / 2);
    half = true;
  }
  const Region& R = a.reg[ri];
  const int rowend = R.row0 + R.rows;
  const int rblk = R.row0 + rb * kB2Rows;
  // tokens of this tile: 256, or 192 (full tiles of a 192-token block), or 128 (half tiles)
  const int ntok = half ? kB2Tokens / 2 : (a.btok > 0 ? a.btok : kB2Tokens);
  const int K = R.kend, kbound = R.kbound;

  extern __shared__ __attribute__((aligned(1024))) uint8_t big_lds[];
  const MatDesc& MD = a.mat[GR ? R.mat : 0];
  const __amdgpu_buffer_rsrc_t rx = rsrc(a.X, a.x_bytes),
                               rv = GR ? rsrc(MD.values, MD.v_bytes) : rsrc(a.values, a.v_bytes),
                               rm = GR ? rsrc(MD.meta, MD.m_bytes) : rsrc(a.meta, a.m_bytes),
                               rd = GR ? rsrc(MD.dense, MD.d_bytes) : rsrc(a.dense, a.d_bytes);
  v4f acc[RPW][TC];
#pragma unroll
  for (int t = 0; t < RPW; ++t)
#pragma unroll
    for (int c = 0; c < TC; ++c) acc[t][c] = (v4f){0.f, 0.f, 0.f, 0.f};

  const int n_sp = (kbound + 127) / 128, n_de = (K - kbound + 127) / 128, nst = n_sp + n_de;
  const int nch_sp = (n_sp + 3) / 4, nch_de = (n_de + 3) / 4;

  // loop-invariant per-lane offsets (kOOB for rows past M or row tiles past the region)
  uint32_t xo[XI];
  int xb[XI];  // the column (bytes) of this lane's 16-byte block inside the step
#pragma unroll
  for (int i = 0; i < XI; ++i) {
    const int blk = wave * XI + i;
    const int r = 8 * blk + (lane >> 3), b = (lane & 7) ^ ((r >> 1) & 7);
    const int m = m0 + r;
    xb[i] = 16 * b;
    xo[i] = m < a.M && r < ntok ? (uint32_t)((int64_t)m * a.ldx_b + 16 * b) : kOOB;
  }
  uint32_t vo[TU], dlo[TU];
#pragma unroll
  for (int u = 0; u < TU; ++u) {
    const int r0 = rblk + 16 * (TU * wave + u);
    const bool ok = r0 < rowend;
    vo[u] = ok ? (uint32_t)(r0 / 16) * (uint32_t)nch_sp * 4096u + 16u * lane : kOOB;
    dlo[u] = ok && r0 >= R.dense_row_off ? (uint32_t)((r0 - R.dense_row_off) / 16) * (uint32_t)nch_de * 8192u + 16u * lane
                                          : kOOB;
  }
  // a 2:4 step's metadata: wave w < MW copies the 256-byte pieces of row tiles 4w .. 4w + 3
  // (lane l: 16 bytes of tile 4w + l / 16); a tile's piece for step s sits 256 s bytes into
  // its metadata
  uint32_t mo1 = kOOB;
  if (wave < MW) {
    const int r0 = rblk + 16 * (4 * wave + (lane >> 4));
    if (r0 < rowend) mo1 = (uint32_t)(r0 / 16) * (uint32_t)nch_sp * 1024u + 16u * li;
  }

  // Load j of this wave for 2:4 step sn into stage stg: activation blocks (j < 4), the value
  // blocks of its two row tiles (j = 4, 5), the metadata gather (j = 6, waves 0-3).
  auto sp_load = [&](auto j_const, int sn, uint8_t* stg) __attribute__((always_inline)) {
    constexpr int j = decltype(j_const)::value;
    if (sn >= n_sp) return;  // uniform
    if constexpr (j < XI) {
      const int ks = 128 * sn;
      uint32_t off = xo[j];
      if (ks + 128 > kbound) off = ks + xb[j] < kbound ? off : kOOB;  // the region's last, partial step
      lds_load16<0>(rx, stg + (wave * XI + j) * 1024, off, ks);
    } else if constexpr (j < XI + TU) {
      constexpr int u = j - XI;
      lds_load16<kTiledNT>(rv, stg + kB2XSlot + (TU * wave + u) * 1024, vo[u], 1024 * sn);
    } else {
      if (wave < MW) lds_load16<kTiledNT>(rm, stg + kB2XSlot + NT * 1024 + wave * 1024, mo1, 256 * sn);
    }
  };
  // Load j of this wave for dense step sn into stage stg: activation blocks (j < 4), then
  // the two halves of its two row tiles.
  auto de_load = [&](auto j_const, int sn, uint8_t* stg) __attribute__((always_inline)) {
    constexpr int j = decltype(j_const)::value;
    if (sn >= nst) return;  // uniform
    if constexpr (j < XI) {
      const int ks = kbound + 128 * (sn - n_sp);
      uint32_t off = xo[j];
      if (ks + 128 > K) off = ks + xb[j] < K ? off : kOOB;
      lds_load16<0>(rx, stg + (wave * XI + j) * 1024, off, ks);
    } else {
      constexpr int u = (j - XI) % TU, half = (j - XI) / TU;
      lds_load16<kTiledNT>(rd, stg + kB2XSlot + (TU * wave + u) * 2048 + 1024 * half, dlo[u],
                           2048 * (sn - n_sp) + 1024 * half);
    }
  };

  // B fragments of the wave's 4 token tiles from a stage
  auto read_b = [&](v8i (&bq)[TC], const uint8_t* xs) __attribute__((always_inline)) {
#pragma unroll
    for (int c = 0; c < TC; ++c) {
      const int r = 16 * (TC * wc + c) + li;
      bq[c] = cat8(*reinterpret_cast<const v4i*>(xs + r * 128 + ((lq ^ ((r >> 1) & 7)) << 4)),
                   *reinterpret_cast<const v4i*>(xs + r * 128 + (((4 + lq) ^ ((r >> 1) & 7)) << 4)));
    }
  };

  // 2:4 step s from stage cur; the loads of step s + 2 go to stage nxt.  Per row tile t the
  // A fragment of tile t + 1 is read (other register set) before the 4 MMAs of tile t.
  // ACT = false: a wave without tokens (token quarters past a 128- or 192-token tile) only copies.
  auto sp_step = [&](auto act_const, int s, const uint8_t* cur, uint8_t* nxt) __attribute__((always_inline)) {
    constexpr bool ACT = decltype(act_const)::value;
    // this wave's loads of step s have landed once at most those of step s + 1 are pending
    if (s + 1 < n_sp) {
      if (wave < MW)
        barrier_vm_lgkm0<XI + TU + 1>();
      else
        barrier_vm_lgkm0<XI + TU>();
    } else {
      barrier_vm_lgkm0<0>();
    }
    v8i bq[TC];
    const uint8_t* vl = cur + kB2XSlot + (RPW * wr) * 1024 + 16 * lane;
    const uint8_t* ml = cur + kB2XSlot + NT * 1024 + (RPW * wr) * 256 + 16 * li + 4 * lq;
    v4i av[2];
    int aix[2];
    if constexpr (ACT) {
      read_b(bq, cur);
      av[0] = *reinterpret_cast<const v4i*>(vl);
      aix[0] = *reinterpret_cast<const int*>(ml);
    }
    static_for<RPW>([&](auto t_const) {
      constexpr int t = decltype(t_const)::value;
      constexpr int q = t & 1;
      if constexpr (ACT && t + 1 < RPW) {
        av[1 - q] = *reinterpret_cast<const v4i*>(vl + (t + 1) * 1024);
        aix[1 - q] = *reinterpret_cast<const int*>(ml + (t + 1) * 256);
      }
      if constexpr (t == 0) static_for<XI>([&](auto j) { sp_load(j, s + 2, nxt); });
      if constexpr (t == 2) {
        sp_load(std::integral_constant<int, XI>(), s + 2, nxt);
        sp_load(std::integral_constant<int, XI + 1>(), s + 2, nxt);
        sp_load(std::integral_constant<int, XI + 2>(), s + 2, nxt);
      }
      if constexpr (ACT) {
#pragma unroll
        for (int c = 0; c < TC; ++c)
          acc[t][c] = mma_sparse(av[q], bq[c], acc[t][c], aix[q], std::integral_constant<int, kFP8>());
      }
      __builtin_amdgcn_sched_barrier(0);
    });
  };

  // dense step s from stage cur; the loads of step s + 1 go to stage nxt
  auto de_step = [&](auto act_const, int s, const uint8_t* cur, uint8_t* nxt) __attribute__((always_inline)) {
    constexpr bool ACT = decltype(act_const)::value;
    barrier_vm_lgkm0<0>();
    v8i bq[TC];
    const uint8_t* wl = cur + kB2XSlot + (RPW * wr) * 2048 + 16 * lane;
    v4i alo[2], ahi[2];
    if constexpr (ACT) {
      read_b(bq, cur);
      alo[0] = *reinterpret_cast<const v4i*>(wl);
      ahi[0] = *reinterpret_cast<const v4i*>(wl + 1024);
    }
    static_for<RPW>([&](auto t_const) {
      constexpr int t = decltype(t_const)::value;
      constexpr int q = t & 1;
      if constexpr (ACT && t + 1 < RPW) {
        alo[1 - q] = *reinterpret_cast<const v4i*>(wl + (t + 1) * 2048);
        ahi[1 - q] = *reinterpret_cast<const v4i*>(wl + (t + 1) * 2048 + 1024);
      }
      if constexpr (t == 0 || t == 2) {
        de_load(std::integral_constant<int, 2 * t>(), s + 1, nxt);
        de_load(std::integral_constant<int, 2 * t + 1>(), s + 1, nxt);
        de_load(std::integral_constant<int, 2 * t + 2>(), s + 1, nxt);
        de_load(std::integral_constant<int, 2 * t + 3>(), s + 1, nxt);
      }
      if constexpr (ACT) {
#pragma unroll
        for (int c = 0; c < TC; ++c)
          acc[t][c] = mma_dense(cat8(alo[q], ahi[q]), bq[c], acc[t][c], std::integral_constant<int, kFP8>());
      }
      __builtin_amdgcn_sched_barrier(0);
    });
  };

  auto run = [&](auto act_const) __attribute__((always_inline)) {
    int s = 0;
    if (n_sp > 0) {
      static_for<XI + TU + 1>([&](auto j) { sp_load(j, 0, big_lds); });
      static_for<XI + TU + 1>([&](auto j) { sp_load(j, 1, big_lds + kB2SStage); });
      int k = 0;  // stage of step s
      for (; s < n_sp; ++s) {
        const int k2 = k == 0 ? 2 : k - 1;  // stage of step s + 2
        sp_step(act_const, s, big_lds + k * kB2SStage, big_lds + k2 * kB2SStage);
        k = k == 2 ? 0 : k + 1;
      }
      xdl_fence();
    }
    if (n_de > 0) {
      if (n_sp > 0) barrier_vm_lgkm0<0>();  // every wave is done with the 2:4 stages
      static_for<RPW>([&](auto j) { de_load(j, s, big_lds); });
      for (; s < nst; ++s) {
        const int k = (s - n_sp) & 1;
        de_step(act_const, s, big_lds + k * kB2DStage, big_lds + (1 - k) * kB2DStage);
      }
      xdl_fence();
    }
  };
  // bf16 output with 16-byte aligned rows leaves through LDS as whole token rows
  // (out_tile_write); the waves of token quarters past the tile's tokens (2 and 3 of a 256
  // x 128 tile, 3 of a 256 x 192 one) then only help with the stores
  const bool idle = wc * (kB2Tokens / 4) >= ntok;
  const bool via_lds = !a.out_f32 && ((uintptr_t)MD.Y % 16 == 0) && (MD.ldy % 8 == 0) && (rblk % 8 == 0);
  if (idle) {
    run(std::false_type());
    if (!via_lds) return;
  } else {
    run(std::true_type());
  }
  EpiScales<RPW, TC> es;
  if (!idle) epi_scales(es, MD.sw, a.sx, a.M, rblk + 16 * RPW * wr + 4 * lq, m0 + 16 * TC * wc + li, rowend);
  if (!via_lds) {
#pragma unroll
    for (int t = 0; t < RPW; ++t)
#pragma unroll
      for (int c = 0; c < TC; ++c) {
        const int m = m0 + 16 * (TC * wc + c) + li;
        const int n0 = rblk + 16 * (RPW * wr + t) + 4 * lq;
        if (m < a.M && n0 < rowend) store4e(MD.Y, MD.ldy, MD.sw != nullptr, MD.vec_store, a, es, t, c, acc[t][c], m, n0, rowend);
      }
    return;
  }
  barrier_vm_lgkm0<0>();  // every wave's last operand reads and copies are done
  if (!idle) out_tile_write<RPW, TC, kB2Rows / 8>(big_lds, acc, es, MD.sw != nullptr, wr, wc, li, lq);
  barrier_vm_lgkm0<0>();
  out_tile_store<kB2Rows / 8, 512>(big_lds, ntok, m0, a.M, rblk, rowend, MD.Y, MD.ldy);
}

}  // namespace

hipError_t launch_big2(const GemmArgs& a, hipStream_t s) {
  static_assert(kB2Lds <= 160 * 1024, "LDS of a CU");
  if (!a.tiled) return hipErrorInvalidValue;  // the planner sends row-major weights to the 128 x 256 kernel
  const bool gr = a.nmat > 1;
  auto k = gr ? spense_gemm_big2_kernel<true> : spense_gemm_big2_kernel<false>;
  hipError_t e = set_big_lds(k, 1, gr ? 3 : 2, kB2Lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k, dim3(a.groups), dim3(512), kB2Lds, s, a);
  return hipGetLastError();
}

}  // namespace spense
