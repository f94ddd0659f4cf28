// The 128-row large-M kernel (spense_gemm.hip has the overview of all GEMM kernels).
#include "spense_gemm_device.h"

namespace spense {
namespace {

// Between decode and the 256 x 256 grid, and for bf16 every many-token shape: a workgroup
// computes 128 weight rows x 128 tokens, optionally over a slice of K (fp32 partial sums,
// added by splitk_reduce_kernel).  fp8 weights in the tiled layout (one or several, MatDesc),
// bf16 weights row-major.
//
// Eight waves compute, the rows split over four of them and the tokens in two 64-token halves
// (32 rows x 64 tokens each), and four (one per SIMD) only copy.  A wave that issues a copy
// into LDS is held there until the CU's load path takes it (~18 clocks per kilobyte, all waves
// together), and LDS reads
// behind it in the same wave wait too, while copies and reads of different waves do not slow
// each other (measured: 32 KB copied in 606 clocks and 64 KB read in 690 at once, 585 and 687
// alone).  With every wave copying its share, a 128-column step took 1370 clocks.
//
// A step is 128 bytes of every token: 128 columns in fp8, 64 in bf16, whose operand layouts
// are the same in bytes (16 bytes of kept values per lane of a 16-row tile; activations and
// dense weights bytes [16 q, 16 q + 16) and [64 + 16 q, 64 + 16 q + 16) for lane group q).
// Steps go through a ring of NS stages in LDS that 2:4 and dense steps share
// (a stage: the activations, and 16 KB for the row tiles' values and metadata or dense
// halves), so an input-split weight runs across its boundary without draining the ring.
// Per step one barrier; after it every computing wave holds the step's fragments in
// registers, so its stage is free for the copies of step s + NS, and the fragments of step
// s + 1 are read into the other register set between the MMAs of step s.
//
// Measured (graph replay, us, the planner's choice before -> this kernel): 5120 x 8192
// input-split M = 448 / 640 / 768 37 / 46 / 45 -> 34 / 35 / 38, 8192 x 5120 M = 288 / 448 /
// 512 31 / 37 / 40 -> 28 / 27 / 29, 5120 x 25600 M = 512 / 640 103 / 124 -> 94 / 94 and in
// 6 / 3 / 2 slices at M = 128 / 224 / 288 39 / 57 / 75 -> 35 / 49 / 64.  A step takes 0.43 us,
// of which the copies alone take 0.40 (26 loads issued behind one barrier) and the barrier,
// reads and MMAs alone 0.25.  64 x 64 tokens a wave instead of 64 x 32 (256-token blocks)
// does not fit the registers of twelve waves.
constexpr int kMidRows = 128, kMidTok = 128, kMidX = kMidTok * 128, kMidStage = kMidX + 16384;
constexpr int kMidStages = 5, kMidLds = kMidStages * kMidStage;

template <int DT>
__global__ __launch_bounds__(768) void spense_gemm_mid_kernel(GemmArgs a) {
  constexpr bool TL = DT == kFP8;  // tiled weights; bf16 reads the row-major layout
  constexpr int ES = Traits<DT>::ES;
  typedef std::integral_constant<int, DT> Dt;
  constexpr int RPW = 2, TC = 4;  // row tiles and token tiles of a wave
  constexpr int NS = kMidStages, XB = kMidX, SB = kMidStage;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int li = lane & 15, lq = lane >> 4;
  const bool copies = wave >= 8;
  const int wr = wave & 3, wc = (wave >> 2) & 1;  // row quarter and token half of a computing wave
  const int cw = wave & 3;                        // number of a copying wave
  int g = blockIdx.x;
  if (a.xgt > 0 && g < a.xg1) {  // XCD-aware order, as in the 256 x 256 kernel
    const int T = a.tblocks, GT = a.xgt, RC = a.xrc, TGc = T / GT;
    const int x = g & 7, l = g >> 3, tg = x % TGc, rc = x / TGc;
    g = ((l / GT) * RC + rc) * T + tg * GT + l % GT;
  }
  int ri = 0;
  for (int i = 1; i < a.nreg; ++i)
    if (g >= a.reg[i].wg0) ri = i;
  const Region& R = a.reg[ri];
  const int S = R.ksplit, rs = (g - R.wg0) / a.tblocks;
  const int rb = rs / S, slice = rs - rb * S;
  const int m0 = (g - R.wg0) % a.tblocks * kMidTok;
  const int rowend = R.row0 + R.rows, rblk = R.row0 + rb * kMidRows;
  const int K = R.kend * ES, kbound = R.kbound * ES;  // bytes of an activation row
  const int n_sp = (kbound + 127) / 128, n_de = (K - kbound + 127) / 128;
  const int nch_sp = (n_sp + 3) / 4, nch_de = (n_de + 3) / 4;
  // this slice's steps: 2:4 steps [s0, s0 + ns), then dense steps [d0, d0 + nd)
  const int c0 = S > 1 ? R.cut[slice] : 0, c1 = S > 1 ? R.cut[slice + 1] : nch_sp + nch_de;
  const int s0 = min(4 * c0, n_sp), ns = min(4 * c1, n_sp) - s0;
  const int d0 = min(4 * max(c0 - nch_sp, 0), n_de), nd = min(4 * max(c1 - nch_sp, 0), n_de) - d0;
  const int n = ns + nd;

  extern __shared__ __attribute__((aligned(1024))) uint8_t mid_lds[];
  const MatDesc& MD = a.mat[R.mat];
  const __amdgpu_buffer_rsrc_t rx = rsrc(a.X, a.x_bytes), rv = rsrc(MD.values, MD.v_bytes), rm = rsrc(MD.meta, MD.m_bytes),
                               rd = rsrc(MD.dense, MD.d_bytes);
  v4f acc[RPW][TC];
#pragma unroll
  for (int t = 0; t < RPW; ++t)
#pragma unroll
    for (int c = 0; c < TC; ++c) acc[t][c] = (v4f){0.f, 0.f, 0.f, 0.f};

  // Copying wave cw: four activation blocks of 8 tokens, the weight blocks of row tiles 2 cw
  // and 2 cw + 1 and, in 2:4 steps, waves 0 and 1 the metadata pieces of row tiles 4 cw ..
  // 4 cw + 3.
  auto run_copies = [&]() __attribute__((always_inline)) {
    constexpr int XL = 4;
    const int xb = 16 * ((lane & 7) ^ (lane >> 4));  // column of this lane's 16 bytes in a step; odd blocks xb ^ 64
    uint32_t xo[XL], vo[2], dof[4], mo = kOOB;  // loop-invariant per-lane offsets, kOOB past M or the region
    int vc = 0;  // row-major values: the byte of this lane's piece inside the step
#pragma unroll
    for (int i = 0; i < XL; ++i) {
      const int m = m0 + 8 * (XL * cw + i) + (lane >> 3);
      xo[i] = m < a.M ? (uint32_t)((int64_t)m * a.ldx_b + (xb ^ (64 * (i & 1)))) : kOOB;
    }
    if constexpr (TL) {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int r0 = rblk + 16 * (2 * cw + u);
        vo[u] = r0 < rowend ? (uint32_t)(r0 / 16) * (uint32_t)nch_sp * 4096u + 16u * lane : kOOB;
        dof[2 * u] = r0 < rowend && r0 >= R.dense_row_off
                         ? (uint32_t)((r0 - R.dense_row_off) / 16) * (uint32_t)nch_de * 8192u + 16u * lane
                         : kOOB;
        dof[2 * u + 1] = dof[2 * u];
      }
      const int r0 = rblk + 16 * (4 * cw + (lane >> 4));
      if (cw < 2 && r0 < rowend) mo = (uint32_t)(r0 / 16) * (uint32_t)nch_sp * 1024u + 16u * li;
    } else {
      // values: lane l the 16-byte piece (l % 4) ^ (row / 4 % 4) of row l / 4 of the tile, so
      // that the four lane groups' reads of 16 rows meet in no bank; dense rows like the
      // activations, eight per block; metadata: lane l word l % 2 of row l / 2 of 32
      vc = 16 * ((lane & 3) ^ ((lane >> 4) & 3));
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int r = rblk + 16 * (2 * cw + u) + (lane >> 2);
        vo[u] = r < rowend ? (uint32_t)(r * a.v_ld_b + vc) : kOOB;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int r = rblk + 32 * cw + 8 * u + (lane >> 3);
        dof[u] = r < rowend && r >= R.dense_row_off
                     ? (uint32_t)((r - R.dense_row_off) * a.d_ld_b + (kbound - R.dense_col_off * ES) + (xb ^ (64 * (u & 1))))
                     : kOOB;
      }
      const int r = rblk + 32 * cw + (lane >> 1);
      if (r < rowend) mo = (uint32_t)(r * a.m_ld_b + 4 * (lane & 1));
    }
    auto copy = [&](int s, int k) __attribute__((always_inline)) {  // ring step s into stage k
      if (s >= n) return;
      uint8_t* const st = mid_lds + k * SB;
      const bool sp = s < ns;
      const int ss = sp ? s0 + s : d0 + s - ns;  // step inside its kind
      const int ks = sp ? 128 * ss : kbound + 128 * ss, ke = sp ? kbound : K;
      const bool part = ks + 128 > ke;  // the kind's last, partial step
      static_for<XL>([&](auto i_const) {
        constexpr int i = decltype(i_const)::value;
        uint32_t off = xo[i];
        if (part) off = ks + (xb ^ (64 * (i & 1))) < ke ? off : kOOB;
        lds_load16<0>(rx, st + (XL * cw + i) * 1024, off, ks);
      });
      if constexpr (TL) {
        if (sp) {
          lds_load16<kTiledNT>(rv, st + XB + (2 * cw) * 1024, vo[0], 1024 * ss);
          lds_load16<kTiledNT>(rv, st + XB + (2 * cw + 1) * 1024, vo[1], 1024 * ss);
          if (cw < 2) lds_load16<kTiledNT>(rm, st + XB + 8192 + cw * 1024, mo, 256 * ss);
        } else {
#pragma unroll
          for (int u = 0; u < 4; ++u)
            lds_load16<kTiledNT>(rd, st + XB + (4 * cw + u) * 1024, dof[u], 2048 * ss + 1024 * (u & 1));
        }
      } else if (sp) {  // rows are not padded: a partial step's weights past the region read as zeros too
#pragma unroll
        for (int u = 0; u < 2; ++u)
          lds_load16<kNT>(rv, st + XB + (2 * cw + u) * 1024, part && ks + 2 * vc >= ke ? kOOB : vo[u], 64 * ss);
        lds_load4<kNT>(rm, st + XB + 8192 + cw * 256, part && ks + 64 * (lane & 1) >= ke ? kOOB : mo, 8 * ss);
      } else {
        static_for<4>([&](auto u_const) {
          constexpr int u = decltype(u_const)::value;
          uint32_t off = dof[u];
          if (part) off = ks + (xb ^ (64 * (u & 1))) < ke ? off : kOOB;
          lds_load16<kNT>(rd, st + XB + (4 * cw + u) * 1024, off, 128 * ss);
        });
      }
    };
    // Wait until the copies of all but the last k steps in flight have landed.  A 2:4 step is
    // XL + 3 loads (tiled: XL + 2 on waves 2 and 3), a dense one XL + 4; where both are in
    // flight the smaller count waits longer than needed.
    auto wait_steps = [&](bool sp, int k) __attribute__((always_inline)) {
      static_for<NS>([&](auto i_const) {
        constexpr int i = NS - 1 - decltype(i_const)::value;
        if (k == i) {
          if (!sp)
            wait_vm<i * (XL + 4)>();
          else if (!TL || cw < 2)
            wait_vm<i * (XL + 3)>();
          else
            wait_vm<i * (XL + 2)>();
        }
      });
    };
    static_for<NS>([&](auto s_const) { copy(decltype(s_const)::value, decltype(s_const)::value); });
    int k = 0;  // stage of step s
    for (int s = 0; s < n; ++s) {
      const bool sp = s < ns;
      if (s == 0 || s == ns) {  // the first step of a kind
        wait_steps(sp, min(n - 1 - s, NS - 1));
        barrier_lgkm0();
      }
      wait_steps(sp, max(min(n - 2 - s, NS - 2), 0));
      barrier_lgkm0();
      copy(s + NS, k);
      k = k == NS - 1 ? 0 : k + 1;
    }
  };

  const int xc0 = (lq ^ ((li >> 1) & 7)) << 4, xc1 = ((4 + lq) ^ ((li >> 1) & 7)) << 4;
  const int xrow = (16 * TC * wc + li) * 128;
  auto run = [&](auto act_const) __attribute__((always_inline)) {
    constexpr bool ACT = decltype(act_const)::value;
    int k = 0, s = 0;  // stage of step s, step
    // steps [s, hi) of one kind
    auto loop = [&](auto sp_const, const int hi) __attribute__((always_inline)) {
      constexpr bool SP = decltype(sp_const)::value;
      if (s >= hi) return;
      v8i bq[2][TC];
      v4i alo[2][RPW], ahi[2][RPW];
      int aix[2][RPW];
      auto read_b = [&](auto p_const, auto c_const, const uint8_t* st) __attribute__((always_inline)) {
        constexpr int p = decltype(p_const)::value, c = decltype(c_const)::value;
        const uint8_t* xs = st + xrow + c * 2048;
        bq[p][c] = cat8(*reinterpret_cast<const v4i*>(xs + xc0), *reinterpret_cast<const v4i*>(xs + xc1));
      };
      auto read_a = [&](auto p_const, auto t_const, const uint8_t* st) __attribute__((always_inline)) {
        constexpr int p = decltype(p_const)::value, t = decltype(t_const)::value;
        const uint8_t* ws = st + XB;
        if constexpr (SP && TL) {
          alo[p][t] = *reinterpret_cast<const v4i*>(ws + (RPW * wr + t) * 1024 + 16 * lane);
          aix[p][t] = *reinterpret_cast<const int*>(ws + 8192 + (RPW * wr + t) * 256 + 16 * li + 4 * lq);
        } else if constexpr (SP) {
          alo[p][t] = *reinterpret_cast<const v4i*>(ws + (RPW * wr + t) * 1024 + 64 * li + 16 * (lq ^ (li >> 2)));
          aix[p][t] = *reinterpret_cast<const int*>(ws + 8192 + (RPW * wr + t) * 128 + 8 * li + 4 * (lq >> 1));
        } else if constexpr (!TL) {
          alo[p][t] = *reinterpret_cast<const v4i*>(ws + (RPW * wr + t) * 2048 + 128 * li + xc0);
          ahi[p][t] = *reinterpret_cast<const v4i*>(ws + (RPW * wr + t) * 2048 + 128 * li + xc1);
        } else {
          alo[p][t] = *reinterpret_cast<const v4i*>(ws + (RPW * wr + t) * 2048 + 16 * lane);
          ahi[p][t] = *reinterpret_cast<const v4i*>(ws + (RPW * wr + t) * 2048 + 1024 + 16 * lane);
        }
      };
      typedef std::integral_constant<int, 0> Z;
      barrier_lgkm0();  // the first step has landed
      if constexpr (ACT) {
        static_for<TC>([&](auto c) { read_b(Z(), c, mid_lds + k * SB); });
        static_for<RPW>([&](auto t) { read_a(Z(), t, mid_lds + k * SB); });
      }
      auto step = [&](auto p_const) __attribute__((always_inline)) {
        constexpr int P = decltype(p_const)::value;
        typedef std::integral_constant<int, 1 - P> Q;
        k = k == NS - 1 ? 0 : k + 1;
        const uint8_t* const sn = mid_lds + k * SB;
        barrier_lgkm0();  // this step's fragments are in registers, the next step has landed
        __builtin_amdgcn_sched_barrier(0);
        static_for<RPW>([&](auto t_const) {
          constexpr int t = decltype(t_const)::value;
          // after the kind's last step these read a stage in flight or of the other kind; unused
          if constexpr (ACT) {
            read_a(Q(), t_const, sn);
            read_b(Q(), std::integral_constant<int, 2 * t>(), sn);
            read_b(Q(), std::integral_constant<int, 2 * t + 1>(), sn);
#pragma unroll
            for (int c = 0; c < TC; ++c) {
              if constexpr (SP) {
                acc[t][c] = mma_sparse(alo[P][t], bq[P][c], acc[t][c], TL ? aix[P][t] : (int)((uint32_t)aix[P][t] >> (16 * (lq & 1))), Dt());
              } else if constexpr (TL) {
                acc[t][c] = mma_dense(cat8(alo[P][t], ahi[P][t]), bq[P][c], acc[t][c], Dt());
              } else {
                acc[t][c] = mma_dense(cat8(alo[P][t], alo[P][t]), bq[P][c], acc[t][c], Dt());
                acc[t][c] = mma_dense(cat8(ahi[P][t], ahi[P][t]), __builtin_shufflevector(bq[P][c], bq[P][c], 4, 5, 6, 7, 4, 5, 6, 7),
                                      acc[t][c], Dt());
              }
            }
          }
          __builtin_amdgcn_sched_barrier(0);
        });
        ++s;
      };
      for (; s + 2 <= hi;) {
        step(std::integral_constant<int, 0>());
        step(std::integral_constant<int, 1>());
      }
      if (s < hi) step(std::integral_constant<int, 0>());
      xdl_fence();
    };
    loop(std::true_type(), ns);
    loop(std::false_type(), n);
  };
  const bool idle = copies || m0 + 16 * TC * wc >= a.M;  // no tokens: the wave only keeps the barriers
  if (copies)
    run_copies();
  else if (idle)
    run(std::false_type());
  else
    run(std::true_type());

  if (S > 1) {  // unscaled fp32 partials of this K slice, one 16-byte store where it can
    if (idle) return;
#pragma unroll
    for (int t = 0; t < RPW; ++t)
#pragma unroll
      for (int c = 0; c < TC; ++c) {
        const int m = m0 + 16 * (TC * wc + c) + li, n0 = rblk + 16 * (RPW * wr + t) + 4 * lq;
        if (m >= a.M || n0 >= rowend) continue;
        float* pp = a.part + ((int64_t)slice * a.M + m) * a.N + n0;
        if (a.part_vec && n0 + 3 < rowend) {
          *reinterpret_cast<v4f*>(pp) = acc[t][c];
        } else {
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (n0 + r < rowend) pp[r] = acc[t][c][r];
        }
      }
    return;
  }
  const bool via_lds = !a.out_f32 && ((uintptr_t)MD.Y % 16 == 0) && (MD.ldy % 8 == 0) && (rblk % 8 == 0);
  EpiScales<RPW, TC> es;
  if (!idle) epi_scales(es, MD.sw, a.sx, a.M, rblk + 16 * RPW * wr + 4 * lq, m0 + 16 * TC * wc + li, rowend);
  if (!via_lds) {
    if (idle) return;
#pragma unroll
    for (int t = 0; t < RPW; ++t)
#pragma unroll
      for (int c = 0; c < TC; ++c) {
        const int m = m0 + 16 * (TC * wc + c) + li, n0 = rblk + 16 * (RPW * wr + t) + 4 * lq;
        if (m < a.M && n0 < rowend) store4e(MD.Y, MD.ldy, MD.sw != nullptr, MD.vec_store, a, es, t, c, acc[t][c], m, n0, rowend);
      }
    return;
  }
  barrier_vm_lgkm0<0>();  // every wave's last operand reads and copies are done
  if (!idle) out_tile_write<RPW, TC, kMidRows / 8>(mid_lds, acc, es, MD.sw != nullptr, wr, wc, li, lq);
  barrier_vm_lgkm0<0>();
  out_tile_store<kMidRows / 8, 768>(mid_lds, kMidTok, m0, a.M, rblk, rowend, MD.Y, MD.ldy);
}

}  // namespace

hipError_t launch_mid(int dtype, const GemmArgs& a, hipStream_t s) {
  static_assert(kMidLds <= 160 * 1024, "LDS of a CU");
  // fp8 row-major weights go to the 128 x 256 kernel, bf16 ones have no tiled layout
  if ((dtype == kFP8) != (a.tiled != 0)) return hipErrorInvalidValue;
  for (int i = 0; i < a.nreg; ++i)
    if (a.reg[i].ksplit > 1 && !a.part) return hipErrorInvalidValue;
  auto k = dtype == kFP8 ? spense_gemm_mid_kernel<kFP8> : spense_gemm_mid_kernel<kBF16>;
  hipError_t e = set_big_lds(k, 1, dtype == kFP8 ? 0 : 1, kMidLds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k, dim3(a.groups), dim3(768), kMidLds, s, a);
  return hipGetLastError();
}

}  // namespace spense
