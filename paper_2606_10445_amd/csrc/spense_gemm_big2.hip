// The 256 x 256 large-M kernel (spense_gemm.hip has the overview of all GEMM kernels).
#include "spense_gemm_device.h"

namespace spense {
namespace {

// ---------------------------------------------------------------- large-M kernel, 256 x 256 tiles
// Both operands through LDS as in spense_gemm_big_kernel, with twice the rows per
// workgroup and per wave: a workgroup computes 256 weight rows x 256 tokens, its 8 waves a
// grid of 2 row halves x 4 token quarters, each wave 128 rows (8 row tiles) x 64 tokens (4
// token tiles, 128 accumulators).  Each B fragment read from LDS feeds 8 MMAs, each A
// fragment 4.  fp8 weights in the tiled layout, bf16 weights row-major.
//
// Tiles of fewer tokens (128-token tail tiles, 192-token blocks, the block that M ends in): the
// four waves of a row half share them, 32, 48 or 64 each (NT = 2, 3, 4 token tiles).  With 64 each
// and waves without tokens, a 128-token tile took 0.9 of a whole one's time (one wave a SIMD hides
// no latency, and in dense steps its slot stays as long) and a 192-token one all of it: gate / up M
// = 540 / 640 88 / 90 us, now 83 / 85.
//
// What bounds a step (all measured on MI355X): the CU's load path moves about 57 bytes per
// clock from L2 and a load instruction costs at least ~18 clocks however few bytes it moves,
// so every copy moves 1 KB; a wave reads LDS at ~25 bytes per clock (16 bytes a lane) alone on
// its SIMD and two at ~45 together; copies into LDS and reads from it do not slow each other;
// the matrix cores take ~24 clocks per 2:4 and ~45 per dense instruction on random data with
// every CU busy (17 and 32 on zeros: the clock gives way).  A step's copies, reads and MMAs
// are each close to its MMA time, so they have to run at once, and the two kinds of steps do
// that in two ways:
//   - 2:4 steps (52 KB of copies, 147 KB of reads, 256 MMAs): every wave reads the next
//     step's B fragments into a second register set and the A fragments two row tiles ahead
//     between its MMAs, and spreads its copies over the step; one barrier per step, early in
//     it.  With copies and B reads bunched in the second half of the step it took 0.85 us on
//     5120 x 25600 at M = 2048, spread 0.80 (0.95 with all reads at the start of the step).
//   - dense steps (64 KB, 192 KB, 256 MMAs of twice the length): no registers for a second B
//     set and whole A tiles, so the waves of a SIMD take turns: waves 4-7 run one slot behind
//     waves 0-3, and while one half issues the 32 MMAs of a step back to back, the other reads
//     its fragments and issues its copies.  gate/up with every row dense, M = 2048: 259 ->
//     231 us, 2.3 PFLOP/s, in a step the random-data MMA rate above; M = 300 66 -> 54 us.
// Measured, before (both kinds: reads one row tile ahead, copies in two bunches) -> now, us, on
// one box: gate/up M = 300 / 540 / 640 / 1024 / 2048 64 / 81 / 86 / 109 / 201 -> 49 / 83 / 85 / 103 /
// 188; M = 2048 down 207 -> 179, o 74 -> 65, q 70 -> 61.  bf16 (row-major weights, a step is 64 columns: the same bytes and
// MMA clocks), 128 x 128 kernel -> this one: 8192 x 5120 M = 2048 182 -> 108, 25600 x 5120
// M = 1024 / 2048 299 / 568 -> 185 / 380 (0.88 PFLOP/s).
//
// The activations have two stages (the B fragments of a step are in registers before its
// MMAs, so its stage is free again half a step in), the weights four (2:4, 20 KB each) or
// three (dense, 32 KB): they come from HBM or the MALL and need the longer lead.
constexpr int kB2Rows = 256, kB2Tokens = 256, kB2RowTiles = 16;
constexpr int kB2XSlot = kB2Tokens * 128;                            // activations of one step
constexpr int kB2SWgt = kB2RowTiles * 1024 + kB2RowTiles * 256;      // 2:4 values, metadata of one step
constexpr int kB2DWgt = kB2RowTiles * 2048;                          // both dense halves of one step
constexpr int kB2Lds = 2 * kB2XSlot + (4 * kB2SWgt > 3 * kB2DWgt ? 4 * kB2SWgt : 3 * kB2DWgt);

// MODE 1: a grouped launch (several weights sharing X and K): up to kMaxRegions regions, each
// reading its weight's buffers, output and scales from a.mat[R.mat].
// MODE 2: the gate / up pair (a.mat[0], a.mat[1], one geometry): a workgroup takes the same 128
// rows of both weights, row tiles 8 wr + [0, 4) of the 16 gate's and 8 wr + [4, 8) up's, so
// that each wave holds g and u of the same outputs and writes h = u silu(g) (fp32) and its row
// maxima.  G and U written in fp32 and read again cost a 25600 x 5120 pair 420 MB more per
// 2048 tokens than H does: GEMM and GLU quantisation 450 + 124 us, now 366 + 46 (the
// quantisation reads and writes 5.7 TB/s); the whole MLP at M = 256 142 -> 126 us.
// Keeps a kernel argument in its scalar registers: the compiler else loads it again where it is
// used, in the prologue's and the epilogue's branches one memory round trip after the other.
template <typename T>
__device__ __forceinline__ void keep_scalar(T& v) {
  asm volatile("" : "+s"(v));
}

enum { kB2Plain = 0, kB2Grouped = 1, kB2Glu = 2 };

template <int DT, int MODE>
__global__ __launch_bounds__(512) void spense_gemm_big2_kernel(GemmArgs a) {
  constexpr bool TL = DT == kFP8;  // tiled weights; bf16 reads the row-major layout
  constexpr int ES = Traits<DT>::ES;
  typedef std::integral_constant<int, DT> Dt;
  static_assert(TL || MODE == kB2Plain, "grouped and paired launches are fp8");
  constexpr bool GR = MODE == kB2Grouped, GL = MODE == kB2Glu;
  constexpr int kRows = GL ? kB2Rows / 2 : kB2Rows;  // weight rows of a tile (each of both weights)
  constexpr int RPW = 8;  // row tiles of a wave
  // the tile's first row of row tile r; the weight it belongs to is (r >> 2) & 1 in a pair
  auto tile_row = [](int r) __attribute__((always_inline)) { return 16 * (GL ? (r >> 3) * 4 + (r & 3) : r); };
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int li = lane & 15, lq = lane >> 4;
  const bool late = wave >= 4;  // dense steps: the half of the waves that runs one slot behind
  const int w4 = wave & 3, wr = wave >> 2, wc = w4;
  // Workgroups [0, hg0): 256 x 256 tiles, in the XCD-aware order when it is on.  From
  // hg0 on (dispatched last, so that they fill the tail of the grid): the row blocks
  // hrb0 .. of the last region as 256 x 128 tiles, hper per row block.
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
  const int rblk = R.row0 + rb * kRows;
  // tokens of this tile: 256, or 192 (full tiles of a 192-token block), or 128 (half tiles), and
  // those that M ends before; its four waves a row half take 16 NT of them each
  const int ntok = min(half ? kB2Tokens / 2 : (a.btok > 0 ? a.btok : kB2Tokens), a.M - m0);
  const int K = R.kend * ES, kbound = R.kbound * ES;  // bytes of an activation row
  uint32_t ldx = (uint32_t)a.ldx_b;  // X spans less than 2 GiB
  keep_scalar(ldx);
  int dense_row_off = R.dense_row_off;
  keep_scalar(dense_row_off);

  extern __shared__ __attribute__((aligned(1024))) uint8_t big_lds[];
  const MatDesc& MD = a.mat[GR ? R.mat : 0];
  // a pair: the weight whose row tiles this wave copies (values 2 wave, 2 wave + 1, metadata
  // 4 wave .. 4 wave + 3, dense 4 w4 .. 4 w4 + 3)
  const MatDesc& MV = GL ? a.mat[(wave >> 1) & 1] : MD;
  const MatDesc& MM = GL ? a.mat[wave & 1] : MD;
  const __amdgpu_buffer_rsrc_t rx = rsrc(a.X, a.x_bytes),
                               rv = GR || GL ? rsrc(MV.values, MV.v_bytes) : rsrc(a.values, a.v_bytes),
                               rm = GR || GL ? rsrc(MM.meta, MM.m_bytes) : rsrc(a.meta, a.m_bytes),
                               rd = GR || GL ? rsrc(MM.dense, MM.d_bytes) : rsrc(a.dense, a.d_bytes);
  const int n_sp = (kbound + 127) / 128, n_de = (K - kbound + 127) / 128;
  const int nch_sp = (n_sp + 3) / 4, nch_de = (n_de + 3) / 4;

  uint8_t* const sx = big_lds;                 // two activation stages
  uint8_t* const sw = big_lds + 2 * kB2XSlot;  // weight stages: values then metadata (four), or both dense halves (three)

  auto tile = [&](auto nt_const) __attribute__((always_inline)) {
  constexpr int NT = decltype(nt_const)::value;  // token tiles of a wave
  v4f acc[RPW][NT];
#pragma unroll
  for (int t = 0; t < RPW; ++t)
#pragma unroll
    for (int c = 0; c < NT; ++c) acc[t][c] = (v4f){0.f, 0.f, 0.f, 0.f};

  const uint8_t* const xr = sx + (16 * NT * wc + li) * 128;  // (r >> 1) & 7 of the wave's rows r is (li >> 1) & 7
  const int xc0 = (lq ^ ((li >> 1) & 7)) << 4, xc1 = ((4 + lq) ^ ((li >> 1) & 7)) << 4;

  // The 2:4 steps.
  auto run_sparse = [&]() __attribute__((always_inline)) {
    constexpr int NW = 4, AQ = 4, AD = 2, TB = 2;  // weight stages, A register sets, row tiles read ahead, barrier
    // This wave's copies (loop-invariant per-lane offsets, kOOB for rows past M or row tiles
    // past the region): activation blocks 4 wave .. 4 wave + 3 (8 tokens each), the values of
    // row tiles 2 wave and 2 wave + 1 and, waves 0-3, the metadata pieces of row tiles 4 wave
    // .. 4 wave + 3 (lane l: 16 bytes of tile 4 wave + l / 16, 256 s bytes in for step s).
    const int xb = 16 * ((lane & 7) ^ (lane >> 4));  // column of this lane's 16 bytes in a step; odd blocks xb ^ 64
    uint32_t xo[4], wo[2], mo = kOOB;
    // row-major values: lane l takes the 16-byte piece (l % 4) ^ (row / 4 % 4) of row l / 4 of
    // its tile, so that the four lane groups' reads of 16 rows meet in no bank; metadata: word
    // l % 2 of row l / 2 of the wave's 32
    const int vc = 16 * ((lane & 3) ^ ((lane >> 4) & 3));
    const bool meta_wave = !TL || wave < 4;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = 32 * wave + 8 * i + (lane >> 3), m = m0 + r;
      xo[i] = m < a.M && r < ntok ? (uint32_t)m * ldx + (xb ^ (64 * (i & 1))) : kOOB;
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int r0 = rblk + tile_row(2 * wave + u) + (TL ? 0 : lane >> 2);
      wo[u] = r0 >= rowend ? kOOB
              : TL         ? (uint32_t)(r0 / 16) * (uint32_t)nch_sp * 4096u + 16u * lane
                           : (uint32_t)(r0 * a.v_ld_b + vc);
    }
    if constexpr (!TL) {
      const int r0 = rblk + 32 * wave + (lane >> 1);
      if (r0 < rowend) mo = (uint32_t)(r0 * a.m_ld_b + 4 * (lane & 1));
    } else if (wave < 4) {
      const int r0 = rblk + tile_row(4 * wave + (lane >> 4));
      if (r0 < rowend) mo = (uint32_t)(r0 / 16) * (uint32_t)nch_sp * 1024u + 16u * li;
    }
    // A copy past the last step reads (and writes) zeros, so that every step issues the same
    // number of loads.
    auto x_copy = [&](auto i_const, int s, int st) __attribute__((always_inline)) {
      constexpr int i = decltype(i_const)::value;
      uint32_t off = xo[i];
      if (128 * s + 128 > kbound) off = 128 * s + (xb ^ (64 * (i & 1))) < kbound ? off : kOOB;
      lds_load16<0>(rx, sx + st * kB2XSlot + (4 * wave + i) * 1024, off, 128 * s);
    };
    auto w_copy = [&](auto u_const, int s, int k) __attribute__((always_inline)) {
      constexpr int u = decltype(u_const)::value;
      if constexpr (TL)
        lds_load16<kTiledNT>(rv, sw + k * kB2SWgt + (2 * wave + u) * 1024, s < n_sp ? wo[u] : kOOB, 1024 * s);
      else  // rows are not padded: weights past the region read as zeros too
        lds_load16<kNT>(rv, sw + k * kB2SWgt + (2 * wave + u) * 1024, 128 * s + 2 * vc < kbound ? wo[u] : kOOB, 64 * s);
    };
    auto m_copy = [&](int s, int k) __attribute__((always_inline)) {
      if constexpr (!TL)
        lds_load4<kNT>(rm, sw + k * kB2SWgt + kB2RowTiles * 1024 + wave * 256,
                       128 * s + 64 * (lane & 1) < kbound ? mo : kOOB, 8 * s);
      else if (wave < 4)
        lds_load16<kTiledNT>(rm, sw + k * kB2SWgt + kB2RowTiles * 1024 + wave * 1024, s < n_sp ? mo : kOOB, 256 * s);
    };
    auto wait_w = [&](auto n_const) __attribute__((always_inline)) {  // all but the last n steps' weight copies
      constexpr int n = decltype(n_const)::value;
      if (meta_wave)
        wait_vm<3 * n>();
      else
        wait_vm<2 * n>();
    };
    v8i bq[2][NT];
    v4i av[AQ];
    int aix[AQ];
    auto read_b = [&](v8i& b, int st, int c) __attribute__((always_inline)) {
      const uint8_t* p = xr + st * kB2XSlot + c * 2048;
      b = cat8(*reinterpret_cast<const v4i*>(p + xc0), *reinterpret_cast<const v4i*>(p + xc1));
    };
    auto read_a = [&](auto q_const, int t, int k) __attribute__((always_inline)) {
      constexpr int q = decltype(q_const)::value;
      const uint8_t* const wt = sw + k * kB2SWgt + (RPW * wr + t) * 1024;
      const uint8_t* const mt = sw + k * kB2SWgt + kB2RowTiles * 1024;
      av[q] = *reinterpret_cast<const v4i*>(wt + (TL ? 16 * lane : 64 * li + 16 * (lq ^ (li >> 2))));
      aix[q] = *reinterpret_cast<const int*>(TL ? mt + (RPW * wr + t) * 256 + 16 * li + 4 * lq
                                                : mt + (RPW * wr + t) * 128 + 8 * li + 4 * (lq >> 1));
    };
    static_for<4>([&](auto i) { x_copy(i, 0, 0); });
    static_for<2>([&](auto u) { w_copy(u, 0, 0); });
    m_copy(0, 0);
    static_for<4>([&](auto i) { x_copy(i, 1, 1); });
    static_for<2>([&](auto u) { w_copy(u, 1, 1); });
    m_copy(1, 1);
    static_for<2>([&](auto u) { w_copy(u, 2, 2); });
    if (meta_wave)
      wait_vm<4 + 3 + 2>();
    else
      wait_vm<4 + 2 + 2>();
    barrier_lgkm0();
    static_for<NT>([&](auto c) { read_b(bq[0][decltype(c)::value], 0, decltype(c)::value); });
    static_for<AD>([&](auto t) { read_a(t, decltype(t)::value, 0); });
    int k = 0;  // weight stage of step s
    // Step s with the B fragments of set P (its activation stage too).  Before row tile TB, a
    // barrier: the next step's blocks have landed for every wave, and the stages of this
    // step's activations and the last step's weights are free.  After it the next step's B
    // fragments are read between the MMAs, and the copies of step s + 2 (activations) and
    // s + 3 (weights) go out, spread over the step.
    auto step = [&](auto p_const, const int s) __attribute__((always_inline)) {
      constexpr int P = decltype(p_const)::value;
      const int kn = k == NW - 1 ? 0 : k + 1, kp = k == 0 ? NW - 1 : k - 1;
      static_for<RPW>([&](auto t_const) {
        constexpr int t = decltype(t_const)::value;
        if constexpr (t == 0) m_copy(s + 2, k < 2 ? k + 2 : k - 2);
        if constexpr (t == TB) {
          wait_w(std::integral_constant<int, 1>());
          asm volatile("s_barrier" ::: "memory");
          __builtin_amdgcn_sched_barrier(0);
        }
        typedef std::integral_constant<int, (t + AD) % AQ> Q;
        if constexpr (t + AD < RPW)
          read_a(Q(), t + AD, k);
        else
          read_a(Q(), t + AD - RPW, kn);
        if constexpr (t >= 3 && t < 3 + NT) read_b(bq[1 - P][t - 3], 1 - P, t - 3);
        if constexpr (t >= TB && t < TB + 4) x_copy(std::integral_constant<int, t - TB>(), s + 2, P);
        if constexpr (t >= 6) w_copy(std::integral_constant<int, t - 6>(), s + 3, kp);
        constexpr int q = t % AQ;
#pragma unroll
        for (int c = 0; c < NT; ++c)
          acc[t][c] = mma_sparse(av[q], bq[P][c], acc[t][c], TL ? aix[q] : (int)((uint32_t)aix[q] >> (16 * (lq & 1))), Dt());
        __builtin_amdgcn_sched_barrier(0);
      });
      k = kn;
    };
    int s = 0;
    for (; s + 2 <= n_sp; s += 2) {
      step(std::integral_constant<int, 0>(), s);
      step(std::integral_constant<int, 1>(), s + 1);
    }
    if (s < n_sp) step(std::integral_constant<int, 0>(), s);
    xdl_fence();
    barrier_vm_lgkm0<0>();  // every wave is done with the stages, and no copy is in flight
  };

  // The dense steps.  Waves 0-3 copy the activations (eight blocks each, of tokens [64 w4,
  // 64 w4 + 64)), waves 4-7 the weights (both halves of row tiles 4 w4 .. 4 w4 + 3).
  auto run_dense = [&]() __attribute__((always_inline)) {
    const int xb = 16 * ((lane & 7) ^ (lane >> 4));
    uint32_t lo[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      if (late) {
        // row-major rows like the activations, eight per block
        const int r0 = rblk + (TL ? tile_row(4 * w4 + (i >> 1)) : 64 * w4 + 8 * i + (lane >> 3));
        lo[i] = !(r0 < rowend && r0 >= dense_row_off) ? kOOB
                : TL ? (uint32_t)((r0 - dense_row_off) / 16) * (uint32_t)nch_de * 8192u + 16u * lane
                     : (uint32_t)((r0 - dense_row_off) * a.d_ld_b + (kbound - R.dense_col_off * ES) + (xb ^ (64 * (i & 1))));
      } else {
        const int r = 64 * w4 + 8 * i + (lane >> 3), m = m0 + r;
        lo[i] = m < a.M && r < ntok ? (uint32_t)m * ldx + kbound + (xb ^ (64 * (i & 1))) : kOOB;
      }
    }
    auto x_copy = [&](int s) __attribute__((always_inline)) {
      static_for<8>([&](auto i_const) {
        constexpr int i = decltype(i_const)::value;
        uint32_t off = lo[i];
        if (kbound + 128 * s + 128 > K) off = kbound + 128 * s + (xb ^ (64 * (i & 1))) < K ? off : kOOB;
        lds_load16<0>(rx, sx + (s & 1) * kB2XSlot + (8 * w4 + i) * 1024, off, 128 * s);
      });
    };
    auto w_copy = [&](int s, int k) __attribute__((always_inline)) {
      static_for<8>([&](auto i_const) {
        constexpr int i = decltype(i_const)::value;
        if constexpr (TL) {
          lds_load16<kTiledNT>(rd, sw + k * kB2DWgt + (8 * w4 + i) * 1024, lo[i], 2048 * s + 1024 * (i & 1));
        } else {
          uint32_t off = lo[i];
          if (kbound + 128 * s + 128 > K) off = kbound + 128 * s + (xb ^ (64 * (i & 1))) < K ? off : kOOB;
          lds_load16<kNT>(rd, sw + k * kB2DWgt + (8 * w4 + i) * 1024, off, 128 * s);
        }
      });
    };
    if (!late) {
      x_copy(0);
      wait_vm<0>();
    } else {
      w_copy(0, 0);
      if (n_de > 1) {
        w_copy(1, 1);
        wait_vm<8>();
      } else {
        wait_vm<0>();
      }
    }
    barrier_lgkm0();
    if (late) barrier_lgkm0();
    int k = 0;  // weight stage of step s (activation stage s % 2)
    for (int s = 0; s < n_de; ++s) {
      v8i bq[NT], av[RPW];
      const uint8_t* wl = sw + k * kB2DWgt + (RPW * wr) * 2048 + (TL ? 16 * lane : 128 * li);
      const int wc0 = TL ? 0 : xc0, wc1 = TL ? 1024 : xc1;
#pragma unroll
      for (int c = 0; c < NT; ++c) {
        const uint8_t* p = xr + (s & 1) * kB2XSlot + c * 2048;
        bq[c] = cat8(*reinterpret_cast<const v4i*>(p + xc0), *reinterpret_cast<const v4i*>(p + xc1));
      }
#pragma unroll
      for (int t = 0; t < RPW; ++t)
        av[t] = cat8(*reinterpret_cast<const v4i*>(wl + t * 2048 + wc0), *reinterpret_cast<const v4i*>(wl + t * 2048 + wc1));
      __builtin_amdgcn_sched_barrier(0);
      // activations of step s + 1 (awaited after this step's MMAs), weights of step s + 2
      if (!late) {
        if (s + 1 < n_de) x_copy(s + 1);
      } else if (s + 2 < n_de) {
        w_copy(s + 2, k == 0 ? 2 : k - 1);
        wait_vm<8>();
      } else {
        wait_vm<0>();
      }
      barrier_lgkm0();
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_setprio(1);
#pragma unroll
      for (int t = 0; t < RPW; ++t)
#pragma unroll
        for (int c = 0; c < NT; ++c) {
          acc[t][c] = mma_dense(av[t], bq[c], acc[t][c], Dt());
          if constexpr (!TL)
            acc[t][c] = mma_dense(__builtin_shufflevector(av[t], av[t], 4, 5, 6, 7, 4, 5, 6, 7),
                                  __builtin_shufflevector(bq[c], bq[c], 4, 5, 6, 7, 4, 5, 6, 7), acc[t][c], Dt());
        }
      __builtin_amdgcn_s_setprio(0);
      __builtin_amdgcn_sched_barrier(0);
      if (!late) wait_vm<0>();
      barrier_lgkm0();
      k = k == 2 ? 0 : k + 1;
    }
    if (!late) barrier_lgkm0();
    xdl_fence();
  };

  if (n_sp > 0) run_sparse();
  if (n_de > 0) run_dense();
  // bf16 output with 16-byte aligned rows leaves through LDS as whole token rows
  // (out_tile_write)
  const bool via_lds = !GL && !a.out_f32 && ((uintptr_t)MD.Y % 16 == 0) && (MD.ldy % 8 == 0) && (rblk % 8 == 0);
  const int mw = m0 + 16 * NT * wc + li;
  if constexpr (GL) {
    const float* const sg = a.mat[0].sw;
    const float* const su = a.mat[1].sw;
    const int nw = rblk + 64 * wr + 4 * lq;
    EpiScales<RPW / 2, NT> eg;
    EpiScales<RPW / 2, 1> eu;
    epi_scales(eg, sg, a.sx, a.M, nw, mw, rowend);
    epi_scales(eu, su, nullptr, a.M, nw, mw, rowend);
    // the row block's number over both regions: its two slots of the row maxima
    const int slot = 2 * (R.wg0 / a.tblocks + rb) + wr;
#pragma unroll
    for (int c = 0; c < NT; ++c) {
      const int m = mw + 16 * c;
      float tmax = 0.0f;
#pragma unroll
      for (int t = 0; t < RPW / 2; ++t) {
        const int n0 = nw + 16 * t;
        float h[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          float gg = acc[t][c][r], uu = acc[t + RPW / 2][c][r];
          if (sg) gg = gg * eg.w[t][r];
          if (su) uu = uu * eu.w[t][r];
          h[r] = glu_silu(gg * eg.x[c], uu * eg.x[c]);
          if (n0 + r < rowend) tmax = fmaxf(tmax, fabsf(h[r]));
        }
        if (m < a.M && n0 < rowend) put4(MD.Y, MD.ldy, MD.vec_store, a, h, m, n0, rowend);
      }
      if (a.hmax) {
        tmax = fmaxf(tmax, __shfl_xor(tmax, 16, 64));
        tmax = fmaxf(tmax, __shfl_xor(tmax, 32, 64));
        if (lq == 0 && m < a.M) a.hmax[(int64_t)m * a.hmax_ld + slot] = tmax;
      }
    }
    return;
  }
  EpiScales<RPW, NT> es;
  epi_scales(es, MD.sw, a.sx, a.M, rblk + 16 * RPW * wr + 4 * lq, mw, rowend);
  if (!via_lds) {
    void* Y = MD.Y;
    int64_t ldy = MD.ldy;
    int vec_store = MD.vec_store;
    keep_scalar(Y);
    keep_scalar(ldy);
    keep_scalar(vec_store);
#pragma unroll
    for (int t = 0; t < RPW; ++t)
#pragma unroll
      for (int c = 0; c < NT; ++c) {
        const int m = mw + 16 * c;
        const int n0 = rblk + 16 * (RPW * wr + t) + 4 * lq;
        if (m < a.M && n0 < rowend) store4e(Y, ldy, MD.sw != nullptr, vec_store, a, es, t, c, acc[t][c], m, n0, rowend);
      }
    return;
  }
  barrier_vm_lgkm0<0>();  // every wave's last operand reads and copies are done
  out_tile_write<RPW, NT, kB2Rows / 8>(big_lds, acc, es, MD.sw != nullptr, wr, wc, li, lq);
  barrier_vm_lgkm0<0>();
  out_tile_store<kB2Rows / 8, 512>(big_lds, ntok, m0, a.M, rblk, rowend, MD.Y, MD.ldy);
  };
  if (ntok > 192)
    tile(std::integral_constant<int, 4>());
  else if (ntok > 128)
    tile(std::integral_constant<int, 3>());
  else
    tile(std::integral_constant<int, 2>());
}

}  // namespace

hipError_t launch_big2(int dtype, const GemmArgs& a, hipStream_t s) {
  static_assert(kB2Lds <= 160 * 1024, "LDS of a CU");
  // the planner sends row-major fp8 weights to the 128 x 256 kernel; bf16 has no tiled layout
  if ((dtype == kFP8) != (a.tiled != 0)) return hipErrorInvalidValue;
  const int mode = a.hmax_ld > 0 ? kB2Glu : (a.nmat > 1 ? kB2Grouped : kB2Plain);
  if ((mode == kB2Glu && a.nmat != 2) || (mode != kB2Plain && dtype != kFP8)) return hipErrorInvalidValue;
  auto k = dtype != kFP8        ? spense_gemm_big2_kernel<kBF16, kB2Plain>
           : mode == kB2Glu     ? spense_gemm_big2_kernel<kFP8, kB2Glu>
           : mode == kB2Grouped ? spense_gemm_big2_kernel<kFP8, kB2Grouped>
                                : spense_gemm_big2_kernel<kFP8, kB2Plain>;
  hipError_t e = set_big_lds(k, a.tiled ? 1 : 0, 2 + mode, kB2Lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k, dim3(a.groups), dim3(512), kB2Lds, s, a);
  return hipGetLastError();
}

}  // namespace spense
