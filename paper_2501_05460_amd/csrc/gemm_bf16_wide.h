// bf16 MFMA GEMM on large tiles with persistent workgroups:  C[M,N] = A[M,K] * W[N,K]^T with the fused epilogues.
//
// What bounds it: over a long K the chip's power, under which the clock falls to 1.5 to 2.05 GHz of 2.4; at K = 1024 as much the
// epilogue, in which all waves of the one workgroup a CU holds stand together (106496 rows: the matrix pipe is busy 63 to 67 %
// of a product, 56 % of a residual one, at 1.95 to 2.06 GHz).  The energy of a flop counts in both.  Hence
//   * v_mfma_f32_16x16x32_bf16, not v_mfma_f32_32x32x16_bf16: a register-resident loop on normal deviates runs 2.02
//     PFLOP/s with the first and 1.74 with the second (constant operands: both near 2.45).  An element's k-steps are added
//     in the same order inside the instruction: two 32x32x16 steps and one 16x16x32 step leave the same bits.
//   * the MFMAs of a k-step walk the wave's blocks in serpentine order: consecutive ones share an operand fragment
//     (such a loop on another card: 2.10 PFLOP/s, row-major 2.06, both operands new every time 1.95).
// A workgroup per CU walks the tile sequence.  Both operand slabs (64 deep) go from global memory straight into one of two
// LDS buffers; the fragments of a k-step (32 deep) are read while the MFMAs of the step before it run, so that a slab's
// buffer is free, and the slab after the next is fetched into it, as soon as the slab's first k-step is multiplied: the
// loads issue through the second k-step and are waited for behind the next slab's first, so that the first has nearly a slab's time to
// arrive (1.3 us, 1.6 to 1.9 over cold operands) and the last half of one; a slab costs one barrier.  Reads and loads sit one by one between the MFMAs.
// The loads past a tile's last slab fetch the next tile's first two.  A wave stages its part of the finished tile through
// LDS behind the buffers, 4 to 6 KiB at a time and without a workgroup barrier, so that global memory sees whole lines.
//
// Measured stand-alone beside the 32x32x16 kernels this replaces (us; on one card, random operands): 106496 rows, N x K
// 2048 x 1024 380 -> 339, value projection 204 -> 179, out-projection 283 -> 262, 4096 x 1024 with GELU 829 -> 730,
// 1024 x 4096 residual 838 -> 782; 8192^3 775 -> 706 (1.56 PFLOP/s); 10240 rows, 1152 x 4352 residual 101 -> 95.
// With the lines of a slab pair asked for ahead (`touch`) and bands of one width (us, operands cold as in a running encoder): 10240 rows,
// 1152 x 4352 residual, 256 x 192 tiles 111 -> 95; 106496 rows, 1024 x 4096 residual 790 -> 735, 1024 x 1024 residual 294 -> 276, 4096 x 1024
// with GELU 772 -> 745; 40960 rows, 9600 x 3200 1895 -> 1805, 12800 x 3200 with GELU 2595 -> 2490; 3200 x 12800 residual 2930 -> 2830.
// One line a row at a time gives two thirds of that; four lines, or two pairs ahead, the same or less.
// A slab of 256 x 256 reads 192 KiB of LDS and writes 64, as many cycles at 128 bytes each as its products take: 2200 cycles on a CU by
// itself, 2600 to 3000 with all of them at work under the power limit.
// Tried and not kept: both operands slab by slab in memory ([K / 64][rows][64], 1 to 3 % on top of the lines asked for ahead); the stream
// rows' lines asked for ahead of a last tile's epilogue (13312 rows, 1024 x 1024 residual 41 -> 50: they return in order, in front of the
// rows themselves); the direct loads in the first half or three quarters of their k-step (0 to + 4 %); four waves of 128 x 128 (a third fewer fragment reads: 8192^3 equal, K = 1024 2 to 6 % slower, their
// epilogue runs on half as many waves); a staggered start of the workgroups (residual products -1 to -5 %, FC1 + 1 %); a
// wait that leaves the epilogue's stores in flight over the next tile's first slab (equal).
#pragma once
#include <type_traits>

#include "kernels.h"

namespace epd {

namespace {

constexpr int BK = 64;
#define SWZ(row) (((row) >> 1) & 7)

template <int N, int I = 0, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<N, I + 1>(f);
  }
}

// Waves stand WAVES_M x WAVES_N, each on TM x TN blocks of 16 x 16.
template <int TM, int TN, int WAVES_M, int WAVES_N>
struct Wide {
  static constexpr int NT = 64 * WAVES_M * WAVES_N, WM = 16 * TM, WN = 16 * TN, ROWS = WM * WAVES_M, COLS = WN * WAVES_N;
  static constexpr int SLAB = (ROWS + COLS) * BK * 2;                 // bytes of a slab of both operands
  static constexpr int WM64 = (WM + 63) / 64 * 64;
  static constexpr int STG = WN * 64 > WM64 * 32 ? WN * 64 : WM64 * 32;   // staging bytes of a wave: 16 fp32 rows, 32 bf16 rows, or 16 features of the transposed store
  static constexpr size_t LDS = 2 * (size_t)SLAB + (size_t)STG * WAVES_M * WAVES_N;
  static_assert(LDS <= 160 * 1024, "LDS of a CU");
};

// DUAL (EPI_BIAS): tile columns from Npad on are a second product over the same activations, the value projection, whose tiles run
// with the operand roles of EPI_VT and leave through its store (GemmParams::n2).
// NEAR: the output goes THROUGH, stream rows are read without a hint (NEAR_OUT, NEAR_ROWS).  Compiled apart: with both ways in one kernel the residual
// one spills, and the others take 0.5 to 2 % longer at 104 slices.
template <int EPI, bool DUAL, int TM, int TN, int WAVES_M, int WAVES_N, bool NEAR>
__global__ __launch_bounds__(64 * WAVES_M * WAVES_N, 1) void k_gemm_bf16_wide(const GemmParams p, const int gm, const int gw,
                                                                              const int gn, const int n_tiles, const int ahead) {
  using S = Wide<TM, TN, WAVES_M, WAVES_N>;
  constexpr int NT = S::NT, WM = S::WM, WN = S::WN, ROWS = S::ROWS, COLS = S::COLS, SLAB = S::SLAB;
  constexpr int RPL = NT / 8;                       // rows covered by one direct load of the workgroup
  constexpr int LA = (ROWS + RPL - 1) / RPL, LB = COLS / RPL, LPS = LA + LB;
  constexpr bool PART = ROWS % RPL != 0;            // the last load of the activations is the first waves' alone
  static_assert(ROWS % (RPL / 2) == 0 && COLS % RPL == 0, "whole loads");
  static_assert(!DUAL || EPI == EPI_BIAS, "the second product rides on the plain bias epilogue");
  constexpr bool F32_OUT = EPI == EPI_BIAS_RESIDUAL || EPI == EPI_BIAS_POS;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WAVES_N, wn = wave % WAVES_N;
  const int l16 = lane & 15, lg = lane >> 4;
  const int KT = p.K / BK;   // even, at least 2

  // position in the launch order -> tile: XCD x (workgroups are dealt round-robin; a workgroup keeps pos % 8) takes a
  // contiguous run of the tile sequence, which walks bands of gw tile columns top to bottom
  auto tile_at = [&](int pos, int& tm, int& tn) {
    const int x = pos & 7, slot = pos >> 3;
    const int q = n_tiles >> 3, r = n_tiles & 7;
    const int id = x * q + (x < r ? x : r) + slot;
    const int band_tiles = gm * gw;
    const int full_bands = gn / gw;
    int band = id / band_tiles, in_band = id % band_tiles, bw = gw;
    if (band >= full_bands) { band = full_bands; in_band = id - full_bands * band_tiles; bw = gn - full_bands * gw; }
    tm = (in_band / bw) * ROWS;
    tn = (band * gw + in_band % bw) * COLS;
  };
  // Tiles of a height that does not divide 256: a last one begins where it ends with the activations' last whole 256-row tile and
  // computes rows of the tile above again, the same bits.  Only residual rows must not be added to twice (`first_row`).
  auto tile_of = [&](int pos, int& m0, int& n0) {
    tile_at(pos, m0, n0);
    if (256 % ROWS != 0) m0 = min(m0, (p.M + 255) / 256 * 256 - ROWS);
  };

  // Direct loads: LDS rows of 64 elements, 16-byte chunks XOR-swizzled by the row; the lane that lands on physical chunk
  // ld_c of its row fetches logical chunk ld_c ^ SWZ(row).  One scalar base per operand walks along K.  (Rows past M are
  // read like any other: A holds whole 256-row tiles.)  As assembly because the compiler would make every later LDS read
  // wait for all of them.
  const int ld_row = tid >> 3, ld_c = tid & 7;
  const unsigned a_voff = ((unsigned)ld_row * (unsigned)p.lda + ((ld_c ^ SWZ(ld_row)) * 8)) * 2;
  const unsigned b_voff = ((unsigned)ld_row * (unsigned)p.K + ((ld_c ^ SWZ(ld_row)) * 8)) * 2;
  const long a_step = (long)RPL * p.lda * 2, b_step = (long)RPL * p.K * 2;
  const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) void*)smem + wave * 1024;
  const char *ga, *gb;      // first row of the slab to fetch next
  auto issue = [&](int i, int buf) {
    if (PART && i == LA - 1 && wave >= WAVES_M * WAVES_N / 2) return;   // uniform
    const char* g = i < LA ? ga + i * a_step : gb + (i - LA) * b_step;
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                 :: "v"(i < LA ? a_voff : b_voff), "s"(g), "s"(lds0 + buf * SLAB + (i < LA ? i * RPL : ROWS + (i - LA) * RPL) * 128) : "memory", "m0");
  };
  // The last of a slab's direct loads have half a slab's time to arrive (0.65 to 0.95 us), less than a line takes that is not in the L2 yet.  So the
  // lines of the two slabs behind the ones under way are asked for a pair of slabs ahead, each by one workgroup of the XCD
  // (they share panels: slot % gw picks the part of the activation rows, slot / gw that of the weight rows) and two lines of a
  // row by two lanes, 256 contiguous bytes.  The load wants a destination: a dword a lane into the wave's staging area, which
  // nobody uses until the epilogue.  A lane that would ask for a line of its own where few share a panel asks for some only:
  // the load is a hint, any address inside the operands is right.  `ahead` 0: all lanes ask for the slab's first line.
  constexpr int HALF_T = NT / 2;
  const bool a_half = wave < WAVES_M * WAVES_N / 2;   // the first waves ask for activations, the others for weights
  unsigned t_voff = 0;
  if (ahead) {
    const int slot = blockIdx.x >> 3, lt = tid & (HALF_T - 1);
    const int parts = a_half ? gw : max(1, (int)((gridDim.x + 7) >> 3) / gw), rows = a_half ? ROWS : COLS;
    const int n = (rows + parts - 1) / parts, ix = 2 * n <= HALF_T ? lt * 2 * n / HALF_T : lt;
    const int row = min((a_half ? slot % gw : slot / gw % parts) * n + (ix >> 1), rows - 1);
    t_voff = ((unsigned)row * (unsigned)(a_half ? p.lda : (long)p.K) + (ix & 1) * BK) * 2;
  }
  const unsigned t_lds = (unsigned)(size_t)(__attribute__((address_space(3))) void*)smem + 2 * SLAB + wave * S::STG;
  const char *tg, *tgn;   // slab pair to ask for next, and the pairs behind the tile's last: those of the next tile
  int t_left;             // slabs up to there
  auto touch = [&]() {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1" :: "v"(t_voff), "s"(tg), "s"(t_lds) : "memory", "m0");
    tg += 2 * BK * 2;
    if ((t_left -= 2) == 0) { tg = tgn; t_left = KT; }
  };
  auto wait_vm = [&](auto n) {   // at most n vector-memory accesses of the wave outstanding (they complete in order)
    constexpr int N = decltype(n)::value;
    __builtin_amdgcn_s_waitcnt((N & 0xf) | ((N >> 4) << 14) | (0x7 << 4) | (0xf << 8));
  };

  // v_mfma_f32_16x16x32_bf16: lane l supplies row l % 16 of the left operand and column l % 16 of the right one, k = 8 (l / 16)
  // .. + 7; result register e of lane l is D[4 (l / 16) + e][l % 16].  The weights are the left operand (a lane owns a token
  // and four consecutive features), for the transposed store the tokens are.
  f32x4 acc[TM][TN];
  bf16x8 fa[2][TM], fb[2][TN];
  constexpr int NR = TM + TN;   // fragment reads of a k-step
  // LDS offsets of fragment 0 by buffer and k-step (opaque: the compiler would keep one register per fragment otherwise)
  unsigned fa0[2][2], fb0[2][2];
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      fa0[b][ks] = (unsigned)(b * SLAB + (wm * WM + l16) * 128 + (((lg + 4 * ks) ^ SWZ(l16)) * 16));
      fb0[b][ks] = (unsigned)(b * SLAB + (ROWS + wn * WN + l16) * 128 + (((lg + 4 * ks) ^ SWZ(l16)) * 16));
      asm volatile("" : "+v"(fa0[b][ks]), "+v"(fb0[b][ks]));
    }
  // fragment r of k-step ks of the slab in buffer buf: the weight fragments first, every row of blocks needs all of them
  auto read = [&](auto set, int buf, int ks, int r) {
    constexpr int X = decltype(set)::value;
    if (r < TN) fb[X][r < TN ? r : 0] = *reinterpret_cast<const bf16x8*>(smem + fb0[buf][ks] + r * 2048);
    else fa[X][r < TN ? 0 : r - TN] = *reinterpret_cast<const bf16x8*>(smem + fa0[buf][ks] + (r - TN) * 2048);
  };
  using S0 = std::integral_constant<int, 0>;
  using S1 = std::integral_constant<int, 1>;
  constexpr int MM = TM * TN;
  // The MFMAs of a k-step from register set `set`, with fn(m) behind MFMA m.  In the main loop as assembly that keeps an
  // accumulator in place (the compiler's form moves it from register to register, and spills).  The compiler does not see
  // the wait states behind such an MFMA, so nothing but MFMAs may touch an accumulator between the zeros in front of a tile
  // and the tile's last k-step, which is the compiler's own form.
  auto mma = [&](auto tok, auto set, auto own, auto fn) {
    constexpr bool TOK = decltype(tok)::value;
    constexpr int X = decltype(set)::value;
    static_for<MM>([&](auto m) {
      constexpr int i = m / TN, j = i % 2 ? TN - 1 - m % TN : m % TN;
      const bf16x8 l = TOK ? fa[X][i] : fb[X][j], r = TOK ? fb[X][j] : fa[X][i];
      if constexpr (decltype(own)::value) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(l, r, acc[i][j], 0, 0, 0);
      else asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(acc[i][j]) : "v"(l), "v"(r));
      __builtin_amdgcn_sched_barrier(0);
      fn(m);
      __builtin_amdgcn_sched_barrier(0);
    });
  };

  // fp32 epilogues: pass i adds stream (or position) rows 16 i .. + 15 of the wave's tile, XCH chunks of 16 bytes a row
  constexpr int XCH = 4 * TN, XPER = 16 * XCH / 64;
  constexpr int XAHEAD = TN > 4 ? 2 : 4;              // passes whose rows are fetched ahead,
  constexpr int XFIRST = EPI == EPI_BIAS_POS ? 0 : 1;   // and those of them that are fetched under the tile's last k-step (as many as the registers hold)
  static_assert(TM >= XAHEAD, "passes");
  __amdgpu_buffer_rsrc_t rsrc_x = __builtin_amdgcn_make_buffer_rsrc(
      p.R, 0, EPI == EPI_BIAS_RESIDUAL ? (int)(unsigned)(((long)(p.M - 1) * p.ldr + p.N) * 4) : 0, 0x00020000);
  __amdgpu_buffer_rsrc_t rsrc_c = __builtin_amdgcn_make_buffer_rsrc(
      p.C, 0, (EPI == EPI_VT || F32_OUT || !p.C) ? 0 : (int)(unsigned)(((long)(p.M - 1) * p.ldc + p.N) * 2), 0x00020000);

  // V^T, T x heads x hd_pad rows of n_tok (written through only while it is small)
  __amdgpu_buffer_rsrc_t rsrc_v = __builtin_amdgcn_make_buffer_rsrc(
      p.VT, 0, (EPI == EPI_VT || DUAL) && NEAR ? (int)(unsigned)((long)p.M * p.heads * p.hd_pad * 2) : 0, 0x00020000);

  int pos = blockIdx.x, m0, n0, m0n, n0n;
  tile_of(pos, m0, n0);
  ga = reinterpret_cast<const char*>(p.A + (long)m0 * p.lda);
  gb = reinterpret_cast<const char*>(p.W + (long)n0 * p.K);
#pragma unroll
  for (int b = 0; b < 2; ++b) {
#pragma unroll
    for (int i = 0; i < LPS; ++i) issue(i, b);
    ga += BK * 2; gb += BK * 2;
  }
  tgn = a_half ? ga - 4 * BK : gb - 4 * BK;   // K = 128: the pair behind the first one is the first one again
  tg = KT > 2 ? tgn + 4 * BK : tgn;
  t_left = KT > 2 ? KT - 2 : KT;
  touch();
  wait_vm(std::integral_constant<int, LPS - PART + 1>{});
  __syncthreads();

  for (;;) {
    const int nxt = pos + (int)gridDim.x;
    const bool has_next = nxt < n_tiles;
    if (has_next) tile_of(nxt, m0n, n0n); else { m0n = m0; n0n = n0; }
    const char* gan = reinterpret_cast<const char*>(p.A + (long)m0n * p.lda);
    const char* gbn = reinterpret_cast<const char*>(p.W + (long)n0n * p.K);
    tgn = a_half ? gan : gbn;
    int first_row = 0;
    if constexpr (256 % ROWS != 0 && EPI == EPI_BIAS_RESIDUAL) { int tn; tile_at(pos, first_row, tn); }
    auto tile = [&](auto tok) {
    constexpr bool TOK = decltype(tok)::value;   // token-major MFMA result, stored transposed
#pragma unroll
    for (int r = 0; r < NR; ++r) read(S0{}, 0, 0, r);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        asm volatile("" : "+v"(acc[i][j]));   // the zeros are in their registers here, not in front of their first use
      }
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 7" ::: "memory");     // wait states between them and the first MFMA
    __builtin_amdgcn_sched_barrier(0);

    f32x4 xr[F32_OUT ? XAHEAD : 1][F32_OUT ? XPER : 1];
    auto xload = [&](int lane, int i) {
      if constexpr (F32_OUT) {
#pragma unroll
        for (int u = 0; u < XPER; ++u) {
          const int q = lane + 64 * u, r = q / XCH, c = q % XCH;
          const int row = m0 + wm * WM + i * 16 + r, col = n0 + wn * WN + c * 4;
          if constexpr (EPI == EPI_BIAS_RESIDUAL)   // the whole offset is the lane's, so that the range check sees it: rows past M come back as zero
            xr[i % XAHEAD][u] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(
                rsrc_x, ((unsigned)row * (unsigned)p.ldr + (unsigned)col) * 4u, 0, NEAR ? 0 : STREAM));
          else
            xr[i % XAHEAD][u] = *reinterpret_cast<const f32x4*>(p.pos + (long)(row % p.n_pos) * p.N + (col < p.N ? col : 0));
        }
      }
    };
    f32x4 bias4[TOK ? 1 : TN];
    float bias1[TOK ? TN : 1];
    // One slab, in buffer buf with its first fragments in set 0: slab kt + 1 lands in the other buffer meanwhile, slab
    // kt + 2 is fetched into this one behind the barrier.  phase 0: inside the tile; 1: the slab before the last, behind
    // which the next tile's slabs are fetched, if there is one; 2: the last slab.  Buffer 0's slabs end with a touch, the
    // newest access when the next slab waits.
    auto slab = [&](int buf, auto phase) {
      constexpr int PHASE = decltype(phase)::value;
      constexpr int H = MM * 3 / 4;   // the reads go behind the first three quarters of the MFMAs
      mma(tok, S0{}, std::false_type{}, [&](auto m) {
        static_for<NR>([&](auto r) {
          if constexpr (r * H / NR == m) read(S1{}, buf, 1, r);
        });
      });
      if constexpr (PHASE == 1) { ga = gan; gb = gbn; }
      // the wave's part of the next slab has landed
      if constexpr (PHASE == 2) {
        if (has_next) wait_vm(std::integral_constant<int, 1>{});
        else wait_vm(std::integral_constant<int, 0>{});
      } else if (buf == 0) {
        wait_vm(std::integral_constant<int, 0>{});
      } else {
        wait_vm(std::integral_constant<int, 1>{});
      }
      __syncthreads();                             // everyone's has, and everyone holds this slab's fragments: its buffer is free
      if constexpr (PHASE == 2) {
        if constexpr (TOK) {
#pragma unroll
          for (int j = 0; j < TN; ++j) bias1[j] = p.bias[n0 + wn * WN + j * 16 + l16];
        } else {
#pragma unroll
          for (int j = 0; j < TN; ++j) bias4[j] = *reinterpret_cast<const f32x4*>(p.bias + n0 + wn * WN + j * 16 + lg * 4);
        }
#pragma unroll
        for (int i = 0; i < XFIRST; ++i) xload(lane, i);   // into the registers of fragment set 0, which nobody reads any more
      }
      mma(tok, S1{}, std::integral_constant<bool, PHASE == 2>{}, [&](auto m) {
        if constexpr (PHASE < 2)
          static_for<NR>([&](auto r) {
            if constexpr (r * H / NR == m) read(S0{}, buf ^ 1, 0, r);
          });
        static_for<LPS>([&](auto i) {
          if constexpr (i * MM / LPS + 1 == m) {
            if (PHASE == 0 || has_next) issue(i, buf);
          }
        });
      });
      ga += BK * 2; gb += BK * 2;
      if (buf == 0 && (PHASE == 0 || has_next)) touch();
    };
    using P0 = std::integral_constant<int, 0>;
    for (int kt = 0; kt < KT - 2; kt += 2) { slab(0, P0{}); slab(1, P0{}); }
    slab(0, std::integral_constant<int, 1>{});
    slab(1, std::integral_constant<int, 2>{});
    // LDS buffer 0 holds slab 0 of the next tile, its slab 1 is on its way to buffer 1; the touch in front of it has left
    wait_vm(std::integral_constant<int, LPS - PART>{});   // the staging area

    {
      // The epilogue's addresses derive from an opaque copy of the thread index, made anew for every tile: computed in
      // front of the tile loop they would occupy registers through the main loop.
      int tid_opaque = threadIdx.x;
      asm volatile("" : "+v"(tid_opaque));
      const int lane = tid_opaque & 63, l16 = lane & 15, lg = lane >> 4;
      unsigned char* stg = smem + 2 * SLAB + wave * S::STG;
      auto wave_sync = [&]() {   // LDS written by one lane, read by another of the same wave
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
      };
      // staging rows of NCH 16-byte chunks; chunk c of row r sits at c ^ key(r), which spreads the 16 rows of an access over
      // the banks
      auto at = [&](auto nch, int r, int c) {
        constexpr int NCH = decltype(nch)::value;
        static_assert(NCH % 4 == 0, "the swizzle stays inside a row");
        return stg + r * (NCH * 16) + ((c ^ (NCH % 16 == 0 ? r & 15 : NCH % 8 == 0 ? (r >> 1) & 7 : (r >> 1) & 3)) << 4);
      };
      if constexpr (F32_OUT) {
        using NCH = std::integral_constant<int, XCH>;
#pragma unroll
        for (int i = XFIRST; i < XAHEAD; ++i) xload(lane, i);
#pragma unroll
        for (int i = 0; i < TM; ++i) {
#pragma unroll
          for (int j = 0; j < TN; ++j) {
            f32x4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = acc[i][j][e] + bias4[j][e];
            *reinterpret_cast<f32x4*>(at(NCH{}, l16, j * 4 + lg)) = v;
          }
          wave_sync();
#pragma unroll
          for (int u = 0; u < XPER; ++u) {
            const int q = lane + 64 * u, r = q / XCH, c = q % XCH;
            const int row = m0 + wm * WM + i * 16 + r, col = n0 + wn * WN + c * 4;
            const f32x4 v = *reinterpret_cast<const f32x4*>(at(NCH{}, r, c));
            if (row >= first_row && row < p.M && col < p.N) {   // read next by a row kernel, not by this launch
              if constexpr (EPI == EPI_BIAS_POS)   // through the slice layout
                *reinterpret_cast<f32x4*>(p.R + p.xrows.row(row) * p.ldr + col) = v + xr[i % XAHEAD][u];
              else if constexpr (NEAR)
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, xr[i % XAHEAD][u] + v), rsrc_x,
                                                       ((unsigned)row * (unsigned)p.ldr + (unsigned)col) * 4u, 0, THROUGH);
              else
                __builtin_nontemporal_store(xr[i % XAHEAD][u] + v, reinterpret_cast<f32x4*>(p.R + (long)row * p.ldr + col));
            }
          }
          wave_sync();
          if (i + XAHEAD < TM) xload(lane, i + XAHEAD);
        }
      } else if constexpr (TOK) {
        using NCH = std::integral_constant<int, (2 * TM + 7) / 8 * 8>;   // chunks of 8 tokens, 2 TM of them in use
#pragma unroll
        for (int j = 0; j < TN; ++j) {
#pragma unroll
          for (int i = 0; i < TM; ++i) {
            bf16x4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = (bf16_t)(acc[i][j][e] + bias1[j]);
            *reinterpret_cast<bf16x4*>(at(NCH{}, l16, i * 2 + (lg >> 1)) + ((lg & 1) << 3)) = o;
          }
          wave_sync();
#pragma unroll
          for (int u = 0; u < 16 * NCH::value / 64; ++u) {
            const int q = lane + 64 * u, r = q / NCH::value, c = q % NCH::value;
            const int f = n0 + wn * WN + j * 16 + r - (DUAL ? p.Npad : 0), tok = m0 + wm * WM + c * 8;   // n_tok % 8 == 0: the eight tokens share a slice
            if (c < 2 * TM && f < (DUAL ? p.n2 : p.N) && tok < p.M) {
              const u32x4 v = *reinterpret_cast<const u32x4*>(at(NCH{}, r, c));
              const int t = tok / p.n_tok, n = tok % p.n_tok;
              // feature h * hd_pad + d of slice t: row ((t * heads + h) * hd_pad + d) = t * heads * hd_pad + f of V^T
              if constexpr (NEAR)
                __builtin_amdgcn_raw_buffer_store_b128(v, rsrc_v, ((unsigned)(t * p.heads * p.hd_pad + f) * (unsigned)p.n_tok + (unsigned)n) * 2u, 0, THROUGH);
              else
                __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(p.VT + ((long)t * p.heads * p.hd_pad + f) * p.n_tok + n));
            }
          }
          wave_sync();
        }
      } else {
        using NCH = std::integral_constant<int, 2 * TN>;   // chunks of 8 columns, two rows of blocks a pass
        auto pass = [&](int i2, auto store) {
#pragma unroll
          for (int i = i2; i < i2 + 2 && i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) {
              bf16x4 o;
#pragma unroll
              for (int e = 0; e < 4; ++e) o[e] = (bf16_t)apply_act_fast<EPI>(acc[i][j][e] + bias4[j][e]);
              *reinterpret_cast<bf16x4*>(at(NCH{}, (i - i2) * 16 + l16, j * 2 + (lg >> 1)) + ((lg & 1) << 3)) = o;
            }
          wave_sync();
#pragma unroll
          for (int u = 0; u < (i2 + 1 < TM ? 32 : 16) * NCH::value / 64; ++u) {
            const int q = lane + 64 * u, r = q / NCH::value, c = q % NCH::value;
            store(m0 + wm * WM + i2 * 16 + r, n0 + wn * WN + c * 8, *reinterpret_cast<const u32x4*>(at(NCH{}, r, c)));
          }
          wave_sync();
        };
        if (p.row_map) {   // paged output: rows go through the block map
#pragma unroll
          for (int i2 = 0; i2 < TM; i2 += 2)
            pass(i2, [&](int row, int col, u32x4 v) {
              if (row < p.M && col < p.N) {
                const long orow = (long)p.row_map[row / p.block_tokens] * p.block_tokens + row % p.block_tokens;
                __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(p.C + orow * p.ldc + col));
              }
            });
        } else {
          // buffer stores whose whole offset is the lane's: the range check drops the rows past M
#pragma unroll
          for (int i2 = 0; i2 < TM; i2 += 2)
            pass(i2, [&](int row, int col, u32x4 v) {
              if (col < p.N)
                __builtin_amdgcn_raw_buffer_store_b128(v, rsrc_c, ((unsigned)row * (unsigned)p.ldc + (unsigned)col) * 2u, 0, NEAR ? THROUGH : STREAM);
            });
        }
      }
    }
    };
    if constexpr (DUAL) {
      if (n0 >= p.Npad) tile(std::true_type{});   // uniform over the workgroup
      else tile(std::false_type{});
    } else {
      tile(std::integral_constant<bool, EPI == EPI_VT>{});
    }
    if (!has_next) break;
    pos = nxt; m0 = m0n; n0 = n0n;
  }
}

template <int EPI, bool DUAL, int TM, int TN, int WAVES_M, int WAVES_N>
hipError_t launch_wide(const GemmParams& p, int cus, hipStream_t st) {
  using S = Wide<TM, TN, WAVES_M, WAVES_N>;
  // tile columns that hold nothing but padding are not launched (the weights are packed to 256 rows)
  const int n_last = DUAL ? p.n2 : p.N, pad_last = DUAL ? p.n2_pad : p.Npad, cols_last = (n_last + S::COLS - 1) / S::COLS;
  if (cols_last * S::COLS > pad_last || (DUAL && p.Npad % S::COLS != 0)) return hipErrorInvalidValue;
  const int gm = (p.M + S::ROWS - 1) / S::ROWS, gn = (DUAL ? p.Npad / S::COLS : 0) + cols_last, n_tiles = gm * gn;
  if (n_tiles == 0) return hipSuccess;
  int gw = band_columns(gn, (double)S::ROWS * p.K * sizeof(bf16_t), (double)S::COLS * p.K * sizeof(bf16_t), (n_tiles < cus ? n_tiles + 7 : cus) / 8);
  if (p.band > 0 && p.band <= gn) gw = p.band;
  // one round of short tiles has nothing to gain (13312 rows, 1024 x 1024 residual, us without | with: 40.7 | 41.6)
  const int ahead = n_tiles > cus || p.K >= 2048;
  const dim3 grid(n_tiles < cus ? n_tiles : cus), block(S::NT);
  constexpr bool HAS_NEAR = EPI != EPI_BIAS_POS;
  if (HAS_NEAR && (EPI == EPI_BIAS_RESIDUAL ? 4.0 * p.M * p.N <= NEAR_ROWS : 2.0 * p.M * (p.N > p.n2 ? p.N : p.n2) <= NEAR_OUT))
    k_gemm_bf16_wide<EPI, DUAL, TM, TN, WAVES_M, WAVES_N, HAS_NEAR><<<grid, block, S::LDS, st>>>(p, gm, gw, gn, n_tiles, ahead);
  else
    k_gemm_bf16_wide<EPI, DUAL, TM, TN, WAVES_M, WAVES_N, false><<<grid, block, S::LDS, st>>>(p, gm, gw, gn, n_tiles, ahead);
  return hipGetLastError();
}
template <int EPI, bool DUAL, int TM, int TN, int WAVES_M, int WAVES_N>
hipError_t set_attr_wide() {
  constexpr int LDS = (int)Wide<TM, TN, WAVES_M, WAVES_N>::LDS;
  const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_gemm_bf16_wide<EPI, DUAL, TM, TN, WAVES_M, WAVES_N, false>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
  if (e != hipSuccess || EPI == EPI_BIAS_POS) return e;
  return hipFuncSetAttribute(reinterpret_cast<const void*>(&k_gemm_bf16_wide<EPI, DUAL, TM, TN, WAVES_M, WAVES_N, EPI != EPI_BIAS_POS>),
                             hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
}
}  // namespace

}  // namespace epd
