// bf16 MFMA GEMM for launches of a few slices:  C[M,N] = A[M,K] * W[N,K]^T on 64 x 64, 128 x 64 and 128 x 128 tiles.
//
// A call of one to some ten slices does not fill the chip with 256 x 256 tiles.  What bounds a launch of smaller tiles
// is the chain one wave walks per 64-deep slab: a wave issues in order, so the barrier, the fragment reads, the direct
// loads (which wait for their turn in the address unit) and the MFMAs add up unless they are laid under one another.
//   * Both operand slabs go from global memory straight into an LDS ring of RING stages (global_load_lds), RING slabs
//     ahead: a stage is free as soon as every wave holds its slab's fragments in registers.
//   * The fragments of a whole slab are read while the MFMAs of the slab before it run (two register sets); reads and
//     direct loads sit one by one between the MFMAs.
//   * The slab is straight-line code: no branch decides about the tail (the last slabs are unrolled), one scalar base
//     per operand walks along K.  (With the waits chosen by branches and addresses computed per load, 573 instead of
//     377 cycles a slab for a 64 x 64 tile; reads in front of all MFMAs, 885 instead of 733 for a 128 x 128 tile, whose
//     MFMAs alone are 512.)
//   * What the epilogue reads (bias, residual rows) is fetched in front of the main loop.
//   * Four waves (2 x 2) of 32 WTM x 32 WTN each: a 64 x 64 wave tile reads half as many LDS bytes per flop as the
//     32 x 64 wave tiles of an eight-wave 128 x 128 tile.
//   * v_mfma_f32_16x16x32_bf16, for the reason given in gemm_bf16_wide.h.
// An element's k-steps are added in the order of every other form (k ascending): same bits.
// Measured stand-alone, K = 4096, N = 1024: 1024 rows 21.8 us with the 64 x 64 form this replaces, 15.4 now; 3096 rows
// 56.4 us with eight-wave 128 x 128 tiles, 30.5 now.  In the running encoder, weights cold: 24.4 -> 22.9, 55.8 -> 41.5.
// A deeper ring (8 / 6 / 5 stages, one workgroup per CU) changed nothing in the encoder.  A fifth wave that asks for the panels' lines
// ahead, as gemm_bf16_wide.h does, costs 5 to 40 %.  LDS is half of a slab (a 64 x 64 one is 32 KiB read and 16 KiB written, 384
// cycles at 128 bytes a cycle; a 128 x 128 one 768): FC2 of 3096 rows of the 1024-wide encoder, one 128 x 128 tile on each of 200 CUs,
// takes 41 us in the encoder, 1500 cycles a slab, of which the products are 512.  Its waves spend 17 % of their cycles waiting for data or
// a barrier and 53 % waiting for an instruction to issue (counters); which instruction, is not measured.
//
// The epilogue goes through LDS wave by wave (a wave stages 32 rows of its own tile and reads them back, no
// workgroup barrier), so that global memory sees 16-byte pieces of whole 128-byte row parts; bias, activation,
// residual and position rows are applied on the way out, where a lane keeps one column chunk.
#include <type_traits>

#include "kernels.h"

namespace epd {

namespace {

constexpr int BK = 64;
#define SWZ(row) (((row) >> 1) & 7)


// acc += a b with the accumulator kept in place (the compiler's form moves it from register to register).  The compiler does
// not see the wait states around it: nothing but MFMAs may touch an accumulator between the zeros in front of the main loop
// and the pause behind it.
__device__ __forceinline__ void mfma_in_place(bf16x8 a, bf16x8 b, f32x4& c) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(a), "v"(b));
}

template <int WTM, int WTN>
constexpr int stage_elems() { return 64 * (WTM + WTN) * BK; }   // activation slab, then weight slab
template <int WTM, int WTN, int RING>
constexpr size_t ring_lds() { return (size_t)RING * stage_elems<WTM, WTN>() * sizeof(bf16_t); }

// DUAL (EPI_BIAS): tile columns from Npad on are a second product over the same activations, the value projection,
// whose tiles run with the operand roles of EPI_VT and leave through its store (GemmParams::n2).
template <int EPI, bool DUAL, int WTM, int WTN, int RING, int OCC>
__global__ __launch_bounds__(256, OCC) void k_gemm_bf16_ring(const GemmParams p, const int gm, const int bw_) {
  static_assert(!DUAL || EPI == EPI_BIAS, "the second product rides on the plain bias epilogue");
  constexpr int TM = 64 * WTM, TN = 64 * WTN;   // block tile
  constexpr int STAGE = stage_elems<WTM, WTN>();
  constexpr int LPS = 2 * (WTM + WTN);          // direct loads per thread and slab (32 rows each)
  constexpr bool tok_major = (EPI == EPI_VT);
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  bf16_t* ring = reinterpret_cast<bf16_t*>(smem);

  // XCD x (workgroups are dealt round-robin) takes a contiguous run of the tile sequence; the sequence walks
  // bands of bw_ tile columns top to bottom, so the tiles an XCD holds at once share few operand panels
  const int gn = (p.Npad + (DUAL ? p.n2_pad : 0)) / TN;
  int id = blockIdx.x;
  {
    const int nb = gridDim.x, x = id & 7, slot = id >> 3, q = nb >> 3, r = nb & 7;
    id = x * q + (x < r ? x : r) + slot;
  }
  const int band_tiles = gm * bw_, full_bands = gn / bw_;
  int band = id / band_tiles, in_band = id % band_tiles, bw = bw_;
  if (band >= full_bands) { band = full_bands; in_band = id - full_bands * band_tiles; bw = gn - full_bands * bw_; }
  const int m0 = (in_band / bw) * TM;
  const int n0 = (band * bw_ + in_band % bw) * TN;
  const bool vt_tile = tok_major || (DUAL && n0 >= p.Npad);   // uniform over the workgroup

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int l16 = lane & 15, lg = lane >> 4;
  constexpr int BM = 2 * WTM, BN = 2 * WTN;   // 16 x 16 blocks of a wave
  const int ld_row = tid >> 3, ld_c = tid & 7;
  // the lane that lands on physical chunk ld_c of its LDS row fetches logical chunk ld_c ^ SWZ(row).  One scalar base per
  // operand walks along K; where a load's 32 rows lie relative to it is a lane offset fixed for the whole kernel.
  unsigned voff[LPS];
#pragma unroll
  for (int i = 0; i < LPS; ++i) {
    const bool a_op = i < 2 * WTM;
    const unsigned ld = (unsigned)(a_op ? p.lda : (long)p.K), row = (unsigned)(ld_row + 32 * (a_op ? i : i - 2 * WTM));
    voff[i] = (row * ld + ((ld_c ^ SWZ(ld_row)) * 8)) * 2;
  }
  const char* ga = reinterpret_cast<const char*>(p.A + (long)m0 * p.lda);
  const char* gb = reinterpret_cast<const char*>(p.W + (long)n0 * p.K);
  const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) void*)ring + wave * 1024;
  const int KT = p.K / BK;   // even, at least 2

  // the next slab -> ring stage at byte offset so (rows of a ragged last tile past M are read like any other: A holds
  // whole 256-row tiles; their results are never stored)
  auto issue_some = [&](int from, int to, unsigned so) {
#pragma unroll
    for (int i = 0; i < LPS; ++i) {
      if (i < from || i >= to) continue;
      asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                   :: "v"(voff[i]), "s"(i < 2 * WTM ? ga : gb), "s"(lds0 + so + 4096 * i) : "memory", "m0");
    }
  };
  auto advance = [&]() { ga += BK * 2; gb += BK * 2; };
  auto wait_vm = [&](auto n) {
    constexpr int N = decltype(n)::value;
    __builtin_amdgcn_s_waitcnt((N & 0xf) | ((N >> 4) << 14) | (0x7 << 4) | (0xf << 8));
  };

  f32x4 acc[BM][BN];

  // byte offsets of the fragments inside a stage; k-step kk (32 deep) sits at chunk (4 kk + lg) ^ swizzle = chunk 0's ^ 4 kk
  const unsigned fa0 = (unsigned)(((wm * 32 * WTM + l16) * BK + ((lg ^ SWZ(l16)) * 8)) * 2);
  const unsigned fb0 = (unsigned)((TM * BK + (wn * 32 * WTN + l16) * BK + ((lg ^ SWZ(l16)) * 8)) * 2);
  bf16x8 fa[2][2][BM], fb[2][2][BN];
  constexpr int RPK = BM + BN, NRD = 2 * RPK;   // fragment reads per k-step and per slab
  auto read_some = [&](auto set, unsigned so, int from, int to) {
    constexpr int S = decltype(set)::value;
#pragma unroll
    for (int r = 0; r < NRD; ++r) {
      if (r < from || r >= to) continue;
      const int kk = r / RPK, x = r % RPK;
      if (x < BM) fa[S][kk][x < BM ? x : 0] = *reinterpret_cast<const bf16x8*>(smem + ((fa0 ^ (64u * kk)) + so) + x * 16 * BK * 2);
      else fb[S][kk][x < BM ? 0 : x - BM] = *reinterpret_cast<const bf16x8*>(smem + ((fb0 ^ (64u * kk)) + so) + (x - BM) * 16 * BK * 2);
    }
  };

  // What the epilogue reads is fetched in front of the main loop: bias, and the residual / position rows (chunk c of
  // pass i), whose latency would otherwise stand behind the last MFMA (up to 2000 cycles of a 10000-cycle tile).
  constexpr bool F32_OUT = EPI == EPI_BIAS_RESIDUAL || EPI == EPI_BIAS_POS;
  constexpr int XCH = 8 * WTN;            // 16-byte fp32 chunks per row of the wave's tile
  constexpr int XPER = 32 * XCH / 64;     // per lane and pass of 32 rows
  f32x4 xr[F32_OUT ? WTM : 1][F32_OUT ? XPER : 1];
  const int x_row = m0 + wm * 32 * WTM + lane / XCH;            // + (64 / XCH) c + 32 i
  const int x_col = n0 + wn * 32 * WTN + (lane % XCH) * 4;
  // VT tiles: a lane reads back chunks of one feature row each, row lane / VCH + (64 / VCH) u of 32-row group j
  constexpr int VCH = 4 * WTM, VU = 32 * VCH / 64;
  constexpr bool HAS_VT = tok_major || DUAL;
  float vb[HAS_VT ? WTN : 1][HAS_VT ? VU : 1];
  f32x4 bias0 = {0.f, 0.f, 0.f, 0.f}, bias1 = {0.f, 0.f, 0.f, 0.f};   // the columns a lane reads back: x_col .. + 3, or c_col .. + 7
  constexpr int NCH = 4 * WTN;   // bf16 output: chunks of 8 columns per row
  const int c_col = n0 + wn * 32 * WTN + (lane % NCH) * 8;
  auto epilogue_loads = [&]() {
    if (HAS_VT && vt_tile) {
#pragma unroll
      for (int j = 0; j < WTN; ++j)
#pragma unroll
        for (int u = 0; u < VU; ++u) vb[j][u] = p.bias[n0 + wn * 32 * WTN + j * 32 + lane / VCH + (64 / VCH) * u];
    } else if constexpr (F32_OUT) {
      bias0 = *reinterpret_cast<const f32x4*>(p.bias + x_col);
#pragma unroll
      for (int i = 0; i < WTM; ++i)
#pragma unroll
        for (int c = 0; c < XPER; ++c) {
          const int row = x_row + 32 * i + (64 / XCH) * c;
          // RESIDUAL: R holds whole 256-row tiles and a padded row's slack, so every lane reads; POS: a valid row and column
          xr[i][c] = *reinterpret_cast<const f32x4*>(
              EPI == EPI_BIAS_RESIDUAL ? p.R + (long)row * p.ldr + x_col
                                       : p.pos + (long)(row % p.n_pos) * p.N + (x_col < p.N ? x_col : 0));
        }
    } else {
      bias0 = *reinterpret_cast<const f32x4*>(p.bias + c_col);
      bias1 = *reinterpret_cast<const f32x4*>(p.bias + c_col + 4);
    }
  };

  using S0 = std::integral_constant<int, 0>;
  using S1 = std::integral_constant<int, 1>;
  constexpr unsigned SB = STAGE * 2;                       // bytes of a stage
  constexpr int TAIL = (RING + 1) / 2 * 2;                 // last slabs, with nothing (more) to fetch
#pragma unroll
  for (int s = 0; s < 2; ++s) { issue_some(0, LPS, s * SB); advance(); }   // KT >= 2
  epilogue_loads();
  auto main_loop = [&](auto tm) {
    constexpr bool TOKM = decltype(tm)::value;
#pragma unroll
    for (int i = 0; i < BM; ++i)
#pragma unroll
      for (int j = 0; j < BN; ++j) {
        acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        asm volatile("" : "+v"(acc[i][j]));   // the zeros are in their registers here (see mfma_in_place)
      }
    asm volatile("s_nop 7" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    unsigned so = 0;   // stage of the slab being multiplied, as a byte offset
    // One slab: its fragments are in register set `cur`; slab kt + 1 moves into the other set and slab kt + RING into
    // the stage slab kt has left.  AHEAD: slabs issued behind slab kt + 1 (loads complete in order, so it has landed
    // once at most their loads are outstanding); MORE: there is a slab kt + RING; NEXT: there is a slab kt + 1.
    auto step = [&](auto cur, auto nxt, auto ahead, auto more, auto next) {
      constexpr int S = decltype(cur)::value;
      constexpr bool MORE = decltype(more)::value, NEXT = decltype(next)::value;
      unsigned son = so + SB == RING * SB ? 0 : so + SB;
      if constexpr (NEXT) {
        wait_vm(std::integral_constant<int, decltype(ahead)::value * LPS>{});
        // everyone's part of slab kt + 1 is in LDS, and everyone holds slab kt in registers: its stage is free
        __syncthreads();
      }
      // A wave issues in order: a fragment read waits for its turn in LDS, a direct load for its turn in the address
      // unit.  Each goes between two MFMAs and passes under the one in front of it: the reads, which the next slab
      // waits for, in the first half, the loads that refill the stage in the second.
      // (Blocks in serpentine order: consecutive MFMAs share a fragment, which saves power.)
      constexpr int MM = 2 * BM * BN, HALF = MM / 2;
#pragma unroll
      for (int m = 0; m < MM; ++m) {
        const int kk = m / (BM * BN), i = m / BN % BM, j = i % 2 ? BN - 1 - m % BN : m % BN;
        const bf16x8 l = TOKM ? fa[S][kk][i] : fb[S][kk][j], r = TOKM ? fb[S][kk][j] : fa[S][kk][i];
        mfma_in_place(l, r, acc[i][j]);
        if constexpr (NEXT) {
          __builtin_amdgcn_sched_barrier(0);
          if (m < HALF) read_some(nxt, son, m * NRD / HALF, (m + 1) * NRD / HALF);
          else if constexpr (MORE) issue_some((m - HALF) * LPS / HALF, (m + 1 - HALF) * LPS / HALF, so);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      if constexpr (MORE) advance();
      so = son;
    };
    using AH = std::integral_constant<int, RING - 2>;
    using YES = std::true_type;
    using NO = std::false_type;
    // slab KT - TAIL + t of the last ones: slab kt + RING is behind it only while t + RING < TAIL
    auto last = [&](auto t_) {
      constexpr int t = decltype(t_)::value;
      constexpr int behind = TAIL - 2 - t < RING - 2 ? TAIL - 2 - t : RING - 2;
      step(std::integral_constant<int, t % 2>{}, std::integral_constant<int, 1 - t % 2>{},
           std::integral_constant<int, (behind > 0 ? behind : 0)>{}, std::integral_constant<bool, (t + RING < TAIL)>{},
           std::integral_constant<bool, (t + 1 < TAIL)>{});
    };
    static_assert(TAIL == 4, "the tail is unrolled that far");
    wait_vm(std::integral_constant<int, LPS>{});   // slab 0 (slab 1 and the epilogue's loads are newer)
    __syncthreads();
    read_some(S0{}, 0, 0, NRD);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 2; s < RING; ++s)
      if (s < KT) { issue_some(0, LPS, s * SB); advance(); }
    for (int left = KT - TAIL; left > 0; left -= 2) {   // KT and TAIL are even
      step(S0{}, S1{}, AH{}, YES{}, YES{});
      step(S1{}, S0{}, AH{}, YES{}, YES{});
    }
    if (KT >= TAIL) {   // K = 128: two slabs
      last(std::integral_constant<int, 0>{});
      last(std::integral_constant<int, 1>{});
    }
    last(std::integral_constant<int, 2>{});
    last(std::integral_constant<int, 3>{});
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 15\n\ts_nop 7" ::: "memory");   // the last MFMAs have written
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < BM; ++i)
#pragma unroll
      for (int j = 0; j < BN; ++j) asm volatile("" : "+v"(acc[i][j]));
  };
  if (DUAL && vt_tile) main_loop(std::true_type{});
  else main_loop(std::integral_constant<bool, tok_major>{});

  // ------------------------------------------------------------ epilogue ----
  __syncthreads();   // every wave is done reading the ring
  auto wave_sync = [&]() {   // LDS written by one lane, read by another of the same wave
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  // the output the tile is part of: V^T, rows of the stream or C (each under 4 GiB; what these tiles write is under NEAR_OUT)
  const __amdgpu_buffer_rsrc_t rsrc =
      vt_tile ? __builtin_amdgcn_make_buffer_rsrc(p.VT, 0, (int)(unsigned)((long)p.M * p.heads * p.hd_pad * 2), 0x00020000)
      : F32_OUT ? __builtin_amdgcn_make_buffer_rsrc(p.R, 0, (int)(unsigned)(((long)(p.M - 1) * p.ldr + p.N) * 4), 0x00020000)
                : __builtin_amdgcn_make_buffer_rsrc(p.C, 0, (int)(unsigned)(((long)(p.M - 1) * p.ldc + p.N) * 2), 0x00020000);
  if (vt_tile) {
    constexpr int ROWF = 32 * WTM + 4;      // floats per staging row (16 bytes of padding: rows start 4 banks apart)
    float* stg = reinterpret_cast<float*>(smem) + wave * 32 * ROWF;
    const int c = lane % VCH;               // chunk of 8 tokens
    const int tok = m0 + wm * 32 * WTM + c * 8;   // n_tok % 8 == 0: the eight tokens share a slice
    const int t = tok / p.n_tok, n = tok % p.n_tok;
#pragma unroll
    for (int j = 0; j < WTN; ++j) {
#pragma unroll
      for (int j2 = 0; j2 < 2; ++j2)
#pragma unroll
        for (int i = 0; i < BM; ++i)
          *reinterpret_cast<f32x4*>(stg + (j2 * 16 + l16) * ROWF + i * 16 + 4 * lg) = acc[i][2 * j + j2];
      wave_sync();
#pragma unroll
      for (int u = 0; u < VU; ++u) {
        const int r = lane / VCH + (64 / VCH) * u;
        const int f = n0 + wn * 32 * WTN + j * 32 + r - (DUAL ? p.Npad : 0);   // feature of the value projection
        if (f < (DUAL ? p.n2 : p.N) && tok < p.M) {
          const f32x4 lo = *reinterpret_cast<const f32x4*>(stg + r * ROWF + c * 8);
          const f32x4 hi = *reinterpret_cast<const f32x4*>(stg + r * ROWF + c * 8 + 4);
          bf16x8 o;
#pragma unroll
          for (int e = 0; e < 4; ++e) { o[e] = (bf16_t)(lo[e] + vb[HAS_VT ? j : 0][HAS_VT ? u : 0]); o[4 + e] = (bf16_t)(hi[e] + vb[HAS_VT ? j : 0][HAS_VT ? u : 0]); }
          // feature h * hd_pad + d of slice t: row ((t * heads + h) * hd_pad + d) = t * heads * hd_pad + f of V^T
          __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, o), rsrc, ((unsigned)(t * p.heads * p.hd_pad + f) * (unsigned)p.n_tok + (unsigned)n) * 2u, 0, THROUGH);
        }
      }
      wave_sync();
    }
    return;
  }
  constexpr int ROWF = 32 * WTN + 4;
  float* stg = reinterpret_cast<float*>(smem) + wave * 32 * ROWF;
  auto stage_rows = [&](int i) {
#pragma unroll
    for (int i2 = 0; i2 < 2; ++i2)
#pragma unroll
      for (int j = 0; j < BN; ++j)
        *reinterpret_cast<f32x4*>(stg + (i2 * 16 + l16) * ROWF + j * 16 + 4 * lg) = acc[2 * i + i2][j];
    wave_sync();
  };
  if constexpr (F32_OUT) {
#pragma unroll
    for (int i = 0; i < WTM; ++i) {
      stage_rows(i);
#pragma unroll
      for (int c = 0; c < XPER; ++c) {
        const int row = x_row + 32 * i + (64 / XCH) * c;
        if (row < p.M && x_col < p.N) {
          const f32x4 v = *reinterpret_cast<const f32x4*>(stg + (lane / XCH + (64 / XCH) * c) * ROWF + (lane % XCH) * 4) + bias0;
          if constexpr (EPI == EPI_BIAS_RESIDUAL)
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, xr[i][c] + v), rsrc, ((unsigned)row * (unsigned)p.ldr + (unsigned)x_col) * 4u, 0, THROUGH);
          else *reinterpret_cast<f32x4*>(p.R + p.xrows.row(row) * p.ldr + x_col) = v + xr[i][c];   // through the slice layout
        }
      }
      wave_sync();
    }
  } else {
#pragma unroll
    for (int i = 0; i < WTM; ++i) {
      stage_rows(i);
#pragma unroll
      for (int u = 0; u < 32 * NCH / 64; ++u) {
        const int r = lane / NCH + (64 / NCH) * u;
        const int row = m0 + wm * 32 * WTM + 32 * i + r;
        if (row < p.M && c_col < p.N) {
          const f32x4 lo = *reinterpret_cast<const f32x4*>(stg + r * ROWF + (lane % NCH) * 8) + bias0;
          const f32x4 hi = *reinterpret_cast<const f32x4*>(stg + r * ROWF + (lane % NCH) * 8 + 4) + bias1;
          bf16x8 o;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            o[e] = (bf16_t)apply_act_fast<EPI>(lo[e]);
            o[4 + e] = (bf16_t)apply_act_fast<EPI>(hi[e]);
          }
          if (p.row_map)   // paged output: rows go through the block map
            *reinterpret_cast<bf16x8*>(p.C + ((long)p.row_map[row / p.block_tokens] * p.block_tokens + row % p.block_tokens) * p.ldc + c_col) = o;
          else
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, o), rsrc, ((unsigned)row * (unsigned)p.ldc + (unsigned)c_col) * 2u, 0, THROUGH);
        }
      }
      wave_sync();
    }
  }
}

// The forms: 64 x 64 and 128 x 64 tiles, two workgroups per CU (64 / 72 KiB of ring each), and 128 x 128 tiles, one
// workgroup per CU (128 KiB).
template <int EPI, bool DUAL, int WTM, int WTN, int RING, int OCC>
hipError_t launch_ring(const GemmParams& p, hipStream_t st) {
  constexpr int TM = 64 * WTM, TN = 64 * WTN;
  if (p.Npad % TN != 0 || p.n2_pad % TN != 0) return hipErrorInvalidValue;
  const int gm = (p.M + TM - 1) / TM, gn = (p.Npad + (DUAL ? p.n2_pad : 0)) / TN;
  if (gm * gn == 0) return hipSuccess;
  if ((EPI == EPI_VT || DUAL) && (long)p.M * p.heads * p.hd_pad * 2 >= (1L << 32)) return hipErrorInvalidValue;   // V^T through 32-bit offsets
  // bands of up to eight tile columns, equally wide: within 2 % of four at any size, 4 % ahead on average with 128 x 64 tiles
  const int bands = (gn + 7) / 8;
  k_gemm_bf16_ring<EPI, DUAL, WTM, WTN, RING, OCC><<<dim3(gm * gn), dim3(256), ring_lds<WTM, WTN, RING>(), st>>>(p, gm, (gn + bands - 1) / bands);
  return hipGetLastError();
}
template <int EPI, bool DUAL, int WTM, int WTN, int RING, int OCC>
hipError_t set_attr_ring() {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(&k_gemm_bf16_ring<EPI, DUAL, WTM, WTN, RING, OCC>),
                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)ring_lds<WTM, WTN, RING>());
}
template <int EPI, bool DUAL = false>
hipError_t set_attr_tiles() {
  hipError_t e = set_attr_ring<EPI, DUAL, 1, 1, 4, 2>();
  if (e == hipSuccess) e = set_attr_ring<EPI, DUAL, 2, 1, 3, 2>();
  return e != hipSuccess ? e : set_attr_ring<EPI, DUAL, 2, 2, 4, 1>();
}
template <int EPI, bool DUAL = false>
hipError_t launch_tile(const GemmParams& p, int tile, hipStream_t st) {
  switch (tile) {
    case RING_64x64: return launch_ring<EPI, DUAL, 1, 1, 4, 2>(p, st);
    case RING_128x64: return launch_ring<EPI, DUAL, 2, 1, 3, 2>(p, st);
    case RING_128x128: return launch_ring<EPI, DUAL, 2, 2, 4, 1>(p, st);
  }
  return hipErrorInvalidValue;
}
}  // namespace

hipError_t bf16_gemm_ring_init() {
  hipError_t e = set_attr_tiles<EPI_BIAS>();
  if (e == hipSuccess) e = set_attr_tiles<EPI_BIAS, true>();
  if (e == hipSuccess) e = set_attr_tiles<EPI_BIAS_GELU_ERF>();
  if (e == hipSuccess) e = set_attr_tiles<EPI_BIAS_GELU_TANH>();
  if (e == hipSuccess) e = set_attr_tiles<EPI_BIAS_RESIDUAL>();
  if (e == hipSuccess) e = set_attr_tiles<EPI_BIAS_POS>();
  return e != hipSuccess ? e : set_attr_tiles<EPI_VT>();
}

hipError_t bf16_gemm_ring(const GemmParams& p, int tile, hipStream_t st) {
  if (p.stats || p.xb) return hipErrorInvalidValue;   // neither the folded pre-norm nor the bf16 copy of the residual rows
  if (p.n2_pad > 0) return p.epi == EPI_BIAS ? launch_tile<EPI_BIAS, true>(p, tile, st) : hipErrorInvalidValue;
  switch (p.epi) {
    case EPI_BIAS: return launch_tile<EPI_BIAS>(p, tile, st);
    case EPI_BIAS_GELU_ERF: return launch_tile<EPI_BIAS_GELU_ERF>(p, tile, st);
    case EPI_BIAS_GELU_TANH: return launch_tile<EPI_BIAS_GELU_TANH>(p, tile, st);
    case EPI_BIAS_RESIDUAL: return launch_tile<EPI_BIAS_RESIDUAL>(p, tile, st);
    case EPI_BIAS_POS: return launch_tile<EPI_BIAS_POS>(p, tile, st);
    case EPI_VT: return launch_tile<EPI_VT>(p, tile, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace epd
