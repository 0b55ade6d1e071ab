// bf16 MFMA GEMM for launches of a few slices:  C[M,N] = A[M,K] * W[N,K]^T on 64 x 64, 128 x 64 and 128 x 128 tiles,
// and on 64 x 96, 128 x 96 and 128 x 192 ones where those make one round of two (ring_wider).
//
// A call of one to some ten slices does not fill the chip with 256 x 256 tiles.  What bounds a launch of smaller tiles
// is the chain one wave walks per 64-deep slab: a wave issues in order, so the barrier, the fragment reads, the direct
// loads (which wait for their turn in the address unit) and the MFMAs add up unless they are laid under one another.
//   * Both operand slabs go from global memory straight into an LDS ring of RING stages (global_load_lds), RING slabs
//     ahead: a stage is free as soon as every wave holds its slab's last fragments in registers.
//   * The fragments of a k-step (32 deep, two a slab) are read while the MFMAs of the one before it run; reads and
//     direct loads sit one by one between the MFMAs.
//   * The slab is straight-line code: no branch decides about the tail (the last slabs are unrolled), one scalar base
//     per operand walks along K.  (With the waits chosen by branches and addresses computed per load, 573 instead of
//     377 cycles a slab for a 64 x 64 tile; reads in front of all MFMAs, 885 instead of 733 for a 128 x 128 tile, whose
//     MFMAs alone are 512.)
//   * What the epilogue reads (bias, residual rows) is fetched in front of the main loop; the bias of two products in a launch behind it.
//   * Four waves (2 x 2), each on BM x BN blocks of 16 x 16: a 64 x 64 wave tile reads half as many LDS bytes per flop as the
//     32 x 64 wave tiles of an eight-wave 128 x 128 tile.
//   * v_mfma_f32_16x16x32_bf16, for the reason given in gemm_bf16_wide.h.
// An element's k-steps are added in the order of every other form (k ascending): same bits.
// Measured stand-alone, K = 4096, N = 1024: 1024 rows 21.8 us with the 64 x 64 form this replaces, 15.4 now; 3096 rows
// 56.4 us with eight-wave 128 x 128 tiles, 30.5 now.  In the running encoder, weights cold: 24.4 -> 22.9, 55.8 -> 41.5.
// A deeper ring (8 / 6 / 5 stages, one workgroup per CU) changed nothing in the encoder.  A fifth wave that asks for the panels' lines
// ahead, as gemm_bf16_wide.h does, costs 5 to 40 %.  LDS is half of a slab (a 64 x 64 one is 32 KiB read and 16 KiB written, 384
// cycles at 128 bytes a cycle; a 128 x 128 one 768): FC2 of 3096 rows of the 1024-wide encoder, one 128 x 128 tile on each of 200 CUs,
// takes 41 us in the encoder, 1500 cycles a slab, of which the products are 512.  Its waves spend 17 % of their cycles waiting for data or
// a barrier and 53 % waiting for an instruction to issue (counters of the loop that held fragments of whole slabs); which instruction, is not measured.
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


template <int N, int I = 0, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<N, I + 1>(f);
  }
}

// acc += a b with the accumulator kept in place (the compiler's form moves it from register to register).  The compiler does
// not see the wait states around it: nothing but MFMAs may touch an accumulator between the zeros in front of the main loop
// and the pause behind it.
__device__ __forceinline__ void mfma_in_place(bf16x8 a, bf16x8 b, f32x4& c) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(a), "v"(b));
}

// A tile: 2 x 2 waves of BM x BN blocks of 16 x 16
template <int BM, int BN>
constexpr int stage_elems() { return 32 * (BM + BN) * BK; }   // activation slab, then weight slab
template <int BM, int BN, int RING>
constexpr size_t ring_lds() { return (size_t)RING * stage_elems<BM, BN>() * sizeof(bf16_t); }

// DUAL (EPI_BIAS): tile columns from Npad on are a second product over the same activations, the value projection,
// whose tiles run with the operand roles of EPI_VT and leave through its store (GemmParams::n2).
template <int EPI, bool DUAL, int BM, int BN, int RING, int OCC>
__global__ __launch_bounds__(256, OCC) void k_gemm_bf16_ring(const GemmParams p, const int gm, const int bw_) {
  static_assert(!DUAL || EPI == EPI_BIAS, "the second product rides on the plain bias epilogue");
  constexpr int TM = 32 * BM, TN = 32 * BN;     // block tile
  constexpr int WTM = BM / 2, WTN = BN / 2;     // a wave's part in units of 32 (BN odd: only the row-major stores, which do not count in them)
  static_assert(BM % 2 == 0 && (BN % 2 == 0 || !(DUAL || EPI == EPI_VT)), "passes of 32 rows");
  constexpr int STAGE = stage_elems<BM, BN>();
  constexpr int LPS = BM + BN;                  // direct loads per thread and slab (32 rows each)
  constexpr bool tok_major = (EPI == EPI_VT);
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  bf16_t* ring = reinterpret_cast<bf16_t*>(smem);

  // XCD x (workgroups are dealt round-robin) takes a contiguous run of the tile sequence; the sequence walks
  // bands of bw_ tile columns top to bottom, so the tiles an XCD holds at once share few operand panels
  const int gn = ((p.Npad + (DUAL ? p.n2_pad : 0)) + TN - 1) / TN;
  int id = blockIdx.x;
  {
    const int nb = gridDim.x, x = id & 7, slot = id >> 3, q = nb >> 3, r = nb & 7;
    id = x * q + (x < r ? x : r) + slot;
  }
  const int band_tiles = gm * bw_, full_bands = gn / bw_;
  int band = id / band_tiles, in_band = id % band_tiles, bw = bw_;
  if (band >= full_bands) { band = full_bands; in_band = id - full_bands * band_tiles; bw = gn - full_bands * bw_; }
  const int m0 = (in_band / bw) * TM;
  // a last tile column past the weights begins where it ends with them and computes columns of the one beside it again, the same bits (not of rows
  // that are added to: see launch_ring)
  const int n_at = (band * bw_ + in_band % bw) * TN, n0 = 128 % TN == 0 ? n_at : min(n_at, p.Npad - TN);
  const bool vt_tile = tok_major || (DUAL && n0 >= p.Npad);   // uniform over the workgroup

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int l16 = lane & 15, lg = lane >> 4;
  const int ld_row = tid >> 3, ld_c = tid & 7;
  // the lane that lands on physical chunk ld_c of its LDS row fetches logical chunk ld_c ^ SWZ(row).  One scalar base per
  // operand walks along K; where a load's 32 rows lie relative to it is a lane offset fixed for the whole kernel.
  unsigned voff[LPS];
#pragma unroll
  for (int i = 0; i < LPS; ++i) {
    const bool a_op = i < BM;
    const unsigned ld = (unsigned)(a_op ? p.lda : (long)p.K), row = (unsigned)(ld_row + 32 * (a_op ? i : i - BM));
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
                   :: "v"(voff[i]), "s"(i < BM ? ga : gb), "s"(lds0 + so + 4096 * i) : "memory", "m0");
    }
  };
  auto advance = [&]() { ga += BK * 2; gb += BK * 2; };
  auto wait_vm = [&](auto n) {
    constexpr int N = decltype(n)::value;
    __builtin_amdgcn_s_waitcnt((N & 0xf) | ((N >> 4) << 14) | (0x7 << 4) | (0xf << 8));
  };

  f32x4 acc[BM][BN];

  // byte offsets of the fragments inside a stage; k-step kk (32 deep) sits at chunk (4 kk + lg) ^ swizzle = chunk 0's ^ 4 kk
  const unsigned fa0 = (unsigned)(((wm * 16 * BM + l16) * BK + ((lg ^ SWZ(l16)) * 8)) * 2);
  const unsigned fb0 = (unsigned)((TM * BK + (wn * 16 * BN + l16) * BK + ((lg ^ SWZ(l16)) * 8)) * 2);
  bf16x8 fa[2][BM], fb[2][BN];   // of a k-step each
  constexpr int RPK = BM + BN, NRD = 2 * RPK;   // fragment reads per k-step and per slab
  auto read_some = [&](unsigned so, int from, int to) {
#pragma unroll
    for (int r = 0; r < NRD; ++r) {
      if (r < from || r >= to) continue;
      const int kk = r / RPK, x = r % RPK;
      if (x < BM) fa[kk][x < BM ? x : 0] = *reinterpret_cast<const bf16x8*>(smem + ((fa0 ^ (64u * kk)) + so) + x * 16 * BK * 2);
      else fb[kk][x < BM ? 0 : x - BM] = *reinterpret_cast<const bf16x8*>(smem + ((fb0 ^ (64u * kk)) + so) + (x - BM) * 16 * BK * 2);
    }
  };

  // What the epilogue reads is fetched in front of the main loop: bias, and the residual / position rows (chunk c of
  // pass i), whose latency would otherwise stand behind the last MFMA (up to 2000 cycles of a 10000-cycle tile).
  constexpr bool F32_OUT = EPI == EPI_BIAS_RESIDUAL || EPI == EPI_BIAS_POS;
  constexpr int XCH = 4 * BN;             // 16-byte fp32 chunks per row of the wave's tile
  constexpr int XPER = 32 * XCH / 64;     // per lane and pass of 32 rows: chunk (lane + 64 c) % XCH of row (lane + 64 c) / XCH, which
  constexpr int XB = 64 % XCH == 0 ? 1 : 3;      // is the same for every c, or for every third (XCH 12 or 24)
  f32x4 xr[F32_OUT ? WTM : 1][F32_OUT ? XPER : 1];
  const int x_row0 = m0 + wm * 16 * BM;   // + 32 i
  auto xr_of = [&](int c) { return XB == 1 ? lane / XCH + (64 / XCH) * c : (lane + 64 * c) / XCH; };
  auto xc_of = [&](int c) { return XB == 1 ? lane % XCH : (lane + 64 * c) % XCH; };
  auto x_col = [&](int c) { return n0 + wn * 16 * BN + xc_of(c) * 4; };
  // VT tiles: a lane reads back chunks of one feature row each, row lane / VCH + (64 / VCH) u of 32-row group j
  constexpr int VCH = 4 * WTM, VU = 32 * VCH / 64;
  constexpr bool HAS_VT = tok_major || DUAL;
  float vb[HAS_VT ? WTN : 1][HAS_VT ? VU : 1];
  constexpr int NCH = 2 * BN, CPER = 32 * NCH / 64, CB = 64 % NCH == 0 ? 1 : 3;   // bf16 output: chunks of 8 columns per row, dealt like the fp32 ones
  auto cr_of = [&](int u) { return CB == 1 ? lane / NCH + (64 / NCH) * u : (lane + 64 * u) / NCH; };
  auto cc_of = [&](int u) { return CB == 1 ? lane % NCH : (lane + 64 * u) % NCH; };
  auto c_col = [&](int u) { return n0 + wn * 16 * BN + cc_of(u) * 8; };
  constexpr int NB = F32_OUT ? XB : CB;
  f32x4 bias0[NB], bias1[F32_OUT ? 1 : NB];   // the columns a lane reads back: x_col .. + 3, or c_col .. + 7
  auto epilogue_loads = [&]() {
    if (HAS_VT && vt_tile) {
#pragma unroll
      for (int j = 0; j < WTN; ++j)
#pragma unroll
        for (int u = 0; u < VU; ++u) vb[j][u] = p.bias[n0 + wn * 32 * WTN + j * 32 + lane / VCH + (64 / VCH) * u];
    } else if constexpr (F32_OUT) {
#pragma unroll
      for (int c = 0; c < XB; ++c) bias0[c] = *reinterpret_cast<const f32x4*>(p.bias + x_col(c));
#pragma unroll
      for (int i = 0; i < WTM; ++i)
#pragma unroll
        for (int c = 0; c < XPER; ++c) {
          const int row = x_row0 + 32 * i + xr_of(c);
          // RESIDUAL: R holds whole 256-row tiles and a padded row's slack, so every lane reads; POS: a valid row and column
          xr[i][c] = *reinterpret_cast<const f32x4*>(
              EPI == EPI_BIAS_RESIDUAL ? p.R + (long)row * p.ldr + x_col(c)
                                       : p.pos + (long)(row % p.n_pos) * p.N + (x_col(c) < p.N ? x_col(c) : 0));
        }
    } else {
#pragma unroll
      for (int u = 0; u < CB; ++u) {
        bias0[u] = *reinterpret_cast<const f32x4*>(p.bias + c_col(u));
        bias1[F32_OUT ? 0 : u] = *reinterpret_cast<const f32x4*>(p.bias + c_col(u) + 4);
      }
    }
  };

  constexpr unsigned SB = STAGE * 2;                       // bytes of a stage
  constexpr int TAIL = (RING + 1) / 2 * 2;                 // last slabs, with nothing (more) to fetch
#pragma unroll
  for (int s = 0; s < 2; ++s) { issue_some(0, LPS, s * SB); advance(); }   // KT >= 2
  // Of two products in a launch behind the loop: 2048 rows, 3072 columns, K = 1024 on 128 x 128 tiles 26.0 | 23.8 us; with an activation the other
  // way round (4096 columns over 1024 rows 14.4 | 16.4).
  if (!DUAL) epilogue_loads();
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
    // One slab, the fragments of its first k-step in registers: those of a k-step are read while the MFMAs of the one before run.  The barrier
    // stands between the two: slab kt + 1 is read behind it, and slab kt + RING goes into the stage slab kt has left.  (Fragments of whole slabs in
    // two register sets, the barrier in front of a slab: twice the registers, the same times but for 128 x 64 tiles, 2048 rows, residual
    // 1024 x 4096 34.2 us for 33.0.)  AHEAD: slabs issued behind slab kt + 1 (loads complete in order, so it has landed
    // once at most their loads are outstanding); MORE: there is a slab kt + RING; NEXT: there is a slab kt + 1.
    auto step = [&](auto ahead, auto more, auto next) {
      constexpr bool MORE = decltype(more)::value, NEXT = decltype(next)::value;
      unsigned son = so + SB == RING * SB ? 0 : so + SB;
      // A wave issues in order: a fragment read waits for its turn in LDS, a direct load for its turn in the address
      // unit.  Each goes between two MFMAs and passes under the one in front of it, the reads behind the first three quarters of a k-step's.
      // (Blocks in serpentine order: consecutive MFMAs share a fragment, which saves power.)
      constexpr int MM = BM * BN, H = MM * 3 / 4;
      static_for<2 * MM>([&](auto m_) {   // not a loop: 48 steps are too many for the compiler to unroll (128 x 192 tiles 68 us for 21)
        constexpr int kk = m_ / MM, m = m_ % MM, i = m / BN, j = i % 2 ? BN - 1 - m % BN : m % BN;
        if constexpr (kk == 1 && m == 0 && NEXT) {
          wait_vm(std::integral_constant<int, decltype(ahead)::value * LPS>{});
          // everyone's part of slab kt + 1 is in LDS, and everyone holds the rest of slab kt in registers: its stage is free
          __syncthreads();
          __builtin_amdgcn_sched_barrier(0);
        }
        mfma_in_place(TOKM ? fa[kk][i] : fb[kk][j], TOKM ? fb[kk][j] : fa[kk][i], acc[i][j]);
        __builtin_amdgcn_sched_barrier(0);
        constexpr int from = m * RPK / H < RPK ? m * RPK / H : RPK, to = (m + 1) * RPK / H < RPK ? (m + 1) * RPK / H : RPK;
        if constexpr (kk == 0) read_some(so, RPK + from, RPK + to);
        else if constexpr (NEXT) {
          read_some(son, from, to);
          if constexpr (MORE) issue_some(m * LPS / MM, (m + 1) * LPS / MM, so);
        }
        __builtin_amdgcn_sched_barrier(0);
      });
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
      step(std::integral_constant<int, (behind > 0 ? behind : 0)>{}, std::integral_constant<bool, (t + RING < TAIL)>{},
           std::integral_constant<bool, (t + 1 < TAIL)>{});
    };
    static_assert(TAIL == 4, "the tail is unrolled that far");
    wait_vm(std::integral_constant<int, LPS>{});   // slab 0 (slab 1 and the epilogue's loads are newer)
    __syncthreads();
    read_some(0, 0, RPK);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 2; s < RING; ++s)
      if (s < KT) { issue_some(0, LPS, s * SB); advance(); }
    for (int left = KT - TAIL; left > 0; left -= 2) {   // KT and TAIL are even
      step(AH{}, YES{}, YES{});
      step(AH{}, YES{}, YES{});
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
  if (DUAL) epilogue_loads();
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
  constexpr int ROWF = 16 * BN + 4;
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
        const int row = x_row0 + 32 * i + xr_of(c);
        if (row < p.M && x_col(c) < p.N) {
          const f32x4 v = *reinterpret_cast<const f32x4*>(stg + xr_of(c) * ROWF + xc_of(c) * 4) + bias0[c % XB];
          if constexpr (EPI == EPI_BIAS_RESIDUAL)
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, xr[i][c] + v), rsrc, ((unsigned)row * (unsigned)p.ldr + (unsigned)x_col(c)) * 4u, 0, THROUGH);
          else *reinterpret_cast<f32x4*>(p.R + p.xrows.row(row) * p.ldr + x_col(c)) = v + xr[i][c];   // through the slice layout
        }
      }
      wave_sync();
    }
  } else {
#pragma unroll
    for (int i = 0; i < WTM; ++i) {
      stage_rows(i);
#pragma unroll
      for (int u = 0; u < CPER; ++u) {
        const int r = cr_of(u), row = m0 + wm * 16 * BM + 32 * i + r;
        if (row < p.M && c_col(u) < p.N) {
          const f32x4 lo = *reinterpret_cast<const f32x4*>(stg + r * ROWF + cc_of(u) * 8) + bias0[u % CB];
          const f32x4 hi = *reinterpret_cast<const f32x4*>(stg + r * ROWF + cc_of(u) * 8 + 4) + bias1[F32_OUT ? 0 : u % CB];
          bf16x8 o;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            o[e] = (bf16_t)apply_act_fast<EPI>(lo[e]);
            o[4 + e] = (bf16_t)apply_act_fast<EPI>(hi[e]);
          }
          if (p.row_map)   // paged output: rows go through the block map
            *reinterpret_cast<bf16x8*>(p.C + ((long)p.row_map[row / p.block_tokens] * p.block_tokens + row % p.block_tokens) * p.ldc + c_col(u)) = o;
          else
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, o), rsrc, ((unsigned)row * (unsigned)p.ldc + (unsigned)c_col(u)) * 2u, 0, THROUGH);
        }
      }
      wave_sync();
    }
  }
}

// The forms: 64 x 64 and 128 x 64 tiles, two workgroups per CU (64 / 72 KiB of ring each), and 128 x 128 tiles, one
// workgroup per CU (128 KiB).  Half as wide again where ring_wider says so: 64 x 96 (80 KiB, two per CU), 128 x 96 and 128 x 192 (112, 120).
template <int EPI, bool DUAL, int BM, int BN, int RING, int OCC>
hipError_t launch_ring(const GemmParams& p, hipStream_t st) {
  constexpr int TM = 32 * BM, TN = 32 * BN;
  if (128 % TN == 0 ? p.Npad % TN != 0 || p.n2_pad % TN != 0 : p.Npad < TN || p.n2_pad > 0 || (EPI == EPI_BIAS_RESIDUAL && p.Npad % TN != 0)) return hipErrorInvalidValue;
  const int gm = (p.M + TM - 1) / TM, gn = (p.Npad + (DUAL ? p.n2_pad : 0) + TN - 1) / TN;
  if (gm * gn == 0) return hipSuccess;
  if ((EPI == EPI_VT || DUAL) && (long)p.M * p.heads * p.hd_pad * 2 >= (1L << 32)) return hipErrorInvalidValue;   // V^T through 32-bit offsets
  // bands of up to eight tile columns, equally wide: within 2 % of four at any size, 4 % ahead on average with 128 x 64 tiles
  const int bands = (gn + 7) / 8;
  k_gemm_bf16_ring<EPI, DUAL, BM, BN, RING, OCC><<<dim3(gm * gn), dim3(256), ring_lds<BM, BN, RING>(), st>>>(p, gm, (gn + bands - 1) / bands);
  return hipGetLastError();
}
template <int EPI, bool DUAL, int BM, int BN, int RING, int OCC>
hipError_t set_attr_ring() {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(&k_gemm_bf16_ring<EPI, DUAL, BM, BN, RING, OCC>),
                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)ring_lds<BM, BN, RING>());
}
constexpr bool gelu(int epi) { return epi == EPI_BIAS_GELU_ERF || epi == EPI_BIAS_GELU_TANH; }
template <int EPI, bool DUAL = false>
hipError_t set_attr_tiles() {
  hipError_t e = set_attr_ring<EPI, DUAL, 2, 2, 4, 2>();
  if (e == hipSuccess) e = set_attr_ring<EPI, DUAL, 4, 2, 3, 2>();
  if constexpr (EPI == EPI_BIAS_RESIDUAL) {
    if (e == hipSuccess) e = set_attr_ring<EPI, DUAL, 2, 3, 4, 2>();
    if (e == hipSuccess) e = set_attr_ring<EPI, DUAL, 4, 3, 4, 1>();
  }
  if constexpr (gelu(EPI)) {
    if (e == hipSuccess) e = set_attr_ring<EPI, DUAL, 4, 6, 3, 1>();
  }
  return e != hipSuccess ? e : set_attr_ring<EPI, DUAL, 4, 4, 4, 1>();
}
template <int EPI, bool DUAL = false>
hipError_t launch_tile(const GemmParams& p, int tile, hipStream_t st) {
  const bool wide = ring_wider(p.epi, p.M, p.Npad, p.K, tile);
  switch (tile) {
    case RING_64x64:
      if constexpr (EPI == EPI_BIAS_RESIDUAL) {
        if (wide) return launch_ring<EPI, DUAL, 2, 3, 4, 2>(p, st);
      }
      return launch_ring<EPI, DUAL, 2, 2, 4, 2>(p, st);
    case RING_128x64:
      if constexpr (EPI == EPI_BIAS_RESIDUAL) {
        if (wide) return launch_ring<EPI, DUAL, 4, 3, 4, 1>(p, st);
      }
      return launch_ring<EPI, DUAL, 4, 2, 3, 2>(p, st);
    case RING_128x128:
      if constexpr (gelu(EPI)) {
        if (wide) return launch_ring<EPI, DUAL, 4, 6, 3, 1>(p, st);
      }
      return launch_ring<EPI, DUAL, 4, 4, 4, 1>(p, st);
  }
  return hipErrorInvalidValue;
}
}  // namespace

// Where a launch makes some more tiles than there are CUs, a few CUs have two and all wait for them; tiles half as wide again then fit one round, and read
// a sixth fewer LDS bytes per flop.  Residual products of a width that is a multiple of 96 (no column may be added to twice), and activations: the
// others have not been compiled.  us among other kernels, cold: 1024 rows, residual 1152 x 4352 (288 | 192 tiles) 32.2 | 30.9, 1152 x 1152 11.4 | 10.9;
// 2048 (288 | 192) 43.4 | 39.2, 18.1 | 16.5; GELU 4304 x 1152 over 1024 rows (272 | 184) 25.6 | 20.9, 4096 x 1024 over 1088 (288 | 198) 23.2 | 19.1.
// Encoder calls, where the attention has asked for the weights, gain more: 1152-wide, one slice 2640 | 2330 (231 of them by the residual ones), two
// 3705 | 3550, three of 729 tokens 3668 | 3527; 1024-wide, one of 1025 tokens 2206 | 2152.
// 128 x 96 tiles over a K up to 1536 as long as they leave a sixteenth of the CUs idle: fuller rounds (2600 rows, 1152 x 1152: 18.0, on 128 x 128 tiles 19.4)
// stay where the tests of the dispatch hold them.
bool ring_wider(int epi, int M, int n_cols, int K, int tile) {
  const long cus = cu_count();
  auto one_round = [&](int tm, int tn, long most) {
    const long rows = (M + tm - 1) / tm;
    return rows * ((n_cols + tn - 1) / tn) > cus && rows * ((n_cols + tn * 3 / 2 - 1) / (tn * 3 / 2)) <= most;
  };
  switch (tile) {
    case RING_64x64: return epi == EPI_BIAS_RESIDUAL && n_cols % 96 == 0 && one_round(64, 64, cus);
    case RING_128x64: return epi == EPI_BIAS_RESIDUAL && n_cols % 96 == 0 && one_round(128, 64, K <= 1536 ? cus / 16 * 15 : cus);
    default: return gelu(epi) && n_cols >= 192 && one_round(128, 128, cus);
  }
}

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
