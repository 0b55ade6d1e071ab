// bf16 MFMA GEMM for gfx950:  C[M,N] = A[M,K] * W[N,K]^T, fp32 accumulate,
// fused epilogues (bias, GELU, residual add into the fp32 stream, position
// embedding, transposed store of the attention values).
//
// Block tile 256 x BN x 64 (BN = 256 or 128; 128 x 128 x 64 for small launches), 8 waves of 64 lanes.  Both
// operands are K-contiguous, staged through LDS as [row][64] bf16 with the
// 16-byte chunks of a row XOR-swizzled by the row so that the 32 rows a
// wave reads for one MFMA operand fall into different banks (64 banks, 16
// lanes per 128-bit access phase: rows r and r+1 share a chunk column, so the
// XOR key is (row >> 1) & 7).  One barrier per slab, two LDS buffers.
//
// What runs here: the products with a folded pre-norm or emitted rows (EPD_NORM_MODE), and the forms that tests hold the others
// against.  All other products run on gemm_bf16_wide.h and gemm_bf16_ring.hip; the dispatch at the end of this file chooses.
//
// Main loop of the 256 x 256 shape (PIPE = 1): the activation slab is read two
// slabs ahead into registers through a buffer descriptor (L2 / Infinity-Cache
// latency is longer than one slab of MFMA work) and stored to the other LDS
// buffer a slab later; the weight slab, which sits in L2, goes from global
// memory straight into the other LDS buffer one slab ahead (global_load_lds,
// no staging registers).  The MFMA operand fragments of k-step kk+1 are read
// from LDS into a second register set while the MFMAs of k-step kk issue back
// to back.  PIPE = 0 is the plain form (both operands staged in registers,
// fragment reads left to the compiler), kept for the other tile shapes.
//
// v_mfma_f32_32x32x16_bf16 operand layout (checked on the device by
// mfma_probe): lane l supplies row (l % 32) of the 32 x 16 left operand /
// column (l % 32) of the 16 x 32 right operand, k = 8*(l / 32) + 0..7;
// result register i of lane l is D[8*(i/4) + 4*(l/32) + i%4][l % 32].
// The weight fragment is fed as the LEFT operand, so a lane owns one token
// and four consecutive output features per register group: 8-byte bf16 /
// 16-byte fp32 accesses in the epilogue.  For the attention values (EPI_VT)
// the roles are swapped, so a lane owns four consecutive tokens of one
// feature, which is what the transposed value layout wants.
#include <cmath>
#include <cstdlib>
#include <type_traits>

#include "kernels.h"

namespace epd {

namespace {

constexpr int BM = 256;
constexpr int BK = 64;

// XOR swizzle of the 16-byte chunk index by the row
#define SWZ(row) (((row) >> 1) & 7)

__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// Configurations (BN, 512 threads, 64-wide wave tiles), one workgroup per CU, two LDS buffers:
//   BN = 256  256x256 tile, 128x64 per wave (PIPE = 1: pipelined loop; PIPE = 0:
//             both operands two slabs ahead in two register sets, fragment reads left to the
//             compiler: the reference the pipelined loop is checked against bit for bit);
//   BN = 128  256x128 tile, 64x64 per wave, PIPE = 0: one round of tiles over long K, outputs narrower than 256 columns;
//   BN = 128, BM = 128  128x128 tile, 32x64 per wave, PIPE = 0 or 2, two workgroups per CU: launches of a few
//             slices with a folded pre-norm (the others take the tiles of gemm_bf16_ring.hip).
// (Tried and dropped, none faster on the six workloads: 4 waves of 128x128 with AGPR
// accumulators, 256x128 tiles with two 4-wave workgroups per CU, 32-deep slabs.)
template <int BN, int NT, int BM_ = BM>
constexpr size_t smem_main_bytes() {
  // operand slabs, or the epilogue staging tile (BM x BN bf16 / 64 x BN fp32), whichever is larger
  constexpr size_t operands = (size_t)2 * (BM_ + BN) * BK * sizeof(bf16_t);
  constexpr size_t staging = (size_t)BM_ * BN * sizeof(bf16_t);
  return operands > staging ? operands : staging;
}

// FOLD (compiled apart so that the plain kernels keep their code and registers).  bf16-output epilogues: 2 = apply a
// folded pre-norm (GemmParams::stats).  Residual epilogue: 1 = also store the updated rows as bf16
// (GemmParams::xb), 2 = and their statistics pairs (GemmParams::stats_out).
template <int BN, int NTHREADS, int WN, int EPI, int PIPE, int BM_ = 256, int FOLD = 0>
__global__ __launch_bounds__(NTHREADS, BM_ == 128 && PIPE == 0 ? 2 : 1) void k_gemm_bf16(const GemmParams p, const int gm_, const int gw) {
  constexpr int BM = BM_;   // token rows of the tile: 256, or 128 for launches of a few slices
  static_assert(BM_ == 256 ? (PIPE <= 1 || PIPE == 3) : (BM_ == 128 && BN == 128 && (PIPE == 0 || PIPE == 2)), "tile shapes compiled");
  constexpr int NWAVES = NTHREADS / 64;
  constexpr int WAVES_N = BN / WN;           // 4 | 2
  constexpr int WAVES_M = NWAVES / WAVES_N;  // 2 | 4 | 2
  constexpr int WM = BM / WAVES_M;           // 128 | 64 | 128
  constexpr int TM = WM / 32;                // 4 | 2 | 4
  constexpr int TN = WN / 32;                // 2 | 4
  constexpr int A_LD = BM * 8 / NTHREADS;    // 16-byte chunks per thread per slab
  constexpr int B_LD = BN * 8 / NTHREADS;
  constexpr int NBUF = 2;  // LDS slab buffers
  // register sets the global loads land in = slabs they run ahead of the MFMAs.  PIPE = 2 (128 x 128
  // tiles of launches with at most one tile per CU): four, because such a launch is bound by the bytes
  // it keeps in flight, not by the matrix cores
  constexpr int NSET = PIPE == 2 ? 4 : 2;
  constexpr int ROWS_PER_LD = NTHREADS / 8;      // rows covered by one 16-byte load per thread

  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  // weight slabs first: their LDS addresses (<= 64 KiB) also serve as the 16-bit base of the
  // direct global-to-LDS loads
  bf16_t* sB = reinterpret_cast<bf16_t*>(smem);  // [NBUF][BN][64]
  bf16_t* sA = sB + NBUF * BN * BK;              // [NBUF][BM][64]
  float* sBias = reinterpret_cast<float*>(smem + smem_main_bytes<BN, NTHREADS, BM>());  // [BN]
  float* sCol = sBias + BN;   // [BN] column sums of the weights (folded pre-norm)
  float* sMu = sCol + BN;     // [BM] mean of the tile's rows
  float* sRs = sMu + BM;      // [BM] 1 / sqrt(variance + eps)
  constexpr bool BF16_OUT = !(EPI == EPI_BIAS_RESIDUAL || EPI == EPI_BIAS_POS);
  constexpr bool fold = BF16_OUT && FOLD == 2;
  constexpr bool emit = EPI == EPI_BIAS_RESIDUAL && FOLD >= 1;        // bf16 rows
  constexpr bool emit_stats = EPI == EPI_BIAS_RESIDUAL && FOLD == 2;  // and their statistics

  // Workgroups are dealt round-robin to the 8 XCDs, each with its own L2.
  // XCD x takes a contiguous run of the tile sequence, and the sequence walks
  // a band of `gw` tile columns top to bottom before moving to the next
  // band: the band's weight panel (gw * BN rows) stays L2-resident while the
  // activation panels stream through once per band.
  const int gn = p.Npad / BN;
  int id = blockIdx.x;
  {
    const int nb = gridDim.x;
    const int x = id & 7, slot = id >> 3;
    const int q = nb >> 3, r = nb & 7;
    id = x * q + (x < r ? x : r) + slot;
  }
  const int band_tiles = gm_ * gw;
  const int full_bands = gn / gw;                 // the last band may be narrower
  int band = id / band_tiles, in_band = id % band_tiles, bw = gw;
  if (band >= full_bands) { band = full_bands; in_band = id - full_bands * band_tiles; bw = gn - full_bands * gw; }
  const int m0 = (in_band / bw) * BM;
  const int n0 = (band * gw + in_band % bw) * BN;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WAVES_N, wn = wave % WAVES_N;
  (void)NWAVES;
  const int l32 = lane & 31, lh = lane >> 5;

  const int KT_ = p.K / BK;  // even (K % 128 == 0)
  // the tile's bias values wait in LDS for the epilogue (a global load there
  // would sit exposed between the last MFMA and the first store)
  if (tid < BN) sBias[tid] = p.bias[n0 + tid];
  if (fold) {   // read by the epilogue, many barriers from here
    if (tid < BN) sCol[tid] = p.colsum[n0 + tid];
    if (tid < BM) {
      const float* pairs = p.stats + (long)(m0 + tid < p.M ? m0 + tid : p.M - 1) * p.n_part * 2;   // rows past M: any valid row, never stored
      RowPairs rp;
      rp.load(pairs, p.n_part);
      float mu, rs;
      rp.finish(p.n_part, p.stat_group, p.norm_dim, p.norm_rms, p.norm_eps, mu, rs);
      sMu[tid] = mu;
      sRs[tid] = rs;
    }
  }
  const int ld_row = tid >> 3, ld_c = tid & 7;
  const int st_off = ld_row * BK + ((ld_c ^ SWZ(ld_row)) * 8);

  // global addresses = wave-uniform base (scalar registers) + one 32-bit lane offset per operand
  const unsigned a_voff = ((unsigned)ld_row * (unsigned)p.lda + ld_c * 8) * 2;   // bytes
  const unsigned b_voff = ((unsigned)ld_row * (unsigned)p.K + ld_c * 8) * 2;

  // Residual epilogue: the tile's fp32 rows are added in passes of 64 token
  // rows; the rows of pass p wait in register set p % 2, loaded two passes
  // ahead (the first two while the last slabs are multiplied), so the
  // read-modify-write never waits for memory with the MFMA pipe idle.
  constexpr int XROWS = 64;                          // token rows per fp32 epilogue pass
  constexpr int XNCH = BN * 4 / 16;                  // 16-byte chunks per staging row
  constexpr int XPER_T = XROWS * XNCH / NTHREADS;    // chunks per thread and pass
  constexpr int XSTEP = NTHREADS / XNCH;             // rows between a thread's consecutive chunks
  static_assert(NTHREADS % XNCH == 0, "a thread keeps one chunk column");
  // chunk i of a thread: tile row tid / XNCH + XSTEP * i (the same for a whole
  // wave), column chunk tid % XNCH: one lane offset serves every access, the
  // row part of the address is wave-uniform
  const int x_r0 = XNCH % 64 == 0 ? __builtin_amdgcn_readfirstlane(tid / XNCH) : tid / XNCH;  // wave-uniform when a row is >= 64 chunks
  const int x_col = n0 + (tid % XNCH) * 4;
  const bool x_col_ok = x_col < p.N;
  const unsigned x_voff = (unsigned)x_r0 * (unsigned)p.ldr + (unsigned)x_col;
  // PIPE == 1: the weight slab goes from global memory straight into LDS (no
  // staging registers), one slab ahead; only the activation slab is staged in
  // registers, two slabs ahead.
  constexpr bool B_DIRECT = PIPE == 1 || PIPE == 3;
  // PIPE == 3: the activation slab goes straight into LDS as well, one slab ahead (no staging registers at all)
  constexpr bool A_DIRECT = PIPE == 3;
  // the operand register sets can carry residual rows of the first passes when the counts match:
  // both sets = passes 0 and 1 (A and B staged), or both sets = the two halves of pass 0 (A staged only)
  constexpr bool X_IN_LOOP = EPI == EPI_BIAS_RESIDUAL &&
                             (A_DIRECT || (B_DIRECT ? XPER_T == 2 * A_LD : XPER_T == A_LD + B_LD));
  f32x4 xr[2][X_IN_LOOP ? XPER_T : 1];
  auto xload = [&](auto set, int pass) {
    if constexpr (X_IN_LOOP) {
      constexpr int S = decltype(set)::value;
      if (x_col_ok) {
#pragma unroll
        for (int i = 0; i < XPER_T; ++i) {
          const int row0 = m0 + pass * XROWS + XSTEP * i;            // uniform
          if (row0 + x_r0 < p.M) xr[S][i] = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(p.R + (long)row0 * p.ldr + x_voff));
        }
      }
    }
  };


  // Global operands are read through buffer descriptors: descriptor + scalar offset + one lane
  // offset per operand, so no per-load address arithmetic touches vector registers.  The range
  // check of a descriptor covers the lane offset only, not the scalar one: the rows of a ragged
  // last tile past M are read like any other (A and R hold round_up(M, 256) rows) and their
  // results never stored.  The host launcher checks that every extent fits 32 bits.
  __amdgpu_buffer_rsrc_t rsrc_a = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<bf16_t*>(p.A), 0, (int)(unsigned)(((long)(p.M - 1) * p.lda + p.K) * 2), 0x00020000);
  __amdgpu_buffer_rsrc_t rsrc_b = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<bf16_t*>(p.W), 0, (int)(unsigned)((long)p.Npad * p.K * 2), 0x00020000);
  __amdgpu_buffer_rsrc_t rsrc_x = __builtin_amdgcn_make_buffer_rsrc(
      p.R, 0, EPI == EPI_BIAS_RESIDUAL ? (int)(unsigned)(((long)(p.M - 1) * p.ldr + p.N) * 4) : 0, 0x00020000);

  // Two register sets: the loads of slab k+2 are in flight while slab k is
  // multiplied and slab k+1 (loaded one iteration earlier) moves to LDS.
  u32x4 ra[NSET][A_LD], rb[NSET][B_DIRECT ? 1 : B_LD];
  auto gload = [&](auto set, int kt) {
    constexpr int S = decltype(set)::value;
    // Residual epilogue: the two loads past the last slab (kt == KT_ into set
    // 0, KT_ + 1 into set 1) fetch fp32 rows of the first epilogue passes into
    // the same registers instead of re-reading operands.  Chunk c of a pass =
    // rows XSTEP * c + x_r0 of the pass, this lane's 16-byte column chunk.
    // Staged A and B: set s holds pass s, chunks 0 .. XPER_T-1; staged A only:
    // set s holds chunks s * A_LD .. of pass 0.
    const bool past = kt >= KT_;
    const int xpass = kt - KT_;
    kt = past ? KT_ - 1 : kt;  // past the end (other epilogues): re-read the last slab, result unused
    if (X_IN_LOOP && past && xpass >= 2) return;   // four register sets: only two of them carry residual rows
    if (X_IN_LOOP && past) {   // one uniform branch per slab, taken for the last two slabs of a tile
      auto so_x = [&](int c) {
        const int pass = B_DIRECT ? 0 : xpass, ci = B_DIRECT ? xpass * A_LD + c : c;
        return (unsigned)(m0 + pass * XROWS + XSTEP * ci) * (unsigned)p.ldr * 4u;
      };
#pragma unroll
      for (int i = 0; i < A_LD; ++i) ra[S][i] = __builtin_amdgcn_raw_buffer_load_b128(rsrc_x, x_voff * 4u, so_x(i), 2);
      if constexpr (!B_DIRECT) {
#pragma unroll
        for (int i = 0; i < B_LD; ++i)
          rb[S][i] = __builtin_amdgcn_raw_buffer_load_b128(rsrc_x, x_voff * 4u, so_x(A_LD + i), 2);
      }
    } else {
#pragma unroll
      for (int i = 0; i < A_LD; ++i) {
        const unsigned so = ((unsigned)(m0 + ROWS_PER_LD * i) * (unsigned)p.lda + (unsigned)(kt * BK)) * 2u;
        ra[S][i] = __builtin_amdgcn_raw_buffer_load_b128(rsrc_a, a_voff, so, 0);
      }
      if constexpr (!B_DIRECT) {
#pragma unroll
        for (int i = 0; i < B_LD; ++i) {
          const unsigned so = ((unsigned)(n0 + ROWS_PER_LD * i) * (unsigned)p.K + (unsigned)(kt * BK)) * 2u;
          rb[S][i] = __builtin_amdgcn_raw_buffer_load_b128(rsrc_b, b_voff, so, 0);
        }
      }
    }
  };
  // Weight slab kt -> LDS buffer buf without passing through registers.  The
  // hardware puts lane l's 16 bytes at (wave-uniform LDS base) + 16 l, so a
  // wave fills 1 KiB = 8 slab rows linearly; the swizzle is applied on the
  // global side instead: the lane that lands on physical chunk ld_c of its row
  // fetches logical chunk ld_c ^ SWZ(row).
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);
  const unsigned bd_voff = ((unsigned)ld_row * (unsigned)p.K + ((ld_c ^ SWZ(ld_row)) * 8)) * 2;
  auto bload = [&](int buf, int kt) {
    if constexpr (B_DIRECT) {
#pragma unroll
      for (int i = 0; i < B_LD; ++i) {
        const bf16_t* g = p.W + (long)(n0 + ROWS_PER_LD * i) * p.K + kt * BK;   // uniform
        bf16_t* l = sB + buf * BN * BK + (wave_u * 64 + NTHREADS * i) * 8;
        // Written as assembly on purpose: for the builtin form the compiler makes every later
        // LDS read wait for ALL outstanding vector-memory loads (it cannot tell the two LDS
        // buffers apart), which would serialise the pipeline.  Completion is awaited
        // explicitly (wait_vm) in front of the barrier that publishes the buffer.
        const unsigned lds_addr = (unsigned)(size_t)(__attribute__((address_space(3))) void*)l;
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                     :: "v"(bd_voff), "s"(g), "s"(lds_addr) : "memory", "m0");
      }
    }
  };
  // PIPE == 3: activation slab kt -> LDS buffer buf, same scheme (LDS-DMA reaches the whole LDS through M0 on gfx950)
  const unsigned ad_voff = ((unsigned)ld_row * (unsigned)p.lda + ((ld_c ^ SWZ(ld_row)) * 8)) * 2;
  auto aload = [&](int buf, int kt) {
    if constexpr (A_DIRECT) {
#pragma unroll
      for (int i = 0; i < A_LD; ++i) {
        const bf16_t* g = p.A + (long)(m0 + ROWS_PER_LD * i) * p.lda + kt * BK;   // uniform
        bf16_t* l = sA + buf * BM * BK + (wave_u * 64 + NTHREADS * i) * 8;
        const unsigned lds_addr = (unsigned)(size_t)(__attribute__((address_space(3))) void*)l;
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                     :: "v"(ad_voff), "s"(g), "s"(lds_addr) : "memory", "m0");
      }
    }
  };
  // wait until at most n of this wave's vector-memory loads are outstanding (they complete in order)
  auto wait_vm = [&](auto n) {
    constexpr int N = decltype(n)::value;
    __builtin_amdgcn_s_waitcnt((N & 0xf) | ((N >> 4) << 14) | (0x7 << 4) | (0xf << 8));
  };
  auto sstore = [&](auto set, int buf) {
    constexpr int S = decltype(set)::value;
#pragma unroll
    for (int i = 0; i < A_LD; ++i)
      *reinterpret_cast<u32x4*>(sA + buf * BM * BK + ROWS_PER_LD * i * BK + st_off) = ra[S][i];
    if constexpr (!B_DIRECT) {
#pragma unroll
      for (int i = 0; i < B_LD; ++i)
        *reinterpret_cast<u32x4*>(sB + buf * BN * BK + ROWS_PER_LD * i * BK + st_off) = rb[S][i];
    }
  };

  // attention values: token-major MFMA result, stored transposed
  constexpr bool tok_major = (EPI == EPI_VT);

  f32x16 acc[TM][TN];
  const int frag_sw = SWZ(l32);
  auto compute = [&](int buf) {
    const bf16_t* a_s = sA + buf * BM * BK + (wm * WM + l32) * BK;
    const bf16_t* b_s = sB + buf * BN * BK + (wn * WN + l32) * BK;
    if constexpr (TM * TN <= 2) {
      // Small tiles run alone on their CU and their time is the chain LDS read -> MFMA of one wave:
      // all fragments of the slab are read first (two k-steps' worth per batch of registers), so the
      // LDS latency is paid once per half slab instead of once per k-step.  The k-steps of an element
      // are still added in order.
#pragma unroll
      for (int k2 = 0; k2 < BK / 16; k2 += 2) {
        bf16x8 xf[2][TM], wf[2][TN];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const int coff = (((2 * (k2 + q) + lh) ^ frag_sw) * 8);
#pragma unroll
          for (int i = 0; i < TM; ++i) xf[q][i] = *reinterpret_cast<const bf16x8*>(a_s + i * 32 * BK + coff);
#pragma unroll
          for (int j = 0; j < TN; ++j) wf[q][j] = *reinterpret_cast<const bf16x8*>(b_s + j * 32 * BK + coff);
        }
        __builtin_amdgcn_sched_barrier(0);   // the scheduler would otherwise sink each read to its MFMA
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
          for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
              acc[i][j] = tok_major ? mfma32(xf[q][i], wf[q][j], acc[i][j]) : mfma32(wf[q][j], xf[q][i], acc[i][j]);
      }
      return;
    }
#pragma unroll
    for (int kk = 0; kk < BK / 16; ++kk) {
      const int coff = (((2 * kk + lh) ^ frag_sw) * 8);
      bf16x8 xf[TM], wf[TN];
#pragma unroll
      for (int i = 0; i < TM; ++i) xf[i] = *reinterpret_cast<const bf16x8*>(a_s + i * 32 * BK + coff);
#pragma unroll
      for (int j = 0; j < TN; ++j) wf[j] = *reinterpret_cast<const bf16x8*>(b_s + j * 32 * BK + coff);
      if (tok_major) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j) acc[i][j] = mfma32(xf[i], wf[j], acc[i][j]);
      } else {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j) acc[i][j] = mfma32(wf[j], xf[i], acc[i][j]);
      }
    }
  };

  using S0 = std::integral_constant<int, 0>;
  using S1 = std::integral_constant<int, 1>;

#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
  if constexpr (PIPE == 1 || PIPE == 3) {
    // The operand fragments run one k-step ahead of the MFMAs in a second
    // register set, so a wave issues its MFMAs back to back instead of
    // waiting for LDS in front of every k-step; the slab hand-over (LDS
    // stores of the next slab + barrier) sits in front of the LAST k-step,
    // whose MFMAs cover the first fragment reads from the other buffer.
    bf16x8 fa[2][TM], fb[2][TN];
    auto ldfrag = [&](auto set, int buf, int kk) {
      constexpr int S = decltype(set)::value;
      const bf16_t* a_s = sA + buf * BM * BK + (wm * WM + l32) * BK;
      const bf16_t* b_s = sB + buf * BN * BK + (wn * WN + l32) * BK;
      const int coff = (((2 * kk + lh) ^ frag_sw) * 8);
#pragma unroll
      for (int i = 0; i < TM; ++i) fa[S][i] = *reinterpret_cast<const bf16x8*>(a_s + i * 32 * BK + coff);
#pragma unroll
      for (int j = 0; j < TN; ++j) fb[S][j] = *reinterpret_cast<const bf16x8*>(b_s + j * 32 * BK + coff);
    };
    auto mma = [&](auto set) {
      constexpr int S = decltype(set)::value;
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = tok_major ? mfma32(fa[S][i], fb[S][j], acc[i][j]) : mfma32(fb[S][j], fa[S][i], acc[i][j]);
    };
    // scheduling hint: spread the TM + TN LDS reads of the next k-step over the TM * TN MFMAs of this one
    auto interleave = [&]() {
      constexpr int PER = (TM * TN) / (TM + TN) > 0 ? (TM * TN) / (TM + TN) : 1;
#pragma unroll
      for (int i = 0; i < TM + TN; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, PER, 0);  // MFMA
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);    // DS read
      }
    };
    // The hand-over is unconditional so that a slab is straight-line code: behind the last slab it
    // re-reads the last weight slab and parks stale registers in the idle buffer, nobody reads them.
    auto slab = [&](auto lset, auto sset, int buf, int kt) {
      bload(buf ^ 1, kt + 1 < KT_ ? kt + 1 : KT_ - 1);  // the other buffer is free since the last barrier
      gload(lset, kt + 2);   // past the last slab: residual rows of the first epilogue passes (see gload)
      // the loads stay in front of the slab's arithmetic: moved down by the scheduler they would
      // share registers with the fragments and lose half of their head start
      __builtin_amdgcn_sched_barrier(0);
      ldfrag(S1{}, buf, 1); mma(S0{}); interleave();
      ldfrag(S0{}, buf, 2); mma(S1{}); interleave();
      ldfrag(S1{}, buf, 3); mma(S0{}); interleave();
      __builtin_amdgcn_sched_barrier(0);   // the LDS stores wait for loads issued a slab ago: keep them late
      sstore(sset, buf ^ 1);
      if constexpr (B_DIRECT) wait_vm(std::integral_constant<int, A_LD>{});  // all but the newest A loads: the weight slab has landed
      __syncthreads();
      ldfrag(S0{}, buf ^ 1, 0); mma(S1{}); interleave();
    };
    // PIPE == 3: both slabs of step kt + 1 are in flight towards the other buffer while step kt is multiplied.
    // The last two steps also start the residual rows of the first two epilogue passes (PHASE 1: the step
    // before the last, whose wait leaves those newest loads in flight; PHASE 2: the last step, which has
    // nothing to fetch for the product).
    // residual rows of an epilogue pass through the buffer descriptor: every lane of every wave issues exactly
    // XPER_T loads whatever the tile's position (rows past M are read like any other, columns past N come back
    // as zero), so the wait below can count them
    auto xload_all = [&](auto set, int pass) {
      if constexpr (X_IN_LOOP) {
        constexpr int S = decltype(set)::value;
#pragma unroll
        for (int i = 0; i < XPER_T; ++i)
          xr[S][i] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(
              rsrc_x, x_voff * 4u, (unsigned)(m0 + pass * XROWS + XSTEP * i) * (unsigned)p.ldr * 4u, 2));
      }
    };
    auto slab_direct = [&](int buf, int kt, auto phase) {
      constexpr int PHASE = decltype(phase)::value;
      if constexpr (PHASE < 2) { bload(buf ^ 1, kt + 1); aload(buf ^ 1, kt + 1); }
      if constexpr (PHASE == 1) xload_all(S0{}, 0);
      if constexpr (PHASE == 2) xload_all(S1{}, 1);
      __builtin_amdgcn_sched_barrier(0);
      ldfrag(S1{}, buf, 1); mma(S0{}); interleave();
      ldfrag(S0{}, buf, 2); mma(S1{}); interleave();
      ldfrag(S1{}, buf, 3); mma(S0{}); interleave();
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (PHASE < 2) {
        // both slabs have landed in the other buffer (loads complete in order: the residual rows are newer)
        wait_vm(std::integral_constant<int, (PHASE == 1 && X_IN_LOOP) ? XPER_T : 0>{});
        __syncthreads();
        ldfrag(S0{}, buf ^ 1, 0);
      }
      mma(S1{});
      if constexpr (PHASE < 2) interleave();
    };
    using P0 = std::integral_constant<int, 0>;
    using P1 = std::integral_constant<int, 1>;
    using P2 = std::integral_constant<int, 2>;
    if constexpr (A_DIRECT) {
      bload(0, 0);
      aload(0, 0);
      wait_vm(std::integral_constant<int, 0>{});
      __syncthreads();
      ldfrag(S0{}, 0, 0);
      for (int kt = 0; kt < KT_ - 2; kt += 2) {
        slab_direct(0, kt, P0{});
        slab_direct(1, kt + 1, P0{});
      }
      slab_direct(0, KT_ - 2, P1{});
      slab_direct(1, KT_ - 1, P2{});
    } else {
    bload(0, 0);
    gload(S0{}, 0);
    gload(S1{}, 1);
    sstore(S0{}, 0);
    // loads complete in order: once all but the newest A_LD (slab 1's) are done, weight slab 0 has landed
    if constexpr (B_DIRECT) wait_vm(std::integral_constant<int, A_LD>{});
    __syncthreads();
    ldfrag(S0{}, 0, 0);
    for (int kt = 0; kt < KT_; kt += 2) {
      slab(S0{}, S1{}, 0, kt);
      slab(S1{}, S0{}, 1, kt + 1);
    }
    }
    if constexpr (X_IN_LOOP && B_DIRECT && !A_DIRECT) {
#pragma unroll
      for (int i = 0; i < XPER_T; ++i) xr[0][i] = __builtin_bit_cast(f32x4, ra[i / A_LD][i % A_LD]);
      xload(S1{}, 1);   // into the registers the operand fragments have left
    } else if constexpr (X_IN_LOOP && !A_DIRECT) {
#pragma unroll
      for (int i = 0; i < XPER_T; ++i) {
        xr[0][i] = __builtin_bit_cast(f32x4, i < A_LD ? ra[0][i < A_LD ? i : 0] : rb[0][i < A_LD ? 0 : i - A_LD]);
        xr[1][i] = __builtin_bit_cast(f32x4, i < A_LD ? ra[1][i < A_LD ? i : 0] : rb[1][i < A_LD ? 0 : i - A_LD]);
      }
    }
  } else if constexpr (PIPE == 2) {
    // four slabs ahead (the launcher takes this form only for K % 256 == 0)
    using S2 = std::integral_constant<int, 2>;
    using S3 = std::integral_constant<int, 3>;
    gload(S0{}, 0);
    gload(S1{}, 1);
    gload(S2{}, 2);
    gload(S3{}, 3);
    sstore(S0{}, 0);
    __syncthreads();
    for (int kt = 0; kt < KT_; kt += 4) {
      gload(S0{}, kt + 4);   // past the last slab: residual rows of epilogue pass 0 (see gload)
      compute(0);
      sstore(S1{}, 1);
      __syncthreads();
      gload(S1{}, kt + 5);   // ... and of pass 1
      compute(1);
      sstore(S2{}, 0);
      __syncthreads();
      gload(S2{}, kt + 6);
      compute(0);
      sstore(S3{}, 1);
      __syncthreads();
      gload(S3{}, kt + 7);
      compute(1);
      if (X_IN_LOOP && kt + 4 >= KT_) break;   // nothing left to hand over
      sstore(S0{}, 0);
      __syncthreads();
    }
    if constexpr (X_IN_LOOP) {
#pragma unroll
      for (int i = 0; i < XPER_T; ++i) {
        xr[0][i] = __builtin_bit_cast(f32x4, i < A_LD ? ra[0][i < A_LD ? i : 0] : rb[0][i < A_LD ? 0 : i - A_LD]);
        xr[1][i] = __builtin_bit_cast(f32x4, i < A_LD ? ra[1][i < A_LD ? i : 0] : rb[1][i < A_LD ? 0 : i - A_LD]);
      }
    }
  } else {
    gload(S0{}, 0);
    gload(S1{}, 1);
    sstore(S0{}, 0);
    __syncthreads();
    for (int kt = 0; kt < KT_; kt += 2) {
      gload(S0{}, kt + 2);   // past the last slab: residual rows of epilogue pass 0 (see gload)
      compute(0);
      sstore(S1{}, 1);
      __syncthreads();
      gload(S1{}, kt + 3);   // ... and of pass 1
      compute(1);
      if (X_IN_LOOP && kt + 2 >= KT_) break;   // nothing left to hand over
      sstore(S0{}, 0);
      __syncthreads();
    }
    if constexpr (X_IN_LOOP) {
#pragma unroll
      for (int i = 0; i < XPER_T; ++i) {
        xr[0][i] = __builtin_bit_cast(f32x4, i < A_LD ? ra[0][i < A_LD ? i : 0] : rb[0][i < A_LD ? 0 : i - A_LD]);
        xr[1][i] = __builtin_bit_cast(f32x4, i < A_LD ? ra[1][i < A_LD ? i : 0] : rb[1][i < A_LD ? 0 : i - A_LD]);
      }
    }
  }

  // ------------------------------------------------------------ epilogue ----
  // The accumulators go through LDS (the operand buffers are idle now) so
  // that global memory sees whole 16-byte chunks of consecutive rows: a lane
  // owns one staging row (l32) and four consecutive columns per register
  // group; chunk c of staging row r sits at physical chunk c ^ (r & 15), which
  // spreads the 16 rows of an access phase over all banks.
  __syncthreads();  // every wave is done reading the operand buffers
  unsigned char* stage = smem;

  if (EPI == EPI_BIAS_RESIDUAL || EPI == EPI_BIAS_POS) {
    // fp32 staging, XROWS token rows per pass: [XROWS][BN] floats
    constexpr int ROWB = BN * 4;          // bytes per staging row
    constexpr int PASSES = BM / XROWS;
    auto fp32_pass = [&](auto set, int pass) {
      constexpr int S = decltype(set)::value;
      if (pass > 0) __syncthreads();
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const int base = wm * WM + i * 32;            // first tile row of this 32-row group
        if (base / XROWS != pass) continue;            // wave-uniform
        const int r = base % XROWS + l32;
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int gi = 0; gi < 4; ++gi) {
            const int cl = wn * WN + j * 32 + gi * 8 + lh * 4;  // column inside the tile
            const float4 b4 = *reinterpret_cast<const float4*>(sBias + cl);
            f32x4 v = {acc[i][j][gi * 4 + 0] + b4.x, acc[i][j][gi * 4 + 1] + b4.y,
                       acc[i][j][gi * 4 + 2] + b4.z, acc[i][j][gi * 4 + 3] + b4.w};
            *reinterpret_cast<f32x4*>(stage + r * ROWB + (((cl >> 2) ^ (r & 15)) << 4)) = v;
          }
      }
      __syncthreads();
      // The sums leave through global stores.  The 128-bit buffer store with a scalar offset is no
      // alternative here: the compiler puts no wait state behind that form, and with the next chunk's
      // additions rewriting its data registers in the following cycle a stored row was wrong once in
      // about 1e8 stores on gfx950 (gone with one s_nop behind each store, no faster than this form).
      if constexpr (emit) {
        // The updated rows also leave as bf16 (the operand of the next product, whose pre-norm is folded into
        // its weights) together with their statistics pairs.  A half-wave holds one row's 128-column group,
        // four values per lane, whatever the tile shape, so the pairs carry the same bits for every shape.
        const int c = tid % XNCH;
        const int grp = x_col / STAT_GROUP;
        const int left = p.N - grp * STAT_GROUP;
        const float inv_cnt = left <= 0 ? 0.f : 1.0f / (float)(left < STAT_GROUP ? left : STAT_GROUP);
#pragma unroll
        for (int i = 0; i < XPER_T; ++i) {
          const int r = x_r0 + XSTEP * i;
          const int row = m0 + pass * XROWS + XSTEP * i + x_r0;
          const bool ok = x_col_ok && row < p.M;
          f32x4 sum = {0.f, 0.f, 0.f, 0.f};
          if (ok) {
            const f32x4 v = *reinterpret_cast<const f32x4*>(stage + r * ROWB + ((c ^ (r & 15)) << 4));
            f32x4* dst = reinterpret_cast<f32x4*>(p.R + (long)(row - x_r0) * p.ldr + x_voff);
            if constexpr (X_IN_LOOP) { sum = xr[S][i] + v; __builtin_nontemporal_store(sum, dst); }
            else { sum = *dst + v; *dst = sum; }
            bf16x4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = (bf16_t)sum[e];
            *reinterpret_cast<bf16x4*>(p.xb + (long)row * p.ldxb + x_col) = o;
          }
          if constexpr (emit_stats) {
            float mean, m2;
            group_mean_m2(sum, ok, inv_cnt, mean, m2);
            if ((tid & 31) == 0 && row < p.M && grp < p.n_part_out)
              *reinterpret_cast<float2*>(p.stats_out + ((long)row * p.n_part_out + grp) * 2) = make_float2(mean, m2);
          }
        }
      } else if (x_col_ok) {
        const int c = tid % XNCH;
#pragma unroll
        for (int i = 0; i < XPER_T; ++i) {
          const int r = x_r0 + XSTEP * i;
          const int row0 = m0 + pass * XROWS + XSTEP * i;              // uniform
          if (row0 + x_r0 < p.M) {
            const f32x4 v = *reinterpret_cast<const f32x4*>(stage + r * ROWB + ((c ^ (r & 15)) << 4));
            f32x4* dst = reinterpret_cast<f32x4*>(p.R + (long)row0 * p.ldr + x_voff);
            if (EPI == EPI_BIAS_RESIDUAL) {
              if constexpr (X_IN_LOOP) __builtin_nontemporal_store(xr[S][i] + v, dst);   // streamed: read next by a row kernel, not by this launch
              else *dst = *dst + v;      // other tile shapes: plain read-modify-write
            } else {   // patch embedding: position row by patch index, output row through the slice layout
              const int row = row0 + x_r0;
              *reinterpret_cast<f32x4*>(p.R + p.xrows.row(row) * p.ldr + x_col) =
                  v + *reinterpret_cast<const f32x4*>(p.pos + (long)(row % p.n_pos) * p.N + x_col);
            }
          }
        }
      }
      if (pass + 2 < PASSES) xload(set, pass + 2);
    };
#pragma unroll
    for (int pass = 0; pass < PASSES; pass += 2) {
      fp32_pass(S0{}, pass);
      fp32_pass(S1{}, pass + 1);
    }
  } else {
  // bf16 staging of the whole tile: rows = MFMA lane dimension
  constexpr int SROWS = tok_major ? BN : BM;   // staging rows
  constexpr int SCOLS = tok_major ? BM : BN;   // staging columns
  constexpr int ROWB = SCOLS * 2;
  constexpr int NCH = ROWB / 16;
  constexpr int PER_T = SROWS * NCH / NTHREADS;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      // lane dimension: feature (tok_major) or token; register dimension: the other one
      const int r = tok_major ? (wn * WN + j * 32 + l32) : (wm * WM + i * 32 + l32);
      // the lane's own scalars: bias and column sum of its feature (tok_major), or mean / rstd of its token
      float bl = 0.f, cs = 0.f, mu = 0.f, rs = 1.f;
      if (tok_major) { bl = sBias[r]; if (fold) cs = sCol[r]; }
      else if (fold) { mu = sMu[r]; rs = sRs[r]; }
#pragma unroll
      for (int gi = 0; gi < 4; ++gi) {
        const int cl = (tok_major ? (wm * WM + i * 32) : (wn * WN + j * 32)) + gi * 8 + lh * 4;
        float v[4];
        if (tok_major) {
          if (fold) {   // rstd_t (acc - mean_t colsum) + bias over four consecutive tokens t
            const f32x4 m4 = *reinterpret_cast<const f32x4*>(sMu + cl), r4 = *reinterpret_cast<const f32x4*>(sRs + cl);
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = __builtin_fmaf(r4[e], __builtin_fmaf(-m4[e], cs, acc[i][j][gi * 4 + e]), bl);
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = acc[i][j][gi * 4 + e] + bl;
          }
        } else {
          const f32x4 b4 = *reinterpret_cast<const f32x4*>(sBias + cl);
          if (fold) {
            const f32x4 c4 = *reinterpret_cast<const f32x4*>(sCol + cl);
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = __builtin_fmaf(rs, __builtin_fmaf(-mu, c4[e], acc[i][j][gi * 4 + e]), b4[e]);
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = acc[i][j][gi * 4 + e] + b4[e];
          }
        }
        bf16x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = (bf16_t)apply_act_fast<EPI>(v[e]);
        *reinterpret_cast<bf16x4*>(stage + r * ROWB + (((cl >> 3) ^ (r & 15)) << 4) + ((cl & 4) << 1)) = o;
      }
    }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < PER_T; ++i) {
    const int q = tid + NTHREADS * i;
    const int r = q / NCH, c = q % NCH;
    const u32x4 v = *reinterpret_cast<const u32x4*>(stage + r * ROWB + ((c ^ (r & 15)) << 4));
    if (tok_major) {
      const int f = n0 + r, tok = m0 + c * 8;
      if (f < p.N && tok < p.M) {
        const int h = f / p.hd_pad, d = f % p.hd_pad;
        const int t = tok / p.n_tok, n = tok % p.n_tok;
        __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(p.VT + (((long)t * p.heads + h) * p.hd_pad + d) * p.n_tok + n));
      }
    } else {
      const int row = m0 + r, col = n0 + c * 8;
      if (row < p.M && col < p.N) {
        const long orow = p.row_map ? (long)p.row_map[row / p.block_tokens] * p.block_tokens + row % p.block_tokens : row;
        __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(p.C + orow * p.ldc + col));
      }
    }
  }
  }  // staging kind
}


// ---------------------------------------------------------------------------
// Persistent form of the default shape (256 x 256 x 64 tile, 8 waves, pipelined
// loop) for the epilogues with bf16 output.  One workgroup per CU walks the
// tile sequence with stride gridDim.x.  The loads that would run past the last
// slab of a tile fetch the first two slabs of the workgroup's NEXT tile instead
// (slab 0 into LDS buffer 0, slab 1 into a register set), and the epilogue
// stages the finished tile through LDS buffer 1 only, in two passes of 128
// rows: the next tile's main loop starts right behind the last store, without
// the launch gap and the exposed first-slab latency a fresh workgroup pays.
// ---------------------------------------------------------------------------
// For products with a folded pre-norm; the others run on gemm_bf16_wide.h.
template <int EPI>
__global__ __launch_bounds__(512, 1) void k_gemm_bf16_persist(const GemmParams p, const int gm_, const int gw,
                                                              const int n_tiles) {
  constexpr int BN = 256, NTHREADS = 512, WN = 64, WAVES_N = 4, WM = 128, TM = 4, TN = 2;
  constexpr int A_LD = 4, B_LD = 4, ROWS_PER_LD = 64;
  constexpr bool tok_major = (EPI == EPI_VT);
  static_assert(EPI != EPI_BIAS_RESIDUAL && EPI != EPI_BIAS_POS, "bf16-output epilogues only");

  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  bf16_t* sB = reinterpret_cast<bf16_t*>(smem);  // [2][BN][64]: bytes 0 .. 64 Ki
  bf16_t* sA = sB + 2 * BN * BK;                 // [2][BM][64]: bytes 64 Ki .. 128 Ki
  float* sBias = reinterpret_cast<float*>(smem + smem_main_bytes<BN, NTHREADS>());
  float* sCol = sBias + BN;   // column sums of the weights, mean and rstd of the tile's rows (folded pre-norm)
  float* sMu = sCol + BN;
  float* sRs = sMu + BM;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WAVES_N, wn = wave % WAVES_N;
  const int l32 = lane & 31, lh = lane >> 5;
  const int KT_ = p.K / BK;  // even
  const int gn = p.Npad / BN;
  // Per-tile scalars of the epilogue: bias, the column sums of the weights and
  // mean / rstd of the tile's rows.  The statistics pairs of the NEXT tile's rows are loaded into registers at
  // the start of a tile's epilogue (one thread per row, one batch of independent loads whose latency passes
  // under the epilogue) and combined at its end, when nobody reads the current tile's scalars any more.
  // (The register copy of the pairs lives inside one epilogue: a variable carried around the tile loop would
  // occupy its registers through the main loop as well.)
  // (t: the calling thread's index, handed in so that the epilogue can pass its opaque copy, see there)
  auto pairs_of = [&](int t, int mrow0) {
    return p.stats + (long)(mrow0 + t < p.M ? mrow0 + t : p.M - 1) * p.n_part * 2;   // rows past M: any valid row, never stored
  };
  auto stats_load = [&](int t, RowPairs& rp, int mrow0) { if (t < BM) rp.load(pairs_of(t, mrow0), p.n_part); };
  auto tile_scalars = [&](int t, const RowPairs& rp, int mrow0, int ncol0) {
    if (t < BN) { sBias[t] = p.bias[ncol0 + t]; sCol[t] = p.colsum[ncol0 + t]; }
    if (t < BM) {
      float mu, rs;
      rp.finish(p.n_part, p.stat_group, p.norm_dim, p.norm_rms, p.norm_eps, mu, rs);
      sMu[t] = mu;
      sRs[t] = rs;
    }
  };

  // position in the launch order -> tile (same XCD-aware band order as the one-tile kernel; a
  // persistent workgroup keeps pos % 8, i.e. its XCD)
  auto tile_of = [&](int pos, int& m0, int& n0) {
    const int x = pos & 7, slot = pos >> 3;
    const int q = n_tiles >> 3, r = n_tiles & 7;
    const int id = x * q + (x < r ? x : r) + slot;
    const int band_tiles = gm_ * gw;
    const int full_bands = gn / gw;
    int band = id / band_tiles, in_band = id % band_tiles, bw = gw;
    if (band >= full_bands) { band = full_bands; in_band = id - full_bands * band_tiles; bw = gn - full_bands * gw; }
    m0 = (in_band / bw) * BM;
    n0 = (band * gw + in_band % bw) * BN;
  };

  const int ld_row = tid >> 3, ld_c = tid & 7;
  const int st_off = ld_row * BK + ((ld_c ^ SWZ(ld_row)) * 8);
  const unsigned a_voff = ((unsigned)ld_row * (unsigned)p.lda + ld_c * 8) * 2;
  const unsigned bd_voff = ((unsigned)ld_row * (unsigned)p.K + ((ld_c ^ SWZ(ld_row)) * 8)) * 2;
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);
  __amdgpu_buffer_rsrc_t rsrc_a = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<bf16_t*>(p.A), 0, (int)(unsigned)(((long)(p.M - 1) * p.lda + p.K) * 2), 0x00020000);

  __amdgpu_buffer_rsrc_t rsrc_c = __builtin_amdgcn_make_buffer_rsrc(
      p.C, 0, (tok_major || !p.C) ? 0 : (int)(unsigned)(((long)(p.M - 1) * p.ldc + p.N) * 2), 0x00020000);

  u32x4 ra[2][A_LD];
  auto gload = [&](auto set, int mrow0, int kt) {   // activation slab kt of the tile rows mrow0 ..
    constexpr int S = decltype(set)::value;
#pragma unroll
    for (int i = 0; i < A_LD; ++i) {
      const unsigned so = ((unsigned)(mrow0 + ROWS_PER_LD * i) * (unsigned)p.lda + (unsigned)(kt * BK)) * 2u;
      ra[S][i] = __builtin_amdgcn_raw_buffer_load_b128(rsrc_a, a_voff, so, 0);
    }
  };
  auto bload = [&](int buf, int ncol0, int kt) {    // weight slab kt of the tile columns ncol0 .. -> LDS
#pragma unroll
    for (int i = 0; i < B_LD; ++i) {
      const bf16_t* g = p.W + (long)(ncol0 + ROWS_PER_LD * i) * p.K + kt * BK;   // uniform
      bf16_t* l = sB + buf * BN * BK + (wave_u * 64 + NTHREADS * i) * 8;
      const unsigned lds_addr = (unsigned)(size_t)(__attribute__((address_space(3))) void*)l;
      asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                   :: "v"(bd_voff), "s"(g), "s"(lds_addr) : "memory", "m0");
    }
  };
  auto sstore = [&](auto set, int buf) {
    constexpr int S = decltype(set)::value;
#pragma unroll
    for (int i = 0; i < A_LD; ++i)
      *reinterpret_cast<u32x4*>(sA + buf * BM * BK + ROWS_PER_LD * i * BK + st_off) = ra[S][i];
  };
  auto wait_vm = [&](auto n) {
    constexpr int N = decltype(n)::value;
    __builtin_amdgcn_s_waitcnt((N & 0xf) | ((N >> 4) << 14) | (0x7 << 4) | (0xf << 8));
  };

  f32x16 acc[TM][TN];
  bf16x8 fa[2][TM], fb[2][TN];
  const int frag_sw = SWZ(l32);
  auto ldfrag = [&](auto set, int buf, int kk) {
    constexpr int S = decltype(set)::value;
    const bf16_t* a_s = sA + buf * BM * BK + (wm * WM + l32) * BK;
    const bf16_t* b_s = sB + buf * BN * BK + (wn * WN + l32) * BK;
    const int coff = (((2 * kk + lh) ^ frag_sw) * 8);
#pragma unroll
    for (int i = 0; i < TM; ++i) fa[S][i] = *reinterpret_cast<const bf16x8*>(a_s + i * 32 * BK + coff);
#pragma unroll
    for (int j = 0; j < TN; ++j) fb[S][j] = *reinterpret_cast<const bf16x8*>(b_s + j * 32 * BK + coff);
  };
  auto mma = [&](auto set) {
    constexpr int S = decltype(set)::value;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
        acc[i][j] = tok_major ? mfma32(fa[S][i], fb[S][j], acc[i][j]) : mfma32(fb[S][j], fa[S][i], acc[i][j]);
  };
  auto interleave = [&]() {
#pragma unroll
    for (int i = 0; i < TM + TN; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);  // DS read
    }
  };
  using S0 = std::integral_constant<int, 0>;
  using S1 = std::integral_constant<int, 1>;
  using VM_A = std::integral_constant<int, A_LD>;

  int pos = blockIdx.x, m0, n0, m0n, n0n;
  tile_of(pos, m0, n0);
  {
    RowPairs rp0;
    stats_load(tid, rp0, m0);
    tile_scalars(tid, rp0, m0, n0);
  }
  bload(0, n0, 0);
  gload(S0{}, m0, 0);
  gload(S1{}, m0, 1);
  sstore(S0{}, 0);
  wait_vm(VM_A{});   // loads complete in order: all but slab 1's are done, weight slab 0 has landed
  __syncthreads();

  for (;;) {
    ldfrag(S0{}, 0, 0);   // (the copy the last hand-over of the previous tile read is not kept across the epilogue)
    const int nxt = pos + (int)gridDim.x;
    const bool has_next = nxt < n_tiles;
    if (has_next) tile_of(nxt, m0n, n0n); else { m0n = m0; n0n = n0; }   // no next tile: harmless re-reads
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

    // slab kt sits in LDS buffer `buf` with its first fragments in set 0; slab kt+1 in the register
    // set `sset`.  Slab indices past the tile's end name the first slabs of the next tile.
    auto slab = [&](auto lset, auto sset, int buf, int kt) {
      const bool w_own = kt + 1 < KT_, a_own = kt + 2 < KT_;
      bload(buf ^ 1, w_own ? n0 : n0n, w_own ? kt + 1 : kt + 1 - KT_);
      gload(lset, a_own ? m0 : m0n, a_own ? kt + 2 : kt + 2 - KT_);
      __builtin_amdgcn_sched_barrier(0);
      ldfrag(S1{}, buf, 1); mma(S0{}); interleave();
      ldfrag(S0{}, buf, 2); mma(S1{}); interleave();
      ldfrag(S1{}, buf, 3); mma(S0{}); interleave();
      __builtin_amdgcn_sched_barrier(0);
      sstore(sset, buf ^ 1);
      wait_vm(VM_A{});
      __syncthreads();
      ldfrag(S0{}, buf ^ 1, 0); mma(S1{}); interleave();
    };
    for (int kt = 0; kt < KT_; kt += 2) {
      slab(S0{}, S1{}, 0, kt);
      slab(S1{}, S0{}, 1, kt + 1);
    }
    // Here LDS buffer 0 holds slab 0 of the next tile and register set 1 holds its slab 1; nobody reads buffer 1 any more (the reads of the last slab were
    // complete at the barrier inside its hand-over).

    // ---- epilogue through LDS buffer 1: staging rows 0..63 of a pass in sB[1], 64..127 in sA[1] ----
    {
    // The epilogue's addresses derive from the thread index through an opaque copy, made anew for every tile:
    // computed once in front of the tile loop (they are loop invariants) they would sit in registers, that is
    // in scratch memory, through the main loop, and every tile would wait for their reloads before its
    // epilogue; recomputing them is a few dozen integer operations.
    int tid_opaque = threadIdx.x;
    asm volatile("" : "+v"(tid_opaque));
    const int tid = tid_opaque, lane = tid & 63, wave = tid >> 6;
    const int wm = wave / WAVES_N, wn = wave % WAVES_N;
    const int l32 = lane & 31, lh = lane >> 5;
    constexpr int ROWB = 512, NCH = 32;
    auto stage_row = [&](int r) -> unsigned char* {   // r = 0..127 inside the pass
      return reinterpret_cast<unsigned char*>(r < 64 ? sB + BN * BK : sA + BM * BK) + (r & 63) * ROWB;
    };
    // Every wave stages half of its own sub-tiles per pass (token-major result: its 32-row group
    // j == pass of both halves i; otherwise its groups i = 2 pass, 2 pass + 1), so a pass holds 128
    // staging rows: slot (r / G) * G + r % G  <->  tile row (slot / G) * 2G + pass * G + slot % G,
    // G = 32 (token-major) or 64.
    constexpr int G = tok_major ? 32 : 64;
    RowPairs rp;
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
      if (pass > 0) {
        __syncthreads();       // pass 0 has been read out
        stats_load(tid, rp, m0n);   // half of the accumulators are gone: room for the next tile's pairs (no next tile: m0n = m0, harmless re-read)
      }
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          if ((tok_major ? j : i / 2) != pass) continue;
          // lane dimension: feature (tok_major) or token; register dimension: the other one
          const int rg = tok_major ? (wn * WN + j * 32 + l32) : (wm * WM + i * 32 + l32);
          const int r = (rg / (2 * G)) * G + rg % G;
          float bl = 0.f, cs = 0.f, mu = 0.f, rs = 1.f;
          if (tok_major) { bl = sBias[rg]; cs = sCol[rg]; }
          else { mu = sMu[rg]; rs = sRs[rg]; }
          unsigned char* srow = stage_row(r);
#pragma unroll
          for (int gi = 0; gi < 4; ++gi) {
            const int cl = (tok_major ? (wm * WM + i * 32) : (wn * WN + j * 32)) + gi * 8 + lh * 4;
            float v[4];
            if (tok_major) {
              const f32x4 m4 = *reinterpret_cast<const f32x4*>(sMu + cl), r4 = *reinterpret_cast<const f32x4*>(sRs + cl);
#pragma unroll
              for (int e = 0; e < 4; ++e) v[e] = __builtin_fmaf(r4[e], __builtin_fmaf(-m4[e], cs, acc[i][j][gi * 4 + e]), bl);
            } else {
              const f32x4 b4 = *reinterpret_cast<const f32x4*>(sBias + cl), c4 = *reinterpret_cast<const f32x4*>(sCol + cl);
#pragma unroll
              for (int e = 0; e < 4; ++e) v[e] = __builtin_fmaf(rs, __builtin_fmaf(-mu, c4[e], acc[i][j][gi * 4 + e]), b4[e]);
            }
            bf16x4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = (bf16_t)apply_act_fast<EPI>(v[e]);
            *reinterpret_cast<bf16x4*>(srow + (((cl >> 3) ^ (r & 15)) << 4) + ((cl & 4) << 1)) = o;
          }
        }
      __syncthreads();
      if (pass == 1 && has_next) tile_scalars(tid, rp, m0n, n0n);   // every read of this tile's scalars is behind us
      // read-out: all LDS reads first, then the stores.  Thread tid owns 16-byte chunk tid % 32 of
      // staging rows tid / 32 + 16 i.
      constexpr int PER_T = 128 * NCH / NTHREADS;   // 8
      u32x4 v[PER_T];
      const int c = tid % NCH;
#pragma unroll
      for (int i = 0; i < PER_T; ++i) {
        const int r = tid / NCH + (NTHREADS / NCH) * i;
        v[i] = *reinterpret_cast<const u32x4*>(stage_row(r) + ((c ^ (r & 15)) << 4));
      }
      if (tok_major) {
#pragma unroll
        for (int i = 0; i < PER_T; ++i) {
          const int r = tid / NCH + (NTHREADS / NCH) * i;
          const int rg = (r / G) * 2 * G + pass * G + r % G;
          const int f = n0 + rg, tok = m0 + c * 8;
          if (f < p.N && tok < p.M) {
            const int h = f / p.hd_pad, d = f % p.hd_pad;
            const int t = tok / p.n_tok, n = tok % p.n_tok;
            __builtin_nontemporal_store(v[i], reinterpret_cast<u32x4*>(p.VT + (((long)t * p.heads + h) * p.hd_pad + d) * p.n_tok + n));
          }
        }
      } else if (p.row_map) {   // paged output: rows go through the block map
#pragma unroll
        for (int i = 0; i < PER_T; ++i) {
          const int r = tid / NCH + (NTHREADS / NCH) * i;
          const int row = m0 + (r / G) * 2 * G + pass * G + r % G, col = n0 + c * 8;
          if (row < p.M && col < p.N) {
            const long orow = (long)p.row_map[row / p.block_tokens] * p.block_tokens + row % p.block_tokens;
            __builtin_nontemporal_store(v[i], reinterpret_cast<u32x4*>(p.C + orow * p.ldc + col));
          }
        }
      } else if (n0 + c * 8 < p.N) {
        // buffer stores: the whole byte offset is the lane offset (the only part the descriptor's range
        // check sees; a scalar offset is outside it), so a row past M is dropped by the hardware.  The
        // data registers are not written again before the next barrier.
        const unsigned voff = ((unsigned)(tid / NCH) * (unsigned)p.ldc + (unsigned)(n0 + c * 8)) * 2u;
#pragma unroll
        for (int i = 0; i < PER_T; ++i) {
          const int r0 = (NTHREADS / NCH) * i;                                  // staging row of lane row 0
          const int row0 = m0 + (r0 / G) * 2 * G + pass * G + r0 % G;           // uniform (G % 16 == 0)
          __builtin_amdgcn_raw_buffer_store_b128(v[i], rsrc_c, voff + (unsigned)row0 * (unsigned)p.ldc * 2u, 0, 2);   // streamed (nt): read by a later launch
        }
      }
    }
    }
    if (!has_next) break;
    __syncthreads();   // buffer 1 has been read out: the next tile's first hand-over may fill it
    pos = nxt; m0 = m0n; n0 = n0n;
  }
}

// behind the operand slabs: the tile's bias values, and for a folded pre-norm the column sums of its
// weights and the mean / rstd of its rows
template <int BN, int NT, int BM_ = BM>
constexpr size_t smem_bytes() { return smem_main_bytes<BN, NT, BM_>() + (2 * BN + 2 * BM_) * sizeof(float); }

thread_local long g_kernel_launches = 0;   // kernels launched by bf16_gemm on this host thread so far (a product may be cut into two launches)

template <int BN, int NT, int WN, int EPI, int PIPE, int BM_ = BM, int FOLD = 0>
hipError_t launch(const GemmParams& p, hipStream_t st) {
  const int gm = (p.M + BM_ - 1) / BM_, gn = p.Npad / BN;
  const int n_tiles = gm * gn;
  if (n_tiles == 0) return hipSuccess;
  // Band width.  The ~32 workgroups an XCD runs at once cover (32 / gw) tile rows x gw tile
  // columns and move through K together, so per wave of tiles the L2 pulls 32 / gw activation
  // panels and gw weight panels (256 x K each) over the fabric; the weight panels are not
  // pulled again by later waves while a band's whole weight panel fits the 4 MiB L2.
  const double panel = 256.0 * p.K * sizeof(bf16_t);
  int gw = 1;
  double best = 1e30;
  for (int c = 1; c <= gn && c <= 32; ++c) {
    const bool resident = c * (double)BN * p.K * sizeof(bf16_t) <= 2.5 * (1 << 20);
    const double cost = (32.0 / c) * panel + (resident ? 0.0 : c * panel * (BN / 256.0));
    if (cost < best * 0.999) { best = cost; gw = c; }
  }
  if (p.band > 0 && p.band <= gn) gw = p.band;
  k_gemm_bf16<BN, NT, WN, EPI, PIPE, BM_, FOLD><<<dim3(n_tiles), dim3(NT), smem_bytes<BN, NT, BM_>(), st>>>(p, gm, gw);
  ++g_kernel_launches;
  return hipGetLastError();
}

}  // namespace
// The calling thread's device when first asked, for good: every GPU this code runs on is of one kind.  A function-local
// constant, so that threads that ask at once wait for one answer.
int cu_count() {
  static const int n = [] {
    int dev = 0, v = 0;
    const bool ok = hipGetDevice(&dev) == hipSuccess &&
                    hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0;
    return ok ? v : 256;
  }();
  return n;
}
namespace {

// the ring kernel has neither the folded pre-norm nor the bf16 copy of the residual rows
bool ring_has(const GemmParams& p) { return !p.stats && !p.xb; }

// Tile columns that hold nothing but padding are not launched by the 64- and 128-wide forms: a width of 1152 is padded to
// 1280 and has nine columns of 128 (residual products of 5888 rows of the SigLIP shape, ten columns: 33 + 94 us, nine: 32
// + 90).  A second product begins behind the padded first one.
int whole_128(int n) { return (n + 127) / 128 * 128; }
GemmParams without_padded_columns(GemmParams p) {
  if (p.n2_pad > 0) p.n2_pad = whole_128(p.n2);
  else p.Npad = whole_128(p.N);
  return p;
}
hipError_t launch_ring(const GemmParams& p, int tile, hipStream_t st) {
  ++g_kernel_launches;
  return bf16_gemm_ring(without_padded_columns(p), tile, st);
}

// Times of a product by form, in microseconds, as the dispatch compares them: a workgroup's chain of KT 64-deep slabs plus its
// fixed cost (first slab, epilogue), times the rounds the launch's tiles make on the CUs, and a part that grows with the
// tiles alone (the CUs share memory and power).  Fitted to the products of the running encoder, each form forced for one
// product at a time (three shapes, 256 to 65536 rows, K 1024 to 12800, weights cold; rms 4-7 %), when the 256-wide tiles
// still ran on v_mfma_f32_32x32x16_bf16: those are 5 to 14 % faster now, the ring tiles 2 %.  They order the forms for the second
// stage below, whose choice tests hold against times of the present kernels.  Figures below that give one form only are of the earlier kernels.
struct RingPick { int tile; double us; };
bool f32_rows(int epi) { return epi == EPI_BIAS_RESIDUAL || epi == EPI_BIAS_POS; }   // reads and writes rows of the stream
bool has_gelu(int epi) { return epi == EPI_BIAS_GELU_ERF || epi == EPI_BIAS_GELU_TANH; }
// ring tiles half as wide again (ring_wider), one round of them; fitted to 11 products with cold operands, 960 to 2688 rows
double wider_us(int tile, double kt) {
  return tile == RING_64x64 ? 3.7 + 0.40 * kt : tile == RING_128x64 ? 8.3 + 0.455 * kt : 11.1 + 0.54 * kt;
}
// One round of 128 x 128 tiles takes 1 us less than the fit for values and pairs (epi EPI_VT), since fragments are read by k-step and pairs read their bias behind
// the loop, and 2.3 with an activation: pairs, 736 rows of 2304 and 1152 columns 16.6 us on 64 x 64 tiles, 14.6 on 128 x 128; values, 4096 rows, 1024 x 1024
// 18.1 on 128 x 64, 15.5; activation, 1024 rows, 4096 x 1024 16.9, 14.7.  Over more rounds 128 x 64 tiles stay ahead.  (The plain bias likewise would part the
// pair of two slices of the 1024-wide encoder: 2368 | 2399 us a call.)
RingPick best_ring(int M, int n_cols, int K, int epi) {
  const double cus = cu_count(), kt = K / BK;
  const bool f32 = f32_rows(epi);
  auto per_cu = [&](int tm, int tn) { return (double)((M + tm - 1) / tm) * ((n_cols + tn - 1) / tn) / cus; };
  auto wider = [&](int tile) { return ring_wider(epi, M, whole_128(n_cols), K, tile); };
  const double t0 = wider(RING_64x64) ? wider_us(RING_64x64, kt) : f32 ? 6.0 + 0.09 * kt + fmax(1.0, per_cu(64, 64)) * (0.4 + 0.217 * kt)
                        : 5.0 + 0.12 * kt + fmax(1.0, per_cu(64, 64)) * 0.198 * kt;
  RingPick best = {RING_64x64, t0};
  const double r1 = ceil(per_cu(128, 64));   // two workgroups share a CU: a tile alone on its CU takes 3/4 of two
  const double t1 = wider(RING_128x64) ? wider_us(RING_128x64, kt) : f32 ? 6.2 + (r1 == 1.0 ? 2.15 + 0.445 * kt : r1 * (1.2 + 0.33 * kt))
                        : 5.4 + (r1 == 1.0 ? 0.35 + 0.42 * kt : r1 * 0.318 * kt) + (has_gelu(epi) ? 0.8 : 0.0);
  if (t1 < best.us) best = {RING_128x64, t1};
  const double r2 = per_cu(128, 128);
  const double t2 = wider(RING_128x128) ? wider_us(RING_128x128, kt) : f32 ? 5.5 + ceil(r2) * (4.5 + 0.4 * kt) + r2 * 0.187 * kt
                        : 5.8 + ceil(r2) * (2.3 + 0.34 * kt) + r2 * 0.18 * kt + (r2 > 1.0 ? (has_gelu(epi) ? 1.7 : 0.0) : has_gelu(epi) ? -0.6 : epi == EPI_VT ? -1.0 : 0.0);
  if (t2 < best.us) best = {RING_128x128, t2};
  return best;
}
// one round of 256 x 256 tiles, `tiles` of them
double round_256(double tiles, int K, int epi) {
  const double kt = K / BK, fill = tiles / cu_count();
  if (f32_rows(epi)) return 18.0 + 1.36 * kt + fill * (1.0 + 0.29 * kt);
  return 9.0 + 1.45 * kt + fill * (0.02 * kt - 1.0) + (has_gelu(epi) ? 1.4 : 0.0);
}
// one round of 256 x 192 tiles (residual products only)
double round_192(double tiles, int K) {
  const double kt = K / BK;
  return 13.7 + 1.27 * kt + tiles / cu_count() * (0.234 * kt - 0.5);
}
// 256 x 128 tiles, one workgroup per CU: a launch that is one round of them (6400 columns over 1024 rows of K = 3200: 54 us,
// 66 on 128 x 128 ring tiles; 1152 columns over 6144 rows of K = 4352: 91 against 94); not launched for more
double one_round_128(const GemmParams& p) {
  const double kt = p.K / BK, tiles = (double)((p.M + BM - 1) / BM) * (whole_128(p.N) / 128), fill = tiles / cu_count();
  if (fill > 1.0) return INFINITY;
  if (f32_rows(p.epi)) return 16.6 + 0.765 * kt + fill * (5.5 + 0.253 * kt);
  return 7.5 + 0.79 * kt + fill * (0.3 + 0.247 * kt) + (has_gelu(p.epi) ? 1.8 : 0.0);
}
// `tiles` tiles in rounds of one per CU
template <typename F>
double rounds_of(long tiles, F round) {
  const long cus = cu_count(), full = tiles / cus, rem = tiles % cus;
  return full * round((double)cus) + (rem > 0 ? round((double)rem) : 0.0);
}
// The rows behind a cut, as a second launch.  Ring tiles always: 256 x 128 tiles there were measured beside them on 230
// products, up to 54 us slower and never more than 5 us (0.5 %) faster (3072 rows of 2304 columns, K = 1152, one whole round
// of them: equal; FC1 of a 13-slice call of the 1024-wide encoder: 128 against 120 us with its 3 whole rounds).
double behind_cut(const GemmParams& p, long rows_a) {
  return 4.0 + best_ring(p.M - (int)(rows_a * BM), p.N, p.K, p.epi).us;
}
// The tile rows of a launch of 256 x 256 tiles that go ahead as whole rounds when the rows of its last, partly filled
// round are cut off as a launch of ring tiles (every form sums an element's k-steps in the same order: same bits).
// 0: no cut, because the ring launch would take longer than the partly filled round.  The
// cut keeps a slice (transposed store) or a cache block (row map) on one side.
long cut_rows(const GemmParams& p) {
  const long cus = cu_count(), gn = p.Npad / 256, gm = (p.M + BM - 1) / BM, tiles = gm * gn, full = tiles / cus, rem = tiles % cus;
  if (full < 1 || rem == 0 || p.epi == EPI_BIAS_POS) return 0;
  // A cut pays only when at most half of the CUs are left with a tile (75264 rows of the 1024-wide encoder, 4.6 rounds:
  // +1.2 % on the call with the last 152 tiles cut), and past a few rounds, where the chip sits against its power limit
  // and an idle tail is paid back in clock, only for the long residual products (40 slices of the 6B shape with all
  // products cut: +1.4 %).
  if (full > 4 && !(p.epi == EPI_BIAS_RESIDUAL && p.K >= 2048)) return 0;
  long rows_a = full * cus / gn, unit = 1;
  if (p.epi == EPI_VT) { if (p.n_tok % BM != 0) return 0; unit = p.n_tok / BM; }
  rows_a -= rows_a % unit;
  if (rows_a < 1 || rows_a >= gm) return 0;
  if (p.row_map && (p.block_tokens < 1 || (rows_a * BM) % p.block_tokens != 0)) return 0;
  if ((gm - rows_a) * gn * 2 > cus) return 0;
  auto round = [&](double n) { return round_256(n, p.K, p.epi); };
  return rounds_of(rows_a * gn, round) + behind_cut(p, rows_a) < rounds_of(tiles, round) ? rows_a : 0;
}

// Residual products of this file's 256 x 256 tiles (emitted rows, EPD_PERSIST_RES=0): activation slabs straight into LDS
// (no register hop) when K is long (FC2 -1 %; the short out-projection is 1 % faster with its rows staged in registers
// two slabs ahead).  EPD_A_DIRECT=0 keeps the register-staged form for both.
bool a_direct() {
  static const bool on = !(getenv("EPD_A_DIRECT") && getenv("EPD_A_DIRECT")[0] == '0');
  return on;
}

template <int EPI>
hipError_t launch_persist(const GemmParams& p, hipStream_t st) {
  const int gm = (p.M + BM - 1) / BM, gn = p.Npad / 256;
  const int n_tiles = gm * gn;
  if (n_tiles == 0) return hipSuccess;
  const double panel = 256.0 * p.K * sizeof(bf16_t);
  // a search of its own: with band_columns, which counts the narrower last band, 104 slices of the 1024-wide encoder take 83.4 ms for 83.2
  int gw = 1;
  double best = 1e30;
  for (int c = 1; c <= gn && c <= 32; ++c) {
    const bool resident = c * 256.0 * p.K * sizeof(bf16_t) <= 2.5 * (1 << 20);
    const double cost = (32.0 / c) * panel + (resident ? 0.0 : c * panel);
    if (cost < best * 0.999) { best = cost; gw = c; }
  }
  if (p.band > 0 && p.band <= gn) gw = p.band;
  const int grid = n_tiles < cu_count() ? n_tiles : cu_count();
  k_gemm_bf16_persist<EPI><<<dim3(grid), dim3(512), smem_bytes<256, 512>(), st>>>(p, gm, gw, n_tiles);
  ++g_kernel_launches;
  return hipGetLastError();
}

bool persist_res() {   // EPD_PERSIST_RES=0: the residual products stay on the one-tile-per-workgroup kernels (ring tiles and this file's 256 x 256 ones)
  static const bool on = !(getenv("EPD_PERSIST_RES") && getenv("EPD_PERSIST_RES")[0] == '0');
  return on;
}

hipError_t launch_wide(const GemmParams& p, int tile, hipStream_t st) {
  ++g_kernel_launches;
  return bf16_gemm_wide(p, tile, cu_count(), st);
}

bool tiles_192() {   // EPD_TILES_192=0: widths like 1152 stay on the 256-wide tiles
  static const bool on = !(getenv("EPD_TILES_192") && getenv("EPD_TILES_192")[0] == '0');
  return on;
}

hipError_t dispatch_persist(const GemmParams& p, hipStream_t st) {   // all but the residual epilogue, on 256 x 256 tiles
  if (!p.stats) return launch_wide(p, WIDE_256, st);
  switch (p.epi) {
    case EPI_BIAS: return launch_persist<EPI_BIAS>(p, st);
    case EPI_BIAS_GELU_ERF: return launch_persist<EPI_BIAS_GELU_ERF>(p, st);
    case EPI_BIAS_GELU_TANH: return launch_persist<EPI_BIAS_GELU_TANH>(p, st);
    case EPI_VT: return launch_persist<EPI_VT>(p, st);
  }
  return hipErrorInvalidValue;
}

template <int EPI>
hipError_t set_attr_persist() {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(&k_gemm_bf16_persist<EPI>),
                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem_bytes<256, 512>());
}

template <int BN, int NT, int WN, int PIPE = 0, int BM_ = BM>
hipError_t dispatch(const GemmParams& p, hipStream_t st) {
  if (p.stats) {   // folded pre-norm (bf16-output epilogues)
    switch (p.epi) {
      case EPI_BIAS: return launch<BN, NT, WN, EPI_BIAS, PIPE, BM_, 2>(p, st);
      case EPI_BIAS_GELU_ERF: return launch<BN, NT, WN, EPI_BIAS_GELU_ERF, PIPE, BM_, 2>(p, st);
      case EPI_BIAS_GELU_TANH: return launch<BN, NT, WN, EPI_BIAS_GELU_TANH, PIPE, BM_, 2>(p, st);
      case EPI_VT: return launch<BN, NT, WN, EPI_VT, PIPE, BM_, 2>(p, st);
    }
    return hipErrorInvalidValue;
  }
  if (p.xb) {      // residual epilogue that also stores the rows as bf16, with or without their statistics
    if (p.epi != EPI_BIAS_RESIDUAL) return hipErrorInvalidValue;
    return p.stats_out ? launch<BN, NT, WN, EPI_BIAS_RESIDUAL, PIPE, BM_, 2>(p, st)
                       : launch<BN, NT, WN, EPI_BIAS_RESIDUAL, PIPE, BM_, 1>(p, st);
  }
  if constexpr (BN == 256) {
    switch (p.epi) {
      case EPI_BIAS: return launch<BN, NT, WN, EPI_BIAS, PIPE, BM_>(p, st);
      case EPI_BIAS_GELU_ERF: return launch<BN, NT, WN, EPI_BIAS_GELU_ERF, PIPE, BM_>(p, st);
      case EPI_BIAS_GELU_TANH: return launch<BN, NT, WN, EPI_BIAS_GELU_TANH, PIPE, BM_>(p, st);
      case EPI_BIAS_RESIDUAL: return launch<BN, NT, WN, EPI_BIAS_RESIDUAL, PIPE, BM_>(p, st);
      case EPI_VT: return launch<BN, NT, WN, EPI_VT, PIPE, BM_>(p, st);
      case EPI_BIAS_POS: return launch<BN, NT, WN, EPI_BIAS_POS, PIPE, BM_>(p, st);
    }
  }
  return hipErrorInvalidValue;   // 256 x 128 tiles: folded pre-norms and emitted rows only
}

// 128 x 128 tiles: compiled for the folded pre-norm and the emitting residual epilogues only (ring tiles otherwise)
template <int PIPE>
hipError_t dispatch_128_fold(const GemmParams& p, hipStream_t st) {
  if (p.stats) {
    switch (p.epi) {
      case EPI_BIAS: return launch<128, 512, 64, EPI_BIAS, PIPE, 128, 2>(p, st);
      case EPI_BIAS_GELU_ERF: return launch<128, 512, 64, EPI_BIAS_GELU_ERF, PIPE, 128, 2>(p, st);
      case EPI_BIAS_GELU_TANH: return launch<128, 512, 64, EPI_BIAS_GELU_TANH, PIPE, 128, 2>(p, st);
      case EPI_VT: return launch<128, 512, 64, EPI_VT, PIPE, 128, 2>(p, st);
    }
    return hipErrorInvalidValue;
  }
  if (p.epi != EPI_BIAS_RESIDUAL || !p.xb) return hipErrorInvalidValue;
  return p.stats_out ? launch<128, 512, 64, EPI_BIAS_RESIDUAL, PIPE, 128, 2>(p, st)
                     : launch<128, 512, 64, EPI_BIAS_RESIDUAL, PIPE, 128, 1>(p, st);
}

template <int BN, int NT, int WN, int EPI, int PIPE, int BM_, int FOLD = 0>
hipError_t set_attr() {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(&k_gemm_bf16<BN, NT, WN, EPI, PIPE, BM_, FOLD>),
                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem_bytes<BN, NT, BM_>());
}

template <int BN, int NT, int WN, int PIPE = 0, int BM_ = BM>
hipError_t set_attr_all() {
  hipError_t e;
  if constexpr (BN == 256) {
    if ((e = set_attr<BN, NT, WN, EPI_BIAS, PIPE, BM_>()) != hipSuccess) return e;
    if ((e = set_attr<BN, NT, WN, EPI_BIAS_GELU_ERF, PIPE, BM_>()) != hipSuccess) return e;
    if ((e = set_attr<BN, NT, WN, EPI_BIAS_GELU_TANH, PIPE, BM_>()) != hipSuccess) return e;
    if ((e = set_attr<BN, NT, WN, EPI_BIAS_RESIDUAL, PIPE, BM_>()) != hipSuccess) return e;
    if ((e = set_attr<BN, NT, WN, EPI_VT, PIPE, BM_>()) != hipSuccess) return e;
    if ((e = set_attr<BN, NT, WN, EPI_BIAS_POS, PIPE, BM_>()) != hipSuccess) return e;
  }
  if ((e = set_attr<BN, NT, WN, EPI_BIAS, PIPE, BM_, 2>()) != hipSuccess) return e;
  if ((e = set_attr<BN, NT, WN, EPI_BIAS_GELU_ERF, PIPE, BM_, 2>()) != hipSuccess) return e;
  if ((e = set_attr<BN, NT, WN, EPI_BIAS_GELU_TANH, PIPE, BM_, 2>()) != hipSuccess) return e;
  if ((e = set_attr<BN, NT, WN, EPI_BIAS_RESIDUAL, PIPE, BM_, 1>()) != hipSuccess) return e;
  if ((e = set_attr<BN, NT, WN, EPI_BIAS_RESIDUAL, PIPE, BM_, 2>()) != hipSuccess) return e;
  return set_attr<BN, NT, WN, EPI_VT, PIPE, BM_, 2>();
}

template <int PIPE>
hipError_t set_attr_128_fold() {
  hipError_t e;
  if ((e = set_attr<128, 512, 64, EPI_BIAS, PIPE, 128, 2>()) != hipSuccess) return e;
  if ((e = set_attr<128, 512, 64, EPI_BIAS_GELU_ERF, PIPE, 128, 2>()) != hipSuccess) return e;
  if ((e = set_attr<128, 512, 64, EPI_BIAS_GELU_TANH, PIPE, 128, 2>()) != hipSuccess) return e;
  if ((e = set_attr<128, 512, 64, EPI_BIAS_RESIDUAL, PIPE, 128, 1>()) != hipSuccess) return e;
  if ((e = set_attr<128, 512, 64, EPI_BIAS_RESIDUAL, PIPE, 128, 2>()) != hipSuccess) return e;
  return set_attr<128, 512, 64, EPI_VT, PIPE, 128, 2>();
}

}  // namespace

long bf16_gemm_kernel_launches() { return g_kernel_launches; }

hipError_t bf16_gemm_init() {
  hipError_t e = set_attr_all<256, 512, 64>();
  if (e != hipSuccess) return e;
  if ((e = set_attr_all<256, 512, 64, 1>()) != hipSuccess) return e;
  if ((e = set_attr_all<256, 512, 64, 3>()) != hipSuccess) return e;
  if ((e = set_attr_persist<EPI_BIAS>()) != hipSuccess) return e;
  if ((e = set_attr_persist<EPI_BIAS_GELU_ERF>()) != hipSuccess) return e;
  if ((e = set_attr_persist<EPI_BIAS_GELU_TANH>()) != hipSuccess) return e;
  if ((e = set_attr_persist<EPI_VT>()) != hipSuccess) return e;
  if ((e = bf16_gemm_wide_init()) != hipSuccess) return e;
  if ((e = set_attr_all<128, 512, 64>()) != hipSuccess) return e;
  if ((e = set_attr_128_fold<0>()) != hipSuccess) return e;
  if ((e = set_attr_128_fold<2>()) != hipSuccess) return e;
  if ((e = bf16_gemm_ring_init()) != hipSuccess) return e;
  return hipSuccess;
}

// Products without a folded pre-norm or emitted rows: the form with the smallest estimated time.  All forms leave the same
// bits: a tile shape changes which lane holds an element, never the order in which its k-steps are summed.
enum PlainForm { PLAIN_RING, PLAIN_256x128, PLAIN_256, PLAIN_192, PLAIN_COLUMNS };
struct Plain { PlainForm form; int tile; long rows_a; double us; };   // tile: of the ring launch (whole or behind the cut); rows_a: see cut_rows
static bool few_128_tiles(const GemmParams& p) {
  return p.Npad % 256 != 0 || (long)((p.M + 127) / 128) * ((whole_128(p.N) + (p.n2_pad > 0 ? whole_128(p.n2) : 0)) / 128) <= 8L * cu_count();
}
static Plain choose_plain(const GemmParams& p) {
  const bool residual = p.epi == EPI_BIAS_RESIDUAL;
  const long gm = (p.M + BM - 1) / BM, cus = cu_count();
  const RingPick ring = best_ring(p.M, p.N, p.K, p.epi);
  // Ring tiles are for launches of a few slices.  Past eight 128 x 128 tiles per CU they were never ahead, and there the
  // stream's rows make them 10 to 25 % slower than estimated (47104 rows of 1152 by K = 1152: 225 us, 177 on 256 x 256 tiles).
  const bool few = few_128_tiles(p);
  Plain best = {PLAIN_RING, ring.tile, 0, few ? ring.us : INFINITY};
  auto offer = [&](PlainForm form, int tile, long rows_a, double us) { if (us < best.us) best = {form, tile, rows_a, us}; };
  // 128 columns over many rows stream the activations at the memory's rate: 256 x 128 tiles fetch each row once (the cut
  // columns of the 6B shape's FC2, 40960 rows: 277 us, on 128 x 64 ring tiles 315)
  const bool persistent = !residual || persist_res();
  if (p.Npad == 128 && gm * 2 > cus && persistent) return {PLAIN_256x128, 0, 0, ring.us};
  if (persistent) offer(PLAIN_256x128, 0, 0, one_round_128(p));
  if (p.Npad % 256 != 0) return best;
  const long tiles = gm * (p.Npad / 256);
  // A width like 3200 leaves the last 256-wide tile column half used.  When that column is also what
  // spills the launch into a nearly empty last round (at most a quarter of the CUs busy), the residual
  // product is cut by columns: the whole 256-wide tile columns, and the last 128 columns as a launch of
  // their own (weight rows, bias and residual columns are pointer offsets): -4 % on the 6B shape's FC2,
  // +1 % on a SigLIP-shaped batch of 480 slices whose 2560 tiles are ten full rounds anyway.  Not for multiples of 192, which
  // 256 x 192 tiles take whole (1152 columns, 41216 rows, out-projection and FC2 together: 667 us by columns, 606 on those
  // tiles; 26624 rows, K = 4352: 314 us by columns, 287 cut by rows).
  if (residual && p.N > 256 && p.N % 192 != 0 && p.N % 256 != 0 && p.N % 256 <= 128 && tiles >= cus && tiles % cus != 0 && (tiles % cus) * 4 <= cus)
    return {PLAIN_COLUMNS, 0, 0, 0.0};
  const long rows_a = cut_rows(p);
  auto round = [&](double n) { return round_256(n, p.K, p.epi); };
  if (rows_a == 0) offer(PLAIN_256, 0, 0, rounds_of(tiles, round));
  else offer(PLAIN_256, best_ring(p.M - (int)(rows_a * BM), p.N, p.K, p.epi).tile, rows_a, rounds_of(rows_a * (p.Npad / 256), round) + behind_cut(p, rows_a));
  // A width of 1152 is four and a half 256-wide tile columns and six 192-wide ones: 240 tiles in one round instead of
  // 200 for the residual products of the 10-slice SigLIP-shaped request (-8 % on both), but 6 rounds for 5 in 64 slices
  // (FC2 642 us on 256 x 256 tiles, 677 on these).
  if (residual && persistent && tiles_192() && p.N % 192 == 0 && p.N % 256 != 0)
    offer(PLAIN_192, 0, 0, rounds_of(gm * (p.N / 192), [&](double n) { return round_192(n, p.K); }));
  return best;
}

// ---- second stage: the shape that runs ----
// choose_plain weighs the forms there were when its estimates were fitted; this stage takes another shape of the persistent kernel where it
// is faster on the present kernels.  us = c + ck kt + up (u + uk kt) + r (v + vk kt): kt 64-deep slabs, r tiles per CU, up its rounds
// (64 x 64 tiles, which share a CU: at least 1).  Fitted to products with cold operands and among their own kind, each in up to nine shapes
// (encoders of 1024, 1152 and 3200 columns, 736 to 106496 rows; rms 2 to 7 %, no coefficient below zero).  Against 410 products and pairs
// among other kernels (tests/golden/product_times.txt, which tests/product_times.py takes) what runs is behind the fastest form by, on
// average: pairs 0.5 %, bias 1.9, activation 0.3, residual 0.9, values 0.5; furthest 1024 rows of 5120 columns over K = 12800, 199 us on ring tiles,
// 151 on 256 x 128 ones.  Which ring tiles, only the first stage says: alone and in the running encoder they differ most.
static void cut_columns(const GemmParams& p, GemmParams& a, GemmParams& b) {   // whole 256-wide tile columns, and the rest
  const int n_a = p.N / 256 * 256;
  a = b = p;
  a.N = n_a; a.Npad = n_a;
  b.N = p.N - n_a; b.Npad = 128;
  b.W = p.W + (long)n_a * p.K; b.bias = p.bias + n_a; b.R = p.R + n_a;
}
enum Shape { S_64x64, S_128x64, S_128x128, S_256x128, S_256, S_224, S_192_ROWS, S_160_ROWS, S_192, N_SHAPES };
constexpr int SHAPE_ROWS[N_SHAPES] = {64, 128, 128, 256, 256, 224, 192, 160, 256};
constexpr int SHAPE_COLS[N_SHAPES] = {64, 64, 128, 128, 256, 256, 256, 256, 192};
enum Kind { K_PAIR, K_BIAS, K_GELU, K_RESIDUAL, K_VT, N_KINDS };
struct Fit { float c, ck, u, uk, v, vk; };   // all zero: not compiled for this kind
constexpr Fit RING_FIT_64 = {0, 0.202f, 0.211f, 0.093f, 0.211f, 0.093f}, RING_FIT_128x64 = {0, 0.163f, 0, 0.173f, 0.890f, 0.119f},
              RING_FIT_128 = {0, 0.101f, 0, 0.396f, 4.261f, 0.043f}, NO_FIT = {0, 0, 0, 0, 0, 0};
static const Fit FITS[N_KINDS][N_SHAPES] = {
    {RING_FIT_64, RING_FIT_128x64, RING_FIT_128, NO_FIT, {0, 0.226f, 4.699f, 0.788f, 0.840f, 0.571f}, {0, 0.100f, 4.297f, 0.871f, 0, 0.424f},
     {0, 0.078f, 3.675f, 0.845f, 0, 0.321f}, {0, 0.131f, 2.768f, 0.769f, 0.698f, 0.268f}, {0.013f, 0.002f, 1.862f, 0.969f, 0.551f, 0.277f}},
    {RING_FIT_64, RING_FIT_128x64, RING_FIT_128, {0, 0.099f, 1.078f, 0.716f, 0, 0.211f}, {0.985f, 0, 0.831f, 1.061f, 5.395f, 0.272f}},
    {{0, 0.149f, 0.568f, 0.087f, 0.568f, 0.087f}, {0, 0.132f, 0, 0.247f, 2.094f, 0.023f}, {0, 0.181f, 0.460f, 0.390f, 5.288f, 0.009f},
     {0, 0.168f, 0.076f, 0.874f, 2.415f, 0.038f}, {0, 0.162f, 6.232f, 0.835f, 0, 0.611f}, {0, 0.114f, 1.584f, 1.041f, 3.835f, 0.282f}},
    {{0, 0.143f, 0.965f, 0, 0.265f, 0.207f}, {0, 0.178f, 0.119f, 0.211f, 2.808f, 0.095f}, {0, 0.042f, 0, 0.486f, 8.305f, 0.037f},
     {3.683f, 0.003f, 0.601f, 0.813f, 8.356f, 0.141f}, {4.777f, 0, 1.948f, 1.191f, 19.052f, 0.139f}, {0.187f, 0.021f, 7.756f, 0.994f, 10.328f, 0.278f},
     NO_FIT, NO_FIT, {0, 0, 6.672f, 0.951f, 10.647f, 0.200f}},
    {RING_FIT_64, RING_FIT_128x64, RING_FIT_128, {0, 0, 2.208f, 0.825f, 0, 0.168f}, {0, 0, 3.195f, 1.110f, 4.354f, 0.227f}},
};
static Kind kind_of(const GemmParams& p) {
  return p.n2_pad > 0 ? K_PAIR : p.epi == EPI_BIAS_RESIDUAL ? K_RESIDUAL : p.epi == EPI_VT ? K_VT : has_gelu(p.epi) ? K_GELU : K_BIAS;
}
static int ring_tile(int shape) { return shape == S_64x64 ? RING_64x64 : shape == S_128x64 ? RING_128x64 : RING_128x128; }
static double shape_us(const GemmParams& p, int shape) {
  if (shape <= S_128x128 && p.n2_pad == 0 && ring_wider(p.epi, p.M, whole_128(p.N), p.K, ring_tile(shape))) return wider_us(ring_tile(shape), p.K / BK);
  const Fit& f = FITS[kind_of(p)][shape];
  const int tm = SHAPE_ROWS[shape], tn = SHAPE_COLS[shape];
  auto columns = [&](int n) { return ((tn <= 128 ? whole_128(n) : n) + tn - 1) / tn; };
  const double kt = p.K / BK, cols = p.n2_pad > 0 ? (double)p.Npad / tn + columns(p.n2) : columns(p.N);
  const double r = (double)((p.M + tm - 1) / tm) * cols / cu_count(), up = shape == S_64x64 ? fmax(1.0, r) : ceil(r);
  // Among other kernels a launch of the persistent one takes 4 us longer than among its own kind, where the fit was taken (3 slices of the
  // 1024-wide encoder: q/k/v on 160 x 256 tiles 25.5 for 21.7 us, FC1 on 224 x 256 29.5 for 25.6); one of ring tiles does not (29.7, 30.3).
  // Residual products over a short K (up to 1536) 7 us: with 4, the out-projection of nine and ten slices of that encoder left 128 x 64 ring tiles
  // for 224 x 256 ones, and the calls took 8609 for 8536 and 8818 for 8748 us.  us, ring | persistent: 10240 rows, 1024 x 1024 35.9 | 40.6;
  // 8192 30.2 | 34.5; 6144, 1152 x 1152 31.7 | 33.6; 4608, 1536 x 1536 36.8 | 40.7; over K = 4096 4 us are right: 6144 rows 65.4 | 59.6.
  const double start = shape < S_256x128 ? 0.0 : kind_of(p) == K_RESIDUAL && kt <= 24 ? 7.0 : 4.0;
  return start + f.c + f.ck * kt + up * (f.u + f.uk * kt) + r * (f.v + f.vk * kt);
}
static bool shape_runs(const GemmParams& p, int shape) {
  const Fit& f = FITS[kind_of(p)][shape];
  if (f.uk == 0 && f.vk == 0) return false;
  if (shape <= S_128x128) return few_128_tiles(p);
  if (kind_of(p) == K_RESIDUAL && !persist_res()) return false;
  if (shape == S_256x128) return true;
  const int tn = SHAPE_COLS[shape], n = p.n2_pad > 0 ? p.n2 : p.N, pad = p.n2_pad > 0 ? p.n2_pad : p.Npad;
  if (p.n2_pad > 0 && p.Npad % tn != 0) return false;
  if (shape == S_192 && (!tiles_192() || n % 192 != 0)) return false;
  return (n + tn - 1) / tn * tn <= pad;
}
static hipError_t launch_shape(const GemmParams& p, int shape, hipStream_t st) {
  static const int tile[N_SHAPES] = {RING_64x64, RING_128x64, RING_128x128, WIDE_128, WIDE_256, WIDE_224, WIDE_192_ROWS, WIDE_160_ROWS, WIDE_192};
  return shape <= S_128x128 ? launch_ring(p, tile[shape], st) : launch_wide(p, tile[shape], st);
}
static int ring_shape(int tile) { return tile == RING_64x64 ? S_64x64 : tile == RING_128x64 ? S_128x64 : S_128x128; }
struct Choice { Plain first; int shape; double us; };   // shape -1: the first stage's
static Choice choose(const GemmParams& p) {
  const Plain c = choose_plain(p);
  if (p.epi == EPI_BIAS_POS) return {c, -1, c.us};
  double us = INFINITY;
  switch (c.form) {
    case PLAIN_RING: us = shape_us(p, ring_shape(c.tile)); break;
    case PLAIN_256x128: us = shape_us(p, S_256x128); break;
    case PLAIN_192: us = shape_us(p, S_192); break;
    case PLAIN_256: {
      GemmParams a = p, b = p;
      if (c.rows_a > 0) { a.M = (int)(c.rows_a * BM); b.M = p.M - a.M; }
      us = shape_us(a, S_256) + (c.rows_a > 0 ? 2.5 + shape_us(b, ring_shape(c.tile)) : 0.0);
      break;
    }
    case PLAIN_COLUMNS: {
      GemmParams a, b;
      cut_columns(p, a, b);
      us = choose(a).us + choose(b).us + 2.5;
      break;
    }
  }
  Choice best = {c, -1, us * 0.97};   // of two forms closer than that the first stage's stays
  for (int shape = S_256x128; shape < N_SHAPES; ++shape)   // which ring tiles, the first stage says: its estimates are from the running encoder
    if (shape_runs(p, shape) && shape_us(p, shape) < best.us) best = {c, shape, shape_us(p, shape)};
  if (best.shape < 0) best.us = us;
  return best;
}

static hipError_t dispatch_plain(const GemmParams& p, hipStream_t st);
static hipError_t launch_first(const GemmParams& p, const Plain& c, hipStream_t st) {
  const bool residual = p.epi == EPI_BIAS_RESIDUAL;
  GemmParams a = p, b = p;
  auto wide = [&](const GemmParams& g) {
    if (!residual || persist_res()) return launch_wide(g, WIDE_256, st);
    return (a_direct() && g.K >= 2048) ? dispatch<256, 512, 64, 3>(g, st) : dispatch<256, 512, 64, 1>(g, st);
  };
  switch (c.form) {
    case PLAIN_RING: return launch_ring(p, c.tile, st);
    case PLAIN_256x128: return launch_wide(p, WIDE_128, st);
    case PLAIN_192: return launch_wide(p, WIDE_192, st);
    case PLAIN_256: {
      if (c.rows_a == 0) return wide(p);
      a.M = (int)(c.rows_a * BM);
      b.M = p.M - a.M;
      b.A = p.A + (long)a.M * p.lda;
      if (residual) b.R = p.R + (long)a.M * p.ldr;
      else if (p.epi == EPI_VT) b.VT = p.VT + (long)a.M * p.heads * p.hd_pad;   // whole slices: a.M / n_tok of [heads * hd_pad][n_tok]
      else if (p.row_map) b.row_map = p.row_map + a.M / p.block_tokens;
      else b.C = p.C + (long)a.M * p.ldc;
      const hipError_t e = wide(a);
      return e != hipSuccess ? e : launch_ring(b, c.tile, st);
    }
    case PLAIN_COLUMNS: {
      cut_columns(p, a, b);
      const hipError_t e = dispatch_plain(a, st);
      return e != hipSuccess ? e : dispatch_plain(b, st);
    }
  }
  return hipErrorInvalidValue;
}
static hipError_t dispatch_plain(const GemmParams& p, hipStream_t st) {
  const Choice c = choose(p);
  return c.shape >= 0 ? launch_shape(p, c.shape, st) : launch_first(p, c.first, st);
}
// the two cuts as forms of their own (tests, timing): by rows where cut_rows finds one, by columns where the last tile column is half empty
static hipError_t launch_cut_rows(const GemmParams& p, hipStream_t st) {
  const long rows_a = p.Npad % 256 == 0 ? cut_rows(p) : 0;
  if (rows_a == 0) return hipErrorInvalidValue;
  return launch_first(p, {PLAIN_256, best_ring(p.M - (int)(rows_a * BM), p.N, p.K, p.epi).tile, rows_a, 0.0}, st);
}
static hipError_t launch_cut_columns(const GemmParams& p, hipStream_t st) {
  if (p.epi != EPI_BIAS_RESIDUAL || p.N <= 256 || p.N % 256 == 0 || p.N % 256 > 128) return hipErrorInvalidValue;
  return launch_first(p, {PLAIN_COLUMNS, 0, 0, 0.0}, st);
}

// The q/k and the value projection as one launch, where that is estimated to take less than the two launches each in its own
// best shape and the 2.5 us a second launch costs.  us, cold, two launches | one: 1024-wide encoder, one slice 14.7 | 11.3 (ring
// tiles), three 29.4 | 21.7 (192 x 256 tiles), ten 81.8 | 55.7, 13 78.4 | 75.9 (224 x 256), 26 155 | 135, 104 551 | 549; 1152-wide, ten
// 85.9 | 72.2 (256 x 192); 3200-wide, 40 1954 | 1830.
static bool residual_or_gelu(int epi) { return epi == EPI_BIAS_RESIDUAL || has_gelu(epi); }
static bool pair_shape(const GemmParams& p) {
  return p.epi == EPI_BIAS && p.n2_pad > 0 && p.n2_pad % 128 == 0 && p.Npad % 128 == 0 && ring_has(p) && !p.row_map;
}
struct Pair { int shape; double us; };
static Pair choose_pair(const GemmParams& p) {
  Pair best = {-1, INFINITY};
  const int ring = ring_shape(best_ring(p.M, p.Npad + whole_128(p.n2), p.K, EPI_VT).tile);
  if (shape_runs(p, ring)) best = {ring, shape_us(p, ring)};
  for (int shape = S_256x128; shape < N_SHAPES; ++shape)
    if (shape_runs(p, shape) && shape_us(p, shape) < best.us) best = {shape, shape_us(p, shape)};
  return best;
}
bool bf16_gemm_pair_fits(const GemmParams& p) {
  if (p.cfg != 0 || !pair_shape(p)) return false;
  GemmParams q = p, v = p;
  q.n2_pad = v.n2_pad = 0; v.epi = EPI_VT; v.N = p.n2; v.Npad = p.n2_pad;
  return choose_pair(p).us < choose(q).us + choose(v).us + 2.5;
}

// For tests: what runs, by its number in GemmParams::cfg (5 and 18: the cuts by rows and by columns); of a pair 0: two products
int bf16_gemm_shape(const GemmParams& p) {
  static const int number[N_SHAPES] = {11, 13, 14, 1, 9, 15, 16, 17, 12};
  if (p.n2_pad > 0) return bf16_gemm_pair_fits(p) ? number[choose_pair(p).shape] : 0;
  const Choice c = choose(p);
  const bool residual = p.epi == EPI_BIAS_RESIDUAL;
  if (c.shape >= 0) return c.shape == S_256 && residual ? 10 : number[c.shape];
  switch (c.first.form) {
    case PLAIN_RING: return number[ring_shape(c.first.tile)];
    case PLAIN_256x128: return 1;
    case PLAIN_192: return 12;
    case PLAIN_256: return c.first.rows_a > 0 ? 5 : !residual ? 9 : persist_res() ? 10 : a_direct() && p.K >= 2048 ? 8 : 7;
    case PLAIN_COLUMNS: return 18;
  }
  return -1;
}

hipError_t bf16_gemm(const GemmParams& p, hipStream_t st) {
  if (p.K % (2 * BK) != 0 || p.Npad % 128 != 0 || p.N % 4 != 0) return hipErrorInvalidValue;
  if (p.stats && (p.n_part < 1 || p.n_part > STAT_REGS || p.stat_group < 1 || !p.colsum)) return hipErrorInvalidValue;
  // operands are addressed through 32-bit buffer offsets
  if ((long)p.M * p.lda * 2 >= (1L << 32) || (long)p.Npad * p.K * 2 >= (1L << 32) ||
      (p.R && (long)p.M * p.ldr * 4 >= (1L << 32)) || (p.C && !p.row_map && (long)p.M * p.ldc * 2 >= (1L << 32)))
    return hipErrorInvalidValue;
  const bool f32_out = p.epi == EPI_BIAS_RESIDUAL || p.epi == EPI_BIAS_POS;
  if (!f32_out && p.epi != EPI_VT && (p.N % 8 != 0 || p.ldc % 8 != 0)) return hipErrorInvalidValue;
  if (p.n2_pad > 0) {
    if (!pair_shape(p)) return hipErrorInvalidValue;
    switch (p.cfg) {
      case 0: { const Pair c = choose_pair(p); return c.shape < 0 ? hipErrorInvalidValue : launch_shape(p, c.shape, st); }
      case 11: return launch_ring(p, RING_64x64, st);
      case 13: return launch_ring(p, RING_128x64, st);
      case 14: return launch_ring(p, RING_128x128, st);
      case 9: return launch_wide(p, WIDE_256, st);
      case 12: return launch_wide(p, WIDE_192, st);
      case 15: return launch_wide(p, WIDE_224, st);
      case 16: return launch_wide(p, WIDE_192_ROWS, st);
      case 17: return launch_wide(p, WIDE_160_ROWS, st);
    }
    return hipErrorInvalidValue;
  }
  switch (p.cfg) {
    case 1: return ring_has(p) ? launch_wide(p, WIDE_128, st) : dispatch<128, 512, 64>(p, st);
    case 2: return ring_has(p) ? launch_ring(p, RING_128x128, st) : dispatch_128_fold<0>(p, st);
    case 3: if (!ring_has(p)) { if (p.K % 256 == 0) return dispatch_128_fold<2>(p, st); break; } return launch_ring(p, RING_128x128, st);
    case 5: return ring_has(p) ? launch_cut_rows(p, st) : hipErrorInvalidValue;
    case 6: if (p.Npad % 256 == 0) return dispatch<256, 512, 64, 0>(p, st); break;
    case 7: if (p.Npad % 256 == 0) return dispatch<256, 512, 64, 1>(p, st); break;
    case 8: if (p.Npad % 256 == 0) return dispatch<256, 512, 64, 3>(p, st); break;
    case 9: if (p.Npad % 256 == 0 && p.epi != EPI_BIAS_RESIDUAL) return dispatch_persist(p, st); break;
    case 10: if (p.Npad % 256 == 0 && p.epi == EPI_BIAS_RESIDUAL && !p.xb) return launch_wide(p, WIDE_256, st); break;
    case 11: if (ring_has(p)) return launch_ring(p, RING_64x64, st); break;
    case 13: if (ring_has(p)) return launch_ring(p, RING_128x64, st); break;
    case 14: if (ring_has(p)) return launch_ring(p, RING_128x128, st); break;
    case 15: if (p.Npad % 256 == 0 && ring_has(p) && (residual_or_gelu(p.epi))) return launch_wide(p, WIDE_224, st); break;
    case 12: if (p.N % 192 == 0 && p.epi == EPI_BIAS_RESIDUAL && !p.xb) return launch_wide(p, WIDE_192, st); break;
    case 18: return ring_has(p) ? launch_cut_columns(p, st) : hipErrorInvalidValue;
  }
  if (ring_has(p)) return dispatch_plain(p, st);
  // from here on: products with a folded pre-norm or an emitting residual epilogue (EPD_NORM_MODE)
  if (p.Npad % 256 != 0) return dispatch<128, 512, 64>(p, st);
  // A width like 3200 leaves the last 256-wide tile column half used.  When that column is also what
  // spills the launch into a nearly empty last round (at most a quarter of the CUs busy), the residual
  // product is cut by columns: the whole 256-wide tile columns, and the last 128 columns as a launch of
  // 128-wide tiles (weight rows, bias and residual columns are pointer offsets).  Same bits.  A 128-wide
  // tile takes about as long as a 256-wide one, so the cut pays only then: -4 % on the 6B shape's FC2,
  // +1 % on a SigLIP-shaped batch of 480 slices whose 2560 tiles are ten full rounds anyway.
  const long tiles_all = (long)((p.M + BM - 1) / BM) * (p.Npad / 256), cus = cu_count();
  if (p.cfg == 0 && p.epi == EPI_BIAS_RESIDUAL && p.N > 256 && p.N % 256 != 0 && p.N % 256 <= 128 &&
      tiles_all >= cus && tiles_all % cus != 0 && (tiles_all % cus) * 4 <= cus) {
    const int n_a = p.N / 256 * 256;
    GemmParams a = p, b = p;
    a.N = n_a; a.Npad = n_a;
    b.N = p.N - n_a; b.Npad = 128;
    b.W = p.W + (long)n_a * p.K; b.bias = p.bias + n_a; b.R = p.R + n_a;
    if (p.xb) { b.xb = p.xb + n_a; b.stats_out = p.stats_out + (n_a / STAT_GROUP) * 2; }   // n_a % 256 == 0
    const hipError_t e = bf16_gemm(a, st);
    return e != hipSuccess ? e : bf16_gemm(b, st);
  }
  // Small batches: when 256-wide tiles would leave half of the CUs without one, 128 x 128 tiles
  // quadruple the number of workgroups (two of them fit a CU) and shorten the one round there is; with at
  // most one such tile per CU with the loop that loads four slabs ahead (K in whole groups of four slabs).
  const long tiles256 = (long)((p.M + BM - 1) / BM) * (p.Npad / 256);
  if (tiles256 * 4 <= cu_count() && p.K % 256 == 0) return dispatch_128_fold<2>(p, st);
  if (tiles256 * 2 <= cu_count()) return dispatch_128_fold<0>(p, st);
  if (p.epi != EPI_BIAS_RESIDUAL) {
    // A batch of a few rounds whose last round fills at most half of the CUs is cut by rows like the long-K residual
    // products below: whole rounds on the persistent kernel, the remaining rows as one round of 256 x 128 tiles, whose
    // plain loop is slower per flop, so that the cut pays only while the last round is a large part of the launch.
    if (p.cfg == 0 && p.epi != EPI_VT && (!p.row_map || p.block_tokens > 0)) {
      const long cu = cu_count(), gn = p.Npad / 256, gm = (p.M + BM - 1) / BM;
      const long rounds = tiles256 / cu, rem = tiles256 % cu;
      const long rows_a = rounds * cu / gn;
      const long tiles_b = (gm - rows_a) * gn;
      if (rounds >= 1 && rounds <= 4 && rem > 0 && rows_a >= 1 && rows_a < gm && tiles_b * 2 <= cu &&
          (!p.row_map || (rows_a * BM) % p.block_tokens == 0)) {
        GemmParams a = p, b = p;
        a.M = (int)(rows_a * BM);
        b.M = p.M - a.M;
        b.A = p.A + (long)a.M * p.lda;
        b.stats = p.stats + (long)a.M * p.n_part * 2;
        if (p.row_map) b.row_map = p.row_map + a.M / p.block_tokens;
        else b.C = p.C + (long)a.M * p.ldc;
        const hipError_t e = dispatch_persist(a, st);
        return e != hipSuccess ? e : dispatch<128, 512, 64>(b, st);
      }
    }
    return dispatch_persist(p, st);
  }
  // A last round that fills at most half of the CUs costs a whole tile time.  The residual product
  // (rows are independent, all addressing is by pointer) is cut by rows instead: whole rounds of
  // 256-wide tiles, then the remaining rows as one round of 128-wide tiles, half as long.  Same bits.
  // Measured: -4 % on the K = 12800 product of the 6B shape, -1 % at K = 4096, +2 % at K = 1024 (the
  // second launch costs more than the short tiles save; +0.6 % with the persistent kernel), hence the K limit.
  if (p.K >= 2048) {
    const long cu = cu_count(), gn = p.Npad / 256, gm = (p.M + BM - 1) / BM;
    const long rounds = tiles256 / cu, rem = tiles256 % cu;
    const long rows_a = rounds * cu / gn;                    // tile rows of the whole rounds
    const long tiles_b = (gm - rows_a) * gn;
    if (rounds >= 1 && rem > 0 && rows_a >= 1 && rows_a < gm && tiles_b * 2 <= cu) {
      GemmParams a = p, b = p;
      a.M = (int)(rows_a * BM);
      b.M = p.M - a.M;
      b.A = p.A + (long)a.M * p.lda;
      b.R = p.R + (long)a.M * p.ldr;
      b.xb = p.xb + (long)a.M * p.ldxb; b.stats_out = p.stats_out + (long)a.M * p.n_part_out * 2;
      const hipError_t e = a_direct() ? dispatch<256, 512, 64, 3>(a, st) : dispatch<256, 512, 64, 1>(a, st);   // K >= 2048 here
      return e != hipSuccess ? e : dispatch<128, 512, 64>(b, st);
    }
  }
  return (a_direct() && p.K >= 2048) ? dispatch<256, 512, 64, 3>(p, st) : dispatch<256, 512, 64, 1>(p, st);
}

}  // namespace epd
