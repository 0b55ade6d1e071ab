// MXFP8 operands for the large products of an encoder layer on gfx950.
//
// Format (OCP Microscaling Formats specification v1.0, MXFP8 with E4M3 elements): along the contraction
// dimension K, 32 consecutive elements form a block that shares one power-of-two scale (one byte, value
// 2^(byte - 127)); an element is an OCP FP8 E4M3 number.  Conversion of a block: shared exponent =
// floor(log2(max |v|)) - 8, element = nearest E4M3 value of v / scale (ties to even), saturated to +-448.
//
// Layout in HBM: codes [rows][K] bytes, K contiguous; scales [K / 128][rows] 32-bit words, word (s, r) holding
// the four scale bytes of row r's blocks 4 s .. 4 s + 3 (byte b = block 4 s + b): one K slab of 128 elements
// of a 256-row tile reads 256 consecutive words.
//
// Product: C[M,N] = A[M,K] W[N,K]^T with v_mfma_scale_f32_16x16x128_f8f6f4, which takes the block scales as operands and
// applies them inside the instruction: lane l supplies row l % 16 of its 16 x 128 operand; its registers 0-3 hold k =
// 16 (l / 16) .. + 15 and its registers 4-7 k = 64 + 16 (l / 16) .. + 15, its scale register carries the scale byte of the
// row's block l / 16 (k = 32 (l / 16) .. + 31); result register e of lane l is D[4 (l / 16) + e][l % 16].  (The same bits as two
// v_mfma_scale_f32_32x32x64_f8f6f4 steps; a register-resident loop runs 4.6 PFLOP/s with it and 4.25 with those.)
//
// What bounds it: at the depths of an encoder layer (8 to 32 slabs) as much the epilogue and the fill of the chip as the
// products, hence persistent workgroups (the slabs past a tile's last are the next tile's), staging wave by wave without a
// workgroup barrier, and small tiles, two workgroups per CU, where large ones leave CUs idle or would all reach their fp32
// epilogue at once.  Slabs of 128 go from global memory straight into one of two LDS buffers (rows of 128 bytes, 16-byte chunks
// XOR-swizzled by (row >> 1) & 7), two slabs ahead; the fragments of a slab are read between its products and one barrier a
// slab frees the buffer.  us, one workgroup per tile on 32x32x64 -> this: 1024 rows, 2048 x 1024 16.3 -> 8.2, 4096 x 1024 with
// GELU 21.3 -> 10.4, 1024 x 4096 residual 46.7 -> 26.6; 26624 rows 74.7 -> 58.7, 151 -> 137, 128 -> 124, 1024 x 1024 residual
// 63.4 -> 54.7; 53248 rows 128 -> 105, 281 -> 255, 246 -> 244, 116 -> 103.
#include <cstring>
#include <type_traits>

#include "kernels.h"

namespace epd {

namespace {

typedef int i32x8 __attribute__((ext_vector_type(8)));
typedef unsigned char u8;

constexpr int BKB = 128;               // K elements (= bytes) per slab
constexpr int TN = 4;                  // a wave's blocks of 16 columns

// Waves stand WAVES_M x WAVES_N, each on TM x TN blocks of 16 x 16.
template <int TM, int WAVES_M, int WAVES_N>
struct MxTile {
  static constexpr int NT = 64 * WAVES_M * WAVES_N, WM = 16 * TM, WN = 16 * TN, BM = WM * WAVES_M, BN = WN * WAVES_N;
  static constexpr int AR = TM == 7 ? 256 : BM;                    // rows of A in a slab: 224-row tiles fetch 256, so that the buffers and the loads stay as they are
  static constexpr unsigned SLAB = (AR + BN) * BKB;                // bytes of a slab of both operands,
  static constexpr unsigned SCALES = (AR + BN) * sizeof(unsigned); // of its scale words: one per row of A and of W,
  static constexpr unsigned STAGE = 2048;                          // of a wave's staging space
  static constexpr size_t LDS = 2 * (size_t)SLAB + 2 * SCALES + NT / 64 * STAGE;
  static_assert(LDS <= 160 * 1024, "LDS of a CU");
  static_assert((SLAB & (SLAB - 1)) == 0 && (SCALES & (SCALES - 1)) == 0, "the buffers are told apart by one bit");
  static_assert(SCALES == NT * 4 && AR % 64 == 0, "a wave loads 64 scale words, of A or of W");
  static_assert(TM % 4 == 0 || TM == 7, "fragment slots");
  // The register slot of fragment i of A: no other than those of i + 1 and i + 2, and the last two's not those of 0 and 1, which are read for
  // the next slab while the last two are in use.
  static constexpr int slot(int i) { return TM % 4 == 0 ? i % 4 : i < TM - 1 ? i % 3 : 3; }
};

#define SWZ(row) (((row) >> 1) & 7)

// ---- conversion: mx_scale_byte / mx_inv_scale / mx_pack4 live in common.h (the attention kernel converts its output too) ----
template <typename C>
__device__ __forceinline__ float dpp_f(float x, C) {
  return __uint_as_float((unsigned)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(x), C::value, 0xf, 0xf, true));
}

__device__ __forceinline__ float max4abs(float a, float b, float c, float d) {
  return fmaxf(fmaxf(fabsf(a), fabsf(b)), fmaxf(fabsf(c), fabsf(d)));
}

// ---- rows -> MXFP8 (optionally behind a LayerNorm / RMSNorm) ----------------------------------------------
// One wave per row; lane l owns the 4-element chunks l + 64 i, so a block of 32 elements is 8 neighbouring
// lanes and a slab of 128 elements the 32 lanes of a half-wave.  The row stays in registers (NV chunks per
// lane; NV = 0: read again for every pass).
// PRE (a norm, kind 0 or 1): gain and shift are fetched in front of the sums.  It pays while they fit beside the row, with
// NV the row's own count of chunks (65536 rows of 768 | 1024 | 1152 in us: 45.3 -> 44.4 | 55.9 -> 53.6 | 65.2 -> 64.2,
// 1152 with NV = 8 77.7); at six chunks and more it loses (1536 | 2048: 94.3 -> 96.2 | 128.7 -> 137.5).
// NEAR: rows of the stream that are in the Infinity Cache, codes that go THROUGH (NEAR_ROWS_MX).
template <bool IN_BF16, int NV, bool PRE, bool NEAR>
__global__ __launch_bounds__(256) void k_mx_rows(const MxRowParams p) {
  const long R = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (R >= p.rows) return;
  const int lane = threadIdx.x & 63;
  const int nchunk = p.dim >> 2;
  auto load = [&](int c) -> float4 {
    if (IN_BF16) {
      const bf16x4 t = *(reinterpret_cast<const bf16x4*>(reinterpret_cast<const bf16_t*>(p.in) + R * p.ld_in) + c);
      return make_float4((float)t[0], (float)t[1], (float)t[2], (float)t[3]);
    }
    const f32x4* at = reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(p.in) + R * p.ld_in) + c;
    const f32x4 t = NEAR ? *at : __builtin_nontemporal_load(at);
    return make_float4(t[0], t[1], t[2], t[3]);
  };
  constexpr int NVR = NV > 0 ? NV : 1;
  float4 v[NVR];
  if (NV > 0) {
#pragma unroll
    for (int i = 0; i < NV; ++i) v[i] = lane + 64 * i < nchunk ? load(lane + 64 * i) : make_float4(0.f, 0.f, 0.f, 0.f);
  }
  // gain and shift in front of the sums: behind them their latency would stand between the statistics and the store
  float4 gpre[PRE ? NV : 1], bpre[PRE ? NV : 1];
  if constexpr (PRE) {
#pragma unroll
    for (int i = 0; i < NV; ++i)
      if (lane + 64 * i < nchunk) {
        gpre[i] = *(reinterpret_cast<const float4*>(p.gamma) + lane + 64 * i);
        if (p.kind == 0) bpre[i] = *(reinterpret_cast<const float4*>(p.beta) + lane + 64 * i);
      }
  }
  float mean = 0.f, rstd = 1.f;
  if (p.kind != 2) {
    float s = 0.f;
    if (p.kind == 0) {
      if (NV > 0) {
#pragma unroll
        for (int i = 0; i < NV; ++i) s += v[i].x + v[i].y + v[i].z + v[i].w;
      } else {
        for (int c = lane; c < nchunk; c += 64) { const float4 a = load(c); s += a.x + a.y + a.z + a.w; }
      }
      mean = wave_sum(s) / p.dim;
    }
    float qs = 0.f;
    auto sq = [&](float4 t) {
      const float a = t.x - mean, b = t.y - mean, cc = t.z - mean, d = t.w - mean;
      qs += a * a + b * b + cc * cc + d * d;
    };
    if (NV > 0) {
#pragma unroll
      for (int i = 0; i < NV; ++i)
        if (lane + 64 * i < nchunk) sq(v[i]);
    } else {
      for (int c = lane; c < nchunk; c += 64) sq(load(c));
    }
    rstd = 1.0f / sqrtf(wave_sum(qs) / p.dim + p.eps);
  }
  unsigned* codes = reinterpret_cast<unsigned*>(p.codes + R * p.ld_codes);
  // every lane of the wave takes part (the exchanges below are wave-wide); lanes past the row carry zeros
  auto emit = [&](int c, float4 a, bool in_row, const float4* gk, const float4* bk) {
#pragma clang fp contract(off)   // the same bits for every NV
    float r[4] = {a.x, a.y, a.z, a.w};
    if (p.kind != 2 && in_row) {
      const float4 gm = *gk;
      r[0] = (r[0] - mean) * rstd * gm.x;
      r[1] = (r[1] - mean) * rstd * gm.y;
      r[2] = (r[2] - mean) * rstd * gm.z;
      r[3] = (r[3] - mean) * rstd * gm.w;
      if (p.kind == 0) {
        const float4 bt = *bk;
        r[0] += bt.x; r[1] += bt.y; r[2] += bt.z; r[3] += bt.w;
      }
    }
    // largest magnitude of the block's eight lanes: three exchanges inside a row of 16 lanes (no LDS traffic)
    float amax = max4abs(r[0], r[1], r[2], r[3]);
    amax = fmaxf(amax, dpp_f(amax, std::integral_constant<int, 0xB1>{}));    // quad_perm [1, 0, 3, 2]
    amax = fmaxf(amax, dpp_f(amax, std::integral_constant<int, 0x4E>{}));    // quad_perm [2, 3, 0, 1]
    amax = fmaxf(amax, dpp_f(amax, std::integral_constant<int, 0x141>{}));   // row_half_mirror: the other quad of the eight
    const unsigned byte = mx_scale_byte(amax);
    const float inv = mx_inv_scale(byte);
    const unsigned word = mx_pack4(r[0] * inv, r[1] * inv, r[2] * inv, r[3] * inv);
    if (in_row) {
      if constexpr (NEAR)   // a relaxed store at the device's scope is one that goes THROUGH
        __hip_atomic_store(codes + c, word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      else
        codes[c] = word;
      // block c / 8 of the row = byte (c / 8) % 4 of scale word (c / 32, R): the block's first lane stores it
      if ((lane & 7) == 0) reinterpret_cast<unsigned char*>(p.scales + (long)(c >> 5) * p.ld_scales + R)[(c >> 3) & 3] = (unsigned char)byte;
    }
  };
  if (NV > 0) {
#pragma unroll
    for (int i = 0; i < NV; ++i)
      if (64 * i < nchunk) {
        if constexpr (PRE) emit(lane + 64 * i, v[i], lane + 64 * i < nchunk, &gpre[i], &bpre[i]);
        else emit(lane + 64 * i, v[i], lane + 64 * i < nchunk, reinterpret_cast<const float4*>(p.gamma) + lane + 64 * i,
                  reinterpret_cast<const float4*>(p.beta) + lane + 64 * i);
      }
  } else {
    for (int c0 = 0; c0 < nchunk; c0 += 64) {
      const bool in_row = c0 + lane < nchunk;
      emit(c0 + lane, in_row ? load(c0 + lane) : make_float4(0.f, 0.f, 0.f, 0.f), in_row,
           reinterpret_cast<const float4*>(p.gamma) + c0 + lane, reinterpret_cast<const float4*>(p.beta) + c0 + lane);
    }
  }
}

// ---- product ------------------------------------------------------------------------------------------------
template <int N, int I = 0, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<N, I + 1>(f);
  }
}

// DUAL (EPI_BIAS): the tile columns behind the first product's gq are a second product over the same rows, the value projection
// (MxGemmParams::n2).  Its tiles read their fragments with the operands' LDS regions exchanged: so the products, which stay as they
// are, leave four tokens of a feature in a lane, and the bits are EPI_VT's.  (A second main loop with the roles exchanged in
// the products instead spills 64 registers.)
// NEAR: the output goes THROUGH, stream rows are read without a hint (NEAR_OUT, NEAR_ROWS_MX); compiled apart as in gemm_bf16_wide.h.
template <int EPI, bool DUAL, int TM, int WAVES_M, int WAVES_N, bool NEAR>
__global__ __launch_bounds__(64 * WAVES_M * WAVES_N, 512 / (64 * WAVES_M * WAVES_N)) void k_gemm_mxfp8(const MxGemmParams p, const int gm, const int gw, const int gn, const int gq, const int n_tiles) {
  using T = MxTile<TM, WAVES_M, WAVES_N>;
  constexpr int NT = T::NT, WM = T::WM, WN = T::WN, BM = T::BM, BN = T::BN, AR = T::AR;
  constexpr unsigned SLAB = T::SLAB, SCALES = T::SCALES, STAGE = T::STAGE;
  constexpr bool TOK = EPI == EPI_VT;
  static_assert(!DUAL || (EPI == EPI_BIAS && BM == BN), "the second product rides on the plain bias epilogue, on square tiles");
  constexpr bool MX_OUT = EPI == EPI_BIAS_GELU_ERF || EPI == EPI_BIAS_GELU_TANH;
  constexpr bool F32_OUT = EPI == EPI_BIAS_RESIDUAL;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];   // slab buffers 0, 1 | scale words 0, 1 | staging by wave

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WAVES_N, wn = wave % WAVES_N;
  const int l16 = lane & 15, lg = lane >> 4;
  const int KT = p.K / BKB;

  // position in the launch order -> tile: XCD x (workgroups are dealt round-robin; a workgroup keeps pos % 8) takes a
  // contiguous run of the tile sequence, which walks bands of gw tile columns top to bottom
  auto tile_of = [&](int pos, int& m0, int& n0) {
    const int x = pos & 7, slot = pos >> 3;
    const int q = n_tiles >> 3, r = n_tiles & 7;
    const int id = x * q + (x < r ? x : r) + slot;
    const int band_tiles = gm * gw;
    const int full_bands = gn / gw;
    int band = id / band_tiles, in_band = id % band_tiles, bw = gw;
    if (band >= full_bands) { band = full_bands; in_band = id - full_bands * band_tiles; bw = gn - full_bands * gw; }
    m0 = (in_band / bw) * BM;
    n0 = (band * gw + in_band % bw) * BN;   // of the second product: from gq * BN on
  };

  // Direct loads: a wave fills 8 slab rows of 128 bytes linearly; the lane that lands on physical chunk ld_c of its row
  // fetches logical chunk ld_c ^ SWZ(row).  The first AR / 64 waves fetch the scale words of A rows, the
  // others those of W rows.
  const int ld_row = tid >> 3, ld_c = tid & 7;
  const unsigned a_voff = (unsigned)ld_row * (unsigned)p.lda + (unsigned)((ld_c ^ SWZ(ld_row)) * 16);
  const unsigned b_voff = (unsigned)ld_row * (unsigned)p.K + (unsigned)((ld_c ^ SWZ(ld_row)) * 16);
  const unsigned s_voff = (unsigned)lane * 4u;
  const long a_step = (long)(NT / 8) * p.lda, b_step = (long)(NT / 8) * p.K;
  constexpr int SA_WAVES = AR / 64;
  long s_step = (wave < SA_WAVES ? p.sa_ld : (long)p.Npad) * 4;
  constexpr int LA = AR * 8 / NT, LPS = LA + BN * 8 / NT + 1;
  const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) void*)smem;
  // the slab to fetch next: its position, its index in the tile, its first rows
  int lpos = blockIdx.x, lk = 0;
  unsigned lbuf = 0;
  const u8 *ga, *gb, *gs;
  const int last_rows = ((p.M + 255) & ~255) - AR;   // AR != BM: a tile past them fetches the rows from there on
  auto aim = [&]() {
    int m, n;
    tile_of(lpos, m, n);
    const bool v = DUAL && n >= gq * BN;
    if (v) n -= gq * BN;
    if (AR != BM) m = min(m, last_rows);
    ga = p.A + (long)m * p.lda;
    gb = (v ? p.W2 : p.W) + (long)n * p.K;
    gs = reinterpret_cast<const u8*>(wave < SA_WAVES ? p.SA + m + 64 * wave : (v ? p.SW2 : p.SW) + n + 64 * (wave - SA_WAVES));
    if (DUAL && wave >= SA_WAVES) s_step = (v ? (long)p.n2_pad : (long)p.Npad) * 4;
  };
  auto issue = [&](int i) {
    if (i < LPS - 1) {
      const u8* g = i < LA ? ga + i * a_step : gb + (i - LA) * b_step;
      asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
                   :: "v"(i < LA ? a_voff : b_voff), "s"(g), "s"(lds0 + lbuf * SLAB + wave * 1024 + i * (NT * 16)) : "memory", "m0");
    } else {
      asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1"
                   :: "v"(s_voff), "s"(gs), "s"(lds0 + 2 * SLAB + lbuf * SCALES + wave * 256) : "memory", "m0");
    }
  };
  auto advance = [&]() {
    lbuf ^= 1;
    ga += BKB; gb += BKB; gs += s_step;
    if (++lk == KT) {
      lk = 0;
      lpos += (int)gridDim.x;
      if (lpos < n_tiles) aim();
    }
  };
  auto wait_all = [&](bool but_one) {   // LDS reads and all vector-memory accesses, or all but the newest
    if (but_one) __builtin_amdgcn_s_waitcnt(1 | (0x7 << 4));
    else __builtin_amdgcn_s_waitcnt(0x7 << 4);
  };
  // The lines of the slab behind the newest one under way are asked for a slab ahead, each by one workgroup of the XCD (see
  // gemm_bf16_wide.h), with a dword a lane into the wave's staging area, which nobody uses until the epilogue.
  const bool a_half = wave < NT / 128;
  unsigned t_voff;
  {
    const int slot = blockIdx.x >> 3, lt = tid & (NT / 2 - 1), parts = a_half ? gw : max(1, (int)((gridDim.x + 7) >> 3) / gw), rows = a_half ? AR : BN;
    const int n = (rows + parts - 1) / parts, row = min((a_half ? slot % gw : slot / gw % parts) * n + lt * n / (NT / 2), rows - 1);
    t_voff = (unsigned)row * (unsigned)(a_half ? p.lda : (long)p.K);
  }
  bool touched = false;   // the newest access is such a load
  auto touch = [&]() {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1"
                 :: "v"(t_voff), "s"(a_half ? ga : gb), "s"(lds0 + 2 * SLAB + 2 * SCALES + wave * STAGE) : "memory", "m0");
    touched = true;
  };

  // Fragments: 16-byte chunks lg and 4 + lg of a row (k = 16 lg .. + 15 and 64 + 16 lg .. + 15), byte lg of its scale word.
  // Addresses of fragment 0 in the buffer of the slab at hand; the buffers lie a power of two apart.
  unsigned a_lo = (unsigned)((wm * WM + l16) * BKB + ((lg ^ SWZ(l16)) * 16)), a_hi = a_lo ^ 64u;
  unsigned b_lo = (unsigned)(AR * BKB + (wn * WN + l16) * BKB + ((lg ^ SWZ(l16)) * 16)), b_hi = b_lo ^ 64u;
  unsigned sc_a = (unsigned)(2 * SLAB + (wm * WM + l16) * 4 + lg), sc_b = (unsigned)(2 * SLAB + (AR + wn * WN + l16) * 4 + lg);
  auto other_buffer = [&]() { a_lo ^= SLAB; a_hi ^= SLAB; b_lo ^= SLAB; b_hi ^= SLAB; sc_a ^= SCALES; sc_b ^= SCALES; };
  auto frag = [&](unsigned lo, unsigned hi, int r) {
    const u32x4 x = *reinterpret_cast<const u32x4*>(smem + lo + r * (16 * BKB)), y = *reinterpret_cast<const u32x4*>(smem + hi + r * (16 * BKB));
    return __builtin_bit_cast(i32x8, __builtin_shufflevector(x, y, 0, 1, 2, 3, 4, 5, 6, 7));
  };
  f32x4 acc[TM][TN];
  i32x8 fa[4], fb[TN];   // fragment i of A in slot(i)
  int sa[4], sb[TN];
  auto read_a = [&](int i) { fa[T::slot(i)] = frag(a_lo, a_hi, i); sa[T::slot(i)] = smem[sc_a + i * 64]; };
  auto read_b = [&](int j) { fb[j] = frag(b_lo, b_hi, j); sb[j] = smem[sc_b + j * 64]; };
  // In place, as assembly: the compiler's form moves accumulators from register to register, and spills.  It does not see
  // the wait states such an instruction needs.  Behind it: nothing but products touches an accumulator between the zeros in
  // front of a tile and the nops behind it.  In front of it: an operand that a vector instruction wrote is read two wait
  // states later at the earliest.  The codes come from LDS as they are, but the compiler widens a scale byte wherever it
  // likes, also next to the product: hence the s_nop of every product.  It costs nothing (a product holds the matrix core
  // for eight wait states; 40 products with it in front of all and of two products a slab: equal to within two runs of one).
  auto mma = [&](auto i, auto j) {
    constexpr int I = decltype(i)::value, J = decltype(j)::value, S = T::slot(I);
    if constexpr (TOK)
      asm volatile("s_nop 1\n\tv_mfma_scale_f32_16x16x128_f8f6f4 %0, %1, %2, %0, %3, %4 op_sel_hi:[0,0,0]" : "+v"(acc[I][J]) : "v"(fa[S]), "v"(fb[J]), "v"(sa[S]), "v"(sb[J]));
    else
      asm volatile("s_nop 1\n\tv_mfma_scale_f32_16x16x128_f8f6f4 %0, %1, %2, %0, %3, %4 op_sel_hi:[0,0,0]" : "+v"(acc[I][J]) : "v"(fb[J]), "v"(fa[S]), "v"(sb[J]), "v"(sa[S]));
    __builtin_amdgcn_sched_barrier(0);
  };

  // fp32 epilogue: pass q adds rows 16 (q / 2) .. + 15, columns 32 (q % 2) .. + 31 of the wave's tile; the rows of four passes
  // are on their way
  constexpr int XAHEAD = 4, PASSES = 2 * TM;
  __amdgpu_buffer_rsrc_t rsrc_x = __builtin_amdgcn_make_buffer_rsrc(
      p.R, 0, F32_OUT ? (int)(unsigned)(((long)(p.M - 1) * p.ldr + p.N) * 4) : 0, 0x00020000);
  // the outputs that go THROUGH (each under 4 GiB: see NEAR_OUT)
  __amdgpu_buffer_rsrc_t rsrc_v = __builtin_amdgcn_make_buffer_rsrc(
      p.VT, 0, NEAR && (TOK || DUAL) ? (int)(unsigned)((long)p.M * p.heads * p.hd_pad * 2) : 0, 0x00020000);
  __amdgpu_buffer_rsrc_t rsrc_c = __builtin_amdgcn_make_buffer_rsrc(
      p.C, 0, NEAR && !MX_OUT && !F32_OUT && !TOK ? (int)(unsigned)(((long)(p.M - 1) * p.ldc + p.N) * 2) : 0, 0x00020000);
  __amdgpu_buffer_rsrc_t rsrc_q = __builtin_amdgcn_make_buffer_rsrc(
      p.Cq, 0, NEAR && MX_OUT ? (int)(unsigned)((long)(p.M - 1) * p.ldcq + p.ncq) : 0, 0x00020000);

  aim();
#pragma unroll
  for (int i = 0; i < LPS; ++i) issue(i);
  advance();
  if (lpos < n_tiles) {
#pragma unroll
    for (int i = 0; i < LPS; ++i) issue(i);
    advance();
  }
  wait_all(false);
  __syncthreads();

  bool v_tile = false;   // uniform
  int shift = 0;         // of the tile's rows against those fetched
  for (int pos = blockIdx.x;;) {
    int m0, n0;
    tile_of(pos, m0, n0);
    if constexpr (DUAL) {
      const bool v = n0 >= gq * BN;
      if (v != v_tile) {   // the regions are powers of two apart
        a_lo ^= BM * BKB; a_hi ^= BM * BKB; b_lo ^= BM * BKB; b_hi ^= BM * BKB;
        sc_a ^= BM * 4; sc_b ^= BM * 4;
        v_tile = v;
      }
      if (v) n0 -= gq * BN;
    }
    if constexpr (AR != BM) {   // rows the buffer does not hold are none of the operand's: what stands behind it is multiplied and not stored
      const int sh = max(0, m0 - last_rows), d = sh - shift;   // multiples of 32: a row's swizzle stays
      a_lo += d * BKB; a_hi += d * BKB; sc_a += d * 4;
      shift = sh;
    }
#pragma unroll
    for (int j = 0; j < TN; ++j) read_b(j);
    read_a(0);
    read_a(1);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        asm volatile("" : "+v"(acc[i][j]));   // the zeros are in their registers here, not in front of their first use
      }
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 7" ::: "memory");     // wait states between them and the first product
    __builtin_amdgcn_sched_barrier(0);

    f32x4 xr[F32_OUT ? XAHEAD : 1][2];
    auto xload = [&](int lane, int q) {
      if constexpr (F32_OUT) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const int r = (lane + 64 * u) / 8, c = lane % 8;
          const int row = m0 + wm * WM + (q / 2) * 16 + r, col = n0 + wn * WN + (q % 2) * 32 + c * 4;
          xr[q % XAHEAD][u] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(   // rows past M come back as zero
              rsrc_x, ((unsigned)row * (unsigned)p.ldr + (unsigned)col) * 4u, 0, NEAR ? 0 : STREAM));
        }
      }
    };
    // One slab.  Rows 0 .. 5 of blocks with the fragments of row i + 2 read meanwhile; then everyone holds what it needs of the
    // slab: behind the barrier the slab after the next is fetched into its buffer, and rows 6 and 7 run column by column,
    // each column's fragment of the next slab read into the registers the column has left.
    auto slab = [&](auto last) {
      constexpr bool LAST = decltype(last)::value;
      static_for<TM - 2>([&](auto i) {
        static_for<TN>([&](auto jj) {
          constexpr int J = i % 2 ? TN - 1 - jj : jj;
          mma(i, std::integral_constant<int, J>{});
          if constexpr (jj == 0 && i < TM - 3) read_a(i + 2);
          if constexpr (jj == 2 && i == TM - 4) read_a(TM - 1);
          __builtin_amdgcn_sched_barrier(0);
        });
      });
      wait_all(touched);   // the wave's part of the next slab has landed, its fragments of this one are in registers
      __syncthreads();   // everyone's has, and everyone holds this slab's fragments: its buffer is free
      other_buffer();
      if constexpr (LAST) {
#pragma unroll
        for (int q = 0; q < 2; ++q) xload(lane, q);
      } else {
        read_a(0);
        read_a(1);
      }
      __builtin_amdgcn_sched_barrier(0);
      const bool more = lpos < n_tiles;
      static_for<TN>([&](auto j) {
        constexpr int FIRST = j % 2 ? TM - 1 : TM - 2;
        mma(std::integral_constant<int, FIRST>{}, j);
        if (more) { issue(2 * j); issue(2 * j + 1); }
        mma(std::integral_constant<int, 2 * TM - 3 - FIRST>{}, j);
        if constexpr (!LAST) read_b(j);
        __builtin_amdgcn_sched_barrier(0);
      });
      touched = false;
      if (more) {
        issue(LPS - 1);
        advance();
        if (!LAST && lpos < n_tiles) touch();
      }
    };
#pragma clang loop unroll(disable)
    for (int kt = 0; kt < KT - 1; ++kt) slab(std::false_type{});
    slab(std::true_type{});
    __builtin_amdgcn_s_waitcnt((LPS & 0xf) | ((LPS >> 4) << 14) | (0x7 << 4) | (0xf << 8));   // the last touch has left the staging area
    asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7" ::: "memory");
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) asm volatile("" : "+v"(acc[i][j]));
    __builtin_amdgcn_sched_barrier(0);

    {
      // The epilogue's addresses derive from an opaque copy of the thread index, made anew for every tile: computed in
      // front of the tile loop they would occupy registers through the main loop.
      int tid_opaque = threadIdx.x;
      asm volatile("" : "+v"(tid_opaque));
      const int lane = tid_opaque & 63, l16 = lane & 15, lg = lane >> 4;
      u8* stg = smem + 2 * SLAB + 2 * SCALES + wave * STAGE;
      auto wave_sync = [&]() {   // LDS written by one lane, read by another of the same wave
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
      };
      auto at = [&](int r, int c) { return stg + r * 128 + ((c ^ SWZ(r)) << 4); };   // 16 rows of eight 16-byte chunks
      if (DUAL && v_tile) {   // rows of blocks are features, columns of blocks tokens
        float c1[TM], b1[TM];
#pragma unroll
        for (int i = 0; i < TM; ++i) {
          const int col = n0 + wm * WM + i * 16 + l16;
          b1[i] = p.bias2[col];
          c1[i] = p.cscale2 ? p.cscale2[col] : 1.0f;
        }
#pragma unroll
        for (int i = 0; i < TM; ++i) {
#pragma unroll
          for (int j = 0; j < TN; ++j) {
            bf16x4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = (bf16_t)__builtin_fmaf(acc[i][j][e], c1[i], b1[i]);
            *reinterpret_cast<bf16x4*>(at(l16, j * 2 + (lg >> 1)) + ((lg & 1) << 3)) = o;
          }
          wave_sync();
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            const int r = (lane + 64 * u) / 8, c = lane % 8;
            const int f = n0 + wm * WM + i * 16 + r, tok = m0 + wn * WN + c * 8;   // n_tok % 8 == 0: the eight tokens share a slice
            if (f < p.n2 && tok < p.M) {
              const u32x4 v = *reinterpret_cast<const u32x4*>(at(r, c));
              const int t = tok / p.n_tok, n = tok % p.n_tok;
              if constexpr (NEAR)
                __builtin_amdgcn_raw_buffer_store_b128(v, rsrc_v, ((unsigned)(t * p.heads * p.hd_pad + f) * (unsigned)p.n_tok + (unsigned)n) * 2u, 0, THROUGH);
              else
                __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(p.VT + ((long)t * p.heads * p.hd_pad + f) * p.n_tok + n));
            }
          }
          wave_sync();
        }
      } else {
      // per-column factor and bias: of feature l16 of block j (transposed store), of features 4 lg .. + 3 otherwise
      f32x4 c4[TOK ? 1 : TN], b4[TOK ? 1 : TN];
      float c1[TOK ? TN : 1], b1[TOK ? TN : 1];
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int col = n0 + wn * WN + j * 16;
        if constexpr (TOK) {
          b1[j] = p.bias[col + l16];
          c1[j] = p.cscale ? p.cscale[col + l16] : 1.0f;
        } else {
          b4[j] = *reinterpret_cast<const f32x4*>(p.bias + col + lg * 4);
          c4[j] = p.cscale ? *reinterpret_cast<const f32x4*>(p.cscale + col + lg * 4) : f32x4{1.f, 1.f, 1.f, 1.f};
        }
      }
      if constexpr (F32_OUT) {
#pragma unroll
        for (int q = 2; q < XAHEAD; ++q) xload(lane, q);
#pragma unroll
        for (int q = 0; q < PASSES; ++q) {
#pragma unroll
          for (int jj = 0; jj < 2; ++jj) {
            const int j = (q % 2) * 2 + jj;
            f32x4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = __builtin_fmaf(acc[q / 2][j][e], c4[j][e], b4[j][e]);
            *reinterpret_cast<f32x4*>(at(l16, jj * 4 + lg)) = v;
          }
          wave_sync();
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            const int r = (lane + 64 * u) / 8, c = lane % 8;
            const int row = m0 + wm * WM + (q / 2) * 16 + r, col = n0 + wn * WN + (q % 2) * 32 + c * 4;
            const f32x4 v = *reinterpret_cast<const f32x4*>(at(r, c));
            if (row < p.M && col < p.N) {   // read next by a row kernel, not by this launch
              if constexpr (NEAR)
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, xr[q % XAHEAD][u] + v), rsrc_x,
                                                       ((unsigned)row * (unsigned)p.ldr + (unsigned)col) * 4u, 0, THROUGH);
              else
                __builtin_nontemporal_store(xr[q % XAHEAD][u] + v, reinterpret_cast<f32x4*>(p.R + (long)row * p.ldr + col));
            }
          }
          wave_sync();
          if (q + XAHEAD < PASSES) xload(lane, q + XAHEAD);
        }
      } else if constexpr (TOK) {
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int h = 0; h < TM / 4; ++h) {   // 64 tokens each
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              bf16x4 o;
#pragma unroll
              for (int e = 0; e < 4; ++e) o[e] = (bf16_t)__builtin_fmaf(acc[h * 4 + i][j][e], c1[j], b1[j]);
              *reinterpret_cast<bf16x4*>(at(l16, i * 2 + (lg >> 1)) + ((lg & 1) << 3)) = o;
            }
            wave_sync();
#pragma unroll
            for (int u = 0; u < 2; ++u) {
              const int r = (lane + 64 * u) / 8, c = lane % 8;
              const int f = n0 + wn * WN + j * 16 + r, tok = m0 + wm * WM + h * 64 + c * 8;   // n_tok % 8 == 0: the eight tokens share a slice
              if (f < p.N && tok < p.M) {
                const u32x4 v = *reinterpret_cast<const u32x4*>(at(r, c));
                const int t = tok / p.n_tok, n = tok % p.n_tok;
                if constexpr (NEAR)
                  __builtin_amdgcn_raw_buffer_store_b128(v, rsrc_v, ((unsigned)(t * p.heads * p.hd_pad + f) * (unsigned)p.n_tok + (unsigned)n) * 2u, 0, THROUGH);
                else
                  __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(p.VT + ((long)t * p.heads * p.hd_pad + f) * p.n_tok + n));
              }
            }
            wave_sync();
          }
      } else if constexpr (MX_OUT) {
        // act(acc * cscale + bias) converted to MXFP8 along the output features (the contraction dimension of the next
        // product).  Blocks 2 b and 2 b + 1 of a token's four lanes are one block of 32 features, eight in each lane.  Codes of
        // 32 rows are staged as rows of 64 bytes, 16-byte chunk c of row r at c ^ (r / 4) % 4.
        auto code_at = [&](int r, int c) { return stg + r * 64 + ((c ^ ((r >> 2) & 3)) << 4); };
#pragma unroll
        for (int i2 = 0; i2 < TM; i2 += 2) {
#pragma unroll
          for (int i = i2; i < i2 + 2; ++i) {
            unsigned bytes[2];
#pragma unroll
            for (int b = 0; b < 2; ++b) {
              float v[8], amax = 0.f;
#pragma unroll
              for (int e = 0; e < 8; ++e) {
                const int j = 2 * b + (e >> 2);
                v[e] = apply_act_fast<EPI>(__builtin_fmaf(acc[i][j][e & 3], c4[j][e & 3], b4[j][e & 3]));
                amax = fmaxf(amax, fabsf(v[e]));
              }
              amax = fmaxf(amax, __shfl_xor(amax, 16, 64));
              amax = fmaxf(amax, __shfl_xor(amax, 32, 64));
              bytes[b] = mx_scale_byte(amax);
              const float inv = mx_inv_scale(bytes[b]);
#pragma unroll
              for (int x = 0; x < 2; ++x)
                *reinterpret_cast<unsigned*>(code_at((i - i2) * 16 + l16, 2 * b + x) + lg * 4) =
                    mx_pack4(v[4 * x] * inv, v[4 * x + 1] * inv, v[4 * x + 2] * inv, v[4 * x + 3] * inv);
            }
            // the wave's 64 features are half of a scale word
            const int row = m0 + wm * WM + i * 16 + l16, col = n0 + wn * WN;
            if (lg == 0 && row < p.M && col < p.ncq)
              reinterpret_cast<unsigned short*>(p.SC + (long)(col / BKB) * p.sc_ld + row)[wn & 1] = (unsigned short)(bytes[0] | bytes[1] << 8);
          }
          wave_sync();
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            const int r = (lane + 64 * u) / 4, c = lane % 4;
            const int row = m0 + wm * WM + i2 * 16 + r, col = n0 + wn * WN + c * 16;
            if (row < p.M && col < p.ncq) {
              const u32x4 v = *reinterpret_cast<const u32x4*>(code_at(r, c));
              if constexpr (NEAR) __builtin_amdgcn_raw_buffer_store_b128(v, rsrc_q, (unsigned)row * (unsigned)p.ldcq + (unsigned)col, 0, THROUGH);
              else __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(p.Cq + (long)row * p.ldcq + col));
            }
          }
          wave_sync();
        }
      } else {
#pragma unroll
        for (int i = 0; i < TM; ++i) {
#pragma unroll
          for (int j = 0; j < TN; ++j) {
            bf16x4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = (bf16_t)__builtin_fmaf(acc[i][j][e], c4[j][e], b4[j][e]);
            *reinterpret_cast<bf16x4*>(at(l16, j * 2 + (lg >> 1)) + ((lg & 1) << 3)) = o;
          }
          wave_sync();
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            const int r = (lane + 64 * u) / 8, c = lane % 8;
            const int row = m0 + wm * WM + i * 16 + r, col = n0 + wn * WN + c * 8;
            if (row < p.M && col < p.N) {
              const u32x4 v = *reinterpret_cast<const u32x4*>(at(r, c));
              if constexpr (NEAR) __builtin_amdgcn_raw_buffer_store_b128(v, rsrc_c, ((unsigned)row * (unsigned)p.ldc + (unsigned)col) * 2u, 0, THROUGH);
              else __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(p.C + (long)row * p.ldc + col));
            }
          }
          wave_sync();
        }
      }
      }
    }
    pos += (int)gridDim.x;
    if (pos >= n_tiles) break;
  }
}

// One instruction on caller-supplied registers: lane l gets a[l][0..7], b[l][0..7] and the scale registers
// sa[l], sb[l] (byte 0 is used) and leaves its four result registers in d[l][0..3].
__global__ __launch_bounds__(64) void k_mx_mfma_probe(const int* a, const int* b, const int* sa, const int* sb, float* d) {
  const int l = threadIdx.x;
  i32x8 fa, fb;
#pragma unroll
  for (int e = 0; e < 8; ++e) { fa[e] = a[l * 8 + e]; fb[e] = b[l * 8 + e]; }
  const f32x4 acc = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(fa, fb, f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0, sa[l], 0, sb[l]);
#pragma unroll
  for (int e = 0; e < 4; ++e) d[l * 4 + e] = acc[e];
}

template <int EPI, bool DUAL, int TM, int WAVES_M, int WAVES_N>
hipError_t launch_tile(const MxGemmParams& p, int cols, hipStream_t st) {
  using T = MxTile<TM, WAVES_M, WAVES_N>;
  const int gm = (p.M + T::BM - 1) / T::BM, gq = (cols + T::BN - 1) / T::BN, gv = DUAL ? (p.n2 + T::BN - 1) / T::BN : 0, gn = gq + gv, n_tiles = gm * gn, slots = cu_count() * (512 / T::NT);
  const int at_once = slots / 8, gw = band_columns(gn, (double)T::BM * p.K, (double)T::BN * p.K, n_tiles < 8 * at_once ? (n_tiles + 7) / 8 : at_once);
  if (gq * T::BN > p.Npad || gv * T::BN > p.n2_pad) return hipErrorInvalidValue;
  constexpr bool MX_OUT = EPI == EPI_BIAS_GELU_ERF || EPI == EPI_BIAS_GELU_TANH;
  const dim3 grid((unsigned)(n_tiles < slots ? n_tiles : slots)), block(T::NT);
  if (EPI == EPI_BIAS_RESIDUAL ? 4.0 * p.M * p.N <= NEAR_ROWS_MX : (double)p.M * (MX_OUT ? p.ncq : 2 * (p.N > p.n2 ? p.N : p.n2)) <= NEAR_OUT)
    k_gemm_mxfp8<EPI, DUAL, TM, WAVES_M, WAVES_N, true><<<grid, block, T::LDS, st>>>(p, gm, gw, gn, gq, n_tiles);
  else
    k_gemm_mxfp8<EPI, DUAL, TM, WAVES_M, WAVES_N, false><<<grid, block, T::LDS, st>>>(p, gm, gw, gn, gq, n_tiles);
  return hipGetLastError();
}

// tile columns that hold nothing but padding are not launched (the weights are packed to 256 rows)
template <int EPI>
int launched_columns(const MxGemmParams& p) { return (EPI == EPI_BIAS_GELU_ERF || EPI == EPI_BIAS_GELU_TANH) && p.ncq > p.N ? p.ncq : p.N; }

template <int EPI, bool DUAL = false>
int tile_for(const MxGemmParams& p) {
  const int cols = launched_columns<EPI>(p);
  // 256 x 256 tiles, a workgroup of eight waves per CU, 128 x 128 ones, two of four waves, or, for the residual product over more
  // than a round, 224 x 256 ones: the one estimated to take least.  us = start + rounds (fixed + slabs) + rounds without rounding up
  // (fixed + slabs): the residual product's workgroups drift apart, and over several rounds one's epilogue stands under
  // another's products.  The small tiles' last round counts 0.7 while one per CU holds it.  Fitted to products of 1024 to 106496 rows, 1024 to
  // 3200 columns and K 1024 to 12800; residual ones with 4 us for a start of large tiles behind another kernel, which those did
  // not hold, and 3 % that the 224-row ones have to be ahead.  Against the 372 products and pairs of tests/golden/product_times.txt the tile
  // taken is 0.2 to 0.6 % behind the fastest on average, 13 % at most (8256 rows, residual 1024 x 4096: 62.4 us, 224-row tiles 55.4).  us, 256 x 256 | 128 x 128 | 224 x 256: 1024 rows, 2048 x 1024 15.4 | 9.1, residual 1024 x 4096 51.0 | 24.7 | 47.2;
  // 26624 rows, 1152 x 1152 91.9 | 73.9 | 83.8, 1024 x 4096 130 | 151 | 127; 53248, 1024 x 4096 257 | 283 | 247; 106496, 1152 x 4352
  // 620 | 726 | 633.  In one round the 224-row tiles gain nothing that the 128 x 128 ones do not: 10240, 1152 x 4352 67.0 | 76.8 | 68.6.
  struct Cost { double start, round, round_slab, work, work_slab; };
  constexpr bool MX = EPI == EPI_BIAS_GELU_ERF || EPI == EPI_BIAS_GELU_TANH, RES = EPI == EPI_BIAS_RESIDUAL;
  constexpr Cost LARGE = RES ? Cost{6.54, 9.32, 1.21, 12.25, 0.27} : Cost{0.0, MX ? 9.7 : 5.3, 1.25, 0.0, 0.0};
  constexpr Cost SMALL = RES ? Cost{3.59, 2.41, 0.75, 6.11, 0.33} : Cost{2.0, MX ? 3.9 : 0.8, 0.93, 0.0, 0.0};
  const long cus = cu_count(), kt = p.K / BKB;
  const int cols2 = DUAL ? p.n2 : 0;
  const auto estimate = [&](const Cost& c, int bm, int bn, long slots, double half_round) {
    const long tiles = (p.M + bm - 1) / bm * (long)((cols + bn - 1) / bn + (cols2 + bn - 1) / bn), rem = tiles % slots;
    const double rounds = (double)(tiles / slots) + (rem == 0 ? 0.0 : 2 * rem <= slots ? half_round : 1.0);
    return c.start + rounds * (c.round + c.round_slab * kt) + (double)tiles / slots * (c.work + c.work_slab * kt);
  };
  double best = estimate(LARGE, 256, 256, cus, 1.0);
  int tile = 1;
  const auto offer = [&](double us, int t) { if (us < best) { best = us; tile = t; } };
  offer(estimate(SMALL, 128, 128, 2 * cus, 0.7), 2);
  if constexpr (RES)
    if ((p.M + 223) / 224 * (long)((cols + 255) / 256) > cus) offer(1.03 * estimate(Cost{6.58, 8.30, 1.10, 9.21, 0.31}, 224, 256, cus, 1.0), 3);
  return tile;
}

template <int EPI, bool DUAL = false>
hipError_t launch(const MxGemmParams& p, hipStream_t st) {
  const int cols = launched_columns<EPI>(p), tile = p.tile > 0 ? p.tile : tile_for<EPI, DUAL>(p);
  if constexpr (EPI == EPI_BIAS_RESIDUAL) {
    if (tile == 3) return launch_tile<EPI, DUAL, 7, 2, 4>(p, cols, st);
  }
  if (tile == 2) return launch_tile<EPI, DUAL, 4, 2, 2>(p, cols, st);
  return launch_tile<EPI, DUAL, 8, 2, 4>(p, cols, st);
}

// The two products of a pair in one launch: where that saves a round of 256 x 256 tiles, or the start of a launch among few
// rounds.  Encodes of 448-pixel slices, two launches | one, us: 1 slice, 300M 2541 | 2294; 10, SigLIP (3 rounds, none saved) 9179 |
// 9073; 16, 300M (3) 9495 | 9315; 40, SigLIP (9, one saved) 32694 | 32374; none saved and more of them, two launches: 48, 300M (9)
// 26239 | 26320, 104 (20) 55802 | 56182.
bool together(const MxGemmParams& p) {
  const long cus = cu_count(), rows = (p.M + 255) / 256, q = rows * ((p.N + 255) / 256), v = rows * ((p.n2 + 255) / 256);
  const auto rounds = [cus](long tiles) { return (tiles + cus - 1) / cus; };
  return rounds(q + v) <= 4 || rounds(q + v) < rounds(q) + rounds(v);
}

template <int EPI, bool DUAL, int TM, int WAVES_M, int WAVES_N>
hipError_t set_attr_tile() {
  constexpr int LDS = (int)MxTile<TM, WAVES_M, WAVES_N>::LDS;
  const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_gemm_mxfp8<EPI, DUAL, TM, WAVES_M, WAVES_N, true>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
  return e != hipSuccess ? e : hipFuncSetAttribute(reinterpret_cast<const void*>(&k_gemm_mxfp8<EPI, DUAL, TM, WAVES_M, WAVES_N, false>),
                                                   hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
}
template <int EPI, bool DUAL = false>
hipError_t set_attr() {
  hipError_t e = set_attr_tile<EPI, DUAL, 8, 2, 4>();
  if constexpr (EPI == EPI_BIAS_RESIDUAL) {
    if (e == hipSuccess) e = set_attr_tile<EPI, DUAL, 7, 2, 4>();
  }
  return e != hipSuccess ? e : set_attr_tile<EPI, DUAL, 4, 2, 2>();
}

}  // namespace

hipError_t mx_gemm_init() {
  static const hipError_t once = [] {
    hipError_t e;
    if ((e = set_attr<EPI_BIAS>()) != hipSuccess) return e;
    if ((e = set_attr<EPI_BIAS, true>()) != hipSuccess) return e;
    if ((e = set_attr<EPI_VT>()) != hipSuccess) return e;
    if ((e = set_attr<EPI_BIAS_GELU_ERF>()) != hipSuccess) return e;
    if ((e = set_attr<EPI_BIAS_GELU_TANH>()) != hipSuccess) return e;
    return set_attr<EPI_BIAS_RESIDUAL>();
  }();
  return once;
}

int mx_gemm_tile(const MxGemmParams& p) {
  switch (p.epi) {
    case EPI_BIAS: return p.n2 == 0 ? tile_for<EPI_BIAS>(p) : together(p) ? tile_for<EPI_BIAS, true>(p) : 0;
    case EPI_VT: return tile_for<EPI_VT>(p);
    case EPI_BIAS_GELU_ERF: return tile_for<EPI_BIAS_GELU_ERF>(p);
    case EPI_BIAS_GELU_TANH: return tile_for<EPI_BIAS_GELU_TANH>(p);
    case EPI_BIAS_RESIDUAL: return tile_for<EPI_BIAS_RESIDUAL>(p);
  }
  return -1;
}

hipError_t mx_gemm(const MxGemmParams& p, hipStream_t st) {
  // what the kernel assumes, checked where the launch is made (buffers hold whole 256-row tiles)
  constexpr int BM = 256, BN = 256;
  const long a_extent = ((long)(p.M + BM - 1) / BM * BM) * p.lda;
  if (p.M <= 0 || p.K <= 0 || p.K % BKB || p.Npad <= 0 || p.Npad % BN || p.N > p.Npad || p.lda < p.K || p.lda % 16 ||
      p.sa_ld < (long)(p.M + BM - 1) / BM * BM || a_extent >= (1L << 32) || (long)p.Npad * p.K >= (1L << 32) ||
      !p.A || !p.SA || !p.W || !p.SW || !p.bias)
    return hipErrorInvalidValue;
  switch (p.epi) {
    case EPI_BIAS:
      if (!p.C || p.N % 8) return hipErrorInvalidValue;
      if (p.n2 == 0) return launch<EPI_BIAS>(p, st);
      if (p.n2 < 0 || p.n2_pad % BN || p.n2 > p.n2_pad || (long)p.n2_pad * p.K >= (1L << 32) || !p.W2 || !p.SW2 || !p.bias2 || !p.VT || p.n_tok % 8 || p.hd_pad <= 0)
        return hipErrorInvalidValue;
      if (p.tile == 0 && !together(p)) {
        MxGemmParams q = p, v = p;
        q.n2 = 0;
        v.epi = EPI_VT; v.W = p.W2; v.SW = p.SW2; v.bias = p.bias2; v.cscale = p.cscale2; v.N = p.n2; v.Npad = p.n2_pad; v.n2 = 0;
        const hipError_t e = launch<EPI_BIAS>(q, st);
        return e != hipSuccess ? e : launch<EPI_VT>(v, st);
      }
      return launch<EPI_BIAS, true>(p, st);
    case EPI_VT: return p.VT && p.n_tok % 8 == 0 && p.hd_pad > 0 ? launch<EPI_VT>(p, st) : hipErrorInvalidValue;
    case EPI_BIAS_GELU_ERF:
    case EPI_BIAS_GELU_TANH:
      if (!p.Cq || !p.SC || p.ncq <= 0 || p.ncq % BKB || p.ldcq < p.ncq || p.ldcq % 16 || p.sc_ld < (long)(p.M + BM - 1) / BM * BM) return hipErrorInvalidValue;
      return p.epi == EPI_BIAS_GELU_ERF ? launch<EPI_BIAS_GELU_ERF>(p, st) : launch<EPI_BIAS_GELU_TANH>(p, st);
    case EPI_BIAS_RESIDUAL:   // the stream rows are addressed through 32-bit offsets
      if (!p.R || p.N % 4 || p.ldr < p.N || ((long)(p.M + BM - 1) / BM * BM) * p.ldr * 4 >= (1L << 32)) return hipErrorInvalidValue;
      return launch<EPI_BIAS_RESIDUAL>(p, st);
    default: return hipErrorInvalidValue;
  }
}

hipError_t mx_rows(const MxRowParams& p, hipStream_t st) {
  if (p.rows == 0) return hipSuccess;
  if (p.dim <= 0 || p.dim % 128 || p.ld_codes < p.dim || p.ld_codes % 4 || p.ld_scales < p.rows || !p.in || !p.codes ||
      !p.scales || (p.kind != 2 && !p.gamma) || (p.kind == 0 && !p.beta) || p.kind < 0 || p.kind > 2)
    return hipErrorInvalidValue;
  const dim3 grid((unsigned)((p.rows + 3) / 4)), block(256);
  const int per_lane = (p.dim / 4 + 63) / 64;
  const bool near = !p.in_bf16 && 4.0 * p.rows * p.dim <= NEAR_ROWS_MX;
#define MX_ROWS(BF, NV, PRE) (near ? k_mx_rows<BF, NV, PRE, true> : k_mx_rows<BF, NV, PRE, false>)<<<grid, block, 0, st>>>(p)
  if (p.in_bf16) {
    if (per_lane <= 4) MX_ROWS(true, 4, false); else if (per_lane <= 8) MX_ROWS(true, 8, false);
    else if (per_lane <= 16) MX_ROWS(true, 16, false); else MX_ROWS(true, 0, false);
  } else if (p.kind != 2 && per_lane <= 5) {
    switch (per_lane) {
      case 1: MX_ROWS(false, 1, true); break;
      case 2: MX_ROWS(false, 2, true); break;
      case 3: MX_ROWS(false, 3, true); break;
      case 4: MX_ROWS(false, 4, true); break;
      case 5: MX_ROWS(false, 5, true); break;
    }
  } else {
    if (per_lane <= 4) MX_ROWS(false, 4, false); else if (per_lane <= 8) MX_ROWS(false, 8, false);
    else if (per_lane <= 16) MX_ROWS(false, 16, false); else MX_ROWS(false, 0, false);
  }
#undef MX_ROWS
  return hipGetLastError();
}

void mx_mfma_probe(const int* a, const int* b, const int* sa, const int* sb, float* d, hipStream_t st) {
  k_mx_mfma_probe<<<dim3(1), dim3(64), 0, st>>>(a, b, sa, sb, d);
}

}  // namespace epd
