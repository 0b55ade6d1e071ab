// Tile-local flash attention for gfx950 (bf16 MFMA, fp32 online softmax).
//
// One workgroup = 4 waves, each owning QT sub-tiles of 16 queries of one (slice, head).  Keys and values of the same slice
// stream through LDS in blocks of 64 keys (double buffered, one barrier per block); the online softmax advances in steps
// of 32 keys.  Everything is computed transposed so that a lane always owns ONE query per sub-tile:
//     S^T = K Q^T        (left operand: key rows from LDS, right: Q from registers)
//     O^T += V^T P^T     (left operand: V^T rows from LDS, right: P^T from the S^T registers)
// on v_mfma_f32_16x16x32_bf16 (register e of lane l = row 4 (l / 16) + e, column l % 16; operands: k = 8 (l / 16) .. + 7).
// The rows of a key block are dealt to the two S^T blocks of a step such that a lane's eight results are keys
// 8 (l / 16) .. + 7 of its query: exponentiated they are the second product's right operand as they stand, and V^T is
// read in the order it has in memory.  A K / V^T fragment read from LDS feeds all QT sub-tiles of the wave.
// Values arrive pre-transposed ([slice, head, hd, token]) from the value GEMM.
//
// What bounds it: the SIMD's issue port, which exponentials and products share, and in calls of one or two slices the chain
// product -> exponentials -> product of a wave.  Beside the v_mfma_f32_32x32x16_bf16 kernel this replaces (32 queries per
// wave, V^T through registers; us per launch, 1024 tokens, on one card): 104 slices x 16 heads of 64 517 -> 511, 13 slices
// 71.3 -> 67.7; 10 slices x 16 heads of 72 69.9 -> 62.9, 23 of 729 tokens 108 -> 83; 40 slices x 25 heads of 128
// 649 -> 581; one slice 16.9 -> 14.0 (64), 22.1 -> 16.1 (72), 27.9 -> 23.5 (128), three of 1025 tokens 26.4 -> 24.9.
// What gave it: head dim 72 takes 96 + 80 rows of products a step instead of 80 + 96 of twice the width, and no pass of the
// values through registers leaves the registers for three workgroups; a query's maximum is exchanged between lanes only
// when the reference moves.
//
// The queries arrive carrying the logit scale: q = (1 / sqrt(hd)) log2(e) x (the projection that makes them has
// the factor folded into its weights), so the S^T registers are the logits in the log2 domain as they stand
// and the weights are exp2 of them with no arithmetic in between.
//
// The reference value m that is subtracted from a query's logits follows the
// running maximum lazily: it moves (and the accumulators are rescaled) only
// when a logit exceeds it by more than RESCALE_LOG2 in the log2 domain, which
// bounds the weights by 2^RESCALE_LOG2 instead of by 1: harmless for bf16
// weights and fp32 sums, and it takes the rescaling out of almost every step
// (with the exact running maximum some query of a wave moves it at most steps).
// The sum of the weights is taken over the rounded values the second product
// uses: two per v_dot2_f32_bf16, or, where V^T has a spare row past the head dim
// (hd = 72 in 80 rows), by a row of ones in V^T, so that the sum comes out of the
// second product itself.  Where the sum is taken on the VALU
// the common step computes no maximum at all: a step whose weights sum to
// more than 2^RESCALE_LOG2 (or overflow) is what triggers the maximum, the
// move of the reference and a second round of exponentials.
#include <algorithm>
#include <type_traits>

#include "kernels.h"

namespace epd {

namespace {

constexpr int BKEY = 64;  // keys per LDS block
constexpr float RESCALE_LOG2 = 8.0f;   // a logit may exceed the reference by this much (log2 domain)
constexpr float RESCALE_SUM = 256.0f;  // 2^RESCALE_LOG2: what a lane's 8 weights of a step may sum to

// maximum over the four lanes l, l ^ 16, l ^ 32, l ^ 48, which share a query: a swap of a register with itself leaves the
// even rows' values in one result and the odd rows' in the other
__device__ __forceinline__ float max_over_query(float x) {
  const unsigned a = __float_as_uint(x);
  const auto r = __builtin_amdgcn_permlane16_swap(a, a, false, false);
  const unsigned b = __float_as_uint(fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1])));
  const auto t = __builtin_amdgcn_permlane32_swap(b, b, false, false);
  return fmaxf(__uint_as_float(t[0]), __uint_as_float(t[1]));
}

// HD = head dim as stored in q, k, v^T.  The products run over HD rounded up to the MFMA shapes (32 for q.k, 16 rows of
// O^T).  Head dim 72, the one that is no such multiple, holds no padding: q is zero past it in registers, the key
// fragments past it are read from 16 bytes of zeros, and the one spare V^T row that exists, of ones, stands for all seven.
template <int HD>
struct AttnSmem {
  static_assert(HD == 64 || HD == 72 || HD == 96 || HD == 128, "head dims");
  static constexpr int KS = (HD + 31) / 32;         // k-steps of S^T
  static constexpr int OB = (HD + 15) / 16;         // 16-row blocks of O^T
  static constexpr bool ONES = HD % 16 != 0;        // a spare V^T row of ones makes the second product sum the weights
  static constexpr int V_ROWS = HD + (ONES ? 1 : 0);
  static constexpr int K_ELEMS = BKEY * HD;
  static constexpr int V_ELEMS = V_ROWS * BKEY;
  static constexpr size_t BYTES = (size_t)2 * (K_ELEMS + V_ELEMS) * sizeof(bf16_t) + (ONES ? 16 : 0);
  // Rows are unpadded (a load puts 64 lanes' chunks next to each other): the 16 rows of a read of one logical 16-byte chunk
  // are spread over the 64 banks by where the chunk sits in its row.  Key rows are read as {0-3, 8-11, 16-19, 24-27} + 4 b,
  // in the PAIRED order as {0-7, 16-23} + 8 b.
  template <bool PAIRED>
  static __device__ __forceinline__ int k_chunk(int row, int c) {
    if (PAIRED) {
      const int a = (row >> 4) & 1;
      return HD == 64 ? c ^ (a << 2 | ((row >> 1) & 3)) : HD == 96 ? c ^ (a << 1 | ((row >> 2) & 1)) : HD == 128 ? c ^ (a << 3 | (row & 7)) : c < 8 ? c ^ a : c;
    }
    const int a = (row >> 3) & 3;
    return HD == 64 ? c ^ (a << 1 | ((row >> 1) & 1)) : HD == 96 ? c ^ a : HD == 128 ? c ^ (a << 2 | (row & 3)) : c < 8 ? c ^ ((a >> 1) << 2) : c;
  }
  static __device__ __forceinline__ int v_chunk(int row, int c) { return c ^ ((row >> 1) & 7); }
};

// The accumulators of the second product live in registers named here (sub-tile u, block b: v[64 + 32 u + 4 b : + 3]) and are
// touched by assembly alone: left to the compiler they move from register to register at every product and around every
// branch that may change them.  The compiler does not see the wait states such assembly needs: two between a vector
// instruction that wrote an operand and the product (an s_nop in front of a step's products), 24 between a product and
// anything else that touches its accumulator.
#define EPD_ACC_LIST(X) \
  X(0, 64, 65, 66, 67) X(1, 68, 69, 70, 71) X(2, 72, 73, 74, 75) X(3, 76, 77, 78, 79) \
  X(4, 80, 81, 82, 83) X(5, 84, 85, 86, 87) X(6, 88, 89, 90, 91) X(7, 92, 93, 94, 95) \
  X(8, 96, 97, 98, 99) X(9, 100, 101, 102, 103) X(10, 104, 105, 106, 107) X(11, 108, 109, 110, 111) \
  X(12, 112, 113, 114, 115) X(13, 116, 117, 118, 119) X(14, 120, 121, 122, 123) X(15, 124, 125, 126, 127)

template <int I>   // acc += l r
__device__ __forceinline__ void acc_mfma(f32x4& acc, bf16x8 l, bf16x8 r) {
#define X(N, R0, R1, R2, R3)                                                                                          \
  if constexpr (I == N)                                                                                               \
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+{v[" #R0 ":" #R3 "]}"(acc) : "v"(l), "v"(r));
  EPD_ACC_LIST(X)
#undef X
}
template <int I>   // the accumulator is in its register here
__device__ __forceinline__ void acc_pin(f32x4& acc) {
#define X(N, R0, R1, R2, R3) \
  if constexpr (I == N) asm volatile("" : "+{v[" #R0 ":" #R3 "]}"(acc));
  EPD_ACC_LIST(X)
#undef X
}
// All accumulators of sub-tile U times f if `moved` (uniform) is not 0.
template <int U, int OB>
__device__ __forceinline__ void acc_scale(f32x4 (&a)[OB], int moved, float f) {
#define MUL(R) "v_mul_f32 v" #R ", %[f], v" #R "\n\t"
#define MUL4(R0, R1, R2, R3) MUL(R0) MUL(R1) MUL(R2) MUL(R3)
#define HEAD "s_cmp_eq_u32 %[m], 0\n\ts_cbranch_scc1 .Lacc_kept%=\n\ts_nop 7\n\ts_nop 7\n\ts_nop 7\n\t"
#define TAIL ".Lacc_kept%=:"
#define FOUR_0 MUL4(64, 65, 66, 67) MUL4(68, 69, 70, 71) MUL4(72, 73, 74, 75) MUL4(76, 77, 78, 79)
#define FOUR_1 MUL4(96, 97, 98, 99) MUL4(100, 101, 102, 103) MUL4(104, 105, 106, 107) MUL4(108, 109, 110, 111)
#define OUT_0 "+{v[64:67]}"(a[0]), "+{v[68:71]}"(a[1]), "+{v[72:75]}"(a[2]), "+{v[76:79]}"(a[3])
#define OUT_1 "+{v[96:99]}"(a[0]), "+{v[100:103]}"(a[1]), "+{v[104:107]}"(a[2]), "+{v[108:111]}"(a[3])
#define IN [m] "s"(moved), [f] "v"(f) : "scc"
  static_assert(OB == 4 || OB == 5 || OB == 6 || OB == 8, "blocks");
  if constexpr (U == 0) {
    if constexpr (OB == 4) asm volatile(HEAD FOUR_0 TAIL : OUT_0 : IN);
    if constexpr (OB == 5) asm volatile(HEAD FOUR_0 MUL4(80, 81, 82, 83) TAIL : OUT_0, "+{v[80:83]}"(a[4]) : IN);
    if constexpr (OB == 6)
      asm volatile(HEAD FOUR_0 MUL4(80, 81, 82, 83) MUL4(84, 85, 86, 87) TAIL : OUT_0, "+{v[80:83]}"(a[4]), "+{v[84:87]}"(a[5]) : IN);
    if constexpr (OB == 8)
      asm volatile(HEAD FOUR_0 MUL4(80, 81, 82, 83) MUL4(84, 85, 86, 87) MUL4(88, 89, 90, 91) MUL4(92, 93, 94, 95) TAIL
                   : OUT_0, "+{v[80:83]}"(a[4]), "+{v[84:87]}"(a[5]), "+{v[88:91]}"(a[6]), "+{v[92:95]}"(a[7]) : IN);
  } else {
    if constexpr (OB == 4) asm volatile(HEAD FOUR_1 TAIL : OUT_1 : IN);
    if constexpr (OB == 5) asm volatile(HEAD FOUR_1 MUL4(112, 113, 114, 115) TAIL : OUT_1, "+{v[112:115]}"(a[4]) : IN);
    if constexpr (OB == 6)
      asm volatile(HEAD FOUR_1 MUL4(112, 113, 114, 115) MUL4(116, 117, 118, 119) TAIL : OUT_1, "+{v[112:115]}"(a[4]), "+{v[116:119]}"(a[5]) : IN);
    if constexpr (OB == 8)
      asm volatile(HEAD FOUR_1 MUL4(112, 113, 114, 115) MUL4(116, 117, 118, 119) MUL4(120, 121, 122, 123) MUL4(124, 125, 126, 127) TAIL
                   : OUT_1, "+{v[112:115]}"(a[4]), "+{v[116:119]}"(a[5]), "+{v[120:123]}"(a[6]), "+{v[124:127]}"(a[7]) : IN);
  }
#undef MUL
#undef MUL4
#undef HEAD
#undef TAIL
#undef FOUR_0
#undef FOUR_1
#undef OUT_0
#undef OUT_1
#undef IN
}

template <int N, int I = 0, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<N, I + 1>(f);
  }
}

// A launch of a few slices leaves the memory idle, and the products behind it wait for weights that come from memory (a slab of a
// 128 x 128 tile takes 1500 cycles with 72, 128 or 200 tiles at work, 1100 with its weights in the Infinity Cache).  So `wgs` workgroups in
// front of the attention's read every line of the weights of the out-projection, of both MLP products and of the next layer's q, k and v.
// us without | with: attention of one slice of 16 heads of 64 12.5 | 14.9 (24 MB), FC2 behind it 21.0 | 16.0, FC1 15.0 | 13.4, out-projection
// 8.1 | 6.8; of three slices of 1025 tokens 27.1 | 28.9, FC2 40.3 | 32.5, out-projection 15.5 | 13.7.  Two loads in flight a thread: with
// eight on half as many workgroups the attention takes 16.2; on 32 of them 22.5 (they end last); one dword a line 15.9.
__device__ __forceinline__ void ask_for(const Ahead& a, int wgs) {
  const unsigned from = blockIdx.x * 256 + threadIdx.x, step = wgs * 256;
#pragma clang loop unroll(disable)
  for (int r = 0; r < a.n; ++r) {
    const u32x4* p = reinterpret_cast<const u32x4*>(a.at[r]);
    const unsigned n = a.pieces[r];
#pragma clang loop unroll(disable)
    for (unsigned i = from; i < n; i += 2 * step) {
      const u32x4 v = p[i], w = p[min(i + step, n - 1)];
      asm volatile("" :: "v"(v), "v"(w));
    }
  }
}

// QT sub-tiles of 16 queries per wave, four waves.
// LEAN: one step's S^T registers and weights only, no step issued ahead, so that four (head dim 64), three (72, 96) workgroups
// share a CU (112, 142, 144 registers; up to 128, 155, 162 with MASK and PAIRED); at head dim 128, where LDS holds two, the
// S^T product of step i + 1 is issued ahead of the softmax of step i.  So it is with 16 queries per wave at head dims 64 and 96, whose
// few waves leave the registers (us, lean | ahead: 64, one slice of 1024 tokens 14.1 | 12.5, three 22.4 | 21.6; 96, one 17.3 | 15.8, three
// 27.9 | 27.1; 72 and masked slices: equal, lean).  A third LDS buffer, loads two blocks ahead, gives nothing: a step is the wave's chain.
// PAIRED: a lane's eight keys of a step are 16 (l / 32) + 4 (l / 16 % 2) + {0..3, 8..11}, V^T fragments are two 8-byte halves, and
// the row sum on the VALU runs over a lane pair's sixteen weights in a row: the order of summation of a kernel on
// v_mfma_f32_32x32x16_bf16, whose bits this gives.  For calls whose output is converted to MXFP8: there a change of the last
// bit anywhere re-draws the conversion's rounding in all that follows (6 % of an encoder's output).  It costs twice
// the instructions of the row sums, 4 to 18 % of a launch (26 slices of 16 heads of 64, bf16 output | this: 136 | 160), and at
// head dim 64 more than this kernel gains: with this output the 32x32x16 kernel took 151 (five slices 36.2, this 41.6; one 18.1,
// 18.6); 96, 13 slices of 16 heads 124 -> 110; 128, ten of 25 heads 172 -> 160.  V^T as whole chunks whose halves two lane groups
// then exchange (v_permlane16_swap): the same bits, 2 to 5 % slower.
// MASK: the slices carry rows past n_keys (compiled apart: the unmasked kernel keeps its registers and its step free of
// the key-index compare).
template <int HD, int QT>
constexpr int per_cu() { return HD == 64 || (HD == 72 && QT == 1) ? 4 : HD <= 96 ? 3 : 2; }   // workgroups that share a CU
template <int HD, int QT, bool MASK, bool PAIRED>
__global__ __launch_bounds__(256, (per_cu<HD, QT>())) void k_attention_bf16(const bf16_t* __restrict__ q, const bf16_t* __restrict__ k,
                                                        const bf16_t* __restrict__ vt,
                                                        bf16_t* __restrict__ o, int n_tok, int n_keys, int n_q,
                                                        int q_shared, int heads, int n_pairs, long ld_qk,
                                                        long ld_o, unsigned char* __restrict__ oq,
                                                        unsigned* __restrict__ so, long ld_so, int n_ahead, const Ahead ahead) {
  if ((int)blockIdx.x < n_ahead) {   // uniform over the workgroup
    ask_for(ahead, n_ahead);
    return;
  }
  using SM = AttnSmem<HD>;
  constexpr bool LEAN = HD <= 96 && !(QT == 1 && HD != 72 && !MASK);
  constexpr int BQ = 64 * QT;   // queries per workgroup
  constexpr int KS = SM::KS, OB = SM::OB;
  constexpr int KCH = HD / 8;   // 16-byte chunks per key row
  constexpr int K_TOTAL = BKEY * KCH, V_TOTAL = HD * (BKEY / 8);   // chunks per block, whole waves of them
  constexpr int K_LOADS = (K_TOTAL + 255) / 256;
  constexpr int V_LOADS = (V_TOTAL + 255) / 256;
  constexpr bool K_RIGID = HD == 64;   // a load covers 32 whole rows: the loads of a thread differ by a uniform offset

  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  bf16_t* sK = reinterpret_cast<bf16_t*>(smem);       // [2][BKEY][HD]
  bf16_t* sV = sK + 2 * SM::K_ELEMS;                  // [2][V_ROWS][BKEY]

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, lg = lane >> 4;
  // Workgroups are dealt round-robin to the 8 XCDs: keep the q-blocks of one
  // (slice, head) on one XCD so that its K / V^T block is fetched into one L2.
  const int n_qb = (n_q + BQ - 1) / BQ;
  const int xcd = blockIdx.x & 7, seq = (blockIdx.x - n_ahead) >> 3;   // n_ahead % 8 == 0
  const int pair = (seq / n_qb) * 8 + xcd;          // (slice, head) index
  if (pair >= n_pairs) return;                      // whole workgroup leaves before any barrier
  const int qb = seq % n_qb, h = pair % heads, t = pair / heads;
  const long row0 = (long)t * n_tok;
  const int q0 = qb * BQ + wave * 16 * QT;
  // A sub-tile that begins inside the slice is computed whole: its rows past the last query are read like any other
  // (at most 15 of them) and never stored.
  bool act[QT];
  bool any_act = false;
#pragma unroll
  for (int u = 0; u < QT; ++u) { act[u] = q0 + u * 16 < n_q; any_act = any_act || act[u]; }
  const long q_row0 = q_shared ? 0 : row0;   // learned queries: the same rows for every slice

  const bf16_t* kbase = k + row0 * ld_qk + (long)h * HD;
  const bf16_t* vbase = vt + ((long)t * heads + h) * HD * (long)n_tok;

  // Q fragments: lane = query, 8 consecutive head-dim elements per k-step
  bf16x8 qf[QT][KS];
#pragma unroll
  for (int u = 0; u < QT; ++u) {
    const int qrow = act[u] ? q0 + u * 16 + l16 : 0;  // inactive sub-tiles read a valid row, result unused
    const bf16_t* qp = q + (q_row0 + qrow) * ld_qk + (long)h * HD + lg * 8;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      if (s * 32 + 32 <= HD || s * 32 + lg * 8 < HD) {
        qf[u][s] = *reinterpret_cast<const bf16x8*>(qp + s * 32);
      } else {   // head-dim positions past HD
#pragma unroll
        for (int e = 0; e < 8; ++e) qf[u][s][e] = (bf16_t)0.f;
      }
    }
  }

  // Both blocks go from global memory straight into LDS (no staging registers, no LDS stores by the waves); the hardware
  // puts lane l's 16 bytes at a wave-uniform base + 16 l, so the swizzle is applied on the global side.  A thread's chunks
  // keep their place inside every block: 32-bit byte offsets once, the block's base stays in scalar registers.
  unsigned koff[K_RIGID ? 1 : K_LOADS];
#pragma unroll
  for (int i = 0; i < (K_RIGID ? 1 : K_LOADS); ++i) {
    const int c = tid + 256 * i < K_TOTAL ? tid + 256 * i : 0;   // (waves past the block's end load nothing)
    const int row = c / KCH;
    koff[i] = (unsigned)(((long)row * ld_qk + SM::template k_chunk<PAIRED>(row, c % KCH) * 8) * 2);
  }
  const unsigned voff = (unsigned)(((long)(tid >> 3) * n_tok + SM::v_chunk(tid >> 3, tid & 7) * 8) * 2);   // 32 rows a load
  const unsigned ldsk = (unsigned)(size_t)(__attribute__((address_space(3))) void*)sK + wave * 1024;
  const unsigned ldsv = (unsigned)(size_t)(__attribute__((address_space(3))) void*)sV + wave * 1024;
  auto dma = [&](unsigned off, const bf16_t* base, unsigned dst) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" :: "v"(off), "s"(base), "s"(dst) : "memory", "m0");
  };
  auto gload = [&](int buf, int kb) {   // key block kb and its values -> LDS buffers buf
    const bf16_t* kblk = kbase + (long)kb * BKEY * ld_qk;   // uniform
    const bf16_t* vblk = vbase + (long)kb * BKEY;
#pragma unroll
    for (int i = 0; i < K_LOADS; ++i)
      if (256 * i + 256 <= K_TOTAL || wave * 64 + 256 * i < K_TOTAL)   // uniform
        dma(koff[K_RIGID ? 0 : i], K_RIGID ? kblk + (long)(256 / KCH) * i * ld_qk : kblk, ldsk + buf * (SM::K_ELEMS * 2) + i * 4096);
#pragma unroll
    for (int i = 0; i < V_LOADS; ++i)
      if (256 * i + 256 <= V_TOTAL || wave * 64 + 256 * i < V_TOTAL)
        dma(voff, vblk + (long)32 * i * n_tok, ldsv + buf * (SM::V_ELEMS * 2) + i * 4096);
  };
  // the thread's parts of key block kb have landed in buffers buf
  auto landed = [&](int buf, int kb) {
    __builtin_amdgcn_s_waitcnt(0 | (0x7 << 4) | (0xf << 8));   // vmcnt(0)
    asm volatile("" ::: "memory");
    if (MASK && (kb + 1) * BKEY > n_keys) {   // uniform: only the last block(s) of a slice whose rows are padded
      // Values of keys past n_keys are no part of the slice (the next slice's, or whatever an earlier call left in the
      // workspace): their weights are exactly zero, but 0 * NaN or 0 * Inf would still poison the sum, so a thread clears
      // them in the chunks it has loaded.  Word j of a chunk holds keys key0 + 2j, + 2j + 1.
      const int key0 = kb * BKEY + SM::v_chunk(tid >> 3, tid & 7) * 8;
#pragma unroll
      for (int i = 0; i < V_LOADS; ++i)
        if (256 * i + 256 <= V_TOTAL || wave * 64 + 256 * i < V_TOTAL) {
          u32x4* at = reinterpret_cast<u32x4*>(sV + buf * SM::V_ELEMS) + tid + 256 * i;
          u32x4 v = *at;
#pragma unroll
          for (int j = 0; j < 4; ++j)
            v[j] &= (key0 + 2 * j < n_keys ? 0x0000ffffu : 0u) | (key0 + 2 * j + 1 < n_keys ? 0xffff0000u : 0u);
          *at = v;
        }
    }
  };

  constexpr bool SUM_MFMA = SM::ONES;
  f32x4 oacc[QT][OB];
  // m_ref: the reference subtracted from this query's logits (log2 domain);
  // l_run: this lane's share of the running sum of weights (unused with SUM_MFMA)
  float m_ref[QT], l_run[QT];
  // Wave-uniform: some query of the wave has a reference other than 0.  While it is false (the common case:
  // logits of a few units) the exponentials are taken of the S^T registers as they are.
  bool shifted = false;
#pragma unroll
  for (int u = 0; u < QT; ++u) {
    m_ref[u] = 0.f;
    l_run[u] = 0.f;
#pragma unroll
    for (int b = 0; b < OB; ++b) oacc[u][b] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  auto acc_here = [&]() {
    static_for<QT>([&](auto u) { static_for<OB>([&](auto b) { acc_pin<u * 8 + b>(oacc[u][b]); }); });
  };
  acc_here();

  // S^T of one 32-key step for all sub-tiles: row i of key block b is key 8 (i / 4) + 4 b + i % 4, so that s[u][b] holds keys
  // 8 lg + 4 b + 0..3 of query l16, and the exponentials of both are the second product's operand as they stand: keys
  // 8 lg .. + 7.  (Fragment addresses: the swizzle depends on l16 alone.)
  const int krow = PAIRED ? 16 * (l16 >> 3) + (l16 & 7) : 8 * (l16 >> 2) + (l16 & 3);
  unsigned kfo[KS];
#pragma unroll
  for (int st = 0; st < KS; ++st) kfo[st] = (unsigned)(krow * HD + SM::template k_chunk<PAIRED>(krow, (st * 4 + lg) % KCH) * 8);
  auto issue_s = [&](f32x4 (&s)[QT][2], int buf, int kt) {
    const bf16_t* ks = sK + buf * SM::K_ELEMS;
    // fragments two k-steps ahead: the LDS latency is paid once per step, in front of it
    bf16x8 kf[2][2];
    auto read_k = [&](int st) {
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        const bf16_t* a = ks + kfo[st] + (kt * 32 + b * (PAIRED ? 8 : 4)) * HD;
        if (SM::ONES && st == KS - 1) a = lg == 0 ? a : sV + 2 * SM::V_ELEMS;   // past the head dim: the zeros behind V^T
        kf[st & 1][b] = *reinterpret_cast<const bf16x8*>(a);
      }
    };
    read_k(0);
    read_k(1);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int st = 0; st < KS; ++st) {
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int u = 0; u < QT; ++u)
          s[u][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[st & 1][b], qf[u][st], st == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : s[u][b], 0, 0, 0);
      if (st + 2 < KS) {
        __builtin_amdgcn_sched_barrier(0);
        read_k(st + 2);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
  // Where the softmax of a step follows its S^T product directly.  The compiler keeps the eight wait states behind a product
  // on the way through the rare shift of the logits, but not past it: its search does not look at the direct way, and
  // the first exponential stood three behind.  (Everywhere else a second product or the next S^T product lies in between.)
  // us with 8 | 5 wait states here: one slice of 16 heads of 64 14.4 | 14.3, 13 68.3 | 68.4, 104 529.6 | 526.1; of 72 10 64.4 | 64.4.
  auto settle = [&](f32x4 (&s)[QT][2]) {
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < QT; ++u) asm volatile("" : "+v"(s[u][0]), "+v"(s[u][1]));
    asm volatile("s_nop 7" ::: "memory");
#pragma unroll
    for (int u = 0; u < QT; ++u) asm volatile("" : "+v"(s[u][0]), "+v"(s[u][1]));
    __builtin_amdgcn_sched_barrier(0);
  };
  // weights of one step from its shifted logits, and (unless the second product sums them) their
  // sum over the rounded values that product uses, two per instruction
  auto weights = [&](const f32x4 (&sv)[2], bf16x8& pv, float& psum) {
#pragma unroll
    for (int e = 0; e < 8; ++e) pv[e] = (bf16_t)__builtin_amdgcn_exp2f(sv[e >> 2][e & 3]);
    psum = 0.f;
    if (!SUM_MFMA) {
      const bf16x2 ones = {(bf16_t)1.0f, (bf16_t)1.0f};
      auto add = [&](float x) {
        x = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pv, pv, 0, 1), ones, x, false);
        x = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pv, pv, 2, 3), ones, x, false);
        x = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pv, pv, 4, 5), ones, x, false);
        return __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(pv, pv, 6, 7), ones, x, false);
      };
      psum = add(0.f);
      if (PAIRED) {   // lanes 32 .. 63 go on from the sums of lanes 0 .. 31 and hold the sixteen weights', the others their own eight's
        const unsigned z = __float_as_uint(psum);
        const auto r = __builtin_amdgcn_permlane32_swap(0u, z, false, false);   // r[0]: 0 | the low lanes' sums
        psum = add(__uint_as_float(r[0]));
      }
    }
  };
  // Online softmax of one step, one query of each sub-tile per lane (shared with three others).  `force`: the first
  // step of a slice takes its own maximum as the reference, whatever its size.
  auto softmax = [&](f32x4 (&s)[QT][2], bf16x8 (&pf)[QT], int key0, bool force) {
    if (MASK && key0 + 32 > n_keys) {   // uniform; only the last steps of a slice whose rows are padded
      // rows past n_keys are no tokens: logit -inf, weight 0 (the first step always holds a real key,
      // so the reference is finite by the time a step is masked entirely)
#pragma unroll
      for (int u = 0; u < QT; ++u)
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (key0 + (PAIRED ? 16 * (lg >> 1) + 8 * (e >> 2) + 4 * (lg & 1) + (e & 3) : 8 * lg + e) >= n_keys) s[u][e >> 2][e & 3] = -INFINITY;
    }
    // logits relative to the reference as it stands (log2 domain already: q carries the scale)
    if (shifted) {
#pragma unroll
      for (int u = 0; u < QT; ++u)
#pragma unroll
        for (int e = 0; e < 8; ++e) s[u][e >> 2][e & 3] -= m_ref[u];
    }
    // the lane's part of the maximum, by three-input maxima (the two-input form would first quieten its inputs)
    auto lane_max = [&](int u) {
      float mx = fmaxf(fmaxf(s[u][0][0], s[u][0][1]), s[u][0][2]);
      mx = fmaxf(fmaxf(mx, s[u][0][3]), s[u][1][0]);
      mx = fmaxf(fmaxf(mx, s[u][1][1]), s[u][1][2]);
      return fmaxf(fmaxf(mx, s[u][1][3]), s[u][1][3]);
    };
    // What a lane's share of a query is judged by.  Where the sum is taken on the VALU the weights are taken against the
    // reference as it stands, no maximum, and their sum tells whether one of them was too large (a logit above
    // RESCALE_LOG2 alone makes the sum exceed 2^RESCALE_LOG2; an overflowed weight makes it infinite).  Where the sum sits
    // in the accumulator of the second product, by the maximum.
    float psum[QT], gauge[QT];
    bool any_high = false;
    constexpr float LIMIT = SUM_MFMA ? RESCALE_LOG2 : RESCALE_SUM;
#pragma unroll
    for (int u = 0; u < QT; ++u) {
      if constexpr (SUM_MFMA) {
        gauge[u] = lane_max(u);
        any_high = any_high || gauge[u] > LIMIT;
      } else {
        weights(s[u], pf[u], psum[u]);
        gauge[u] = psum[u];
        any_high = any_high || !(gauge[u] <= LIMIT);
      }
    }
    int moved = 0;   // uniform
    float alpha[QT];
#pragma unroll
    for (int u = 0; u < QT; ++u) alpha[u] = 1.0f;
    if (force || __builtin_amdgcn_ballot_w64(any_high) != 0) {
      moved = 1;
#pragma unroll
      for (int u = 0; u < QT; ++u) {
        const float mx = max_over_query(lane_max(u));
        // Whether THIS query's reference moves depends on its own logits only (the move is entered when any
        // query of the wave asks for it): a query's bits must not depend on which other queries share its
        // wave, which in slices whose rows are padded can be rows of the next slice.
        const bool high = SUM_MFMA ? gauge[u] > LIMIT : !(gauge[u] <= LIMIT);
        const bool mine = force || max_over_query(high ? 1.0f : 0.f) > 0.f;
        // this query's reference moves by d: to the step's maximum (a sum above 2^RESCALE_LOG2 over 8 weights
        // means a logit above RESCALE_LOG2 - 3).  First step: unless that maximum is within a few units of 0
        // already (then the reference stays 0 and the step's weights stay below 2^4 each)
        const float d = !mine ? 0.f : (force ? (fabsf(mx) > 4.0f ? mx : 0.f) : mx);
        shifted = shifted || __builtin_amdgcn_ballot_w64(d != 0.f) != 0;
        // nothing has been accumulated before the first step (and the factor would overflow for a
        // first maximum below -127)
        alpha[u] = force ? 1.0f : __builtin_amdgcn_exp2f(-d);
        l_run[u] *= alpha[u];
#pragma unroll
        for (int e = 0; e < 8; ++e) s[u][e >> 2][e & 3] -= d;
        m_ref[u] += d;
        if (!SUM_MFMA) weights(s[u], pf[u], psum[u]);   // again, against the new reference
      }
    }
#pragma unroll
    for (int u = 0; u < QT; ++u) {
      if (SUM_MFMA) weights(s[u], pf[u], psum[u]);
      else l_run[u] += psum[u];
    }
    static_for<QT>([&](auto u) { acc_scale<u>(oacc[u], moved, alpha[u]); });
  };
  // O^T += V^T P^T for one step; rows past the head dim all read the row of ones.  The first PRE fragments are read ahead
  // (in front of the S^T products or the softmax before it), fragment b + PRE behind the products of fragment b.
  constexpr int PRE = QT == 1 && HD == 64 ? OB : 2;
  unsigned vfo[2], vfo_last[2];   // by step of the block
#pragma unroll
  for (int kt = 0; kt < 2; ++kt) {
    vfo[kt] = (unsigned)(l16 * BKEY + SM::v_chunk(l16, kt * 4 + (PAIRED ? lg & 2 : lg)) * 8 + (PAIRED ? (lg & 1) * 4 : 0));
    vfo_last[kt] = SM::ONES && l16 > HD % 16 ? (unsigned)(HD % 16 * BKEY) : vfo[kt];
  }
  bf16x8 vf[PRE];
  auto read_v = [&](int buf, int kt, int b) {
    const unsigned o = b == OB - 1 ? vfo_last[kt] : vfo[kt];
    const bf16_t* v = sV + buf * SM::V_ELEMS + b * 16 * BKEY;
    if constexpr (PAIRED) {   // the other half of the keys: the neighbouring chunk, which the swizzle keeps in the pair
      const bf16x4 x = *reinterpret_cast<const bf16x4*>(v + o), y = *reinterpret_cast<const bf16x4*>(v + (o ^ 8u));
      vf[b % PRE] = __builtin_shufflevector(x, y, 0, 1, 2, 3, 4, 5, 6, 7);
    } else {
      vf[b % PRE] = *reinterpret_cast<const bf16x8*>(v + o);
    }
  };
  auto pre_pv = [&](int buf, int kt) {
#pragma unroll
    for (int b = 0; b < PRE; ++b) read_v(buf, kt, b);
  };
  auto issue_pv = [&](bf16x8 (&pf)[QT], int buf, int kt) {
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < QT; ++u) asm volatile("" : "+v"(pf[u]));   // the weights are written in front of the nop
    asm volatile("s_nop 1");
    static_for<OB>([&](auto b) {
      static_for<QT>([&](auto u) { acc_mfma<u * 8 + b>(oacc[u][b], vf[b % PRE], pf[u]); });
      __builtin_amdgcn_sched_barrier(0);
      if (b + PRE < OB) read_v(buf, kt, b + PRE);
      __builtin_amdgcn_sched_barrier(0);
    });
  };

  // NB blocks hold keys (the last one may reach past them: masked), NF of them in both steps; a single step over the first
  // half of the last block is the rest.
  const int NB = (n_keys + BKEY - 1) / BKEY, NF = MASK ? (n_keys + 31) / 64 : NB;
  gload(0, 0);
  if constexpr (SM::ONES) {
    if (tid < 2 * BKEY) sV[(tid / BKEY) * SM::V_ELEMS + HD * BKEY + tid % BKEY] = (bf16_t)1.0f;
    if (tid < 8) sV[2 * SM::V_ELEMS + tid] = (bf16_t)0.f;
  }
  landed(0, 0);
  __syncthreads();

  if (!any_act) {   // uniform: the wave's queries lie past the slice; it only loads
#pragma clang loop unroll(disable)
    for (int kb = 0; kb + 1 < NB; ++kb) {
      gload((kb & 1) ^ 1, kb + 1);
      landed((kb & 1) ^ 1, kb + 1);
      __syncthreads();
    }
    return;
  }
  int first = 1;   // opaque and kept in a loop that is not peeled
  asm volatile("" : "+s"(first));
  if constexpr (LEAN) {
    f32x4 s0[QT][2];
    bf16x8 p0[QT];
#pragma clang loop unroll(disable)
    for (int kb = 0; kb < NF; ++kb) {
      const int buf = kb & 1;
      const bool more = kb + 1 < NB;
      if (more) gload(buf ^ 1, kb + 1);   // the other buffer: nobody reads it after the previous barrier
      issue_s(s0, buf, 0);
      settle(s0);
      softmax(s0, p0, kb * BKEY, first);
      first = 0;
      pre_pv(buf, 0);
      issue_s(s0, buf, 1);   // the weights of step 0 are out of the S^T registers: step 1's product starts
      issue_pv(p0, buf, 0);  // under the second product of step 0
      pre_pv(buf, 1);
      softmax(s0, p0, kb * BKEY + 32, false);
      issue_pv(p0, buf, 1);
      if (more) {
        landed(buf ^ 1, kb + 1);
        __syncthreads();
      }
    }
    // (a loop of at most one turn: around a branch the compiler would copy the accumulators)
#pragma clang loop unroll(disable)
    for (int kb = NF; kb < NB; ++kb) {
      issue_s(s0, kb & 1, 0);
      settle(s0);
      softmax(s0, p0, kb * BKEY, first);
      pre_pv(kb & 1, 0);
      issue_pv(p0, kb & 1, 0);
    }
  } else {
    // the S^T MFMAs of the next step are in flight while the VALU does the softmax of the current one; s0 of a
    // block is issued right after the barrier that published the block
    f32x4 s0[QT][2], s1[QT][2];
    bf16x8 p0[QT], p1[QT];
    issue_s(s0, 0, 0);
#pragma clang loop unroll(disable)
    for (int kb = 0; kb < NF; ++kb) {
      const int buf = kb & 1;
      const bool more = kb + 1 < NB;
      if (more) gload(buf ^ 1, kb + 1);   // the other buffer: nobody reads it after the previous barrier
      issue_s(s1, buf, 1);
      pre_pv(buf, 0);
      softmax(s0, p0, kb * BKEY, first);
      first = 0;
      issue_pv(p0, buf, 0);
      pre_pv(buf, 1);
      softmax(s1, p1, kb * BKEY + 32, false);
      issue_pv(p1, buf, 1);
      if (more) {
        landed(buf ^ 1, kb + 1);
        __syncthreads();
        issue_s(s0, buf ^ 1, 0);
      }
    }
#pragma clang loop unroll(disable)
    for (int kb = NF; kb < NB; ++kb) {
      pre_pv(kb & 1, 0);
      settle(s0);
      softmax(s0, p0, kb * BKEY, first);
      issue_pv(p0, kb & 1, 0);
    }
  }
  asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7" ::: "memory");
  acc_here();
#pragma unroll
  for (int u = 0; u < QT; ++u) {
    if (!act[u]) continue;
    // SUM_MFMA: row HD of O^T holds the sum, in the 16 lanes of one group
    float l_tot;
    if constexpr (SUM_MFMA) {
      l_tot = __shfl(oacc[u][OB - 1][0], (HD % 16 / 4) * 16 + l16, 64);
    } else {
      l_tot = l_run[u] + __shfl_xor(l_run[u], 16, 64);
      if (PAIRED) l_tot = __shfl(l_tot, lane | 32, 64);   // whole in the upper lanes
      else l_tot += __shfl_xor(l_tot, 32, 64);
    }
    if (q0 + u * 16 + l16 >= n_q) continue;   // the slice's queries need not fill its last sub-tile (nor its rows a wave)
    const float inv = 1.0f / l_tot;
    if constexpr (HD % 32 == 0) {
      if (oq) {
        // MXFP8 output (the out-projection's operand): block b of this head = 32 head-dim rows = O^T blocks 2 b and
        // 2 b + 1, eight rows in each of the query's four lanes, so the block's largest magnitude is two exchanges
        // away; codes [row][ld_o bytes], scale words [column / 128][ld_so].
        const long row = (long)t * n_q + q0 + u * 16 + l16;
#pragma unroll
        for (int b = 0; b < HD / 32; ++b) {
          float v[8];
          float amax = 0.f;
#pragma unroll
          for (int e = 0; e < 8; ++e) { v[e] = oacc[u][2 * b + (e >> 2)][e & 3] * inv; amax = fmaxf(amax, fabsf(v[e])); }
          amax = fmaxf(amax, __shfl_xor(amax, 16, 64));   // the four lanes share a query: all of them are here
          amax = fmaxf(amax, __shfl_xor(amax, 32, 64));
          const unsigned byte = mx_scale_byte(amax);
          const float sc = mx_inv_scale(byte);
          const int col0 = h * HD + b * 32;
#pragma unroll
          for (int i = 0; i < 2; ++i)
            *reinterpret_cast<unsigned*>(oq + row * ld_o + col0 + i * 16 + lg * 4) =
                mx_pack4(v[i * 4] * sc, v[i * 4 + 1] * sc, v[i * 4 + 2] * sc, v[i * 4 + 3] * sc);
          if (lg == 0) reinterpret_cast<unsigned char*>(so + (long)(col0 >> 7) * ld_so + row)[(col0 >> 5) & 3] = (unsigned char)byte;
        }
        continue;
      }
    }
    bf16_t* op = o + ((long)t * n_q + q0 + u * 16 + l16) * ld_o + (long)h * HD;
#pragma unroll
    for (int b = 0; b < OB; ++b) {
      const int d0 = b * 16 + lg * 4;
      if (HD % 16 != 0 && d0 >= HD) continue;   // rows of O^T past the head dim
      bf16x4 ov;
#pragma unroll
      for (int e = 0; e < 4; ++e) ov[e] = (bf16_t)(oacc[u][b][e] * inv);
      *reinterpret_cast<bf16x4*>(op + d0) = ov;
    }
  }
}

template <int HD, int QT, bool MASK, bool PAIRED>
hipError_t launch_attn_m(const bf16_t* q, const bf16_t* k, const bf16_t* vt, bf16_t* o, int n_slices,
                         int n_tok, int n_keys, int n_q, int q_shared, int heads, long ld_qk, long ld_o,
                         unsigned char* oq, unsigned* so, long ld_so, const Ahead* ahead, hipStream_t st) {
  constexpr int BQ = 64 * QT;
  const int n_qb = (n_q + BQ - 1) / BQ, n_pairs = n_slices * heads;
  const long n_wg = (long)((n_pairs + 7) / 8) * 8 * n_qb;
  // 256 workgroups ask for the lines, fewer where they would take places of workgroups that could all run at once (three slices of 1025 tokens, 816
  // workgroups and 1024 places: 3.53 ms with 256, 3.46 with 128).  Where they must, the more of them the sooner they leave.
  const long free = (long)cu_count() * per_cu<HD, QT>() - n_wg;
  const int n_ahead = !ahead || ahead->n == 0 ? 0 : free < 128 ? 256 : (int)std::min(256L, free / 64 * 64);
  if (n_wg + n_ahead > 0x7fffffffL) return hipErrorInvalidValue;
  k_attention_bf16<HD, QT, MASK, PAIRED><<<dim3((unsigned)n_wg + n_ahead), dim3(256), AttnSmem<HD>::BYTES, st>>>(
      q, k, vt, o, n_tok, n_keys, n_q, q_shared, heads, n_pairs, ld_qk, ld_o, oq, so, ld_so, n_ahead, n_ahead ? *ahead : Ahead{});
  return hipGetLastError();
}

// 16 queries per wave, or 32: twice as many waves, each with half of a step's chain, while they all run at once.  By the most
// workgroups a CU gets (a (slice, head) keeps to one XCD), of 64 queries and of 128; LDS holds five of 64 at head dim 64,
// four at 72, three at 96 and two at 128.  us, 32 | 16 queries per wave (16 heads of 64 and 72, 12 of 96, 25 of 128; slices of 1024 tokens):
//   two of 64: head dim 128, one slice 26.0 | 23.8; 72, two 21.6 | 20.5
//   three: 64, three slices 25.8 | 20.6; 72 28.8 | 26.4; 96, four 33.7 | 28.9; but 128, one of 1025 tokens 38.2 | 39.9
//   four against two of 128: 64, four slices 27.1 | 25.7, PAIRED 29.3 | 28.9 and three of 1025 29.5 | 30.5; 72, four 30.1 | 33.1; 96, five
//     34.5 | 38.7; 128, two 38.2 | 44.7
//   four against three of 128: 64, seven of 576 tokens 21.0 | 16.3, 17 of 192 10.8 | 8.3; 72, seven of 576 24.9 | 21.8; 96, nine of 576
//     28.0 | 25.4; 128, four of 576 34.0 | 30.2; four of 128 (slices of up to 64 tokens): 64 6.4 | 6.0; 72 10.5 | 9.0; 96 13.0 | 11.7; 128 15.9 | 14.2
// A query's bits are the same.
bool short_waves(int n_slices, int n_q, int heads, int hd, bool paired) {
  const long pairs = ((long)n_slices * heads + 7) / 8, cus = cu_count() >= 8 ? cu_count() / 8 : 1;   // of an XCD
  auto per_cu = [&](int queries) { return (pairs * ((n_q + queries - 1) / queries) + cus - 1) / cus; };
  const long of_64 = per_cu(64), of_128 = per_cu(128);
  return of_64 <= (hd == 128 ? 2 : 3) || (of_64 == 4 && (of_128 >= 3 || (hd == 64 && !paired)));
}

template <int HD, bool PAIRED>
hipError_t launch_attn(const bf16_t* q, const bf16_t* k, const bf16_t* vt, bf16_t* o, int n_slices,
                       int n_tok, int n_keys, int n_q, int q_shared, int heads, long ld_qk, long ld_o,
                       unsigned char* oq, unsigned* so, long ld_so, int queries, const Ahead* ahead, hipStream_t st) {
  const bool mask = n_keys < n_tok || n_tok % BKEY != 0;
  if (queries == 16 || (queries == 0 && short_waves(n_slices, n_q, heads, HD, PAIRED)))
    return mask ? launch_attn_m<HD, 1, true, PAIRED>(q, k, vt, o, n_slices, n_tok, n_keys, n_q, q_shared, heads, ld_qk, ld_o, oq, so, ld_so, ahead, st)
                : launch_attn_m<HD, 1, false, PAIRED>(q, k, vt, o, n_slices, n_tok, n_keys, n_q, q_shared, heads, ld_qk, ld_o, oq, so, ld_so, ahead, st);
  return mask ? launch_attn_m<HD, 2, true, PAIRED>(q, k, vt, o, n_slices, n_tok, n_keys, n_q, q_shared, heads, ld_qk, ld_o, oq, so, ld_so, ahead, st)
              : launch_attn_m<HD, 2, false, PAIRED>(q, k, vt, o, n_slices, n_tok, n_keys, n_q, q_shared, heads, ld_qk, ld_o, oq, so, ld_so, ahead, st);
}

template <int HD, int QT, bool MASK, bool PAIRED>
hipError_t set_attr() {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(&k_attention_bf16<HD, QT, MASK, PAIRED>),
                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)AttnSmem<HD>::BYTES);
}
template <int HD>
hipError_t set_attr_hd() {
  hipError_t e = set_attr<HD, 1, false, false>();
  if (e == hipSuccess) e = set_attr<HD, 1, true, false>();
  if (e == hipSuccess) e = set_attr<HD, 2, false, false>();
  if (e == hipSuccess) e = set_attr<HD, 2, true, false>();
  if (e == hipSuccess) e = set_attr<HD, 1, false, true>();
  if (e == hipSuccess) e = set_attr<HD, 1, true, true>();
  if (e == hipSuccess) e = set_attr<HD, 2, false, true>();
  return e == hipSuccess ? set_attr<HD, 2, true, true>() : e;
}

}  // namespace

hipError_t bf16_attention_init() {
  hipError_t e = set_attr_hd<64>();
  if (e == hipSuccess) e = set_attr_hd<72>();
  if (e == hipSuccess) e = set_attr_hd<96>();
  return e == hipSuccess ? set_attr_hd<128>() : e;
}

int bf16_attention_queries(int n_slices, int n_q, int heads, int hd_pad, bool paired) {
  return short_waves(n_slices, n_q, heads, hd_pad, paired) ? 16 : 32;
}

hipError_t bf16_attention(const bf16_t* q, const bf16_t* k, const bf16_t* vt, bf16_t* o, int n_slices,
                          int n_tok, int n_keys, int n_q, int q_shared, int heads, int hd_pad, long ld_qk,
                          long ld_o, hipStream_t st, unsigned char* oq, unsigned* so, long ld_so, bool paired, int queries,
                          const Ahead* ahead) {
  if (n_slices == 0) return hipSuccess;
  // MXFP8 output: whole blocks of 32 per head only, rows of at least heads * hd_pad bytes, 4-byte pieces
  if (oq && (hd_pad % 32 != 0 || !so || ld_o % 4 != 0 || ld_o < (long)heads * hd_pad || ld_so < (long)n_slices * n_q)) return hipErrorInvalidValue;
  // n_tok % 8: V^T rows are read in 16-byte chunks.  A slice whose rows are no multiple of the key block is
  // read up to 63 rows (q, k) / 63 elements (v^T) past its end: the caller's buffers must reach that far.
  if (n_tok % 8 != 0 || n_tok <= 0 || n_keys < 1 || n_keys > n_tok || n_q < 1) return hipErrorInvalidValue;
  if (!q_shared && n_q != n_tok) return hipErrorInvalidValue;   // a slice's own rows: one query per row
#define LAUNCH(HD)                                                                                                       \
  return paired || oq ? launch_attn<HD, true>(q, k, vt, o, n_slices, n_tok, n_keys, n_q, q_shared, heads, ld_qk, ld_o, oq, so, ld_so, queries, ahead, st) \
                      : launch_attn<HD, false>(q, k, vt, o, n_slices, n_tok, n_keys, n_q, q_shared, heads, ld_qk, ld_o, oq, so, ld_so, queries, ahead, st)
  switch (hd_pad) {
    case 64: LAUNCH(64);
    case 72: LAUNCH(72);
    case 96: LAUNCH(96);
    case 128: LAUNCH(128);
  }
#undef LAUNCH
  return hipErrorInvalidValue;
}

}  // namespace epd
