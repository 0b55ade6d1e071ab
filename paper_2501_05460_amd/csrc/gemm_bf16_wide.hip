// The forms of the product on large tiles (gemm_bf16_wide.h), the plain bias, the transposed store and the patch embedding.
#include "gemm_bf16_wide.h"

namespace epd {

namespace {
template <int EPI>
hipError_t init() {
  const hipError_t e = set_attr_wide<EPI, false, 8, 4, 2, 4>();
  return e != hipSuccess ? e : set_attr_wide<EPI, false, 4, 4, 4, 2>();
}
template <int EPI>
hipError_t launch(const GemmParams& p, int tile, int cus, hipStream_t st) {
  switch (tile) {
    case WIDE_256: return launch_wide<EPI, false, 8, 4, 2, 4>(p, cus, st);
    case WIDE_128: return launch_wide<EPI, false, 4, 4, 4, 2>(p, cus, st);
  }
  return hipErrorInvalidValue;
}
}  // namespace

hipError_t bf16_gemm_wide_init() {
  hipError_t e = init<EPI_BIAS>();
  if (e == hipSuccess) e = init<EPI_BIAS_POS>();
  if (e == hipSuccess) e = init<EPI_VT>();
  if (e == hipSuccess) e = bf16_gemm_wide_gelu_init();
  if (e == hipSuccess) e = bf16_gemm_wide_residual_init();
  return e != hipSuccess ? e : bf16_gemm_wide_pair_init();
}

hipError_t bf16_gemm_wide(const GemmParams& p, int tile, int cus, hipStream_t st) {
  if (p.stats || p.xb) return hipErrorInvalidValue;   // neither a folded pre-norm nor the bf16 copy of the residual rows
  if (p.n2_pad > 0) return p.epi == EPI_BIAS ? bf16_gemm_wide_pair(p, tile, cus, st) : hipErrorInvalidValue;
  switch (p.epi) {
    case EPI_BIAS: return launch<EPI_BIAS>(p, tile, cus, st);
    case EPI_BIAS_GELU_ERF:
    case EPI_BIAS_GELU_TANH: return bf16_gemm_wide_gelu(p, tile, cus, st);
    case EPI_BIAS_RESIDUAL: return bf16_gemm_wide_residual(p, tile, cus, st);
    case EPI_BIAS_POS: return launch<EPI_BIAS_POS>(p, tile, cus, st);
    case EPI_VT: return launch<EPI_VT>(p, tile, cus, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace epd
