// The forms of the product on large tiles (gemm_bf16_wide.h), the epilogues with an activation.
#include "gemm_bf16_wide.h"

namespace epd {

namespace {
template <int EPI>
hipError_t init() {
  hipError_t e = set_attr_wide<EPI, false, 8, 4, 2, 4>();
  if (e == hipSuccess) e = set_attr_wide<EPI, false, 7, 4, 2, 4>();
  return e != hipSuccess ? e : set_attr_wide<EPI, false, 4, 4, 4, 2>();
}
template <int EPI>
hipError_t launch(const GemmParams& p, int tile, int cus, hipStream_t st) {
  switch (tile) {
    case WIDE_256: return launch_wide<EPI, false, 8, 4, 2, 4>(p, cus, st);
    case WIDE_224: return launch_wide<EPI, false, 7, 4, 2, 4>(p, cus, st);
    case WIDE_128: return launch_wide<EPI, false, 4, 4, 4, 2>(p, cus, st);
  }
  return hipErrorInvalidValue;
}
}  // namespace

hipError_t bf16_gemm_wide_gelu_init() {
  const hipError_t e = init<EPI_BIAS_GELU_ERF>();
  return e != hipSuccess ? e : init<EPI_BIAS_GELU_TANH>();
}

hipError_t bf16_gemm_wide_gelu(const GemmParams& p, int tile, int cus, hipStream_t st) {
  return p.epi == EPI_BIAS_GELU_ERF ? launch<EPI_BIAS_GELU_ERF>(p, tile, cus, st) : launch<EPI_BIAS_GELU_TANH>(p, tile, cus, st);
}

}  // namespace epd
