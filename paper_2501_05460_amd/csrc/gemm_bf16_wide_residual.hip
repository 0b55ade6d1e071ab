// The forms of the product on large tiles (gemm_bf16_wide.h), the residual epilogue.
#include "gemm_bf16_wide.h"

namespace epd {

hipError_t bf16_gemm_wide_residual_init() {
  hipError_t e = set_attr_wide<EPI_BIAS_RESIDUAL, false, 8, 4, 2, 4>();
  if (e == hipSuccess) e = set_attr_wide<EPI_BIAS_RESIDUAL, false, 7, 4, 2, 4>();
  if (e == hipSuccess) e = set_attr_wide<EPI_BIAS_RESIDUAL, false, 4, 6, 4, 2>();
  return e != hipSuccess ? e : set_attr_wide<EPI_BIAS_RESIDUAL, false, 4, 4, 4, 2>();
}

hipError_t bf16_gemm_wide_residual(const GemmParams& p, int tile, int cus, hipStream_t st) {
  switch (tile) {
    case WIDE_256: return launch_wide<EPI_BIAS_RESIDUAL, false, 8, 4, 2, 4>(p, cus, st);
    case WIDE_224: return launch_wide<EPI_BIAS_RESIDUAL, false, 7, 4, 2, 4>(p, cus, st);
    case WIDE_192: return launch_wide<EPI_BIAS_RESIDUAL, false, 4, 6, 4, 2>(p, cus, st);
    case WIDE_128: return launch_wide<EPI_BIAS_RESIDUAL, false, 4, 4, 4, 2>(p, cus, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace epd
