// The forms of the product on large tiles (gemm_bf16_wide.h), two products over the same activations: q/k and value projection.
#include "gemm_bf16_wide.h"

namespace epd {

hipError_t bf16_gemm_wide_pair_init() {
  hipError_t e = set_attr_wide<EPI_BIAS, true, 8, 4, 2, 4>();
  if (e == hipSuccess) e = set_attr_wide<EPI_BIAS, true, 7, 4, 2, 4>();
  if (e == hipSuccess) e = set_attr_wide<EPI_BIAS, true, 4, 6, 4, 2>();
  return e != hipSuccess ? e : bf16_gemm_wide_pair_low_init();
}

hipError_t bf16_gemm_wide_pair(const GemmParams& p, int tile, int cus, hipStream_t st) {
  switch (tile) {
    case WIDE_256: return launch_wide<EPI_BIAS, true, 8, 4, 2, 4>(p, cus, st);
    case WIDE_224: return launch_wide<EPI_BIAS, true, 7, 4, 2, 4>(p, cus, st);
    case WIDE_192_ROWS:
    case WIDE_160_ROWS: return bf16_gemm_wide_pair_low(p, tile, cus, st);
    case WIDE_192: return launch_wide<EPI_BIAS, true, 4, 6, 4, 2>(p, cus, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace epd
