// The forms of the product on large tiles (gemm_bf16_wide.h), two products over the same activations on tiles of 192 and 160 rows.
#include "gemm_bf16_wide.h"

namespace epd {

hipError_t bf16_gemm_wide_pair_low_init() {
  const hipError_t e = set_attr_wide<EPI_BIAS, true, 6, 4, 2, 4>();
  return e != hipSuccess ? e : set_attr_wide<EPI_BIAS, true, 5, 4, 2, 4>();
}

hipError_t bf16_gemm_wide_pair_low(const GemmParams& p, int tile, int cus, hipStream_t st) {
  switch (tile) {
    case WIDE_192_ROWS: return launch_wide<EPI_BIAS, true, 6, 4, 2, 4>(p, cus, st);
    case WIDE_160_ROWS: return launch_wide<EPI_BIAS, true, 5, 4, 2, 4>(p, cus, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace epd
