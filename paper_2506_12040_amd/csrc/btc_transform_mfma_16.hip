// btc_transform for several rows, n2 a multiple of 16.
#define BTC_TRANSFORM_ALIGN
#include "btc_transform_mfma.h"

namespace btc {
namespace transform {

btc_status mfma_16(hipStream_t q, const void* X, int is_bf16, int M, int n1, int n2, const uint32_t* sign_bits, const float* P1,
                   const float* P2, void* Y, int y_dtype) {
  return run_mfma<16>(q, X, is_bf16, M, n1, n2, sign_bits, P1, P2, Y, y_dtype);
}

}  // namespace transform
}  // namespace btc
