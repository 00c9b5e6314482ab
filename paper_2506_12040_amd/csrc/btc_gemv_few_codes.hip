// The decode engine for few activation rows (btc_gemv_few.h) on 8-bit codes.  Widening the codes, the product and the epilogue
// were launches of their own: 12 us per call with two rows on 1152 x 1152, 6 us here.
#include "btc_gemv_few.h"

namespace btc {

btc_status gemm_few_codes(hipStream_t q, const Dims& d, const uint32_t* packed, const uint32_t* codebook, const float* alpha,
                          const float* mu, const float* wsum, const uint8_t* Q, const float* lo, const float* step, int M,
                          void* Y, int y_dtype) {
  return few::run<few::kCodes>(q, d, packed, codebook, alpha, mu, Q, few::CodeArgs{wsum, lo, step}, M, Y, y_dtype);
}

}  // namespace btc
