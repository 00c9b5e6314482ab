// The decode engine for few activation rows (btc_gemv_few.h) on fp16 and bf16 activations.
#include "btc_gemv_few.h"

namespace btc {

bool gemv_few_covers(const Dims& d, int batch) {
  return batch >= 1 && batch <= 16 && (d.v == 9 || d.v == 10) && d.b >= 7 && d.b <= 10 &&
         (long long)d.out * d.wpr * 4 < (1LL << 31) && (long long)batch * d.in * 2 < (1LL << 31) - 4;
}

double gemv_few_estimate_us(const Dims& d, int batch) { return few::make_plan(d, batch).us; }

btc_status gemv_few(hipStream_t q, const Dims& d, const uint32_t* packed, const uint32_t* codebook, const float* alpha,
                    const float* mu, const void* x, int is_bf16, int batch, void* y, int y_dtype) {
  if (is_bf16) return few::run<few::kBf16>(q, d, packed, codebook, alpha, mu, x, few::CodeArgs{}, batch, y, y_dtype);
  return few::run<few::kF16>(q, d, packed, codebook, alpha, mu, x, few::CodeArgs{}, batch, y, y_dtype);
}

}  // namespace btc
