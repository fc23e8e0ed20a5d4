// Prefill down projection (scatter variant of gemm_prefill.h).
#include "gemm_prefill.h"

namespace coco {

hipError_t launch_prefill_scatter_bf16(const uint16_t* A, const uint16_t* W, int M, int N, int K,
                                       const float* x1, uint16_t* out, const int32_t* out_idx,
                                       int num_cus, hipStream_t st) {
  if (M <= 0) return hipSuccess;
  if (!x1 || !out) return hipErrorInvalidValue;
  PrefillEpiArgs ea{};
  ea.x1_in = x1;
  ea.out = out;
  ea.out_idx = out_idx;
  return prefill::launch_mode<prefill::kScatter>(A, W, M, N, K, 1, ea, num_cus, st);
}

}  // namespace coco
