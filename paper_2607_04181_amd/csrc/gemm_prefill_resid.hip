// Prefill O projection (residual variant of gemm_prefill.h).
#include "gemm_prefill.h"

namespace coco {

hipError_t launch_prefill_resid_bf16(const uint16_t* A, const uint16_t* W, int M, int N, int K,
                                     const uint16_t* res_x, const int32_t* res_idx,
                                     const uint16_t* gamma, float* x1, uint16_t* h,
                                     float* ss_part, int num_cus, hipStream_t st) {
  if (M <= 0) return hipSuccess;
  if (!res_x || !gamma || !x1 || !h || !ss_part) return hipErrorInvalidValue;
  PrefillEpiArgs ea{};
  ea.res_x = res_x;
  ea.res_idx = res_idx;
  ea.gamma = gamma;
  ea.x1 = x1;
  ea.h = h;
  ea.ss_part = ss_part;
  return prefill::launch_mode<prefill::kResid>(A, W, M, N, K, 1, ea, num_cus, st);
}

}  // namespace coco
