// Decode projections of large batches (partial variant of gemm_prefill.h).
#include "gemm_prefill.h"

namespace coco {

hipError_t launch_tile_partial_bf16(const uint16_t* A, const uint16_t* W, float* part, int M,
                                    int N, int K, int S, int num_cus, hipStream_t st) {
  if (M <= 0) return hipSuccess;
  if (!part) return hipErrorInvalidValue;
  PrefillEpiArgs ea{};
  ea.x1 = part;
  return prefill::launch_mode<prefill::kPartial>(A, W, M, N, K, S, ea, num_cus, st);
}

}  // namespace coco
