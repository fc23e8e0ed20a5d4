// Prefill QKV projection (QKV variant of gemm_prefill.h).
#include "gemm_prefill.h"

namespace coco {

hipError_t launch_prefill_qkv_bf16(const uint16_t* A, const uint16_t* W_qkv, int M, int K,
                                   const PrefillEpiArgs& ea, int num_cus, hipStream_t st) {
  if (M <= 0) return hipSuccess;
  if (!ea.row_info || !ea.rope || !ea.q_out || !ea.k_cache || !ea.v_cache)
    return hipErrorInvalidValue;
  return prefill::launch_mode<prefill::kQkv>(A, W_qkv, M, (ea.Hq + 2 * ea.Hkv) * 128, K, 1,
                                             ea, num_cus, st);
}

}  // namespace coco
