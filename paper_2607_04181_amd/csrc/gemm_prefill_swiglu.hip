// Prefill gate/up projection (SwiGLU variants of gemm_prefill.h) and the
// tile shape choice of all prefill GEMMs.
#include "gemm_prefill.h"

namespace coco {

namespace prefill {

// Tile shape by an estimate of the time (us) of each shape that divides N:
//   rounds of workgroups x (K / 32 x step + epilogue), where a 32-k step of a
//   CU's n workgroups takes the longest of
//   * the loads' latency over the steps in flight, 0.4 us / ((SLOTS - 1) KS);
//   * its L2 -> LDS loads, n (TM + TN) 64 bytes at 65 GB/s per CU (the
//     loads-only ablation of the 256-row tiles runs at 54-60);
//   * its MFMAs, n TM TN / 64 cycles at an effective 1.47 GHz (the clock under
//     load times the MFMA pipe's share of a stage).
// The four constants are a least-squares fit to 2,100 timed launches (the 13
// shapes other than 192 x 256 and 160 x 256, x 15 row counts from 1 to 2,048 x
// the four projections of the 8B, 32B and 70B layers): 13% rms off the times,
// and the shape it picks takes on average 0.1%, at worst 6% longer than the
// best one. The two fill the gap between 128 and 256 rows, best of the others
// against them (us): 8B gate/up 300 rows 92 -> 80, 380 rows 97 -> 90, 760 rows
// 175 -> 162; 70B gate/up 160 rows 199 -> 183, 380 rows 364 -> 339. Against one 256-row
// shape for every M: 8B, 300 rows: QKV 69 -> 30 us, O 43 -> 24, down 124 ->
// 70; 32B, 512 rows, down 379 -> 212; 70B, 1,000 rows, O 187 -> 113 (256 x 256
// tiles before).
int choose_tile(int M, int N, int K, int S, int num_cus) {
  struct Shape {
    int tm, tn, steps, per_cu;  // steps in flight, workgroups per CU
  };
#define COCO_SHAPE(T, per_cu) {T::TM, T::TN, T::AHEAD * T::KS, per_cu}
  static constexpr Shape shapes[kTileCount] = {
      COCO_SHAPE(T256x224, 1), COCO_SHAPE(T256x192, 1), COCO_SHAPE(T256x160, 1),
      COCO_SHAPE(T256x128, 1), COCO_SHAPE(T192x256, 1), COCO_SHAPE(T160x256, 1),
      COCO_SHAPE(T128x256, 1), COCO_SHAPE(T128x160, 1), COCO_SHAPE(T128x128, 1),
      COCO_SHAPE(T128x64, 1),  COCO_SHAPE(T64x160, 1),  COCO_SHAPE(T64x128, 2),
      COCO_SHAPE(T64x64, 1),   COCO_SHAPE(T64x32, 1),   COCO_SHAPE(T32x32, 1)};
#undef COCO_SHAPE
  int best = -1;
  double best_us = 0.;
  for (int t = 0; t < kTileCount; ++t) {
    const Shape& s = shapes[t];
    if (N % s.tn != 0) continue;
    const int64_t wgs = (int64_t)((M + s.tm - 1) / s.tm) * (N / s.tn) * S;
    const int64_t round = (int64_t)num_cus * s.per_cu, rem = wgs % round;
    auto one = [&](int n) {  // a round with n workgroups per CU
      const double latency = 0.4 / s.steps;
      const double loads = n * (s.tm + s.tn) * 64e-3 / 65.;
      const double mfma = (double)n * s.tm * s.tn / (64e3 * 1.47);
      const double step = latency > loads ? latency : loads;
      return K / S / 32 * (step > mfma ? step : mfma) + 2.7 * n;
    };
    double us = (double)(wgs / round) * one(s.per_cu);
    if (rem != 0) us += one(rem <= num_cus ? 1 : s.per_cu);
    if (best < 0 || us < best_us) {
      best = t;
      best_us = us;
    }
  }
  return best;
}

}  // namespace prefill

hipError_t launch_prefill_swiglu_bf16(const uint16_t* A, const uint16_t* W_gate_up, uint16_t* H,
                                      int M, int F, int K, const float* ss_in, float eps,
                                      int num_cus, hipStream_t st) {
  if (M <= 0) return hipSuccess;
  if (!H || !ss_in) return hipErrorInvalidValue;
  PrefillEpiArgs ea{};
  ea.h = H;
  ea.ss_in = ss_in;
  ea.eps = eps;
  // Persistent when the row tiles divide the 32 workgroups of an XCD and a
  // tile is a whole number of unrolled rounds.
  using T = prefill::T256x192;
  const int tiles_m = (M + T::TM - 1) / T::TM;
  if (prefill::choose_tile(M, 2 * F, K, 1, num_cus) == prefill::k256x192 && num_cus == 256 &&
      32 % tiles_m == 0 && (K / 32) % T::ROUND == 0 && 2 * F % T::TN == 0) {
    COCO_LAUNCH((prefill::gemm_prefill_swiglu_persistent_kernel<T>), dim3(256), dim3(T::NT), 0, st,
                (const bf16_t*)A, (const bf16_t*)W_gate_up, M, F, K, (bf16_t*)H, ss_in, eps);
    return hipGetLastError();
  }
  return prefill::launch_mode<prefill::kSwiglu>(A, W_gate_up, M, 2 * F, K, 1, ea, num_cus, st);
}

hipError_t launch_prefill_swiglu_plain_bf16(const uint16_t* A, const uint16_t* W_gate_up,
                                            uint16_t* H, int M, int F, int K, bool h_tiled,
                                            int num_cus, hipStream_t st) {
  if (M <= 0) return hipSuccess;
  if (!H) return hipErrorInvalidValue;
  PrefillEpiArgs ea{};
  ea.h = H;
  ea.h_rows = !h_tiled;
  return prefill::launch_mode<prefill::kSwigluPlain>(A, W_gate_up, M, 2 * F, K, 1, ea, num_cus, st);
}

}  // namespace coco
