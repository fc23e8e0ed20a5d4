// Weight-streaming GEMM for decode-sized row counts (bf16 MFMA, fp32 out).
//
//   part[s][m][n] = sum over k in K-slice s of A[m][k] * W[n][k]
//
// A: [M][K] activations, bf16. W: the [N][K] weights (nn.Linear layout) in
// tile order (pack_tile_order below): every 16 rows x 32 k of W are one
// contiguous 1 KB block laid out as the B operand of a
// v_mfma_f32_16x16x32_bf16 step, lane by lane.
// Decode is bound by reading W once from HBM, so the kernel is built around
// that stream:
//   * a workgroup of WAVES waves owns 16*WAVES output columns and one K-slice;
//     each wave streams the 16 weight rows of its columns straight into VGPRs
//     (each 16-byte-per-lane load one contiguous 1 KB block; plain loads
//     measured faster here than non-temporal ones), keeping two stages of
//     128 k in flight: ~56 KB per CU at 7 waves covers HBM latency, and deeper
//     rings measured slower (more requests queued behind each other);
//   * the activation tile [rows][128 k] of a stage is shared by the waves
//     through LDS (double-buffered); its 16-byte chunks are XOR-swizzled
//     with the row (chunk ^ row % 16), so both the row-wise stores and the
//     16-rows-per-instruction fragment reads hit distinct banks;
//   * each 16x16 output tile is accumulated with v_mfma_f32_16x16x32_bf16 in
//     ascending k.
// It covers up to 128 rows; larger batches, and the plans whose grid the tiles
// match, run the tile kernel of gemm_prefill.h on the same K-slices.
// The NORM variant (decode QKV projection) folds the row gather and the
// first RMSNorm into the activation staging: it reads the layer input rows
// x[row_idx[m]] directly, stages bf16(x * gamma), and writes each row's sum
// of x^2 over its K-slice; the 1/rms factor of a row is a scalar that the
// consumer applies to the summed partials.
// The plan (WAVES, split count S) is chosen from (N, K) alone (skinny_plan);
// every output element is
// summed in the same k order for any M, so a row's result does not depend on
// the other rows in the call (batch invariance). Partials of the S slices
// are added in slice order by the consumer epilogue.
#include <math.h>

#include "common.h"
#include "kernels.h"

namespace coco {

namespace {

constexpr int kBK = 128;       // k per pipeline stage
constexpr int kCUs = 256;

// LDS element offset of 16-byte chunk c (0..15) of activation row r.
__device__ __forceinline__ int a_swz(int r, int c) { return r * kBK + ((c ^ (r & 15)) << 3); }

// t plus the squares of eight packed elements, in order.
__device__ __forceinline__ float sum_squares8(u32x4_t u, float t) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float lo = __uint_as_float(u[e] << 16), hi = __uint_as_float(u[e] & 0xFFFF0000u);
    t = fmaf(lo, lo, t);
    t = fmaf(hi, hi, t);
  }
  return t;
}

// NORM row sums, by one wave: ss[blockIdx.y][r] = sum of x^2 over the K-slice
// for rows r = r_first, r_first + gridDim.x, ... below r_end (each row by one
// workgroup of the slice), per lane in chunk order, then a fixed
// butterfly: a row's sum never depends on the batch.
__device__ __forceinline__ void norm_row_sums(const bf16_t* __restrict__ A,
                                              const int32_t* __restrict__ row_idx, int M, int K,
                                              int k_begin, int k_slice, int r_first, int r_end,
                                              float* __restrict__ ss, int lane) {
  for (int r = r_first; r < r_end; r += gridDim.x) {
    const bf16_t* xr = A + (int64_t)((row_idx != nullptr) ? row_idx[r] : r) * K + k_begin;
    float t = 0.f;
    for (int c = lane; c < k_slice / 8; c += 64) {
      t = sum_squares8(*(const u32x4_t*)(xr + c * 8), t);
    }
    t = wave_sum(t);
    if (lane == 0) ss[(int64_t)blockIdx.y * M + r] = t;
  }
}

// bf16(x * gamma) of eight packed elements, the product in fp32.
__device__ __forceinline__ u32x4_t scale_bf16x8(u32x4_t x, u32x4_t g) {
  u32x4_t y;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float lo = __uint_as_float(x[e] << 16), hi = __uint_as_float(x[e] & 0xFFFF0000u);
    const float glo = __uint_as_float(g[e] << 16), ghi = __uint_as_float(g[e] & 0xFFFF0000u);
    y[e] = pack_bf16x2(lo * glo, hi * ghi);
  }
  return y;
}

// The NORM variant's staging as a kernel of its own, for batches whose QKV
// projection runs on the tile kernel: wave s of row i's workgroup writes K-slice
// s of bf16(x * gamma) in tile order and the slice's sum of squares, both with
// the arithmetic and order of the folded form.
__global__ void gather_scale_kernel(const bf16_t* __restrict__ x,
                                    const int32_t* __restrict__ row_idx, int M, int K,
                                    const bf16_t* __restrict__ gamma, bf16_t* __restrict__ h,
                                    float* __restrict__ ss) {
  // Consecutive rows on one XCD (blockIdx % 8): the 16 rows of a tile-order
  // block fill it in that XCD's L2.
  constexpr int kXCDs = 8;
  const int nb = gridDim.x, b = blockIdx.x, full = (nb / kXCDs) * kXCDs;
  const int i = b < full ? (b % kXCDs) * (nb / kXCDs) + b / kXCDs : b;
  const int lane = threadIdx.x & 63, s = threadIdx.x >> 6, S = blockDim.x >> 6;
  const int k_slice = K / S, k_begin = s * k_slice;
  const bf16_t* xr = x + (int64_t)(row_idx != nullptr ? row_idx[i] : i) * K + k_begin;
  float t = 0.f;
  for (int c = lane; c < k_slice / 8; c += 64) {
    const u32x4_t u = *(const u32x4_t*)(xr + c * 8);
    const u32x4_t g = *(const u32x4_t*)(gamma + k_begin + c * 8);
    t = sum_squares8(u, t);
    *(u32x4_t*)(h + tile_off(i, k_begin + c * 8, K)) = scale_bf16x8(u, g);
  }
  t = wave_sum(t);
  if (lane == 0) ss[(int64_t)s * M + i] = t;
}

// FUSE: W is the [2F][K] gate/up matrix (N = 2F, one K-slice), interleaved
// (launch_pack_gate_up): lanes c16 < 8 of a wave stream gate rows o0..o0+7 and
// lanes c16 >= 8 the matching up rows, so the epilogue pairs lanes c16 and
// c16+8 and writes h = silu(gate) * up in bf16 to H[M][F] instead of fp32
// partials.
// NORM: A holds the layer input rows, row m of the call at A[row_idx[m]]
// (row_idx null: row m); the staged operand is bf16(A * gamma) and
// ss[blockIdx.y][m] receives the row's sum of squares over the K-slice
// (row m by the workgroup of the slice with blockIdx.x == m % gridDim.x).
template <int WAVES, int MT, bool FUSE, bool NORM>
__global__ __launch_bounds__(WAVES * 64) void gemm_skinny_kernel(
    const bf16_t* __restrict__ A, const bf16_t* __restrict__ W, float* __restrict__ part,
    bf16_t* __restrict__ H, int M, int N, int K, int k_slice,
    const int32_t* __restrict__ row_idx, const bf16_t* __restrict__ gamma,
    float* __restrict__ ss, bool h_tiled) {
  constexpr int NT = WAVES * 64;
  constexpr int PF = 2;  // weight stages in flight
  constexpr int kChunks = MT * 16 * (kBK / 8);  // 16-byte A chunks per stage
  constexpr int kPerT = (kChunks + NT - 1) / NT;
  __shared__ __attribute__((aligned(16))) bf16_t lds[2][MT * 16 * kBK];

  const int tid = threadIdx.x;
  const int lane = tid & 63, wv = tid >> 6;
  const int c16 = lane & 15, j4 = lane >> 4;
  const int o0 = (blockIdx.x * WAVES + wv) * 8;  // fused: this wave's 8 outputs
  const int n_col = blockIdx.x * (16 * WAVES) + wv * 16 + c16;  // this lane's weight row
  const int k_begin = blockIdx.y * k_slice;
  const int stages = k_slice / kBK;
  float* out = FUSE ? nullptr : part + (int64_t)blockIdx.y * M * N;

  // This lane's chunk of the stage's step t (row n_col, k = k_begin + 128 st +
  // 32 t + 8 j4) in tile order: block (n_col / 16) * (K / 32) + k / 32, chunk
  // j4 * 16 + n_col % 16; a wave's load of one step is one 1 KB block.
  const bf16_t* wrow =
      W + ((int64_t)(n_col >> 4) * (K / 32) + k_begin / 32) * 512 + (j4 * 16 + (n_col & 15)) * 8;

  // The steady-state loop is branch-free so that the compiler can wait for
  // exactly the loads each step consumes: prefetches past the slice are
  // clamped to its last stage (an L2 hit, never used), and stages past the
  // slice in the final group get a zero activation tile (adding exact zeros
  // leaves every sum unchanged).
  const int groups = (stages + PF - 1) / PF;
  f32x4_t acc[MT];
#pragma unroll
  for (int t = 0; t < MT; ++t) acc[t] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  // Weight ring: PF stages x 4 k-steps of 8 bf16 per lane.
  u32x4_t wreg[PF][4];
  auto load_w = [&](int st, int u) {
    const bf16_t* src = wrow + min(st, stages - 1) * (kBK / 32) * 512;
#pragma unroll
    for (int t = 0; t < 4; ++t) wreg[u][t] = *(const u32x4_t*)(src + t * 512);
  };
#pragma unroll
  for (int u = 0; u < PF; ++u) load_w(u, u);

  // Activation ring: stage x lives in register slot x % 2 from the start of
  // stage x-2 until it is copied to LDS buffer x % 2 at the end of stage
  // x-1, so its L2 latency is hidden behind two stages of weight streaming.
  // A thread stages the same (row, 16-byte chunk column) of every stage:
  // rows (tid + v * NT) / 16 and chunk column tid % 16 (NT is a multiple of
  // 16), so under NORM it needs one gain chunk per stage and keeps one sum
  // of squares per row it stages.
  u32x4_t areg[2][kPerT];
  u32x4_t greg[2];
  int arow[kPerT];  // source row of each staged chunk (32-bit to spare registers)
#pragma unroll
  for (int v = 0; v < kPerT; ++v) {
    const int q = min(tid + v * NT, kChunks - 1);
    const int m = min(q >> 4, M - 1);
    arow[v] = (NORM && row_idx) ? row_idx[m] : m;
  }
  const bf16_t* a_col = A + k_begin + (tid & 15) * 8;  // NT % 16 == 0: column tid % 16
  auto load_a = [&](int st, int slot) {
    const int sc = min(st, stages - 1);
#pragma unroll
    for (int v = 0; v < kPerT; ++v)
      areg[slot][v] = *(const u32x4_t*)(a_col + (int64_t)arow[v] * K + sc * kBK);
    if (NORM) greg[slot] = *(const u32x4_t*)(gamma + k_begin + sc * kBK + (tid & 15) * 8);
  };
  auto store_a = [&](int st, int slot, int buf) {
#pragma unroll
    for (int v = 0; v < kPerT; ++v) {
      const int q = tid + v * NT;
      const bool live = st < stages && (q >> 4) < M;
      u32x4_t val = live ? areg[slot][v] : u32x4_t{0u, 0u, 0u, 0u};
      if (NORM) val = scale_bf16x8(val, greg[slot]);  // x * gamma in fp32, rounded to bf16
      if (q < kChunks) *(u32x4_t*)(&lds[buf][a_swz(q >> 4, q & 15)]) = val;
    }
  };

  load_a(0, 0);
  load_a(1, 1);
  // Row sums of squares while the first weight stages are in flight.
  if (NORM && wv == 0)
    norm_row_sums(A, row_idx, M, K, k_begin, k_slice, blockIdx.x, M, ss, lane);
  store_a(0, 0, 0);
  __syncthreads();

  static_assert(PF % 2 == 0, "ring slots are indexed by stage parity");
  for (int g = 0; g < groups; ++g) {
#pragma unroll
    for (int u = 0; u < PF; ++u) {
      const int st = g * PF + u;
      const int buf = u & 1;  // == st & 1 since PF is even
      load_a(st + 2, u & 1);
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const bf16x8_t b = __builtin_bit_cast(bf16x8_t, wreg[u][t]);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
          const bf16x8_t a = __builtin_bit_cast(
              bf16x8_t, *(const u32x4_t*)(&lds[buf][a_swz(mt * 16 + c16, t * 4 + j4)]));
          acc[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc[mt], 0, 0, 0);
        }
      }
      load_w(st + PF, u);
      store_a(st + 1, (u + 1) & 1, buf ^ 1);
      __syncthreads();
    }
  }

  // D layout: lane holds rows 4*j4 + r of column c16 of each 16x16 tile.
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = mt * 16 + j4 * 4 + r;
      if (FUSE) {
        // The up value of this lane's output sits 8 lanes up.
        const float u = __shfl_down(acc[mt][r], 8, 16);
        const float g = acc[mt][r];
        if (c16 < 8 && m < M)
          H[h_tiled ? tile_off(m, o0 + c16, N / 2) : (int64_t)m * (N / 2) + o0 + c16] =
              (bf16_t)f32_to_bf16(silu_mul(g, u));
      } else if (m < M) {
        // Non-temporal: the partials are read once, by the next kernel.
        __builtin_nontemporal_store(acc[mt][r], out + (int64_t)m * N + n_col);
      }
    }
  }
}

struct NormArgs {
  const int32_t* row_idx = nullptr;
  const uint16_t* gamma = nullptr;
  float* ss = nullptr;
};

template <int WAVES, int MT, bool FUSE, bool NORM>
hipError_t launch_plan(const uint16_t* A, const uint16_t* W, float* part, uint16_t* H, int M,
                       int N, int K, int S, NormArgs na, bool h_tiled, hipStream_t st) {
  if (M > MT * 16) return hipErrorInvalidValue;
  COCO_LAUNCH((gemm_skinny_kernel<WAVES, MT, FUSE, NORM>), dim3(N / (16 * WAVES), S),
                     dim3(WAVES * 64), 0, st, A, W, part, H, M, N, K, K / S, na.row_idx,
                     (const bf16_t*)na.gamma, na.ss, h_tiled);
  return hipGetLastError();
}

template <int WAVES, bool FUSE, bool NORM>
hipError_t launch_waves(const uint16_t* A, const uint16_t* W, float* part, uint16_t* H, int M,
                        int N, int K, int S, NormArgs na, bool h_tiled, hipStream_t st) {
  if (M <= 64)
    return launch_plan<WAVES, 4, FUSE, NORM>(A, W, part, H, M, N, K, S, na, h_tiled, st);
  return launch_plan<WAVES, 8, FUSE, NORM>(A, W, part, H, M, N, K, S, na, h_tiled, st);
}

template <bool FUSE, bool NORM>
hipError_t launch_any(const uint16_t* A, const uint16_t* W, float* part, uint16_t* H, int M,
                      int N, int K, SkinnyPlan plan, NormArgs na, bool h_tiled,
                      hipStream_t st) {
  switch (plan.waves) {
    case 4: return launch_waves<4, FUSE, NORM>(A, W, part, H, M, N, K, plan.S, na, h_tiled, st);
    case 5: return launch_waves<5, FUSE, NORM>(A, W, part, H, M, N, K, plan.S, na, h_tiled, st);
    case 6: return launch_waves<6, FUSE, NORM>(A, W, part, H, M, N, K, plan.S, na, h_tiled, st);
    case 7: return launch_waves<7, FUSE, NORM>(A, W, part, H, M, N, K, plan.S, na, h_tiled, st);
    default: return launch_waves<8, FUSE, NORM>(A, W, part, H, M, N, K, plan.S, na, h_tiled, st);
  }
}

}  // namespace

// Grid plan from (N, K) only (so a row's sums never depend on the batch).
// Measured on the decode shapes: the best plans fill the 256 CUs with exactly
// one round of workgroups; among those, K-slices of at least 1024 (eight
// stages) and then more waves per workgroup win. Without such a plan, the
// unsplit weight stream wins (split-K partials and short slices cost more),
// with the fullest last round of workgroups and then the most waves: on the
// 70B gate/up shape (N = 57344, K = 8192, 128 rows) 7 waves (two full rounds)
// took 206 us against 220 us for 8 waves (448 workgroups). The wave count
// does not change any output's k order.
SkinnyPlan skinny_plan(int N, int K) {
  auto valid = [&](int waves, int S) {
    if (N % (16 * waves)) return false;
    if (K % (S * kBK)) return false;
    if (S > 1 && K / S < 4 * kBK) return false;
    return true;
  };
  SkinnyPlan best{0, 0};
  int best_rank = -1;
  for (int waves = 4; waves <= 8; ++waves)
    for (int S = 1; S <= 16; S *= 2) {
      if (!valid(waves, S)) continue;
      const int wgs = (N / (16 * waves)) * S;
      if (wgs != kCUs) continue;
      const int rank = (K / S >= 8 * kBK ? 100 : 0) + waves * 2 + (S == 1 ? 1 : 0);
      if (rank > best_rank) {
        best_rank = rank;
        best = SkinnyPlan{waves, S};
      }
    }
  if (best.waves) return best;
  int64_t best_fill = -1;  // workgroups * 2^16 / (rounds * 256): last-round fill
  for (int waves = 8; waves >= 4; --waves) {
    if (!valid(waves, 1)) continue;
    const int64_t wgs = N / (16 * waves);
    const int64_t rounds = (wgs + kCUs - 1) / kCUs;
    const int64_t fill = (wgs << 16) / (rounds * kCUs);
    if (fill > best_fill) {
      best_fill = fill;
      best = SkinnyPlan{waves, 1};
    }
  }
  return best;  // {0, 0}: no plan (N not a multiple of 64 or K of 128)
}

hipError_t launch_gemm_skinny_bf16(const uint16_t* A, const uint16_t* W, float* part, int M,
                                   int N, int K, SkinnyPlan plan, hipStream_t st) {
  if (M <= 0) return hipSuccess;
  if (plan.waves < 4 || plan.waves > 8 || N % (16 * plan.waves) != 0 ||
      K % (plan.S * kBK) != 0)
    return hipErrorInvalidValue;
  return launch_any<false, false>(A, W, part, nullptr, M, N, K, plan, NormArgs{}, false, st);
}

hipError_t launch_gather_scale_bf16(const uint16_t* src, const int32_t* row_idx, int M, int d,
                                    const uint16_t* gamma, uint16_t* h_out, float* ss, int S,
                                    hipStream_t st) {
  if (M <= 0) return hipSuccess;
  if (S < 1 || S > 16 || d % (128 * S) != 0) return hipErrorInvalidValue;
  COCO_LAUNCH(gather_scale_kernel, dim3(M), dim3(64 * S), 0, st, src, row_idx, M, d, gamma, h_out,
              ss);
  return hipGetLastError();
}

hipError_t launch_gemm_skinny_norm_bf16(const uint16_t* X, const int32_t* row_idx,
                                        const uint16_t* gamma, const uint16_t* W, float* part,
                                        float* ss, int M, int N, int K, SkinnyPlan plan,
                                        hipStream_t st) {
  if (M <= 0) return hipSuccess;
  if (plan.waves < 4 || plan.waves > 8 || N % (16 * plan.waves) != 0 ||
      K % (plan.S * kBK) != 0)
    return hipErrorInvalidValue;
  NormArgs na;
  na.row_idx = row_idx;
  na.gamma = gamma;
  na.ss = ss;
  return launch_any<false, true>(X, W, part, nullptr, M, N, K, plan, na, false, st);
}

hipError_t launch_gemm_skinny_swiglu_bf16(const uint16_t* A, const uint16_t* W_gate_up,
                                          uint16_t* H, int M, int F, int K, SkinnyPlan plan,
                                          bool h_tiled, hipStream_t st) {
  if (M <= 0) return hipSuccess;
  if (plan.S != 1 || plan.waves < 4 || plan.waves > 8 || (2 * F) % (16 * plan.waves) != 0 ||
      K % kBK != 0)
    return hipErrorInvalidValue;
  return launch_any<true, false>(A, W_gate_up, nullptr, H, M, 2 * F, K, plan, NormArgs{},
                                 h_tiled, st);
}

// ----------------------------------------------------------------------------
// Tile order of a bf16 weight matrix [N][K] (N % 16 == 0, K % 32 == 0): the
// 1 KB block b = (n / 16) * (K / 32) + k / 32 holds rows 16 (n / 16) .. + 15
// and columns 32 (k / 32) .. + 31 as 64 chunks of 8 consecutive k, chunk
// ((k % 32) / 8) * 16 + n % 16 -- lane j4 * 16 + c16 of the B operand of a
// v_mfma_f32_16x16x32_bf16 step (row c16, k 8 j4 .. + 7). One thread per
// 16-byte chunk, in the order of the packed rows.
// ----------------------------------------------------------------------------
namespace {
// F > 0: rows interleaved as launch_pack_gate_up says (N = 2F). Threads go by
// packed row, so that the rows of a block are written side by side in time
// whatever their order in w (by row of w, gate and up halves of a block apart,
// coco_layer_init of a 32B layer took 1.08 ms against 1.03).
__global__ __launch_bounds__(256) void pack_tile_order_kernel(const u32x4_t* __restrict__ w,
                                                              int64_t n_chunks, int K, int F,
                                                              u32x4_t* __restrict__ out) {
  const int64_t chunk = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (chunk >= n_chunks) return;
  const int64_t per_row = K / 8;
  const int64_t n = chunk / per_row, kc = chunk - n * per_row;
  const int64_t row = F > 0 ? (n >> 4) * 8 + (n & 7) + (n & 8 ? F : 0) : n;
  out[((n >> 4) * (K / 32) + (kc >> 2)) * 64 + (kc & 3) * 16 + (n & 15)] = w[row * per_row + kc];
}

hipError_t pack(const uint16_t* W, int64_t N, int K, int F, uint16_t* out, hipStream_t st) {
  const int64_t n_chunks = N * K / 8;
  COCO_LAUNCH(pack_tile_order_kernel, dim3((unsigned)((n_chunks + 255) / 256)), dim3(256), 0, st,
              (const u32x4_t*)W, n_chunks, K, F, (u32x4_t*)out);
  return hipGetLastError();
}
}  // namespace

hipError_t launch_pack_tile_order(const uint16_t* W, int N, int K, uint16_t* out,
                                  hipStream_t st) {
  if (N <= 0 || K <= 0 || N % 16 != 0 || K % 32 != 0) return hipErrorInvalidValue;
  return pack(W, N, K, 0, out, st);
}

hipError_t launch_pack_gate_up(const uint16_t* W, int F, int K, uint16_t* out, hipStream_t st) {
  if (F <= 0 || K <= 0 || F % 8 != 0 || K % 32 != 0) return hipErrorInvalidValue;
  return pack(W, 2LL * F, K, F, out, st);
}

}  // namespace coco
