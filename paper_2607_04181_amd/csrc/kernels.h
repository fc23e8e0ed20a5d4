// Host-side launchers of the gfx950 kernels (internal to libcoco).
#pragma once

#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace coco {

// Per-kernel timing (benchmark mode): events that the next kernel launch of
// this thread passes to hipExtLaunchKernelGGL, which timestamps them at the
// kernel's own start and end, then clears. Null events: a plain launch.
struct LaunchEvents {
  hipEvent_t start = nullptr, stop = nullptr;
};
LaunchEvents& launch_events();

#define COCO_LAUNCH(kernel, grid, block, shmem, stream, ...)                                  \
  do {                                                                                        \
    ::coco::LaunchEvents& le_ = ::coco::launch_events();                                      \
    hipExtLaunchKernelGGL(kernel, grid, block, shmem, stream, le_.start, le_.stop, 0,         \
                          __VA_ARGS__);                                                       \
    le_ = ::coco::LaunchEvents{};                                                             \
  } while (0)

// ---------------------------------------------------------------- row kernels
// Prefill row slots (optional output of the gather kernel): row_info[2i] =
// positions[i] clamped to [0, rope_rows), row_info[2i + 1] = the cache block
// of that position in row i's sequence (rows of a sequence contiguous).
struct RowSlotArgs {
  const int32_t* positions = nullptr;
  const int32_t* seq_starts = nullptr;
  const int32_t* block_table = nullptr;
  int32_t* row_info = nullptr;  // null: not written
  int n_seqs = 0, max_blocks = 0, rope_rows = 0;
};

// h_out[i] = RMSNorm(src[row_idx ? row_idx[i] : i]) * gamma, in tile order
// (tile_off), the prefill GEMM's A operand layout; and the rows' slots.
hipError_t launch_gather_rmsnorm_bf16(const uint16_t* src, const int32_t* row_idx, int M, int d,
                                      const uint16_t* gamma, float eps, uint16_t* h_out,
                                      const RowSlotArgs& rs, hipStream_t st);

// Decode batches whose QKV projection runs on the tile kernel: h_out[i] =
// bf16(x * gamma) of row src[row_idx ? row_idx[i] : i] in tile order, and
// ss[s][i] = the row's sum of squares over K-slice s, with the bits of
// launch_gemm_skinny_norm_bf16.
hipError_t launch_gather_scale_bf16(const uint16_t* src, const int32_t* row_idx, int M, int d,
                                    const uint16_t* gamma, uint16_t* h_out, float* ss, int S,
                                    hipStream_t st);

// RoPE table rope[p][j] = (cos, sin)(p * inv_freq[j]) for p < n_pos and
// j < half, angle and both functions in fp64 (as the QKV epilogue computes
// them), stored as fp32 pairs.
hipError_t launch_rope_table(const double* inv_freq, int half, int n_pos, float* rope,
                             hipStream_t st);

// Decode: sum of S split-K partials of the QKV projection, each row's sums
// scaled by 1 / sqrt(sum_s ss[s][row] / d + eps) (RMSNorm_1, folded into the
// projection), RoPE on query and key heads, queries to q_out [M][Hq*hd],
// keys/values into the paged cache. One workgroup also writes the decode
// attention's work list split_off (layout at launch_attn_decode_bf16) from the
// keys each row attends, min(ctx_lens, positions + 1) (partition counts capped
// at max_splits).
hipError_t launch_qkv_epilogue_bf16(const float* part, int S, int M, int Hq, int Hkv, int hd,
                                    const int32_t* positions, const int32_t* block_table,
                                    int max_blocks, const double* inv_freq, uint16_t* q_out,
                                    uint16_t* k_cache, uint16_t* v_cache,
                                    const int32_t* ctx_lens, int32_t* split_off, int max_splits,
                                    const float* ss, int d, float eps, hipStream_t st);

// x1 = x + sum_s part[s]  (fp32);  h2 = RMSNorm(x1) * gamma. Row i of x is
// x[row_idx ? row_idx[i] : i]. tiled: h2 in tile order.
hipError_t launch_residual_rmsnorm_bf16(const float* part, int S, int M, int d,
                                        const uint16_t* x, const int32_t* row_idx,
                                        const uint16_t* gamma, float eps, float* x1,
                                        uint16_t* h2, bool tiled, hipStream_t st);

// u = silu(sum_s gate) * sum_s up, part rows [2F] in the interleaved order of
// launch_pack_gate_up. tiled: u in tile order.
hipError_t launch_swiglu_bf16(const float* part, int S, int M, int F, uint16_t* u, bool tiled,
                              hipStream_t st);

// dst[m][k] (row-major, at most dst_elems elements) = src (tile order, [M][K]).
hipError_t launch_untile(const uint16_t* src, int M, int K, uint16_t* dst, int64_t dst_elems,
                         hipStream_t st);

// y = x1 + sum_s part[s];  out[row_idx ? row_idx[i] : i] = y.
hipError_t launch_residual_scatter_bf16(const float* part, int S, int M, int d, const float* x1,
                                        uint16_t* out, const int32_t* row_idx, hipStream_t st);

// Bit copy of [n][Hkv][hd] keys/values into the paged cache.
template <typename T>
hipError_t launch_kv_append(const T* k, const T* v, const int32_t* seq_idx,
                            const int32_t* positions, int n, int Hkv, int hd,
                            const int32_t* block_table, int max_blocks, T* k_cache,
                            T* v_cache, hipStream_t st);

// ---------------------------------------------------------------- GEMMs
// Every bf16 GEMM below reads its weights W [N][K] in tile order: the 1 KB
// block (n / 16) * (K / 32) + k / 32 holds rows 16 (n / 16) .. + 15 and k
// 32 (k / 32) .. + 31 as 64 chunks of 8 k, chunk ((k % 32) / 8) * 16 + n % 16.
// launch_pack_tile_order writes that layout from nn.Linear layout (N % 16 ==
// 0, K % 32 == 0).
hipError_t launch_pack_tile_order(const uint16_t* W, int N, int K, uint16_t* out,
                                  hipStream_t st);
// The gate/up matrix [W_g; W_u] ([2F][K], F % 8 == 0) in tile order with its
// rows interleaved: packed rows 16b .. 16b + 7 are gate rows 8b .. 8b + 7,
// packed rows 16b + 8 .. 16b + 15 the matching up rows, so both factors of an
// output come out of one 16-column MFMA tile.
hipError_t launch_pack_gate_up(const uint16_t* W, int F, int K, uint16_t* out, hipStream_t st);

// part[s][m][n] = sum_{k in slice s} A[m][k] * W[n][k]   (bf16 in, fp32 out)
// The plan (split count S, workgroup width) and the K-order of every output element depend only on
// (N, K), never on M: rows are independent and batch-invariant.
struct SkinnyPlan {
  int waves;  // 16-column wave groups per workgroup (4..8)
  int S;      // K-slices (split-K)
};
SkinnyPlan skinny_plan(int N, int K);
hipError_t launch_gemm_skinny_bf16(const uint16_t* A, const uint16_t* W, float* part, int M,
                                   int N, int K, SkinnyPlan plan, hipStream_t st);
// Same with the gather and RMSNorm_1 folded in: the operand of row m is
// bf16(X[row_idx ? row_idx[m] : m] * gamma), and ss[s][m] = sum of X^2 over
// K-slice s (the consumer scales row m's sums by its 1/rms).
hipError_t launch_gemm_skinny_norm_bf16(const uint16_t* X, const int32_t* row_idx,
                                        const uint16_t* gamma, const uint16_t* W, float* part,
                                        float* ss, int M, int N, int K, SkinnyPlan plan,
                                        hipStream_t st);
// Decode gate/up GEMM with the SwiGLU epilogue: H[M][F] = bf16(silu(A W_g^T) *
// (A W_u^T)), W_gate_up [2F][K] interleaved (launch_pack_gate_up);
// plan = skinny_plan(2F, K) with S == 1.
// h_tiled: H in tile order (for a down projection that reads it so).
hipError_t launch_gemm_skinny_swiglu_bf16(const uint16_t* A, const uint16_t* W_gate_up,
                                          uint16_t* H, int M, int F, int K, SkinnyPlan plan,
                                          bool h_tiled, hipStream_t st);
// Prefill GEMMs (bf16, any M): A in tile order (tile_off; its buffer holds M
// rounded up to 16 rows), W in tile order, N and K multiples of 128, unsplit
// along K. The tile shape is chosen by (M, N, K) and the number of CUs and
// changes no result. Epilogue inputs of the variants (unused fields zero):
struct PrefillEpiArgs {
  // residual variant (O projection; x1: also the partial variant's output)
  const uint16_t* res_x = nullptr;   // residual rows [*][N] (bf16)
  const int32_t* res_idx = nullptr;  // row m's residual row (null: m)
  const uint16_t* gamma = nullptr;   // RMSNorm_2 gains [N]
  float* x1 = nullptr;               // [M][N] fp32
  uint16_t* h = nullptr;             // bf16(x1 * gamma), tile order
  float* ss_part = nullptr;          // [M][N / 32] row sums of x1^2 per 32 columns
  // scatter variant (down projection)
  const float* x1_in = nullptr;      // [M][N] fp32 residual
  uint16_t* out = nullptr;           // output rows [*][N] (bf16)
  const int32_t* out_idx = nullptr;  // row m's output row (null: m)
  // SwiGLU variant (gate/up projection, RMSNorm_2 folded in); h above is
  // its output [M][N / 2] in tile order
  const float* ss_in = nullptr;      // [M][K / 32] from the residual variant
  float eps = 0.f;
  bool h_rows = false;               // h row-major instead (SwiGLU without 1/rms only)
  // QKV variant (head_dim 128)
  const int32_t* row_info = nullptr;  // [M][2] row slots from the gather kernel
  const float* rope = nullptr;        // [rope_rows][64] (cos, sin) pairs
  uint16_t* q_out = nullptr;
  uint16_t* k_cache = nullptr;
  uint16_t* v_cache = nullptr;
  int Hq = 0, Hkv = 0;
};
// O projection with the residual and the first half of RMSNorm_2 in its
// epilogue: x1[m] = A W^T + res_x[res_idx ? res_idx[m] : m] (fp32),
// h[m] = bf16(x1 * gamma) in tile order, ss_part[m][g] = sum of x1^2 over
// columns 32g .. 32g + 31, in a fixed order.
hipError_t launch_prefill_resid_bf16(const uint16_t* A, const uint16_t* W, int M, int N, int K,
                                     const uint16_t* res_x, const int32_t* res_idx,
                                     const uint16_t* gamma, float* x1, uint16_t* h,
                                     float* ss_part, int num_cus, hipStream_t st);
// Gate/up projection with RMSNorm_2's 1/rms and the SwiGLU in its epilogue:
// H[m] = bf16(silu(g) * u) in tile order [M][F], where (g, u) = (A W_g^T,
// A W_u^T)[m] / sqrt(sum_g ss_in[m][g] / K + eps), and W_gate_up [2F][K] is in
// the interleaved order of launch_pack_gate_up.
hipError_t launch_prefill_swiglu_bf16(const uint16_t* A, const uint16_t* W_gate_up, uint16_t* H,
                                      int M, int F, int K, const float* ss_in, float eps,
                                      int num_cus, hipStream_t st);
// The same SwiGLU epilogue without the 1/rms (A already normalised), for
// decode batches. Every output is the v_mfma_f32_16x16x32_bf16 chain over k in
// ascending 32-steps of the decode GEMMs, with the same epilogue arithmetic,
// so the bits equal theirs. h_tiled: H in tile order, else row-major.
hipError_t launch_prefill_swiglu_plain_bf16(const uint16_t* A, const uint16_t* W_gate_up,
                                            uint16_t* H, int M, int F, int K, bool h_tiled,
                                            int num_cus, hipStream_t st);
// Decode projections of large batches: part[s][m][n] = sum over K-slice s (of
// S) of A[m][k] * W[n][k], A in tile order; the same chain of MFMAs, and bits,
// as launch_gemm_skinny_bf16 with that S (K a multiple of 128 S).
hipError_t launch_tile_partial_bf16(const uint16_t* A, const uint16_t* W, float* part, int M,
                                    int N, int K, int S, int num_cus, hipStream_t st);
// QKV projection with RoPE and the cache append in its epilogue (head_dim
// 128): queries to q_out [M][Hq*128] in bf16, keys (rotated) and values into
// the paged cache tiles.
hipError_t launch_prefill_qkv_bf16(const uint16_t* A, const uint16_t* W_qkv, int M, int K,
                                   const PrefillEpiArgs& ea, int num_cus, hipStream_t st);
// Down projection with the residual and the scatter in its epilogue:
// out[out_idx ? out_idx[m] : m] = bf16(x1[m] + A W^T).
hipError_t launch_prefill_scatter_bf16(const uint16_t* A, const uint16_t* W, int M, int N, int K,
                                       const float* x1, uint16_t* out, const int32_t* out_idx,
                                       int num_cus, hipStream_t st);

// ---------------------------------------------------------------- fp32 layer
// The four GEMMs of an fp32 layer (row-major, nn.Linear weights; K a multiple
// of 4), with the layer's row work in their prologues and epilogues. Epilogue
// inputs (unused fields zero):
struct F32EpiArgs {
  const float* gamma = nullptr;       // QKV, SwiGLU: RMSNorm gains [K]
  float eps = 0.f;
  float* h = nullptr;                 // QKV, SwiGLU: the normalised rows [M][K]
  const int32_t* row_idx = nullptr;   // QKV: row m's source row; residual: its row of res;
                                      // scatter: its row of out (null: m)
  const float* res = nullptr;         // residual, scatter: what is added
  float* out = nullptr;               // residual: x1 [M][N]; SwiGLU: u [M][F]; scatter: rows [*][N]
  // QKV
  const int32_t* positions = nullptr;
  const int32_t* seq_starts = nullptr;
  const int32_t* block_table = nullptr;
  const double* inv_freq = nullptr;
  float* q_out = nullptr;
  float* k_cache = nullptr;
  float* v_cache = nullptr;
  int n_seqs = 0, max_blocks = 0, Hq = 0, Hkv = 0, hd = 0;
};
// RMSNorm_1, QKV projection, RoPE, queries to q_out [M][Hq*hd], keys and
// values into the paged cache.
hipError_t launch_f32_qkv(const float* x, const float* w_qkv, int M, int d, const F32EpiArgs& ea,
                          hipStream_t st);
// out[m] = res[row_idx[m]] + o[m] W_o^T.
hipError_t launch_f32_resid(const float* o, const float* w_o, int M, int d, int qd,
                            const F32EpiArgs& ea, hipStream_t st);
// RMSNorm_2, gate/up projection ([2F][d]: gate rows, then up rows), SwiGLU.
hipError_t launch_f32_swiglu(const float* x1, const float* w_gate_up, int M, int F, int d,
                             const F32EpiArgs& ea, hipStream_t st);
// out[row_idx[m]] = res[m] + u[m] W_down^T.
hipError_t launch_f32_scatter(const float* u, const float* w_down, int M, int d, int F,
                              const F32EpiArgs& ea, hipStream_t st);

// ---------------------------------------------------------------- attention
constexpr int kDecodeSplit = 256;  // tokens per split-KV partition
int decode_max_splits(int max_blocks_per_seq);
bool attn_combine_fits(int max_splits);

// split_off (at most 2 n_seqs + 2 entries, written by the QKV epilogue of the
// same call): [0 .. n_seqs] the exclusive prefix sum of each sequence's full
// 256-key partitions; [n_seqs + 1] the number of sequences whose last
// partition is partial; [n_seqs + 2 ..] those sequences, longest last
// partition first.
// Decode row s attends min(ctx_lens[s], positions[s] + 1) keys.
hipError_t launch_attn_decode_bf16(const uint16_t* q, const uint16_t* k_cache,
                                   const uint16_t* v_cache, const int32_t* block_table,
                                   int max_blocks, const int32_t* ctx_lens,
                                   const int32_t* positions, const int32_t* split_off,
                                   int n_seqs, int Hq, int Hkv, float* part_o, float* part_ml,
                                   int max_splits, int num_cus, hipStream_t st);
// tiled: o in tile order (for an O projection that reads it so).
hipError_t launch_attn_combine_bf16(const float* part_o, const float* part_ml,
                                    const int32_t* ctx_lens, const int32_t* positions,
                                    int n_seqs, int Hq, int max_splits, uint16_t* o, bool tiled,
                                    hipStream_t st);

// Causal attention of prefill rows over their sequences' caches; o [n_rows]
// [Hq * 128] is written in tile order (the O projection's A operand).
hipError_t launch_attn_prefill_bf16(const uint16_t* q, const uint16_t* k_cache,
                                    const uint16_t* v_cache, const int32_t* block_table,
                                    int max_blocks, const int32_t* ctx_lens,
                                    const int32_t* positions, const int32_t* seq_starts,
                                    int n_seqs, int n_rows, int Hq, int Hkv, uint16_t* o,
                                    int num_cus, hipStream_t st);

// fp32 path, decode and prefill alike (hd a multiple of 32, at most 256).
hipError_t launch_attn_f32(const float* q, const float* k_cache, const float* v_cache,
                           const int32_t* block_table, int max_blocks,
                           const int32_t* ctx_lens, const int32_t* positions,
                           const int32_t* seq_starts, int n_seqs, int n_rows, int Hq,
                           int Hkv, int hd, float* o, hipStream_t st);

}  // namespace coco
