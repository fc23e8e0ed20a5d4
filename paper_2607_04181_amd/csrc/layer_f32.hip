// fp32 layer: four GEMM kernels with the layer's row work in their prologue
// and epilogue, so a layer is five launches with the attention.
//
//   acc[m][n] = sum_k A[m][k] * W[n][k]     v_mfma_f32_16x16x4_f32, fp32 in and out
//
//   * QKV: A = x * gamma (rows gathered); the row's 1/rms, from the sums of
//     squares of the very operands, scales the accumulators; RoPE, queries to
//     q, keys and values into the paged cache;
//   * residual (O projection): x1 = x + acc;
//   * SwiGLU (gate/up): A = x1 * gamma, 1/rms as above, u = silu(g) * u;
//   * scatter (down): out[row_idx[m]] = x1 + acc.
// fp32 layers are small (test and reference configurations), so a call is
// bound by latency: launches and chains of dependent loads. A workgroup owns
// 16 * RT rows x two 16-column tiles and its eight waves split K: wave w takes
// the 32-k chunks w, w + 8, ..., one loaded while the one before is
// multiplied; the waves' sums meet in LDS in wave order. At K = 256 every load
// of the kernel is one round trip. A wave loads whole 128-byte lines (eight
// lanes a row) and turns them to MFMA operands through LDS of its own, so the
// loop has no barrier: loaded straight into the operand layout, where
// neighbouring lanes hold different rows, a load touches 16 lines and takes
// ~75 cycles (gate/up of 200 rows, d = 1024: 60 against 39 us). Against 16 x 16 LDS
// tiles, one output per thread, and ten launches: tiny layer (d = 256, 4
// rows) 103 -> 28 us, d = 1024, 200-row prefill 588 -> 109 us.
// The order of every sum depends on K (or d) alone, not on M, RT or the other
// rows.
#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace coco {

namespace {

constexpr int kFWaves = 8, kFThreads = 64 * kFWaves;
constexpr int kFChunk = 32;  // k per wave and step

enum { kFQkv = 0, kFResid = 1, kFSwiglu = 2, kFScatter = 3 };

template <int MODE, int RT>
__global__ __launch_bounds__(kFThreads) void layer_f32_gemm_kernel(const float* __restrict__ A,
                                                                   const float* __restrict__ W,
                                                                   int M, int N, int K,
                                                                   F32EpiArgs ea) {
  constexpr bool kNorm = MODE == kFQkv || MODE == kFSwiglu;
  constexpr int TM = 16 * RT;
  // Each wave's chunk (32 k of TM rows of A, then 32 of W, as 16-byte pieces
  // at piece ^ (row / 2) % 8: conflict-free both ways); after the loop the
  // waves' sums.
  constexpr int kRows = TM + 32;
  __shared__ f32x4_t stage[kFWaves][kRows * 8];
  f32x4_t(*const part)[RT][2][64] = reinterpret_cast<f32x4_t(*)[RT][2][64]>(stage);
  static_assert(RT * 2 * 64 <= kRows * 8, "the sums fit");
  __shared__ float ssw[kNorm ? kFWaves : 1][TM];
  __shared__ float inv[TM];
  __shared__ int arow[TM];     // source (QKV: hidden) or output (scatter) row
  __shared__ int pos_s[TM];    // QKV: position
  __shared__ int64_t blk_s[TM];  // QKV: cache block
  __shared__ float rot[MODE == kFQkv ? TM * 16 : 1][2];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c16 = lane & 15, j4 = lane >> 4;
  const int m0 = blockIdx.y * TM;
  // W row of column x (0..31) of the tile. QKV: dims j and j + hd/2 of one
  // head, j = j0 + x % 16; SwiGLU: output o's gate and up rows; else 32 columns
  // side by side. Columns past N read the last one and are never stored.
  const int F = N / 2;
  int head = 0, j0 = 0;
  if constexpr (MODE == kFQkv) {
    const int per = ea.hd / 32;
    head = blockIdx.x / per;
    j0 = 16 * (blockIdx.x - head * per);
  }
  auto w_row = [&](int x) -> int {
    const int t = x >> 4, c = x & 15;
    if constexpr (MODE == kFQkv) return head * ea.hd + j0 + c + t * (ea.hd / 2);
    if constexpr (MODE == kFSwiglu) return t * F + min((int)blockIdx.x * 16 + c, F - 1);
    return min((int)blockIdx.x * 32 + x, N - 1);
  };

  // Loads: lane l takes 16-byte piece l % 8 of rows l / 8 + 8 i of the chunk.
  // Pieces past K (a multiple of 4) are zero in both operands.
  constexpr int kLd = kRows / 8, kLdA = TM / 8;
  const int lr = lane >> 3, pc = lane & 7;
  const float* src[kLd];
#pragma unroll
  for (int i = 0; i < kLd; ++i) {
    const int r = lr + 8 * i;
    if (i < kLdA) {
      const int m = min(m0 + r, M - 1);
      src[i] = A + (int64_t)((MODE == kFQkv && ea.row_idx) ? ea.row_idx[m] : m) * K;
    } else {
      src[i] = W + (int64_t)w_row(r - TM) * K;
    }
  }
  f32x4_t v[kLd], gv;
  auto load = [&](int c) {
    const int k = min(kFChunk * c + 4 * pc, K - 4);
#pragma unroll
    for (int i = 0; i < kLd; ++i) v[i] = *(const f32x4_t*)(src[i] + k);
    if (kNorm) gv = *(const f32x4_t*)(ea.gamma + k);
  };
  f32x4_t acc[RT][2];
#pragma unroll
  for (int t = 0; t < RT; ++t) acc[t][0] = acc[t][1] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  float ss[kLdA];
#pragma unroll
  for (int i = 0; i < kLdA; ++i) ss[i] = 0.f;
  f32x4_t* const mine = stage[wv];
  auto put = [&](int c) {
    const bool live = kFChunk * c + 4 * pc < K;
#pragma unroll
    for (int i = 0; i < kLd; ++i) {
      const int r = lr + 8 * i;
      f32x4_t x;
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] = live ? v[i][e] : 0.f;
      if (kNorm && i < kLdA) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          ss[i] = fmaf(x[e], x[e], ss[i]);
          x[e] *= live ? gv[e] : 0.f;
        }
      }
      mine[r * 8 + (pc ^ ((r >> 1) & 7))] = x;
    }
  };
  // Operand lane (c16, j4): k = 8 j4 + 0..7 of the chunk, step e takes k 8 j4 + e.
  auto mul = [&]() {
    auto get = [&](int r, int h) { return mine[r * 8 + ((2 * j4 + h) ^ ((r >> 1) & 7))]; };
    f32x4_t a[RT][2], w[2][2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int t = 0; t < RT; ++t) a[t][h] = get(16 * t + c16, h);
#pragma unroll
      for (int u = 0; u < 2; ++u) w[u][h] = get(TM + 16 * u + c16, h);
    }
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int t = 0; t < RT; ++t)
#pragma unroll
          for (int u = 0; u < 2; ++u)
            acc[t][u] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[t][h][e], w[u][h][e], acc[t][u], 0,
                                                            0, 0);
  };
  const int chunks = (K + kFChunk - 1) / kFChunk;
  load(wv);

  // Row data of the epilogue while the first chunk is on its way.
  if (tid < TM) {
    const int m = min(m0 + tid, M - 1);
    if constexpr (MODE == kFQkv) {
      const int pos = ea.positions[m];
      const int seq = row_to_seq(ea.seq_starts, ea.n_seqs, m);
      arow[tid] = ea.row_idx ? ea.row_idx[m] : m;
      pos_s[tid] = pos;
      blk_s[tid] = ea.block_table[(int64_t)seq * ea.max_blocks + pos / kBlockTokens];
    } else if constexpr (MODE == kFScatter || MODE == kFResid) {
      arow[tid] = ea.row_idx ? ea.row_idx[m] : m;
    }
  }
  if constexpr (MODE == kFQkv) {
    // The rows' rotation angles, cosine and sine in fp64.
    for (int i = tid; i < TM * 16; i += kFThreads) {
      double sn, cn;
      sincos((double)ea.positions[min(m0 + (i >> 4), M - 1)] * ea.inv_freq[j0 + (i & 15)], &sn,
             &cn);
      rot[i][0] = (float)cn;
      rot[i][1] = (float)sn;
    }
  }

  for (int c = wv; c < chunks; c += kFWaves) {
    put(c);
    load(c + kFWaves);
    wave_lds_order();  // other lanes' pieces
    mul();
    wave_lds_order();  // read before the next chunk overwrites them
  }

  // The waves' sums, in wave order; a wave's worth of threads per row tile
  // finishes them.
  if constexpr (kNorm) {
#pragma unroll
    for (int i = 0; i < kLdA; ++i) {
      float s = ss[i];  // the row's eight lanes
      s += __shfl_xor(s, 1, kWave);
      s += __shfl_xor(s, 2, kWave);
      s += __shfl_xor(s, 4, kWave);
      if (pc == 0) ssw[wv][lr + 8 * i] = s;
    }
  }
  __syncthreads();  // every wave is done with its chunks
#pragma unroll
  for (int t = 0; t < RT; ++t) {
    part[wv][t][0][lane] = acc[t][0];
    part[wv][t][1][lane] = acc[t][1];
  }
  __syncthreads();
  if constexpr (kNorm) {
    if (tid < TM) {
      float s = 0.f;
#pragma unroll
      for (int w = 0; w < kFWaves; ++w) s += ssw[w][tid];
      inv[tid] = 1.0f / sqrtf(s / (float)K + ea.eps);
    }
    __syncthreads();
    // The normalised rows themselves, spread over the columns' workgroups (by
    // the first of them alone, their dependent loads took as long as the GEMM).
    for (int i = blockIdx.x * kFThreads + tid; i < TM * (K / 4); i += gridDim.x * kFThreads) {
      const int r = i / (K / 4), k = 4 * (i - r * (K / 4));
      if (m0 + r >= M) break;  // rows ascend with i
      const int64_t src = MODE == kFQkv ? arow[r] : m0 + r;
      const f32x4_t x = *(const f32x4_t*)(A + src * K + k);
      const f32x4_t g = *(const f32x4_t*)(ea.gamma + k);
      f32x4_t y;
#pragma unroll
      for (int e = 0; e < 4; ++e) y[e] = x[e] * inv[r] * g[e];
      *(f32x4_t*)(ea.h + (int64_t)(m0 + r) * K + k) = y;
    }
  }
  if (tid >= RT * 64) return;
  const int t = tid >> 6;
  f32x4_t s0 = part[0][t][0][lane], s1 = part[0][t][1][lane];
#pragma unroll
  for (int w = 1; w < kFWaves; ++w) {
    s0 += part[w][t][0][lane];
    s1 += part[w][t][1][lane];
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int rl = 16 * t + 4 * j4 + r, m = m0 + rl;
    if (m >= M) continue;
    float v0 = s0[r], v1 = s1[r];
    if constexpr (kNorm) {
      v0 *= inv[rl];
      v1 *= inv[rl];
    }
    if constexpr (MODE == kFQkv) {
      const int hd = ea.hd, j = j0 + c16;
      if (head < ea.Hq + ea.Hkv) {
        const float cn = rot[rl * 16 + c16][0], sn = rot[rl * 16 + c16][1];
        const float lo = v0 * cn - v1 * sn, hi = v1 * cn + v0 * sn;
        v0 = lo;
        v1 = hi;
      }
      if (head < ea.Hq) {
        float* dst = ea.q_out + ((int64_t)m * ea.Hq + head) * hd + j;
        dst[0] = v0;
        dst[hd / 2] = v1;
      } else {
        const int slot = pos_s[rl] % kBlockTokens;
        const bool key = head < ea.Hq + ea.Hkv;
        const int g = head - ea.Hq - (key ? 0 : ea.Hkv);
        float* tile = (key ? ea.k_cache : ea.v_cache) +
                      (blk_s[rl] * ea.Hkv + g) * (int64_t)(kBlockTokens * hd);
        tile[key ? k_tile_offset(slot, j) : v_tile_offset(slot, j)] = v0;
        tile[key ? k_tile_offset(slot, j + hd / 2) : v_tile_offset(slot, j + hd / 2)] = v1;
      }
    } else if constexpr (MODE == kFSwiglu) {
      const int o = blockIdx.x * 16 + c16;
      if (o < F) ea.out[(int64_t)m * F + o] = silu_mul(v0, v1);
    } else {
      // Residual: x1[m] = x[arow] + acc; scatter: out[arow] = x1[m] + acc.
      const int64_t rx = (int64_t)(MODE == kFResid ? arow[rl] : m) * N;
      const int64_t ro = (int64_t)(MODE == kFResid ? m : arow[rl]) * N;
      const int n = blockIdx.x * 32 + c16;
      if (n < N) ea.out[ro + n] = ea.res[rx + n] + v0;
      if (n + 16 < N) ea.out[ro + n + 16] = ea.res[rx + n + 16] + v1;
    }
  }
}

// Two row tiles per workgroup above 16 rows: the W operands serve both. Four
// above 64 leave the chip short of workgroups (d = 1024, us for two / four: 130
// rows 89 / 130, 512 rows 221 / 245).
template <int MODE>
hipError_t launch_f32(const float* A, const float* W, int M, int N, int K, int cols,
                      const F32EpiArgs& ea, hipStream_t st) {
  if (M <= 0) return hipSuccess;
  if (K % 4 != 0 || K < 4 || cols <= 0) return hipErrorInvalidValue;
  if (M <= 16)
    COCO_LAUNCH((layer_f32_gemm_kernel<MODE, 1>), dim3(cols, 1), dim3(kFThreads), 0, st, A, W, M,
                N, K, ea);
  else
    COCO_LAUNCH((layer_f32_gemm_kernel<MODE, 2>), dim3(cols, (M + 31) / 32), dim3(kFThreads), 0,
                st, A, W, M, N, K, ea);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_f32_qkv(const float* x, const float* w_qkv, int M, int d, const F32EpiArgs& ea,
                          hipStream_t st) {
  const int N = (ea.Hq + 2 * ea.Hkv) * ea.hd;
  if (ea.hd % 32 != 0) return hipErrorInvalidValue;
  return launch_f32<kFQkv>(x, w_qkv, M, N, d, N / 32, ea, st);
}

hipError_t launch_f32_resid(const float* o, const float* w_o, int M, int d, int qd,
                            const F32EpiArgs& ea, hipStream_t st) {
  return launch_f32<kFResid>(o, w_o, M, d, qd, (d + 31) / 32, ea, st);
}

hipError_t launch_f32_swiglu(const float* x1, const float* w_gate_up, int M, int F, int d,
                             const F32EpiArgs& ea, hipStream_t st) {
  return launch_f32<kFSwiglu>(x1, w_gate_up, M, 2 * F, d, (F + 15) / 16, ea, st);
}

hipError_t launch_f32_scatter(const float* u, const float* w_down, int M, int d, int F,
                              const F32EpiArgs& ea, hipStream_t st) {
  return launch_f32<kFScatter>(u, w_down, M, d, F, (d + 31) / 32, ea, st);
}

// ---------------------------------------------------------------- attention
// One workgroup per (row, GH query heads of one key/value head); its eight
// waves take the 16-token blocks w, w + 8, ... of the row's keys, each with an
// online softmax, and meet in LDS in wave order. In a block, lane (t, j) =
// (lane % 16, lane / 16) scores token t over the dims it holds of the key
// tile (8 per 32, contiguous), the four lanes of a token are added, and for
// the values lane (h, q) = (lane % 16, lane / 16) holds dims h and h + 16 of
// each 32 at tokens 4q .. 4q + 3: every load is 32 contiguous bytes per lane,
// a wave's 2 KB. The keys a wave sees depend on the row's own length only.
// One wave per (row, head), one key at a time, took 33 us for 65 keys and
// 146 us for the 200-row prefill (16 heads of 64); now 5 and 23 us.
namespace {

constexpr int kAWaves = 8;

template <int HS, int GH>  // hd = 32 HS
__global__ __launch_bounds__(64 * kAWaves) void attn_f32_kernel(
    const float* __restrict__ q, const float* __restrict__ k_cache,
    const float* __restrict__ v_cache, const int32_t* __restrict__ block_table, int max_blocks,
    const int32_t* __restrict__ ctx_lens, const int32_t* __restrict__ positions,
    const int32_t* __restrict__ seq_starts, int n_seqs, int Hq, int Hkv, float* __restrict__ o) {
  constexpr int hd = 32 * HS;
  __shared__ float sm_m[kAWaves][GH], sm_l[kAWaves][GH];
  __shared__ float sm_o[kAWaves][GH][hd];
  const int i = blockIdx.x, h0 = blockIdx.y * GH;
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int t = lane & 15, j4 = lane >> 4;
  const int s = row_to_seq(seq_starts, n_seqs, i);
  const int g = h0 / (Hq / Hkv);
  const int n = min(ctx_lens[s], positions[i] + 1);
  const int blocks = (n + kBlockTokens - 1) / kBlockTokens;
  const int32_t* bt = block_table + (int64_t)s * max_blocks;
  const float scale = 1.0f / sqrtf((float)hd);

  // This lane's part of the queries: dims 32 p + 8 j4 .. + 7.
  f32x4_t qv[GH][HS][2];
#pragma unroll
  for (int e = 0; e < GH; ++e)
#pragma unroll
    for (int p = 0; p < HS; ++p)
#pragma unroll
      for (int f = 0; f < 2; ++f)
        qv[e][p][f] =
            *(const f32x4_t*)(q + ((int64_t)i * Hq + h0 + e) * hd + 32 * p + 8 * j4 + 4 * f);

  float m[GH], l[GH], acc[GH][HS][2];
#pragma unroll
  for (int e = 0; e < GH; ++e) {
    m[e] = -INFINITY;
    l[e] = 0.f;
#pragma unroll
    for (int p = 0; p < HS; ++p) acc[e][p][0] = acc[e][p][1] = 0.f;
  }
  for (int b = wv; b < blocks; b += kAWaves) {
    const int64_t tile = ((int64_t)bt[b] * Hkv + g) * (kBlockTokens * hd);
    f32x4_t kf[HS][2], vf[HS][2];
#pragma unroll
    for (int p = 0; p < HS; ++p)
#pragma unroll
      for (int f = 0; f < 2; ++f) {
        kf[p][f] = *(const f32x4_t*)(k_cache + tile + (p * 64 + lane) * 8 + 4 * f);
        vf[p][f] = *(const f32x4_t*)(v_cache + tile + (p * 64 + lane) * 8 + 4 * f);
      }
    const bool live = b * kBlockTokens + t < n;
    // Slots past the row's keys may hold anything: their values are not used.
    const int left = n - (b * kBlockTokens + 4 * j4);  // live tokens of this lane's four
#pragma unroll
    for (int e = 0; e < GH; ++e) {
      float z = 0.f;
#pragma unroll
      for (int p = 0; p < HS; ++p)
#pragma unroll
        for (int f = 0; f < 2; ++f)
#pragma unroll
          for (int c = 0; c < 4; ++c) z = fmaf(qv[e][p][f][c], kf[p][f][c], z);
      z += __shfl_xor(z, 16, kWave);
      z += __shfl_xor(z, 32, kWave);
      z = live ? z * scale : -INFINITY;
      float mx = z;
#pragma unroll
      for (int d = 8; d > 0; d >>= 1) mx = fmaxf(mx, __shfl_xor(mx, d, kWave));
      const float m_new = fmaxf(m[e], mx);
      // A block of keys that all score -inf leaves m at -inf.
      const float m_ref = m_new == -INFINITY ? 0.f : m_new;
      const float alpha = expf(m[e] - m_ref);
      const float pr = expf(z - m_ref);
      float ls = pr;
#pragma unroll
      for (int d = 8; d > 0; d >>= 1) ls += __shfl_xor(ls, d, kWave);
      l[e] = l[e] * alpha + ls;
      m[e] = m_new;
      float p4[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) p4[c] = __shfl(pr, 4 * j4 + c, kWave);
#pragma unroll
      for (int p = 0; p < HS; ++p)
#pragma unroll
        for (int f = 0; f < 2; ++f) {
          float a = acc[e][p][f] * alpha;
#pragma unroll
          for (int c = 0; c < 4; ++c) a = fmaf(p4[c], c < left ? vf[p][f][c] : 0.f, a);
          acc[e][p][f] = a;
        }
    }
  }
#pragma unroll
  for (int e = 0; e < GH; ++e) {
    if (lane == 0) {
      sm_m[wv][e] = m[e];
      sm_l[wv][e] = l[e];
    }
#pragma unroll
    for (int p = 0; p < HS; ++p)
#pragma unroll
      for (int f = 0; f < 2; ++f) {
        float a = acc[e][p][f];  // dim 32 p + 16 f + lane % 16, tokens 4 j4 ..
        a += __shfl_xor(a, 16, kWave);
        a += __shfl_xor(a, 32, kWave);
        if (j4 == 0) sm_o[wv][e][32 * p + 16 * f + t] = a;
      }
  }
  __syncthreads();
  for (int x = threadIdx.x; x < GH * hd; x += 64 * kAWaves) {
    const int e = x / hd, dim = x - e * hd;
    float mx = sm_m[0][e];
#pragma unroll
    for (int w = 1; w < kAWaves; ++w) mx = fmaxf(mx, sm_m[w][e]);
    const float ref = mx == -INFINITY ? 0.f : mx;
    float a = 0.f, L = 0.f;
#pragma unroll
    for (int w = 0; w < kAWaves; ++w) {
      const float f = expf(sm_m[w][e] - ref);
      a = fmaf(f, sm_o[w][e][dim], a);
      L = fmaf(f, sm_l[w][e], L);
    }
    o[((int64_t)i * Hq + h0 + e) * hd + dim] = n > 0 ? a / L : 0.f;
  }
}

}  // namespace

hipError_t launch_attn_f32(const float* q, const float* k_cache, const float* v_cache,
                           const int32_t* block_table, int max_blocks, const int32_t* ctx_lens,
                           const int32_t* positions, const int32_t* seq_starts, int n_seqs,
                           int n_rows, int Hq, int Hkv, int hd, float* o, hipStream_t st) {
  if (n_rows <= 0) return hipSuccess;
  // Heads per workgroup: they share the key/value loads; the queries they
  // keep in registers (hd / 4 floats per lane each) bound their number.
  const int G = Hq / Hkv;
  const int gh = (G % 4 == 0 && hd <= 64) ? 4 : (G % 2 == 0 && hd <= 128) ? 2 : 1;
  const dim3 grid(n_rows, Hq / gh);
#define COCO_ATT(HS, GH)                                                                       \
  COCO_LAUNCH((attn_f32_kernel<HS, GH>), grid, dim3(64 * kAWaves), 0, st, q, k_cache, v_cache, \
              block_table, max_blocks, ctx_lens, positions, seq_starts, n_seqs, Hq, Hkv, o)
#define COCO_ATT4(HS) \
  if (gh == 4) COCO_ATT(HS, 4); else if (gh == 2) COCO_ATT(HS, 2); else COCO_ATT(HS, 1)
#define COCO_ATT2(HS) \
  if (gh == 2) COCO_ATT(HS, 2); else COCO_ATT(HS, 1)
  switch (hd) {
    case 32: COCO_ATT4(1); break;
    case 64: COCO_ATT4(2); break;
    case 96: COCO_ATT2(3); break;
    case 128: COCO_ATT2(4); break;
    case 160: COCO_ATT(5, 1); break;
    case 192: COCO_ATT(6, 1); break;
    case 224: COCO_ATT(7, 1); break;
    case 256: COCO_ATT(8, 1); break;
    default: return hipErrorInvalidValue;
  }
#undef COCO_ATT4
#undef COCO_ATT2
#undef COCO_ATT
  return hipGetLastError();
}

}  // namespace coco
