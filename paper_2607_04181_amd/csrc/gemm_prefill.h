// Prefill GEMMs (bf16 MFMA), each unsplit along K with its consumer's work in
// the epilogue.
//
//   acc[m][n] = sum_k A[m][k] * W[n][k]      A: [M][K], W: [N][K], both bf16
//
// A and W are in tile order (tile_off / pack_tile_order): every 16 rows x
// 32 k is one contiguous 1 KB block, laid out lane by lane as a
// v_mfma_f32_16x16x32_bf16 operand, so one 16-byte-per-lane load copies a
// block to LDS unchanged and one 16-byte LDS read per lane is a fragment.
// Epilogue variants:
//   * residual (O projection): x1 = acc + residual row (fp32 out),
//     h = bf16(x1 * gamma) in tile order for the gate/up projection, and the
//     row's sums of x1^2 per 32 columns (RMSNorm_2's statistics, finished by
//     the gate/up epilogue);
//   * scatter (down projection): out[out_idx[m]] = bf16(x1 + acc), the layer
//     output written straight to its row of the full batch;
//   * SwiGLU (gate/up projection): W interleaves 8 gate rows with the 8
//     matching up rows in every 16-row block (pack_gate_up), so the two
//     factors of an output sit 8 lanes apart; h = silu(gate / rms) * up / rms
//     in tile order;
//   * QKV: a tile holds whole RoPE pairs; queries are rotated into q, keys
//     rotated and values copied into the paged cache;
//   * partial (decode batches): the fp32 sums of K-slice blockIdx.y, for the
//     decode epilogues.
// Main loop:
//   * WM x WN waves; each owns a TM/WM x TN/WN sub-tile as accumulators of
//     16 x 16;
//   * stages of 32 * KS k of both tiles go straight from global memory to LDS
//     (global_load_lds, no register staging) into a ring of SLOTS slots, all
//     but one stage in flight (the loads come from L2, the MALL or HBM, whose
//     latency under this load is several stages of MFMA work);
//   * one barrier per stage, which publishes stage st + 1 and guarantees
//     that the slot the next loads overwrite was read by every wave;
//   * workgroups are remapped so that the tiles sharing a W column slab run
//     on the same XCD (blockIdx % 8) and hit its L2.
// Every output element is one chain of MFMAs over k in ascending 32-steps and
// every epilogue sum has an order fixed by its columns, so a row's result
// depends neither on M and the other rows of the call nor on the tile shape,
// which the launcher is free to choose by M.
#pragma once

#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace coco {
namespace prefill {

constexpr int kNXCDs = 8;
constexpr int kSsCols = 32;  // columns per sum of x1^2, [M][d / 32]

typedef __attribute__((address_space(3))) void lds_void_t;

// kSwigluPlain: the SwiGLU epilogue without RMSNorm_2's 1/rms (the operand is
// already normalised).
enum { kResid = 0, kScatter = 1, kSwiglu = 2, kQkv = 3, kSwigluPlain = 4, kPartial = 5 };

// Tile shape: TM x TN outputs, WM x WN waves, KS 32-k blocks per stage,
// SLOTS ring slots.
template <int TM_, int TN_, int WM_, int WN_, int KS_, int SLOTS_>
struct Tile {
  static constexpr int TM = TM_, TN = TN_, WM = WM_, WN = WN_, KS = KS_, SLOTS = SLOTS_;
  static constexpr int NW = WM * WN, NT = 64 * NW;
  static constexpr int RB = TM / 16 / WM, CB = TN / 16 / WN;  // 16-row / 16-column blocks per wave
  static constexpr int AB = TM / 16 * KS, NB = AB + TN / 16 * KS;  // 1 KB blocks per stage: A, all
  // Loads per stage and wave. Every wave issues the same number, so all wait
  // on the same counts and the loop has no branch around a load: FULL whole
  // blocks, then what is left of NB / NW. A load costs the same whatever its
  // width, so the rest is one more load per wave: a quarter block each (4
  // bytes per lane) where a quarter of the waves' count is left (QUARTER:
  // 256 x 160, down 428 -> 419 us), else a whole block, some waves copying
  // their last block again into a spare block that is never read (SPARE; two
  // or three quarter loads measured 3-8% slower).
  static constexpr int FULL = NB / NW;
  static constexpr bool QUARTER = NB % NW * 4 == NW, SPARE = NB % NW != 0 && !QUARTER;
  static constexpr int LOADS = (NB + NW - 1) / NW;
  // Block of whole load i of wave w. Where the A blocks
  // divide by the waves, a wave takes adjacent ones: strided ones measured
  // 1.5% slower on the large tiles.
  static constexpr bool AEVEN = AB % NW == 0;
  static __device__ __forceinline__ int block(int w, int i) {
    if (AEVEN && i < AB / NW) return w * (AB / NW) + i;
    return w + i * NW;
  }
  // Load i of wave w from the stage's blocks, in quarter blocks.
  static __device__ __forceinline__ int source(int w, int i) {
    if (QUARTER && i == FULL) return 4 * FULL * NW + w;
    int q = block(w, i);
    if (SPARE && q >= NB) q = block(w, i - 1);
    return 4 * q;
  }
  static constexpr int bytes(int i) { return QUARTER && i == FULL ? 4 : 16; }  // per lane
  static constexpr int AHEAD = SLOTS - 1;  // stages in flight
  // Stages per unrolled round: slots and fragment registers (which alternate
  // with the 32-k step) are then known at compile time.
  static constexpr int ROUND = (SLOTS * KS) % 2 ? 2 * SLOTS : SLOTS;
  static_assert(TM % (16 * WM) == 0 && TN % (16 * WN) == 0 && TN % 32 == 0, "tile shape");
  static_assert(SLOTS >= 3 && SLOTS <= 8 && SLOTS > RB && RB <= 5, "ring slots");
  static_assert(LOADS * (AHEAD - 1) < 64, "vmcnt range");
};

// A row's sum of x1^2 over its groups of 32 columns (ss: [M][K / 32], n4 =
// K / 128 vectors of four groups per row), in two halves by two threads: the
// vectors of half h added in order, then (0 + 1) + (2 + 3); the row's sum is
// half 0 + half 1. The first kSsVec vectors (all of them for K <= 5120) are
// one round of loads, issued by ss_load.
constexpr int kSsVec = 20;
struct SsPart {
  f32x4_t v[kSsVec];
};
__device__ __forceinline__ void ss_load(SsPart& s, const float* __restrict__ ss, int m, int h,
                                        int n4) {
  const int nh = (n4 + 1) / 2;
  const f32x4_t* p = (const f32x4_t*)ss + (int64_t)m * n4;
#pragma unroll
  for (int c = 0; c < kSsVec; ++c) s.v[c] = p[min(h * nh + c, n4 - 1)];
}
__device__ __forceinline__ float ss_half(const SsPart& s, const float* __restrict__ ss, int m,
                                         int h, int n4) {
  const int nh = (n4 + 1) / 2, n = min(nh, n4 - h * nh);
  const f32x4_t* p = (const f32x4_t*)ss + (int64_t)m * n4 + h * nh;
  f32x4_t t = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int c = 0; c < kSsVec; ++c) {
    const f32x4_t v = s.v[c];
#pragma unroll
    for (int e = 0; e < 4; ++e) t[e] += c < n ? v[e] : 0.f;
  }
  for (int c = kSsVec; c < n; ++c) t += p[c];
  return (t[0] + t[1]) + (t[2] + t[3]);
}

// SwiGLU of one accumulator of an interleaved gate/up block: lane c16 < 8
// holds the gates of output c16 (rows 0..3 of its quad), lane c16 + 8 the
// matching ups. The lanes swap halves, then lane c16 < 8 finishes rows 0 and
// 1 of the quad and lane c16 >= 8 rows 2 and 3 of output c16 - 8. rs: the
// row scales of the two rows.
__device__ __forceinline__ void swiglu_quad(const f32x4_t a, float rs0, float rs1, float* y) {
  // Lanes c16 >= 8 (upper) or c16 < 8 (lower) get lane (c16 + 8) % 16's
  // `other` (row_ror:8 under a bank mask), the rest keep `own`.
  auto upper = [](float own, float other) {
    return __int_as_float(__builtin_amdgcn_update_dpp(
        __float_as_int(own), __float_as_int(other), 0x128, 0xF, 0xC, false));
  };
  auto lower = [](float own, float other) {
    return __int_as_float(__builtin_amdgcn_update_dpp(
        __float_as_int(own), __float_as_int(other), 0x128, 0xF, 0x3, false));
  };
  const float g0 = upper(a[0], a[2]), u0 = lower(a[2], a[0]);
  const float g1 = upper(a[1], a[3]), u1 = lower(a[3], a[1]);
  y[0] = silu_mul(g0 * rs0, u0 * rs0);
  y[1] = silu_mul(g1 * rs1, u1 * rs1);
}

template <class T, int MODE>
__global__ __launch_bounds__(T::NT) void gemm_prefill_kernel(const bf16_t* __restrict__ A,
                                                              const bf16_t* __restrict__ W, int M,
                                                              int N, int K, PrefillEpiArgs ea) {
  constexpr bool kSwi = MODE == kSwiglu || MODE == kSwigluPlain;
  constexpr int TM = T::TM, TN = T::TN, WM = T::WM, KS = T::KS, RB = T::RB, CB = T::CB;
  constexpr int NW = T::NW, NT = T::NT, AB = T::AB, NB = T::NB, LOADS = T::LOADS;
  constexpr int SLOTS = T::SLOTS, AHEAD = T::AHEAD, ROUND = T::ROUND;
  constexpr int kSlot = NB * 512;  // elements
  // One LDS object per ring slot, so the compiler tracks each slot's pending
  // direct loads on its own and never drains the ring before a fragment read.
  __shared__ __attribute__((aligned(16))) bf16_t s0[kSlot], s1[kSlot], s2[kSlot], s3[kSlot],
      s4[kSlot], s5[kSlot], s6[kSlot], s7[kSlot];
  __shared__ __attribute__((aligned(16))) bf16_t spare[512];
  __shared__ __attribute__((aligned(16))) int rowv[2 * TM];  // a row's epilogue value(s)
  bf16_t* const ring[8] = {s0, s1, s2, s3, s4, s5, s6, s7};

  const int tiles_m = (M + TM - 1) / TM;
  const int nb = gridDim.x;
  const int b = blockIdx.x;
  const int full = (nb / kNXCDs) * kNXCDs;
  const int lid = b < full ? (b % kNXCDs) * (nb / kNXCDs) + b / kNXCDs : b;
  const int m0 = (lid % tiles_m) * TM;
  const int n0 = (lid / tiles_m) * TN;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wv % WM, wn = wv / WM;
  const int c16 = lane & 15, j4 = lane >> 4;

  // W block (16 rows) of the tile's column block blk. QKV: rotation pair
  // p = 64 hh + j holds dims j and j + 64 of head hh; the tile holds pairs
  // TN/2 (n0/TN) .. + TN/2 - 1 as TN/32 groups of 16, the j dims of group q
  // in block q, the j + 64 dims in block TN/32 + q.
  auto w_block = [&](int blk) -> int {
    if constexpr (MODE == kQkv) {
      const int h = blk / (TN / 32), q = blk % (TN / 32);
      const int p0 = 16 * ((n0 / TN) * (TN / 32) + q);
      return ((p0 >> 6) * 128 + (p0 & 63) + 64 * h) >> 4;
    }
    return (n0 >> 4) + blk;
  };
  // This wave's blocks of a stage, of the slot, which holds
  // the A blocks (row group, 32-k step), then the W blocks (column block,
  // 32-k step). Row groups past the last row read the last group; their rows
  // are never stored.
  const int k_slice = MODE == kPartial ? K / (int)gridDim.y : K;
  const int stages = k_slice / (32 * KS);
  const int64_t k_off = MODE == kPartial ? (int64_t)blockIdx.y * (k_slice / 32) * 1024 : 0;
  const char* src[LOADS];
#pragma unroll
  for (int i = 0; i < LOADS; ++i) {
    const int t = T::source(wv, i), q = t >> 2;
    const bool a = q < AB;
    const int qq = a ? q : q - AB;
    const int blk = a ? min((m0 >> 4) + qq / KS, (M - 1) >> 4) : w_block(qq / KS);
    src[i] = (const char*)(a ? A : W) + ((int64_t)blk * (K / 32) + qq % KS) * 1024 +
             k_off + (t & 3) * 256 + lane * T::bytes(i);
  }
  // Loads past the last stage repeat it (never multiplied).
  auto issue = [&](int st, int slot) {
    const int64_t off = (int64_t)min(st, stages - 1) * (KS * 1024);
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
      bf16_t* dst = ring[slot] + T::source(wv, i) * 128;
      if (T::SPARE && i == LOADS - 1) dst = T::block(wv, i) < NB ? dst : spare;
      if (T::bytes(i) == 4)
        __builtin_amdgcn_global_load_lds((const void*)(src[i] + off), (lds_void_t*)dst, 4, 0, 0);
      else
        __builtin_amdgcn_global_load_lds((const void*)(src[i] + off), (lds_void_t*)dst, 16, 0, 0);
    }
  };

  f32x4_t acc[RB][CB];
#pragma unroll
  for (int i = 0; i < RB; ++i)
#pragma unroll
    for (int j = 0; j < CB; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  auto read_frags = [&](const bf16_t* s, int ks, bf16x8_t* a, bf16x8_t* w) {
#pragma unroll
    for (int i = 0; i < RB; ++i)
      a[i] = __builtin_bit_cast(
          bf16x8_t, *(const u32x4_t*)(s + ((wm * RB + i) * KS + ks) * 512 + lane * 8));
#pragma unroll
    for (int j = 0; j < CB; ++j)
      w[j] = __builtin_bit_cast(
          bf16x8_t, *(const u32x4_t*)(s + (AB + (wn * CB + j) * KS + ks) * 512 + lane * 8));
  };
  auto mfma_step = [&](const bf16x8_t* a, const bf16x8_t* w, auto loads) {
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
      for (int j = 0; j < CB; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], w[j], acc[i][j], 0, 0, 0);
    // Large sub-tiles: in the step that issues a stage's direct loads, those
    // after the first four MFMAs (the MFMA pipe restarts right after the
    // barrier), then the fragment reads of the next step interleaved with these
    // MFMAs.
    if constexpr (RB * CB >= 8 + RB + CB) {
      constexpr int kFirst = decltype(loads)::value ? 4 : 0;
      if constexpr (kFirst != 0) {
        __builtin_amdgcn_sched_group_barrier(0x008, kFirst, 0);  // MFMA
        __builtin_amdgcn_sched_group_barrier(0x020, LOADS, 0);   // VMEM read
      }
      for (int g = 0; g < RB + CB; ++g) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);  // DS read
      }
      __builtin_amdgcn_sched_group_barrier(0x008, RB * CB - kFirst - RB - CB, 0);
    }
  };

  // The epilogue's row of each tile row (residual, output) or its cache slot.
  int erow = 0;
  u32x2_t rinfo = {0u, 0u};
  if (tid < TM) {
    const int m = min(m0 + tid, M - 1);
    if constexpr (MODE == kQkv) {
      rinfo = *(const u32x2_t*)(ea.row_info + 2 * m);
    } else if constexpr (MODE == kResid || MODE == kScatter) {
      const int32_t* idx = MODE == kResid ? ea.res_idx : ea.out_idx;
      erow = idx ? idx[m] : m;
    }
  }
  // SwiGLU: the rows' sums of x1^2, two threads per row, loaded ahead of the
  // ring and added while its first stages land.
  SsPart sp;
  const int n4 = K / (4 * kSsCols);
  static_assert(MODE != kSwiglu || NT >= 2 * TM, "two threads per row");
  if constexpr (MODE == kSwiglu) ss_load(sp, ea.ss_in, min(m0 + tid % TM, M - 1), (tid / TM) & 1, n4);
#pragma unroll
  for (int st = 0; st < AHEAD; ++st) issue(st, st);
  if constexpr (MODE == kSwiglu) {
    const float t = ss_half(sp, ea.ss_in, min(m0 + tid % TM, M - 1), (tid / TM) & 1, n4);
    if (tid < 2 * TM) rowv[tid] = __float_as_int(t);
  }
  wait_vmcnt<(AHEAD - 1) * LOADS>();  // this wave's stage-0 loads are in LDS
  stage_barrier();                    // every wave's
  bf16x8_t fa[2][RB], fw[2][CB];
  read_frags(ring[0], 0, fa[0], fw[0]);
  // One unrolled round: stages st0 .. st0 + ROUND - 1. In the last, partial
  // round (masked) stages past the end load the last stage again and multiply
  // nothing.
  auto ring_round = [&](int st0, auto masked) {
#pragma unroll
    for (int u = 0; u < ROUND; ++u) {
      const int st = st0 + u;
      wait_vmcnt<(AHEAD - 2) * LOADS>();  // this wave's loads of stage st + 1 are in LDS
      stage_barrier();  // every wave's: stage st + 1 published, stage st - 1 read
      issue(st + AHEAD, (u + AHEAD) % SLOTS);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const int cur = (u * KS + ks) & 1;
        if (ks + 1 < KS)
          read_frags(ring[u % SLOTS], ks + 1, fa[cur ^ 1], fw[cur ^ 1]);
        else
          read_frags(ring[(u + 1) % SLOTS], 0, fa[cur ^ 1], fw[cur ^ 1]);
        if (!decltype(masked)::value || st < stages) {
          if (ks == 0)
            mfma_step(fa[cur], fw[cur], std::true_type{});
          else
            mfma_step(fa[cur], fw[cur], std::false_type{});
        }
      }
    }
  };
  const int full_end = stages - stages % ROUND;
  auto main_loop = [&]() {
    for (int st0 = 0; st0 < full_end; st0 += ROUND) ring_round(st0, std::false_type{});
    if (full_end < stages) ring_round(full_end, std::true_type{});
  };
  main_loop();
  wait_vmcnt<0>();  // no direct load outlives the workgroup

  // Epilogues, in the idle ring. The residual, scatter and QKV epilogues
  // work one row group (the TM/WM rows of a wave) at a time: its waves put
  // their fp32 accumulators in LDS as rows of TN + 4 floats (16 rows per
  // slot; the 4-float pad spreads the four rows a wave store touches over
  // all banks), then every thread takes 8-column pieces of those rows, so
  // each load and store is 16 contiguous bytes per lane.
  if constexpr (MODE == kPartial) {
    // Lane (j4, c16) of block (i, j): rows 16 (RB wm + i) + 4 j4 + r, column
    // 16 (CB wn + j) + c16. Non-temporal: read once, by the next kernel.
    float* const out = ea.x1 + (int64_t)blockIdx.y * M * N;
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = m0 + 16 * (RB * wm + i) + 4 * j4 + r;
        if (m >= M) continue;
        float* const row = out + (int64_t)m * N + n0 + 16 * CB * wn + c16;
#pragma unroll
        for (int j = 0; j < CB; ++j) __builtin_nontemporal_store(acc[i][j][r], row + 16 * j);
      }
    return;
  }
  __syncthreads();  // every wave is done with the ring
  if (tid < TM) {
    if constexpr (MODE == kQkv) {
      ((u32x2_t*)rowv)[tid] = rinfo;
    } else if constexpr (MODE == kSwiglu) {
      const float t = __int_as_float(rowv[tid]) + __int_as_float(rowv[TM + tid]);
      rowv[tid] = __float_as_int(1.0f / sqrtf(t / (float)K + ea.eps));
    } else {
      rowv[tid] = kSwi ? __float_as_int(1.f) : erow;
    }
  }
  __syncthreads();
  constexpr int RG = TM / WM;  // rows of a group
  constexpr int TNP = TN + 4;  // staged row stride (floats)
  static_assert(16 * TNP * 4 <= kSlot * 2, "16 staged rows fit a slot");
  auto st_row = [&](int rq) -> float* {  // row rq of the staged group
    if constexpr (RB == 1) return (float*)s0 + rq * TNP;
    const int g = rq >> 4;
    float* const hi = (float*)(RB > 4 && g > 3 ? s4 : s3);
    return (g == 0 ? (float*)s0 : g == 1 ? (float*)s1 : g == 2 ? (float*)s2 : hi) +
           (rq & 15) * TNP;
  };
  // Accumulator layout: lane (j4, c16) of block (i, j) holds rows
  // 16 (RB wm + i) + 4 j4 + r, r < 4, of column 16 (CB wn + j) + c16.
  auto stage_group = [&](int p) {
    if (wm == p) {
#pragma unroll
      for (int i = 0; i < RB; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          float* const row = st_row(16 * i + 4 * j4 + r);
#pragma unroll
          for (int j = 0; j < CB; ++j) row[16 * (CB * wn + j) + c16] = acc[i][j][r];
        }
    }
  };
  constexpr int kCh = TN / 8;                    // 8-column pieces per row
  constexpr int kPer = (RG * kCh + NT - 1) / NT;  // pieces per thread and group
  if constexpr (MODE == kResid) {
    // x1 = acc + residual row (fp32 out), h = bf16(x1 * gamma) in tile
    // order, and the row's sums of x1^2 per 32 columns: per piece in column
    // order, then the four pieces in order.
    float* const ssp = (float*)ring[RB];
    static_assert(RG * kCh * 4 <= kSlot * 2, "the pieces' sums fit a slot");
    // A thread's residual pieces of all groups and its gamma pieces (the
    // same columns in every group), for clamped pieces (no branch), before
    // the first group: one memory round trip for the epilogue.
    u32x4_t rv[WM][kPer], gv[kPer];
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
      const int it = min(tid + u * NT, RG * kCh - 1);
      const int rq = it / kCh, ch = it - rq * kCh;
      gv[u] = *(const u32x4_t*)(ea.gamma + n0 + 8 * ch);
#pragma unroll
      for (int p = 0; p < WM; ++p)
        rv[p][u] = *(const u32x4_t*)(ea.res_x + (int64_t)rowv[RG * p + rq] * N + n0 + 8 * ch);
    }
#pragma unroll
    for (int p = 0; p < WM; ++p) {
      stage_group(p);
      __syncthreads();
#pragma unroll
      for (int u = 0; u < kPer; ++u) {
        const int it = tid + u * NT;
        if (it >= RG * kCh) continue;
        const int rq = it / kCh, ch = it - rq * kCh;
        const float* a = st_row(rq) + 8 * ch;
        const f32x4_t a0 = *(const f32x4_t*)a, a1 = *(const f32x4_t*)(a + 4);
        float x1[8], y[8];
        float sq = 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          x1[2 * e] = (e < 2 ? a0[2 * e] : a1[2 * e - 4]) + bf16_to_f32(rv[p][u][e] & 0xFFFFu);
          x1[2 * e + 1] = (e < 2 ? a0[2 * e + 1] : a1[2 * e - 3]) + bf16_to_f32(rv[p][u][e] >> 16);
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          sq = fmaf(x1[e], x1[e], sq);
          y[e] = x1[e] * bf16_to_f32(e & 1 ? gv[u][e >> 1] >> 16 : gv[u][e >> 1] & 0xFFFFu);
        }
        ssp[rq * kCh + ch] = sq;
        const int m = m0 + RG * p + rq;
        if (m < M) {
          float* xo = ea.x1 + (int64_t)m * N + n0 + 8 * ch;
          *(f32x4_t*)xo = f32x4_t{x1[0], x1[1], x1[2], x1[3]};
          *(f32x4_t*)(xo + 4) = f32x4_t{x1[4], x1[5], x1[6], x1[7]};
          *(u32x4_t*)(ea.h + tile_off(m, n0 + 8 * ch, N)) =
              u32x4_t{pack_bf16x2(y[0], y[1]), pack_bf16x2(y[2], y[3]), pack_bf16x2(y[4], y[5]),
                      pack_bf16x2(y[6], y[7])};
        }
      }
      __syncthreads();
      constexpr int kGroups = TN / kSsCols;
      for (int t = tid; t < RG * kGroups; t += NT) {
        const int rq = t / kGroups, g = t % kGroups;
        const float* s = ssp + rq * kCh + 4 * g;
        if (m0 + RG * p + rq < M)
          ea.ss_part[(int64_t)(m0 + RG * p + rq) * (N / kSsCols) + n0 / kSsCols + g] =
              ((s[0] + s[1]) + s[2]) + s[3];
      }
      __syncthreads();  // the group's staging and sums are read
    }
  } else if constexpr (MODE == kScatter) {
    // out[out_idx[m]] = bf16(x1 + acc), 8 columns per piece. A thread's x1
    // pieces of all groups are loaded before the first group.
    f32x4_t xv[WM][kPer][2];
#pragma unroll
    for (int p = 0; p < WM; ++p)
#pragma unroll
      for (int u = 0; u < kPer; ++u) {
        const int it = min(tid + u * NT, RG * kCh - 1);
        const int rq = it / kCh, ch = it - rq * kCh;
        const float* xr = ea.x1_in + (int64_t)min(m0 + RG * p + rq, M - 1) * N + n0 + 8 * ch;
        xv[p][u][0] = *(const f32x4_t*)xr;
        xv[p][u][1] = *(const f32x4_t*)(xr + 4);
      }
#pragma unroll
    for (int p = 0; p < WM; ++p) {
      stage_group(p);
      __syncthreads();
#pragma unroll
      for (int u = 0; u < kPer; ++u) {
        const int it = tid + u * NT;
        if (it >= RG * kCh) continue;
        const int rq = it / kCh, ch = it - rq * kCh;
        const int m = m0 + RG * p + rq;
        if (m >= M) continue;
        const float* a = st_row(rq) + 8 * ch;
        const f32x4_t a0 = *(const f32x4_t*)a, a1 = *(const f32x4_t*)(a + 4);
        const f32x4_t y0 = xv[p][u][0] + a0, y1 = xv[p][u][1] + a1;
        *(u32x4_t*)(ea.out + (int64_t)rowv[RG * p + rq] * N + n0 + 8 * ch) =
            u32x4_t{pack_bf16x2(y0[0], y0[1]), pack_bf16x2(y0[2], y0[3]),
                    pack_bf16x2(y1[0], y1[1]), pack_bf16x2(y1[2], y1[3])};
      }
      __syncthreads();  // the group's staging is read
    }
  } else if constexpr (MODE == kQkv) {
    // Column block q < TN/32 holds dims j of pair group q, block TN/32 + q
    // the dims j + 64, so a staged row has both halves of each pair. Per
    // row group: queries and keys in pieces of 8 pairs (rotate-half RoPE with
    // the table's fp32 cos/sin of (position, j), then 16-byte stores of the 8
    // j dims and of the 8 j + 64 dims: q_out [M][Hq][128], or the key tile
    // of the row's cache slot); values (not rotated) as 8-byte runs of four
    // tokens (the value tile order) where four staged rows fill slots
    // 4a .. 4a + 3 of one block, element by element otherwise.
    constexpr int kHd = 128, kTile = kBlockTokens * kHd;
    constexpr int PG = TN / 32;      // pair groups of the tile
    const u32x2_t* const slots = (const u32x2_t*)rowv;
    const int g0 = (n0 / TN) * PG;   // first pair group of the tile
    constexpr int kQK = RG * PG * 2;  // (row, group, 8-pair half) pieces per row group
    constexpr int kQKPer = (kQK + NT - 1) / NT;
    // The (cos, sin) of 8 pairs per piece, one row group ahead.
    f32x4_t cs[2][kQKPer][4];
    auto load_cs = [&](int p, f32x4_t (&dst)[kQKPer][4]) {
#pragma unroll
      for (int u = 0; u < kQKPer; ++u) {
        const int it = min(tid + u * NT, kQK - 1);
        const int c8 = it & 1, q = (it >> 1) % PG, rq = (it >> 1) / PG;
        const int jd0 = 16 * ((g0 + q) & 3) + 8 * c8;
        const f32x4_t* t =
            (const f32x4_t*)(ea.rope + ((int64_t)slots[RG * p + rq].x * (kHd / 2) + jd0) * 2);
#pragma unroll
        for (int v = 0; v < 4; ++v) dst[u][v] = t[v];
      }
    };
    load_cs(0, cs[0]);
#pragma unroll
    for (int p = 0; p < WM; ++p) {
      if (p + 1 < WM) load_cs(p + 1, cs[(p + 1) & 1]);
      stage_group(p);
      __syncthreads();
#pragma unroll
      for (int u = 0; u < kQKPer; ++u) {
        const int it = tid + u * NT;
        if (it >= kQK) continue;
        const int c8 = it & 1, q = (it >> 1) % PG, rq = (it >> 1) / PG;
        const int hh = (g0 + q) >> 2;
        const int m = m0 + RG * p + rq;
        if (m >= M || hh >= ea.Hq + ea.Hkv) continue;  // values below
        const float* lo = st_row(rq) + 16 * q + 8 * c8;
        const float* up = st_row(rq) + 16 * (PG + q) + 8 * c8;
        uint32_t wl[4], wu[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float rl[2], ru[2];
#pragma unroll
          for (int f = 0; f < 2; ++f) {
            const int k = 2 * e + f;  // pair k of the piece
            const float c = cs[p & 1][u][k >> 1][2 * (k & 1)];
            const float sn = cs[p & 1][u][k >> 1][2 * (k & 1) + 1];
            rl[f] = lo[k] * c - up[k] * sn;
            ru[f] = up[k] * c + lo[k] * sn;
          }
          wl[e] = pack_bf16x2(rl[0], rl[1]);
          wu[e] = pack_bf16x2(ru[0], ru[1]);
        }
        const int jd0 = 16 * ((g0 + q) & 3) + 8 * c8;
        const u32x4_t vl = {wl[0], wl[1], wl[2], wl[3]}, vu = {wu[0], wu[1], wu[2], wu[3]};
        if (hh < ea.Hq) {
          bf16_t* dst = ea.q_out + ((int64_t)m * ea.Hq + hh) * kHd + jd0;
          *(u32x4_t*)dst = vl;
          *(u32x4_t*)(dst + 64) = vu;
        } else {
          const u32x2_t sl = slots[RG * p + rq];
          const int slot = (int)sl.x % kBlockTokens;
          bf16_t* tile = ea.k_cache + ((int64_t)(int)sl.y * ea.Hkv + (hh - ea.Hq)) * kTile;
          *(u32x4_t*)(tile + k_tile_offset(slot, jd0)) = vl;
          *(u32x4_t*)(tile + k_tile_offset(slot, jd0 + 64)) = vu;
        }
      }
      // Values: (row quad, group, 32 dims), the dim fastest.
      constexpr int kV = (RG / 4) * PG * 32;
      for (int it = tid; it < kV; it += NT) {
        const int d32 = it & 31, q = (it >> 5) % PG, quad = (it >> 5) / PG;
        const int hh = (g0 + q) >> 2;
        if (hh < ea.Hq + ea.Hkv) continue;  // queries and keys above
        const int dim = 64 * (d32 >> 4) + 16 * ((g0 + q) & 3) + (d32 & 15);
        const int col = 16 * ((d32 >> 4) * PG + q) + (d32 & 15);  // staged column
        const int lr0 = RG * p + 4 * quad;
        bf16_t* const vbase = ea.v_cache + (int64_t)(hh - ea.Hq - ea.Hkv) * kTile;
        uint32_t e4[4];
        u32x2_t sl[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          e4[e] = f32_to_bf16(st_row(4 * quad + e)[col]);
          sl[e] = slots[lr0 + e];
        }
        const int t0 = (int)sl[0].x % kBlockTokens;
        bool run = m0 + lr0 + 3 < M && t0 % 4 == 0;
#pragma unroll
        for (int e = 1; e < 4; ++e)
          run = run && sl[e].y == sl[0].y && (int)sl[e].x % kBlockTokens == t0 + e;
        if (run) {
          *(u32x2_t*)(vbase + (int64_t)(int)sl[0].y * ea.Hkv * kTile + v_tile_offset(t0, dim)) =
              u32x2_t{e4[0] | (e4[1] << 16), e4[2] | (e4[3] << 16)};
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (m0 + lr0 + e < M)
              vbase[(int64_t)(int)sl[e].y * ea.Hkv * kTile +
                    v_tile_offset((int)sl[e].x % kBlockTokens, dim)] = (bf16_t)e4[e];
        }
      }
      __syncthreads();  // the group's staging is read
    }
  } else {
    // h = silu(gate) * up of outputs n0/2 + 8 (CB wn + j) + c16 % 8, 16 rows
    // at a time through a buffer of this wave's own, then in 16-byte pieces
    // of 8 outputs, 16 rows (256 contiguous bytes of tile order) side by side.
    constexpr int kWO = CB * 8 + 8;  // outputs of a wave and row, padded for the banks
    static_assert(NW * 16 * kWO <= kSlot, "the waves' output buffers fit a slot");
    const int F = N / 2;
    bf16_t* const mine = s0 + wv * 16 * kWO;
    const bool up = c16 >= 8;
    const int row2 = 4 * j4 + (up ? 2 : 0);  // this lane's two rows of a block
#pragma unroll
    for (int i = 0; i < RB; ++i) {
      const int rb = 16 * (RB * wm + i);
      const float rs0 = __int_as_float(rowv[rb + row2]), rs1 = __int_as_float(rowv[rb + row2 + 1]);
#pragma unroll
      for (int j = 0; j < CB; ++j) {
        float y[2];
        swiglu_quad(acc[i][j], rs0, rs1, y);
        mine[row2 * kWO + 8 * j + (c16 & 7)] = (bf16_t)f32_to_bf16(y[0]);
        mine[(row2 + 1) * kWO + 8 * j + (c16 & 7)] = (bf16_t)f32_to_bf16(y[1]);
      }
      wave_lds_order();  // the rows just written, by this wave's other lanes
#pragma unroll
      for (int c0 = 0; c0 < 16 * CB; c0 += 64) {
        const int row = (c0 + lane) & 15, pc = (c0 + lane) >> 4;
        if (16 * CB % 64 == 0 || pc < CB) {
          const u32x4_t v = *(const u32x4_t*)(mine + row * kWO + 8 * pc);
          const int m = m0 + rb + row, o = n0 / 2 + 8 * (CB * wn + pc);
          const bool rows = MODE == kSwigluPlain && ea.h_rows;
          if (m < M) *(u32x4_t*)(ea.h + (rows ? (int64_t)m * F + o : tile_off(m, o, F))) = v;
        }
      }
      wave_lds_order();  // read before the next block overwrites them
    }
  }
}

// Persistent SwiGLU variant (gate/up projection with RMSNorm_2 folded in):
// one workgroup per CU keeps a row tile and walks a list of column tiles, so
// the direct-load ring streams on across tile boundaries (the next tile's
// first stages load while a tile's epilogue runs, and no workgroup starts
// cold after the first), and the rows' 1/rms are taken once. Same main loop,
// stage order and epilogue arithmetic as gemm_prefill_kernel's SwiGLU mode,
// so every output is bit-identical to it.
//   * Grid: 256 workgroups, 32 per XCD (blockIdx % 8). Workgroup k of XCD x
//     takes row tile k % tiles_m and the column tiles
//     x + 8 (k / tiles_m + ng s), s = 0, 1, ..., ng = 32 / tiles_m: at each
//     step the workgroups of one XCD share ng W tiles in its L2, each read by
//     tiles_m of them.
//   * The ring's slots are in use during an epilogue, so each wave stages its
//     SwiGLU outputs through a private 16-row buffer and writes them as
//     16-byte tile-order pieces. After an epilogue all vector memory
//     operations are waited for: the partial wait counts of the ring assume
//     that only its loads are outstanding.
// A tile is a whole number of unrolled rounds (K / (32 KS) % ROUND == 0) and
// the row tiles divide 32 (host checks).
template <class T>
__global__ __launch_bounds__(T::NT) void gemm_prefill_swiglu_persistent_kernel(
    const bf16_t* __restrict__ A, const bf16_t* __restrict__ W, int M, int F, int K,
    bf16_t* __restrict__ H, const float* __restrict__ ss_in, float eps) {
  constexpr int TM = T::TM, TN = T::TN, WM = T::WM, KS = T::KS, RB = T::RB, CB = T::CB;
  constexpr int NW = T::NW, NT = T::NT, AB = T::AB, NB = T::NB, LOADS = T::LOADS;
  constexpr int SLOTS = T::SLOTS, AHEAD = T::AHEAD, ROUND = T::ROUND;
  constexpr int kSlot = NB * 512;  // elements
  constexpr int kWO = CB * 8 + 8;  // outputs of a wave and row, padded for the banks
  static_assert(AHEAD < ROUND && NT >= 2 * TM && KS == 1, "tile shape");
  __shared__ __attribute__((aligned(16))) bf16_t s0[kSlot], s1[kSlot], s2[kSlot], s3[kSlot],
      s4[kSlot], s5[kSlot], s6[kSlot], s7[kSlot];
  __shared__ __attribute__((aligned(16))) bf16_t spare[512];
  __shared__ __attribute__((aligned(16))) bf16_t stg[NW][16 * kWO];  // per-wave output rows
  __shared__ float rn[2 * TM];  // the rows' half sums, then 1/rms
  bf16_t* const ring[8] = {s0, s1, s2, s3, s4, s5, s6, s7};

  const int tiles_m = (M + TM - 1) / TM;
  const int tiles_n = 2 * F / TN;
  const int x = blockIdx.x % kNXCDs, kx = blockIdx.x / kNXCDs;
  const int ng = 32 / tiles_m;
  const int n_first = x + kNXCDs * (kx / tiles_m), n_step = kNXCDs * ng;
  const int tiles = n_first < tiles_n ? (tiles_n - 1 - n_first) / n_step + 1 : 0;
  if (tiles == 0) return;  // the whole workgroup leaves
  const int m0 = (kx % tiles_m) * TM;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wv % WM, wn = wv / WM;
  const int c16 = lane & 15, j4 = lane >> 4;
  const int stages = K / 32;

  // Blocks as in gemm_prefill_kernel; the W blocks of later tiles are n_step
  // tiles, a fixed number of blocks, further.
  const int64_t blk_elems = (int64_t)(K / 32) * 512;
  const int64_t w_step = (int64_t)n_step * (TN / 16) * blk_elems;
  // (The first AB / NW loads of a wave are A blocks.)
  static_assert(T::AEVEN && AB < NB, "whole loads of A");
  constexpr int ALOADS = AB / NW;
  const char* src[LOADS];
#pragma unroll
  for (int i = 0; i < LOADS; ++i) {
    const int t = T::source(wv, i), q = t >> 2;
    const int blk = i < ALOADS ? min((m0 >> 4) + q, (M - 1) >> 4) : n_first * (TN / 16) + q - AB;
    src[i] = (const char*)((i < ALOADS ? A : W) + blk * blk_elems) + (t & 3) * 256 +
             lane * T::bytes(i);
  }
  // Stage st of the tile whose W blocks are w_off past the first tile's.
  // The stage offsets pass through empty asm statements: the compiler then
  // forms each address where it is used, instead of keeping precomputed
  // addresses of the unrolled stages (and of the prologue's, which the last
  // round's next-tile loads repeat) in registers.
  auto issue = [&](int64_t w_off, int st, int slot) {
    int64_t oa = (int64_t)st * 1024, ow = 2 * w_off + (int64_t)st * 1024;
    asm volatile("" : "+s"(oa), "+s"(ow));
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
      bf16_t* dst = ring[slot] + T::source(wv, i) * 128;
      if (T::SPARE && i == LOADS - 1) dst = T::block(wv, i) < NB ? dst : spare;
      const void* p = (const void*)(src[i] + (i < ALOADS ? oa : ow));
      if (T::bytes(i) == 4)
        __builtin_amdgcn_global_load_lds(p, (lds_void_t*)dst, 4, 0, 0);
      else
        __builtin_amdgcn_global_load_lds(p, (lds_void_t*)dst, 16, 0, 0);
    }
  };

  f32x4_t acc[RB][CB];
  auto read_frags = [&](const bf16_t* s, bf16x8_t* a, bf16x8_t* w) {
#pragma unroll
    for (int i = 0; i < RB; ++i)
      a[i] = __builtin_bit_cast(bf16x8_t, *(const u32x4_t*)(s + (wm * RB + i) * 512 + lane * 8));
#pragma unroll
    for (int j = 0; j < CB; ++j)
      w[j] = __builtin_bit_cast(bf16x8_t,
                                *(const u32x4_t*)(s + (AB + wn * CB + j) * 512 + lane * 8));
  };
  auto mfma_step = [&](const bf16x8_t* a, const bf16x8_t* w) {
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
      for (int j = 0; j < CB; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], w[j], acc[i][j], 0, 0, 0);
    __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);      // MFMA
    __builtin_amdgcn_sched_group_barrier(0x020, LOADS, 0);  // VMEM read
    for (int g = 0; g < RB + CB; ++g) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);  // DS read
    }
    __builtin_amdgcn_sched_group_barrier(0x008, RB * CB - 4 - RB - CB, 0);
  };

  {
    const int m = min(m0 + tid % TM, M - 1), h = (tid / TM) & 1, n4 = K / (4 * kSsCols);
    SsPart sp;
    ss_load(sp, ss_in, m, h, n4);
#pragma unroll
    for (int st = 0; st < AHEAD; ++st) issue(0, st, st);
    const float t = ss_half(sp, ss_in, m, h, n4);
    if (tid < 2 * TM) rn[tid] = t;
    __syncthreads();
    const float r = tid < TM ? 1.0f / sqrtf((rn[tid] + rn[TM + tid]) / (float)K + eps) : 0.f;
    __syncthreads();
    if (tid < TM) rn[tid] = r;
  }
  __syncthreads();  // stage 0 and the 1/rms are in LDS
  bf16x8_t fa[2][RB], fw[2][CB];
  read_frags(ring[0], fa[0], fw[0]);
  // One unrolled round: stages st0 .. st0 + ROUND - 1 of the tile at w_off.
  // Only in a tile's last round do the loads run into the next tile (at
  // w_next; after the last tile, that tile again: loaded, never multiplied),
  // and that round leaves the next tile's first fragments unread, so they are
  // not held through the epilogue.
  auto ring_round = [&](int st0, int64_t w_off, int64_t w_next, auto last) {
#pragma unroll
    for (int u = 0; u < ROUND; ++u) {
      wait_vmcnt<(AHEAD - 2) * LOADS>();
      stage_barrier();
      if (!decltype(last)::value || u + AHEAD < ROUND)
        issue(w_off, st0 + u + AHEAD, (u + AHEAD) % SLOTS);
      else
        issue(w_next, u + AHEAD - ROUND, (u + AHEAD) % SLOTS);
      if (!decltype(last)::value || u + 1 < ROUND)
        read_frags(ring[(u + 1) % SLOTS], fa[(u + 1) & 1], fw[(u + 1) & 1]);
      mfma_step(fa[u & 1], fw[u & 1]);
    }
  };
  bf16_t* const mine = stg[wv];
  const bool up = c16 >= 8;
  const int row2 = 4 * j4 + (up ? 2 : 0);  // this lane's two rows of a block
  for (int s = 0; s < tiles; ++s) {
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
      for (int j = 0; j < CB; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    if (s > 0) {
      // After an epilogue: every vector memory operation done (its stores
      // too, which the ring's partial wait counts do not allow for), then
      // the tile's first stage is published and read.
      wait_vmcnt<0>();
      stage_barrier();
      read_frags(ring[0], fa[0], fw[0]);
    }
    const int64_t w_off = (int64_t)s * w_step;
    const int64_t w_next = s + 1 < tiles ? w_off + w_step : w_off;
    for (int st0 = 0; st0 + ROUND < stages; st0 += ROUND)
      ring_round(st0, w_off, w_off, std::false_type{});
    ring_round(stages - ROUND, w_off, w_next, std::true_type{});
    // Epilogue as in gemm_prefill_kernel. tile_off(m, o0 + 8 pc, F) for
    // m = mr + row (mr a multiple of 16) splits into a wave-uniform block
    // offset and a lane part, so the address is a scalar base plus a 32-bit
    // offset.
    const int o0 = (n_first + n_step * s) * (TN / 2) + CB * 8 * wn;
#pragma unroll
    for (int i = 0; i < RB; ++i) {
      const int rb = 16 * (RB * wm + i);
      const float rs0 = rn[rb + row2], rs1 = rn[rb + row2 + 1];
#pragma unroll
      for (int j = 0; j < CB; ++j) {
        float y[2];
        swiglu_quad(acc[i][j], rs0, rs1, y);
        mine[row2 * kWO + 8 * j + (c16 & 7)] = (bf16_t)f32_to_bf16(y[0]);
        mine[(row2 + 1) * kWO + 8 * j + (c16 & 7)] = (bf16_t)f32_to_bf16(y[1]);
      }
      wave_lds_order();  // the rows just written, by this wave's other lanes
      const int mr = m0 + rb;
      bf16_t* const hb = H + ((int64_t)(mr >> 4) * (F >> 5) + (o0 >> 5)) * 512;
#pragma unroll
      for (int c0 = 0; c0 < 16 * CB; c0 += 64) {
        const int row = (c0 + lane) & 15, pc = (c0 + lane) >> 4;
        const int kk = (o0 & 31) + 8 * pc;
        if (16 * CB % 64 == 0 || pc < CB) {
          const u32x4_t v = *(const u32x4_t*)(mine + row * kWO + 8 * pc);
          if (mr + row < M)
            *(u32x4_t*)(hb + ((kk >> 5) * 512 + ((kk & 31) >> 3) * 128 + row * 8)) = v;
        }
      }
      wave_lds_order();  // read before the next block overwrites them
    }
  }
  wait_vmcnt<0>();  // no direct load outlives the workgroup
}

// The tile shapes choose_tile picks from (gemm_prefill_swiglu.hip). T64x128 is
// small enough for two workgroups per CU; the others fill a CU's LDS with
// their ring.
using T256x224 = Tile<256, 224, 4, 2, 1, 5>;
using T256x192 = Tile<256, 192, 4, 2, 1, 5>;
using T256x160 = Tile<256, 160, 4, 2, 1, 6>;
using T256x128 = Tile<256, 128, 4, 2, 1, 6>;
using T192x256 = Tile<192, 256, 4, 2, 1, 5>;
using T160x256 = Tile<160, 256, 2, 4, 1, 6>;
using T128x256 = Tile<128, 256, 4, 2, 1, 6>;
using T128x160 = Tile<128, 160, 4, 2, 1, 6>;
using T128x128 = Tile<128, 128, 4, 2, 2, 4>;
using T128x64 = Tile<128, 64, 4, 2, 2, 6>;
using T64x160 = Tile<64, 160, 4, 2, 1, 8>;
using T64x128 = Tile<64, 128, 2, 2, 1, 6>;
using T64x64 = Tile<64, 64, 2, 2, 2, 8>;
using T64x32 = Tile<64, 32, 4, 1, 4, 6>;
using T32x32 = Tile<32, 32, 2, 2, 4, 8>;
enum TileId {
  k256x224, k256x192, k256x160, k256x128, k192x256, k160x256, k128x256, k128x160, k128x128,
  k128x64, k64x160, k64x128, k64x64, k64x32, k32x32, kTileCount
};
// The shape for an [M] x [N] x [K] product, run as S products of K / S; -1 if
// none divides N.
int choose_tile(int M, int N, int K, int S, int num_cus);

template <class T, int MODE>
hipError_t launch_one(const uint16_t* A, const uint16_t* W, int M, int N, int K,
                      int S, const PrefillEpiArgs& ea, hipStream_t st) {
  if (N % T::TN != 0 || S < 1 || K % (32 * T::KS * S) != 0) return hipErrorInvalidValue;
  const int64_t grid = (int64_t)((M + T::TM - 1) / T::TM) * (N / T::TN);
  if (grid > 0x7fffffff) return hipErrorInvalidValue;
  COCO_LAUNCH((gemm_prefill_kernel<T, MODE>), dim3((unsigned)grid, S), dim3(T::NT), 0, st,
              (const bf16_t*)A, (const bf16_t*)W, M, N, K, ea);
  return hipGetLastError();
}

template <int MODE>
hipError_t launch_mode(const uint16_t* A, const uint16_t* W, int M, int N, int K, int S,
                       const PrefillEpiArgs& ea, int num_cus, hipStream_t st) {
  switch (choose_tile(M, N, K, S, num_cus)) {
    case k256x224: return launch_one<T256x224, MODE>(A, W, M, N, K, S, ea, st);
    case k256x192: return launch_one<T256x192, MODE>(A, W, M, N, K, S, ea, st);
    case k256x160: return launch_one<T256x160, MODE>(A, W, M, N, K, S, ea, st);
    case k256x128: return launch_one<T256x128, MODE>(A, W, M, N, K, S, ea, st);
    case k192x256: return launch_one<T192x256, MODE>(A, W, M, N, K, S, ea, st);
    case k160x256: return launch_one<T160x256, MODE>(A, W, M, N, K, S, ea, st);
    case k128x256: return launch_one<T128x256, MODE>(A, W, M, N, K, S, ea, st);
    case k128x160: return launch_one<T128x160, MODE>(A, W, M, N, K, S, ea, st);
    case k128x128: return launch_one<T128x128, MODE>(A, W, M, N, K, S, ea, st);
    case k128x64: return launch_one<T128x64, MODE>(A, W, M, N, K, S, ea, st);
    case k64x160: return launch_one<T64x160, MODE>(A, W, M, N, K, S, ea, st);
    case k64x128: return launch_one<T64x128, MODE>(A, W, M, N, K, S, ea, st);
    case k64x64: return launch_one<T64x64, MODE>(A, W, M, N, K, S, ea, st);
    case k64x32: return launch_one<T64x32, MODE>(A, W, M, N, K, S, ea, st);
    case k32x32: return launch_one<T32x32, MODE>(A, W, M, N, K, S, ea, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace prefill
}  // namespace coco
