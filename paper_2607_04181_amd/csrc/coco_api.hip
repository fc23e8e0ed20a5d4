// C ABI of the layer-replica hot path: handle, workspace, argument checks and
// the launch sequence of one decoder layer / one span of layers.
#include <math.h>
#include <stdarg.h>
#include <stdio.h>
#include <type_traits>

#include <mutex>
#include <vector>

#include "../../include/coco.h"
#include "common.h"
#include "kernels.h"

using namespace coco;

namespace {

// Message of the last failure on this thread (a fixed buffer: reporting an
// error allocates nothing).
thread_local char g_err[512];

int fail(int code, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof g_err, fmt, ap);
  va_end(ap);
  return code;
}

#define HIPCHK(expr)                                                                  \
  do {                                                                                \
    hipError_t e_ = (expr);                                                           \
    if (e_ != hipSuccess) return fail(COCO_EHIP, "%s: %s", #expr, hipGetErrorString(e_)); \
  } while (0)

}  // namespace

// Per-call buffers of the launch sequence, carved out of one region (the
// handle's workspace, or the static scratch array of the no-alloc entry
// point).
struct Work {
  void *x = nullptr, *h = nullptr, *q = nullptr, *o = nullptr, *h2 = nullptr, *u = nullptr;
  float *x1 = nullptr, *part = nullptr, *attn_o = nullptr, *attn_ml = nullptr;
  // Row sums of squares per K-slice (decode QKV with RMSNorm_1 folded in). The
  // prefill O projection's, per 32 columns ([rows][d / 32]), are in `part`,
  // which prefill has no other use for.
  float* ss = nullptr;
  int32_t* split_off = nullptr;  // decode attention work list
  int32_t* row_info = nullptr;   // prefill row slots [rows][2] (position, cache block)
};

struct coco_layer {
  coco_layer_config cfg;
  std::vector<coco_layer_weights> layers;
  int device = 0;
  int num_cus = 0;  // compute units of `device` (persistent grid sizes)
  bool validate = false;
  char* ws = nullptr;
  size_t ws_bytes = 0;
  // bf16: the library's tile-order copies of every layer's four weight
  // matrices (layers[l].w_* point into it after init).
  char* packed = nullptr;
  size_t packed_bytes = 0;
  Work w;  // the workspace's per-call buffers, sized for max_rows
  double* inv_freq = nullptr;
  float* rope = nullptr;  // RoPE table [rope_rows][head_dim / 2] (cos, sin)
  int rope_rows = 0;      // positions the configuration admits
  size_t act_rows_bytes[7] = {};
  int max_splits = 0;
  int dec_rows = 0;
  // Which of the last regular call's activations h, o, h2, u are in tile
  // order (act_layout), read back row-major by coco_layer_workspace, and
  // that call's rows.
  bool ws_tiled[7] = {};
  int last_rows = 0;
  // Per-kernel timing (benchmark mode).
  bool timing = false;
  std::vector<hipEvent_t> ev;  // pairs: start, stop
  std::vector<int> ev_kind;    // kind of each recorded pair
  bool ev_overflow = false;
  hipStream_t ev_stream = nullptr;
  // Recorded at the end of every call made outside graph capture.
  hipEvent_t done = nullptr;
};

namespace coco {
LaunchEvents& launch_events() {
  thread_local LaunchEvents le;
  return le;
}
}  // namespace coco

namespace {

constexpr int kTimingPairs = 4096;

// Times the one kernel launched in its scope when timing is on: the launch
// timestamps the event pair at the kernel's own start and end. A scope that
// launches nothing (empty work) records an empty interval.
struct KernelTimer {
  coco_layer* H;
  int kind;
  int pair = -1;
  KernelTimer(coco_layer* h, int k, hipStream_t st) : H(h), kind(k) {
    if (!H->timing) return;
    const int n = (int)H->ev_kind.size();
    if (n >= kTimingPairs) {
      H->ev_overflow = true;
      return;
    }
    pair = n;
    H->ev_kind.push_back(kind);
    H->ev_stream = st;
    coco::launch_events() = coco::LaunchEvents{H->ev[2 * pair], H->ev[2 * pair + 1]};
  }
  ~KernelTimer() {
    if (pair < 0) return;
    coco::LaunchEvents& le = coco::launch_events();
    if (le.start != nullptr) {
      (void)hipEventRecord(le.start, H->ev_stream);
      (void)hipEventRecord(le.stop, H->ev_stream);
      le = coco::LaunchEvents{};
    }
  }
};

}  // namespace

namespace {

size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

int elem_bytes(int dtype) { return dtype == COCO_BF16 ? 2 : 4; }

// Fp32 partials [splits][rows][N] that `part` counts: the decode GEMMs'
// K-slices, and at least one per 8192 k (up to four) where N <= 12,032. The
// prefill and fp32 GEMMs write none; the floor and fp32's one split keep the
// size of a call's buffers, and with it which calls the no-alloc entry point
// takes.
int part_splits(const coco_layer_config& c, int N, int K) {
  if (c.dtype != COCO_BF16) return 1;
  int S = 1;
  if ((N + 255) / 256 < 48) {
    S = (K + 4096) / 8192;
    S = S < 1 ? 1 : S > 4 ? 4 : S;
    while (S > 1 && (K / 128) % S != 0) --S;
  }
  const int a = skinny_plan(N, K).S;
  return a > S ? a : S;
}

// Lays out the per-call buffers for `rows` call rows and `dec_seqs` decode
// sequences from `base`, each piece 256-byte aligned, and returns the bytes
// they take (base == nullptr: sizes only; `w` may then be null). *used: the
// bytes that must be there; an fp32 layer touches nothing past x1.
size_t carve_work(const coco_layer_config& c, int64_t rows, int64_t dec_seqs, int max_splits,
                  char* base, Work* w, size_t* used = nullptr) {
  const int eb = elem_bytes(c.dtype);
  const int64_t R = rows, d = c.d_model, F = c.d_ffn;
  const int64_t qd = (int64_t)c.n_q_heads * c.head_dim;
  const int64_t nqkv = (int64_t)(c.n_q_heads + 2 * c.n_kv_heads) * c.head_dim;
  int64_t part_elems = 0;
  const int64_t shapes[4][2] = {{nqkv, d}, {d, qd}, {2 * F, d}, {d, F}};
  for (auto& sh : shapes) {
    const int64_t e = (int64_t)part_splits(c, (int)sh[0], (int)sh[1]) * R * sh[0];
    if (e > part_elems) part_elems = e;
  }
  const bool bf = c.dtype == COCO_BF16;
  // The prefill GEMMs' A operands (h, o, h2, u) are in tile order, read in
  // whole 16-row groups: room for the rows rounded up to 16.
  const int64_t R16 = (R + 15) / 16 * 16;
  const size_t sizes[13] = {
      align256(R * d * eb),      // x
      align256(R16 * d * eb),    // h
      align256(R * qd * eb),     // q
      align256(R16 * qd * eb),   // o
      align256(R16 * d * eb),    // h2
      align256(R16 * F * eb),    // u
      align256(R * d * 4),     // x1
      align256(part_elems * 4),  // part
      bf ? align256((size_t)dec_seqs * c.n_q_heads * max_splits * 128 * 4) : 0,  // attn_o
      bf ? align256((size_t)dec_seqs * c.n_q_heads * max_splits * 2 * 4) : 0,    // attn_ml
      align256((size_t)(2 * dec_seqs + 2) * 4),  // split_off (decode attention work list)
      // ss: per-slice row sums of squares (decode QKV, at most 16 K-slices)
      align256((size_t)32 * R * 4),
      align256(R * 8)};  // row_info
  size_t off[13], total = 0;
  for (int i = 0; i < 13; ++i) {
    off[i] = total;
    total += sizes[i];
  }
  if (used) *used = bf ? total : off[7];
  if (base && w) {
    w->x = base + off[0];
    w->h = base + off[1];
    w->q = base + off[2];
    w->o = base + off[3];
    w->h2 = base + off[4];
    w->u = base + off[5];
    w->x1 = (float*)(base + off[6]);
    if (!bf) return total;
    w->part = (float*)(base + off[7]);
    w->attn_o = (float*)(base + off[8]);
    w->attn_ml = (float*)(base + off[9]);
    w->split_off = (int32_t*)(base + off[10]);
    w->ss = (float*)(base + off[11]);
    w->row_info = (int32_t*)(base + off[12]);
  }
  return total;
}

int check_config(const coco_layer_config* c) {
  if (!c) return fail(COCO_EINVAL, "config is NULL");
  if (c->d_model <= 0 || c->n_q_heads <= 0 || c->n_kv_heads <= 0 || c->head_dim <= 0 ||
      c->d_ffn <= 0 || c->n_layers <= 0 || c->max_rows <= 0 || c->max_seqs <= 0 ||
      c->max_blocks_per_seq <= 0)
    return fail(COCO_EINVAL, "config sizes must be positive");
  if (c->block_size != kBlockTokens) return fail(COCO_EINVAL, "block_size must be 16");
  if (c->max_blocks_per_seq > (1 << 24))
    return fail(COCO_EINVAL, "max_blocks_per_seq must be <= 2^24 (positions fit in int32)");
  if (c->n_q_heads % c->n_kv_heads) return fail(COCO_EINVAL, "n_q_heads %% n_kv_heads != 0");
  if (!(c->rms_eps >= 0.f) || !(c->rope_theta > 0.f))
    return fail(COCO_EINVAL, "rms_eps must be >= 0 and rope_theta > 0");
  if (c->dtype == COCO_BF16) {
    if (c->head_dim != 128) return fail(COCO_EINVAL, "bf16 path needs head_dim == 128");
    if (c->n_q_heads / c->n_kv_heads > 16)
      return fail(COCO_EINVAL, "bf16 path needs n_q_heads / n_kv_heads <= 16");
    if (c->d_model % 128 || c->d_ffn % 128)
      return fail(COCO_EINVAL, "bf16 path needs d_model and d_ffn multiples of 128");
    if (c->d_model > 16384) return fail(COCO_EINVAL, "bf16 path needs d_model <= 16384");
    // The decode partition merge keeps two floats per 256-token partition in LDS.
    if (!attn_combine_fits(decode_max_splits(c->max_blocks_per_seq)))
      return fail(COCO_EINVAL,
                  "max_blocks_per_seq = %d: its %d decode partitions exceed what the partition "
                  "merge holds in LDS (max_blocks_per_seq <= %d)",
                  c->max_blocks_per_seq, decode_max_splits(c->max_blocks_per_seq),
                  (65536 - 64) / 8 * (kDecodeSplit / kBlockTokens));
  } else if (c->dtype == COCO_F32) {
    if (c->head_dim % 32 || c->head_dim > 256)
      return fail(COCO_EINVAL, "fp32 path needs head_dim a multiple of 32, <= 256");
    if (c->d_model % 4 || c->d_ffn % 4 || c->d_model > 16384)
      return fail(COCO_EINVAL, "fp32 path needs d_model, d_ffn multiples of 4, d_model <= 16384");
  } else {
    return fail(COCO_EINVAL, "unknown dtype %d", c->dtype);
  }
  return COCO_OK;
}

}  // namespace

// ----------------------------------------------------------------------------
// Static scratch of the no-alloc entry point (coco_layer_forward_noalloc).
// Every GPU the library runs on holds its own copy of this array from module
// load until the process ends. In host code `scratch` names a host-side
// stand-in, not a device address: the device address of the current device's
// copy comes from hipGetSymbolAddress, taken once per device in
// coco_layer_init and kept in g_scratch; only that address is ever passed to
// kernels.
// ----------------------------------------------------------------------------
namespace {

constexpr size_t kScratchBytes = (size_t)64 << 20;
static __device__ __align__(256) char scratch[kScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
char* g_scratch[kMaxDevices] = {};

// With `dev` current: look up and keep this device's scratch address.
int scratch_setup(int dev) {
  if (dev < 0 || dev >= kMaxDevices)
    return fail(COCO_EINVAL, "device %d beyond the %d the library tracks", dev, kMaxDevices);
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch[dev] != nullptr) return COCO_OK;
  void* p = nullptr;
  const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
  if (e != hipSuccess || p == nullptr) {
    (void)hipGetLastError();
    return fail(COCO_EHIP, "hipGetSymbolAddress(scratch) on device %d: %s", dev,
                hipGetErrorString(e));
  }
  g_scratch[dev] = (char*)p;
  return COCO_OK;
}

char* scratch_ptr(int dev) {
  if (dev < 0 || dev >= kMaxDevices) return nullptr;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  return g_scratch[dev];
}

}  // namespace

namespace {

// bf16: copy every layer's weight matrices into one library-owned buffer in
// tile order (the layout the bf16 GEMM kernels read) and point the handle's
// layer structs at the copies. The caller's matrices are not read again.
int pack_weights(coco_layer* H) {
  const coco_layer_config& c = H->cfg;
  if (c.dtype != COCO_BF16) return COCO_OK;
  const int64_t d = c.d_model, F = c.d_ffn, qd = (int64_t)c.n_q_heads * c.head_dim;
  const int64_t nqkv = qd + 2LL * c.n_kv_heads * c.head_dim;
  struct Mat {
    int64_t N, K;
  };
  const Mat mats[4] = {{nqkv, d}, {d, qd}, {2 * F, d}, {d, F}};
  size_t per_layer = 0;
  for (const Mat& m : mats) per_layer += align256((size_t)(m.N * m.K * 2));
  H->packed_bytes = per_layer * c.n_layers;
  if (hipMalloc((void**)&H->packed, H->packed_bytes) != hipSuccess) {
    (void)hipGetLastError();
    H->packed = nullptr;
    return fail(COCO_ENOMEM, "tile-order weight copies of %zu bytes do not fit", H->packed_bytes);
  }
  char* p = H->packed;
  for (int l = 0; l < c.n_layers; ++l) {
    coco_layer_weights& w = H->layers[l];
    const void** src[4] = {&w.w_qkv, &w.w_o, &w.w_gate_up, &w.w_down};
    for (int i = 0; i < 4; ++i) {
      const hipError_t e =
          i == 2 ? launch_pack_gate_up((const uint16_t*)*src[i], c.d_ffn, c.d_model,
                                       (uint16_t*)p, nullptr)
                 : launch_pack_tile_order((const uint16_t*)*src[i], (int)mats[i].N,
                                          (int)mats[i].K, (uint16_t*)p, nullptr);
      if (e != hipSuccess) {
        (void)hipGetLastError();
        (void)hipFree(H->packed);
        H->packed = nullptr;
        return fail(COCO_EHIP, "weight packing failed (layer %d)", l);
      }
      *src[i] = p;
      p += align256((size_t)(mats[i].N * mats[i].K * 2));
    }
  }
  if (hipDeviceSynchronize() != hipSuccess) {
    (void)hipGetLastError();
    (void)hipFree(H->packed);
    H->packed = nullptr;
    return fail(COCO_EHIP, "weight packing failed");
  }
  return COCO_OK;
}

}  // namespace

extern "C" {

const char* coco_last_error(void) { return g_err; }

int coco_version(void) { return 100; }

int coco_layer_init(const coco_layer_config* cfg, const coco_layer_weights* layers,
                    coco_layer_t* out) {
  if (!out) return fail(COCO_EINVAL, "out is NULL");
  *out = nullptr;
  int rc = check_config(cfg);
  if (rc) return rc;
  if (!layers) return fail(COCO_EINVAL, "layers is NULL");
  const coco_layer_config& c = *cfg;
  for (int l = 0; l < c.n_layers; ++l) {
    const coco_layer_weights& w = layers[l];
    if (!w.w_qkv || !w.w_o || !w.w_gate_up || !w.w_down || !w.gamma_attn || !w.gamma_mlp ||
        !w.k_cache || !w.v_cache)
      return fail(COCO_EINVAL, "layer %d has a NULL weight or cache pointer", l);
    if (w.num_blocks <= 0) return fail(COCO_EINVAL, "layer %d: num_blocks must be > 0", l);
    // The kernels read weights, gains and cache tiles with 16-byte vector loads.
    const void* ptrs[8] = {w.w_qkv, w.w_o, w.w_gate_up, w.w_down, w.gamma_attn, w.gamma_mlp,
                           w.k_cache, w.v_cache};
    for (const void* ptr : ptrs)
      if ((uintptr_t)ptr % 16) return fail(COCO_EINVAL, "layer %d: a weight or cache pointer is not 16-byte aligned", l);
  }

  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      cus <= 0)
    return fail(COCO_EHIP, "cannot query the current device");
  if ((rc = scratch_setup(dev))) return rc;
  coco_layer* H = new coco_layer();
  H->cfg = c;
  H->layers.assign(layers, layers + c.n_layers);
  H->device = dev;
  H->num_cus = cus;

  const int eb = elem_bytes(c.dtype);
  const int64_t R = c.max_rows, d = c.d_model, F = c.d_ffn;
  const int64_t qd = (int64_t)c.n_q_heads * c.head_dim;
  H->max_splits = decode_max_splits(c.max_blocks_per_seq);
  H->dec_rows = c.max_rows < c.max_seqs ? c.max_rows : c.max_seqs;

  // Per-call buffers for max_rows rows, then the handle's constants: RoPE
  // inverse frequencies and (bf16) the RoPE table of the fused prefill QKV
  // epilogue.
  H->rope_rows = c.dtype == COCO_BF16 ? c.max_blocks_per_seq * kBlockTokens : 0;
  size_t work_bytes = 0;
  carve_work(c, R, H->dec_rows, H->max_splits, nullptr, nullptr, &work_bytes);
  const size_t freq_bytes = align256((size_t)(c.head_dim / 2) * 8);
  const size_t rope_bytes = align256((size_t)H->rope_rows * (c.head_dim / 2) * 8);
  H->ws_bytes = work_bytes + freq_bytes + rope_bytes;
  if (hipMalloc((void**)&H->ws, H->ws_bytes) != hipSuccess) {
    (void)hipGetLastError();
    const size_t want = H->ws_bytes;
    delete H;
    return fail(COCO_ENOMEM, "workspace of %zu bytes does not fit", want);
  }
  carve_work(c, R, H->dec_rows, H->max_splits, H->ws, &H->w);
  H->inv_freq = (double*)(H->ws + work_bytes);
  H->rope = (float*)(H->ws + work_bytes + freq_bytes);
  H->act_rows_bytes[COCO_WS_X] = R * d * eb;
  H->act_rows_bytes[COCO_WS_H] = R * d * eb;
  H->act_rows_bytes[COCO_WS_Q] = R * qd * eb;
  H->act_rows_bytes[COCO_WS_O] = R * qd * eb;
  H->act_rows_bytes[COCO_WS_X1] = R * d * 4;
  H->act_rows_bytes[COCO_WS_H2] = R * d * eb;
  H->act_rows_bytes[COCO_WS_U] = R * F * eb;

  // RoPE inverse frequencies theta^(-2j/hd), in fp64.
  std::vector<double> inv(c.head_dim / 2);
  for (int j = 0; j < c.head_dim / 2; ++j)
    inv[j] = pow((double)c.rope_theta, -2.0 * j / (double)c.head_dim);
  if (hipMemcpy(H->inv_freq, inv.data(), inv.size() * 8, hipMemcpyHostToDevice) != hipSuccess ||
      hipMemset(H->ws, 0, work_bytes) != hipSuccess ||
      hipEventCreateWithFlags(&H->done, hipEventDisableTiming) != hipSuccess ||
      (H->rope_rows > 0 &&
       (launch_rope_table(H->inv_freq, c.head_dim / 2, H->rope_rows, H->rope, nullptr) !=
            hipSuccess ||
        hipDeviceSynchronize() != hipSuccess))) {
    (void)hipGetLastError();
    if (H->done) (void)hipEventDestroy(H->done);
    (void)hipFree(H->ws);
    delete H;
    return fail(COCO_EHIP, "workspace initialisation failed");
  }
  if ((rc = pack_weights(H))) {
    (void)hipEventDestroy(H->done);
    (void)hipFree(H->ws);
    delete H;
    return rc;
  }
  *out = H;
  return COCO_OK;
}

void coco_layer_destroy(coco_layer_t H) {
  if (!H) return;
  int cur = 0;
  (void)hipGetDevice(&cur);
  (void)hipSetDevice(H->device);
  // The handle's last call outside graph capture recorded `done` after its
  // last kernel; calls on one handle are ordered (they share the workspace),
  // so this waits for all of its enqueued work and nothing else.
  if (H->done) {
    (void)hipEventSynchronize(H->done);
    (void)hipEventDestroy(H->done);
  }
  for (auto& e : H->ev) (void)hipEventDestroy(e);
  (void)hipFree(H->ws);
  if (H->packed) (void)hipFree(H->packed);
  (void)hipSetDevice(cur);
  delete H;
}

int coco_layer_set_validate(coco_layer_t H, int32_t on) {
  if (!H) return fail(COCO_EINVAL, "handle is NULL");
  H->validate = on != 0;
  return COCO_OK;
}

int coco_layer_set_timing(coco_layer_t H, int32_t on) {
  if (!H) return fail(COCO_EINVAL, "handle is NULL");
  HIPCHK(hipSetDevice(H->device));
  if (on && H->ev.empty()) {
    H->ev.resize(2 * kTimingPairs);
    for (auto& e : H->ev) HIPCHK(hipEventCreate(&e));
    H->ev_kind.reserve(kTimingPairs);  // timed calls then never allocate
  }
  H->timing = on != 0;
  H->ev_kind.clear();
  H->ev_overflow = false;
  return COCO_OK;
}

int coco_layer_read_timing(coco_layer_t H, double* ms, int64_t* launches, int32_t n_kinds) {
  if (!H || !ms || !launches) return fail(COCO_EINVAL, "NULL argument");
  if (n_kinds < 0 || n_kinds > COCO_K_COUNT) return fail(COCO_EINVAL, "bad n_kinds");
  for (int k = 0; k < n_kinds; ++k) {
    ms[k] = 0.0;
    launches[k] = 0;
  }
  const bool overflow = H->ev_overflow;
  HIPCHK(hipSetDevice(H->device));
  for (size_t p = 0; p < H->ev_kind.size(); ++p) {
    HIPCHK(hipEventSynchronize(H->ev[2 * p + 1]));
    float t = 0.f;
    HIPCHK(hipEventElapsedTime(&t, H->ev[2 * p], H->ev[2 * p + 1]));
    const int k = H->ev_kind[p];
    if (k < n_kinds) {
      ms[k] += t;
      launches[k] += 1;
    }
  }
  H->ev_kind.clear();
  H->ev_overflow = false;
  if (overflow) return fail(COCO_ESTATE, "more than %d timed launches between reads", kTimingPairs);
  return COCO_OK;
}

int coco_layer_workspace(coco_layer_t H, int32_t which, void* dst, int64_t dst_bytes,
                         coco_stream_t stream) {
  if (!H || !dst) return fail(COCO_EINVAL, "NULL argument");
  void* p[7] = {H->w.x, H->w.h, H->w.q, H->w.o, H->w.x1, H->w.h2, H->w.u};
  if (which < 0 || which > 6) return fail(COCO_EINVAL, "unknown workspace id %d", which);
  if (dst_bytes < 0) return fail(COCO_EINVAL, "dst_bytes < 0");
  const size_t n = (size_t)dst_bytes < H->act_rows_bytes[which] ? (size_t)dst_bytes
                                                                 : H->act_rows_bytes[which];
  HIPCHK(hipSetDevice(H->device));
  const coco_layer_config& c = H->cfg;
  const int cols[7] = {c.d_model, c.d_model, c.n_q_heads * c.head_dim,
                       c.n_q_heads * c.head_dim, c.d_model, c.d_model, c.d_ffn};
  if (H->ws_tiled[which]) {
    HIPCHK(launch_untile((const uint16_t*)p[which], H->last_rows, cols[which],
                         (uint16_t*)dst, (int64_t)(n / 2), (hipStream_t)stream));
    return COCO_OK;
  }
  HIPCHK(hipMemcpyAsync(dst, p[which], n, hipMemcpyDeviceToDevice, (hipStream_t)stream));
  return COCO_OK;
}

}  // extern "C"

// ----------------------------------------------------------------------------
// Validation of device-side index arrays (debug mode; synchronises).
// ----------------------------------------------------------------------------
namespace {

template <typename V>
int fetch(std::vector<V>& dst, const V* src, size_t n, hipStream_t st) {
  dst.resize(n);
  if (n == 0) return COCO_OK;
  HIPCHK(hipMemcpyAsync(dst.data(), src, n * sizeof(V), hipMemcpyDeviceToHost, st));
  HIPCHK(hipStreamSynchronize(st));
  return COCO_OK;
}

int validate_batch(coco_layer* H, int64_t hidden_rows, const int32_t* row_idx, int n_rows,
                   const int32_t* positions, const int32_t* seq_starts, int n_seqs,
                   const int32_t* block_table, const int32_t* ctx_lens, int first_layer,
                   int n_layers, hipStream_t st) {
  const coco_layer_config& c = H->cfg;
  std::vector<int32_t> ri, pos, ss, bt, cl;
  int rc;
  if ((rc = fetch(ri, row_idx, n_rows, st)) || (rc = fetch(pos, positions, n_rows, st)) ||
      (rc = fetch(cl, ctx_lens, n_seqs, st)) ||
      (rc = fetch(bt, block_table, (size_t)n_seqs * c.max_blocks_per_seq, st)))
    return rc;
  if (seq_starts) {
    if ((rc = fetch(ss, seq_starts, n_seqs + 1, st))) return rc;
  } else {
    ss.resize(n_seqs + 1);
    for (int s = 0; s <= n_seqs; ++s) ss[s] = s;
  }
  std::vector<char> seen(hidden_rows, 0);
  for (int i = 0; i < n_rows; ++i) {
    if (ri[i] < 0 || ri[i] >= hidden_rows)
      return fail(COCO_EINVAL, "row_idx[%d] = %d out of range [0, %lld)", i, ri[i],
                  (long long)hidden_rows);
    if (seen[ri[i]]) return fail(COCO_EINVAL, "row_idx[%d] = %d is a duplicate", i, ri[i]);
    seen[ri[i]] = 1;
  }
  if (ss[0] != 0 || ss[n_seqs] != n_rows)
    return fail(COCO_EINVAL, "seq_starts must run from 0 to n_rows");
  int64_t min_blocks = INT64_MAX;
  for (int l = first_layer; l < first_layer + n_layers; ++l)
    if (H->layers[l].num_blocks < min_blocks) min_blocks = H->layers[l].num_blocks;
  for (int s = 0; s < n_seqs; ++s) {
    if (ss[s + 1] < ss[s]) return fail(COCO_EINVAL, "seq_starts not monotone at %d", s);
    if (cl[s] < 1 || cl[s] > c.max_blocks_per_seq * kBlockTokens)
      return fail(COCO_EINVAL, "ctx_lens[%d] = %d out of range", s, cl[s]);
    for (int i = ss[s]; i < ss[s + 1]; ++i) {
      if (pos[i] < 0 || pos[i] >= cl[s])
        return fail(COCO_EINVAL, "positions[%d] = %d not in [0, ctx_lens[%d] = %d)", i, pos[i],
                    s, cl[s]);
      if (i > ss[s] && pos[i] <= pos[i - 1])
        return fail(COCO_EINVAL, "positions of sequence %d not increasing at row %d", s, i);
    }
    const int nb = (cl[s] + kBlockTokens - 1) / kBlockTokens;
    for (int b = 0; b < nb; ++b) {
      const int32_t v = bt[(size_t)s * c.max_blocks_per_seq + b];
      if (v < 0 || v >= min_blocks)
        return fail(COCO_EINVAL, "block_table[%d][%d] = %d out of range [0, %lld)", s, b, v,
                    (long long)min_blocks);
    }
  }
  return COCO_OK;
}

// ----------------------------------------------------------------------------
// Launch sequence.
// ----------------------------------------------------------------------------
// Which kernel a decode projection of M rows runs: the weight-streaming one
// (skinny_plan: split-K from (N, K) only), or the prefill tile kernel on the
// same K-slices, with the same bits.
//   * Above 128 rows the skinny kernel reads the weights twice (us, skinny /
//     tiles): 8B O 160 rows 25.5 / 13.5, 32B down 160 rows 136 / 79, 70B QKV
//     200 rows 120 / 55 + 8 for its operand.
//   * 4- and 8-wave plans of one full round: 64- and 128-column tiles make the
//     same round. 8B O 1 row 10.7 / 7.6, 64 rows 12.1 / 9.4, 128 rows 16.3 /
//     12.3; 8B down 64 rows 27.4 / 26.5; 70B O 64 rows 31.8 / 29.0, 70B down
//     128 rows 102 / 97, 1 row 82.6 / 82.2. (8-wave plans of another grid:
//     above 64 rows, where the skinny kernel stages 128.)
//   * The rest stay: 32B O (5 waves) 64 rows 15.4 / 16.3, down 128 rows 74 / 80.
bool tile_partial(const coco_layer* H, int N, int K, int M) {
  const SkinnyPlan p = skinny_plan(N, K);
  if (p.waves == 0) return false;
  const bool round = N / (16 * p.waves) * p.S == H->num_cus;
  return M > 128 || (round && (p.waves == 4 || p.waves == 8)) || (M > 64 && p.waves == 8);
}

// QKV: the tile kernel needs gather_scale's operand first (4-8 us), which the
// skinny kernel folds in, so it pays where the weights are large too. 70B (84 M
// weights) 65 rows 57 / 42 + 7, 128 rows 62 / 50 + 7; 32B (37 M) 128 rows 26.5 /
// 22.7 + 4.6, 8B (25 M) 96 rows 20.4 / 17.0 + 4.2.
bool tile_qkv(const coco_layer* H, int M) {
  const coco_layer_config& c = H->cfg;
  const int64_t N = (int64_t)(c.n_q_heads + 2 * c.n_kv_heads) * c.head_dim;
  return M > 128 || (M > 64 && N * c.d_model >= (64 << 20));
}

// The decode GEMMs that write fp32 partials.
int gemm(const coco_layer* H, float* part, const bf16_t* A, const bf16_t* W, int M, int N, int K,
         int* S, hipStream_t st) {
  const SkinnyPlan plan = skinny_plan(N, K);
  if (plan.waves == 0) return fail(COCO_EINVAL, "no GEMM plan for N=%d K=%d", N, K);
  *S = plan.S;
  if (tile_partial(H, N, K, M))
    HIPCHK(launch_tile_partial_bf16(A, W, part, M, N, K, plan.S, H->num_cus, st));
  else
    HIPCHK(launch_gemm_skinny_bf16(A, W, part, M, N, K, plan, st));
  return COCO_OK;
}

// Decode: whether the (unsplit, bf16) gate/up projection of M rows runs on the
// tile kernel: above 128 rows, and above 64 for 8-wave plans and where a grid
// of 128 x 256 tiles fills at least three quarters of the CUs. Measured, skinny
// kernel against tiles (us): 8B 128 rows 56.2 / 55.9, 160 rows 74.4 / 65.0, 400
// rows 154 / 89; 32B (216 tiles) 65 rows 121 / 106, 128 rows 135 / 116; 70B
// (224 tiles) 80 rows 186 / 176, 128 rows 200 / 177, 256 rows 310 / 210. 8B
// (112 such tiles, 7 waves) 80 rows 49.3 / 51.6, and at 64 rows 45.4 / 46.5
// (70B 172 / 174): those stay.
bool tile_swiglu(const coco_layer* H, int M) {
  const int F = H->cfg.d_ffn;
  const SkinnyPlan p = skinny_plan(2 * F, H->cfg.d_model);
  return p.S == 1 &&
         (M > 128 || (M > 64 && (p.waves == 8 || 2 * F / 256 >= H->num_cus * 3 / 4)));
}

// Layout of the four projections' A operands in a call: tile order
// (tile_off) wherever the consuming GEMM reads it so -- every bf16 prefill
// GEMM, and the decode GEMMs that run the tile kernel -- else row-major.
struct ActLayout {
  bool h = false, o = false, h2 = false, u = false;
};
ActLayout act_layout(const coco_layer* H, bool prefill, int M) {
  const coco_layer_config& c = H->cfg;
  ActLayout a;
  if (c.dtype != COCO_BF16) return a;
  if (prefill) {
    a.h = a.o = a.h2 = a.u = true;
    return a;
  }
  const int d = c.d_model, F = c.d_ffn, qd = c.n_q_heads * c.head_dim;
  a.o = tile_partial(H, d, qd, M);
  a.h2 = skinny_plan(2 * F, d).S == 1 ? tile_swiglu(H, M) : tile_partial(H, 2 * F, d, M);
  a.u = tile_partial(H, d, F, M);
  return a;
}

int attention(coco_layer* H, const Work& W, const coco_layer_weights& w, int M,
              const int32_t* positions, const int32_t* seq_starts, int n_seqs, const int32_t* bt,
              const int32_t* ctx, bool o_tiled, hipStream_t st) {
  const coco_layer_config& c = H->cfg;
  if (!seq_starts) {
    {
      KernelTimer t(H, COCO_K_ATTENTION, st);
      HIPCHK(launch_attn_decode_bf16((const bf16_t*)W.q, (const bf16_t*)w.k_cache,
                                     (const bf16_t*)w.v_cache, bt, c.max_blocks_per_seq, ctx,
                                     positions, W.split_off, n_seqs, c.n_q_heads, c.n_kv_heads,
                                     W.attn_o, W.attn_ml, H->max_splits, H->num_cus, st));
    }
    KernelTimer t(H, COCO_K_ATTN_COMBINE, st);
    HIPCHK(launch_attn_combine_bf16(W.attn_o, W.attn_ml, ctx, positions, n_seqs, c.n_q_heads,
                                    H->max_splits, (bf16_t*)W.o, o_tiled, st));
  } else {
    KernelTimer t(H, COCO_K_ATTENTION, st);
    HIPCHK(launch_attn_prefill_bf16((const bf16_t*)W.q, (const bf16_t*)w.k_cache,
                                    (const bf16_t*)w.v_cache, bt, c.max_blocks_per_seq, ctx,
                                    positions, seq_starts, n_seqs, M, c.n_q_heads, c.n_kv_heads,
                                    (bf16_t*)W.o, H->num_cus, st));
  }
  return COCO_OK;
}

#define TIMED(kind, stmt)                     \
  do {                                        \
    KernelTimer timer_(H, kind, st);          \
    stmt;                                     \
  } while (0)

// One bf16 prefill layer: x_src[x_idx] (null: in place) to y[y_idx]. Six
// kernels; every GEMM runs its consumer's work in its epilogue: the QKV
// projection RoPE and the cache append, the O projection the residual and
// RMSNorm_2's first half (bf16(x1 * gamma) with sums of x1^2), gate/up the
// 1/rms and the SwiGLU, down the residual and the scatter. rs: row slots for
// the QKV epilogue, written by the first layer's gather.
int prefill_layer(coco_layer* H, const Work& W, const coco_layer_weights& w, const bf16_t* x_src,
                  const int32_t* x_idx, bf16_t* y, const int32_t* y_idx, int M,
                  const int32_t* positions, const int32_t* seq_starts, int n_seqs,
                  const int32_t* bt, const int32_t* ctx, const RowSlotArgs& rs, hipStream_t st) {
  const coco_layer_config& c = H->cfg;
  const int d = c.d_model, F = c.d_ffn, qd = c.n_q_heads * c.head_dim;
  bf16_t *h = (bf16_t*)W.h, *o = (bf16_t*)W.o, *h2 = (bf16_t*)W.h2, *u = (bf16_t*)W.u;
  TIMED(COCO_K_GATHER_NORM,
        HIPCHK(launch_gather_rmsnorm_bf16(x_src, x_idx, M, d, (const bf16_t*)w.gamma_attn,
                                          c.rms_eps, h, rs, st)));
  PrefillEpiArgs qa;
  qa.row_info = W.row_info;
  qa.rope = H->rope;
  qa.q_out = (uint16_t*)W.q;
  qa.k_cache = (uint16_t*)w.k_cache;
  qa.v_cache = (uint16_t*)w.v_cache;
  qa.Hq = c.n_q_heads;
  qa.Hkv = c.n_kv_heads;
  TIMED(COCO_K_GEMM_QKV,
        HIPCHK(launch_prefill_qkv_bf16(h, (const bf16_t*)w.w_qkv, M, d, qa, H->num_cus, st)));
  int rc;
  if ((rc = attention(H, W, w, M, positions, seq_starts, n_seqs, bt, ctx, true, st)))
    return rc;
  float* const ss = W.part;
  TIMED(COCO_K_GEMM_O,
        HIPCHK(launch_prefill_resid_bf16(o, (const bf16_t*)w.w_o, M, d, qd, x_src, x_idx,
                                         (const bf16_t*)w.gamma_mlp, W.x1, h2, ss, H->num_cus,
                                         st)));
  TIMED(COCO_K_GEMM_GATE_UP,
        HIPCHK(launch_prefill_swiglu_bf16(h2, (const bf16_t*)w.w_gate_up, u, M, F, d, ss,
                                          c.rms_eps, H->num_cus, st)));
  TIMED(COCO_K_GEMM_DOWN,
        HIPCHK(launch_prefill_scatter_bf16(u, (const bf16_t*)w.w_down, M, d, F, W.x1, y, y_idx,
                                           H->num_cus, st)));
  return COCO_OK;
}

// One bf16 decode layer. The gather and RMSNorm_1 are folded into the QKV
// projection: its operand is bf16(x * gamma), staged straight from the input
// rows (large batches: written by a kernel of its own), and the QKV epilogue
// applies each row's 1/rms.
int decode_layer(coco_layer* H, const Work& W, const coco_layer_weights& w, const bf16_t* x_src,
                 const int32_t* x_idx, bf16_t* y, const int32_t* y_idx, int M,
                 const int32_t* positions, const int32_t* bt, const int32_t* ctx,
                 hipStream_t st) {
  const coco_layer_config& c = H->cfg;
  const int d = c.d_model, Hq = c.n_q_heads, Hkv = c.n_kv_heads, hd = c.head_dim, F = c.d_ffn;
  const int nqkv = (Hq + 2 * Hkv) * hd;
  const ActLayout lay = act_layout(H, false, M);
  bf16_t *q = (bf16_t*)W.q, *o = (bf16_t*)W.o, *h2 = (bf16_t*)W.h2, *u = (bf16_t*)W.u;
  int S, rc;
  const SkinnyPlan plan = skinny_plan(nqkv, d);
  if (plan.waves == 0) return fail(COCO_EINVAL, "no GEMM plan for N=%d K=%d", nqkv, d);
  if (tile_qkv(H, M)) {
    TIMED(COCO_K_GATHER_NORM,
          HIPCHK(launch_gather_scale_bf16(x_src, x_idx, M, d, (const bf16_t*)w.gamma_attn,
                                          (bf16_t*)W.h, W.ss, plan.S, st)));
    TIMED(COCO_K_GEMM_QKV,
          HIPCHK(launch_tile_partial_bf16((const bf16_t*)W.h, (const bf16_t*)w.w_qkv, W.part, M,
                                          nqkv, d, plan.S, H->num_cus, st)));
  } else {
    TIMED(COCO_K_GEMM_QKV,
          HIPCHK(launch_gemm_skinny_norm_bf16(x_src, x_idx, (const bf16_t*)w.gamma_attn,
                                              (const bf16_t*)w.w_qkv, W.part, W.ss, M, nqkv, d,
                                              plan, st)));
  }
  // RoPE, local cache append.
  TIMED(COCO_K_QKV_EPILOGUE,
        HIPCHK(launch_qkv_epilogue_bf16(W.part, plan.S, M, Hq, Hkv, hd, positions, bt,
                                        c.max_blocks_per_seq, H->inv_freq, q,
                                        (bf16_t*)w.k_cache, (bf16_t*)w.v_cache, ctx, W.split_off,
                                        H->max_splits, W.ss, d, c.rms_eps, st)));
  // Attention over the paged cache.
  if ((rc = attention(H, W, w, M, positions, nullptr, M, bt, ctx, lay.o, st))) return rc;
  // O projection + residual + RMSNorm_2.
  TIMED(COCO_K_GEMM_O,
        if ((rc = gemm(H, W.part, o, (const bf16_t*)w.w_o, M, d, Hq * hd, &S, st))) return rc);
  TIMED(COCO_K_RESIDUAL_NORM,
        HIPCHK(launch_residual_rmsnorm_bf16(W.part, S, M, d, x_src, x_idx,
                                            (const bf16_t*)w.gamma_mlp, c.rms_eps, W.x1, h2,
                                            lay.h2, st)));
  // SwiGLU MLP: in the gate/up GEMM's epilogue whenever that GEMM is not split
  // along K.
  if (tile_swiglu(H, M)) {
    TIMED(COCO_K_GEMM_GATE_UP,
          HIPCHK(launch_prefill_swiglu_plain_bf16(h2, (const bf16_t*)w.w_gate_up, u, M, F, d,
                                                  lay.u, H->num_cus, st)));
  } else if (skinny_plan(2 * F, d).S == 1) {
    TIMED(COCO_K_GEMM_GATE_UP,
          HIPCHK(launch_gemm_skinny_swiglu_bf16(h2, (const bf16_t*)w.w_gate_up, u, M, F, d,
                                                skinny_plan(2 * F, d), lay.u, st)));
  } else {
    TIMED(COCO_K_GEMM_GATE_UP,
          if ((rc = gemm(H, W.part, h2, (const bf16_t*)w.w_gate_up, M, 2 * F, d, &S, st))) return rc);
    TIMED(COCO_K_SWIGLU, HIPCHK(launch_swiglu_bf16(W.part, S, M, F, u, lay.u, st)));
  }
  // Down projection and residual.
  TIMED(COCO_K_GEMM_DOWN,
        if ((rc = gemm(H, W.part, u, (const bf16_t*)w.w_down, M, d, F, &S, st))) return rc);
  TIMED(COCO_K_RESIDUAL_SCATTER,
        HIPCHK(launch_residual_scatter_bf16(W.part, S, M, d, W.x1, y, y_idx, st)));
  return COCO_OK;
}

// One fp32 layer, decode and prefill alike: five kernels.
int f32_layer(coco_layer* H, const Work& W, const coco_layer_weights& w, const float* x_src,
              const int32_t* x_idx, float* y, const int32_t* y_idx, int M,
              const int32_t* positions, const int32_t* seq_starts, int n_seqs, const int32_t* bt,
              const int32_t* ctx, hipStream_t st) {
  const coco_layer_config& c = H->cfg;
  const int d = c.d_model, Hq = c.n_q_heads, Hkv = c.n_kv_heads, hd = c.head_dim, F = c.d_ffn;
  F32EpiArgs qa;
  qa.gamma = (const float*)w.gamma_attn;
  qa.eps = c.rms_eps;
  qa.h = (float*)W.h;
  qa.row_idx = x_idx;
  qa.positions = positions;
  qa.seq_starts = seq_starts;
  qa.block_table = bt;
  qa.inv_freq = H->inv_freq;
  qa.q_out = (float*)W.q;
  qa.k_cache = (float*)w.k_cache;
  qa.v_cache = (float*)w.v_cache;
  qa.n_seqs = n_seqs;
  qa.max_blocks = c.max_blocks_per_seq;
  qa.Hq = Hq;
  qa.Hkv = Hkv;
  qa.hd = hd;
  TIMED(COCO_K_GEMM_QKV, HIPCHK(launch_f32_qkv(x_src, (const float*)w.w_qkv, M, d, qa, st)));
  TIMED(COCO_K_ATTENTION,
        HIPCHK(launch_attn_f32((const float*)W.q, (const float*)w.k_cache,
                               (const float*)w.v_cache, bt, c.max_blocks_per_seq, ctx, positions,
                               seq_starts, n_seqs, M, Hq, Hkv, hd, (float*)W.o, st)));
  F32EpiArgs oa;
  oa.row_idx = x_idx;
  oa.res = x_src;
  oa.out = W.x1;
  TIMED(COCO_K_GEMM_O,
        HIPCHK(launch_f32_resid((const float*)W.o, (const float*)w.w_o, M, d, Hq * hd, oa, st)));
  F32EpiArgs ga;
  ga.gamma = (const float*)w.gamma_mlp;
  ga.eps = c.rms_eps;
  ga.h = (float*)W.h2;
  ga.out = (float*)W.u;
  TIMED(COCO_K_GEMM_GATE_UP,
        HIPCHK(launch_f32_swiglu(W.x1, (const float*)w.w_gate_up, M, F, d, ga, st)));
  F32EpiArgs da;
  da.row_idx = y_idx;
  da.res = W.x1;
  da.out = y;
  TIMED(COCO_K_GEMM_DOWN,
        HIPCHK(launch_f32_scatter((const float*)W.u, (const float*)w.w_down, M, d, F, da, st)));
  return COCO_OK;
}

template <typename T>
int run_span(coco_layer* H, const Work& W, int first, int nl, T* hidden, const int32_t* row_idx,
             int M, const int32_t* positions, const int32_t* seq_starts, int n_seqs,
             const int32_t* bt, const int32_t* ctx, hipStream_t st) {
  T* x = (T*)W.x;
  for (int l = first; l < first + nl; ++l) {
    const coco_layer_weights& w = H->layers[l];
    const bool first_l = l == first, last_l = l == first + nl - 1;
    // The residual reads the input rows where they are (hidden[row_idx] in
    // the first layer of the call), so no copy of them is made; the last
    // layer scatters to the full batch.
    const T* x_src = first_l ? hidden : x;
    const int32_t* x_idx = first_l ? row_idx : nullptr;
    T* const y = last_l ? hidden : x;
    const int32_t* y_idx = last_l ? row_idx : nullptr;
    int rc;
    if constexpr (std::is_same<T, float>::value) {
      rc = f32_layer(H, W, w, x_src, x_idx, y, y_idx, M, positions, seq_starts, n_seqs, bt, ctx,
                     st);
    } else if (seq_starts == nullptr) {
      rc = decode_layer(H, W, w, x_src, x_idx, y, y_idx, M, positions, bt, ctx, st);
    } else {
      // Prefill row slots (position, cache block), written once per call by
      // the first layer's gather.
      RowSlotArgs rs;
      if (first_l) {
        rs.positions = positions;
        rs.seq_starts = seq_starts;
        rs.block_table = bt;
        rs.row_info = W.row_info;
        rs.n_seqs = n_seqs;
        rs.max_blocks = H->cfg.max_blocks_per_seq;
        rs.rope_rows = H->rope_rows;
      }
      rc = prefill_layer(H, W, w, x_src, x_idx, y, y_idx, M, positions, seq_starts, n_seqs, bt,
                         ctx, rs, st);
    }
    if (rc) return rc;
  }
  return COCO_OK;
}
#undef TIMED

int check_batch(coco_layer* H, int first, int nl, const void* hidden, int64_t hidden_rows,
                const int32_t* row_idx, int n_rows, const int32_t* positions,
                const int32_t* seq_starts, int n_seqs, const int32_t* bt, const int32_t* ctx) {
  const coco_layer_config& c = H->cfg;
  if (first < 0 || nl < 1 || first + nl > c.n_layers)
    return fail(COCO_EINVAL, "layers [%d, %d) outside [0, %d)", first, first + nl, c.n_layers);
  if (n_rows < 0 || n_rows > c.max_rows)
    return fail(COCO_EINVAL, "n_rows = %d outside [0, max_rows = %d]", n_rows, c.max_rows);
  if (n_rows == 0) return COCO_OK;
  if (!hidden || !row_idx || !positions || !bt || !ctx)
    return fail(COCO_EINVAL, "NULL batch pointer");
  if (hidden_rows < 1) return fail(COCO_EINVAL, "hidden_rows must be >= 1");
  if ((uintptr_t)hidden % 16) return fail(COCO_EINVAL, "hidden is not 16-byte aligned");
  if (n_seqs < 1 || n_seqs > c.max_seqs)
    return fail(COCO_EINVAL, "n_seqs = %d outside [1, max_seqs = %d]", n_seqs, c.max_seqs);
  if (!seq_starts) {
    if (n_seqs != n_rows)
      return fail(COCO_EINVAL, "decode (seq_starts NULL) needs n_seqs == n_rows");
    if (n_seqs > H->dec_rows)
      return fail(COCO_EINVAL, "decode batch larger than min(max_rows, max_seqs)");
  } else if (n_seqs > n_rows) {
    return fail(COCO_EINVAL, "more sequences than rows");
  }
  return COCO_OK;
}

// Records the handle's completion event behind the call's last kernel, unless
// the stream is being captured into a graph (the event would then only fire
// on replays).
int mark_done(coco_layer* H, hipStream_t st) {
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  HIPCHK(hipStreamIsCapturing(st, &cs));
  if (cs == hipStreamCaptureStatusNone) HIPCHK(hipEventRecord(H->done, st));
  return COCO_OK;
}

// use_static: the per-call buffers come from this device's static scratch
// array, sized for the call (no allocation anywhere; validation mode, which
// copies index arrays to the host, is not run).
int forward_impl(coco_layer* H, int first, int nl, void* hidden, int64_t hidden_rows,
                 const int32_t* row_idx, int n_rows, const int32_t* positions,
                 const int32_t* seq_starts, int n_seqs, const int32_t* bt, const int32_t* ctx,
                 coco_stream_t stream, bool use_static = false) {
  if (!H) return fail(COCO_EINVAL, "handle is NULL");
  int rc = check_batch(H, first, nl, hidden, hidden_rows, row_idx, n_rows, positions,
                       seq_starts, n_seqs, bt, ctx);
  if (rc || n_rows == 0) return rc;
  hipStream_t st = (hipStream_t)stream;
  HIPCHK(hipSetDevice(H->device));
  Work W = H->w;
  if (use_static) {
    const int64_t dec_seqs = seq_starts ? 0 : n_seqs;
    const size_t need = carve_work(H->cfg, n_rows, dec_seqs, H->max_splits, nullptr, nullptr);
    if (need > kScratchBytes)
      return fail(COCO_EINVAL,
                  "call needs %zu bytes of scratch; the no-alloc entry point has %zu (%d rows)",
                  need, kScratchBytes, n_rows);
    char* base = scratch_ptr(H->device);
    if (!base) return fail(COCO_ESTATE, "static scratch of device %d not set up", H->device);
    carve_work(H->cfg, n_rows, dec_seqs, H->max_splits, base, &W);
  } else if (H->validate &&
             (rc = validate_batch(H, hidden_rows, row_idx, n_rows, positions, seq_starts, n_seqs,
                                  bt, ctx, first, nl, st))) {
    return rc;
  }
  if (!use_static) {
    const ActLayout a = act_layout(H, seq_starts != nullptr, n_rows);
    for (bool& t : H->ws_tiled) t = false;
    H->ws_tiled[COCO_WS_H] = a.h;
    H->ws_tiled[COCO_WS_O] = a.o;
    H->ws_tiled[COCO_WS_H2] = a.h2;
    H->ws_tiled[COCO_WS_U] = a.u;
    H->last_rows = n_rows;
  }
  if (H->cfg.dtype == COCO_BF16)
    rc = run_span<bf16_t>(H, W, first, nl, (bf16_t*)hidden, row_idx, n_rows, positions,
                          seq_starts, n_seqs, bt, ctx, st);
  else
    rc = run_span<float>(H, W, first, nl, (float*)hidden, row_idx, n_rows, positions,
                         seq_starts, n_seqs, bt, ctx, st);
  if (rc) return rc;
  return mark_done(H, st);
}

}  // namespace

extern "C" {

int coco_layer_forward(coco_layer_t H, int32_t layer, void* hidden, int64_t hidden_rows,
                       const int32_t* row_idx, int32_t n_rows, const int32_t* positions,
                       const int32_t* seq_starts, int32_t n_seqs, const int32_t* block_table,
                       const int32_t* ctx_lens, coco_stream_t stream) {
  return forward_impl(H, layer, 1, hidden, hidden_rows, row_idx, n_rows, positions, seq_starts,
                      n_seqs, block_table, ctx_lens, stream);
}

int coco_layer_forward_noalloc(coco_layer_t H, int32_t layer, void* hidden, int64_t hidden_rows,
                               const int32_t* row_idx, int32_t n_rows, const int32_t* positions,
                               const int32_t* seq_starts, int32_t n_seqs,
                               const int32_t* block_table, const int32_t* ctx_lens,
                               coco_stream_t stream) {
  return forward_impl(H, layer, 1, hidden, hidden_rows, row_idx, n_rows, positions, seq_starts,
                      n_seqs, block_table, ctx_lens, stream, true);
}

int coco_layer_span_forward(coco_layer_t H, int32_t first_layer, int32_t n_layers, void* hidden,
                            int64_t hidden_rows, const int32_t* row_idx, int32_t n_rows,
                            const int32_t* positions, const int32_t* seq_starts, int32_t n_seqs,
                            const int32_t* block_table, const int32_t* ctx_lens,
                            coco_stream_t stream) {
  return forward_impl(H, first_layer, n_layers, hidden, hidden_rows, row_idx, n_rows, positions,
                      seq_starts, n_seqs, block_table, ctx_lens, stream);
}

int coco_kv_append(coco_layer_t H, int32_t layer, const void* k, const void* v,
                   const int32_t* seq_idx, const int32_t* positions, int32_t n_tok,
                   const int32_t* block_table, int32_t n_seqs, coco_stream_t stream) {
  if (!H) return fail(COCO_EINVAL, "handle is NULL");
  const coco_layer_config& c = H->cfg;
  if (layer < 0 || layer >= c.n_layers) return fail(COCO_EINVAL, "layer %d out of range", layer);
  if (n_tok < 0) return fail(COCO_EINVAL, "n_tok < 0");
  if (n_tok == 0) return COCO_OK;
  if (!k || !v || !seq_idx || !positions || !block_table)
    return fail(COCO_EINVAL, "NULL argument");
  if (n_seqs < 1) return fail(COCO_EINVAL, "n_seqs must be >= 1");
  hipStream_t st = (hipStream_t)stream;
  HIPCHK(hipSetDevice(H->device));
  if (H->validate) {
    std::vector<int32_t> si, pos, bt;
    int rc;
    if ((rc = fetch(si, seq_idx, n_tok, st)) || (rc = fetch(pos, positions, n_tok, st)) ||
        (rc = fetch(bt, block_table, (size_t)n_seqs * c.max_blocks_per_seq, st)))
      return rc;
    for (int t = 0; t < n_tok; ++t) {
      if (si[t] < 0 || si[t] >= n_seqs) return fail(COCO_EINVAL, "seq_idx[%d] out of range", t);
      if (pos[t] < 0 || pos[t] >= c.max_blocks_per_seq * kBlockTokens)
        return fail(COCO_EINVAL, "positions[%d] out of range", t);
      const int32_t b = bt[(size_t)si[t] * c.max_blocks_per_seq + pos[t] / kBlockTokens];
      if (b < 0 || b >= H->layers[layer].num_blocks)
        return fail(COCO_EINVAL, "token %d maps to block %d outside the pool", t, b);
    }
  }
  const coco_layer_weights& w = H->layers[layer];
  if (c.dtype == COCO_BF16)
    HIPCHK(launch_kv_append<bf16_t>((const bf16_t*)k, (const bf16_t*)v, seq_idx, positions, n_tok,
                                    c.n_kv_heads, c.head_dim, block_table, c.max_blocks_per_seq,
                                    (bf16_t*)w.k_cache, (bf16_t*)w.v_cache, st));
  else
    HIPCHK(launch_kv_append<float>((const float*)k, (const float*)v, seq_idx, positions, n_tok,
                                   c.n_kv_heads, c.head_dim, block_table, c.max_blocks_per_seq,
                                   (float*)w.k_cache, (float*)w.v_cache, st));
  return mark_done(H, st);
}

}  // extern "C"
