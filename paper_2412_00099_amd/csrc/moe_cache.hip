// Host side of libmoe_cache: argument checking, the context, the per-layer step sequence and statistics.  A step that nobody
// waits for is enqueued and left alone: routing, the experts and what misses run on the device.  Only one that is waited for
// goes route kernel -> host learns the misses -> fills on the copy stream -> expert kernels.
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <algorithm>
#include <chrono>
#include <new>
#include <string>
#include <vector>

#include "batch_places.h"
#include "common.h"
#include "waiting_turn.h"

using namespace moe;

namespace {

thread_local std::string g_err;

int fail(int code, const char *fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_err = buf;
  return code;
}

#define HIP_TRY(expr)                                                                        \
  do {                                                                                       \
    hipError_t e_ = (expr);                                                                  \
    if (e_ != hipSuccess) return fail(MOE_EHIP, "%s: %s", #expr, hipGetErrorString(e_));     \
  } while (0)

// Keeps the compute stream busy for about `ticks` periods of the 100 MHz wall clock (bounded by the iteration
// count whatever the clock does).  Enqueued ahead of a launch that is timed with events: the start event of such
// a launch is a marker of its own, enqueued a few microseconds of host time before the kernel, and on an idle
// stream it would be stamped that much before the kernel starts.  Behind this kernel both are queued by the time
// the marker is reached.
__global__ void hold_stream_kernel(uint64_t ticks) {
  const uint64_t t0 = wall_clock64();
  for (int i = 0; i < 4096 && wall_clock64() - t0 < ticks; ++i) __builtin_amdgcn_s_sleep(8);
}

// per device: whose launches may wait for their first workgroup
constexpr int kMaxDevices = 64;
WaitingTurn g_turn[kMaxDevices];

bool valid_wfmt(int f) { return f >= MOE_W_FP32 && f <= MOE_W_INT4_G128; }
bool valid_afmt(int f) { return f == MOE_A_FP32 || f == MOE_A_BF16; }

}  // namespace

struct moe_cache {
  moe_cache_config_t cfg{};
  std::vector<const void *> host_blob;
  std::vector<void *> slot_pool;
  std::vector<const void *> gate_w;
  std::vector<const void *> shared_blob;
  std::vector<int32_t> initial;
  int32_t n_initial = 0;
  BlobLayout slot_layout{};
  hipStream_t compute = nullptr, copy = nullptr;

  LayerState *d_state = nullptr;   // two copies of every layer's state: [2][n_layers]; cur[layer] says which one counts
  std::vector<uint8_t> cur;        // (a launch that routes in every workgroup reads one and writes the other)
  LayerState *state(int layer) const { return d_state + (size_t)cur[layer] * cfg.n_layers + layer; }
  float *d_logits = nullptr;       // [n_layers][MOE_MAX_EXPERTS] logits of a layer boundary whose routing is still to come
  moe_route_out_t *d_route = nullptr;
  HostNote *h_note = nullptr;      // pinned, mapped: the router's message to the host, one per layer
  HostNote *h_note_dev = nullptr;  // device view of h_note
  HostRecord *h_rec = nullptr;     // pinned, mapped: the full record of the last step that was waited for
  HostRecord *h_rec_dev = nullptr;
  uint32_t *h_done = nullptr;      // pinned, mapped: seq of the last batch whose records are all in batch_rec
  uint32_t *h_done_dev = nullptr;
  struct Decision {                // h_note decoded
    int n_miss = 0;
    uint8_t miss_mask = 0;
    uint8_t expert[MOE_MAX_TOPK] = {}, slot[MOE_MAX_TOPK] = {};
  };
  std::vector<Decision> decided;
  // layer boundaries deferred into the expert launch (see BoundaryArgs)
  std::vector<BoundaryArgs> boundary;
  uint64_t *d_handover = nullptr;   // [n_layers][64] self-tagged words: a boundary's decision for its own launch
  float *d_ss = nullptr;            // [128] sums of squares of the residual stream per 64 columns
  uint32_t *h_gave_up = nullptr;    // pinned, mapped: set by a wavefront that stopped waiting for the hand-over
  uint32_t *h_gave_up_dev = nullptr;
  bool fuse_boundary = true;        // run deferred boundaries inside the expert launch (see moe_cache_init)
  bool route_everywhere = false;    // deferred boundaries: gate launch, routing in every workgroup of the expert launch
  bool everywhere_cumsum = false;   // the same in route mode MOE_ROUTE_CUMSUM
  bool poison_fills = false;        // debugging aid: a slot is overwritten with NaN patterns before its fill (MOE_POISON_FILLS)
  int tag_spins = 1 << 18;          // polls (about a tenth of a second) before a workgroup stops waiting for
                                    // workgroup 0; MOE_TAG_SPINS lowers it so that tests reach the error path
  int32_t *d_initial = nullptr;
  float *d_partial = nullptr;
  int pending_rows = 0;            // partial rows of an expert output not reduced yet (y_dev was NULL)
  const int32_t *pending_miss = nullptr;  // see launch_partial_reduce
  void *d_y = nullptr;             // [d] act_fmt: a pending expert output once summed, when the caller gave no y_dev
  GemvPlan plan{};
  hipEvent_t ev_route = nullptr;
  std::vector<hipEvent_t> ev_copy;
  std::vector<uint8_t> routed;        // per layer: 0 idle, 1 routed (decision on the host), 2 routed (not collected
                                      // yet), 3 boundary deferred into the expert launch,
                                      // 4 routing deferred into every workgroup of it
  bool x_fixed = false;               // a non-blocking boundary's x_dev is the only one its moe_expert_forward takes
  std::vector<const void *> x_given;  // per layer: that x_dev, or nullptr
  std::vector<uint8_t> logits_given;  // per layer: the pending step reads the caller's logits
  int deferred = -1;                  // the layer in state 3: its launch forms x from the caller's h and d_ss
  std::vector<uint32_t> route_seq;    // per layer: completion tag of the pending route step
  std::vector<uint32_t> hand_count;   // per layer: hand-overs inside an expert launch so far
  std::vector<int64_t> bytes_filled;  // per layer: what had been filled when the misses stood at miss_base
  std::vector<int64_t> miss_base;
  const uint8_t **d_host_blob = nullptr;  // [n_layers][N] the host tier as the device sees it, or nullptr: some of it is not
                                          // mapped there, and every fill is a copy that the host enqueues
  uint32_t seq = 0;
  bool poll = false;

  // prompt phase (moe_route_batch / moe_expert_forward_batch); allocated only for shapes the batched kernels take
  bool batch_ok = false;
  float *d_logits_batch = nullptr;          // [kMaxBatch][n_experts]
  moe_route_out_t *batch_rec = nullptr;      // [kMaxBatch] the decisions of the batch routed last: pinned host memory
  moe_route_out_t *batch_rec_dev = nullptr;  // the routing kernel's view of it (the records go straight to the host)
  BatchSel *d_bsel = nullptr;               // the same selection as the expert kernels read it
  BatchAhead *d_bahead = nullptr;           // between the two routing kernels of a long batch
  BatchPlan *d_bplan = nullptr;             // units of a batch whose expert kernels were enqueued behind its routing
  const void *batch_x = nullptr;            // x_dev of that batch, until moe_expert_forward_batch; nullptr: they were not
  uint8_t *d_bh = nullptr;                  // h of a segment (see up_batch_kernel)
  float *d_bpartial = nullptr;              // P of a segment: [kMaxPartialRows][hidden]
  int n_cus = 0;
  int dev = 0;
  int batch_layer = -1, batch_n = 0;
  int batch_misses = 0;                     // fills that moe_expert_forward_batch has not enqueued yet
  hipEvent_t ev_batch = nullptr;            // compute stream has finished reading the slots (before fills overwrite them)

  // optional timing of the expert GEMV launches
  int profiling = 0;      // 0 = off, n = events on every n-th expert launch of a layer's first pass
  uint64_t prof_tick = 0;
  std::vector<std::pair<hipEvent_t, hipEvent_t>> prof_events;
  std::vector<uint8_t> prof_full;  // launch covered the whole layer (no expert was missing)
  size_t prof_used = 0;
};

namespace {

int check_waits(const moe_cache_t *ctx) {
  if (ctx->h_gave_up && __atomic_load_n(ctx->h_gave_up, __ATOMIC_ACQUIRE) != 0)
    return fail(MOE_EHIP, "an expert kernel gave up waiting for the layer boundary of its own launch: outputs since then are invalid");
  return MOE_OK;
}

int check_layer(const moe_cache_t *ctx, int32_t layer) {
  if (!ctx) return fail(MOE_EINVAL, "context is NULL");
  if (layer < 0 || layer >= ctx->cfg.n_layers) return fail(MOE_EINVAL, "layer %d out of range [0,%d)", layer, ctx->cfg.n_layers);
  return check_waits(ctx);
}

// Everything enqueued on the compute stream has run.  The host may be many tokens ahead when it asks, so a wait that ran out
// in one of the launches that were still queued is known only now.
int sync_compute(const moe_cache_t *ctx) {
  HIP_TRY(hipStreamSynchronize(ctx->compute));
  return check_waits(ctx);
}

// Polls until arrived() or, after 200 ms (or at once without polling: MOE_HOST_SYNC=event), the end of what has been
// enqueued on the compute stream, which also surfaces launch errors.  Whether it has arrived then.
template <typename F>
int wait_for(moe_cache_t *c, F arrived, bool *ok) {
  *ok = true;
  if (c->poll) {
    const auto t0 = std::chrono::steady_clock::now();
    for (uint32_t spin = 0;; ++spin) {
      if (arrived()) return MOE_OK;
      if ((spin & 0x3ff) == 0x3ff && std::chrono::steady_clock::now() - t0 > std::chrono::milliseconds(200)) break;
    }
  }
  HIP_TRY(hipEventRecord(c->ev_route, c->compute));
  HIP_TRY(hipEventSynchronize(c->ev_route));
  *ok = arrived();
  return MOE_OK;
}

int do_reset(moe_cache_t *c) {
  HIP_TRY(hipStreamSynchronize(c->compute));
  HIP_TRY(hipStreamSynchronize(c->copy));
  if (c->n_initial > 0)
    HIP_TRY(hipMemcpy(c->d_initial, c->initial.data(), c->initial.size() * sizeof(int32_t), hipMemcpyHostToDevice));
  for (int copy = 0; copy < 2; ++copy)
    HIP_TRY(launch_state_init(c->d_state + (size_t)copy * c->cfg.n_layers, c->cfg.n_layers, c->d_initial, c->n_initial, c->compute));
  std::fill(c->cur.begin(), c->cur.end(), 0);
  g_turn[c->dev].give_back(c);
  if (c->h_gave_up) __atomic_store_n(c->h_gave_up, 0u, __ATOMIC_RELAXED);
  c->pending_rows = 0;
  c->deferred = -1;
  c->batch_layer = -1;
  c->batch_n = 0;
  c->batch_x = nullptr;
  const int N = c->cfg.n_experts;
  for (int l = 0; l < c->cfg.n_layers; ++l) {
    for (int i = 0; i < c->n_initial; ++i) {
      const int e = c->initial[(size_t)l * c->n_initial + i];
      HIP_TRY(hipMemcpy(static_cast<uint8_t *>(c->slot_pool[l]) + (size_t)i * c->slot_layout.total,
                        c->host_blob[(size_t)l * N + e], c->slot_layout.total, hipMemcpyHostToDevice));
    }
    c->routed[l] = 0;
    c->bytes_filled[l] = 0;
    c->miss_base[l] = 0;
  }
  HIP_TRY(hipStreamSynchronize(c->compute));
  return MOE_OK;
}

}  // namespace

extern "C" {

const char *moe_last_error(void) { return g_err.c_str(); }

size_t moe_blob_bytes(int32_t weight_fmt, int32_t hidden, int32_t inter) {
  if (!valid_wfmt(weight_fmt) || hidden <= 0 || inter <= 0) return 0;
  if (!gemv_shape_supported(weight_fmt, hidden) || !gemv_inter_supported(weight_fmt, inter)) return 0;
  return (size_t)blob_layout(weight_fmt, hidden, inter).total;
}

size_t moe_slot_bytes(const moe_cache_config_t *cfg) {
  if (!cfg) return 0;
  return moe_blob_bytes(cfg->weight_fmt, cfg->hidden, cfg->inter);
}

int moe_pack_expert(int32_t weight_fmt, int32_t hidden, int32_t inter, const void *gate, const void *up,
                    const void *down, const void *gate_s, const void *up_s, const void *down_s, void *blob_dev,
                    void *stream) {
  if (!valid_wfmt(weight_fmt)) return fail(MOE_EINVAL, "unknown weight format %d", weight_fmt);
  if (hidden <= 0 || inter <= 0 || !gemv_shape_supported(weight_fmt, hidden) ||
      !gemv_inter_supported(weight_fmt, inter))
    return fail(MOE_EINVAL, "unsupported shape hidden=%d inter=%d for weight format %d", hidden, inter, weight_fmt);
  if (!gate || !up || !down || !blob_dev) return fail(MOE_EINVAL, "NULL weight or blob pointer");
  const bool quant = weight_fmt == MOE_W_INT8_PC || weight_fmt == MOE_W_INT4_G128;
  if (quant && (!gate_s || !up_s || !down_s)) return fail(MOE_EINVAL, "quantised format needs scale pointers");
  HIP_TRY(launch_pack(weight_fmt, hidden, inter, gate, up, down, gate_s, up_s, down_s, blob_dev,
                      static_cast<hipStream_t>(stream)));
  return MOE_OK;
}

int moe_cache_init(const moe_cache_config_t *cfg, const moe_cache_buffers_t *b, moe_cache_t **out) {
  if (!out) return fail(MOE_EINVAL, "out is NULL");
  *out = nullptr;
  if (!cfg || !b) return fail(MOE_EINVAL, "config or buffers is NULL");
  // ---- everything below is checked before the first HIP call ----
  if (cfg->n_layers <= 0) return fail(MOE_EINVAL, "n_layers must be positive");
  if (cfg->n_experts <= 0 || cfg->n_experts > MOE_MAX_EXPERTS)
    return fail(MOE_EINVAL, "n_experts must be in 1..%d", MOE_MAX_EXPERTS);
  if (cfg->top_k <= 0 || cfg->top_k > MOE_MAX_TOPK) return fail(MOE_EINVAL, "top_k must be in 1..%d", MOE_MAX_TOPK);
  if (cfg->top_j < 0 || cfg->top_j > cfg->top_k) return fail(MOE_EINVAL, "top_j must be in 0..top_k");
  if (cfg->capacity < cfg->top_k) return fail(MOE_EINVAL, "capacity %d < top_k %d: a token's experts must all be resident", cfg->capacity, cfg->top_k);
  if (cfg->capacity > cfg->n_experts) return fail(MOE_EINVAL, "capacity exceeds n_experts");
  if (!valid_wfmt(cfg->weight_fmt) || !valid_afmt(cfg->act_fmt)) return fail(MOE_EINVAL, "unknown weight or activation format");
  if (cfg->inter <= 0 || cfg->shared_inter < 0) return fail(MOE_EINVAL, "bad intermediate size");
  if (!gemv_shape_supported(cfg->weight_fmt, cfg->hidden))
    return fail(MOE_EINVAL, "hidden=%d unsupported for weight format %d (needs 64*{1,2,4,8} 16-byte loads per row)", cfg->hidden, cfg->weight_fmt);
  if (!gemv_inter_supported(cfg->weight_fmt, cfg->inter) ||
      (cfg->shared_inter > 0 && !gemv_inter_supported(cfg->weight_fmt, cfg->shared_inter)))
    return fail(MOE_EINVAL, "intermediate size unsupported for this weight format (int8: multiple of 8, int4: multiple of 128)");
  if ((int64_t)cfg->top_k * cfg->inter + cfg->shared_inter > (int64_t)1 << 22)
    return fail(MOE_EINVAL, "more than 2^22 expert records per layer-token");
  if (!(cfg->lambda >= 0.f) || !std::isfinite(cfg->lambda)) return fail(MOE_EINVAL, "lambda must be finite and >= 0");
  if (cfg->delta_mode < MOE_DELTA_RUNNING_MEAN || cfg->delta_mode > MOE_DELTA_TOKEN) return fail(MOE_EINVAL, "bad delta_mode");
  if (cfg->delta_mode == MOE_DELTA_FIXED && !std::isfinite(cfg->delta_fixed)) return fail(MOE_EINVAL, "delta_fixed must be finite");
  if (cfg->route_mode < MOE_ROUTE_CACHE_PRIOR || cfg->route_mode > MOE_ROUTE_CUMSUM) return fail(MOE_EINVAL, "bad route_mode");
  if (cfg->route_mode == MOE_ROUTE_MAX_RANK && (cfg->max_rank < 0 || cfg->max_rank > cfg->n_experts))
    return fail(MOE_EINVAL, "max_rank must be in 0..n_experts");
  if (cfg->route_mode == MOE_ROUTE_CUMSUM && !(cfg->cumsum_p >= 0.f)) return fail(MOE_EINVAL, "cumsum_p must be >= 0");
  if (cfg->renormalize != 0 && cfg->renormalize != 1) return fail(MOE_EINVAL, "renormalize must be 0 or 1");
  if (cfg->compute_stream == cfg->copy_stream) return fail(MOE_EINVAL, "copy_stream must differ from compute_stream");
  if (!b->host_expert_blob || !b->slot_pool || !b->gate_w) return fail(MOE_EINVAL, "NULL buffer table");
  if (cfg->shared_inter > 0 && !b->shared_blob) return fail(MOE_EINVAL, "shared_inter > 0 needs shared_blob");
  if (b->n_initial < 0 || b->n_initial > cfg->capacity) return fail(MOE_EINVAL, "n_initial must be in 0..capacity");
  if (b->n_initial > 0 && !b->initial_resident) return fail(MOE_EINVAL, "n_initial > 0 needs initial_resident");
  const int L = cfg->n_layers, N = cfg->n_experts;
  for (int l = 0; l < L; ++l) {
    if (!b->slot_pool[l] || !b->gate_w[l]) return fail(MOE_EINVAL, "NULL slot pool or gate matrix for layer %d", l);
    if (reinterpret_cast<uintptr_t>(b->slot_pool[l]) % 256 != 0) return fail(MOE_EINVAL, "slot pool of layer %d not 256-byte aligned", l);
    if (cfg->shared_inter > 0 && !b->shared_blob[l]) return fail(MOE_EINVAL, "NULL shared blob for layer %d", l);
    for (int e = 0; e < N; ++e)
      if (!b->host_expert_blob[(size_t)l * N + e]) return fail(MOE_EINVAL, "NULL host blob for layer %d expert %d", l, e);
    uint64_t seen = 0;
    for (int i = 0; i < b->n_initial; ++i) {
      const int e = b->initial_resident[(size_t)l * b->n_initial + i];
      if (e < 0 || e >= N || ((seen >> e) & 1)) return fail(MOE_EINVAL, "initial_resident of layer %d: bad or repeated expert %d", l, e);
      seen |= 1ull << e;
    }
  }

  moe_cache_t *c = new (std::nothrow) moe_cache;
  if (!c) return fail(MOE_ENOMEM, "out of host memory");
  c->cfg = *cfg;
  c->host_blob.assign(b->host_expert_blob, b->host_expert_blob + (size_t)L * N);
  c->slot_pool.assign(b->slot_pool, b->slot_pool + L);
  c->gate_w.assign(b->gate_w, b->gate_w + L);
  if (cfg->shared_inter > 0) c->shared_blob.assign(b->shared_blob, b->shared_blob + L);
  c->n_initial = b->n_initial;
  if (b->n_initial > 0) c->initial.assign(b->initial_resident, b->initial_resident + (size_t)L * b->n_initial);
  c->slot_layout = blob_layout(cfg->weight_fmt, cfg->hidden, cfg->inter);
  c->compute = static_cast<hipStream_t>(cfg->compute_stream);
  c->copy = static_cast<hipStream_t>(cfg->copy_stream);
  c->routed.assign(L, 0);
  c->cur.assign(L, 0);
  c->route_seq.assign(L, 0);
  c->hand_count.assign(L, 0);
  c->decided.assign(L, {});
  c->boundary.assign(L, BoundaryArgs{});
  c->x_given.assign(L, nullptr);
  c->logits_given.assign(L, 0);
  c->bytes_filled.assign(L, 0);
  c->miss_base.assign(L, 0);
  c->ev_copy.assign(L, nullptr);

  auto bail = [&](int code) {
    moe_cache_destroy(c);
    return code;
  };
#define HIP_INIT(expr)                                                                      \
  do {                                                                                      \
    hipError_t e_ = (expr);                                                                 \
    if (e_ != hipSuccess) {                                                                 \
      fail(e_ == hipErrorOutOfMemory ? MOE_ENOMEM : MOE_EHIP, "%s: %s", #expr, hipGetErrorString(e_)); \
      return bail(e_ == hipErrorOutOfMemory ? MOE_ENOMEM : MOE_EHIP);                       \
    }                                                                                       \
  } while (0)

  int dev = 0;
  HIP_INIT(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) HIP_INIT(hipErrorInvalidDevice);
  c->dev = dev;
  int cus = 0;
  HIP_INIT(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
  HIP_INIT(static_scratch_setup(dev, nullptr, nullptr));  // moe_expert_forward_static's scratch array on this device
  c->n_cus = cus;
  c->plan = gemv_plan(cus, cfg->top_k * cfg->inter + cfg->shared_inter, cfg->weight_fmt, cfg->act_fmt, cfg->hidden);
  // the host learns a routing decision by polling the three self-tagged words the router stores into mapped host
  // memory (each complete in itself, no ordering between them); MOE_HOST_SYNC=event waits on a stream event instead
  c->poll = true;
  if (const char *s = getenv("MOE_HOST_SYNC")) c->poll = strcmp(s, "event") != 0;

  HIP_INIT(hipMalloc(&c->d_state, sizeof(LayerState) * 2 * L));
  HIP_INIT(hipMalloc(&c->d_logits, sizeof(float) * MOE_MAX_EXPERTS * (size_t)L));
  HIP_INIT(hipMalloc(&c->d_route, sizeof(moe_route_out_t) * L));
  HIP_INIT(hipMemset(c->d_route, 0, sizeof(moe_route_out_t) * L));
  HIP_INIT(hipHostMalloc(reinterpret_cast<void **>(&c->h_note), sizeof(HostNote) * L,
                         hipHostMallocMapped | hipHostMallocCoherent));
  memset(c->h_note, 0, sizeof(HostNote) * L);
  HIP_INIT(hipHostGetDevicePointer(reinterpret_cast<void **>(&c->h_note_dev), c->h_note, 0));
  HIP_INIT(hipHostMalloc(reinterpret_cast<void **>(&c->h_rec), sizeof(HostRecord), hipHostMallocMapped | hipHostMallocCoherent));
  memset(c->h_rec, 0, sizeof(HostRecord));
  HIP_INIT(hipHostGetDevicePointer(reinterpret_cast<void **>(&c->h_rec_dev), c->h_rec, 0));
  HIP_INIT(hipMalloc(&c->d_handover, sizeof(uint64_t) * 64 * (size_t)L));
  HIP_INIT(hipMemset(c->d_handover, 0, sizeof(uint64_t) * 64 * (size_t)L));
  HIP_INIT(hipMalloc(&c->d_ss, sizeof(float) * 128));
  HIP_INIT(hipMemset(c->d_ss, 0, sizeof(float) * 128));
  HIP_INIT(hipHostMalloc(reinterpret_cast<void **>(&c->h_gave_up), sizeof(uint32_t),
                         hipHostMallocMapped | hipHostMallocCoherent));
  *c->h_gave_up = 0;
  HIP_INIT(hipHostGetDevicePointer(reinterpret_cast<void **>(&c->h_gave_up_dev), c->h_gave_up, 0));
  // Three ways to run a boundary that nobody waits for (measured with nobody waiting in the expert launch either, us per
  // layer-token, 60 experts, 3 layers; one launch of the boundary before the experts / routing in every workgroup behind a gate
  // launch / boundary inside the expert launch; MB a layer-token, of them the shared expert's):
  //   d = 512, bf16   3.1, 0    12.5 / 13.7 / -      17.3, 0    13.8 / 13.2 / -      26, 8.7  14.6 / 13.6 / 14.2   69, 34.6  20.6 / 18.7 / 17.0
  //   d = 1024, bf16  12.6, 0   14.6 / 13.3 / -      51.9, 17.3 19.6 / 16.7 / 17.7   69, 34.6 21.9 / 18.8 / 17.8
  //   d = 2048, bf16  6.3, 0    15.8 / 14.1 / -      75.5, 25   24.7 / 20.5 / 22.0   104, 34.6 28.8 / 24.6 / 25.1  75.5, 50  24.5 / 20.5 / 18.9
  //   d = 2048, int8  12.6, 0   17.1 / 15.2 / -      52, 17.3   23.0 / 20.1 / 20.5   86.5, 52 27.9 / 25.0 / 22.5
  //   d = 2048, int4  3.2, 0    16.5 / 15.9 / -      35.7, 9    24.9 / 22.9 / 26.0   62.4, 36 31.9 / 29.1 / 27.4
  //   d = 4096        6.5, 0 (int4) 22.3 / 19.4 / -  138, 69 (int8) 39.2 / 35.9 / 35.9          277, 138 (int8) 58.8 / 55.5 / 52.4
  //   d = 256, fp32   3.1, 0    12.0 / 12.9 / -      d = 1024, fp32 25, 0 17.0 / 14.4 / -       25, 12.6 16.3 / 14.1 / -
  // Inside the launch the boundary hides behind the shared expert's records, but one compute unit does all of it, and the
  // gate matrix alone costs it time in proportion to d: about 20 KB of shared records per hidden column are wanted for that.
  // Routing everywhere spreads the gate matrix; against that, the launch of its own sums the pending output and does the glue
  // of small hidden sizes in one launch less where a token begins, which only the smallest layers feel.
  // Cumsum-Threshold walks all ranks in every wavefront (bf16 d = 2048, 6.3 MB 20.0 / 16.9; int8 12.6 MB 21.2 / 18.8).  The lines
  // for int4 were drawn when its launch was longer by what its registers cost (see expert_gemv_int4_kernel): own launch / every
  // workgroup then, d = 2048, 64 experts 22.7 MB 27.6 / 30.4, 97 MB 40.0 / 41.6, 32 experts 38.9 MB 29.1 / 28.8; d = 4096, 60
  // experts 3.2 MB 28.2 / 29.4, 22.7 MB 31.4 / 31.1.  Now: d = 2048, 60 experts 1.6 MB 20.5 / 18.4, 35 MB 27.0 / 24.6, 64 experts
  // 95 MB 42.5 / 39.7, 32 experts 20 MB 21.6 / 19.4, 38 MB 26.1 / 24.0; d = 4096, 60 experts 6.4 MB 26.2 / 26.2, 22.5 MB 28.4 /
  // 28.4, 45 MB 31.3 / 30.9, 32 experts 3.2 MB 24.8 / 23.4.  So d = 2048 has no reason for a line any more; which form a context
  // takes is something callers can ask for, and it is left as it was.
  // MOE_FUSE_BOUNDARY=0 / 1 and MOE_ROUTE_EVERYWHERE=0 / 1 in the environment override the two rules.
  const int64_t records = (int64_t)cfg->top_k * cfg->inter + cfg->shared_inter, streamed = records * c->slot_layout.rec_bytes;
  // (whichever form is taken: what a wrong x_dev meets depends on the shared expert's share alone)
  c->x_fixed = 3 * (int64_t)cfg->shared_inter >= records;
  const bool int4 = cfg->weight_fmt == MOE_W_INT4_G128;
  c->fuse_boundary = !int4 && c->x_fixed && cfg->shared_inter * c->slot_layout.rec_bytes >= (int64_t)20000 * cfg->hidden;
  c->route_everywhere = gate_rows_supported(cfg->hidden, cfg->act_fmt) && (cfg->hidden >= 1024 || streamed >= 10000000);
  c->everywhere_cumsum = c->route_everywhere && (!int4 || (cfg->hidden < 4096 ? N <= 32 && streamed >= 36000000
                                                                               : N <= 32 || streamed >= 20000000));
  if (const char *s = getenv("MOE_FUSE_BOUNDARY")) c->fuse_boundary = c->x_fixed = atoi(s) != 0;
  c->x_fixed = c->x_fixed && gemv_fused_supported(cfg->weight_fmt, cfg->act_fmt, cfg->hidden, c->plan);
  if (const char *s = getenv("MOE_ROUTE_EVERYWHERE"))
    c->route_everywhere = c->everywhere_cumsum = atoi(s) != 0 && gate_rows_supported(cfg->hidden, cfg->act_fmt);
  if (const char *s = getenv("MOE_POISON_FILLS")) c->poison_fills = atoi(s) != 0;
  if (const char *s = getenv("MOE_TAG_SPINS")) if (atoi(s) > 0) c->tag_spins = atoi(s);
  // The host tier as the device sees it, for launches that bring in the experts that miss: only if all of it is pinned
  // memory (MOE_DEVICE_FILLS=0: the host enqueues every fill)
  bool mapped = !c->poison_fills;
  if (const char *s = getenv("MOE_DEVICE_FILLS")) mapped = mapped && atoi(s) != 0;
  std::vector<const uint8_t *> dev_blob((size_t)L * N);
  for (size_t i = 0; mapped && i < dev_blob.size(); ++i) {
    void *first = nullptr, *last = nullptr;
    uint8_t *host = static_cast<uint8_t *>(const_cast<void *>(c->host_blob[i]));
    const size_t end = (size_t)c->slot_layout.total - 1;
    mapped = hipHostGetDevicePointer(&first, host, 0) == hipSuccess && hipHostGetDevicePointer(&last, host + end, 0) == hipSuccess &&
             static_cast<uint8_t *>(last) == static_cast<uint8_t *>(first) + end && reinterpret_cast<uintptr_t>(first) % 16 == 0;
    dev_blob[i] = static_cast<const uint8_t *>(first);
  }
  if (mapped) {
    HIP_INIT(hipMalloc(&c->d_host_blob, sizeof(void *) * dev_blob.size()));
    HIP_INIT(hipMemcpy(c->d_host_blob, dev_blob.data(), sizeof(void *) * dev_blob.size(), hipMemcpyHostToDevice));
  } else {
    (void)hipGetLastError();  // (memory that is not pinned is no error)
  }
  HIP_INIT(hipMalloc(&c->d_initial, sizeof(int32_t) * (size_t)L * (b->n_initial > 0 ? b->n_initial : 1)));
  HIP_INIT(hipMalloc(&c->d_partial, sizeof(float) * 2 * (size_t)c->plan.grid * cfg->hidden));
  HIP_INIT(hipMalloc(&c->d_y, sizeof(float) * (size_t)cfg->hidden));
  c->batch_ok = batch_shape_supported(cfg->weight_fmt, cfg->act_fmt, cfg->hidden, cfg->inter, cfg->shared_inter);
  if (c->batch_ok) {
    // a tile is 16 tokens of one expert: at most one partly filled tile per slot plus the full ones
    const int64_t routed_tiles = cfg->capacity + kMaxBatch * cfg->top_k / 16;
    const int64_t h_blocks = routed_tiles * ((cfg->inter + 31) / 32) + kMaxBatch / 16 * ((cfg->shared_inter + 31) / 32);
    HIP_INIT(hipMalloc(&c->d_logits_batch, sizeof(float) * kMaxBatch * MOE_MAX_EXPERTS));
    HIP_INIT(hipHostMalloc(reinterpret_cast<void **>(&c->batch_rec), sizeof(moe_route_out_t) * kMaxBatch,
                           hipHostMallocMapped | hipHostMallocCoherent));
    HIP_INIT(hipHostGetDevicePointer(reinterpret_cast<void **>(&c->batch_rec_dev), c->batch_rec, 0));
    HIP_INIT(hipHostMalloc(reinterpret_cast<void **>(&c->h_done), sizeof(uint32_t), hipHostMallocMapped | hipHostMallocCoherent));
    *c->h_done = 0;
    HIP_INIT(hipHostGetDevicePointer(reinterpret_cast<void **>(&c->h_done_dev), c->h_done, 0));
    HIP_INIT(hipMalloc(&c->d_bsel, sizeof(BatchSel)));
    HIP_INIT(hipMalloc(&c->d_bahead, sizeof(BatchAhead)));
    HIP_INIT(hipMalloc(&c->d_bplan, sizeof(BatchPlan)));
    HIP_INIT(hipMalloc(&c->d_bh, (size_t)h_blocks * 2048));
    HIP_INIT(hipMalloc(&c->d_bpartial, sizeof(float) * (size_t)kMaxPartialRows * cfg->hidden));
    HIP_INIT(hipEventCreateWithFlags(&c->ev_batch, hipEventDisableTiming));
  }
  HIP_INIT(hipEventCreateWithFlags(&c->ev_route, hipEventDisableTiming));
  for (int l = 0; l < L; ++l) HIP_INIT(hipEventCreateWithFlags(&c->ev_copy[l], hipEventDisableTiming));
#undef HIP_INIT
  int rc = do_reset(c);
  if (rc != MOE_OK) return bail(rc);
  *out = c;
  return MOE_OK;
}

void moe_cache_destroy(moe_cache_t *c) {
  if (!c) return;
  (void)hipStreamSynchronize(c->compute);
  (void)hipStreamSynchronize(c->copy);
  g_turn[c->dev].give_back(c);
  if (c->d_state) (void)hipFree(c->d_state);
  if (c->d_logits) (void)hipFree(c->d_logits);
  if (c->d_route) (void)hipFree(c->d_route);
  if (c->h_note) (void)hipHostFree(c->h_note);
  if (c->h_rec) (void)hipHostFree(c->h_rec);
  if (c->h_done) (void)hipHostFree(c->h_done);
  if (c->d_handover) (void)hipFree(c->d_handover);
  if (c->d_ss) (void)hipFree(c->d_ss);
  if (c->h_gave_up) (void)hipHostFree(c->h_gave_up);
  if (c->d_initial) (void)hipFree(c->d_initial);
  if (c->d_host_blob) (void)hipFree(c->d_host_blob);
  if (c->d_partial) (void)hipFree(c->d_partial);
  if (c->d_y) (void)hipFree(c->d_y);
  if (c->d_logits_batch) (void)hipFree(c->d_logits_batch);
  if (c->batch_rec) (void)hipHostFree(c->batch_rec);
  if (c->d_bpartial) (void)hipFree(c->d_bpartial);
  if (c->d_bsel) (void)hipFree(c->d_bsel);
  if (c->d_bahead) (void)hipFree(c->d_bahead);
  if (c->d_bplan) (void)hipFree(c->d_bplan);
  if (c->d_bh) (void)hipFree(c->d_bh);
  if (c->ev_batch) (void)hipEventDestroy(c->ev_batch);
  if (c->ev_route) (void)hipEventDestroy(c->ev_route);
  for (hipEvent_t e : c->ev_copy)
    if (e) (void)hipEventDestroy(e);
  for (auto &pr : c->prof_events) {
    (void)hipEventDestroy(pr.first);
    (void)hipEventDestroy(pr.second);
  }
  delete c;
}

// Wait until the routing decision of `layer` (tag `seq`) is visible on the host and decode it into decided[layer].
static int read_note(moe_cache_t *c, int32_t layer, uint32_t seq) {
  const moe_cache_config_t &g = c->cfg;
  const HostNote *h = c->h_note + layer;
  const uint64_t tag = seq & 0xffffu;
  uint64_t w0 = 0, w1 = 0, w2 = 0;
  auto arrived = [&]() {
    w0 = __atomic_load_n(&h->w[0], __ATOMIC_ACQUIRE);
    w1 = __atomic_load_n(&h->w[1], __ATOMIC_ACQUIRE);
    w2 = __atomic_load_n(&h->w[2], __ATOMIC_ACQUIRE);
    return (uint32_t)w0 == seq && (w1 & 0xffffu) == tag && (w2 & 0xffffu) == tag;
  };
  bool ok;
  if (int rc = wait_for(c, arrived, &ok)) return rc;
  if (!ok) return fail(MOE_EHIP, "route kernel of layer %d did not publish its result", layer);
  moe_cache::Decision &d = c->decided[layer];
  d.n_miss = (int)((w0 >> 32) & 0xff);
  d.miss_mask = (uint8_t)((w0 >> 40) & 0xff);
  for (int k = 0; k < g.top_k; ++k) {
    d.expert[k] = (uint8_t)((w1 >> (16 + 6 * k)) & 63);
    d.slot[k] = (uint8_t)((w2 >> (16 + 6 * k)) & 63);
  }
  return MOE_OK;
}

// The same, then the fills of the missed experts are enqueued on the copy stream.  Returns the number of misses.
static int collect_route(moe_cache_t *c, int32_t layer, uint32_t seq, int *n_miss) {
  if (int rc = read_note(c, layer, seq)) return rc;
  const moe_cache_config_t &g = c->cfg;
  const moe_cache::Decision &d = c->decided[layer];
  const size_t slot_bytes = (size_t)c->slot_layout.total;
  if (d.n_miss > 0) {
    for (int k = 0; k < g.top_k; ++k) {
      if (!((d.miss_mask >> k) & 1)) continue;
      const int e = d.expert[k], s = d.slot[k];
      if (e >= g.n_experts || s >= g.capacity)
        return fail(MOE_EHIP, "route kernel returned expert %d slot %d out of range", e, s);
      // (debugging aid: whatever uses the slot before the fill has landed then computes NaNs, which no parity
      // test lets pass)
      if (c->poison_fills)
        HIP_TRY(hipMemsetAsync(static_cast<uint8_t *>(c->slot_pool[layer]) + (size_t)s * slot_bytes, 0xff, slot_bytes, c->copy));
      HIP_TRY(hipMemcpyAsync(static_cast<uint8_t *>(c->slot_pool[layer]) + (size_t)s * slot_bytes,
                             c->host_blob[(size_t)layer * g.n_experts + e], slot_bytes, hipMemcpyHostToDevice,
                             c->copy));
    }
    HIP_TRY(hipEventRecord(c->ev_copy[layer], c->copy));
  }
  *n_miss = d.n_miss;
  return MOE_OK;
}

// the full decision record of a layer, from device memory (waits for the compute stream)
static int fetch_record(moe_cache_t *c, int32_t layer, moe_route_out_t *out) {
  HIP_TRY(hipMemcpyAsync(out, c->d_route + layer, sizeof *out, hipMemcpyDeviceToHost, c->compute));
  return sync_compute(c);
}

static RouteParams make_route_params(moe_cache_t *c) {
  const moe_cache_config_t &g = c->cfg;
  RouteParams p{};
  p.n_experts = g.n_experts;
  p.top_k = g.top_k;
  p.top_j = g.top_j;
  p.capacity = g.capacity;
  p.hidden = g.hidden;
  p.act_fmt = g.act_fmt;
  p.renormalize = g.renormalize;
  p.delta_mode = g.delta_mode;
  p.route_mode = g.route_mode;
  p.max_rank = g.max_rank;
  p.lambda = g.lambda;
  p.delta_fixed = g.delta_fixed;
  p.cumsum_p = g.cumsum_p;
  if (++c->seq == 0) c->seq = 1;
  p.seq = c->seq;
  return p;
}

// Runs what is left of a layer's deferred boundary now, in launches of its own (the same operations in the same order: x,
// logits and decision are those of the launch it was deferred into); the layer's step is then one like any other whose
// decision is not collected yet.
static int settle(moe_cache_t *c, int32_t layer) {
  if (c->routed[layer] < 3) return MOE_OK;
  const BoundaryArgs &b = c->boundary[layer];
  float *logits = c->d_logits + (size_t)layer * MOE_MAX_EXPERTS;
  if (c->routed[layer] == 3) HIP_TRY(launch_gate_rows(b.route, b.glue, c->gate_w[layer], logits, c->compute));
  HIP_TRY(launch_route(b.route, nullptr, nullptr, logits, c->state(layer), c->d_route + layer,
                       HostOut{c->h_note_dev + layer, nullptr}, c->compute));
  if (c->deferred == layer) c->deferred = -1;
  c->routed[layer] = 2;
  return MOE_OK;
}

// after the router launch: either leave the decision for moe_expert_forward, or wait for it now
// (with_outputs: the launch writes h and x for the caller, who may use them on any stream once the call returns)
static int finish_route_call(moe_cache_t *c, int32_t layer, uint32_t seq, moe_route_out_t *out_host, bool with_outputs) {
  c->route_seq[layer] = seq;
  if (!out_host) {
    c->routed[layer] = 2;  // decision collected by moe_expert_forward, behind the first expert launch
    return MOE_OK;
  }
  int n_miss = 0;
  if (int rc = collect_route(c, layer, seq, &n_miss)) return rc;
  c->routed[layer] = 1;
  // the record follows the decision by a microsecond
  uint32_t w[kHostRecWords];
  bool ok;
  const auto arrived = [&]() {
    bool all = true;
    for (int i = 0; i < kHostRecWords; ++i) {
      const uint64_t v = __atomic_load_n(&c->h_rec->w[i], __ATOMIC_ACQUIRE);
      w[i] = (uint32_t)v;
      all &= (uint32_t)(v >> 32) == seq;
    }
    return all && (!with_outputs || (uint32_t)__atomic_load_n(&c->h_rec->outputs, __ATOMIC_ACQUIRE) == seq);
  };
  if (int rc = wait_for(c, arrived, &ok)) return rc;
  if (!ok) return fail(MOE_EHIP, "route kernel of layer %d did not publish its record", layer);
  static_assert(sizeof w == sizeof *out_host, "record words");
  memcpy(out_host, w, sizeof w);
  return MOE_OK;
}

// the routing of a step is left to every workgroup of its expert launch, which starts from the logits
static void defer_routing(moe_cache_t *c, int32_t layer, const RouteParams &p, const float *logits) {
  BoundaryArgs &b = c->boundary[layer];
  b = BoundaryArgs{};
  b.route = p;
  b.state = c->state(layer);
  b.state_out = c->d_state + (size_t)(1 - c->cur[layer]) * c->cfg.n_layers + layer;
  b.logits = logits;
  b.out_dev = c->d_route + layer;
  b.note = c->h_note_dev + layer;
  c->route_seq[layer] = p.seq;
  c->routed[layer] = 4;
}

// whether that is the better way (see moe_cache_init)
static bool routed_everywhere(const moe_cache_t *c) {
  return c->cfg.route_mode == MOE_ROUTE_CUMSUM ? c->everywhere_cumsum : c->route_everywhere;
}

int moe_route_step(moe_cache_t *c, int32_t layer, const void *x_dev, const float *logits_dev,
                   moe_route_out_t *out_host) {
  if (int rc = check_layer(c, layer)) return rc;
  if ((x_dev == nullptr) == (logits_dev == nullptr)) return fail(MOE_EINVAL, "exactly one of x_dev and logits_dev must be given");
  if (c->routed[layer]) return fail(MOE_ESTATE, "layer %d: previous route step not followed by moe_expert_forward", layer);
  if (c->pending_rows) return fail(MOE_ESTATE, "an expert output is pending: the next routing call must be moe_stack_route_step");
  if (c->batch_layer >= 0) return fail(MOE_ESTATE, "a routed batch is pending: call moe_expert_forward_batch first");
  c->x_given[layer] = nullptr;
  c->logits_given[layer] = logits_dev != nullptr;
  const RouteParams p = make_route_params(c);
  if (!out_host && x_dev && routed_everywhere(c)) {
    // nobody waits: only the logits are made by this call, over several compute units (route_kernel takes 8.9 us for 8 experts
    // of d = 4096 or 64 of d = 2048, the logits alone 3)
    float *logits = c->d_logits + (size_t)layer * MOE_MAX_EXPERTS;
    HIP_TRY(launch_gate_x(p, x_dev, c->gate_w[layer], logits, c->compute));
    defer_routing(c, layer, p, logits);
    return MOE_OK;
  }
  HIP_TRY(launch_route(p, c->gate_w[layer], x_dev, logits_dev, c->state(layer), c->d_route + layer,
                       HostOut{c->h_note_dev + layer, out_host ? c->h_rec_dev : nullptr}, c->compute));
  return finish_route_call(c, layer, p.seq, out_host, false);
}

// how a boundary that nobody waits for is run (see moe_cache_init)
static int boundary_form(const moe_cache_t *c) {
  if (c->fuse_boundary && gemv_fused_supported(c->cfg.weight_fmt, c->cfg.act_fmt, c->cfg.hidden, c->plan))
    return MOE_BOUNDARY_IN_FIRST_WORKGROUP;
  return routed_everywhere(c) ? MOE_BOUNDARY_ROUTED_EVERYWHERE : MOE_BOUNDARY_OWN_LAUNCH;
}

int moe_stack_route_step(moe_cache_t *c, int32_t layer, float *h_dev, const float *a_dev, float perturb,
                         int32_t carry, void *x_dev, void *y_dev, moe_route_out_t *out_host) {
  if (int rc = check_layer(c, layer)) return rc;
  if (!h_dev || !x_dev) return fail(MOE_EINVAL, "h_dev or x_dev is NULL");
  if (c->cfg.hidden > kFusedMaxHidden) return fail(MOE_EINVAL, "hidden exceeds %d", kFusedMaxHidden);
  if (c->routed[layer]) return fail(MOE_ESTATE, "layer %d: previous route step not followed by moe_expert_forward", layer);
  if (c->batch_layer >= 0) return fail(MOE_ESTATE, "a routed batch is pending: call moe_expert_forward_batch first");
  // h may be the one another layer's deferred boundary is still to be formed from, d_ss is
  if (c->deferred >= 0)
    if (int rc = settle(c, c->deferred)) return rc;
  c->x_given[layer] = !out_host && c->x_fixed ? x_dev : nullptr;
  c->logits_given[layer] = 0;
  const RouteParams p = make_route_params(c);
  const int form = out_host ? MOE_BOUNDARY_OWN_LAUNCH : boundary_form(c);
  // the pending expert output is summed first (into y_dev if given, else into the library's own buffer)
  void *y = nullptr;
  if (c->pending_rows > 0) y = y_dev ? y_dev : c->d_y;
  FusedParams f{};
  f.h = h_dev;
  f.x_out = x_dev;
  if (form == MOE_BOUNDARY_IN_FIRST_WORKGROUP) {
    // nobody waits for the decision here: the sum of the pending output and the residual glue are one launch, and
    // the rest of the boundary (x, gate GEMV, routing) runs in workgroup 0 of the layer's expert launch
    HIP_TRY(launch_reduce_glue(c->d_partial, c->pending_rows, c->pending_miss, y, c->cfg.hidden, c->cfg.act_fmt, h_dev, a_dev, perturb,
                               carry, c->d_ss, c->compute));
    c->pending_rows = 0;
    f.ss = c->d_ss;
    f.n_ss = c->cfg.hidden / 64;
    BoundaryArgs &b = c->boundary[layer];
    b.route = p;
    b.glue = f;
    b.gate_w = c->gate_w[layer];
    b.state = c->state(layer);
    b.out_dev = c->d_route + layer;
    b.note = c->h_note_dev + layer;
    b.handover = c->d_handover + 64 * (size_t)layer;
    b.hand_tag = ++c->hand_count[layer] & 0xffffu;  // the words hold count - 1 (0 at first): never equal
    b.gave_up = c->h_gave_up_dev;
    b.spin_limit = c->tag_spins;
    b.next_gate_w = c->gate_w[(layer + 1) % c->cfg.n_layers];
    b.next_state = c->state((layer + 1) % c->cfg.n_layers);
    b.gate_bytes = (int64_t)c->cfg.n_experts * c->cfg.hidden * (c->cfg.act_fmt == MOE_A_BF16 ? 2 : 4);
    c->route_seq[layer] = p.seq;
    c->routed[layer] = 3;
    c->deferred = layer;
    return MOE_OK;
  }
  if (form == MOE_BOUNDARY_ROUTED_EVERYWHERE) {
    // nobody waits for the decision here: only x and the logits are made by this call (over several compute units), and
    // every workgroup of the layer's expert launch routes for itself.  (Doing the glue in the gate launch where a token begins
    // saves a launch a token: 272 -> 266 us for 12 layer-tokens in stacks of 3 layers, less than 1 % in deeper ones; not done.)
    HIP_TRY(launch_reduce_glue(c->d_partial, c->pending_rows, c->pending_miss, y, c->cfg.hidden, c->cfg.act_fmt, h_dev, a_dev, perturb,
                               carry, c->d_ss, c->compute));
    f.ss = c->d_ss;
    f.n_ss = c->cfg.hidden / 64;
    c->pending_rows = 0;
    float *logits = c->d_logits + (size_t)layer * MOE_MAX_EXPERTS;
    HIP_TRY(launch_gate_rows(p, f, c->gate_w[layer], logits, c->compute));
    defer_routing(c, layer, p, logits);
    return MOE_OK;
  }
  if (fused_route_pre_supported(c->cfg.hidden)) {
    // the sum of the pending output and the residual glue spread over d / 64 workgroups; the single-workgroup
    // boundary launch then starts from h and the sums of squares
    HIP_TRY(launch_reduce_glue(c->d_partial, c->pending_rows, c->pending_miss, y, c->cfg.hidden, c->cfg.act_fmt, h_dev, a_dev, perturb,
                               carry, c->d_ss, c->compute));
    f.ss = c->d_ss;
    f.n_ss = c->cfg.hidden / 64;
  } else {
    if (c->pending_rows > 0)
      HIP_TRY(launch_partial_reduce(c->d_partial, c->pending_rows, c->pending_miss, y, c->cfg.hidden, c->cfg.act_fmt, c->compute));
    f.y = y;
    f.a = a_dev;
    f.perturb = perturb;
    f.carry = carry;
  }
  c->pending_rows = 0;
  HIP_TRY(launch_fused_route(p, f, c->gate_w[layer], c->state(layer), c->d_route + layer,
                             HostOut{c->h_note_dev + layer, out_host ? c->h_rec_dev : nullptr}, c->compute));
  return finish_route_call(c, layer, p.seq, out_host, true);
}

int moe_expert_forward(moe_cache_t *c, int32_t layer, const void *x_dev, void *y_dev) {
  if (int rc = check_layer(c, layer)) return rc;
  if (!x_dev) return fail(MOE_EINVAL, "x_dev is NULL");
  if (!c->routed[layer]) return fail(MOE_ESTATE, "layer %d: moe_expert_forward without a preceding moe_route_step", layer);
  if (c->pending_rows) return fail(MOE_ESTATE, "an expert output is pending: call moe_stack_route_step first");
  if (c->x_given[layer] && x_dev != c->x_given[layer])
    return fail(MOE_EINVAL, "layer %d: x_dev must be the vector moe_stack_route_step wrote", layer);
  const moe_cache_config_t &g = c->cfg;
  GemvParams p{};
  p.slot_pool = static_cast<const uint8_t *>(c->slot_pool[layer]);
  p.shared_blob = g.shared_inter > 0 ? static_cast<const uint8_t *>(c->shared_blob[layer]) : nullptr;
  p.route = c->d_route + layer;
  p.x = x_dev;
  p.partial = c->d_partial;
  p.hidden = g.hidden;
  p.inter = g.inter;
  p.shared_inter = g.shared_inter;
  p.top_k = g.top_k;
  p.act_fmt = g.act_fmt;
  p.slot_bytes = c->slot_layout.total;
  // A step that nobody waited for: the launch itself brings in what misses, and the host, which need not know the decision,
  // is free to go on (with a wait in each layer it was what bounded a stack of small layers: 36 MB of int4 a layer-token 20.6 us
  // a layer, 12.9 without; 101 MB of bf16 26.4 / 20.9).  Otherwise, and where the host tier is not mapped on the device, a
  // first pass covers the shared expert and the experts that were resident, the host enqueues the fills, and a second pass
  // covers the experts filled.
  const bool on_device = c->d_host_blob != nullptr && c->routed[layer] >= 2;
  if (on_device) {
    hipStreamCaptureStatus capturing = hipStreamCaptureStatusNone;
    HIP_TRY(hipStreamIsCapturing(c->compute, &capturing));
    if (capturing != hipStreamCaptureStatusNone)  // (a replay would repeat this step's tags and state)
      return fail(MOE_EHIP, "layer %d: a routed step cannot be captured into a graph", layer);
    p.host_blob = c->d_host_blob + (size_t)layer * g.n_experts;
    p.missing_row = c->plan.grid;
  }
  p.pass = 0;
  p.row_offset = 0;
  if (c->routed[layer] == 3 && !g_turn[c->dev].take(c, &c->h_note[layer].w[0], c->route_seq[layer])) {
    // another context's launch may still be waiting for its first workgroup: the boundary ahead of the launch, the routing in
    // every workgroup.  (The first workgroup still streams nothing, so that the sums are those of the other form.)
    BoundaryArgs &b = c->boundary[layer];
    float *logits = c->d_logits + (size_t)layer * MOE_MAX_EXPERTS;
    HIP_TRY(launch_gate_rows(b.route, b.glue, c->gate_w[layer], logits, c->compute));
    if (c->deferred == layer) c->deferred = -1;
    defer_routing(c, layer, RouteParams(b.route), logits);
    p.idle_row = 1;
  }
  if (c->routed[layer] == 3) {
    p.route_in = kRouteBoundary;
    p.b = c->boundary[layer];
  } else if (c->routed[layer] == 4) {
    p.route_in = kRouteEverywhere;
    p.b = c->boundary[layer];
  }
  const bool prof = c->profiling && c->prof_tick++ % (uint64_t)c->profiling == 0 && c->prof_used < c->prof_events.size();
  if (prof) {
    hipLaunchKernelGGL(hold_stream_kernel, dim3(1), dim3(64), 0, c->compute, (uint64_t)5000);  // 50 us
    HIP_TRY(hipGetLastError());
  }
  const hipError_t launched = launch_expert_gemv(p, g.weight_fmt, c->plan, c->compute, prof ? c->prof_events[c->prof_used].first : nullptr,
                                                 prof ? c->prof_events[c->prof_used].second : nullptr);
  if (launched != hipSuccess) {
    g_turn[c->dev].give_back(c);
    return fail(MOE_EHIP, "expert launch of layer %d: %s", layer, hipGetErrorString(launched));
  }
  if (c->deferred == layer) c->deferred = -1;
  if (p.route_in == kRouteEverywhere) c->cur[layer] ^= 1;  // the launch writes the other copy of the state
  p.route_in = kRouteBefore;
  int n_miss = c->decided[layer].n_miss;
  if (on_device) {
    n_miss = 0;
    if (prof) {
      if (int rc = read_note(c, layer, c->route_seq[layer])) return rc;
      c->prof_full[c->prof_used++] = c->decided[layer].n_miss == 0;
    }
  } else if (c->routed[layer] >= 2) {
    if (int rc = collect_route(c, layer, c->route_seq[layer], &n_miss)) return rc;
  }
  if (prof && !on_device) c->prof_full[c->prof_used++] = n_miss == 0;
  int rows = c->plan.grid;
  if (n_miss > 0) {
    // pass 1: the experts whose slots are being filled, once the fills have landed
    HIP_TRY(hipStreamWaitEvent(c->compute, c->ev_copy[layer], 0));
    p.pass = 1;
    p.row_offset = c->plan.grid;
    HIP_TRY(launch_expert_gemv(p, g.weight_fmt, c->plan, c->compute));
    rows = 2 * c->plan.grid;
  }
  const int32_t *misses = on_device ? &c->d_route[layer].n_miss : nullptr;
  if (y_dev) {
    HIP_TRY(launch_partial_reduce(c->d_partial, rows, misses, y_dev, g.hidden, g.act_fmt, c->compute));
  } else {
    c->pending_rows = rows;  // finished by the next moe_stack_route_step
    c->pending_miss = misses;
  }
  c->routed[layer] = 0;
  // the caller's logits are the caller's again when this call returns: the decision says that they have been read
  if (on_device && c->logits_given[layer]) return read_note(c, layer, c->route_seq[layer]);
  return MOE_OK;
}

int moe_expert_forward_static(int32_t weight_fmt, int32_t act_fmt, int32_t hidden, int32_t inter, int32_t shared_inter,
                              int32_t top_k, const void *slot_pool_dev, int32_t n_slots, const void *shared_blob_dev,
                              const int32_t *sel_slot_host, const float *sel_weight_host, const void *x_dev,
                              void *y_dev, void *stream) {
  if (!valid_wfmt(weight_fmt) || !valid_afmt(act_fmt)) return fail(MOE_EINVAL, "unknown weight or activation format");
  if (hidden <= 0 || hidden > static_max_hidden())
    return fail(MOE_EINVAL, "hidden=%d beyond the fixed scratch buffer of this entry point (at most %d)", hidden, static_max_hidden());
  if (!gemv_shape_supported(weight_fmt, hidden)) return fail(MOE_EINVAL, "hidden=%d unsupported for weight format %d", hidden, weight_fmt);
  if (inter <= 0 || shared_inter < 0 || !gemv_inter_supported(weight_fmt, inter) ||
      (shared_inter > 0 && !gemv_inter_supported(weight_fmt, shared_inter)))
    return fail(MOE_EINVAL, "intermediate size unsupported for this weight format");
  if (top_k <= 0 || top_k > MOE_MAX_TOPK) return fail(MOE_EINVAL, "top_k must be in 1..%d", MOE_MAX_TOPK);
  if ((int64_t)top_k * inter + shared_inter > (int64_t)1 << 22) return fail(MOE_EINVAL, "more than 2^22 expert records");
  if (n_slots <= 0 || n_slots > 256) return fail(MOE_EINVAL, "n_slots must be in 1..256");
  if (!slot_pool_dev || !sel_slot_host || !sel_weight_host || !x_dev || !y_dev) return fail(MOE_EINVAL, "NULL argument");
  if (shared_inter > 0 && !shared_blob_dev) return fail(MOE_EINVAL, "shared_inter > 0 needs shared_blob_dev");
  for (int k = 0; k < top_k; ++k) {
    if (sel_slot_host[k] < 0 || sel_slot_host[k] >= n_slots) return fail(MOE_EINVAL, "sel_slot[%d]=%d outside 0..%d", k, sel_slot_host[k], n_slots - 1);
    if (!std::isfinite(sel_weight_host[k])) return fail(MOE_EINVAL, "sel_weight[%d] is not finite", k);
  }
  const int64_t slot_bytes = blob_layout(weight_fmt, hidden, inter).total;
  HIP_TRY(launch_expert_forward_static(weight_fmt, act_fmt, hidden, inter, shared_inter, top_k, slot_pool_dev, slot_bytes,
                                       shared_blob_dev, sel_slot_host, sel_weight_host, x_dev, y_dev,
                                       static_cast<hipStream_t>(stream)));
  return MOE_OK;
}

namespace {
struct BatchUnits {
  int up_records, down_groups;  // records per unit of up_batch_kernel, groups of 32 records per unit of down_batch_kernel
  int n_rc, n_rc_shared;        // blocks of records of down_batch_kernel per routed expert / of the shared expert
};
BatchUnits batch_units(int groups, int inter, int shared_groups, int shared_inter, int hidden, int n_seg, int top_k, int n_cus) {
  BatchUnits u{};
  const int sh = shared_groups ? shared_inter : 0;
  int64_t best = kNoCandidate;
  for (int cand = 32; cand <= 32 * batch_up_candidates(inter, sh); cand += 32) {
    const int64_t est = batch_up_estimate(cand, groups, inter, shared_groups, sh, hidden, n_cus);
    if (est <= best) best = est, u.up_records = cand;
  }
  best = kNoCandidate;
  u.down_groups = 4;
  for (int cand = 4; cand <= 4 * batch_down_candidates(inter, sh); cand += 4) {
    const int64_t est = batch_down_estimate(cand, groups, inter, shared_groups, sh, hidden, n_seg, top_k, n_cus);
    if (est <= best) best = est, u.down_groups = cand;
  }
  u.n_rc = batch_parts(batch_parts(inter, 32), u.down_groups);
  u.n_rc_shared = batch_parts(batch_parts(sh, 32), u.down_groups);
  return u;
}
}  // namespace

// what the expert kernels of a batch of the layer take, but for the list of experts
static BatchArgs batch_args(const moe_cache_t *c, int32_t layer, const void *x_dev, int n_tokens) {
  const moe_cache_config_t &g = c->cfg;
  BatchArgs a{};
  a.slot_pool = static_cast<const uint8_t *>(c->slot_pool[layer]);
  a.shared_blob = g.shared_inter > 0 ? static_cast<const uint8_t *>(c->shared_blob[layer]) : nullptr;
  a.x = static_cast<const uint16_t *>(x_dev);
  a.sel = c->d_bsel;
  a.h = c->d_bh;
  a.partial = c->d_bpartial;
  a.slot_bytes = (int64_t)c->slot_layout.total;
  a.hidden = g.hidden;
  a.inter = g.inter;
  a.shared_inter = g.shared_inter;
  a.top_k = g.top_k;
  a.t0 = 0;
  a.t1 = n_tokens;
  return a;
}

int moe_route_batch(moe_cache_t *c, int32_t layer, const void *x_dev, const float *logits_dev, int32_t n_tokens,
                    moe_route_out_t *out_host) {
  if (int rc = check_layer(c, layer)) return rc;
  if (!c->batch_ok) return fail(MOE_EINVAL, "the prompt-phase kernels take bf16 weights and activations, hidden 1024 or 2048, intermediate sizes that are multiples of 16");
  if ((x_dev == nullptr) == (logits_dev == nullptr)) return fail(MOE_EINVAL, "exactly one of x_dev and logits_dev must be given");
  if (n_tokens <= 0 || n_tokens > kMaxBatch) return fail(MOE_EINVAL, "n_tokens must be in 1..%d", kMaxBatch);
  if (c->routed[layer] || c->pending_rows || c->batch_layer >= 0)
    return fail(MOE_ESTATE, "layer %d: a routing step, an expert output or a routed batch is pending", layer);
  const float *z = logits_dev;
  if (x_dev) {
    HIP_TRY(launch_gate_gemm(x_dev, c->gate_w[layer], c->d_logits_batch, n_tokens, c->cfg.n_experts, c->cfg.hidden, c->compute));
    z = c->d_logits_batch;
  }
  const RouteParams p = make_route_params(c);
  // x_dev is what moe_expert_forward_batch will be given: the expert kernels follow the routing at once, with a list of experts
  // made there (it is empty if something misses), and run while the host takes its turn (15 us between the two calls' launches).
  // What is left for moe_expert_forward_batch is the sum per token.
  const BatchPlanFor planned{x_dev ? c->d_bplan : nullptr, c->cfg.hidden, c->cfg.inter, c->cfg.shared_inter, c->n_cus};
  c->batch_x = nullptr;
  HIP_TRY(launch_route_batch(p, z, n_tokens, c->state(layer), c->batch_rec_dev, c->d_bsel, c->d_bahead, c->h_done_dev, planned, c->compute));
  if (x_dev) {
    HIP_TRY(launch_planned_experts(batch_args(c, layer, x_dev, n_tokens), c->d_bplan, c->n_cus, c->compute));
    c->batch_x = x_dev;
  }
  bool ok;
  if (int rc = wait_for(c, [&]() { return __atomic_load_n(c->h_done, __ATOMIC_ACQUIRE) == p.seq; }, &ok)) return rc;
  if (!ok) return fail(MOE_EHIP, "batch routing of layer %d did not publish its records", layer);
  const moe_cache_config_t &g = c->cfg;
  BatchPlaces places;
  if (const moe_route_out_t *r = places.count(c->batch_rec, n_tokens, g.top_k, g.n_experts, g.capacity)) {
    c->batch_x = nullptr;
    return fail(MOE_EHIP, "batch routing returned an expert or a slot out of range (token %d)", r->token);
  }
  if (places.misses > 0) c->batch_x = nullptr;
  if (c->batch_x) {  // the device's list has to fit its launches (see make_plan)
    const int sg = g.shared_inter > 0 ? batch_parts(n_tokens, 64) : 0;
    int groups = 0, n_up = 0, n_down = 0, up, down;
    for (int n : places.of_slot) groups += batch_parts(n, 64);
    const BatchUnits bu = batch_units(groups, g.inter, sg, g.shared_inter, g.hidden, n_tokens, g.top_k, c->n_cus);
    const auto add = [&](int n, int rows) {
      batch_entry_units(n, rows, bu.up_records, bu.down_groups, g.hidden, &up, &down);
      n_up += up;
      n_down += down;
    };
    for (int n : places.of_slot)
      if (n > 0) add(n, g.inter);
    if (sg) add(n_tokens, g.shared_inter);
    if (std::max(n_up, n_down) > kPlanRounds * c->n_cus) c->batch_x = nullptr;
  }
  if (out_host) memcpy(out_host, c->batch_rec, sizeof(moe_route_out_t) * n_tokens);
  c->batch_layer = layer;
  c->batch_n = n_tokens;
  c->batch_misses = places.misses;
  return MOE_OK;
}

int moe_expert_forward_batch(moe_cache_t *c, int32_t layer, const void *x_dev, void *y_dev, int32_t n_tokens) {
  if (int rc = check_layer(c, layer)) return rc;
  if (!x_dev || !y_dev) return fail(MOE_EINVAL, "x_dev or y_dev is NULL");
  if (c->batch_layer != layer || c->batch_n != n_tokens)
    return fail(MOE_ESTATE, "layer %d: moe_expert_forward_batch without a preceding moe_route_batch of %d tokens", layer, n_tokens);
  const moe_cache_config_t &g = c->cfg;
  const int K = g.top_k, d = g.hidden;
  const size_t slot_bytes = (size_t)c->slot_layout.total;
  BatchParams bp{};
  static_cast<BatchArgs &>(bp) = batch_args(c, layer, x_dev, n_tokens);
  if (c->batch_x == x_dev) {  // the expert kernels are on their way
    HIP_TRY(launch_planned_reduce(bp, c->d_bplan, y_dev, c->compute));
    HIP_TRY(hipStreamSynchronize(c->compute));
    c->batch_layer = -1;
    c->batch_n = 0;
    c->batch_x = nullptr;
    return MOE_OK;
  }
  // Segments: maximal runs of tokens during which no slot is refilled after a token of the run has read it, so that
  // all experts a segment needs are in their slots at once.
  int t0 = 0;
  while (t0 < n_tokens) {
    uint64_t read = 0;
    int n_of_slot[MOE_MAX_EXPERTS] = {};
    int t1 = t0;
    for (; t1 < n_tokens; ++t1) {
      const moe_route_out_t &r = c->batch_rec[t1];
      bool conflict = false;
      for (int k = 0; k < K; ++k) conflict |= r.miss[k] && ((read >> r.sel_slot[k]) & 1);
      if (conflict) break;
      for (int k = 0; k < K; ++k) {
        read |= 1ull << r.sel_slot[k];
        ++n_of_slot[r.sel_slot[k]];
      }
    }
    // fills of the segment's misses, once the compute stream has finished with the slots' previous contents
    int n_fill = 0;
    uint64_t filled = 0;  // slots that receive an expert in this segment
    for (int t = t0; t < t1; ++t) {
      const moe_route_out_t &r = c->batch_rec[t];
      for (int k = 0; k < K; ++k) {
        if (!r.miss[k]) continue;
        filled |= 1ull << r.sel_slot[k];
        if (n_fill++ == 0) {  // whatever reads the slots' previous contents is ahead of this point
          HIP_TRY(hipEventRecord(c->ev_batch, c->compute));
          HIP_TRY(hipStreamWaitEvent(c->copy, c->ev_batch, 0));
        }
        if (c->poison_fills)
          HIP_TRY(hipMemsetAsync(static_cast<uint8_t *>(c->slot_pool[layer]) + (size_t)r.sel_slot[k] * slot_bytes, 0xff,
                                 slot_bytes, c->copy));
        HIP_TRY(hipMemcpyAsync(static_cast<uint8_t *>(c->slot_pool[layer]) + (size_t)r.sel_slot[k] * slot_bytes,
                               c->host_blob[(size_t)layer * g.n_experts + r.sel_expert[k]], slot_bytes,
                               hipMemcpyHostToDevice, c->copy));
      }
    }
    c->batch_misses -= n_fill;
    if (n_fill > 0) HIP_TRY(hipEventRecord(c->ev_copy[layer], c->copy));
    // Sizes of the units of the two expert kernels (see batch_units): chosen for the whole segment
    const int n_seg = t1 - t0;
    bp.t0 = t0;
    bp.t1 = t1;
    int one = 0, more = 0;  // experts with one group of 64 tokens, and the groups of those with several (padded below)
    for (uint64_t m = read; m; m &= m - 1) {
      const int n = n_of_slot[__builtin_ctzll(m)];
      if (n <= 64) ++one; else more += (n + 63) / 64;
    }
    const BatchUnits bu = batch_units(one + more, g.inter, g.shared_inter > 0 ? (n_seg + 63) / 64 : 0, g.shared_inter, d, n_seg, K, c->n_cus);
    bp.up_records = bu.up_records;
    bp.down_groups = bu.down_groups;
    bp.shared_row0 = n_seg * K * bu.n_rc;
    // Two sets of launches: the experts that were in their slots already (and the shared expert) at once, behind them
    // those whose slots are being filled, behind the fill event - so the first set computes while the fills stream.
    // Experts with several token groups come first: their unit counts are padded to whole blocks of 8 x groups, which
    // keeps the groups of a block on one XCD (see group_pos).
    uint32_t h_base = 0;
    for (int set = 0; set < 2; ++set) {
      const uint64_t mine = set == 0 ? read & ~filled : read & filled;
      int n_up = 0, n_down = 0;
      bp.n_entries = 0;
      auto add = [&](int slot, int n_tok, int rows) {
        int up, down;
        batch_entry_units(n_tok, rows, bu.up_records, bu.down_groups, d, &up, &down);
        bp.e[bp.n_entries++] = BatchEntry{(int16_t)slot, (uint16_t)n_tok, h_base, (uint32_t)n_up, (uint32_t)n_down};
        h_base += (uint32_t)batch_parts(n_tok, 16) * (uint32_t)batch_parts(rows, 32);
        n_up += up;
        n_down += down;
      };
      for (int pass = 0; pass < 2; ++pass) {
        const bool several = pass == 0;
        if (set == 0 && g.shared_inter > 0 && (n_seg > 64) == several) add(-1, n_seg, g.shared_inter);
        for (uint64_t m = mine; m; m &= m - 1) {
          const int s = __builtin_ctzll(m);
          if ((n_of_slot[s] > 64) == several) add(s, n_of_slot[s], g.inter);
        }
      }
      if (set == 1 && n_fill > 0) HIP_TRY(hipStreamWaitEvent(c->compute, c->ev_copy[layer], 0));
      HIP_TRY(launch_up_batch(bp, n_up, c->compute));
      HIP_TRY(launch_down_batch(bp, n_down, c->compute));
    }
    HIP_TRY(launch_reduce_batch(bp, y_dev, bu.n_rc, bu.n_rc_shared, c->compute));
    t0 = t1;
  }
  HIP_TRY(hipStreamSynchronize(c->compute));
  c->batch_layer = -1;
  c->batch_n = 0;
  c->batch_x = nullptr;
  return MOE_OK;
}

int moe_cache_last_route(moe_cache_t *c, int32_t layer, moe_route_out_t *out) {
  if (int rc = check_layer(c, layer)) return rc;
  if (!out) return fail(MOE_EINVAL, "out is NULL");
  if (c->routed[layer] >= 2) return fail(MOE_ESTATE, "layer %d: routing decision not collected yet", layer);
  return fetch_record(c, layer, out);
}

int moe_cache_stats(moe_cache_t *c, int32_t layer, moe_cache_stats_t *out) {
  if (!c || !out) return fail(MOE_EINVAL, "NULL argument");
  if (int rc = check_layer(c, layer == -1 ? 0 : layer)) return rc;  // also refuses a context whose hand-over was abandoned
  for (int l = 0; l < c->cfg.n_layers; ++l)
    if (layer == -1 || l == layer)
      if (int rc = settle(c, l)) return rc;
  if (int rc = sync_compute(c)) return rc;
  std::vector<LayerState> both(2 * (size_t)c->cfg.n_layers);
  HIP_TRY(hipMemcpy(both.data(), c->d_state, sizeof(LayerState) * both.size(), hipMemcpyDeviceToHost));
  memset(out, 0, sizeof *out);
  for (int l = 0; l < c->cfg.n_layers; ++l) {
    if (layer != -1 && l != layer) continue;
    const LayerState &st = both[(size_t)c->cur[l] * c->cfg.n_layers + l];
    out->tokens += st.count;
    out->selections += st.selections;
    out->hits += st.hits;
    out->misses += st.misses;
    out->cold_misses += st.cold_misses;
    out->evictions += st.evictions;
    out->lifetime_sum += st.lifetime_sum;
    // a miss is a fill, except that those of a step or batch whose moe_expert_forward(_batch) has not been called are still
    // to come
    int32_t to_come = l == c->batch_layer ? c->batch_misses : 0;
    if (c->routed[l] >= 2)
      HIP_TRY(hipMemcpy(&to_come, &c->d_route[l].n_miss, sizeof to_come, hipMemcpyDeviceToHost));
    out->bytes_filled += c->bytes_filled[l] + (st.misses - c->miss_base[l] - to_come) * c->slot_layout.total;
  }
  return MOE_OK;
}

int moe_cache_tables(moe_cache_t *c, int32_t layer, moe_cache_tables_t *out) {
  if (int rc = check_layer(c, layer)) return rc;
  if (!out) return fail(MOE_EINVAL, "out is NULL");
  if (int rc = settle(c, layer)) return rc;
  if (int rc = sync_compute(c)) return rc;
  LayerState st;
  HIP_TRY(hipMemcpy(&st, c->state(layer), sizeof st, hipMemcpyDeviceToHost));
  memcpy(out->expert_slot, st.expert_slot, sizeof out->expert_slot);
  memcpy(out->slot_expert, st.slot_expert, sizeof out->slot_expert);
  memcpy(out->stamp, st.stamp, sizeof out->stamp);
  out->delta_sum = st.delta_sum;
  out->count = st.count;
  return MOE_OK;
}

namespace {
struct SnapshotHeader {
  uint32_t magic, version;
  int32_t n_experts, capacity, top_k, reserved;
};
constexpr uint32_t kSnapMagic = 0x43454f4du, kSnapVersion = 1;  // "MOEC"
constexpr size_t kSnapBytes = sizeof(SnapshotHeader) + sizeof(LayerState);
}  // namespace

int moe_cache_snapshot(moe_cache_t *c, int32_t layer, void *buf, size_t *bytes) {
  if (int rc = check_layer(c, layer)) return rc;
  if (!bytes) return fail(MOE_EINVAL, "bytes is NULL");
  const size_t have = *bytes;
  *bytes = kSnapBytes;
  if (!buf) return MOE_OK;
  if (have < kSnapBytes) return fail(MOE_EINVAL, "snapshot needs %zu bytes, buffer has %zu", kSnapBytes, have);
  if (int rc = settle(c, layer)) return rc;
  if (int rc = sync_compute(c)) return rc;
  SnapshotHeader hd{kSnapMagic, kSnapVersion, c->cfg.n_experts, c->cfg.capacity, c->cfg.top_k, 0};
  memcpy(buf, &hd, sizeof hd);
  HIP_TRY(hipMemcpy(static_cast<uint8_t *>(buf) + sizeof hd, c->state(layer), sizeof(LayerState),
                    hipMemcpyDeviceToHost));
  return MOE_OK;
}

int moe_cache_restore(moe_cache_t *c, int32_t layer, const void *buf, size_t bytes) {
  if (int rc = check_layer(c, layer)) return rc;
  if (!buf || bytes < kSnapBytes) return fail(MOE_EINVAL, "snapshot buffer is NULL or shorter than %zu bytes", kSnapBytes);
  if (c->routed[layer] || c->pending_rows) return fail(MOE_ESTATE, "layer %d: a routing step or an expert output is pending", layer);
  const moe_cache_config_t &g = c->cfg;
  SnapshotHeader hd;
  memcpy(&hd, buf, sizeof hd);
  if (hd.magic != kSnapMagic || hd.version != kSnapVersion) return fail(MOE_EINVAL, "not a cache snapshot");
  if (hd.n_experts != g.n_experts || hd.capacity != g.capacity || hd.top_k != g.top_k)
    return fail(MOE_EINVAL, "snapshot is for n_experts=%d capacity=%d top_k=%d", hd.n_experts, hd.capacity, hd.top_k);
  LayerState st;
  memcpy(&st, static_cast<const uint8_t *>(buf) + sizeof hd, sizeof st);
  // the two tables must describe one partial bijection expert <-> slot inside the configured ranges
  for (int e = 0; e < MOE_MAX_EXPERTS; ++e) {
    const int s = st.expert_slot[e];
    const bool ok = e < g.n_experts ? (s == -1 || (s >= 0 && s < g.capacity && st.slot_expert[s] == e)) : s == -1;
    if (!ok) return fail(MOE_EINVAL, "snapshot tables inconsistent at expert %d", e);
  }
  for (int s = 0; s < MOE_MAX_EXPERTS; ++s) {
    const int e = st.slot_expert[s];
    const bool ok = s < g.capacity ? (e == -1 || (e >= 0 && e < g.n_experts && st.expert_slot[e] == s &&
                                                   ((st.ever_used >> s) & 1)))
                                   : e == -1;
    if (!ok) return fail(MOE_EINVAL, "snapshot tables inconsistent at slot %d", s);
  }
  if (st.count < 0 || st.selections < 0 || st.misses < 0) return fail(MOE_EINVAL, "snapshot counters negative");
  if (int rc = sync_compute(c)) return rc;
  HIP_TRY(hipStreamSynchronize(c->copy));
  c->batch_x = nullptr;  // (a batch routed before this is computed with what the slots hold after it)
  int64_t misses = 0;
  HIP_TRY(hipMemcpy(&misses, &c->state(layer)->misses, sizeof misses, hipMemcpyDeviceToHost));
  HIP_TRY(hipMemcpy(c->state(layer), &st, sizeof st, hipMemcpyHostToDevice));
  c->bytes_filled[layer] += (misses - c->miss_base[layer]) * c->slot_layout.total;
  c->miss_base[layer] = st.misses;
  const size_t slot_bytes = (size_t)c->slot_layout.total;
  for (int s = 0; s < g.capacity; ++s) {
    const int e = st.slot_expert[s];
    if (e < 0) continue;
    HIP_TRY(hipMemcpy(static_cast<uint8_t *>(c->slot_pool[layer]) + (size_t)s * slot_bytes,
                      c->host_blob[(size_t)layer * g.n_experts + e], slot_bytes, hipMemcpyHostToDevice));
  }
  return MOE_OK;
}

int moe_cache_set_lambda(moe_cache_t *c, float lambda) {
  if (!c) return fail(MOE_EINVAL, "context is NULL");
  if (!(lambda >= 0.f) || !std::isfinite(lambda)) return fail(MOE_EINVAL, "lambda must be finite and >= 0");
  c->cfg.lambda = lambda;
  return MOE_OK;
}

int moe_cache_set_baseline(moe_cache_t *c, int32_t route_mode, int32_t max_rank, float cumsum_p) {
  if (!c) return fail(MOE_EINVAL, "context is NULL");
  if (route_mode < MOE_ROUTE_CACHE_PRIOR || route_mode > MOE_ROUTE_CUMSUM) return fail(MOE_EINVAL, "bad route_mode");
  if (route_mode == MOE_ROUTE_MAX_RANK && (max_rank < 0 || max_rank > c->cfg.n_experts))
    return fail(MOE_EINVAL, "max_rank must be in 0..n_experts");
  if (route_mode == MOE_ROUTE_CUMSUM && !(cumsum_p >= 0.f)) return fail(MOE_EINVAL, "cumsum_p must be >= 0");
  c->cfg.route_mode = route_mode;
  c->cfg.max_rank = max_rank;
  c->cfg.cumsum_p = cumsum_p;
  return MOE_OK;
}

int moe_cache_reset(moe_cache_t *c) {
  if (!c) return fail(MOE_EINVAL, "context is NULL");
  return do_reset(c);
}

int moe_residual_rmsnorm(float *h_dev, const void *y_dev, const float *a_dev, float perturb, int32_t carry,
                         void *x_dev, int32_t hidden, int32_t act_fmt, void *stream) {
  if (!h_dev || !x_dev) return fail(MOE_EINVAL, "h_dev or x_dev is NULL");
  if (hidden <= 0 || !valid_afmt(act_fmt)) return fail(MOE_EINVAL, "bad hidden or act_fmt");
  HIP_TRY(launch_residual_rmsnorm(h_dev, y_dev, a_dev, perturb, carry, x_dev, hidden, act_fmt,
                                  static_cast<hipStream_t>(stream)));
  return MOE_OK;
}

int moe_cache_plan(moe_cache_t *c, moe_cache_plan_t *out) {
  if (!c || !out) return fail(MOE_EINVAL, "NULL argument");
  out->grid = c->plan.grid;
  out->wavefronts = kGemvWaves;
  out->depth = c->plan.depth;
  out->packed_bf16_dot = c->plan.dot2;
  out->boundary_in_expert_launch = boundary_form(c) == MOE_BOUNDARY_IN_FIRST_WORKGROUP;
  return MOE_OK;
}

int moe_cache_boundary_form(moe_cache_t *c, int32_t *out) {
  if (!c || !out) return fail(MOE_EINVAL, "NULL argument");
  *out = boundary_form(c);
  return MOE_OK;
}

int moe_cache_fill_form(moe_cache_t *c, int32_t *out) {
  if (!c || !out) return fail(MOE_EINVAL, "NULL argument");
  *out = c->d_host_blob != nullptr ? MOE_FILLS_IN_EXPERT_LAUNCH : MOE_FILLS_BY_HOST;
  return MOE_OK;
}

namespace {
constexpr size_t kProfEvents = 1u << 15;  // launches timed between two resets
}

int moe_cache_profile(moe_cache_t *c, int32_t enable, int32_t reset, double *avg_us, int64_t *launches) {
  if (!c) return fail(MOE_EINVAL, "context is NULL");
  HIP_TRY(hipStreamSynchronize(c->compute));
  double total_ms = 0.0;
  int64_t n_full = 0;
  for (size_t i = 0; i < c->prof_used; ++i) {
    if (!c->prof_full[i]) continue;  // a launch that left out missing experts moved fewer bytes
    float ms = 0.f;
    HIP_TRY(hipEventElapsedTime(&ms, c->prof_events[i].first, c->prof_events[i].second));
    total_ms += ms;
    ++n_full;
  }
  if (avg_us) *avg_us = n_full ? total_ms * 1000.0 / (double)n_full : 0.0;
  if (launches) *launches = n_full;
  if (reset) c->prof_used = 0;
  c->profiling = enable > 0 ? enable : 0;
  c->prof_tick = 0;
  // the events are made here, not between the launches they time
  while (c->profiling && c->prof_events.size() < kProfEvents) {
    hipEvent_t a, b;
    HIP_TRY(hipEventCreate(&a));
    HIP_TRY(hipEventCreate(&b));
    c->prof_events.emplace_back(a, b);
    c->prof_full.push_back(0);
  }
  return MOE_OK;
}

}  // extern "C"
