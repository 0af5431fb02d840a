// Internal declarations shared by the translation units of libmoe_cache (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <stdint.h>

#include "moe_cache.h"

namespace moe {

constexpr int kWave = 64;

// Per-layer cache state, device resident.  One wavefront owns it during a routing step:
// lane e holds expert e's entries, lane s holds slot s's entry.
struct LayerState {
  int32_t expert_slot[MOE_MAX_EXPERTS];  // expert -> slot, -1 = not resident
  int32_t slot_expert[MOE_MAX_EXPERTS];  // slot -> expert, -1 = empty
  int64_t stamp[MOE_MAX_EXPERTS];        // recency stamp per expert (valid while resident)
  int32_t born[MOE_MAX_EXPERTS];         // token at which the expert was loaded (valid while resident)
  uint64_t ever_used;                    // bit s: slot s has held an expert
  float delta_sum;                       // Eq. 10 accumulator
  int32_t count;                         // tokens routed
  int64_t selections, hits, misses, cold_misses, evictions, lifetime_sum;  // contiguous: updated lane-wise
};

struct RouteParams {
  int32_t n_experts, top_k, top_j, capacity, hidden;
  int32_t act_fmt, renormalize, delta_mode, route_mode, max_rank;
  float lambda, delta_fixed, cumsum_p;
  uint32_t seq;
};

// Glue of a stack fused in front of the router (see fused_route_kernel).
constexpr int kFusedMaxHidden = 8192;
struct FusedParams {
  const void *y;    // [d] act_fmt, the previous layer's expert output, or nullptr
  float *h;         // [d] fp32 residual stream, updated in place
  const float *a;   // [d] fp32 perturbation or nullptr
  float perturb;
  int32_t carry;    // 0: a new token starts, h = perturb * a
  void *x_out;      // [d] act_fmt, the normalised vector (input of this layer)
  // When the glue has been done by reduce_glue_kernel: h already holds the new residual stream and ss its sums
  // of squares over consecutive blocks of 64 columns (n_ss = d / 64 of them); y, a, perturb, carry are unused.
  const float *ss;
  int32_t n_ss;
};

// The layer boundary (x from the new residual stream + routing step, see rt::fused_boundary) when it is run by
// workgroup 0 of the expert launch itself: the other workgroups compute x for themselves, stream the shared
// expert's records meanwhile, and wait for its decision before the first routed record.
struct BoundaryArgs {
  RouteParams route;
  FusedParams glue;
  const void *gate_w;
  LayerState *state;
  moe_route_out_t *out_dev;  // the layer's device record (= GemvParams::route)
  struct HostNote *note;     // the layer's words in mapped host memory
  uint64_t *handover;        // the layer's self-tagged words with slots, miss flags and weights (8 copies of 8)
  uint32_t hand_tag;         // 16-bit tag of this hand-over: the count of the layer's hand-overs so far, so that
                             // what the words still hold (the previous one) can never pass for it
  uint32_t *gave_up;         // mapped host word set when a wavefront stopped waiting for the hand-over
  int spin_limit;            // polls of the hand-over before a wavefront stops waiting (a test lowers it)
  // what the boundary of the layer that follows will read first (its gate matrix and cache state): workgroup 0
  // touches it once its own work is done, which measurably shortens that boundary (nullptr: don't)
  const void *next_gate_w;
  const LayerState *next_state;
  int64_t gate_bytes;
  // routing in every workgroup: the logits, and the copy of the state that receives the step (every workgroup of the
  // launch reads the old one)
  const float *logits;
  LayerState *state_out;
};
// how an expert launch comes by the routing decision
enum RouteIn {
  kRouteBefore = 0,     // from the record an earlier launch wrote
  kRouteBoundary = 1,   // workgroup 0 runs the layer boundary `b`, hands the decision over and writes a zero partial row; the
                        // others wait for it (see WaitingTurn)
  kRouteGiven = 3,      // from the launch's own arguments (given_slots, given_weight): all experts are in their slots
  kRouteEverywhere = 2  // every workgroup routes for itself from b.logits and b.state; the first does the bookkeeping: one
                        // more than plan.grid, or (idle_row) one of them, whose partial row is then zero
};

struct GemvParams {
  const uint8_t *slot_pool;      // this layer's slots
  const uint8_t *shared_blob;    // or nullptr
  const moe_route_out_t *route;  // device record of the layer's routing step (slots, weights, miss flags)
  const void *x;                 // [d] act_fmt
  float *partial;                // [grid][d] fp32
  int32_t hidden, inter, shared_inter, top_k, act_fmt;
  int64_t slot_bytes;
  // the layer's experts in the host tier as the device sees them [N], or nullptr.  Given: one launch covers everything (pass
  // 0), the experts that miss are streamed from there and put into their slots on the way.  nullptr: see pass
  const uint8_t *const *host_blob;
  int32_t pass;        // 0: shared expert + experts that were resident; 1: experts whose slot was just filled
  int32_t row_offset;  // first partial row this launch writes
  int32_t missing_row; // with host_blob: how many rows further on the sums over the experts that missed are written, if any did
  int32_t route_in;    // RouteIn
  int32_t idle_row;    // kRouteEverywhere: 1 = plan.grid workgroups with the first one, which writes a zero row
  // the split of n records over the launch's G streaming workgroups (launch_expert_gemv fills it in): quotient and remainder
  // of the shared and of the routed records, and ceil(2^32 / G) to divide by G with one multiplication
  uint32_t shared_q, shared_r, routed_q, routed_r, inv_g;
  uint64_t given_slots;                // kRouteGiven: 8 bits each, in selection order
  float given_weight[MOE_MAX_TOPK];
  BoundaryArgs b;
};

// Blob geometry (see moe_blob_bytes).
struct BlobLayout {
  int64_t rec_bytes;    // bytes of one record (gate row | up row | down column [| inline scales])
  int64_t row_bytes;    // bytes of one d-long row of weights
  int64_t tail_offset;  // start of the out-of-record scales
  int64_t total;        // whole blob, multiple of 256
};
BlobLayout blob_layout(int fmt, int hidden, int inter);
// int4: bytes of one record - three rows of nibbles and the record's (gate, up) fp16 scale pairs, one pair per group of
// 128 columns, padded so that every record starts on a 128-byte line (a wavefront's 1 KB load then covers 8 lines, not 9)
__host__ __device__ constexpr int64_t int4_record_bytes(int64_t d) { return 3 * (d / 2) + ((d / 128) * 4 + 127) / 128 * 128; }

// What the host needs of a routing decision, written by the router into mapped host memory as three 8-byte words,
// each complete in itself (no ordering between them is assumed):
//   w[0] = seq | n_miss << 32 | miss flags by selection position << 40
//   w[1] = (seq & 0xffff) | expert of position k << (16 + 6k)
//   w[2] = (seq & 0xffff) | slot of position k   << (16 + 6k)
// The host has the decision once all three carry the tag of the step it waits for.
struct HostNote {
  uint64_t w[4];
};

// The full record of a step whose decision the caller waits for, in mapped host memory: word i of the record in the
// low half of w[i], the step's seq in the high half.  Complete once all words carry the seq (no order between the stores
// is assumed), so nobody has to wait for the kernel's end or a copy.  `outputs` carries the seq once everything that a
// layer boundary writes for the caller (h, x) has reached memory, where any stream and the host find it.
constexpr int kHostRecWords = sizeof(moe_route_out_t) / 4;
struct HostRecord {
  uint64_t w[kHostRecWords];
  uint64_t outputs;
};
// where a routing step leaves what the host wants of it (device views of mapped host memory; nullptr: not wanted)
struct HostOut {
  HostNote *note;
  HostRecord *rec;
};

// launchers (each returns the hipError_t of the launch)
hipError_t launch_route(const RouteParams &p, const void *gate_w, const void *x, const float *logits,
                        LayerState *state, moe_route_out_t *out_dev, HostOut host, hipStream_t s);
// launch shape of the expert GEMV
constexpr int kGemvWaves = 8;  // wavefronts per workgroup
// Records in flight per wavefront, by 16-byte loads per row and lane: about 48 KB per compute unit, at least one record.  What
// is requested beyond what a compute unit's L1 keeps in flight only lets some wavefronts have all their records before
// others have their first (static launches, us with 1 / 2 / 3 records: int4 d = 2048, 37 MB - / 12.7 / 13.2; int8 d = 2048, 37 MB
// 12.1 / 12.1 / 12.2; bf16 d = 2048, 101 MB 20.8 / 20.7; bf16 d = 4096 21.5 / 33.3, where two do not fit the registers).
constexpr int gemv_depth(int loads_per_row) { return loads_per_row == 1 ? 2 : 1; }
struct GemvPlan {
  int grid;   // workgroups (= fp32 partial rows written): one per compute unit
  int depth;  // records in flight per wavefront
  bool dot2;  // packed bf16 dot products (bf16 weights and activations)
};
GemvPlan gemv_plan(int n_cus, int total_records, int weight_fmt, int act_fmt, int hidden);
// logits of a layer boundary whose glue launch_reduce_glue has done: x = h / rms to f.x_out, z = W_gate x, one workgroup per
// four experts (needs gate_rows_supported)
bool gate_rows_supported(int hidden, int act_fmt);
hipError_t launch_gate_rows(const RouteParams &p, const FusedParams &f, const void *gate_w, float *logits, hipStream_t s);
// logits of a step on a given x, spread the same way
hipError_t launch_gate_x(const RouteParams &p, const void *x, const void *gate_w, float *logits, hipStream_t s);
bool gemv_fused_supported(int weight_fmt, int act_fmt, int hidden, const GemvPlan &plan);  // a launch variant with the boundary in workgroup 0
// f.ss != nullptr: the glue has been done by launch_reduce_glue (needs fused_route_pre_supported(hidden))
bool fused_route_pre_supported(int hidden);
hipError_t launch_fused_route(const RouteParams &p, const FusedParams &f, const void *gate_w, LayerState *state,
                              moe_route_out_t *out_dev, HostOut host, hipStream_t s);
hipError_t launch_expert_gemv(const GemvParams &p, int weight_fmt, const GemvPlan &plan, hipStream_t s,
                              hipEvent_t start = nullptr, hipEvent_t stop = nullptr);
// n_miss: nullptr, or the number of misses of the step (device): if there are any, n_partial rows more
hipError_t launch_partial_reduce(const float *partial, int n_partial, const int32_t *n_miss, void *y, int hidden, int act_fmt,
                                 hipStream_t s);
// the same plus the residual glue: h = (carry ? h + y : 0) + perturb * a in place, ss[b] = sum of h^2 over columns
// 64b .. 64b+63 (y may be NULL: not stored; n_partial may be 0: y = nothing)
hipError_t launch_reduce_glue(const float *partial, int n_partial, const int32_t *n_miss, void *y, int hidden, int act_fmt, float *h,
                              const float *a, float perturb, int carry, float *ss, hipStream_t s);
hipError_t launch_pack(int fmt, int hidden, int inter, const void *gate, const void *up, const void *down,
                       const void *gs, const void *us, const void *ds, void *blob, hipStream_t s);
hipError_t launch_residual_rmsnorm(float *h, const void *y, const float *a, float perturb, int carry, void *x,
                                   int hidden, int act_fmt, hipStream_t s);
hipError_t launch_state_init(LayerState *state, int n_layers, const int32_t *initial_dev, int n_initial,
                             hipStream_t s);
// ---- prompt phase (expert_batch.hip): a batch of tokens through one layer ----
constexpr int kMaxBatch = 128;        // tokens per moe_route_batch / moe_expert_forward_batch call
// the selection of a batch as the expert kernels read it (slots and weights by selection order, 0xff = none)
struct BatchSel {
  uint8_t slot[kMaxBatch][MOE_MAX_TOPK];
  float weight[kMaxBatch][MOE_MAX_TOPK];
};
// what route_ahead_kernel leaves for route_batch_kernel: per token whether it misses an expert, its experts in touch
// order, and Eq. 10's sum before it (and after the last one)
struct BatchAhead {
  uint8_t touched[kMaxBatch][MOE_MAX_TOPK];
  uint8_t miss[kMaxBatch];
  float dsum[kMaxBatch + 1];
};
// one expert of a launch: its slot (-1: the shared expert), how many tokens of the segment take it, where its h starts
// (in blocks of 16 tokens x 32 records in fp32 = 2 KB) and its first workgroup in the two launches
struct BatchEntry {
  int16_t slot;
  uint16_t n_tok;
  uint32_t h_base, unit0_up, unit0_down;
};
constexpr int kMaxEntries = MOE_MAX_EXPERTS + 1;
constexpr int kMaxPartialRows = 4096;  // rows of P of a segment (P: [rows][hidden] fp32)
struct BatchArgs {
  const uint8_t *slot_pool, *shared_blob;
  const uint16_t *x;    // [B, d] bf16
  const BatchSel *sel;
  uint8_t *h;           // see up_batch_kernel
  float *partial;       // P
  int64_t slot_bytes;
  int32_t hidden, inter, shared_inter, top_k;
  int32_t t0, t1;       // tokens of the segment
  int32_t up_records;   // records per unit of up_batch_kernel (a multiple of 32)
  int32_t down_groups;  // groups of 32 records per unit of down_batch_kernel
  int32_t shared_row0;  // first row of the shared expert in P
  int32_t n_entries;
};
struct BatchParams : BatchArgs {
  BatchEntry e[kMaxEntries];
};
// The same list made on the device (route_batch_kernel), for a batch in which nothing misses: the expert kernels are then
// enqueued behind the routing before the host knows the decisions.
struct BatchPlan {
  int32_t n_up, n_down;  // units of the two expert kernels; 0: something misses, the host sees to the batch
  int32_t up_records, down_groups, n_rc, n_rc_shared, shared_row0, n_entries;
  BatchEntry e[kMaxEntries];
};
// what route_batch_kernel needs for it (plan = nullptr: not wanted)
constexpr int kPlanRounds = 2;  // its launches have that many workgroups per compute unit; a longer list is the host's
struct BatchPlanFor {
  BatchPlan *plan;
  int32_t hidden, inter, shared_inter, n_cus;
};
// Sizes of the units of the two expert kernels.  A unit costs a start-up of about 3 us and then what its compute unit's L1
// takes in (about 23 KB per us: 8 KB a record in `up`, 16 KB a group of 32 records in `down`), and a launch runs in rounds of
// one workgroup per compute unit: the sizes with the smallest rounds x unit time are taken, the larger ones where two are equal.
// The same on the host and on the device (whole numbers).
__host__ __device__ inline int batch_parts(int n, int by) { return (n + by - 1) / by; }
constexpr int64_t kNoCandidate = INT64_MAX;
__host__ __device__ inline int64_t batch_up_estimate(int cand, int groups, int inter, int shared_groups, int shared_inter, int hidden, int n_cus) {
  const int units = groups * batch_parts(inter, cand) + shared_groups * batch_parts(shared_inter, cand);
  return (int64_t)batch_parts(units, n_cus) * (300 * 2048 + (int64_t)36 * hidden * cand);  // 3 us + 0.36 us a record at d = 2048
}
__host__ __device__ inline int batch_up_candidates(int inter, int shared_inter) {  // 32, 64, .. times 1 .. this
  const int longest = inter > shared_inter ? inter : shared_inter, n = batch_parts(longest, 32);
  return n < 32 ? n : 32;
}
// P has to hold the rows: a candidate that makes too many is none
__host__ __device__ inline int64_t batch_down_estimate(int cand, int groups, int inter, int shared_groups, int shared_inter, int hidden, int n_seg,
                                                      int top_k, int n_cus) {
  const int n32 = batch_parts(inter, 32), n32s = shared_groups ? batch_parts(shared_inter, 32) : 0;
  const int rc = batch_parts(n32, cand), rcs = batch_parts(n32s, cand);
  if ((int64_t)n_seg * (top_k * rc + rcs) > kMaxPartialRows) return kNoCandidate;
  const int units = (groups * rc + shared_groups * rcs) * (hidden / 256);
  return (int64_t)batch_parts(units, n_cus) * (40 + 7 * cand);  // 4 us + 0.7 us a group
}
__host__ __device__ inline int batch_down_candidates(int inter, int shared_inter) {  // 4, 8, .. times 1 .. this
  const int longest = inter > shared_inter ? inter : shared_inter;
  return batch_parts(batch_parts(longest, 32), 4);
}
// units of one expert with n_tok tokens and `rows` records in the two kernels (several token groups: see group_pos)
__host__ __device__ inline void batch_entry_units(int n_tok, int rows, int up_records, int down_groups, int hidden, int *up, int *down) {
  const int groups = batch_parts(n_tok, 64);
  *up = batch_parts(rows, up_records);
  *down = batch_parts(batch_parts(rows, 32), down_groups) * (hidden / 256);
  if (groups > 1) {
    *up = (*up + 7) / 8 * 8 * groups;
    *down = (*down + 7) / 8 * 8 * groups;
  }
}
bool batch_shape_supported(int weight_fmt, int act_fmt, int hidden, int inter, int shared_inter);
hipError_t launch_gate_gemm(const void *x, const void *gate_w, float *logits, int B, int N, int hidden, hipStream_t s);
hipError_t launch_route_batch(const RouteParams &p, const float *logits, int B, LayerState *state, moe_route_out_t *out,
                              BatchSel *sel, BatchAhead *ahead, uint32_t *done, const BatchPlanFor &planned, hipStream_t s);
hipError_t launch_up_batch(const BatchParams &p, int n_units, hipStream_t s);
hipError_t launch_down_batch(const BatchParams &p, int n_units, hipStream_t s);
hipError_t launch_reduce_batch(const BatchArgs &p, void *y, int n_rc, int n_rc_shared, hipStream_t s);
// with the list that route_batch_kernel leaves
hipError_t launch_planned_experts(const BatchArgs &p, const BatchPlan *plan, int n_cus, hipStream_t s);
hipError_t launch_planned_reduce(const BatchArgs &p, const BatchPlan *plan, void *y, hipStream_t s);

// the allocation-free entry point (expert_static.hip): device address of its fixed scratch array and the compute-unit
// count of device `dev` (which must be current), looked up once per device
hipError_t static_scratch_setup(int dev, void **ptr, int *cus);
hipError_t launch_expert_forward_static(int weight_fmt, int act_fmt, int hidden, int inter, int shared_inter, int top_k,
                                        const void *slot_pool, int64_t slot_bytes, const void *shared_blob,
                                        const int32_t *sel_slot, const float *sel_weight, const void *x, void *y,
                                        hipStream_t s);
int static_max_hidden();
bool gemv_shape_supported(int weight_fmt, int hidden);
bool gemv_inter_supported(int weight_fmt, int inter);
hipError_t launch_expert_gemv_quant(const GemvParams &p, int weight_fmt, const GemvPlan &plan, hipStream_t s,
                                    hipEvent_t start, hipEvent_t stop);

// ---- device helpers -------------------------------------------------------------------------
#if defined(__HIPCC__)
__device__ __forceinline__ float bf16_lo(uint32_t v) { return __uint_as_float(v << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t v) { return __uint_as_float(v & 0xffff0000u); }
__device__ __forceinline__ uint16_t f32_to_bf16_rne(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40);  // NaN stays NaN
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

template <int CTRL>
__device__ __forceinline__ float dpp_f32(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false));
}
// Sum over the 64 lanes, result in every lane, fixed order (rotations inside rows of 16, then rows).
// Sum of N <= 64 floats in index order, the same in every wavefront that computes it: fetch() has lane i load
// entry i (clamped: no branch around the load), total() adds the entries one by one through lane reads.  N is a
// compile-time constant so that neither part ends up inside a branch.
template <int N>
struct OrderedSum {
  static_assert(N >= 1 && N <= 64, "one entry per lane");
  float s;
  __device__ __forceinline__ void fetch(const float *v, int lane) { s = v[lane < N ? lane : 0]; }
  __device__ __forceinline__ float total() const {
    float tot = 0.f;
#pragma unroll
    for (int i = 0; i < N; ++i) tot += __int_as_float(__builtin_amdgcn_readlane(__float_as_int(s), i));
    return tot;
  }
};

__device__ __forceinline__ float wave_sum(float v) {
  v += dpp_f32<0x128>(v);  // row_ror:8
  v += dpp_f32<0x124>(v);  // row_ror:4
  v += dpp_f32<0x122>(v);  // row_ror:2
  v += dpp_f32<0x121>(v);  // row_ror:1
  float r0 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 0));
  float r1 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 16));
  float r2 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 32));
  float r3 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 48));
  return (r0 + r1) + (r2 + r3);
}
#endif

}  // namespace moe
