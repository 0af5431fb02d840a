// Prompt phase: a batch of B tokens through one MoE layer (paper Sec. 4.5 applies the cache-aware routing during
// generation and lets prompt processing use batched kernels; App. F looks at the prompt length).  The routing of the
// batch is the routing of its tokens one after the other - the cache bitmask m_t of Sec. 3.3 is the state after
// token t-1, also inside a batch - so every decision, slot and miss count equals what B single-token steps give;
// only the arithmetic is batched: the gate logits of all tokens by one small GEMM, the experts by a
// weights-stationary small GEMM per expert over the tokens routed to it (Eq. 1), both on the matrix cores.
//
//  gate_gemm_kernel    logits[B, N] = X[B, d] W_gate[N, d]^T, bf16 inputs, fp32 accumulation
//                      (v_mfma_f32_16x16x32_bf16: a 16-token x 16-expert tile per eight wavefronts, which split d).
//  route_batch_kernel  sixteen wavefronts route sixteen tokens at a time through rt::route_wave against the current
//                      cache state; a token that misses an expert is routed alone and updates the state (see there);
//                      one routing record per token.
//  up_batch_kernel, down_batch_kernel, reduce_batch_kernel
//                      the experts as two weights-stationary products over the tokens routed to them, and the sum per
//                      token in a fixed order (deterministic y).
//  up_planned_kernel, down_planned_kernel
//                      the same products where nobody waits between routing and experts: the units of work are listed on
//                      the device by route_batch_kernel (make_plan), the grids are a few workgroups per compute unit.
#include <type_traits>

#include "common.h"
#include "gemv_common.h"
#include "route_device.h"

namespace moe {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f32x4 mfma_bf16(u32x4 a, u32x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
// ---- gate logits of the batch -------------------------------------------------------------------
// grid = (token tiles of 16, expert tiles of 16), block = kGateSplit wavefronts: wavefront ks multiplies the ks-th
// part of the hidden dimension, all its operands requested at once (one round trip); the parts are added through LDS
// in a fixed order.  A-operand lane l: token l % 16, columns k0 + 8 (l / 16) .. + 8; B-operand lane l: expert
// n0 + l % 16, the same columns; result lane l: expert n0 + l % 16, tokens 4 (l / 16) + v.  Rows past the last token /
// expert re-read the last one and are not stored.
constexpr int kGateSplit = 8;
// STEPS: 32-column steps per wavefront (hidden = 32 * kGateSplit * STEPS)
template <int STEPS>
__global__ __launch_bounds__(kGateSplit *kWave) void gate_gemm_kernel(const uint16_t *x, const uint16_t *gate_w,
                                                                     float *logits, int B, int N, int d) {
  __shared__ f32x4 part[kGateSplit][kWave];
  const int lane = threadIdx.x & 63, ks = threadIdx.x >> 6;
  const int t0 = blockIdx.x * 16, n0 = blockIdx.y * 16;
  const int tok = min(t0 + (lane & 15), B - 1), exp = min(n0 + (lane & 15), N - 1);
  const u32x4 *xa = reinterpret_cast<const u32x4 *>(x + (size_t)tok * d) + (lane >> 4) + (size_t)ks * STEPS * 4;
  const u32x4 *wb = reinterpret_cast<const u32x4 *>(gate_w + (size_t)exp * d) + (lane >> 4) + (size_t)ks * STEPS * 4;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  u32x4 a[STEPS], b[STEPS];
#pragma unroll
  for (int s = 0; s < STEPS; ++s) {
    a[s] = xa[s * 4];
    b[s] = wb[s * 4];
  }
#pragma unroll
  for (int s = 0; s < STEPS; ++s) acc = mfma_bf16(a[s], b[s], acc);
  part[ks][lane] = acc;
  __syncthreads();
  if (ks != 0) return;
#pragma unroll
  for (int q = 1; q < kGateSplit; ++q) {
    const f32x4 t = part[q][lane];
    acc[0] += t[0];
    acc[1] += t[1];
    acc[2] += t[2];
    acc[3] += t[3];
  }
  const int e = n0 + (lane & 15);
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int t = t0 + 4 * (lane >> 4) + v;
    if (t < B && e < N) logits[(size_t)t * N + e] = acc[v];
  }
}

// ---- routing of the batch ---------------------------------------------------------------------------
// The decisions are those of the tokens routed one after the other (the cache mask of Sec. 3.3 is the state after the
// previous token), but a token that misses nothing leaves the cache as it found it except for the recency stamps of
// its experts - and stamps only matter to a later miss.  So sixteen wavefronts route the next sixteen tokens at once
// against the current state (rt::route_wave, unchanged, its record kept in LDS); the tokens up to the first one that
// misses an expert are accepted as they are: records copied out, stamps merged (a later token's stamp is larger, so
// the merge is a maximum), counters advanced.  The token with the miss is then routed by one wavefront against the
// merged state, which it updates, and the window moves on behind it.  What does not depend on the cache - Eq. 10's
// running sum of logit ranges - is prepared for all tokens first (the same additions in the same order).
// Miss-free batches cost one round per sixteen tokens; a miss costs one extra round.
//
// A round is issue-bound (four wavefronts a SIMD, each a long chain of dependent instructions), so longer batches are
// first routed by route_ahead_kernel: one wavefront per token on a SIMD of its own, all against the state before the
// batch.  Up to the first miss these are the decisions; route_batch_kernel then only merges them and walks the rest.
constexpr int kRouteWaves = 16;
struct BatchCacheState {  // LayerState's tables while the batch is routed (LDS)
  int32_t my_slot[MOE_MAX_EXPERTS], slot_exp[MOE_MAX_EXPERTS], born[MOE_MAX_EXPERTS];
  long long stamp[MOE_MAX_EXPERTS];
  long long counter[6];
  uint64_t ever_used;
  int32_t count0;  // tokens routed before this batch
};

__device__ __forceinline__ rt::CacheRegs batch_cache_regs(const BatchCacheState &s, int lane, int t, float dsum_prev) {
  rt::CacheRegs cr;
  cr.my_slot = s.my_slot[lane];
  cr.slot_exp = s.slot_exp[lane];
  cr.born = s.born[lane];
  cr.stamp = s.stamp[lane];
  cr.counter = lane < 6 ? s.counter[lane] : 0;
  cr.ever_used = s.ever_used;
  cr.t = s.count0 + t;
  cr.dsum_prev = dsum_prev;
  return cr;
}

// what the expert kernels need of a token's record: its slots and weights in selection order
__device__ __forceinline__ void store_sel(const uint32_t *rec, int K, int lane, int t, BatchSel *sel) {
  if (lane < MOE_MAX_TOPK) {
    sel->slot[t][lane] = lane < K ? (uint8_t)rec[rt::W_SLOT + lane] : (uint8_t)0xff;
    sel->weight[t][lane] = __uint_as_float(rec[rt::W_WEIGHT + lane]);
  }
}

using rt::lds_barrier;

constexpr int kAheadWaves = 4;
constexpr int kZStride = MOE_MAX_EXPERTS + 1;  // (a thread walks a row: rows start in different banks)

__global__ __launch_bounds__(kAheadWaves *kWave) void route_ahead_kernel(RouteParams p, const float *logits, int B,
                                                                         LayerState *st, moe_route_out_t *out, BatchSel *sel,
                                                                         BatchAhead *ahead) {
  __shared__ float z_s[kMaxBatch * kZStride];
  __shared__ float range_s[kMaxBatch];
  __shared__ __attribute__((aligned(16))) uint32_t rec_s[kAheadWaves][rt::kRecWords];
  const int tid = threadIdx.x, lane = tid & 63, N = p.n_experts, K = p.top_k;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int t = (int)blockIdx.x * kAheadWaves + wave;
  const int n = min(B, ((int)blockIdx.x + 1) * kAheadWaves);  // Eq. 10's sum needs the tokens up to this workgroup's
  rt::CacheRegs cr = rt::load_cache_regs(st, lane, N, p.capacity), next;
  const int e_c = min(lane, N - 1);
#pragma unroll 8
  for (int i = wave; i < n; i += kAheadWaves) z_s[i * kZStride + lane] = logits[i * N + e_c];  // (lanes past N: a copy)
  __syncthreads();
  if (tid < n) {
    // (over the numbers among the logits, as a wavefront's maximum is; where 64 logits are none, it is none either)
    const float *row = z_s + tid * kZStride;
    float lo = N < kWave ? INFINITY : row[0], hi = N < kWave ? -INFINITY : row[0];
#pragma unroll 8
    for (int e = 0; e < N; ++e) {
      lo = fminf(lo, row[e]);
      hi = fmaxf(hi, row[e]);
    }
    range_s[tid] = hi - lo;
  }
  __syncthreads();
  if (t >= B) return;
  {
#pragma clang fp contract(off)
    float acc = cr.dsum_prev;
#pragma unroll 8
    for (int i = 0; i < t; ++i) acc = acc + range_s[i];
    cr.dsum_prev = acc;
  }
  const int count0 = cr.t;
  cr.t = count0 + t;
  int n_miss = 0;
  rt::route_wave(p, z_s + t * kZStride, cr, st, out + t, HostOut{nullptr, nullptr}, rec_s[wave], lane, rt::BoundaryFlags{nullptr, 0}, &next, false,
                 &n_miss);
  store_sel(rec_s[wave], K, lane, t, sel);
  // the experts in touch order: their stamps are token * K + position (0xff: logits that are not numbers select fewer)
  if (lane < MOE_MAX_TOPK) ahead->touched[t][lane] = 0xff;
  if (lane < N && next.stamp != cr.stamp) ahead->touched[t][(int)(next.stamp - (int64_t)cr.t * K)] = (uint8_t)lane;
  if (lane == 0) {
    ahead->miss[t] = (uint8_t)(n_miss > 0);
    ahead->dsum[t] = cr.dsum_prev;
    if (t == B - 1) ahead->dsum[B] = next.dsum_prev;
  }
}

// The list of experts for the expert kernels (BatchPlan), by one wavefront: lane s <-> slot s with count[s] places.  The order
// and the numbers are those the host makes: experts with several groups of 64 tokens first, the shared one ahead of its kind.
__device__ __forceinline__ int wave_sum_i(int v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}
__device__ __forceinline__ int wave_before_i(int v, int lane) {  // sum over the lanes below
  int s = v;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const int t = __shfl_up(s, o);
    if (lane >= o) s += t;
  }
  return s - v;
}
__device__ __forceinline__ int64_t wave_min_i64(int64_t v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = min(v, (int64_t)__shfl_xor((long long)v, o));
  return v;
}
__device__ __forceinline__ int wave_max_i(int v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = max(v, __shfl_xor(v, o));
  return v;
}
__device__ __forceinline__ void make_plan(const BatchPlanFor &f, int B, int top_k, const int *count, uint32_t *order_s, int lane) {
  const int n = count[lane], groups = wave_sum_i(batch_parts(n, 64));
  const int sg = f.shared_inter > 0 ? batch_parts(B, 64) : 0, sh = sg ? f.shared_inter : 0;
  // the best candidate, the largest where several are equal
  int64_t best = kNoCandidate;
  int cand = 0;
  if (lane < batch_up_candidates(f.inter, sh)) {
    cand = 32 * (lane + 1);
    best = batch_up_estimate(cand, groups, f.inter, sg, sh, f.hidden, f.n_cus);
  }
  const int up_records = wave_max_i(best == wave_min_i64(best) ? cand : 0);
  best = kNoCandidate;
  cand = 4;
  for (int c = lane; c < batch_down_candidates(f.inter, sh); c += kWave) {
    const int64_t est = batch_down_estimate(4 * (c + 1), groups, f.inter, sg, sh, f.hidden, B, top_k, f.n_cus);
    if (est <= best) best = est, cand = 4 * (c + 1);
  }
  const int down_groups = wave_max_i(best == wave_min_i64(best) ? cand : 0);
  const int n32 = batch_parts(f.inter, 32), n32s = sg ? batch_parts(f.shared_inter, 32) : 0;
  const int rc = batch_parts(n32, down_groups), rcs = batch_parts(n32s, down_groups);
  // the experts in list order, one per lane
  const uint64_t several = rt::ballot(n > 64), others = rt::ballot(n > 0 && n <= 64), below = (1ull << lane) - 1ull;
  const int n_several = (int)__builtin_popcountll(several), n_slots = n_several + (int)__builtin_popcountll(others);
  if (n > 64) order_s[__builtin_popcountll(several & below)] = (uint32_t)lane | ((uint32_t)n << 8);
  else if (n > 0) order_s[n_several + __builtin_popcountll(others & below)] = (uint32_t)lane | ((uint32_t)n << 8);
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  const uint32_t mine = lane < n_slots ? order_s[lane] : 0u;
  const int n_tok = (int)(mine >> 8);
  int up = 0, down = 0, h = 0, sh_up = 0, sh_down = 0, sh_h = 0;
  if (lane < n_slots) {
    batch_entry_units(n_tok, f.inter, up_records, down_groups, f.hidden, &up, &down);
    h = batch_parts(n_tok, 16) * n32;
  }
  if (sg) {
    batch_entry_units(B, f.shared_inter, up_records, down_groups, f.hidden, &sh_up, &sh_down);
    sh_h = batch_parts(B, 16) * n32s;
  }
  const int up0 = wave_before_i(up, lane), down0 = wave_before_i(down, lane), h0 = wave_before_i(h, lane);
  const int sh_at = B > 64 ? 0 : n_several;  // the shared expert's place
  const bool after = sg && lane >= sh_at;
  BatchPlan *o = f.plan;
  if (lane < n_slots)
    o->e[lane + after] = BatchEntry{(int16_t)(mine & 0xffu), (uint16_t)n_tok, (uint32_t)(h0 + (after ? sh_h : 0)),
                                    (uint32_t)(up0 + (after ? sh_up : 0)), (uint32_t)(down0 + (after ? sh_down : 0))};
  const int up_all = wave_sum_i(up) + sh_up, down_all = wave_sum_i(down) + sh_down, h_all = wave_sum_i(h);
  // (n_slots = 64 and the shared expert behind them all: there is no lane at its place)
  const int su0 = sh_at < kWave ? __shfl(up0, sh_at & 63) : up_all - sh_up, sd0 = sh_at < kWave ? __shfl(down0, sh_at & 63) : down_all - sh_down;
  const int h_at = sh_at < kWave ? __shfl(h0, sh_at & 63) : h_all;
  if (lane == 0) {
    if (sg) o->e[sh_at] = BatchEntry{(int16_t)-1, (uint16_t)B, (uint32_t)h_at, (uint32_t)su0, (uint32_t)sd0};
    const bool fits = max(up_all, down_all) <= kPlanRounds * f.n_cus;
    o->n_up = fits ? up_all : 0;
    o->n_down = fits ? down_all : 0;
    o->up_records = up_records;
    o->down_groups = down_groups;
    o->n_rc = rc;
    o->n_rc_shared = rcs;
    o->shared_row0 = B * top_k * rc;
    o->n_entries = n_slots + (sg ? 1 : 0);
  }
}

__global__ __launch_bounds__(kRouteWaves *kWave) void route_batch_kernel(RouteParams p, const float *logits, int B,
                                                                         LayerState *st, moe_route_out_t *out,
                                                                         BatchSel *sel, const BatchAhead *ahead,
                                                                         uint32_t *done, BatchPlanFor planned) {
  __shared__ float z_all[kMaxBatch * MOE_MAX_EXPERTS];
  __shared__ float range_s[kMaxBatch];
  __shared__ float dsum_s[kMaxBatch + 1];  // Eq. 10's sum before token t
  __shared__ __attribute__((aligned(16))) uint32_t asm_s[kRouteWaves][rt::kRecWords];    // route_wave's work buffer
  __shared__ __attribute__((aligned(16))) uint32_t stage_s[kRouteWaves][rt::kRecWords];  // a wavefront's record
  __shared__ BatchCacheState cs;
  __shared__ int first_miss_s;
  __shared__ int count_s[MOE_MAX_EXPERTS];  // places that name the slot
  __shared__ uint32_t order_s[MOE_MAX_EXPERTS];
  const int tid = threadIdx.x, lane = tid & 63, N = p.n_experts, K = p.top_k;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  bool missed = false;  // (the same in every thread)
  if (tid < MOE_MAX_EXPERTS) count_s[tid] = 0;

  if (wave == 0) {
    const rt::CacheRegs cr = rt::load_cache_regs(st, lane, N, p.capacity);
    cs.my_slot[lane] = cr.my_slot;
    cs.slot_exp[lane] = cr.slot_exp;
    cs.born[lane] = cr.born;
    cs.stamp[lane] = cr.stamp;
    if (lane < 6) cs.counter[lane] = cr.counter;
    if (lane == 0) {
      cs.ever_used = cr.ever_used;
      cs.count0 = cr.t;
      dsum_s[0] = cr.dsum_prev;
    }
  }
  int t0 = 0, fm;  // tokens before t0 are routed; fm: the first of the window that misses an expert
  if (ahead != nullptr) {
    if (tid == 0) first_miss_s = B;
    __syncthreads();
    if (tid < B && ahead->miss[tid]) atomicMin(&first_miss_s, tid);
    if (tid <= B) dsum_s[tid] = ahead->dsum[tid];
    __syncthreads();
    fm = first_miss_s;
    for (int i = tid; i < fm * K; i += kRouteWaves * kWave) {
      const int t = i / K, pos = i - t * K;
      const int e = ahead->touched[t][pos];
      if (e < MOE_MAX_EXPERTS) atomicMax(&cs.stamp[e], (long long)(cs.count0 + t) * K + pos);
      atomicAdd(&count_s[sel->slot[t][pos] & (MOE_MAX_EXPERTS - 1)], 1);
    }
  }
  if (ahead == nullptr || fm < B) {
    for (int i = tid; i < B * N; i += kRouteWaves * kWave) {
      const int t = i / N;
      z_all[t * MOE_MAX_EXPERTS + (i - t * N)] = logits[i];
    }
  }
  __syncthreads();
  if (ahead == nullptr) {
    for (int t = wave; t < B; t += kRouteWaves) {
      const bool active = lane < N;
      const float z = active ? z_all[t * MOE_MAX_EXPERTS + lane] : 0.f;
      const float r = rt::wave_max(active ? z : -INFINITY) - rt::wave_min(active ? z : INFINITY);
      if (lane == 0) range_s[t] = r;
    }
    __syncthreads();
    if (tid == 0) {
#pragma clang fp contract(off)
      float acc = dsum_s[0];
      for (int t = 0; t < B; ++t) {
        acc = acc + range_s[t];
        dsum_s[t + 1] = acc;
      }
    }
  }

  bool routed_ahead = ahead != nullptr;
  while (t0 < B) {  // (t0 and everything that steers the loop is the same in every thread)
    int window_end = B;
    rt::CacheRegs cr, next;
    if (!routed_ahead) {
      if (tid == 0) first_miss_s = B;
      lds_barrier();
      const int t = t0 + wave;
      if (t < B) {
        cr = batch_cache_regs(cs, lane, t, dsum_s[t]);
        int n_miss = 0;
        rt::route_wave(p, z_all + t * MOE_MAX_EXPERTS, cr, st, reinterpret_cast<moe_route_out_t *>(stage_s[wave]), HostOut{nullptr, nullptr},
                       asm_s[wave], lane, rt::BoundaryFlags{nullptr, 0}, &next, false, &n_miss);
        if (n_miss > 0 && lane == 0) atomicMin(&first_miss_s, t);
      }
      lds_barrier();
      window_end = min(t0 + kRouteWaves, B);
      fm = min(first_miss_s, window_end);  // tokens t0 .. fm-1 stand as they are
      if (t < fm) {
        if (lane < rt::kRecWords / 4)
          reinterpret_cast<u32x4 *>(out + t)[lane] = reinterpret_cast<const u32x4 *>(stage_s[wave])[lane];
        if (lane < N && next.stamp != cr.stamp) atomicMax(&cs.stamp[lane], (long long)next.stamp);
        store_sel(stage_s[wave], K, lane, t, sel);
        if (lane < K) atomicAdd(&count_s[stage_s[wave][rt::W_SLOT + lane] & (MOE_MAX_EXPERTS - 1)], 1);
      }
    }
    routed_ahead = false;
    if (tid < 2) cs.counter[tid] += (long long)K * (fm - t0);  // selections and hits
    lds_barrier();
    t0 = fm;
    if (fm < window_end) {
      // token fm misses at least one expert: routed against the merged state, which it updates
      missed = true;
      if (wave == 0) {
        cr = batch_cache_regs(cs, lane, fm, dsum_s[fm]);
        rt::route_wave(p, z_all + fm * MOE_MAX_EXPERTS, cr, st, out + fm, HostOut{nullptr, nullptr}, asm_s[0], lane,
                       rt::BoundaryFlags{nullptr, 0}, &next, false);
        store_sel(asm_s[0], K, lane, fm, sel);
        cs.my_slot[lane] = next.my_slot;
        cs.slot_exp[lane] = next.slot_exp;
        cs.born[lane] = next.born;
        cs.stamp[lane] = next.stamp;
        if (lane < 6) cs.counter[lane] = next.counter;
        if (lane == 0) cs.ever_used = next.ever_used;
      }
      t0 = fm + 1;
    }
  }
  // Every record is on its way to host memory (those of route_ahead_kernel are there since its end): one fence behind the
  // barrier covers the stores of all wavefronts, then the host, which polls, is told.  (A fence in each wavefront wrote
  // the L2 back sixteen times: 11.4 against 7.3 us for 8 tokens.)
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (tid == 0) {
    __threadfence_system();
    __hip_atomic_store(done, p.seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
  if (wave == 1 && planned.plan != nullptr) {
    if (missed) {
      if (lane == 0) planned.plan->n_up = planned.plan->n_down = 0;
    } else {
      make_plan(planned, B, K, count_s, order_s, lane);
    }
  }
  if (wave == 0) {
    if (lane < N) {
      st->expert_slot[lane] = cs.my_slot[lane];
      st->stamp[lane] = cs.stamp[lane];
      st->born[lane] = cs.born[lane];
    }
    if (lane < p.capacity) st->slot_expert[lane] = cs.slot_exp[lane];
    if (lane < 6) (&st->selections)[lane] = cs.counter[lane];
    if (lane == 0) {
      st->ever_used = cs.ever_used;
      st->delta_sum = dsum_s[B];
      st->count = cs.count0 + B;
    }
  }
}

// ---- experts of the batch ---------------------------------------------------------------------------
// Two weights-stationary products per expert over the tokens routed to it (tiles of 16 tokens, up to kGroupTiles of
// them per unit), each weight read once per 64 tokens:
//   up_batch_kernel    h[token][record] = silu(gate . x) (up . x) w           unit = (expert, block of records)
//   down_batch_kernel  P[token, expert][column] = sum of h[token][record] down[record][column]
//                                                                  unit = (expert, 256 columns, block of records)
//   reduce_batch_kernel adds a token's rows of P in a fixed order and rounds to bf16.
// What bounds them: HBM, and below it what one compute unit's L1 can keep in flight (about 58 KB, 23-38 GB/s), so
// every compute unit has to stream evenly and nothing may be read twice.  Hence a workgroup of four wavefronts with
// the whole register file (one wavefront per SIMD): the tokens' activations (up) and the output tile (down) of 64
// tokens stay in registers for the unit, no weights are staged through LDS, and no barrier stands in the load
// stream except one per 16 records of `up`.  A unit finds its tokens itself from the selected slots (1 KB): no tables
// are made on the host or sent.  Measured (60 experts of 1408, shared 5632, top-4, d = 2048; both kernels): 19 distinct
// experts, 128 tokens, 399 MB: 62 + 40 us, against 203 us for one fused kernel over tiles of 16 tokens with the down
// projection on the fp32 matrix instruction; 8 experts, 8 tokens, 208 MB: 28 + 16 us against 47 us.
// (h written as three bf16 planes instead of fp32, split once by `up`: 63 + 42 us; h costs `down` a third of what W does.)
constexpr int kBWaves = 4;
constexpr int kGroupTiles = 4;  // token tiles per unit
constexpr int kHBlock = 16 * 32 * 4;  // bytes of h of one token tile and 32 records

struct UnitPos {
  int entry, unit;  // index into BatchParams::e, and the unit's place inside that entry
};
// the entry a workgroup belongs to: the last one whose first unit is not beyond it
// (P: BatchParams, or BatchPlanned with the list in memory)
struct BatchPlanned : BatchArgs {
  const BatchEntry *e;
};
template <bool DOWN, typename P>
__device__ __forceinline__ UnitPos find_unit(const P &p, int block, int lane) {
  int at = 0;
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int i = lane + 64 * j;
    const int i_c = i < p.n_entries ? i : 0;
    const uint32_t u0 = DOWN ? p.e[i_c].unit0_down : p.e[i_c].unit0_up;
    at += (int)__builtin_popcountll(__builtin_amdgcn_ballot_w64(i < p.n_entries && (int)u0 <= block));
  }
  at = __builtin_amdgcn_readfirstlane(at - 1);
  return UnitPos{at, block - (int)(DOWN ? p.e[at].unit0_down : p.e[at].unit0_up)};
}

// Position of a unit: units of an expert with several token groups are laid out in blocks of 8 x groups, so that the
// groups reading the same weights sit 8 workgroups apart - on one XCD, where they share them in its L2.
struct GroupPos {
  int part, group;
};
__device__ __forceinline__ GroupPos group_pos(int unit, int groups) {
  if (groups == 1) return GroupPos{unit, 0};
  const int blk = unit / (8 * groups), r = unit - blk * 8 * groups;
  return GroupPos{blk * 8 + (r & 7), r >> 3};
}

// The places of group `group` of an expert, in token order: list[i] = token * 8 + k (k: the expert's place in the token's
// selection), by one wavefront into LDS of its own.  list has 64 entries; unused ones name the segment's first token.
// Every place that names the slot is listed, as the host counts them: a token whose logits are not numbers leaves places
// that nothing filled, whose record reads slot 0 with weight 0, so that it may name slot 0 several times.
__device__ __forceinline__ void token_list(const BatchArgs &p, int slot, int group, int n, int lane, uint16_t *list) {
  if (slot < 0) {
    const int t = p.t0 + group * 64 + lane;
    list[lane] = (uint16_t)((lane < n ? t : p.t0 + group * 64) * 8);
  } else {
    int seen = -64 * group;
    uint64_t sel[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int t = min(p.t0 + 64 * j + lane, kMaxBatch - 1);
      sel[j] = *reinterpret_cast<const uint64_t *>(p.sel->slot[t]);
    }
    list[lane] = (uint16_t)(p.t0 * 8);
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int t = p.t0 + 64 * j + lane;
      uint32_t ks = 0;  // the token's places
#pragma unroll
      for (int i = 0; i < MOE_MAX_TOPK; ++i)
        if (i < p.top_k && (int)((sel[j] >> (8 * i)) & 0xffu) == slot) ks |= 1u << i;
      if (t >= p.t1) ks = 0;
      const uint64_t m = __builtin_amdgcn_ballot_w64(ks != 0);
      int at = seen + (int)__builtin_popcountll(m & ((1ull << lane) - 1ull));
      seen += (int)__builtin_popcountll(m);
      for (uint64_t q = __builtin_amdgcn_ballot_w64((ks & (ks - 1u)) != 0); q; q &= q - 1) {  // (rare: several places)
        const int l = (int)__builtin_ctzll(q);
        const int extra = (int)__builtin_popcount((uint32_t)__builtin_amdgcn_readlane((int)ks, l)) - 1;
        if (lane > l) at += extra;
        seen += extra;
      }
      for (; ks; ks &= ks - 1u, ++at)
        if (at >= 0 && at < 64) list[at] = (uint16_t)(t * 8 + (int)__builtin_ctz(ks));
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Eight h of one token (A operand: consecutive records) as three bf16 vectors that add up to them exactly (8 + 8 + 8
// significant bits, truncated): the down projection runs on the bf16 matrix instruction with the precision of a 32-bit h
// (weights are bf16, products exact, fp32 sums).  Where nothing is left for a part of an h other than 0 it is 2^-126 with
// the sign of h, not 0: beside an infinite weight (or of an infinite h) a zero part would make a NaN of the infinity.
__device__ __forceinline__ void split3(const f32x4 &lo, const f32x4 &hi, u32x4 (&out)[3]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    uint32_t part[3][2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const float h = i < 2 ? lo[2 * i + j] : hi[2 * i + j - 4];
      const uint32_t u = __float_as_uint(h);
      // magnitudes from here on (what an infinity leaves is not a number, which fmaxf passes over)
      const float least = __builtin_amdgcn_fmed3f(fabsf(h), 0.f, 0x1p-126f);  // the smaller of |h| and 2^-126
      const float r1 = fmaxf(fabsf(h) - fabsf(__uint_as_float(u & 0xffff0000u)), least);
      const uint32_t u1 = __float_as_uint(r1);
      part[0][j] = u;
      part[1][j] = u1;
      part[2][j] = __float_as_uint(fmaxf(r1 - __uint_as_float(u1 & 0xffff0000u), least));
    }
#pragma unroll
    for (int q = 0; q < 3; ++q) out[q][i] = __builtin_amdgcn_perm(part[q][1], part[q][0], 0x07060302u);
#pragma unroll
    for (int q = 1; q < 3; ++q) out[q][i] |= out[0][i] & 0x80008000u;
  }
}

// D: hidden size.  Wavefront w owns the w-th quarter of the hidden dimension: the tokens' activations there stay in
// registers (B operands), the gate and up rows of 16 records at a time are streamed (A operands), in two halves whose
// loads are requested as soon as the registers are free.  The four partial sums meet in LDS (double buffer, one
// barrier per 16 records); wavefront i then finishes token tile i: h to memory in the order in which down_batch_kernel
// reads it, per (token tile, 32 records) two blocks of [lane][4] fp32, lane = 16 (record / 8) + token: records 0..3 and
// 4..7 of the lane's eight.
template <int D, int NT>
__device__ __forceinline__ void up_unit(const BatchArgs &p, const BatchEntry &e, int part, int group, int lane, int wave,
                                        f32x4 *red, uint16_t *list) {
  constexpr int KQ = D / kBWaves, KS = KQ / 32, HS = KS / 2;
  const int rows = e.slot < 0 ? p.shared_inter : p.inter;
  const int rec0 = part * p.up_records, n_blk = (min(p.up_records, rows - rec0)) / 16;
  const uint8_t *blob = e.slot < 0 ? p.shared_blob : p.slot_pool + (int64_t)e.slot * p.slot_bytes;
  const int64_t row_bytes = (int64_t)D * 2, rec_bytes = 3 * row_bytes;
  const int m16 = lane & 15, kq = lane >> 4;
  const int n_tok = min((int)e.n_tok - 64 * group, 64);

  const uint8_t *row = blob + (int64_t)(rec0 + m16) * rec_bytes + ((int64_t)wave * KQ + kq * 8) * 2;
  u32x4 g0[HS], u0[HS], g1[HS], u1[HS];
  auto load = [&](const uint8_t *q, u32x4 *g, u32x4 *u) {
#pragma unroll
    for (int s = 0; s < HS; ++s) {
      // (plain loads, not streaming ones: a load covers 64 bytes of each of 16 rows, the next one the other half of
      // the same 128-byte lines)
      g[s] = *reinterpret_cast<const u32x4 *>(q + s * 64);
      u[s] = *reinterpret_cast<const u32x4 *>(q + row_bytes + s * 64);
    }
  };
  load(row, g0, u0);
  load(row + HS * 64, g1, u1);

  token_list(p, e.slot, group, n_tok, lane, list);
  u32x4 x[NT][KS];
#pragma unroll
  for (int i = 0; i < NT; ++i) {
    const int t = list[i * 16 + m16] >> 3;
    const uint16_t *xr = p.x + (size_t)t * D + wave * KQ + kq * 8;
#pragma unroll
    for (int s = 0; s < KS; ++s) x[i][s] = *reinterpret_cast<const u32x4 *>(xr + s * 32);
  }
  // what this wavefront finishes: token tile `wave` (if there is one)
  const int my = list[min(wave, NT - 1) * 16 + m16];
  const float wt = e.slot < 0 ? 1.f : p.sel->weight[my >> 3][my & 7];
  const int n32 = (rows + 31) / 32;
  uint8_t *hb = p.h + ((int64_t)e.h_base + (int64_t)(group * kGroupTiles + wave) * n32) * kHBlock;

  int parity = 0;
  auto block = [&](int blk, auto next_tag) {
    constexpr bool NEXT = decltype(next_tag)::value;
    f32x4 g[NT], u[NT];
#pragma unroll
    for (int i = 0; i < NT; ++i) g[i] = u[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < HS; ++s)
#pragma unroll
      for (int i = 0; i < NT; ++i) {
        g[i] = mfma_bf16(g0[s], x[i][s], g[i]);
        u[i] = mfma_bf16(u0[s], x[i][s], u[i]);
      }
    row += 16 * rec_bytes;
    if constexpr (NEXT) load(row, g0, u0);
#pragma unroll
    for (int s = 0; s < HS; ++s)
#pragma unroll
      for (int i = 0; i < NT; ++i) {
        g[i] = mfma_bf16(g1[s], x[i][HS + s], g[i]);
        u[i] = mfma_bf16(u1[s], x[i][HS + s], u[i]);
      }
    if constexpr (NEXT) load(row + HS * 64, g1, u1);
    f32x4 *rb = red + (size_t)parity * (kBWaves * 2 * NT * 64);
    parity ^= 1;
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      rb[((wave * NT + i) * 2 + 0) * 64 + lane] = g[i];
      rb[((wave * NT + i) * 2 + 1) * 64 + lane] = u[i];
    }
    lds_barrier();
    if (wave < NT && wave * 16 < n_tok) {
      f32x4 gs = rb[wave * 2 * 64 + lane], us = rb[(wave * 2 + 1) * 64 + lane];
#pragma unroll
      for (int w = 1; w < kBWaves; ++w) {
        gs += rb[((w * NT + wave) * 2 + 0) * 64 + lane];
        us += rb[((w * NT + wave) * 2 + 1) * 64 + lane];
      }
      // records 4 kq + v of the block, token m16 of the tile
      f32x4 h;
#pragma unroll
      for (int v = 0; v < 4; ++v) h[v] = gs[v] / (1.f + __expf(-gs[v])) * us[v] * wt;
      const int rec = rec0 + blk * 16;
      uint8_t *o = hb + (int64_t)(rec >> 5) * kHBlock + (kq & 1) * (kHBlock / 2) + (((rec >> 3) & 3) + (kq >> 1)) * 256 + m16 * 16;
      *reinterpret_cast<f32x4 *>(o) = h;
      // the second half of the last 32 records may not exist: zeros
      if (rec + 16 == rows && (rows & 31)) *reinterpret_cast<f32x4 *>(o + 512) = f32x4{0.f, 0.f, 0.f, 0.f};
    }
  };
  for (int blk = 0; blk + 1 < n_blk; ++blk) block(blk, std::true_type{});
  block(n_blk - 1, std::false_type{});
}

template <int D, typename P>
__device__ __forceinline__ void up_block(const P &list_in, int block, int lane, int wave, f32x4 *red, uint16_t *list) {
  const UnitPos up = find_unit<false>(list_in, block, lane);
  const BatchEntry e = list_in.e[up.entry];
  const BatchArgs p = list_in;  // (a copy: a reference into the launch's arguments puts them all into scratch)
  const int groups = (e.n_tok + 63) / 64;
  const GroupPos gp = group_pos(up.unit, groups);
  if (gp.part * p.up_records >= (e.slot < 0 ? p.shared_inter : p.inter)) return;  // padding of the unit grid
  const int tiles = (min((int)e.n_tok - 64 * gp.group, 64) + 15) / 16;
  if (tiles == 1) up_unit<D, 1>(p, e, gp.part, gp.group, lane, wave, red, list);
  else if (tiles == 2) up_unit<D, 2>(p, e, gp.part, gp.group, lane, wave, red, list);
  else up_unit<D, 4>(p, e, gp.part, gp.group, lane, wave, red, list);
}
template <int D>
__global__ __launch_bounds__(kBWaves *kWave, 1) void up_batch_kernel(BatchParams p) {
  __shared__ f32x4 red[2 * kBWaves * 2 * kGroupTiles * 64];
  __shared__ uint16_t list_s[kBWaves][64];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  up_block<D>(p, blockIdx.x, threadIdx.x & 63, wave, red, list_s[wave]);
}
// the batch's arguments with what the device decided
__device__ __forceinline__ BatchPlanned planned_args(const BatchArgs &p, const BatchPlan *plan) {
  BatchPlanned a;
  static_cast<BatchArgs &>(a) = p;
  a.up_records = plan->up_records;
  a.down_groups = plan->down_groups;
  a.shared_row0 = plan->shared_row0;
  a.n_entries = plan->n_entries;
  a.e = plan->e;
  return a;
}
// Workgroups past the last unit end at once.  (One workgroup per compute unit that walks the units: the loop costs `down`, which
// fills the register file, spills: 8 tokens 20.1 us instead of 15.9.)
template <int D>
__global__ __launch_bounds__(kBWaves *kWave, 1) void up_planned_kernel(BatchArgs p, const BatchPlan *plan) {
  __shared__ f32x4 red[2 * kBWaves * 2 * kGroupTiles * 64];
  __shared__ uint16_t list_s[kBWaves][64];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if ((int)blockIdx.x >= plan->n_up) return;
  up_block<D>(planned_args(p, plan), blockIdx.x, threadIdx.x & 63, wave, red, list_s[wave]);
}

// Eight rows of eight bf16 columns -> eight columns of eight rows, inside a lane: the record layout keeps the columns of
// W_down as rows, the matrix instruction wants eight consecutive records of one column.
__device__ __forceinline__ void transpose8(const u32x4 (&r)[8], u32x4 (&c)[8]) {
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const uint32_t sel = (j & 1) ? 0x07060302u : 0x05040100u;
#pragma unroll
    for (int q = 0; q < 4; ++q) c[j][q] = __builtin_amdgcn_perm(r[2 * q + 1][j >> 1], r[2 * q][j >> 1], sel);
  }
}

// Wavefront w takes every fourth group of 32 records of the unit's block and accumulates the unit's [tokens][256
// columns] tile over them in registers; the four tiles are added through LDS at the end.  Lane l loads columns
// 8 (l % 16) .. + 8 of records 8 (l / 16) + i: full 128-byte lines, each lane an 8 x 8 block that it transposes.
template <int D, int NT>
__device__ __forceinline__ void down_unit(const BatchArgs &p, const BatchEntry &e, int part, int group, int lane, int wave,
                                          float *red, uint16_t *list) {
  constexpr int CBLKS = D / 256;
  const int rows = e.slot < 0 ? p.shared_inter : p.inter;
  const int cblk = part % CBLKS, rc = part / CBLKS;
  const int n32 = (rows + 31) / 32;
  const int g_begin = rc * p.down_groups, g_end = min(n32, g_begin + p.down_groups);
  const uint8_t *blob = e.slot < 0 ? p.shared_blob : p.slot_pool + (int64_t)e.slot * p.slot_bytes;
  const int64_t row_bytes = (int64_t)D * 2, rec_bytes = 3 * row_bytes;
  const int m16 = lane & 15, kq = lane >> 4;
  const int n_tok = min((int)e.n_tok - 64 * group, 64), tiles = (n_tok + 15) / 16;
  const uint8_t *wbase = blob + 2 * row_bytes + (int64_t)cblk * 512;  // the same in every lane
  const uint8_t *hbase = p.h + ((int64_t)e.h_base + (int64_t)group * kGroupTiles * n32) * kHBlock;

  u32x4 w0[8], w1[8];  // columns 0..127 and 128..255 of 32 records
  auto load_w = [&](int g, int c, u32x4 (&w)[8]) {
    // (in a last group of 16 records the lanes of the missing half read the first half again; zeroed before use)
    const uint8_t *q = wbase + (int64_t)g * 32 * rec_bytes + c * 256;
    const uint32_t off = (uint32_t)(g * 32 + 32 > rows ? kq & 1 : kq) * (uint32_t)(8 * rec_bytes) + (uint32_t)m16 * 16u;
#pragma unroll
    for (int i = 0; i < 8; ++i) w[i] = stream_load(reinterpret_cast<const u32x4 *>(q + i * rec_bytes + off));
  };
  f32x4 h[NT][2];
  auto load_h = [&](int g, int i) {
#pragma unroll
    for (int q = 0; q < 2; ++q)  // (tiles past the last repeat it; their rows are not stored)
      h[i][q] = *reinterpret_cast<const f32x4 *>(hbase + ((int64_t)min(i, tiles - 1) * n32 + g) * kHBlock + q * (kHBlock / 2) +
                                                 (uint32_t)lane * 16u);
  };
  f32x4 acc[NT][2][8];
#pragma unroll
  for (int i = 0; i < NT; ++i)
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int j = 0; j < 8; ++j) acc[i][c][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  // One group of 32 records; NEXT: there is a group after it, whose loads are requested as registers become free.  h is split
  // first, once for both halves of the columns; its registers then take the next group's (requested ahead of its weights:
  // loads complete in order, and h is wanted first).  With four token tiles everything but the accumulators lives in 256
  // registers: the order below is kept as written, or loads of later tiles are moved up and spill.
  auto step = [&](int g, auto next_tag) {
    constexpr bool NEXT = decltype(next_tag)::value;
    u32x4 a[NT][3];
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      split3(h[i][0], h[i][1], a[i]);
      if constexpr (NEXT) load_h(g + kBWaves, i);
      if constexpr (NT > 2) __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      u32x4 (&w)[8] = c == 0 ? w0 : w1;
      if (g * 32 + 32 > rows) {
#pragma unroll
        for (int i = 0; i < 8; ++i)
          if (kq >= 2) w[i] = u32x4{0u, 0u, 0u, 0u};
      }
      u32x4 col[8];
      transpose8(w, col);
      if constexpr (NEXT) load_w(g + kBWaves, c, w);
      if constexpr (NT > 2) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < NT; ++i)
#pragma unroll
        for (int q = 2; q >= 0; --q)  // the small parts first
#pragma unroll
          for (int j = 0; j < 8; ++j) acc[i][c][j] = mfma_bf16(a[i][q], col[j], acc[i][c][j]);
    }
  };
  int g = g_begin + wave, left = g < g_end ? (g_end - g + kBWaves - 1) / kBWaves : 0;
  if (left > 0) {
#pragma unroll
    for (int i = 0; i < NT; ++i) load_h(g, i);
    load_w(g, 0, w0);
    load_w(g, 1, w1);
    for (; left > 1; --left, g += kBWaves) step(g, std::true_type{});
    step(g, std::false_type{});
  }
  // the tiles of the four wavefronts, one token tile at a time: [wave][16 rows][256 columns]
  token_list(p, e.slot, group, n_tok, lane, list);
  const int n_seg = p.t1 - p.t0;
#pragma unroll
  for (int i = 0; i < NT; ++i) {
    if (i * 16 >= n_tok) break;
    if (i > 0) lds_barrier();
    float *mine = red + wave * 4096;
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        float *o = mine + (4 * kq + v) * 256 + c * 128 + m16 * 8;
        *reinterpret_cast<f32x4 *>(o) = f32x4{acc[i][c][0][v], acc[i][c][1][v], acc[i][c][2][v], acc[i][c][3][v]};
        *reinterpret_cast<f32x4 *>(o + 4) = f32x4{acc[i][c][4][v], acc[i][c][5][v], acc[i][c][6][v], acc[i][c][7][v]};
      }
    lds_barrier();
#pragma unroll
    for (int r = 0; r < 4; ++r) {  // wavefront w: rows w, w + 4, ...
      const int t16 = r * 4 + wave;
      if (i * 16 + t16 >= n_tok) break;
      f32x4 v = *reinterpret_cast<const f32x4 *>(red + t16 * 256 + lane * 4);
#pragma unroll
      for (int w = 1; w < kBWaves; ++w) v += *reinterpret_cast<const f32x4 *>(red + w * 4096 + t16 * 256 + lane * 4);
      const int tk = list[i * 16 + t16], t = (tk >> 3) - p.t0;
      const int64_t at = e.slot < 0 ? (int64_t)p.shared_row0 + (int64_t)rc * n_seg + t
                                    : ((int64_t)rc * n_seg + t) * p.top_k + (tk & 7);
      *reinterpret_cast<f32x4 *>(p.partial + at * D + cblk * 256 + lane * 4) = v;
    }
  }
}

template <int D, typename P>
__device__ __forceinline__ void down_block(const P &list_in, int block, int lane, int wave, float *red, uint16_t *list) {
  const UnitPos up = find_unit<true>(list_in, block, lane);
  const BatchEntry e = list_in.e[up.entry];
  const BatchArgs p = list_in;  // (a copy: a reference into the launch's arguments puts them all into scratch)
  const int groups = (e.n_tok + 63) / 64;
  const GroupPos gp = group_pos(up.unit, groups);
  const int rows = e.slot < 0 ? p.shared_inter : p.inter;
  if (gp.part / (D / 256) * p.down_groups * 32 >= rows) return;  // padding of the unit grid
  const int tiles = (min((int)e.n_tok - 64 * gp.group, 64) + 15) / 16;
  if (tiles == 1) down_unit<D, 1>(p, e, gp.part, gp.group, lane, wave, red, list);
  else if (tiles == 2) down_unit<D, 2>(p, e, gp.part, gp.group, lane, wave, red, list);
  else down_unit<D, 4>(p, e, gp.part, gp.group, lane, wave, red, list);
}
template <int D>
__global__ __launch_bounds__(kBWaves *kWave, 1) void down_batch_kernel(BatchParams p) {
  __shared__ __attribute__((aligned(16))) float red[kBWaves * 4096];
  __shared__ uint16_t list_s[kBWaves][64];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  down_block<D>(p, blockIdx.x, threadIdx.x & 63, wave, red, list_s[wave]);
}
template <int D>
__global__ __launch_bounds__(kBWaves *kWave, 1) void down_planned_kernel(BatchArgs p, const BatchPlan *plan) {
  __shared__ __attribute__((aligned(16))) float red[kBWaves * 4096];
  __shared__ uint16_t list_s[kBWaves][64];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if ((int)blockIdx.x >= plan->n_down) return;
  down_block<D>(planned_args(p, plan), blockIdx.x, threadIdx.x & 63, wave, red, list_s[wave]);
}

// y[t] = the sum of token t's rows of P - its experts in selection order, each block of records in turn, then the
// shared expert's blocks - rounded to bf16.  grid = (tokens, d / 256), one wavefront: all of a token's rows are
// requested eight at a time.
__global__ __launch_bounds__(kWave) void reduce_batch_kernel(const float *partial, uint16_t *y, int d, int t0, int n_seg, int top_k,
                                                             int n_rc, int shared_row0, int n_rc_shared, const BatchPlan *plan) {
  if (plan != nullptr) {
    n_rc = plan->n_rc;
    n_rc_shared = plan->n_rc_shared;
    shared_row0 = plan->shared_row0;
  }
  const int t = blockIdx.x, col = blockIdx.y * 256 + threadIdx.x * 4;
  f32x4 s = {0.f, 0.f, 0.f, 0.f};
  for (int rc = 0; rc < n_rc; ++rc) {
    const float *q = partial + ((size_t)(rc * n_seg + t) * top_k) * d + col;
#pragma unroll 8
    for (int k = 0; k < top_k; ++k) s += *reinterpret_cast<const f32x4 *>(q + (size_t)k * d);
  }
  const float *q = partial + ((size_t)shared_row0 + t) * d + col;
#pragma unroll 8
  for (int rc = 0; rc < n_rc_shared; ++rc) s += *reinterpret_cast<const f32x4 *>(q + (size_t)rc * n_seg * d);
  u32x2 o;
  o.x = (uint32_t)f32_to_bf16_rne(s[0]) | ((uint32_t)f32_to_bf16_rne(s[1]) << 16);
  o.y = (uint32_t)f32_to_bf16_rne(s[2]) | ((uint32_t)f32_to_bf16_rne(s[3]) << 16);
  *reinterpret_cast<u32x2 *>(y + (size_t)(t0 + t) * d + col) = o;
}

}  // namespace

bool batch_shape_supported(int weight_fmt, int act_fmt, int hidden, int inter, int shared_inter) {
  return weight_fmt == MOE_W_BF16 && act_fmt == MOE_A_BF16 && (hidden == 1024 || hidden == 2048) && inter % 16 == 0 &&
         shared_inter % 16 == 0;
}

hipError_t launch_gate_gemm(const void *x, const void *gate_w, float *logits, int B, int N, int hidden, hipStream_t s) {
  if (B <= 0 || N <= 0 || N > MOE_MAX_EXPERTS) return hipErrorInvalidValue;
  const dim3 g((B + 15) / 16, (N + 15) / 16), blk(kWave * kGateSplit);
  const uint16_t *xp = static_cast<const uint16_t *>(x), *wp = static_cast<const uint16_t *>(gate_w);
  if (hidden == 32 * kGateSplit * 8)
    hipLaunchKernelGGL(gate_gemm_kernel<8>, g, blk, 0, s, xp, wp, logits, B, N, hidden);
  else if (hidden == 32 * kGateSplit * 4)
    hipLaunchKernelGGL(gate_gemm_kernel<4>, g, blk, 0, s, xp, wp, logits, B, N, hidden);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

// Batches of more tokens than this are routed ahead: up to one window route_batch_kernel has nothing to wait for, from
// the second window on the extra launch pays (moe_route_batch in all, miss-free, without / with it: 24 tokens 29.6 /
// 29.3 us, 32 tokens 31.8 / 29.5, 64 tokens 44.2 / 32.5; 128 tokens: the two kernels 8.9 + 5.1 us against 40).
constexpr int kAheadMinTokens = kRouteWaves;

hipError_t launch_route_batch(const RouteParams &p, const float *logits, int B, LayerState *state, moe_route_out_t *out,
                              BatchSel *sel, BatchAhead *ahead, uint32_t *done, const BatchPlanFor &planned, hipStream_t s) {
  if (B <= 0 || B > kMaxBatch) return hipErrorInvalidValue;
  const bool use_ahead = B > kAheadMinTokens;
  if (use_ahead) {
    hipLaunchKernelGGL(route_ahead_kernel, dim3((B + kAheadWaves - 1) / kAheadWaves), dim3(kAheadWaves * kWave), 0, s, p, logits, B,
                       state, out, sel, ahead);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(route_batch_kernel, dim3(1), dim3(kRouteWaves * kWave), 0, s, p, logits, B, state, out, sel,
                     use_ahead ? ahead : nullptr, done, planned);
  return hipGetLastError();
}

hipError_t launch_up_batch(const BatchParams &p, int n_units, hipStream_t s) {
  if (n_units <= 0) return hipSuccess;
  if (p.hidden == 2048) hipLaunchKernelGGL(up_batch_kernel<2048>, dim3(n_units), dim3(kBWaves * kWave), 0, s, p);
  else if (p.hidden == 1024) hipLaunchKernelGGL(up_batch_kernel<1024>, dim3(n_units), dim3(kBWaves * kWave), 0, s, p);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_down_batch(const BatchParams &p, int n_units, hipStream_t s) {
  if (n_units <= 0) return hipSuccess;
  if (p.hidden == 2048) hipLaunchKernelGGL(down_batch_kernel<2048>, dim3(n_units), dim3(kBWaves * kWave), 0, s, p);
  else if (p.hidden == 1024) hipLaunchKernelGGL(down_batch_kernel<1024>, dim3(n_units), dim3(kBWaves * kWave), 0, s, p);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_reduce_batch(const BatchArgs &p, void *y, int n_rc, int n_rc_shared, hipStream_t s) {
  const int n_seg = p.t1 - p.t0;
  if (n_seg <= 0) return hipSuccess;
  hipLaunchKernelGGL(reduce_batch_kernel, dim3(n_seg, p.hidden / 256), dim3(kWave), 0, s, p.partial, static_cast<uint16_t *>(y),
                     p.hidden, p.t0, n_seg, p.top_k, n_rc, p.shared_row0, n_rc_shared, nullptr);
  return hipGetLastError();
}

hipError_t launch_planned_experts(const BatchArgs &p, const BatchPlan *plan, int n_cus, hipStream_t s) {
  if (n_cus < 1 || (p.hidden != 2048 && p.hidden != 1024)) return hipErrorInvalidValue;
  const dim3 g(kPlanRounds * n_cus), b(kBWaves * kWave);
  if (p.hidden == 2048) hipLaunchKernelGGL(up_planned_kernel<2048>, g, b, 0, s, p, plan);
  else hipLaunchKernelGGL(up_planned_kernel<1024>, g, b, 0, s, p, plan);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (p.hidden == 2048) hipLaunchKernelGGL(down_planned_kernel<2048>, g, b, 0, s, p, plan);
  else hipLaunchKernelGGL(down_planned_kernel<1024>, g, b, 0, s, p, plan);
  return hipGetLastError();
}

hipError_t launch_planned_reduce(const BatchArgs &p, const BatchPlan *plan, void *y, hipStream_t s) {
  const int n_seg = p.t1 - p.t0;
  hipLaunchKernelGGL(reduce_batch_kernel, dim3(n_seg, p.hidden / 256), dim3(kWave), 0, s, p.partial, static_cast<uint16_t *>(y), p.hidden,
                     p.t0, n_seg, p.top_k, 0, 0, 0, plan);
  return hipGetLastError();
}

}  // namespace moe
