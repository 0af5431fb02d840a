// Device helpers shared by the expert GEMV kernels (all weight formats).
#pragma once

#include "common.h"
#include "deal.h"

namespace moe {

constexpr int kRedFloats = 16384;  // LDS floats (64 KB) shared by the wavefronts' rows in the final reduction

// for lambdas that are called in several places: as calls they would keep their captures in memory
#define MOE_INLINE __attribute__((always_inline))

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// weights are read once: mark the loads non-temporal so they do not displace x and the partial rows in L2
__device__ __forceinline__ u32x4 stream_load(const u32x4 *p) { return __builtin_nontemporal_load(p); }

// One record of a blob as a buffer resource.  bytes = 0 makes it an empty one: loads from it return zeros and touch no
// memory, so that a place of a list that holds nothing is loaded by the same instructions as any other (no branch
// around loads, see RecordWalker::step).  base has to be the same in every lane.
typedef __amdgpu_buffer_rsrc_t RecBuffer;
__device__ __forceinline__ RecBuffer record_buffer(const uint8_t *base, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(base), 0, bytes, 0x00020000);
}
// weights are read once: non-temporal (aux 2), so that they do not displace x and the partial rows in L2.  at: the same in
// every lane, off: this lane's offset
__device__ __forceinline__ u32x4 record_load(RecBuffer r, uint32_t at, uint32_t off) {
  return __builtin_amdgcn_raw_buffer_load_b128(r, off, at, 2);
}

// (no scalar offset: behind a 16-byte store that has one the compiler lets the next vector instruction write the registers
// that hold the data, and the last lanes then store what that instruction wrote - seen in one record of 500)
__device__ __forceinline__ void record_store(RecBuffer r, uint32_t off, u32x4 v) {
  __builtin_amdgcn_raw_buffer_store_b128(v, r, off, 0, 0);
}

__device__ __forceinline__ float dot2_bf16(uint32_t w, uint32_t x, float acc) {
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, w), __builtin_bit_cast(bf16x2, x), acc, false);
}

// sums a and b over the wavefront (both results in every lane), the two chains interleaved
__device__ __forceinline__ void wave_sum2(float &a, float &b) {
  a += dpp_f32<0x128>(a);
  b += dpp_f32<0x128>(b);
  a += dpp_f32<0x124>(a);
  b += dpp_f32<0x124>(b);
  a += dpp_f32<0x122>(a);
  b += dpp_f32<0x122>(b);
  a += dpp_f32<0x121>(a);
  b += dpp_f32<0x121>(b);
  float a0 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(a), 0));
  float a1 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(a), 16));
  float a2 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(a), 32));
  float a3 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(a), 48));
  float b0 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(b), 0));
  float b1 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(b), 16));
  float b2 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(b), 32));
  float b3 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(b), 48));
  a = (a0 + a1) + (a2 + a3);
  b = (b0 + b1) + (b2 + b3);
}


// Walks the records one wavefront owns in one launch.
//
// Every workgroup owns a share of the shared expert's records followed by a share of the routed records (the K
// selected slots side by side, I records each); its wavefronts take list entries wave, wave+NW, ...  Shared
// records need nothing from the routing step, so streaming starts at once while the loads of the routing
// record are in flight; the record is unpacked when the first routed entry comes up.  Pass 0 covers the
// shared expert and the experts that were resident; pass 1 covers only the experts whose slots were filled
// for this token, so the first pass can run while the fills stream.  With the host tier at hand (host_blob) the launch walks
// twice instead: like pass 0, then over the experts that missed, straight from there (start_missing).
//
// Shares are equal and fixed.  With equal shares the workgroups do not finish together: the mean finish time of
// a workgroup depends on its XCD (about 1.4 us between the fastest and the slowest of 8, the same from launch to
// launch, nothing else systematic), plus about 0.9 us of launch-to-launch noise.  Neither of the two remedies
// pays: handing records out dynamically with device-scope atomics is far slower (an atomic on a contended
// address costs about 200 ns while HBM is saturated), and shares proportional to measured per-XCD rates (or
// skewed by XCD parity) leave the kernel time unchanged - the XCDs that finish early free bandwidth for the
// late ones, so the spread is not lost time.  Fixed shares keep the summation order of y, hence y itself,
// identical from run to run.
__device__ __forceinline__ u32x4 ld128(const void *p) { return *static_cast<const u32x4 *>(p); }
__device__ __forceinline__ u32x2 ld64(const void *p) { return *static_cast<const u32x2 *>(p); }

// IN (RouteIn) = kRouteBoundary: workgroup 0 of the launch runs the layer boundary; the records are shared among
// workgroups 1..G-1 and the decision is fetched only when the first routed entry comes up, once workgroup 0 has handed it
// over.  kRouteEverywhere: the same split, and the wavefronts of every workgroup work the decision out ahead of their first
// routed record (decide_now: one place in the kernel, where few registers are in use).
// STEP: distance between a wavefront's consecutive list entries (see deal).
//
// The walk is organised in runs - consecutive entries of the wavefront inside one blob (the shared expert, or one
// selected expert) - so that the per-record work is an increment and a decrement; slot, weight and the split of the
// routed index into (expert, row) are worked out once per run.  All of it is wavefront-uniform (scalar registers).
namespace rt {
struct DecideLds;
template <int NW>
__device__ void decide(const RouteParams &p, float z, int my_slot, float dsum_prev, int t, int lane, int wave, const LayerState *fills,
                       DecideLds &lds, uint64_t &slots, uint64_t &experts, uint32_t &miss_mask, float (&weight)[MOE_MAX_TOPK]);
}
template <int NW, int IN = kRouteBefore, int STEP = NW>
struct RecordWalker {
  int sh_at, n_sh;   // the wavefront's shared records: first row, how many (not yet started)
  int r, n_rt;       // its routed entries: next index into the K*I routed records, how many are left to start
  int left;          // records left in the current run
  int next_at;       // row of the current run's next record
  bool run_wanted;   // the pass covers the current run's expert
  bool run_shared;   // the current run is of shared records
  bool decided;      // the routing decision has been unpacked
  // the routing record: loaded at kernel start, unpacked when the first routed run comes up
  u32x4 rw0, rw1, rd;  // sel_weight[0..3], sel_weight[4..7], {tag, slots lo, slots hi, miss mask}
  uint64_t slots;
  uint64_t experts;    // 8 bits each, like slots (kRouteBoundary, kRouteEverywhere)
  uint32_t miss_mask;
  bool no_decision;    // the hand-over did not come
  int q0, nr;          // the workgroup's routed entries: the first one, how many
  bool missing_only;   // the walk covers the experts that missed, not the others
  uint8_t *fill_blob;  // the current run's expert comes from the host tier: the slot it is put into, else nullptr
  float z, dsum;       // kRouteEverywhere: lane's logit, Eq. 10's sum so far
  int my_slot, count;  // lane's expert's slot, tokens so far
  // the record found by step()
  const uint8_t *base;  // blob of the record's expert
  int rows, at;
  float wt;
  uint8_t *fill;        // nullptr, or the slot that the record (with its part of the tail) has to be put into

  // start of part b of n = q G + r records split into G parts: floor(b n / G).  b r < 2^20 (the host limits G to 2^10), so
  // that the product with ceil(2^32 / G) has the exact quotient in its upper half
  static __device__ __forceinline__ int bound(int b, uint32_t q, uint32_t r, uint32_t inv_g) {
    return (int)((uint32_t)b * q + __umulhi((uint32_t)b * r, inv_g));
  }

  // The record is the same for every lane and was written by an earlier launch: it is read through the scalar data
  // path (constant address space), whose completion is counted apart from the vector loads - waiting for it does not
  // wait for the weight loads already queued, and the values arrive in scalar registers.
  __device__ __forceinline__ void load_record(const GemvParams &p) {
    typedef const __attribute__((address_space(4))) u32x4 *cvec;
    cvec rr = (cvec)(reinterpret_cast<uintptr_t>(p.route));
    rw0 = rr[offsetof(moe_route_out_t, sel_weight) / 16];
    rw1 = rr[offsetof(moe_route_out_t, sel_weight) / 16 + 1];
    rd = rr[offsetof(moe_route_out_t, opaque) / 16];
  }

  // FUSED: the decision as workgroup 0 of this launch hands it over - eight 8-byte words, each carrying the
  // hand-over's 16-bit tag beside 48 bits of payload (layout: rt::BoundaryFlags).  The words are taken only when all
  // eight carry the tag, whatever order their stores arrived in; re-read until they do, at most spin_limit times.
  // No agent-scope acquire is involved (it would invalidate the XCD's L2 under thirty-two streaming compute
  // units - measured: the launch ran at half speed): the words are read with agent-scope atomic loads.
  __device__ __forceinline__ bool load_handover(const uint64_t *words, uint32_t tag, int spin_limit) {
    const uint32_t want = tag & 0xffffu;
    for (int i = 0; i < spin_limit; ++i) {
      uint64_t q[8];
      uint32_t tags_ok = 1;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        q[j] = __hip_atomic_load(words + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        tags_ok &= (uint32_t)(((uint32_t)q[j] & 0xffffu) == want);
      }
      if (__builtin_amdgcn_readfirstlane((int)tags_ok)) {
        // the same in every lane: kept in scalar registers from here on
#pragma unroll
        for (int j = 0; j < 8; ++j)
          q[j] = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(q[j] >> 32)) << 16) |
                 (uint64_t)((uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)q[j]) >> 16);
        rd.x = tag;
        rd.y = (uint32_t)q[0];
        rd.z = (uint32_t)(q[0] >> 32) | ((uint32_t)(q[1] & 0xffffu) << 16);
        rd.w = (uint32_t)(q[1] >> 16) & 0xffu;
        rw0.x = (uint32_t)q[2];
        rw0.y = (uint32_t)(q[2] >> 32) | ((uint32_t)q[3] << 16);
        rw0.z = (uint32_t)(q[3] >> 16);
        rw0.w = (uint32_t)q[4];
        rw1.x = (uint32_t)(q[4] >> 32) | ((uint32_t)q[5] << 16);
        rw1.y = (uint32_t)(q[5] >> 16);
        rw1.z = (uint32_t)q[6];
        rw1.w = (uint32_t)(q[6] >> 32) | ((uint32_t)q[7] << 16);
        experts = 0;
        const uint64_t e48 = ((q[1] >> 24) & 0xffffffu) | (((q[7] >> 16) & 0xffffffu) << 24);
#pragma unroll
        for (int k = 0; k < MOE_MAX_TOPK; ++k) experts |= ((e48 >> (6 * k)) & 63u) << (8 * k);
        return true;
      }
      __builtin_amdgcn_s_sleep(2);
    }
    return false;
  }

  __device__ __forceinline__ void init(const GemvParams &p, int wave) {
    constexpr int kFirst = IN == kRouteBefore || IN == kRouteGiven ? 0 : 1;  // workgroups that stream nothing
    const int b = (int)blockIdx.x - kFirst;
    // the routing record, or what it is worked out from, first: it is on its way while the shared records are set up
    if constexpr (IN == kRouteBefore) load_record(p);
    if constexpr (IN == kRouteEverywhere) {
      const int lane = (int)(threadIdx.x & 63), e = min(lane, p.b.route.n_experts - 1);
      z = p.b.logits[e];
      my_slot = p.b.state->expert_slot[e];
      dsum = p.b.state->delta_sum;
      count = p.b.state->count;
      __builtin_amdgcn_sched_barrier(0);
    }
    // the workgroup's list: ns shared records from row s0, then nr routed entries from q0
    const int s0 = bound(b, p.shared_q, p.shared_r, p.inv_g), ns = bound(b + 1, p.shared_q, p.shared_r, p.inv_g) - s0;
    q0 = bound(b, p.routed_q, p.routed_r, p.inv_g);
    nr = bound(b + 1, p.routed_q, p.routed_r, p.inv_g) - q0;
    const Deal mine = deal<NW, STEP>(ns, nr, wave);
    n_sh = mine.n_sh;
    n_rt = mine.n_rt;
    sh_at = s0 + mine.first_sh;
    r = q0 + mine.first_rt;
    left = 0;
    next_at = 0;
    at = 0;
    base = p.slot_pool;
    rows = p.inter;
    wt = 0.f;
    run_wanted = true;
    run_shared = false;
    decided = false;
    no_decision = false;
    fill_blob = fill = nullptr;
    missing_only = p.pass == 1;
    if constexpr (IN == kRouteGiven) {
      const float *w = p.given_weight;
      slots = p.given_slots;
      miss_mask = 0;
      rw0 = u32x4{__float_as_uint(w[0]), __float_as_uint(w[1]), __float_as_uint(w[2]), __float_as_uint(w[3])};
      rw1 = u32x4{__float_as_uint(w[4]), __float_as_uint(w[5]), __float_as_uint(w[6]), __float_as_uint(w[7])};
      decided = true;
    }
  }

  // kRouteEverywhere, after init() and the loads that are wanted ahead of the weights; by all wavefronts of the workgroup
  __device__ __forceinline__ void decide_now(const GemvParams &p, int wave, rt::DecideLds &lds) {
    // (what the decision reads through the scalar data path is wanted here, not where it is used: the compiler moves such
    // loads into the branches behind, one trip to memory each)
    const RouteParams &q = p.b.route;
    asm volatile("" ::"s"(dsum), "s"(count), "s"(q.lambda), "s"(q.delta_fixed), "s"(q.cumsum_p), "s"(q.n_experts), "s"(q.top_k),
                 "s"(q.top_j), "s"(q.renormalize), "s"(q.delta_mode), "s"(q.route_mode), "s"(q.max_rank));
    float w[MOE_MAX_TOPK];
    rt::decide<NW>(p.b.route, z, my_slot, dsum, count, (int)(threadIdx.x & 63), wave, p.host_blob != nullptr ? p.b.state : nullptr,
                   lds, slots, experts, miss_mask, w);
    rw0 = u32x4{__float_as_uint(w[0]), __float_as_uint(w[1]), __float_as_uint(w[2]), __float_as_uint(w[3])};
    rw1 = u32x4{__float_as_uint(w[4]), __float_as_uint(w[5]), __float_as_uint(w[6]), __float_as_uint(w[7])};
    decided = true;
  }

  // masks instead of a select chain: a chain over adjacent members is turned into an indexed load from a
  // memory copy of the struct, which then lives in scratch
  __device__ __forceinline__ float pick_weight(int k) const {
    uint32_t v = 0;
    v |= rw0.x & (0u - (uint32_t)(k == 0));
    v |= rw0.y & (0u - (uint32_t)(k == 1));
    v |= rw0.z & (0u - (uint32_t)(k == 2));
    v |= rw0.w & (0u - (uint32_t)(k == 3));
    v |= rw1.x & (0u - (uint32_t)(k == 4));
    v |= rw1.y & (0u - (uint32_t)(k == 5));
    v |= rw1.z & (0u - (uint32_t)(k == 6));
    v |= rw1.w & (0u - (uint32_t)(k == 7));
    return __uint_as_float(v);
  }

  // list entries this wavefront still owns
  __device__ __forceinline__ int remaining() const { return left + n_sh + n_rt; }
  // its next entry is a shared record, which needs no decision
  __device__ __forceinline__ bool shared_next() const { return n_sh > 0 || (left > 0 && run_shared); }

  // the routing record is unpacked when the first routed run comes up
  __device__ __forceinline__ void ensure_decided(const GemvParams &p) {
    if (decided) return;
    bool ok = true;
    if constexpr (IN == kRouteBoundary) {
      // (one wavefront per workgroup fetching for all eight through LDS was measured: no faster)
      ok = load_handover(p.b.handover + 8 * ((int)blockIdx.x % 8), p.b.hand_tag, p.b.spin_limit);
    }
    if constexpr (IN != kRouteEverywhere && IN != kRouteGiven) {
      slots = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)rd.y) |
              ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)rd.z) << 32);
      miss_mask = (uint32_t)__builtin_amdgcn_readfirstlane((int)rd.w);
    }
    if (!ok) {  // no record: use nothing
      slots = 0;
      miss_mask = 0;
      no_decision = true;
      *p.b.gave_up = 1u;
    }
    decided = true;
  }

  // One launch for everything (p.host_blob): whether a second walk is needed, over the experts that missed, and its start.
  // The first walk has gone over the others as a first pass does; the second one is dealt to the wavefronts as a second pass
  // deals its records, which has no shared ones, so that it adds the same in the same order.  (kRouteBoundary: a second pass
  // streams with one workgroup more, so there the order is another.)
  __device__ __forceinline__ bool any_missing(const GemvParams &p) {
    if (IN == kRouteGiven || p.host_blob == nullptr) return false;
    ensure_decided(p);
    return miss_mask != 0;
  }
  __device__ __forceinline__ void start_missing(int wave) {
    const Deal mine = deal<NW, STEP>(0, nr, wave);
    r = q0 + mine.first_rt;
    n_rt = mine.n_rt;
    n_sh = left = 0;
    missing_only = true;
  }

  // the wavefront's next run (there must be one): its shared records first, then its routed entries expert by expert
  __device__ __forceinline__ void start_run(const GemvParams &p) {
    if (n_sh > 0) {
      base = p.shared_blob;
      rows = p.shared_inter;
      next_at = sh_at;
      run_shared = true;
      left = n_sh;
      n_sh = 0;
      wt = 1.f;
      run_wanted = true;
      fill_blob = nullptr;
      return;
    }
    ensure_decided(p);
    const int I = p.inter;
    int seg = 0;  // r / I, of at most MOE_MAX_TOPK values
#pragma unroll
    for (int k = 1; k < MOE_MAX_TOPK; ++k) seg += r >= k * I;
    const int row = r - seg * I;
    run_shared = false;
    const int in_seg = (I - row + STEP - 1) / STEP;  // this wavefront's entries inside expert `seg` from here on
    left = min(in_seg, n_rt);
    n_rt -= left;
    r += left * STEP;
    base = p.slot_pool + (int64_t)((slots >> (8 * seg)) & 0xffu) * p.slot_bytes;
    rows = I;
    next_at = row;
    wt = pick_weight(seg);
    const bool missing = ((miss_mask >> seg) & 1u) != 0;
    run_wanted = missing == missing_only && !no_decision;
    fill_blob = nullptr;
    if (IN != kRouteGiven && run_wanted && missing && p.host_blob != nullptr) from_host_tier(p, seg);
  }

  // The run's expert was not resident: it is read from the host tier and put into its slot on the way (a rare case, kept out
  // of line of the others).
  __device__ __forceinline__ void from_host_tier(const GemvParams &p, int seg) {
    typedef const __attribute__((address_space(4))) int32_t *cint;
    typedef const __attribute__((address_space(4))) uint64_t *caddr;
    uint32_t expert;
    if constexpr (IN == kRouteBefore) {
      expert = (uint32_t)((cint)(reinterpret_cast<uintptr_t>(p.route)))[seg];
      static_assert(offsetof(moe_route_out_t, sel_expert) == 0, "record layout");
    } else {
      expert = (uint32_t)(experts >> (8 * seg)) & 0xffu;
    }
    fill_blob = const_cast<uint8_t *>(base);
    base = reinterpret_cast<const uint8_t *>(((caddr)(reinterpret_cast<uintptr_t>(p.host_blob)))[expert]);
  }

  // Whether selected expert `seg` missed and the workgroup owns some of its records: which (up to last), and base and
  // fill_blob set as for a run of it.  For what is put into the slot apart from the records.
  __device__ __forceinline__ bool missing_rows(const GemvParams &p, int seg, int &first, int &last) {
    const int I = p.inter;
    first = max(q0 - seg * I, 0);
    last = min(q0 + nr - seg * I, I);
    if (((miss_mask >> seg) & 1u) == 0 || first >= last) return false;
    base = p.slot_pool + (int64_t)((slots >> (8 * seg)) & 0xffu) * p.slot_bytes;
    from_host_tier(p, seg);
    return true;
  }

  // Move to this wavefront's next list entry and describe its record; whether there is one and the pass covers it.  The
  // caller issues the same loads in any case, from an empty resource where the answer is no (record_buffer): the number
  // of loads in flight then depends on nothing, and the compiler can wait for exactly the oldest record.  (Loads inside
  // branches make a wait cover all loads in flight: the wavefronts then did no arithmetic before the last of their first
  // records had arrived.)
  __device__ __forceinline__ bool step(const GemvParams &p) {
    if (left == 0) {
      if (n_sh + n_rt == 0) {
        fill = nullptr;
        return false;
      }
      start_run(p);
    }
    fill = fill_blob;
    at = next_at;
    next_at += STEP;
    --left;
    return run_wanted;
  }
};

// The 16 bytes at each lane's offset from one blob's tail to another's (offsets past the end: nothing is read or written)
__device__ __forceinline__ void copy_tail16(const uint8_t *from, uint8_t *to, int bytes, uint32_t off) {
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_amdgcn_raw_buffer_load_b128(record_buffer(from, bytes), off, 0, 0),
                                         record_buffer(to, bytes), off, 0, 0);
}

// Sum the wavefronts' private outputs through LDS (one barrier per pass) and write the workgroup's fp32
// partial row.  y holds, for load index c and v < VEC, column (c*64 + lane)*VEC + v at y[c*VEC + v].
// Slot (cv*64 + lane) of a wavefront's LDS row holds 4 columns with cv = c_in_pass*(VEC/4) + v4, so
// consecutive lanes hit consecutive 16-byte slots.  Wavefronts are added in index order (deterministic).
template <int NW, int VEC, int LPR>
__device__ __forceinline__ void reduce_and_store(const float *y, float *red, float *out, int tid, int lane, int wave) {
  constexpr int kRedCols = kRedFloats / NW;      // columns per LDS pass
  constexpr int CBF = kRedCols / (kWave * VEC);  // load indices c per pass (0 if a chunk exceeds a pass)
  constexpr int CB = CBF > 0 ? CBF : 1;
  static_assert(CBF > 0, "one 16-byte chunk per lane must fit an LDS pass");
  constexpr int PASSES = (LPR + CB - 1) / CB;
  constexpr int CPP = (LPR < CB ? LPR : CB);  // c per pass actually present
  constexpr int SLOTS = kRedCols / 4;         // float4 slots per wavefront row
  float4 *red4 = reinterpret_cast<float4 *>(red);
#pragma unroll
  for (int ps = 0; ps < PASSES; ++ps) {
    if (ps > 0) __syncthreads();
    float4 *dst = red4 + wave * SLOTS;
#pragma unroll
    for (int cc = 0; cc < CPP; ++cc)
#pragma unroll
      for (int v4 = 0; v4 < VEC / 4; ++v4) {
        const int j = (ps * CB + cc) * VEC + v4 * 4;
        dst[(cc * (VEC / 4) + v4) * kWave + lane] = make_float4(y[j], y[j + 1], y[j + 2], y[j + 3]);
      }
    __syncthreads();
    for (int sl = tid; sl < CPP * (VEC / 4) * kWave; sl += NW * kWave) {
      float4 acc = red4[sl];
#pragma unroll
      for (int w = 1; w < NW; ++w) {
        const float4 t = red4[w * SLOTS + sl];
        acc.x += t.x;
        acc.y += t.y;
        acc.z += t.z;
        acc.w += t.w;
      }
      const int cv = sl / kWave, ln = sl % kWave;
      const int c = ps * CB + cv / (VEC / 4), v4 = cv % (VEC / 4);
      *reinterpret_cast<float4 *>(out + (c * kWave + ln) * VEC + v4 * 4) = acc;
    }
  }
}

}  // namespace moe
