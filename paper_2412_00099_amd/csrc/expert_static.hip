// moe_expert_forward_static: the expert computation of one layer-token (paper Eq. 1) for callers that may not
// allocate - code under HIP graph capture, tight serving loops.  It runs the same kernels as moe_expert_forward.  The
// selection travels in the launch's arguments (a launch that wrote it to memory first cost 1.7 us and a dependent read:
// 6 x 1000 int8 records of d = 2048, 15.2 against 12.9 us a call); what moe_expert_forward keeps in memory the context allocated, the
// fp32 partial rows, one per workgroup, lives here in a fixed device array that is part of the library's code object.
#include <mutex>

#include "common.h"

namespace moe {
namespace {

constexpr int kStaticMaxHidden = 4096;  // every workload shape; bounds the scratch array
constexpr int kStaticMaxGrid = 256;     // workgroups = partial rows
constexpr size_t kScratchBytes = sizeof(float) * (size_t)kStaticMaxGrid * kStaticMaxHidden;

// partial rows: 4 MiB per GPU, held until the process ends
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

constexpr int kMaxDevices = 64;
struct PerDevice {
  void *ptr = nullptr;  // device address of `scratch` on this GPU (each GPU has its own copy of the array)
  int cus = 0;
};
PerDevice g_dev[kMaxDevices];
std::mutex g_mu;

}  // namespace

// Once per device, with that device current: the device address of the scratch array and the number of compute
// units.  The array's name is a host-side handle, not an address; only the address obtained here may be given to
// kernels.  Allocates nothing.
hipError_t static_scratch_setup(int dev, void **ptr, int *cus) {
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_mu);
  PerDevice &d = g_dev[dev];
  if (d.ptr == nullptr) {
    void *p = nullptr;
    hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (p == nullptr) return hipErrorInvalidSymbol;
    int n = 0;
    e = hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return e;
    d.cus = n;
    d.ptr = p;
  }
  if (ptr) *ptr = d.ptr;
  if (cus) *cus = d.cus;
  return hipSuccess;
}

hipError_t launch_expert_forward_static(int weight_fmt, int act_fmt, int hidden, int inter, int shared_inter, int top_k,
                                        const void *slot_pool, int64_t slot_bytes, const void *shared_blob,
                                        const int32_t *sel_slot, const float *sel_weight, const void *x, void *y,
                                        hipStream_t s) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  void *base = nullptr;
  int cus = 0;
  e = static_scratch_setup(dev, &base, &cus);
  if (e != hipSuccess) return e;
  float *partial = static_cast<float *>(base);
  GemvPlan plan = gemv_plan(cus, top_k * inter + shared_inter, weight_fmt, act_fmt, hidden);
  if (plan.grid > kStaticMaxGrid) plan.grid = kStaticMaxGrid;
  GemvParams p{};
  p.slot_pool = static_cast<const uint8_t *>(slot_pool);
  p.shared_blob = shared_inter > 0 ? static_cast<const uint8_t *>(shared_blob) : nullptr;
  p.x = x;
  p.partial = partial;
  p.hidden = hidden;
  p.inter = inter;
  p.shared_inter = shared_inter;
  p.top_k = top_k;
  p.act_fmt = act_fmt;
  p.slot_bytes = slot_bytes;
  p.pass = 0;
  p.row_offset = 0;
  p.route_in = kRouteGiven;
  for (int k = 0; k < top_k; ++k) {
    p.given_slots |= (uint64_t)((uint32_t)sel_slot[k] & 0xffu) << (8 * k);
    p.given_weight[k] = sel_weight[k];
  }
  e = launch_expert_gemv(p, weight_fmt, plan, s);
  if (e != hipSuccess) return e;
  return launch_partial_reduce(partial, plan.grid, nullptr, y, hidden, act_fmt, s);
}

int static_max_hidden() { return kStaticMaxHidden; }

}  // namespace moe
