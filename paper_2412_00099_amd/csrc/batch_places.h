// What the host reads off the records of a routed batch before it uses any of them (plain C++, nothing from HIP).
#pragma once

#include "moe_cache.h"

namespace moe {

struct BatchPlaces {
  int of_slot[MOE_MAX_EXPERTS] = {};  // places that name the slot, of experts that were in it
  int misses = 0;

  // Counts n_tokens records; returns the first one that names an expert or a slot out of range (nothing of it is used), or
  // nullptr.
  const moe_route_out_t *count(const moe_route_out_t *rec, int n_tokens, int top_k, int n_experts, int capacity) {
    for (const moe_route_out_t *r = rec; r != rec + n_tokens; ++r)
      for (int k = 0; k < top_k; ++k) {
        const int e = r->sel_expert[k], s = r->sel_slot[k];
        if (e < 0 || e >= n_experts || s < 0 || s >= capacity || s >= MOE_MAX_EXPERTS) return r;
        if (r->miss[k]) ++misses;
        else ++of_slot[s];
      }
    return nullptr;
  }
};

}  // namespace moe
