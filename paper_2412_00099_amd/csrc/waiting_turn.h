// Whose launches may wait inside a kernel (plain C++, nothing from HIP).
//
// A launch that carries the layer boundary in its first workgroup (kRouteBoundary) has its other workgroups wait for that one,
// each on the compute unit that it occupies.  One such launch always gets on: its first workgroup is the first to be placed.
// Of two that share the device this is not sure.  Workgroups are dealt to 8 dies and to the parts of each, which place them
// independently of each other, so that some of the one launch and some of the other can hold all places that the two first
// workgroups still need, and all of them wait.  (Contexts whose host does not wait are what it takes: three decoders driven
// in turn with several tokens in flight each ended once with a wait that ran out.)
//
// So on a device at most one context at a time has launches of this kind whose decision is not known yet; a context that does
// not have the turn runs the boundary ahead of its expert launch, where nothing waits.  The decision is seen in the word that
// the first workgroup stores into mapped host memory: asking costs one load, no call.  (Several processes on one device do not
// know of each other: there the wait is bounded and its end an error, and MOE_FUSE_BOUNDARY=0 keeps it from happening.)
#pragma once

#include <stdint.h>

#include <mutex>

namespace moe {

class WaitingTurn {
 public:
  // Whether `who` may enqueue such a launch now; if so it has the turn until the low half of *note has reached seq (the word
  // counts up: a later step of the same context may have stored more already).  All launches of one owner are on one stream.
  bool take(const void *who, const uint64_t *note, uint32_t seq) {
    std::lock_guard<std::mutex> lock(mu_);
    if (owner_ != nullptr && owner_ != who && !known()) return false;
    owner_ = who;
    note_ = note;
    seq_ = seq;
    return true;
  }
  // nothing of `who` is on the device any more (its stream has been waited for, or its launch failed)
  void give_back(const void *who) {
    std::lock_guard<std::mutex> lock(mu_);
    if (owner_ == who) owner_ = nullptr;
  }

 private:
  bool known() const { return (int32_t)((uint32_t)__atomic_load_n(note_, __ATOMIC_ACQUIRE) - seq_) >= 0; }
  std::mutex mu_;
  const void *owner_ = nullptr;
  const uint64_t *note_ = nullptr;
  uint32_t seq_ = 0;
};

}  // namespace moe
