// How a workgroup's list of records - ns shared ones, then nr routed ones - is dealt out to its NW wavefronts.  Plain C++
// (nothing from HIP), so that it can be looked at on the CPU.
//
// The order of the list is the order in which a wavefront adds its records up, and with it the rounding of y.  It is part of
// what callers see (the same inputs give the same bits from version to version), so it stays as it is.
#pragma once

#if defined(__HIPCC__)
#define MOE_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define MOE_HOST_DEVICE inline
#endif

namespace moe {

struct Deal {
  int first_sh, n_sh;  // the wavefront's shared records: first_sh, first_sh + STEP, ... (n_sh of them)
  int first_rt, n_rt;  // its routed ones, counted from the first routed record of the list
};

// STEP = NW: the wavefronts take list entries wave, wave + NW, ... so that the workgroup streams one contiguous span.
// STEP = 1: every wavefront takes one contiguous block of the whole list, so that its records stay inside one expert and, for
// int4, inside one scale group of 128 records as far as possible.  (Shared records dealt in turn there, so that every
// wavefront has one to load while the decision is on its way, change the order of the sums: fp32 outputs of one launch moved
// by 1e-5, those of a stack in bf16 by 1.3e-3, at the same distance from the sums in 64 bits.  37 MB at d = 2048, a quarter
// of it shared, timed by events when that launch had 216 registers: 17.9 us in turn, 18.25 like this; 141 now: 16.9.)
template <int NW, int STEP>
MOE_HOST_DEVICE Deal deal(int ns, int nr, int wave) {
  static_assert(STEP == NW || STEP == 1, "interleaved or blocked");
  Deal d;
  const int nl = ns + nr;
  int first;  // list index of the first routed one
  if constexpr (STEP == 1) {
    const int lb = wave * nl / NW, le = (wave + 1) * nl / NW;
    d.first_sh = lb;
    d.n_sh = (le < ns ? le : ns) - lb;
    if (d.n_sh < 0) d.n_sh = 0;
    first = lb > ns ? lb : ns;
    d.n_rt = le > first ? le - first : 0;
  } else {
    d.first_sh = wave;
    d.n_sh = wave < ns ? (ns - wave + NW - 1) / NW : 0;
    first = wave + d.n_sh * NW;
    d.n_rt = first < nl ? (nl - first + NW - 1) / NW : 0;
  }
  d.first_rt = first - ns;
  return d;
}

}  // namespace moe
