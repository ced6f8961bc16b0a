// Transitions grouped by target, spread over waves by transition.
#pragma once

#include <stdint.h>

#include "internal.h"

namespace bisim {

// the last t of [lo, hi] with ptr[t] <= e (ptr non-decreasing, ptr[lo] <= e)
__device__ __forceinline__ uint32_t last_not_above(const uint32_t* __restrict__ ptr, uint32_t lo,
                                                   uint32_t hi, uint32_t e) {
  while (lo < hi) {
    const uint32_t mid = hi - (hi - lo) / 2;
    if (ptr[mid] <= e) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// f(t, e) for every transition e and its target t, of transitions grouped by
// target, by wave `wave` of `waves`: a run of kTransRun consecutive transitions
// at a time, whatever the in-degrees are.  (A thread per target walked all the
// transitions of a hub: the transitions by source of an LTS with a sink of 1M
// in-transitions took 396 ms, now below 1.)
constexpr uint32_t kTransRun = 8 * kWave;
template <class F>
__device__ __forceinline__ void each_in_transition(uint32_t n, const uint32_t* __restrict__ in_ptr,
                                                   uint32_t wave, uint32_t waves, const F& f) {
  const uint64_t m = n ? in_ptr[n] : 0u;
  for (uint64_t r = (uint64_t)wave * kTransRun; r < m; r += (uint64_t)waves * kTransRun) {
    const uint32_t first = (uint32_t)r, last = (uint32_t)((m < r + kTransRun ? m : r + kTransRun) - 1);
    uint32_t lo = last_not_above(in_ptr, 0, n - 1, first);
    const uint32_t hi = last_not_above(in_ptr, lo, n - 1, last);
    for (uint32_t i = 0; i <= last - first; i += kWave) {
      const bool on = i + lane() <= last - first;
      const uint32_t e = on ? first + i + lane() : last;
      const uint32_t t = last_not_above(in_ptr, lo, hi, e);
      if (on) f(t, e);
      lo = (uint32_t)__shfl((int)t, kWave - 1, kWave);
    }
  }
}

}  // namespace bisim
