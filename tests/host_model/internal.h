// Lanes of a workgroup as fibers, for compiling the library's device headers
// with a host compiler (tests only).  A lane runs until it reaches a barrier
// or an operation over its wave; then another runs, in an order that changes
// from time to time.  Lanes of a wave that meet different operations, which a
// wave cannot do, end the program.
#pragma once

#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <ucontext.h>

#include <algorithm>
#include <functional>
#include <random>
#include <vector>

#define __device__
#define __host__
#define __forceinline__ inline

using std::max;
using std::min;

namespace lanes {
constexpr int kMost = 1024;

struct Wave {
  uint64_t in[64], out[64];
  int kind[64];
  uint64_t generation;
  int arrived;
};

inline int g_count, g_current, g_arrived;
inline uint64_t g_generation;
inline ucontext_t g_scheduler, g_lane[kMost];
inline bool g_ended[kMost];
inline Wave g_wave[kMost / 64];
inline std::vector<std::vector<char>> g_stack;
inline std::function<void()> g_body;
inline std::mt19937 g_order(1);

inline void pause() { swapcontext(&g_lane[g_current], &g_scheduler); }

inline void barrier() {
  const uint64_t g = g_generation;
  if (++g_arrived == g_count) {
    g_arrived = 0;
    ++g_generation;
    return;
  }
  while (g_generation == g) pause();
}

// every lane's value to all lanes of the wave
inline const uint64_t* exchange(int kind, uint64_t v, uint64_t* to) {
  Wave& w = g_wave[g_current / 64];
  const int l = g_current & 63;
  w.in[l] = v;
  w.kind[l] = kind;
  const uint64_t g = w.generation;
  if (++w.arrived == 64) {
    w.arrived = 0;
    for (int i = 0; i < 64; ++i)
      if (w.kind[i] != kind) {
        fprintf(stderr, "lanes of a wave in different operations: %d and %d\n", kind, w.kind[i]);
        abort();
      }
    memcpy(w.out, w.in, sizeof w.in);
    ++w.generation;
  } else {
    while (w.generation == g) pause();
  }
  memcpy(to, w.out, sizeof w.out);
  return to;
}

inline void entry() {
  g_body();
  g_ended[g_current] = true;
  swapcontext(&g_lane[g_current], &g_scheduler);
}

// body on `count` lanes, one workgroup
inline void run(int count, uint32_t seed, std::function<void()> body) {
  constexpr size_t kStack = 1 << 16;
  g_count = count;
  g_body = std::move(body);
  g_arrived = 0;
  g_order.seed(seed);
  for (Wave& w : g_wave) w.arrived = 0;
  while ((int)g_stack.size() < count) g_stack.emplace_back(kStack);
  std::vector<int> order(count);
  for (int i = 0; i < count; ++i) {
    order[i] = i;
    g_ended[i] = false;
    getcontext(&g_lane[i]);
    g_lane[i].uc_stack.ss_sp = g_stack[i].data();
    g_lane[i].uc_stack.ss_size = kStack;
    g_lane[i].uc_link = &g_scheduler;
    makecontext(&g_lane[i], entry, 0);
  }
  for (int left = count; left;) {
    if ((g_order() & 15) == 0) std::shuffle(order.begin(), order.end(), g_order);
    for (int i : order)
      if (!g_ended[i]) {
        g_current = i;
        swapcontext(&g_scheduler, &g_lane[i]);
        left -= g_ended[i];
      }
  }
}
}  // namespace lanes

struct ThreadIdx {
  struct X {
    operator uint32_t() const { return (uint32_t)lanes::g_current; }
  } x;
};
inline ThreadIdx threadIdx;
inline void __syncthreads() { lanes::barrier(); }

inline uint64_t __ballot(bool p) {
  uint64_t all[64], bits = 0;
  lanes::exchange(1, p, all);
  for (int i = 0; i < 64; ++i) bits |= (uint64_t)(all[i] != 0) << i;
  return bits;
}
template <class T>
inline T __shfl(T v, int from, int) {
  uint64_t all[64];
  return (T)lanes::exchange(2, (uint64_t)v, all)[from & 63];
}
template <class T>
inline T __shfl_xor(T v, int d, int w) {
  return __shfl(v, (lanes::g_current & 63) ^ d, w);
}
inline int __ffsll(unsigned long long v) { return __builtin_ffsll((long long)v); }
inline int __ffs(int v) { return __builtin_ffs(v); }
inline int __popcll(unsigned long long v) { return __builtin_popcountll(v); }
template <class T, class V>
inline T atomicOr(T* p, V v) {
  const T o = *p;
  *p = o | (T)v;
  return o;
}
template <class T, class V>
inline T atomicAnd(T* p, V v) {
  const T o = *p;
  *p = o & (T)v;
  return o;
}
template <class T, class V>
inline T atomicAdd(T* p, V v) {
  const T o = *p;
  *p = o + (T)v;
  return o;
}
template <class T, class V>
inline T atomicMax(T* p, V v) {
  const T o = *p;
  *p = max(o, (T)v);
  return o;
}
template <class T, class V>
inline T atomicMin(T* p, V v) {
  const T o = *p;
  *p = min(o, (T)v);
  return o;
}
template <class T, class A, class B>
inline T atomicCAS(T* p, A expected, B v) {
  const T o = *p;
  if (o == (T)expected) *p = (T)v;
  return o;
}

inline uint64_t lanes_below() { return (1ull << (lanes::g_current & 63)) - 1; }
#define __builtin_amdgcn_fence(order, scope)
#define __builtin_amdgcn_wave_barrier()      \
  do {                                       \
    uint64_t all_[64];                       \
    lanes::exchange(3, 0, all_);             \
  } while (0)
#define __builtin_amdgcn_readfirstlane(v) (v) /* callers pass the same value on every lane */
#define __builtin_amdgcn_readlane(v, l) __shfl((int)(v), (int)(l), 64)
#define __builtin_amdgcn_mbcnt_lo(m, a) \
  ((uint32_t)__builtin_popcount((uint32_t)(m) & (uint32_t)lanes_below()) + (a))
#define __builtin_amdgcn_mbcnt_hi(m, a) \
  ((uint32_t)__builtin_popcount((uint32_t)(m) & (uint32_t)(lanes_below() >> 32)) + (a))

namespace bisim {
constexpr uint32_t kNone = 0xFFFFFFFFu;
constexpr int kWave = 64;
inline uint32_t lane() { return (uint32_t)lanes::g_current & 63u; }
inline uint32_t wave_incl_scan_u32(uint32_t v) {
  uint64_t all[64];
  lanes::exchange(4, v, all);
  uint32_t sum = 0;
  for (uint32_t i = 0; i <= lane(); ++i) sum += (uint32_t)all[i];
  return sum;
}
inline uint32_t wave_min_u32(uint32_t v) {
  uint64_t all[64];
  lanes::exchange(5, v, all);
  for (int i = 0; i < 64; ++i) v = min(v, (uint32_t)all[i]);
  return v;
}
inline bool test_bit(const uint64_t* words, uint32_t i) { return (words[i >> 6] >> (i & 63)) & 1ull; }
}  // namespace bisim
