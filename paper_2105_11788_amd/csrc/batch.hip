// Batched refinement of many independent LTSs in one launch.
//
// Loading: the instances are shifted into one id space (instance k's states
// start at n_off[k]; its initial blocks stay separate) and preprocessed
// together by the single-instance loader: the preprocessing is per state and
// per transition, and no block ever spans two instances, so the result is
// every instance's own preprocessing side by side.
//
// Refinement: one launch of a kernel whose workgroups claim instances from a
// device queue (largest first).  A workgroup carries out the whole run of its
// instance by rounds (rounds_dev.h): the iterations that split nothing are
// decided many at a time, and every instance gets the same splitter sequence
// and #It as a single-instance run.  The label bitmaps, the table of marks
// and the tables of a split live in LDS; the member lists stay in global
// memory (the L2, for all but the largest instances).  The LDS budget and the
// grid are chosen by an autotuner that times candidate configurations and
// caches the winner per device and batch shape.  The queue reset and the
// launch are captured once into a hipGraph and replayed.
#include <sys/stat.h>

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <new>
#include <string>
#include <vector>

#include "internal.h"
#include "rounds_dev.h"

struct bisim_batch {
  int32_t count = 0;
  int64_t N = 0, M = 0;
  uint32_t n_max = 0;  // states of the largest instance
  int32_t Kmax = 1;
  hipStream_t stream = nullptr;
  hipStream_t own_stream = nullptr;
  int device = 0, num_cu = 0;
  int lds_max = 0;
  bisim_lts* u = nullptr;  // the preprocessed union
  bisim::Chunks mem;       // the device arrays below
  std::vector<int64_t> n_off;
  uint32_t* n_off_d = nullptr;  // [count+1]
  uint32_t* bw_off_d = nullptr; // [count+1] bitmap word offsets
  int32_t* order_d = nullptr;   // instance ids, largest first
  int mask64 = 1;               // 64-bit mark words (else 32-bit)
  // per-state arrays of all instances
  int32_t* blk = nullptr;
  uint64_t* mw = nullptr;
  uint64_t* nlb = nullptr;
  uint64_t *ub = nullptr, *qb = nullptr, *qs = nullptr;
  int32_t* tl = nullptr;
  int32_t* sl = nullptr;
  int32_t *perm = nullptr, *pos = nullptr, *bs = nullptr, *be = nullptr, *cnt = nullptr,
          *fc = nullptr, *gc = nullptr, *tmp = nullptr, *rk = nullptr, *fi = nullptr,
          *ob = nullptr, *ltl = nullptr, *tlb = nullptr,
          *llo = nullptr, *lsz = nullptr;
  uint64_t *us = nullptr, *tmp64 = nullptr, *pin = nullptr;
  uint8_t* trk = nullptr;
  uint32_t* iters_d = nullptr;  // [count]
  uint32_t* ctl_d = nullptr;    // [0] queue head, [1] error
  bisim::RoundsArgs<uint64_t>* args_d = nullptr;  // [count]
  unsigned long long* work_d = nullptr;  // [16] work totals per tier
  // options / tuning
  int opt_wg = 0, opt_grid = 0, opt_lds = 0, opt_retune = 0;
  int wg = 0, grid = 0, lds_bytes = 0;
  bool tuned = false;
  hipGraphExec_t gexec = nullptr;
  int g_wg = -1, g_grid = -1, g_lds = -1;
  int32_t* g_out = nullptr;
  hipEvent_t ev0 = nullptr, ev1 = nullptr;
  double t_pre_ms = 0, t_alg_ms = 0;
  int64_t lds_inst = 0, glob_inst = 0;
};

namespace bisim {
bisim_status lts_create_union(int32_t n, int64_t m, int32_t K, const int32_t* src,
                              const int32_t* lab, const int32_t* dst, const int32_t* init,
                              hipStream_t stream, bisim_lts** out);
void lts_destroy(bisim_lts* h);

namespace {
constexpr int kT = 256;

struct BArgs {
  int32_t count;
  const uint32_t* __restrict__ n_off;
  const uint32_t* __restrict__ bw_off;
  const int32_t* __restrict__ order;
  const int32_t* __restrict__ pre_block;
  const uint32_t* __restrict__ in_ptr;
  const int32_t* __restrict__ in_src;
  const int32_t* __restrict__ in_ord;
  int32_t* blk;
  void* mw;
  uint64_t* nlb;
  uint64_t *ub, *qb, *qs;
  int32_t* tl;
  int32_t* sl;
  int32_t *perm, *pos, *bs, *be, *cnt, *fc, *gc, *tmp, *rk, *fi, *ob, *ltl, *tlb, *llo,
      *lsz;
  uint64_t *us, *tmp64, *pin;
  uint32_t* out_ptr;  // transitions by source
  int32_t *out_dst, *out_ord;
  uint8_t* trk;
  int32_t* out;
  uint32_t* iters;
  uint32_t* ctl;
  unsigned long long* work;  // [2][8] totals per tier (see bisim_batch_stats)
  uint32_t lds_bytes;
};

// An instance of up to this need counts as small in the statistics: its block
// ids, marks, bids and bitmaps are within the LDS budget.
template <class MaskT>
__host__ __device__ inline uint64_t lds_need(uint32_t n) {
  const uint64_t nw = (n + 63u) / 64u;
  return 8ull * 3 * nw + 8ull * n + ((sizeof(MaskT) * (uint64_t)n + 7) & ~7ull) + 4ull * n;
}

// Workgroup sizes.  A launch ends with its slowest instance, whose rounds
// spread over more waves at 1024 threads (one workgroup per CU with the whole
// LDS); where instances are many and tiny, two or more workgroups of 256 per
// CU are ahead.  At 1024 / 512 / 256 threads: 256 instances of up to 40k
// states 88 / 92 / 112 ms, 48 of up to 200k 461 / 500 / 640, 2048 of up to 2k
// 4.6 / 4.4 / 4.5, 8192 of up to 200 2.0 / 1.6 / 1.5.  The autotuner times
// both; 256 is what the option names.
constexpr int kBatchWG = 1024, kBatchWGOption = 256;

template <int WG>
struct Shared {
  RoundsShared<WG> r;
  uint32_t job;
};

// kBm: the label bitmaps of every instance fit the LDS budget beside the
// tables (else they stay in global memory for all of them: a second copy of
// the loop in one kernel spills registers).
template <class MaskT, int WG, bool kBm>
__global__ void __launch_bounds__(WG) k_batch(BArgs a,
                                                    const RoundsArgs<MaskT>* __restrict__ args) {
  extern __shared__ uint64_t lds[];
  __shared__ Shared<WG> sh;
  char* base = reinterpret_cast<char*>(lds);
  for (;;) {
    if (threadIdx.x == 0) sh.job = atomicAdd(&a.ctl[0], 1u);
    if (threadIdx.x < kWorkTotals) sh.r.work[threadIdx.x] = 0;
    __syncthreads();
    // the instance's pointers are read as scalars where they are needed
    // (computed here they spilled: 60-120 bytes per thread)
    const uint32_t job = uniform_u32(sh.job);
    if (job >= (uint32_t)a.count) break;
    const uint32_t k = uniform_u32((uint32_t)a.order[job]);
    const RoundsArgs<MaskT> g = args[k];
    const uint32_t s0 = g.s0, n = g.n;
    uint32_t rc = kRoundsBad, none = 0;
    RoundsResume resume;
    resume.may_track = true;
    if (rounds_setup<MaskT, WG>(g, sh.r, a.pre_block + s0, true))
      rc = rounds_loop<MaskT, WG, kBm, kEither>(g, sh.r, base, a.lds_bytes, 0, resume, none);
    if (rc == kRoundsDone && sh.r.it > g.iter_cap) rc = kRoundsCap;
    for (uint32_t s = threadIdx.x; s < n; s += WG) a.out[s0 + s] = g.blk[s];
    __syncthreads();
    if (threadIdx.x == 0) {
      const uint32_t its = sh.r.it + 1;  // with the final pass
      a.iters[k] = its;
      if (rc == kRoundsCap) atomicOr(&a.ctl[1], 1u);
      if (rc == kRoundsBad) atomicOr(&a.ctl[1], 2u);
      const unsigned long long* x = sh.r.work;
      if (lds_need<MaskT>(n) <= a.lds_bytes) {
        const unsigned long long v[8] = {its, x[0], x[1], x[2], 0, x[5], 0, 1};
#pragma unroll
        for (int i = 0; i < 8; ++i) atomicAdd(&a.work[i], v[i]);
      } else {
        const unsigned long long v[8] = {its, x[0], x[1], x[2], x[3], x[4], x[5], x[6]};
#pragma unroll
        for (int i = 0; i < 8; ++i) atomicAdd(&a.work[8 + i], v[i]);
      }
    }
    __syncthreads();
  }
}

// The loop's arguments of every instance, once per batch (the mark words of
// instances with 32-bit marks take the first half of their 64-bit ones).
__global__ void k_batch_args(BArgs a, RoundsArgs<uint64_t>* __restrict__ out) {
  const int32_t k = (int32_t)(blockIdx.x * blockDim.x + threadIdx.x);
  if (k >= a.count) return;
  const uint32_t s0 = a.n_off[k], n = a.n_off[k + 1] - s0;
  const uint32_t b0 = a.bw_off[k];
  RoundsArgs<uint64_t> g{};
  g.n = n;
  g.s0 = s0;
  g.iter_cap = 3u * n + 1u;
  g.in_ptr = a.in_ptr + s0;
  g.in_src = a.in_src;
  g.in_ord = a.in_ord;
  g.blk = a.blk + s0;
  g.perm = a.perm + s0;
  g.pos = a.pos + s0;
  g.bs = a.bs + s0;
  g.be = a.be + s0;
  g.pin = a.pin + s0;
  g.mw = reinterpret_cast<uint64_t*>(a.mw) + s0;
  g.cnt = a.cnt + s0;
  g.fc = a.fc + s0;
  g.gc = a.gc + s0;
  g.nlb = a.nlb + s0;
  g.tmp64 = a.tmp64 + s0;
  g.ts = a.tl + s0;
  g.tb = a.tlb + s0;
  g.lb = a.ltl + s0;
  g.llo = a.llo + s0;
  g.lsz = a.lsz + s0;
  g.ss = a.sl + s0;
  g.sbk = a.ob + s0;
  g.sr = a.rk + s0;
  g.sfi = a.fi + s0;
  g.sps = a.tmp + s0;
  g.ub = a.ub + b0;
  g.qb = a.qb + b0;
  g.us = a.us + b0;
  g.qs = a.qs + b0;
  g.out_ptr = a.out_ptr ? a.out_ptr + s0 : nullptr;
  g.out_dst = a.out_dst;
  g.out_ord = a.out_ord;
  g.out_cur = nullptr;
  g.trk = a.trk + s0;
  g.mean_deg = n ? (a.in_ptr[s0 + n] - a.in_ptr[s0] + n - 1) / n : 1u;
  out[k] = g;
}

__global__ void k_reset_queue(uint32_t* ctl, unsigned long long* work) {
  if (blockIdx.x == 0 && threadIdx.x < 16) work[threadIdx.x] = 0;
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    ctl[0] = 0;
    ctl[1] = 0;
  }
}

// shift instance-local ids into the union's id space, validating ranges
__device__ __forceinline__ int32_t find_instance(const uint32_t* off, int32_t count, uint64_t x) {
  int32_t lo = 0, hi = count;  // off[lo] <= x < off[hi]
  while (hi - lo > 1) {
    const int32_t mid = (lo + hi) >> 1;
    if ((uint64_t)off[mid] <= x) lo = mid;
    else hi = mid;
  }
  return lo;
}

__global__ void k_globalize(int32_t count, const uint32_t* __restrict__ n_off,
                            const uint32_t* __restrict__ m_off, const int32_t* __restrict__ K,
                            const int32_t* __restrict__ src, const int32_t* __restrict__ lab,
                            const int32_t* __restrict__ dst, const int32_t* __restrict__ init,
                            uint64_t M, uint64_t N, int32_t* __restrict__ gsrc,
                            int32_t* __restrict__ gdst, int32_t* __restrict__ ginit,
                            uint32_t* err) {
  bool bad = false;
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < M; i += stride) {
    const int32_t k = find_instance(m_off, count, i);
    const uint32_t nk = n_off[k + 1] - n_off[k];
    const int32_t s = src[i], d = dst[i], l = lab[i];
    bad |= (uint32_t)s >= nk || (uint32_t)d >= nk || (uint32_t)l >= (uint32_t)K[k];
    gsrc[i] = (int32_t)n_off[k] + ((uint32_t)s < nk ? s : 0);
    gdst[i] = (int32_t)n_off[k] + ((uint32_t)d < nk ? d : 0);
  }
  for (uint64_t s = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; s < N; s += stride) {
    const int32_t k = find_instance(n_off, count, s);
    const uint32_t nk = n_off[k + 1] - n_off[k];
    int32_t v = 0;
    if (init) {
      v = init[s];
      bad |= (uint32_t)v >= nk;
      if ((uint32_t)v >= nk) v = 0;
    }
    ginit[s] = (int32_t)n_off[k] + v;
  }
  if (bad) atomicOr(err, 1u);
}

// device memory from `mem` (an allocation of its own for each of the 40 arrays
// was most of the load of a small batch)
template <class T>
bisim_status dmalloc(Chunks& mem, hipStream_t s, T** p, size_t count) {
  *p = nullptr;
  const size_t bytes = sizeof(T) * (count ? count : 1);
  const hipError_t e = mem.alloc((void**)p, bytes, s);
  if (e != hipSuccess) {
    set_error("device allocation of %zu bytes failed: %s", bytes, hipGetErrorString(e));
    return BISIM_E_NOMEM;
  }
  return BISIM_OK;
}

void free_batch(bisim_batch* b) {
  if (!b) return;
  if (b->stream) (void)hipStreamSynchronize(b->stream);
  if (b->gexec) (void)hipGraphExecDestroy(b->gexec);
  b->mem.release(b->stream);
  if (b->stream) (void)hipStreamSynchronize(b->stream);
  if (b->u) lts_destroy(b->u);
  if (b->ev0) (void)hipEventDestroy(b->ev0);
  if (b->ev1) (void)hipEventDestroy(b->ev1);
  if (b->own_stream) (void)hipStreamDestroy(b->own_stream);
  delete b;
}

BArgs make_args(bisim_batch* b, int32_t* out) {
  BArgs a{};
  a.count = b->count;
  a.n_off = b->n_off_d;
  a.bw_off = b->bw_off_d;
  a.order = b->order_d;
  a.pre_block = b->u->pre_block;
  a.in_ptr = b->u->in_ptr;
  a.in_src = b->u->in_src;
  a.in_ord = b->u->in_ord;
  a.blk = b->blk;
  a.mw = b->mw;
  a.nlb = b->nlb;
  a.ub = b->ub;
  a.qb = b->qb;
  a.qs = b->qs;
  a.tl = b->tl;
  a.sl = b->sl;
  a.perm = b->perm;
  a.pos = b->pos;
  a.bs = b->bs;
  a.be = b->be;
  a.cnt = b->cnt;
  a.fc = b->fc;
  a.gc = b->gc;
  a.tmp = b->tmp;
  a.rk = b->rk;
  a.fi = b->fi;
  a.ob = b->ob;
  a.ltl = b->ltl;
  a.tlb = b->tlb;
  a.llo = b->llo;
  a.lsz = b->lsz;
  a.tmp64 = b->tmp64;
  a.pin = b->pin;
  a.us = b->us;
  a.out_ptr = b->u->lists.out_ptr;
  a.out_dst = b->u->lists.out_dst;
  a.out_ord = b->u->lists.out_ord;
  a.trk = b->trk;
  a.out = out;
  a.iters = b->iters_d;
  a.ctl = b->ctl_d;
  a.work = b->work_d;
  a.lds_bytes = (uint32_t)b->lds_bytes;
  return a;
}

// the kernel of a configuration: workgroup size, mark word and whether the
// largest instance's label bitmaps fit the budget
template <int WG>
const void* kernel_for(const bisim_batch* b, int lds) {
  const bool bm = rounds_bitmap_bytes(b->n_max) + split_bytes<WG>() +
                      table_bytes<uint64_t>(256) <= (uint32_t)lds;
  if (b->mask64)
    return bm ? (const void*)k_batch<uint64_t, WG, true> : (const void*)k_batch<uint64_t, WG, false>;
  return bm ? (const void*)k_batch<uint32_t, WG, true> : (const void*)k_batch<uint32_t, WG, false>;
}
const void* kernel_of(const bisim_batch* b, int wg, int lds) {
  return wg == kBatchWG ? kernel_for<kBatchWG>(b, lds) : kernel_for<kBatchWGOption>(b, lds);
}

bisim_status launch_once(bisim_batch* b, int32_t* out, int wg, int grid, int lds) {
  BArgs a = make_args(b, out);
  a.lds_bytes = (uint32_t)lds;
  hipLaunchKernelGGL(k_reset_queue, dim3(1), dim3(64), 0, b->stream, b->ctl_d, b->work_d);
  if (wg != kBatchWG && wg != kBatchWGOption) {
    set_error("batched kernel: workgroup size %d is not built", wg);
    return BISIM_E_INVALID;
  }
  const void* inst = b->args_d;  // (one layout for both mark words)
  void* args[] = {&a, &inst};
  const void* f = kernel_of(b, wg, lds);
  BISIM_TRY_HIP(hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, b->lds_max));
  BISIM_TRY_HIP(hipLaunchKernel(f, dim3(grid), dim3(wg), args, lds, b->stream));
  BISIM_TRY_HIP(hipGetLastError());
  return BISIM_OK;
}

int max_resident(bisim_batch* b, int wg, int lds) {
  int per_cu = 0;
  if (wg != kBatchWG && wg != kBatchWGOption) return 0;
  const void* f = kernel_of(b, wg, lds);
  (void)hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, b->lds_max);
  hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, f, wg, lds);
  if (e != hipSuccess || per_cu < 1) return 0;
  return per_cu * b->num_cu;
}

std::string tune_key(bisim_batch* b) {
  hipDeviceProp_t p;
  std::string arch = "gpu";
  if (hipGetDeviceProperties(&p, b->device) == hipSuccess) arch = p.gcnArchName;
  for (char& c : arch)
    if (c == ' ' || c == ':') c = '_';
  int lc = 0, ln = 0, lm = 0;
  for (int64_t v = b->count; v > 1; v >>= 1) ++lc;
  for (int64_t v = b->N; v > 1; v >>= 1) ++ln;
  for (int64_t v = b->M; v > 1; v >>= 1) ++lm;
  char buf[256];
  snprintf(buf, sizeof buf, "rounds_%s_cu%d_c%d_n%d_m%d_k%d", arch.c_str(), b->num_cu, lc, ln, lm,
           b->mask64);
  return buf;
}

std::string tune_path() {
  const char* e = getenv("BISIM_TUNE_CACHE");
  if (e && *e) return e;
  const char* h = getenv("HOME");
  return std::string(h && *h ? h : "/tmp") + "/.cache/bisim_tune.txt";
}

bool tune_lookup(const std::string& key, int* wg, int* grid, int* lds) {
  FILE* f = fopen(tune_path().c_str(), "r");
  if (!f) return false;
  char k[256];
  int a, g, l;
  float ms;
  bool found = false;
  while (fscanf(f, "%255s %d %d %d %f", k, &a, &g, &l, &ms) == 5)
    if (key == k) {
      *wg = a;
      *grid = g;
      *lds = l;
      found = true;
    }
  fclose(f);
  return found;
}

void tune_store(const std::string& key, int wg, int grid, int lds, float ms) {
  std::string path = tune_path();
  std::string dir = path.substr(0, path.find_last_of('/'));
  if (!dir.empty()) {
    for (size_t i = 1; i <= dir.size(); ++i)
      if (i == dir.size() || dir[i] == '/') (void)mkdir(dir.substr(0, i).c_str(), 0755);
  }
  FILE* f = fopen(path.c_str(), "a");
  if (!f) return;
  fprintf(f, "%s %d %d %d %.4f\n", key.c_str(), wg, grid, lds, ms);
  fclose(f);
}

// Autotuner: time each candidate (workgroup size, LDS budget, grid = as many
// workgroups as stay resident) on the batch itself and keep the fastest.
bisim_status autotune(bisim_batch* b, int32_t* out) {
  const struct {
    int wg, lds;
  } cands[] = {{kBatchWG, b->lds_max},
               {kBatchWGOption, b->lds_max / 2},
               {kBatchWGOption, b->lds_max / 4}};
  float best = 1e30f;
  int bw = 0, bg = 0, bl = 0;
  for (const auto& c : cands) {
    const int wg = c.wg, lds = c.lds & ~63;
    const int grid = max_resident(b, wg, lds);
    if (grid < 1) continue;
    BISIM_TRY_HIP(hipEventRecord(b->ev0, b->stream));
    BISIM_TRY(launch_once(b, out, wg, grid, lds));
    BISIM_TRY_HIP(hipEventRecord(b->ev1, b->stream));
    BISIM_TRY_HIP(hipEventSynchronize(b->ev1));
    float ms = 0;
    BISIM_TRY_HIP(hipEventElapsedTime(&ms, b->ev0, b->ev1));
    if (ms < best) {
      best = ms;
      bw = wg;
      bg = grid;
      bl = lds;
    }
  }
  if (!bw) {
    set_error("batched kernel: no launch configuration is resident");
    return BISIM_E_DEVICE;
  }
  b->wg = bw;
  b->grid = bg;
  b->lds_bytes = bl;
  tune_store(tune_key(b), bw, bg, bl, best);
  return BISIM_OK;
}
}  // namespace
}  // namespace bisim

using namespace bisim;

extern "C" {

bisim_status lts_batch_load(int32_t count, const int64_t* n_off, const int64_t* m_off,
                            const int32_t* src, const int32_t* label, const int32_t* dst,
                            const int32_t* num_actions, const int32_t* init_partition,
                            void* hip_stream, bisim_batch** out) {
  if (!out) {
    set_error("lts_batch_load: out is NULL");
    return BISIM_E_INVALID;
  }
  *out = nullptr;
  if (count < 1 || !n_off || !m_off || !num_actions) {
    set_error("lts_batch_load: need count >= 1 and host offset/action arrays");
    return BISIM_E_INVALID;
  }
  if (n_off[0] != 0 || m_off[0] != 0) {
    set_error("lts_batch_load: offsets must start at 0");
    return BISIM_E_INVALID;
  }
  int32_t Kmax = 1;
  int64_t n_max = 0;
  for (int32_t k = 0; k < count; ++k) {
    if (n_off[k + 1] < n_off[k] || m_off[k + 1] < m_off[k] || num_actions[k] < 1) {
      set_error("lts_batch_load: offsets must be non-decreasing and num_actions >= 1");
      return BISIM_E_INVALID;
    }
    Kmax = std::max(Kmax, num_actions[k]);
    n_max = std::max(n_max, n_off[k + 1] - n_off[k]);
  }
  const int64_t N = n_off[count], M = m_off[count];
  if (N >= 0x7FFFFFFF || M >= 0xFFFFFFFFll) {
    set_error("lts_batch_load: totals beyond 2^31-1 states / 2^32-1 transitions");
    return BISIM_E_UNSUPPORTED;
  }
  if (M > 0 && (!src || !label || !dst)) {
    set_error("lts_batch_load: NULL transition array");
    return BISIM_E_INVALID;
  }
  bisim_batch* b = new (std::nothrow) bisim_batch;
  if (!b) return BISIM_E_NOMEM;
  b->count = count;
  b->N = N;
  b->M = M;
  b->Kmax = Kmax;
  b->n_max = (uint32_t)n_max;
  b->n_off.assign(n_off, n_off + count + 1);
  bisim_status st = BISIM_OK;
  int32_t *gsrc = nullptr, *gdst = nullptr, *ginit = nullptr, *Kd = nullptr;
  uint32_t *m_off_d = nullptr, *err = nullptr;
  Chunks tmp;  // temporaries of loading
  do {
    hipError_t e = hipGetDevice(&b->device);
    if (e == hipSuccess)
      e = hipDeviceGetAttribute(&b->num_cu, hipDeviceAttributeMultiprocessorCount, b->device);
    if (e == hipSuccess)
      e = hipDeviceGetAttribute(&b->lds_max, hipDeviceAttributeMaxSharedMemoryPerBlock, b->device);
    if (e == hipSuccess) e = hipEventCreate(&b->ev0);
    if (e == hipSuccess) e = hipEventCreate(&b->ev1);
    if (e == hipSuccess && !hip_stream) e = hipStreamCreateWithFlags(&b->own_stream, hipStreamNonBlocking);
    if (e != hipSuccess) {
      set_error("lts_batch_load: %s", hipGetErrorString(e));
      st = BISIM_E_DEVICE;
      break;
    }
    b->lds_max = (b->lds_max - (int)sizeof(Shared<kBatchWG>) - 64) & ~63;
    b->stream = hip_stream ? (hipStream_t)hip_stream : b->own_stream;
    hipStream_t s = b->stream;
    if (hipEventRecord(b->ev0, s) != hipSuccess) { st = BISIM_E_DEVICE; break; }
    std::vector<uint32_t> no(count + 1), mo(count + 1), bo(count + 1);
    bo[0] = 0;
    for (int32_t k = 0; k <= count; ++k) {
      no[k] = (uint32_t)n_off[k];
      mo[k] = (uint32_t)m_off[k];
      if (k < count) bo[k + 1] = bo[k] + (uint32_t)((n_off[k + 1] - n_off[k] + 63) / 64);
    }
    std::vector<int32_t> order(count);
    for (int32_t k = 0; k < count; ++k) order[k] = k;
    std::stable_sort(order.begin(), order.end(), [&](int32_t x, int32_t y) {
      return n_off[x + 1] - n_off[x] > n_off[y + 1] - n_off[y];
    });
    tmp.reserve(8 * (size_t)M + 4 * (size_t)N + 8 * (size_t)count + 8 * 256, s);
    if ((st = dmalloc(b->mem, s, &b->n_off_d, count + 1)) ||
        (st = dmalloc(b->mem, s, &b->bw_off_d, count + 1)) ||
        (st = dmalloc(b->mem, s, &b->order_d, count)) ||
        (st = dmalloc(tmp, s, &m_off_d, count + 1)) || (st = dmalloc(tmp, s, &Kd, count)) ||
        (st = dmalloc(tmp, s, &err, 1)) || (st = dmalloc(tmp, s, &gsrc, (size_t)M)) ||
        (st = dmalloc(tmp, s, &gdst, (size_t)M)) || (st = dmalloc(tmp, s, &ginit, (size_t)N)))
      break;
    e = hipMemcpyAsync(b->n_off_d, no.data(), 4 * (count + 1), hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipMemcpyAsync(m_off_d, mo.data(), 4 * (count + 1), hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipMemcpyAsync(b->bw_off_d, bo.data(), 4 * (count + 1), hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipMemcpyAsync(b->order_d, order.data(), 4 * count, hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipMemcpyAsync(Kd, num_actions, 4 * count, hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipMemsetAsync(err, 0, 4, s);
    if (e != hipSuccess) {
      set_error("lts_batch_load: %s", hipGetErrorString(e));
      st = BISIM_E_DEVICE;
      break;
    }
    int64_t g = (std::max(N, M) + kT - 1) / kT;
    g = std::min<int64_t>(std::max<int64_t>(g, 1), (int64_t)b->num_cu * 16);
    hipLaunchKernelGGL(k_globalize, dim3((unsigned)g), dim3(kT), 0, s, count, b->n_off_d, m_off_d,
                       Kd, src, label, dst, init_partition, (uint64_t)M, (uint64_t)N, gsrc, gdst,
                       ginit, err);
    uint32_t err_h = 0;
    e = hipGetLastError();
    if (e == hipSuccess) e = hipMemcpyAsync(&err_h, err, 4, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) {
      set_error("lts_batch_load: %s", hipGetErrorString(e));
      st = BISIM_E_DEVICE;
      break;
    }
    if (err_h) {
      set_error("lts_batch_load: an instance-local id, label or init value is out of range");
      st = BISIM_E_RANGE;
      break;
    }
    st = lts_create_union((int32_t)N, M, Kmax, gsrc, label, gdst, ginit, s, &b->u);
    if (st != BISIM_OK) break;
    if (!b->u->uniform) {
      set_error("lts_batch_load: a state has more than 64 distinct outgoing actions");
      st = BISIM_E_UNSUPPORTED;
      break;
    }
    // 32-bit mark words suffice when no state has more than 32 actions
    b->mask64 = Kmax > 32;
    const size_t BW = bo[count];
    b->mem.reserve(105 * (size_t)N + 32 * BW +
                       (size_t)count * (4 + sizeof(RoundsArgs<uint64_t>)) + 40 * 256,
                   s);
    int32_t** const state[] = {&b->blk, &b->tl,  &b->sl, &b->perm, &b->pos, &b->bs,
                               &b->be,  &b->cnt, &b->fc, &b->gc,   &b->tmp, &b->rk,
                               &b->fi,  &b->ltl, &b->ob, &b->tlb,  &b->llo, &b->lsz};
    for (int32_t** p : state)
      if (st == BISIM_OK) st = dmalloc(b->mem, s, p, (size_t)N);
    if (st != BISIM_OK || (st = dmalloc(b->mem, s, &b->mw, (size_t)N)) ||
        (st = dmalloc(b->mem, s, &b->nlb, (size_t)N)) ||
        (st = dmalloc(b->mem, s, &b->tmp64, (size_t)N)) ||
        (st = dmalloc(b->mem, s, &b->pin, (size_t)N)) ||
        (st = dmalloc(b->mem, s, &b->trk, (size_t)N)) || (st = dmalloc(b->mem, s, &b->ub, BW)) ||
        (st = dmalloc(b->mem, s, &b->qb, BW)) || (st = dmalloc(b->mem, s, &b->qs, BW)) ||
        (st = dmalloc(b->mem, s, &b->us, BW)) || (st = dmalloc(b->mem, s, &b->iters_d, count)) ||
        (st = dmalloc(b->mem, s, &b->ctl_d, 2)) || (st = dmalloc(b->mem, s, &b->work_d, 16)) ||
        (st = dmalloc(b->mem, s, &b->args_d, (size_t)count)))
      break;
    st = by_source(b->u);
    if (st == BISIM_E_NOMEM) {  // no label is tracked then
      clear_error();
      st = BISIM_OK;
    }
    if (st != BISIM_OK) break;
    if (count > 0)
      hipLaunchKernelGGL(k_batch_args, dim3((unsigned)(count + 255) / 256), dim3(256), 0, s,
                       make_args(b, nullptr), b->args_d);
    if (hipGetLastError() != hipSuccess) {
      st = BISIM_E_DEVICE;
      break;
    }
    float ms = 0;
    if (hipEventRecord(b->ev1, s) != hipSuccess || hipEventSynchronize(b->ev1) != hipSuccess ||
        hipEventElapsedTime(&ms, b->ev0, b->ev1) != hipSuccess) {
      st = BISIM_E_DEVICE;
      break;
    }
    b->t_pre_ms = ms;
  } while (0);
  tmp.release(b->stream);
  if (st != BISIM_OK) {
    free_batch(b);
    return st;
  }
  *out = b;
  return BISIM_OK;
}

bisim_status coarsest_partition_batch(bisim_batch* b, int32_t* block_id, int64_t* iterations,
                                      bisim_batch_stats* st) {
  if (!b || (!block_id && b->N > 0)) {
    set_error("coarsest_partition_batch: NULL handle or output");
    return BISIM_E_INVALID;
  }
  // configuration: explicit options, else the cached or freshly tuned choice
  if (!b->tuned || b->opt_retune) {
    int wg = 0, grid = 0, lds = 0;
    const bool fixed = b->opt_wg || b->opt_grid || b->opt_lds;
    if (fixed) {
      wg = b->opt_wg ? b->opt_wg : kBatchWG;
      lds = b->opt_lds ? std::min(b->opt_lds, b->lds_max) : b->lds_max;
      grid = b->opt_grid ? b->opt_grid : max_resident(b, wg, lds);
      b->wg = wg;
      b->grid = grid;
      b->lds_bytes = lds;
    } else if (!b->opt_retune && tune_lookup(tune_key(b), &wg, &grid, &lds) && wg && grid &&
               lds <= b->lds_max && max_resident(b, wg, lds) >= grid) {
      b->wg = wg;
      b->grid = grid;
      b->lds_bytes = lds;
    } else {
      BISIM_TRY(autotune(b, block_id));
    }
    if (b->grid < 1) {
      set_error("coarsest_partition_batch: configuration not resident");
      return BISIM_E_DEVICE;
    }
    b->tuned = true;
    b->opt_retune = 0;
  }
  // graph of (queue reset, batched kernel); the configuration and the output
  // pointer are baked into it, so it is re-captured when either changes
  const bool need_graph = !b->gexec || b->g_wg != b->wg || b->g_grid != b->grid ||
                          b->g_lds != b->lds_bytes || b->g_out != block_id;
  if (need_graph) {
    if (b->gexec) {
      (void)hipGraphExecDestroy(b->gexec);
      b->gexec = nullptr;
    }
    hipGraph_t graph = nullptr;
    BISIM_TRY_HIP(hipStreamBeginCapture(b->stream, hipStreamCaptureModeThreadLocal));
    bisim_status ls = launch_once(b, block_id, b->wg, b->grid, b->lds_bytes);
    hipError_t ec = hipStreamEndCapture(b->stream, &graph);
    if (ls != BISIM_OK) return ls;
    BISIM_TRY_HIP(ec);
    hipError_t ei = hipGraphInstantiate(&b->gexec, graph, nullptr, nullptr, 0);
    (void)hipGraphDestroy(graph);
    BISIM_TRY_HIP(ei);
    b->g_wg = b->wg;
    b->g_grid = b->grid;
    b->g_lds = b->lds_bytes;
    b->g_out = block_id;
  }
  BISIM_TRY_HIP(hipEventRecord(b->ev0, b->stream));
  BISIM_TRY_HIP(hipGraphLaunch(b->gexec, b->stream));
  BISIM_TRY_HIP(hipEventRecord(b->ev1, b->stream));
  std::vector<uint32_t> its(b->count);
  uint32_t ctl_h[2] = {0, 0};
  BISIM_TRY_HIP(hipMemcpyAsync(its.data(), b->iters_d, 4 * b->count, hipMemcpyDeviceToHost, b->stream));
  BISIM_TRY_HIP(hipMemcpyAsync(ctl_h, b->ctl_d, 8, hipMemcpyDeviceToHost, b->stream));
  unsigned long long work_h[16];
  BISIM_TRY_HIP(hipMemcpyAsync(work_h, b->work_d, sizeof(work_h), hipMemcpyDeviceToHost,
                               b->stream));
  BISIM_TRY_HIP(hipStreamSynchronize(b->stream));
  float ms = 0;
  BISIM_TRY_HIP(hipEventElapsedTime(&ms, b->ev0, b->ev1));
  b->t_alg_ms = ms;
  if (ctl_h[1] & 2u) {
    set_error("coarsest_partition_batch: inconsistent block ranges");
    return BISIM_E_DEVICE;
  }
  if (ctl_h[1]) {
    set_error("coarsest_partition_batch: an instance exceeded its iteration cap");
    return BISIM_E_ITERCAP;
  }
  int64_t mx = 0, sum = 0, nl = 0, ng = 0;
  for (int32_t k = 0; k < b->count; ++k) {
    mx = std::max<int64_t>(mx, its[k]);
    sum += its[k];
    if (iterations) iterations[k] = its[k];
    const uint32_t n = (uint32_t)(b->n_off[k + 1] - b->n_off[k]);
    const uint64_t need = b->mask64 ? lds_need<uint64_t>(n) : lds_need<uint32_t>(n);
    (need <= (uint64_t)b->lds_bytes ? nl : ng) += 1;
  }
  if (st) {
    st->max_iterations = mx;
    st->sum_iterations = sum;
    st->lds_instances = nl;
    st->global_instances = ng;
    st->workgroup_size = b->wg;
    st->grid = b->grid;
    st->t_pre_ms = b->t_pre_ms;
    st->t_alg_ms = b->t_alg_ms;
    for (int i = 0; i < 16; ++i) st->work[i / 8][i % 8] = (int64_t)work_h[i];
  }
  return BISIM_OK;
}

void lts_batch_free(bisim_batch* b) { free_batch(b); }

bisim_status bisim_batch_set_option(bisim_batch* b, int32_t option, int64_t value) {
  if (!b) {
    set_error("bisim_batch_set_option: NULL handle");
    return BISIM_E_INVALID;
  }
  switch (option) {
    case BISIM_BOPT_WG_SIZE:
      if (value != 0 && value != kBatchWGOption) break;
      b->opt_wg = (int)value;
      b->tuned = false;
      return BISIM_OK;
    case BISIM_BOPT_GRID:
      if (value < 0 || value > (1 << 20)) break;
      b->opt_grid = (int)value;
      b->tuned = false;
      return BISIM_OK;
    case BISIM_BOPT_LDS_LIMIT:
      if (value < 0 || value > (1 << 22)) break;
      b->opt_lds = (int)value;
      b->tuned = false;
      return BISIM_OK;
    case BISIM_BOPT_TUNE:
      if (value != 0 && value != 1) break;
      b->opt_retune = (int)value;
      return BISIM_OK;
    default:
      break;
  }
  set_error("bisim_batch_set_option: bad option %d or value %lld", option, (long long)value);
  return BISIM_E_INVALID;
}

}  // extern "C"
