// The library's device allocator (stream-ordered memory, or a caller's
// region for the allocation-free entry point) and a measurement helper: a
// plain streaming copy, used to measure the bandwidth the device actually
// sustains and to calibrate memory-traffic counters.
#include <cstdlib>

#include "internal.h"

namespace bisim {

static thread_local ArenaScope* g_arena = nullptr;
static thread_local Chunks* g_chunks = nullptr;

static size_t piece_bytes(size_t bytes) { return ((bytes ? bytes : 1) + 255) & ~(size_t)255; }

hipError_t Chunks::add(size_t bytes, hipStream_t s) {
  // test hook: BISIM_HANDLE_LIMIT=<bytes> bounds the chunks of one handle
  if (const char* limit = getenv("BISIM_HANDLE_LIMIT")) {
    size_t held = 0;
    for (const Chunk& c : chunks_) held += c.capacity;
    if (held + bytes > strtoull(limit, nullptr, 10)) return hipErrorOutOfMemory;
  }
  void* p = nullptr;
  const hipError_t e = hipMallocAsync(&p, bytes, s);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    return e;
  }
  try {
    chunks_.push_back({(char*)p, bytes, Pieces(bytes)});
  } catch (...) {  // no host memory for the list
    (void)hipFreeAsync(p, s);
    return hipErrorOutOfMemory;
  }
  return hipSuccess;
}
// the newest chunk with room takes the piece (a chunk's rest is not lost when
// a larger request has opened another)
bool Chunks::cut(void** p, size_t need) {
  size_t at = 0;
  for (size_t i = chunks_.size(); i-- > 0;)
    if (chunks_[i].pieces.cut(need, &at)) {
      *p = chunks_[i].base + at;
      return true;
    }
  return false;
}
void Chunks::reserve(size_t bytes, hipStream_t s) {
  for (const Chunk& c : chunks_)
    if (c.capacity - c.pieces.used() >= bytes) return;
  (void)add(piece_bytes(bytes), s);
}
hipError_t Chunks::alloc(void** p, size_t bytes, hipStream_t s) try {
  const size_t need = piece_bytes(bytes);
  if (cut(p, need)) return hipSuccess;
  // beyond what was reserved: 1 MiB at a time for small requests
  hipError_t e = need < (1u << 20) ? add(1u << 20, s) : hipErrorOutOfMemory;
  if (e != hipSuccess) e = add(need, s);
  if (e != hipSuccess) return e;
  return cut(p, need) ? hipSuccess : hipErrorOutOfMemory;
} catch (...) {
  return hipErrorOutOfMemory;
}
bool Chunks::give_back(const void* p) {
  for (Chunk& c : chunks_)
    if ((const char*)p >= c.base && (const char*)p < c.base + c.capacity) {
      c.pieces.give_back((size_t)((const char*)p - c.base));
      return true;
    }
  return false;
}
void Chunks::release(hipStream_t s) {
  for (const Chunk& c : chunks_) (void)hipFreeAsync(c.base, s);
  chunks_.clear();
}
ChunkScope::ChunkScope(Chunks& c) : outer_(g_chunks) { g_chunks = &c; }
ChunkScope::~ChunkScope() { g_chunks = outer_; }

ArenaScope::ArenaScope(char* base, size_t capacity) : base_(base), cap_(capacity), outer_(g_arena) {
  g_arena = this;
}
ArenaScope::~ArenaScope() { g_arena = outer_; }
bool arena_active() { return g_arena != nullptr; }

hipError_t dev_alloc(void** p, size_t bytes, hipStream_t s) {
  *p = nullptr;
  if (bytes == 0) bytes = 1;
  ArenaScope* a = g_arena;
  if (!a) return g_chunks ? g_chunks->alloc(p, bytes, s) : hipMallocAsync(p, bytes, s);
  const size_t at = (a->used_ + 255) & ~(size_t)255;
  if (at > a->cap_ || bytes > a->cap_ - at) return hipErrorOutOfMemory;
  *p = a->base_ + at;
  a->used_ = at + bytes;
  return hipSuccess;
}

hipError_t dev_free(void* p, hipStream_t s) {
  if (!p) return hipSuccess;
  for (ArenaScope* a = g_arena; a; a = a->outer_)
    if ((char*)p >= a->base_ && (char*)p < a->base_ + a->cap_) return hipSuccess;
  if (g_chunks && g_chunks->give_back(p)) return hipSuccess;
  return hipFreeAsync(p, s);
}

namespace {
__global__ void __launch_bounds__(256) k_copy16(const uint4* __restrict__ src,
                                                uint4* __restrict__ dst, uint64_t n16) {
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += stride)
    dst[i] = src[i];
}
}  // namespace
}  // namespace bisim

using namespace bisim;

extern "C" bisim_status bisim_device_copy(void* dst, const void* src, int64_t bytes,
                                          void* hip_stream, double* ms_out) {
  if (!dst || !src || bytes < 0 || (bytes & 15) || ((uintptr_t)dst & 15) || ((uintptr_t)src & 15)) {
    set_error("bisim_device_copy: 16-byte aligned pointers and a multiple of 16 bytes");
    return BISIM_E_INVALID;
  }
  hipStream_t s = (hipStream_t)hip_stream;
  int dev = 0, cu = 0;
  BISIM_TRY_HIP(hipGetDevice(&dev));
  BISIM_TRY_HIP(hipDeviceGetAttribute(&cu, hipDeviceAttributeMultiprocessorCount, dev));
  const uint64_t n16 = (uint64_t)bytes / 16;
  uint64_t g = (n16 + 255) / 256;
  if (g > (uint64_t)cu * 32) g = (uint64_t)cu * 32;
  if (g < 1) g = 1;
  hipEvent_t e0, e1;
  BISIM_TRY_HIP(hipEventCreate(&e0));
  BISIM_TRY_HIP(hipEventCreate(&e1));
  BISIM_TRY_HIP(hipEventRecord(e0, s));
  hipLaunchKernelGGL(k_copy16, dim3((unsigned)g), dim3(256), 0, s, (const uint4*)src, (uint4*)dst,
                     n16);
  BISIM_TRY_HIP(hipGetLastError());
  BISIM_TRY_HIP(hipEventRecord(e1, s));
  BISIM_TRY_HIP(hipEventSynchronize(e1));
  float ms = 0;
  BISIM_TRY_HIP(hipEventElapsedTime(&ms, e0, e1));
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  if (ms_out) *ms_out = ms;
  return BISIM_OK;
}
