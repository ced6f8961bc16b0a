// The splitter-scoring network: y = w3 . relu(W2 relu(W1 x + b1) + b2) + b3,
// hidden width 64, F inputs.  fp32 master parameters; the forward pass uses
// bf16 copies of all parameters and of the input (round to nearest even) and
// accumulates in fp32.  Training: mean squared error, gradients with respect
// to the bf16 copies, Adam on the fp32 masters.
//
// Kernels
//   k_mlp_forward   a wave takes tiles of 16 rows; both hidden layers are
//                   products on the fp32 matrix units (v_mfma_f32_16x16x4:
//                   activations keep their 32 bits), the weights staged in
//                   LDS as fp32.
//   k_mlp_backward  the same forward pass, then dZ2, dH1 = dZ2 W2, and the
//                   weight gradients dZ2^T H1 and dZ1^T X, all on the matrix
//                   units and per wave (a wave only reads its own rows, so
//                   nothing waits at a barrier); the gradients of all its
//                   tiles stay in registers.  The workgroup's waves are summed
//                   in LDS in a fixed order and stored as one row of partials.
//   k_mlp_update    sums the workgroups' partials of each parameter in a fixed
//                   order (no floating-point atomics: a training step is
//                   bitwise reproducible), then the Adam step and the bf16
//                   copy.
//
// A tile of 16 rows takes 244 matrix instructions of 32 cycles, 3.3 us: with
// 32,768 rows a wave of each SIMD has two tiles, and the step is bound by
// those and by its two launches.  One wave per row, the unit's products
// through lane shuffles, took 275 us there, and the sum of its 1,024 partials
// by one thread per parameter 238 us.
#include <cmath>
#include <new>
#include <vector>

#include "internal.h"
#include "mlp_dev.h"

struct bisim_mlp {
  int F = 0;
  int64_t P = 0;
  float* master = nullptr;   // device fp32 [P]
  uint16_t* wbf = nullptr;   // device bf16 [P]
  float* m = nullptr;        // Adam moments
  float* v = nullptr;
  float* grad = nullptr;     // device fp32 [P]
  float* loss = nullptr;     // device fp32 [1]
  float* part = nullptr;     // device fp32 [workgroups][P + 2]: partial sums (+ b3, loss)
  int64_t step = 0;
};

namespace bisim {
namespace {
constexpr int kMT = 256;  // 4 waves per workgroup
constexpr int kMW = kMT / kWave;
constexpr int kTile = 16;  // rows per tile
// LDS row strides: 4 floats past a multiple of 32, so that 16 rows read at 4
// consecutive columns touch 64 different banks
constexpr int kS1 = kMlpMaxF + 4, kS2 = kMlpH + 4;

using f32x4 = __attribute__((ext_vector_type(4))) float;
__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) {
  // A: lane l holds row l % 16, column l / 16; B: row l / 16, column l % 16;
  // C, D: rows 4 (l / 16) + i, column l % 16
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// the parameters (bf16 values as fp32) and one wave's tiles
struct TileLds {
  float *W1, *W2;       // [64][kS1] (columns F.. zero), [64][kS2]
  float *b1, *b2, *w3;  // [64]
  float b3;
  float* X;   // this wave's [16][kS1]
  float* H1;  // this wave's [16][kS2]
  float* DZ;  // this wave's [16][kS2]
};
constexpr int kParamFloats = kMlpH * (kS1 + kS2 + 3), kFwdWave = kTile * (kS1 + kS2),
              kBwdWave = kTile * (kS1 + 2 * kS2);

// whole workgroup cooperates; caller synchronises afterwards
__device__ __forceinline__ TileLds tile_stage(float* base, int per_wave,
                                              const uint16_t* __restrict__ w, int F) {
  const MlpOffsets o = mlp_offsets(F);
  TileLds L;
  L.W1 = base;
  L.W2 = L.W1 + kMlpH * kS1;
  L.b1 = L.W2 + kMlpH * kS2;
  L.b2 = L.b1 + kMlpH;
  L.w3 = L.b2 + kMlpH;
  L.X = base + kParamFloats + (threadIdx.x / kWave) * per_wave;
  L.H1 = L.X + kTile * kS1;
  L.DZ = L.H1 + kTile * kS2;
  // 8 parameters a load (both matrices start at a multiple of 16 bytes): calls
  // on a few rows are bound by this (one by one, and with the sums of waves
  // without rows: a step on 1 row 69 us, now 54; forward 41.9, now 40.6)
  const auto eight = [&](int64_t at, float v[8]) {
    const uint4 x = *reinterpret_cast<const uint4*>(w + at);
    const uint32_t q[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[2 * i] = __uint_as_float(q[i] << 16);
      v[2 * i + 1] = __uint_as_float(q[i] & 0xFFFF0000u);
    }
  };
  for (int i = threadIdx.x; i < kMlpH * kMlpH / 8; i += kMT) {
    float v[8];
    eight(o.W2 + 8 * i, v);
#pragma unroll
    for (int e = 0; e < 8; ++e) L.W2[(i / (kMlpH / 8)) * kS2 + i % (kMlpH / 8) * 8 + e] = v[e];
  }
  for (int i = threadIdx.x; i < kMlpH * F / 8; i += kMT) {
    float v[8];
    eight(o.W1 + 8 * i, v);
    int j = 8 * i / F, f = 8 * i % F;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      L.W1[j * kS1 + f] = v[e];
      if (++f == F) {
        f = 0;
        ++j;
      }
    }
  }
  const int pad = kMlpMaxF - F;
  for (int i = threadIdx.x; i < kMlpH * pad; i += kMT) L.W1[(i / pad) * kS1 + F + i % pad] = 0.f;
  if (threadIdx.x < kMlpH) {
    L.b1[threadIdx.x] = bf16_to_f(w[o.b1 + threadIdx.x]);
    L.b2[threadIdx.x] = bf16_to_f(w[o.b2 + threadIdx.x]);
    L.w3[threadIdx.x] = bf16_to_f(w[o.w3 + threadIdx.x]);
  }
  L.b3 = bf16_to_f(w[o.b3]);
  return L;
}

__device__ __forceinline__ float input_of(const float* x, int64_t i) { return bf16_rne(x[i]); }
__device__ __forceinline__ float input_of(const uint16_t* x, int64_t i) { return bf16_to_f(x[i]); }

// LDS written by this wave is read by its other lanes
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Forward pass of rows [r0, r0 + 16) by one wave.  h1[t], h2[t]: units
// 16 t + l % 16 of rows 4 (l / 16) + i; y[i]: the outputs of those rows, on
// all lanes of the row.  X and H1 stay in LDS.
template <class T>
__device__ __forceinline__ void tile_forward(const TileLds& L, int F, const T* __restrict__ x,
                                             int64_t r0, int64_t rows, f32x4 h1[4], f32x4 h2[4],
                                             f32x4& y) {
  const int l = (int)lane(), c = l & 15, g = l >> 4;
  for (int i = l; i < kTile * kMlpMaxF; i += kWave) {
    const int r = i / kMlpMaxF, f = i % kMlpMaxF;
    L.X[r * kS1 + f] = (f < F && r0 + r < rows) ? input_of(x, (r0 + r) * F + f) : 0.f;
  }
  wave_lds_fence();
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const float b = L.b1[16 * t + c];
    h1[t] = f32x4{b, b, b, b};
  }
  for (int s = 0; s < F; s += 4) {  // columns F.. are zero
    const float a = L.X[c * kS1 + s + g];
#pragma unroll
    for (int t = 0; t < 4; ++t) h1[t] = mfma4(a, L.W1[(16 * t + c) * kS1 + s + g], h1[t]);
  }
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      h1[t][i] = fmaxf(h1[t][i], 0.f);
      L.H1[(4 * g + i) * kS2 + 16 * t + c] = h1[t][i];
    }
  wave_lds_fence();
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const float b = L.b2[16 * t + c];
    h2[t] = f32x4{b, b, b, b};
  }
#pragma unroll 4
  for (int s = 0; s < kMlpH; s += 4) {
    const float a = L.H1[c * kS2 + s + g];
#pragma unroll
    for (int t = 0; t < 4; ++t) h2[t] = mfma4(a, L.W2[(16 * t + c) * kS2 + s + g], h2[t]);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    float v = 0.f;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      h2[t][i] = fmaxf(h2[t][i], 0.f);
      v = fmaf(L.w3[16 * t + c], h2[t][i], v);
    }
#pragma unroll
    for (int d = 8; d >= 1; d >>= 1) v += __shfl_xor(v, d, kWave);
    y[i] = v + L.b3;
  }
}

template <class T>
__global__ void __launch_bounds__(kMT) k_mlp_forward(const uint16_t* __restrict__ w, int F,
                                                      const T* __restrict__ x, int64_t rows,
                                                      float* __restrict__ y) {
  extern __shared__ float sw[];
  const TileLds L = tile_stage(sw, kFwdWave, w, F);
  __syncthreads();
  const int l = (int)lane();
  const int64_t wave = ((int64_t)blockIdx.x * kMT + threadIdx.x) / kWave;
  const int64_t nwaves = (int64_t)gridDim.x * kMW;
  for (int64_t r0 = wave * kTile; r0 < rows; r0 += nwaves * kTile) {
    f32x4 h1[4], h2[4], out;
    tile_forward(L, F, x, r0, rows, h1, h2, out);
    wave_lds_fence();  // X and H1 are read before the next tile writes them
    if ((l & 15) == 0) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int64_t r = r0 + 4 * (l >> 4) + i;
        if (r < rows) y[r] = out[i];
      }
    }
  }
}

__global__ void __launch_bounds__(kMT) k_mlp_backward(const uint16_t* __restrict__ w, int F,
                                                       const float* __restrict__ x,
                                                       const float* __restrict__ t, int64_t rows,
                                                       float* __restrict__ part, int64_t P) {
  extern __shared__ float sw[];
  const TileLds L = tile_stage(sw, kBwdWave, w, F);
  float* red = sw + kParamFloats + kMW * kBwdWave;  // [P + 2] the waves' sums
  __syncthreads();
  const int l = (int)lane(), c = l & 15, g = l >> 4;
  const int wv = threadIdx.x / kWave;
  const int64_t wave = ((int64_t)blockIdx.x * kMT + threadIdx.x) / kWave;
  const int64_t nwaves = (int64_t)gridDim.x * kMW;
  const float inv = 2.0f / (float)rows;
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  // gW2[u][t]: rows 16 u + 4 g + i, columns 16 t + c of the gradient of W2;
  // gW1 the same for W1; gb2, gw3, gb1: unit 16 t + c, this lane's rows
  f32x4 gW2[4][4], gW1[4][kMlpMaxF / 16];
  float gb1[4], gb2[4], gw3[4], gb3 = 0.f, lsum = 0.f;
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    gb1[u] = gb2[u] = gw3[u] = 0.f;
#pragma unroll
    for (int v = 0; v < 4; ++v) gW2[u][v] = zero;
#pragma unroll
    for (int v = 0; v < kMlpMaxF / 16; ++v) gW1[u][v] = zero;
  }
  for (int64_t r0 = wave * kTile; r0 < rows; r0 += nwaves * kTile) {
    f32x4 h1[4], h2[4], yv, dy;
    tile_forward(L, F, x, r0, rows, h1, h2, yv);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int64_t r = r0 + 4 * g + i;
      const float diff = r < rows ? yv[i] - t[r] : 0.f;
      dy[i] = inv * diff;
      lsum += diff * diff;
      gb3 += dy[i];
    }
    // dZ2, its sums over rows, and dH1 = dZ2 W2
    f32x4 dh[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      dh[u] = zero;
      const float w3 = L.w3[16 * u + c];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float d = h2[u][i] > 0.f ? dy[i] * w3 : 0.f;
        gw3[u] += dy[i] * h2[u][i];
        gb2[u] += d;
        L.DZ[(4 * g + i) * kS2 + 16 * u + c] = d;
      }
    }
    wave_lds_fence();
#pragma unroll 4
    for (int s = 0; s < kMlpH; s += 4) {
      const float a = L.DZ[c * kS2 + s + g];
#pragma unroll
      for (int u = 0; u < 4; ++u) dh[u] = mfma4(a, L.W2[(s + g) * kS2 + 16 * u + c], dh[u]);
    }
    // gW2 += dZ2^T H1 over the tile's rows
#pragma unroll
    for (int s = 0; s < kTile; s += 4) {
      float b[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) b[v] = L.H1[(s + g) * kS2 + 16 * v + c];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const float a = L.DZ[(s + g) * kS2 + 16 * u + c];
#pragma unroll
        for (int v = 0; v < 4; ++v) gW2[u][v] = mfma4(a, b[v], gW2[u][v]);
      }
    }
    wave_lds_fence();  // DZ is read before dZ1 takes its place
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float d = h1[u][i] > 0.f ? dh[u][i] : 0.f;
        gb1[u] += d;
        L.DZ[(4 * g + i) * kS2 + 16 * u + c] = d;
      }
    wave_lds_fence();
#pragma unroll
    for (int s = 0; s < kTile; s += 4) {
      float b[kMlpMaxF / 16];
#pragma unroll
      for (int v = 0; v < kMlpMaxF / 16; ++v) b[v] = L.X[(s + g) * kS1 + 16 * v + c];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const float a = L.DZ[(s + g) * kS2 + 16 * u + c];
#pragma unroll
        for (int v = 0; v < kMlpMaxF / 16; ++v) gW1[u][v] = mfma4(a, b[v], gW1[u][v]);
      }
    }
    wave_lds_fence();
  }
  // sums over the row groups of the lanes
#pragma unroll
  for (int u = 0; u < 4; ++u)
#pragma unroll
    for (int d = 16; d <= 32; d <<= 1) {
      gb1[u] += __shfl_xor(gb1[u], d, kWave);
      gb2[u] += __shfl_xor(gb2[u], d, kWave);
      gw3[u] += __shfl_xor(gw3[u], d, kWave);
    }
#pragma unroll
  for (int d = 16; d <= 32; d <<= 1) {
    gb3 += __shfl_xor(gb3, d, kWave);
    lsum += __shfl_xor(lsum, d, kWave);
  }
  // the workgroup's waves in order
  const MlpOffsets o = mlp_offsets(F);
  const int64_t tiles = (rows + kTile - 1) / kTile - (int64_t)blockIdx.x * kMW;
  const int active = tiles < kMW ? (int)tiles : kMW;  // waves that had rows (the first ones)
  for (int q = 0; q < active; ++q) {
    if (wv == q) {
      const auto add = [&](int64_t i, float v) { red[i] = q == 0 ? v : red[i] + v; };
#pragma unroll
      for (int u = 0; u < 4; ++u) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int j = 16 * u + 4 * g + i;
#pragma unroll
          for (int v = 0; v < 4; ++v) add(o.W2 + j * kMlpH + 16 * v + c, gW2[u][v][i]);
#pragma unroll
          for (int v = 0; v < kMlpMaxF / 16; ++v)
            if (16 * v + c < F) add(o.W1 + j * F + 16 * v + c, gW1[u][v][i]);
        }
        if (g == 0) {
          add(o.b1 + 16 * u + c, gb1[u]);
          add(o.b2 + 16 * u + c, gb2[u]);
          add(o.w3 + 16 * u + c, gw3[u]);
        }
      }
      if (l == 0) {
        add(o.b3, gb3);
        add(P + 1, lsum / (float)rows);
      }
    }
    __syncthreads();
  }
  float* mine = part + (int64_t)blockIdx.x * (P + 2);
  for (int64_t i = threadIdx.x; i < P + 2; i += kMT)
    if (i != P) mine[i] = red[i];
}

// Sum of the workgroups' partials (64 parameters per workgroup; each wave sums
// a quarter of the rows in order, then the waves in order; index P + 1 is the
// loss), and the Adam step (lr > 0).
__global__ void __launch_bounds__(kMT) k_mlp_update(const float* __restrict__ part, int nblk,
                                                     int64_t P, float* __restrict__ grad,
                                                     float* __restrict__ loss,
                                                     float* __restrict__ w,
                                                     uint16_t* __restrict__ wbf,
                                                     float* __restrict__ m, float* __restrict__ v,
                                                     float lr, float c1, float c2) {
  __shared__ float sum[kMW][kWave];
  const int wv = threadIdx.x / kWave;
  const int64_t i = (int64_t)blockIdx.x * kWave + lane();
  const int per = (nblk + kMW - 1) / kMW, b0 = wv * per, b1 = min(nblk, b0 + per);
  float s = 0.f;
  if (i < P + 2 && i != P) {
    int b = b0;
    for (; b + 8 <= b1; b += 8) {
      float x[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) x[q] = part[(int64_t)(b + q) * (P + 2) + i];
#pragma unroll
      for (int q = 0; q < 8; ++q) s += x[q];
    }
    for (; b < b1; ++b) s += part[(int64_t)b * (P + 2) + i];
  }
  sum[wv][lane()] = s;
  __syncthreads();
  if (wv != 0 || i >= P + 2 || i == P) return;
  s = 0.f;
  for (int q = 0; q < kMW; ++q) s += sum[q][lane()];
  if (i == P + 1) {
    *loss = s;
    return;
  }
  grad[i] = s;
  if (!(lr > 0.f)) return;
  const float a1 = 0.9f, a2 = 0.999f, eps = 1e-8f;
  const float mi = a1 * m[i] + (1.f - a1) * s;
  const float vi = a2 * v[i] + (1.f - a2) * s * s;
  m[i] = mi;
  v[i] = vi;
  const float wi = w[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
  w[i] = wi;
  wbf[i] = bf16_bits(wi);
}

__global__ void k_to_bf16(const float* __restrict__ w, uint16_t* __restrict__ wbf, int64_t P) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < P;
       i += (int64_t)gridDim.x * blockDim.x)
    wbf[i] = bf16_bits(w[i]);
}

// He-normal initialisation from splitmix64 + Box-Muller (host side)
uint64_t splitmix64(uint64_t& s) {
  uint64_t z = (s += 0x9E3779B97F4A7C15ull);
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}
double normal(uint64_t& s) {
  const double u1 = ((splitmix64(s) >> 11) + 1.0) * (1.0 / 9007199254740993.0);
  const double u2 = (splitmix64(s) >> 11) * (1.0 / 9007199254740992.0);
  return std::sqrt(-2.0 * std::log(u1)) * std::cos(6.283185307179586 * u2);
}

constexpr size_t fwd_lds() { return (kParamFloats + kMW * kFwdWave) * sizeof(float); }
size_t bwd_lds(int64_t P) { return (kParamFloats + kMW * kBwdWave + P + 2) * sizeof(float); }

// workgroups for `rows` rows: a tile per wave, up to `most`
constexpr int kMaxGridFwd = 1024, kMaxGridRows = 256;
unsigned grid_rows(int64_t rows, int most) {
  int64_t g = (rows + kTile * kMW - 1) / (kTile * kMW);
  if (g > most) g = most;
  if (g < 1) g = 1;
  return (unsigned)g;
}

template <class T>
bisim_status forward_on(const bisim_mlp* w, const T* x, int64_t rows, float* y, hipStream_t s) {
  if (rows <= 0) return BISIM_OK;
  const auto k = k_mlp_forward<T>;
  BISIM_TRY_HIP(hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize,
                                    (int)fwd_lds()));
  hipLaunchKernelGGL(k, dim3(grid_rows(rows, kMaxGridFwd)), dim3(kMT), fwd_lds(), s, w->wbf, w->F,
                     x, rows, y);
  BISIM_TRY_HIP(hipGetLastError());
  return BISIM_OK;
}
}  // namespace

const uint16_t* mlp_weights_bf16(const bisim_mlp* w) { return w->wbf; }
int mlp_features(const bisim_mlp* w) { return w->F; }
}  // namespace bisim

using namespace bisim;

extern "C" {

int64_t mlp_num_params(int32_t in_features) {
  if (in_features < 1 || in_features > kMlpMaxF) return -1;
  return mlp_offsets(in_features).total;
}

bisim_status mlp_create(int32_t in_features, const float* init_fp32, uint64_t seed,
                        bisim_mlp** out) {
  if (!out || in_features < 1 || in_features > kMlpMaxF) {
    set_error("mlp_create: need 1 <= in_features <= %d and an output pointer", kMlpMaxF);
    return BISIM_E_INVALID;
  }
  *out = nullptr;
  bisim_mlp* w = new (std::nothrow) bisim_mlp;
  if (!w) return BISIM_E_NOMEM;
  w->F = in_features;
  w->P = mlp_offsets(in_features).total;
  std::vector<float> h((size_t)w->P, 0.f);
  if (init_fp32) {
    for (int64_t i = 0; i < w->P; ++i) h[i] = init_fp32[i];
  } else {
    const MlpOffsets o = mlp_offsets(in_features);
    uint64_t s = seed;
    for (int i = 0; i < kMlpH * in_features; ++i)
      h[o.W1 + i] = (float)(normal(s) * std::sqrt(2.0 / in_features));
    for (int i = 0; i < kMlpH * kMlpH; ++i) h[o.W2 + i] = (float)(normal(s) * std::sqrt(2.0 / kMlpH));
    for (int i = 0; i < kMlpH; ++i) h[o.w3 + i] = (float)(normal(s) * std::sqrt(1.0 / kMlpH));
  }
  hipError_t e = hipMalloc((void**)&w->master, 4 * w->P);
  if (e == hipSuccess) e = hipMalloc((void**)&w->wbf, 2 * w->P);
  if (e == hipSuccess) e = hipMalloc((void**)&w->m, 4 * w->P);
  if (e == hipSuccess) e = hipMalloc((void**)&w->v, 4 * w->P);
  if (e == hipSuccess) e = hipMalloc((void**)&w->grad, 4 * w->P);
  if (e == hipSuccess) e = hipMalloc((void**)&w->loss, 4);
  if (e == hipSuccess) e = hipMalloc((void**)&w->part, 4 * (size_t)kMaxGridRows * (w->P + 2));
  if (e == hipSuccess) e = hipMemcpy(w->master, h.data(), 4 * w->P, hipMemcpyHostToDevice);
  if (e == hipSuccess) e = hipMemset(w->m, 0, 4 * w->P);
  if (e == hipSuccess) e = hipMemset(w->v, 0, 4 * w->P);
  if (e == hipSuccess) {
    hipLaunchKernelGGL(k_to_bf16, dim3(16), dim3(256), 0, nullptr, w->master, w->wbf, w->P);
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = hipDeviceSynchronize();
  if (e != hipSuccess) {
    set_error("mlp_create: %s", hipGetErrorString(e));
    mlp_free(w);
    return BISIM_E_DEVICE;
  }
  *out = w;
  return BISIM_OK;
}

void mlp_free(bisim_mlp* w) {
  if (!w) return;
  (void)hipDeviceSynchronize();
  void* p[] = {w->master, w->wbf, w->m, w->v, w->grad, w->loss, w->part};
  for (void* q : p)
    if (q) (void)hipFree(q);
  delete w;
}

bisim_status mlp_get_params(const bisim_mlp* w, float* host_fp32) {
  if (!w || !host_fp32) {
    set_error("mlp_get_params: NULL argument");
    return BISIM_E_INVALID;
  }
  BISIM_TRY_HIP(hipDeviceSynchronize());
  BISIM_TRY_HIP(hipMemcpy(host_fp32, w->master, 4 * w->P, hipMemcpyDeviceToHost));
  return BISIM_OK;
}

bisim_status mlp_forward(const bisim_mlp* w, const float* x, int64_t rows, float* y,
                         void* hip_stream) {
  if (!w || rows < 0 || (rows > 0 && (!x || !y))) {
    set_error("mlp_forward: bad arguments");
    return BISIM_E_INVALID;
  }
  BISIM_TRY(forward_on(w, x, rows, y, (hipStream_t)hip_stream));
  BISIM_TRY_HIP(hipStreamSynchronize((hipStream_t)hip_stream));
  return BISIM_OK;
}

bisim_status mlp_forward_bf16(const bisim_mlp* w, const void* x_bf16, int64_t rows, float* y,
                              void* hip_stream) {
  if (!w || rows < 0 || (rows > 0 && (!x_bf16 || !y))) {
    set_error("mlp_forward_bf16: bad arguments");
    return BISIM_E_INVALID;
  }
  hipStream_t s = (hipStream_t)hip_stream;
  BISIM_TRY(forward_on(w, (const uint16_t*)x_bf16, rows, y, s));
  BISIM_TRY_HIP(hipStreamSynchronize(s));
  return BISIM_OK;
}

bisim_status mlp_train_step(bisim_mlp* w, const float* x, const float* target, int64_t rows,
                            float lr, float* loss_out, float* grad_out, void* hip_stream) {
  if (!w || rows < 1 || !x || !target || !(lr >= 0.f)) {
    set_error("mlp_train_step: bad arguments");
    return BISIM_E_INVALID;
  }
  hipStream_t s = (hipStream_t)hip_stream;
  const unsigned g = grid_rows(rows, kMaxGridRows);
  const size_t lds = bwd_lds(w->P);
  BISIM_TRY_HIP(hipFuncSetAttribute((const void*)k_mlp_backward,
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
  hipLaunchKernelGGL(k_mlp_backward, dim3(g), dim3(kMT), lds, s, w->wbf, w->F, x, target, rows,
                     w->part, w->P);
  float c1 = 1.f, c2 = 1.f;
  if (lr > 0.f) {
    w->step += 1;
    c1 = 1.f - std::pow(0.9f, (float)w->step);
    c2 = 1.f - std::pow(0.999f, (float)w->step);
  }
  hipLaunchKernelGGL(k_mlp_update, dim3((unsigned)((w->P + 2 + kWave - 1) / kWave)), dim3(kMT), 0,
                     s, w->part, (int)g, w->P, w->grad, w->loss, w->master, w->wbf, w->m, w->v, lr,
                     c1, c2);
  BISIM_TRY_HIP(hipGetLastError());
  if (grad_out)
    BISIM_TRY_HIP(hipMemcpyAsync(grad_out, w->grad, 4 * w->P, hipMemcpyDeviceToDevice, s));
  float l = 0.f;
  BISIM_TRY_HIP(hipMemcpyAsync(&l, w->loss, 4, hipMemcpyDeviceToHost, s));
  BISIM_TRY_HIP(hipStreamSynchronize(s));
  if (loss_out) *loss_out = l;
  return BISIM_OK;
}

}  // extern "C"
