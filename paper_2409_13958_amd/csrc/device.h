// Device helpers shared by the kernel files.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

#include "kernels.h"

namespace pmfem {

// Grid storage (GridParams::gmode). BF16 is the upper half of an FP32 word,
// rounded to nearest even (the grid values are finite); the pair form keeps
// the rounding residual as a second BF16 value, so hi + lo carries 16
// significant bits. Arithmetic stays FP32: values are widened on load.
__device__ __forceinline__ uint16_t f32_to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

__device__ __forceinline__ float bf16_to_f32(uint16_t h) {
  return __uint_as_float((uint32_t)h << 16);
}

__device__ __forceinline__ int64_t grid_points(const GridParams& g) {
  return (int64_t)g.N[0] * g.N[1] * g.N[2];
}

__device__ __forceinline__ void grid_store(float* G, int64_t i, float v, const GridParams& g) {
  if (g.gmode == 0) {
    G[i] = v;
    return;
  }
  uint16_t* H = reinterpret_cast<uint16_t*>(G);
  const uint16_t hi = f32_to_bf16(v);
  H[i] = hi;
  if (g.gmode == 2) H[grid_points(g) + i] = f32_to_bf16(v - bf16_to_f32(hi));
}

__device__ __forceinline__ float grid_load(const float* G, int64_t i, const GridParams& g) {
  if (g.gmode == 0) return G[i];
  const uint16_t* H = reinterpret_cast<const uint16_t*>(G);
  float v = bf16_to_f32(H[i]);
  if (g.gmode == 2) v += bf16_to_f32(H[grid_points(g) + i]);
  return v;
}

// Block-strided copy loop with K loads in flight per thread: load(i) for K
// indices first, then store(i, value) for the same K.
template <int K, class Load, class Store>
__device__ __forceinline__ void batched(int n, Load&& load, Store&& store) {
  for (int i0 = threadIdx.x; i0 < n; i0 += K * blockDim.x) {
    decltype(load(0)) v[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int i = i0 + k * blockDim.x;
      if (i < n) v[k] = load(i);
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int i = i0 + k * blockDim.x;
      if (i < n) store(i, v[k]);
    }
  }
}

// n / d for 0 <= n < 2^20 and 1 <= d < 2^20 without an integer divide, with
// inv_d = recip(d): (n + 1/2) / d lies at least 1 / (2 d) from an integer, and
// the errors of the reciprocal (one unit in the last place) and of the product
// stay below (n / d) 1.5 2^-23.
__device__ __forceinline__ float recip(int d) { return __builtin_amdgcn_rcpf((float)d); }
__device__ __forceinline__ int fdiv(int n, int d, float inv_d) {
  return (int)(((float)n + 0.5f) * inv_d);
}

}  // namespace pmfem
