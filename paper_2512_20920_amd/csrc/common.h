// Shared device/host helpers for the RevFFN HIP library (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

typedef __bf16 bf16;
typedef long long i64;

#define WAVE 64

template <class T> __device__ __forceinline__ float to_f(T v) { return (float)v; }
template <class T> __device__ __forceinline__ T from_f(float v) { return (T)v; }

// Reductions over the 64 lanes in a fixed order, result in every lane: inclusive combination inside the rows of 16 lanes,
// then across rows with the row broadcasts, all as data-parallel-primitive moves (a register-to-register instruction per
// step; __shfl_xor goes through the LDS crossbar, some 100 clocks a step), and lane 63 read back.
template <int CTRL, int ROW_MASK> __device__ __forceinline__ float dpp_f(float keep, float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, keep), __builtin_bit_cast(int, v), CTRL, ROW_MASK, 0xf, false));
}
__device__ __forceinline__ float lane63(float v) { return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63)); }
__device__ __forceinline__ float wave_sum(float v) {
  v += dpp_f<0x111, 0xf>(0.f, v);          // row_shr:1
  v += dpp_f<0x112, 0xf>(0.f, v);          // row_shr:2
  v += dpp_f<0x114, 0xf>(0.f, v);          // row_shr:4
  v += dpp_f<0x118, 0xf>(0.f, v);          // row_shr:8
  v += dpp_f<0x142, 0xa>(0.f, v);          // row_bcast:15 into rows 1 and 3
  v += dpp_f<0x143, 0xc>(0.f, v);          // row_bcast:31 into rows 2 and 3
  return lane63(v);
}
__device__ __forceinline__ float wave_max(float v) {
  v = fmaxf(v, dpp_f<0x111, 0xf>(v, v));
  v = fmaxf(v, dpp_f<0x112, 0xf>(v, v));
  v = fmaxf(v, dpp_f<0x114, 0xf>(v, v));
  v = fmaxf(v, dpp_f<0x118, 0xf>(v, v));
  v = fmaxf(v, dpp_f<0x142, 0xa>(v, v));
  v = fmaxf(v, dpp_f<0x143, 0xc>(v, v));
  return lane63(v);
}

// Block-wide sum for blockDim.x = 256 (4 waves); result valid in every thread.
// red must point at >= 4 floats of LDS.  Fixed combination order -> deterministic.
__device__ __forceinline__ float block_sum_256(float v, float* red) {
  v = wave_sum(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  return (red[0] + red[1]) + (red[2] + red[3]);
}

__device__ __forceinline__ float sigmoid_f(float x) { return 1.0f / (1.0f + __expf(-x)); }

// one of a pair of columns rotated by (cos, sin): the first one is own * cos - other * sin, the second own * cos + other * sin
__device__ __forceinline__ float rope_value(float own, float other, bool second, float2 cs) {
  return second ? own * cs.x + other * cs.y : own * cs.x - other * cs.y;
}
// gradients at gate and up of silu(gate) * up, whose gradient is d
__device__ __forceinline__ void swiglu_grad(float d, float gate, float up, float* dgate, float* dup) {
  const float sg = sigmoid_f(gate);
  *dgate = d * up * sg * (1.f + gate * (1.f - sg));
  *dup = d * gate * sg;
}

static inline int cdiv(i64 a, i64 b) { return (int)((a + b - 1) / b); }

// A kernel's dynamic-LDS limit is an attribute per device: `mask` (one per kernel instantiation) keeps one bit per
// device id.  attr_needed: the current device has not been marked yet (the caller sets the attribute, then calls
// attr_done; several threads may do so at once, which is harmless, and none launches before its own call returned).
#include <atomic>
static inline bool attr_needed(const std::atomic<unsigned long long>& mask) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev > 63) return true;
  return (mask.load(std::memory_order_acquire) & (1ull << dev)) == 0;
}
static inline void attr_done(std::atomic<unsigned long long>& mask) {
  int dev = 0;
  if (hipGetDevice(&dev) == hipSuccess && dev >= 0 && dev <= 63) mask.fetch_or(1ull << dev, std::memory_order_acq_rel);
}
