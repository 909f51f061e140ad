// Operands of the float32 matrix instructions v_mfma_f32_32x32x2_f32 and v_mfma_f32_16x16x4_f32, loaded straight from
// memory into registers.
//
// The instruction wants row l % R of the operand (R = 32, 16) at k = l / R in lane l.  A sum over k may be taken in any
// order as long as both operands agree, so lane group g = l / R takes the 4 consecutive k's 4 (64 / R) j + 4 g .. + 3 of
// group j: operands whose k runs along memory are then loaded 4 elements at a time; operands stored k x rows are loaded
// one k per instruction, R neighbouring rows per lane group.
#pragma once
#include "kernels.h"

typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
#define GKC(R) (1024 / (R))   // k's per chunk of 16 matrix-core steps

typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4_g;
__device__ __forceinline__ void load4(const float* p, float* o) {
  const float4 v = *(const float4*)p;
  o[0] = v.x; o[1] = v.y; o[2] = v.z; o[3] = v.w;
}
__device__ __forceinline__ void load4(const bf16* p, float* o) {
  const bf16x4_g v = *(const bf16x4_g*)p;
#pragma unroll
  for (int i = 0; i < 4; i++) o[i] = (float)v[i];
}

// One operand of one wave: R rows from r0 on (rows at or past r_end repeat the last one; their results are not stored).
// last_row: row r_end - 1 is read there instead (k-contiguous operands).
template <class T, bool TR, int R>
struct Operand {
  const T* base;            // TR: element (k = 0, row = 0); else this lane's row
  i64 ld;
  bool vec;                 // k-contiguous: 4 consecutive k's may be loaded at once
  const int* gather; int div;
  int row;
  unsigned lane_off;        // TR: this lane's distance from element (first k of the group, row 0)
  __device__ __forceinline__ void init(const T* p, i64 ld_, int r0, int r_end, int lane, const int* gather_ = nullptr, int div_ = 1, int k0 = 0,
                                       const T* last_row = nullptr) {
    ld = ld_; gather = gather_; div = div_;
    row = min(r0 + (lane & (R - 1)), r_end - 1);
    if (TR) { base = p; vec = ld < (1 << 24); lane_off = (unsigned)(4 * (lane / R) * ld) + (unsigned)row; }
    else {
      base = p + (gather ? (i64)(gather[row] / div) : (i64)row) * ld;
      if (last_row && row == r_end - 1) base = last_row;
      vec = ((ld | k0) & 3) == 0 && (((uintptr_t)p | (uintptr_t)last_row) & (4 * sizeof(T) - 1)) == 0;
    }
  }
  // the 16 elements of chunk [kc, kc + GKC(R)) that this lane (of group g) feeds to the 16 steps; fast() holds
  __device__ __forceinline__ void load(int kc, int g, float (&v)[16]) const {
#pragma unroll
    for (int j = 0; j < 4; j++) {
      if (!TR) load4(base + kc + 256 / R * j + 4 * g, v + 4 * j);
      else
#pragma unroll
        for (int i = 0; i < 4; i++) v[4 * j + i] = to_f((base + (i64)(kc + 256 / R * j + i) * ld)[lane_off]);   // (wave-uniform pointer + lane offset)
    }
  }
  __device__ __forceinline__ bool fast() const { return vec && !(TR && gather); }
  // the same for any operand and range: k's at or past k_end are zeros
  __device__ __forceinline__ void load_any(int kc, int k_end, int g, float (&v)[16]) const {
#pragma unroll
    for (int j = 0; j < 4; j++)
#pragma unroll
      for (int i = 0; i < 4; i++) {
        const int k = kc + 256 / R * j + 4 * g + i, kk = min(k, k_end - 1);
        float x;
        if (TR) x = to_f(base[(gather ? (i64)(gather[kk] / div) : (i64)kk) * ld + row]);
        else x = to_f(base[kk]);
        v[4 * j + i] = k < k_end ? x : 0.f;
      }
  }
};

// One wave's share of a contraction over [k0, k_end): the chunks first, first + step, ... of nchunk.  Whole chunks of
// operands that allow wide loads run with one chunk in flight while the one before it is multiplied; what is left, one by one.
// mul(a, b) takes the elements of one chunk.
template <int R, int TM, int TN, class OA, class OB, class Mul>
__device__ __forceinline__ void k_loop(const OA (&oa)[TM], const OB (&ob)[TN], int k0, int k_end, int first, int step, int nchunk, int g, Mul mul) {
  int c = first;
  if (oa[0].fast() && ob[0].fast()) {
    const int full = (k_end - k0) / GKC(R);
    float va[2][TM][16], vb[2][TN][16];
    auto fetch = [&](int q, float (&a)[TM][16], float (&b)[TN][16]) {
#pragma unroll
      for (int i = 0; i < TM; i++) oa[i].load(k0 + q * GKC(R), g, a[i]);
#pragma unroll
      for (int j = 0; j < TN; j++) ob[j].load(k0 + q * GKC(R), g, b[j]);
      __builtin_amdgcn_sched_barrier(0);       // (the compiler would move the loads behind the products they are to overlap with)
    };
    if (c < full) {
      fetch(c, va[0], vb[0]);
      for (; c + step < full; c += 2 * step) {
        fetch(c + step, va[1], vb[1]);
        mul(va[0], vb[0]);
        if (c + 2 * step < full) fetch(c + 2 * step, va[0], vb[0]);
        mul(va[1], vb[1]);
      }
      if (c < full) { mul(va[0], vb[0]); c += step; }
    }
  }
  for (; c < nchunk; c += step) {
    float a[TM][16], b[TN][16];
#pragma unroll
    for (int i = 0; i < TM; i++) oa[i].load_any(k0 + c * GKC(R), k_end, g, a[i]);
#pragma unroll
    for (int j = 0; j < TN; j++) ob[j].load_any(k0 + c * GKC(R), k_end, g, b[j]);
    mul(a, b);
  }
}

// one chunk: 16 steps of the matrix instruction
__device__ __forceinline__ f32x16 mfma_f32(float a, float b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }
__device__ __forceinline__ f32x4 mfma_f32(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
// the result of one tile: lane l holds column l % R, and element e is row acc_row<R>(l, e)
template <int R> struct AccOf;
template <> struct AccOf<32> { typedef f32x16 type; };
template <> struct AccOf<16> { typedef f32x4 type; };
template <int R> __device__ __forceinline__ int acc_row(int lane, int e) { return R == 32 ? (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3) : (lane >> 4) * 4 + e; }
