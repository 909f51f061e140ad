// Operands of the float32 matrix instruction v_mfma_f32_32x32x2_f32, loaded straight from memory into registers.
//
// The instruction wants row l & 31 at k = l >> 5 in lane l.  A sum over k may be taken in any order as long as both
// operands agree, so lane half g = l >> 5 takes the 4 consecutive k's 8 j + 4 g .. + 3 of group j: operands whose k runs
// along memory are then loaded 4 elements at a time; operands stored k x rows are loaded one k per instruction, 32
// neighbouring rows per half wave.
#pragma once
#include "kernels.h"

typedef __attribute__((ext_vector_type(16))) float f32x16;
#define GKC 32            // k's per chunk: 16 matrix-core steps

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

// One operand of one wave: 32 rows from r0 on (rows at or past r_end repeat the last one; their results are not stored).
// last_row: row r_end - 1 is read there instead (k-contiguous operands).
template <class T, bool TR>
struct Operand {
  const T* base;            // TR: element (k = 0, row of this lane's half-wave position); else row start of this lane's row
  i64 ld;
  bool vec;                 // 4 consecutive k's may be loaded at once (k-contiguous operands)
  const int* gather; int div;
  const T* all;             // with a gather list on the k rows
  int row;
  __device__ __forceinline__ void init(const T* p, i64 ld_, int r0, int r_end, int lane, const int* gather_ = nullptr, int div_ = 1, int k0 = 0,
                                       const T* last_row = nullptr) {
    ld = ld_; gather = gather_; div = div_; all = p;
    row = min(r0 + (lane & 31), r_end - 1);
    if (TR) { base = p + row; vec = false; }
    else {
      base = p + (gather ? (i64)(gather[row] / div) : (i64)row) * ld;
      if (last_row && row == r_end - 1) base = last_row;
      vec = ((ld | k0) & 3) == 0 && (((uintptr_t)p | (uintptr_t)last_row) & (4 * sizeof(T) - 1)) == 0;
    }
  }
  // the 16 elements of chunk [kc, kc + 32) that this lane feeds to the 16 steps; k's at or past k_end are zeros
  __device__ __forceinline__ void load(int kc, int k_end, int g, float (&v)[16]) const {
    if (kc + GKC <= k_end && !(TR && gather)) {
      if (!TR && vec) {
#pragma unroll
        for (int j = 0; j < 4; j++) load4(base + kc + 8 * j + 4 * g, v + 4 * j);
      } else {
#pragma unroll
        for (int j = 0; j < 4; j++)
#pragma unroll
          for (int i = 0; i < 4; i++) {
            const int k = kc + 8 * j + 4 * g + i;
            v[4 * j + i] = to_f(TR ? base[(i64)k * ld] : base[k]);
          }
      }
      return;
    }
#pragma unroll
    for (int j = 0; j < 4; j++)
#pragma unroll
      for (int i = 0; i < 4; i++) {
        const int k = kc + 8 * j + 4 * g + i, kk = min(k, k_end - 1);
        float x;
        if (TR) x = to_f(gather ? all[(i64)(gather[kk] / div) * ld + row] : base[(i64)kk * ld]);
        else x = to_f(base[kk]);
        v[4 * j + i] = k < k_end ? x : 0.f;
      }
  }
};
