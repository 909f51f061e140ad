// Operands of the float32 matrix instructions v_mfma_f32_32x32x2_f32 and v_mfma_f32_16x16x4_f32: loaded straight from
// memory into registers, or (StagedOperand, the router's) through registers into LDS.
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
  static constexpr bool staged = false;
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

// The same for operands whose k runs along memory, staged.  A load of 4 k's above puts every lane on a cache line of its own
// (94 clocks per wave-load against 16).  Where many waves of a CU load at once (the router kernel: 20 -> 14 us for 37 tokens)
// they are therefore loaded in memory order and reach their lanes through 1024 elements of LDS that belong to the wave (no
// barrier; 4-element unit u of row r in place u ^ (r >> SH), so that neither side meets a bank twice).  Where a wave has
// only a chunk or two, the detour costs more than it saves (float32 GEMMs: no change at k = 512, a step 3 % slower at 64).
template <class T, int R>
struct StagedOperand {
  static constexpr bool staged = true;
  typedef __attribute__((ext_vector_type(4))) T vec4;
  static constexpr int UPR = GKC(R) / 4;                          // 4-element units per row of a chunk
  static constexpr int SH = GKC(R) * sizeof(T) == 256 ? 0 : GKC(R) * sizeof(T) == 128 ? 1 : 2;    // rows per 256 bytes: 2^SH
  static constexpr size_t lds_bytes = 1024 * sizeof(T);
  struct Chunk { vec4 v[4]; };                                    // this lane's share, as it lies in memory
  const T* base;            // this lane's row
  bool vec;                 // 4 consecutive k's may be loaded at once
  const T* src[4];          // where this lane's units of a chunk come from (k = 0), rows (64 / UPR) j + lane / UPR
  vec4 *put, *get;          // where unit 0 of them goes in LDS, and this lane's row there
  int sw_put, sw_get, unit;
  __device__ __forceinline__ void init(const T* p, i64 ld, int r0, int r_end, int lane, void* lds) {
    base = p + (i64)min(r0 + (lane & (R - 1)), r_end - 1) * ld;
    vec = (ld & 3) == 0 && ((uintptr_t)p & (4 * sizeof(T) - 1)) == 0;
    unit = lane & (UPR - 1);
#pragma unroll
    for (int j = 0; j < 4; j++) src[j] = p + (i64)min(r0 + j * (64 / UPR) + lane / UPR, r_end - 1) * ld + unit * 4;
    put = (vec4*)lds + (lane / UPR) * UPR;
    get = (vec4*)lds + (lane & (R - 1)) * UPR;
    sw_put = lane / UPR;
    sw_get = ((lane & (R - 1)) >> SH) & (UPR - 1);
  }
  __device__ __forceinline__ void load(int kc, Chunk& c) const {
#pragma unroll
    for (int j = 0; j < 4; j++) c.v[j] = *(const vec4*)(src[j] + kc);
  }
  // the 16 elements that this lane (of group g) feeds to the 16 steps
  __device__ __forceinline__ void deliver(const Chunk& c, int g, float (&v)[16]) const {
    asm volatile("" ::: "memory");                                // (LDS instructions of one wave run in order)
#pragma unroll
    for (int j = 0; j < 4; j++) put[j * 64 + (unit ^ (((sw_put + j * (64 / UPR)) >> SH) & (UPR - 1)))] = c.v[j];
    asm volatile("" ::: "memory");
#pragma unroll
    for (int j = 0; j < 4; j++) {
      const vec4 x = get[(64 / R * j + g) ^ sw_get];
#pragma unroll
      for (int i = 0; i < 4; i++) v[4 * j + i] = (float)x[i];
    }
  }
  __device__ __forceinline__ bool fast() const { return vec; }
  __device__ __forceinline__ void load_any(int kc, int k_end, int g, float (&v)[16]) const {
#pragma unroll
    for (int j = 0; j < 4; j++)
#pragma unroll
      for (int i = 0; i < 4; i++) {
        const int k = kc + 256 / R * j + 4 * g + i;
        const float x = to_f(base[min(k, k_end - 1)]);
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
    if constexpr (OA::staged) {
      typename OA::Chunk ca[2][TM];
      typename OB::Chunk cb[2][TN];
      auto fetch = [&](int q, typename OA::Chunk (&a)[TM], typename OB::Chunk (&b)[TN]) {
#pragma unroll
        for (int i = 0; i < TM; i++) oa[i].load(k0 + q * GKC(R), a[i]);
#pragma unroll
        for (int j = 0; j < TN; j++) ob[j].load(k0 + q * GKC(R), b[j]);
        __builtin_amdgcn_sched_barrier(0);       // (the compiler would move the loads behind the products they are to overlap with)
      };
      auto use = [&](const typename OA::Chunk (&x)[TM], const typename OB::Chunk (&y)[TN]) {
        float a[TM][16], b[TN][16];
#pragma unroll
        for (int i = 0; i < TM; i++) oa[i].deliver(x[i], g, a[i]);
#pragma unroll
        for (int j = 0; j < TN; j++) ob[j].deliver(y[j], g, b[j]);
        mul(a, b);
      };
      if (c < full) {
        fetch(c, ca[0], cb[0]);
        for (; c + step < full; c += 2 * step) {
          fetch(c + step, ca[1], cb[1]);
          use(ca[0], cb[0]);
          if (c + 2 * step < full) fetch(c + 2 * step, ca[0], cb[0]);
          use(ca[1], cb[1]);
        }
        if (c < full) { use(ca[0], cb[0]); c += step; }
      }
    } else {
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
