// Softmax attention with everything in float32 on the matrix cores (v_mfma_f32_32x32x2_f32): the float32 configuration,
// and bfloat16 storage with head widths that the bf16 kernels do not take.  Head widths 16, 32, 64, 128.
//
// Transposed score tiles as in the bf16 kernels: in S^T[key, query] = K Q^T a lane owns one query, element e of the result
// is key (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3), and that is just what the second product wants as its operand: matrix
// instruction e contracts over the two keys that the two halves of the wave hold in element e.  So probabilities stay
// in the registers they were computed in, at full precision, and nothing goes through LDS: K (Q in the dK/dV kernel) is
// read 16 bytes of its own row per lane, V a row of 32 consecutive columns per half.
// A workgroup is 32 queries (keys) of one head and its 4 waves share the keys (queries) out, tile w, w + 4, ..; partial
// results meet in LDS in wave order.  These are short sequences of few heads, and what bounds them is one wave's chain:
// one workgroup per query on the vector units walked the keys twice, one fused multiply-add per loaded element.
// Forward, dQ, dK/dV: 251 tokens, 3 x 4 heads of 64, bfloat16 storage: 55, 51, 56 -> 13, 14, 22 us; 700 tokens, 4 heads of
// 128, float32: 262, 225, 232 -> 41, 61, 87.  dQ and dK/dV are one launch (251 tokens: 15 + 23 -> 24 us).
#include "kernels.h"

typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;

#define NW 4

__device__ __forceinline__ f32x4 load4(const float* p) { return *(const f32x4*)p; }
__device__ __forceinline__ f32x4 load4(const bf16* p) {
  const bf16x4 v = *(const bf16x4*)p;
  return f32x4{(float)v[0], (float)v[1], (float)v[2], (float)v[3]};
}
// this lane's half of a row as an operand of a product over the head width: columns 8 c + 4 (lane >> 5) .. + 3
template <class T, int DH> __device__ __forceinline__ void load_row(const T* row, int half, float scale, float (&r)[DH / 2]) {
#pragma unroll
  for (int c = 0; c < DH / 8; c++) {
    const f32x4 v = load4(row + c * 8 + half * 4);
#pragma unroll
    for (int i = 0; i < 4; i++) r[c * 4 + i] = v[i] * scale;
  }
}
template <class T, int DH> __device__ __forceinline__ f32x16 scores(const T* row, int half, const float (&r)[DH / 2]) {
  f32x16 a = {};
#pragma unroll
  for (int c = 0; c < DH / 8; c++) {
    const f32x4 v = load4(row + c * 8 + half * 4);
#pragma unroll
    for (int i = 0; i < 4; i++) a = __builtin_amdgcn_mfma_f32_32x32x2f32(v[i], r[c * 4 + i], a, 0, 0, 0);
  }
  return a;
}
__device__ __forceinline__ int elem_row(int e, int half) { return (e >> 2) * 8 + half * 4 + (e & 3); }
// acc^T[column, lane] += X^T[column, row] p[row, lane] over the 32 rows of X that start at r0 (rows past the last one are
// that one: p is zero there)
template <class T, int DH, int DT>
__device__ __forceinline__ void accumulate(f32x16 (&acc)[DT], const T* x, i64 ld, int r0, int last, const f32x16& p, int lane) {
  T v[16][DT];
#pragma unroll
  for (int e = 0; e < 16; e++) {
    const T* row = x + (i64)min(r0 + elem_row(e, lane >> 5), last) * ld + (lane & (DH < 32 ? DH - 1 : 31));
#pragma unroll
    for (int i = 0; i < DT; i++) v[e][i] = row[i * 32];
  }
  // all loads in flight before the first product: left to itself the compiler takes a few at a time as soon as registers
  // are short (128-wide dK/dV at 700 tokens 136 us, 87 like this)
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int e = 0; e < 16; e++)
#pragma unroll
    for (int i = 0; i < DT; i++) acc[i] = __builtin_amdgcn_mfma_f32_32x32x2f32((float)v[e][i], p[e], acc[i], 0, 0, 0);
}
// The same for a wave that starts over because its result was not finite (see finite), on a tile of which lanes see only
// the rows lo .. hi - 1 (p is zero in the others).  A value of X that is not finite enters the product as a zero, so that a
// lane that does not see it keeps the bits it has with any finite value; the lanes that see it then get p times it from the
// same instruction on counts: per result element the +infinities (in units of 1) and the -infinities (of 128) among those
// products, a NaN or an infinity times zero counting as both.
template <class T, int DH, int DT>
__device__ __forceinline__ void accumulate_apart(f32x16 (&acc)[DT], const T* x, i64 ld, int r0, int last, const f32x16& p, int lane,
                                                 int lo, int hi) {
#pragma unroll
  for (int i = 0; i < DT; i++) {
    f32x16 n = {};
#pragma unroll
    for (int e = 0; e < 16; e++) {
      if (e % 4 == 0) {                              // (a few loads at a time: this must not cost the other path registers)
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("" : "+v"(lane), "+v"(lo), "+v"(hi));
      }
      const int r = r0 + elem_row(e, lane >> 5);
      const float v = (float)x[(i64)min(r, last) * ld + (lane & (DH < 32 ? DH - 1 : 31)) + i * 32];
      const float up = v < INFINITY ? 0.f : 1.f, down = v > -INFINITY ? 0.f : 1.f;
      const bool sees = r >= lo && r < hi;
      acc[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(up + down > 0.f ? 0.f : v, p[e], acc[i], 0, 0, 0);
      n = __builtin_amdgcn_mfma_f32_32x32x2f32(up + 128.f * down, sees && !(p[e] < 0.f) ? 1.f : 0.f, n, 0, 0, 0);
      n = __builtin_amdgcn_mfma_f32_32x32x2f32(down + 128.f * up, sees && !(p[e] > 0.f) ? 1.f : 0.f, n, 0, 0, 0);
    }
#pragma unroll
    for (int e = 0; e < 16; e++) {
      const float down = floorf(n[e] * (1.f / 128.f));
      acc[i][e] += n[e] - 128.f * down > 0.f ? INFINITY : 0.f;
      acc[i][e] += down > 0.f ? -INFINITY : 0.f;
    }
  }
}
// On tiles that some lanes see only in part the matrix instruction multiplies the rest by their zero probabilities, and a
// value that is not finite would reach queries before it (keys after it).  That always shows in the result, so the tiles
// are multiplied plainly first (looking at every element on the way: 128-wide forward 46 -> 149 us at 700 tokens) and a
// wave whose result is not finite starts over, keeping such values apart.  It then has accumulators of its own: as a second
// value of the first ones they cost a short sequence 1-2 us of register moves in every call.
template <int DT> __device__ __forceinline__ bool finite(const f32x16 (&acc)[DT]) {
  float z[4] = {0.f, 0.f, 0.f, 0.f};                 // (a value that is not finite times zero is no number)
#pragma unroll
  for (int i = 0; i < DT; i++)
#pragma unroll
    for (int e = 0; e < 16; e++) z[e & 3] = __builtin_fmaf(acc[i][e], 0.f, z[e & 3]);
  return __all((z[0] + z[1]) + (z[2] + z[3]) == 0.f);
}
// the lane for the second pass, so that nothing of the first one is kept in registers for it
__device__ __forceinline__ int opaque(int lane) { asm volatile("" : "+v"(lane)); return lane; }
// a wave's accumulators to its LDS tile [32 rows][DH + 1] (row = lane & 31)
template <int DH, int DT> __device__ __forceinline__ void spill_tile(float* t, const f32x16 (&acc)[DT], int lane) {
#pragma unroll
  for (int i = 0; i < DT; i++)
#pragma unroll
    for (int e = 0; e < 16; e++) {
      const int c = i * 32 + elem_row(e, lane >> 5);
      if (DH >= 32 || c < DH) t[(lane & 31) * (DH + 1) + c] = acc[i][e];
    }
}
// sum of the waves' tiles, times scale, to rows r0 .. of out
template <class T, int DH> __device__ __forceinline__ void store_sum(const float* sm, T* out, i64 ld, int r0, int rows, float scale) {
  for (int i = threadIdx.x; i < 32 * DH; i += NW * 64) {
    const int r = i / DH, c = i % DH;
    if (r0 + r >= rows) return;
    float v = 0.f;
#pragma unroll
    for (int w = 0; w < NW; w++) v += sm[w * 32 * (DH + 1) + r * (DH + 1) + c];
    out[(i64)(r0 + r) * ld + c] = from_f<T>(v * scale);
  }
}

// A wave's share of the forward pass of 32 queries (a lane owns one; its keys are 0 .. seen - 1).  APART: see finite.
template <class T, int DH, bool APART, int DT>
__device__ __forceinline__ void fwd_keys(const T* k, const T* v, i64 ld, int S, int nt, int wv, int lane, int seen,
                                         const float (&qf)[DH / 2], f32x16 (&acc)[DT], float& m, float& l) {
  const int half = lane >> 5;
#pragma unroll
  for (int i = 0; i < DT; i++) acc[i] = f32x16{};
  m = -INFINITY;
  l = 0.f;
  for (int t = wv; t < nt; t += NW) {
    const int kv0 = t * 32;
    f32x16 s = scores<T, DH>(k + (i64)min(kv0 + (lane & 31), S - 1) * ld, half, qf);
    float mx = -INFINITY;
#pragma unroll
    for (int e = 0; e < 16; e++) {
      if (kv0 + elem_row(e, half) >= seen) s[e] = -INFINITY;
      mx = fmaxf(mx, s[e]);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 32, WAVE));
    const float mn = fmaxf(m, mx), ms = mn == -INFINITY ? 0.f : mn;
    float rs = 0.f;
#pragma unroll
    for (int e = 0; e < 16; e++) { s[e] = __expf(s[e] - ms); rs += s[e]; }
    rs += __shfl_xor(rs, 32, WAVE);
    const float alpha = __expf(m - ms);
    l = l * alpha + rs;
    m = mn;
#pragma unroll
    for (int i = 0; i < DT; i++) acc[i] *= alpha;
    if constexpr (APART) accumulate_apart<T, DH, DT>(acc, v, ld, kv0, S - 1, s, lane, 0, seen);
    else accumulate<T, DH, DT>(acc, v, ld, kv0, S - 1, s, lane);
  }
}
template <class T, int DH>
__global__ void __launch_bounds__(NW * 64) attn_fwd_f32_k(const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ v,
                                                          T* __restrict__ o, float* __restrict__ lse, int S, int H, int causal,
                                                          float scale, const unsigned char* __restrict__ row_skip) {
  constexpr int DT = DH < 32 ? 1 : DH / 32;
  extern __shared__ float sm[];                      // NW tiles [32][DH + 1], then m and l of each wave's queries
  float *sM = sm + NW * 32 * (DH + 1), *sL = sM + NW * 32;
  const int q0 = ((int)gridDim.x - 1 - (int)blockIdx.x) * 32, hh = blockIdx.y, b = blockIdx.z;    // long tiles first
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, half = lane >> 5, myq = q0 + (lane & 31);
  // every query of the tile is a finished row of the inverse's iteration: every wave looks at all of them
  if (row_skip && !__any(myq < S && row_skip[(i64)b * S + myq] == 0)) return;
  const i64 ld = (i64)H * DH, base = (i64)b * S * ld + (i64)hh * DH;
  float qf[DH / 2];
  load_row<T, DH>(q + base + (i64)min(myq, S - 1) * ld, half, scale, qf);
  const int nt = ((causal ? min(S, q0 + 32) : S) + 31) / 32;
  const int seen = causal ? min(S, myq + 1) : S;
  f32x16 acc[DT];
  float m, l;
  fwd_keys<T, DH, false>(k + base, v + base, ld, S, nt, wv, lane, seen, qf, acc, m, l);
  float* mine = sm + wv * 32 * (DH + 1);
  if (__builtin_expect(finite<DT>(acc), 1)) spill_tile<DH, DT>(mine, acc, lane);
  else {
    f32x16 again[DT];
    fwd_keys<T, DH, true>(k + base, v + base, ld, S, nt, wv, opaque(lane), seen, qf, again, m, l);
    spill_tile<DH, DT>(mine, again, lane);
  }
  if (half == 0) { sM[wv * 32 + lane] = m; sL[wv * 32 + lane] = l; }
  __syncthreads();
  for (int i = threadIdx.x; i < 32 * DH; i += NW * 64) {
    const int r = i / DH, c = i % DH;
    if (q0 + r >= S) return;
    float M = sM[r];
#pragma unroll
    for (int w = 1; w < NW; w++) M = fmaxf(M, sM[w * 32 + r]);
    const float Ms = M == -INFINITY ? 0.f : M;
    float a = 0.f, tot = 0.f;
#pragma unroll
    for (int w = 0; w < NW; w++) {
      const float f = __expf(sM[w * 32 + r] - Ms);
      a += f * sm[w * 32 * (DH + 1) + r * (DH + 1) + c];
      tot += f * sL[w * 32 + r];
    }
    o[base + (i64)(q0 + r) * ld + c] = from_f<T>(a * (1.0f / tot));
    if (c == 0) lse[((i64)b * H + hh) * S + q0 + r] = M + __logf(tot);
  }
}

// A wave's share of dQ of 32 queries: dS^T = P^T (dP^T - D), dP^T = V dO^T, dQ^T += K^T dS^T
template <class T, int DH, bool APART, int DT>
__device__ __forceinline__ void dq_keys(const T* k, const T* v, i64 ld, int S, int nt, int wv, int lane, int seen, float L, float D,
                                        const float (&qf)[DH / 2], const float (&dof)[DH / 2], f32x16 (&acc)[DT]) {
  const int half = lane >> 5;
#pragma unroll
  for (int i = 0; i < DT; i++) acc[i] = f32x16{};
  for (int t = wv; t < nt; t += NW) {
    const int kv0 = t * 32;
    const i64 row = (i64)min(kv0 + (lane & 31), S - 1) * ld;
    f32x16 s = scores<T, DH>(k + row, half, qf);
    const f32x16 dp = scores<T, DH>(v + row, half, dof);
#pragma unroll
    for (int e = 0; e < 16; e++) s[e] = kv0 + elem_row(e, half) >= seen ? 0.f : __expf(s[e] - L) * (dp[e] - D);
    if constexpr (APART) accumulate_apart<T, DH, DT>(acc, k, ld, kv0, S - 1, s, lane, 0, seen);
    else accumulate<T, DH, DT>(acc, k, ld, kv0, S - 1, s, lane);
  }
}
template <class T, int DH>
__device__ __forceinline__ void bwd_dq(float* sm, int tile, int hh, int b, const T* q, const T* k, const T* v, const T* d_o, const float* lse,
                                       const float* dvec, T* dq, int S, int H, int causal, float scale) {
  constexpr int DT = DH < 32 ? 1 : DH / 32;
  const int q0 = ((S + 31) / 32 - 1 - tile) * 32;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, half = lane >> 5, myq = q0 + (lane & 31), qc = min(myq, S - 1);
  const i64 ld = (i64)H * DH, base = (i64)b * S * ld + (i64)hh * DH, stat = ((i64)b * H + hh) * S;
  float qf[DH / 2], dof[DH / 2];
  load_row<T, DH>(q + base + (i64)qc * ld, half, scale, qf);
  load_row<T, DH>(d_o + base + (i64)qc * ld, half, 1.f, dof);
  const float L = lse[stat + qc], D = dvec[stat + qc];
  const int nt = ((causal ? min(S, q0 + 32) : S) + 31) / 32;
  const int seen = causal ? min(S, myq + 1) : S;
  f32x16 acc[DT];
  dq_keys<T, DH, false>(k + base, v + base, ld, S, nt, wv, lane, seen, L, D, qf, dof, acc);
  float* mine = sm + wv * 32 * (DH + 1);
  if (__builtin_expect(finite<DT>(acc), 1)) spill_tile<DH, DT>(mine, acc, lane);
  else {
    f32x16 again[DT];
    dq_keys<T, DH, true>(k + base, v + base, ld, S, nt, wv, opaque(lane), seen, L, D, qf, dof, again);
    spill_tile<DH, DT>(mine, again, lane);
  }
  __syncthreads();
  store_sum<T, DH>(sm, dq + base, ld, q0, S, scale);
}

// A wave's share of dK, dV of 32 keys (a lane owns one; its queries are first .. S - 1):
// S = Q K^T, dP = dO V^T, dV^T += dO^T P, dK^T += Q^T dS
template <class T, int DH, bool APART, int DT>
__device__ __forceinline__ void dkv_queries(const T* q, const T* d_o, const float* lse, const float* dvec, i64 ld, int S, int t_lo,
                                            int lane, int first, const float (&kf)[DH / 2], const float (&vf)[DH / 2],
                                            f32x16 (&dka)[DT], f32x16 (&dva)[DT]) {
  const int half = lane >> 5, nt = (S + 31) / 32;
#pragma unroll
  for (int i = 0; i < DT; i++) { dka[i] = f32x16{}; dva[i] = f32x16{}; }
  for (int t = t_lo; t < nt; t += NW) {
    const int q0 = t * 32;
    const i64 row = (i64)min(q0 + (lane & 31), S - 1) * ld;
    f32x16 s = scores<T, DH>(q + row, half, kf);
    f32x16 dp = scores<T, DH>(d_o + row, half, vf);
#pragma unroll
    for (int e = 0; e < 16; e++) {
      const int qq = q0 + elem_row(e, half), qs = min(qq, S - 1);
      const bool masked = qq >= S || qq < first;
      const float p = __expf(s[e] - lse[qs]);
      dp[e] = masked ? 0.f : p * (dp[e] - dvec[qs]);
      s[e] = masked ? 0.f : p;
    }
    if constexpr (APART) {
      accumulate_apart<T, DH, DT>(dva, d_o, ld, q0, S - 1, s, lane, first, S);
      accumulate_apart<T, DH, DT>(dka, q, ld, q0, S - 1, dp, lane, first, S);
    } else {
      accumulate<T, DH, DT>(dva, d_o, ld, q0, S - 1, s, lane);
      accumulate<T, DH, DT>(dka, q, ld, q0, S - 1, dp, lane);
    }
  }
}
template <class T, int DH>
__device__ __forceinline__ void bwd_dkv(float* sm, int tile, int hh, int b, const T* q, const T* k, const T* v, const T* d_o, const float* lse,
                                        const float* dvec, T* dk, T* dv, int S, int H, int causal, float scale) {
  constexpr int DT = DH < 32 ? 1 : DH / 32;
  const int k0 = tile * 32;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, half = lane >> 5, myk = k0 + (lane & 31), kc = min(myk, S - 1);
  const i64 ld = (i64)H * DH, base = (i64)b * S * ld + (i64)hh * DH, stat = ((i64)b * H + hh) * S;
  float kf[DH / 2], vf[DH / 2];
  load_row<T, DH>(k + base + (i64)kc * ld, half, scale, kf);
  load_row<T, DH>(v + base + (i64)kc * ld, half, 1.f, vf);
  const int first = causal ? myk : 0, t_lo = (causal ? k0 / 32 : 0) + wv;
  f32x16 dka[DT], dva[DT];
  dkv_queries<T, DH, false>(q + base, d_o + base, lse + stat, dvec + stat, ld, S, t_lo, lane, first, kf, vf, dka, dva);
  const bool as_is = finite<DT>(dva) && finite<DT>(dka);
  float* mine = sm + wv * 32 * (DH + 1);
  auto spill = [&](const f32x16 (&acc)[DT], bool keys) __attribute__((always_inline)) {
    if (__builtin_expect(as_is, 1)) spill_tile<DH, DT>(mine, acc, lane);
    else {
      f32x16 dka2[DT], dva2[DT];                     // (each time, so that the usual way holds no registers for it)
      dkv_queries<T, DH, true>(q + base, d_o + base, lse + stat, dvec + stat, ld, S, t_lo, opaque(lane), first, kf, vf, dka2, dva2);
      if (keys) spill_tile<DH, DT>(mine, dka2, lane);
      else spill_tile<DH, DT>(mine, dva2, lane);
    }
  };
  spill(dka, true);
  __syncthreads();
  store_sum<T, DH>(sm, dk + base, ld, k0, S, scale);
  __syncthreads();
  spill(dva, false);
  __syncthreads();
  store_sum<T, DH>(sm, dv + base, ld, k0, S, 1.f);
}

// Both in one launch, dK/dV of every batch, then dQ: neither fills the chip.  (Grid x: tiles, then heads; y, which a grid limits to
// 65536, is the batch alone.  dK/dV and dQ by turns of a batch: 8 x 200 tokens of 4 heads of 64 41 us instead of 36.)
template <class T, int DH>
__global__ void __launch_bounds__(NW * 64) attn_bwd_f32_k(const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ v,
                                                          const T* __restrict__ d_o, const float* __restrict__ lse,
                                                          const float* __restrict__ dvec, T* __restrict__ dq, T* __restrict__ dk,
                                                          T* __restrict__ dv, int S, int H, int causal, float scale) {
  extern __shared__ float sm[];
  const int tiles = (S + 31) / 32, hh = (int)blockIdx.x / tiles, tile = (int)blockIdx.x - hh * tiles, b = blockIdx.y;
  if (blockIdx.z == 0) bwd_dkv<T, DH>(sm, tile, hh, b, q, k, v, d_o, lse, dvec, dk, dv, S, H, causal, scale);
  else bwd_dq<T, DH>(sm, tile, hh, b, q, k, v, d_o, lse, dvec, dq, S, H, causal, scale);
}

// rows are read 4 elements at a time
static bool takes(int dt, int dh, const void* a, const void* b, const void* c, const void* d) {
  const uintptr_t mask = dt == 0 ? 15 : 7;
  return (dh == 16 || dh == 32 || dh == 64 || dh == 128) &&
         !(((uintptr_t)a | (uintptr_t)b | (uintptr_t)c | (uintptr_t)d) & mask);
}
template <class T, int DH>
static void fwd(const void* q, const void* k, const void* v, void* o, float* lse, int B, int S, int H, int causal,
                hipStream_t s, const unsigned char* row_skip) {
  constexpr size_t smem = (size_t)(NW * 32 * (DH + 1) + 2 * NW * 32) * 4;
  static std::atomic<unsigned long long> attr_mask{0};
  if (attr_needed(attr_mask)) {
    (void)hipFuncSetAttribute((const void*)attn_fwd_f32_k<T, DH>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    attr_done(attr_mask);
  }
  hipLaunchKernelGGL((attn_fwd_f32_k<T, DH>), dim3(cdiv(S, 32), H, B), dim3(NW * 64), smem, s, (const T*)q, (const T*)k,
                     (const T*)v, (T*)o, lse, S, H, causal, 1.0f / sqrtf((float)DH), row_skip);
}
template <class T, int DH>
static void bwd(const void* q, const void* k, const void* v, const void* d_o, const float* lse, const float* dvec, void* dq,
                void* dk, void* dv, int B, int S, int H, int causal, hipStream_t s) {
  constexpr size_t smem = (size_t)NW * 32 * (DH + 1) * 4;
  static std::atomic<unsigned long long> attr_mask{0};
  if (attr_needed(attr_mask)) {
    (void)hipFuncSetAttribute((const void*)attn_bwd_f32_k<T, DH>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    attr_done(attr_mask);
  }
  hipLaunchKernelGGL((attn_bwd_f32_k<T, DH>), dim3(cdiv(S, 32) * H, B, 2), dim3(NW * 64), smem, s, (const T*)q, (const T*)k, (const T*)v,
                     (const T*)d_o, lse, dvec, (T*)dq, (T*)dk, (T*)dv, S, H, causal, 1.0f / sqrtf((float)DH));
}

#define BY_WIDTH(T, call)                                  \
  switch (dh) {                                            \
    case 16: call(T, 16); break;                           \
    case 32: call(T, 32); break;                           \
    case 64: call(T, 64); break;                           \
    default: call(T, 128);                                 \
  }

int launch_attn_fwd_f32(int dt, const void* q, const void* k, const void* v, void* o, float* lse, int B, int S, int H, int dh,
                        int causal, hipStream_t s, const unsigned char* row_skip) {
  if (!takes(dt, dh, q, k, v, q)) return 1;
#define FWD(T, W) fwd<T, W>(q, k, v, o, lse, B, S, H, causal, s, row_skip)
  if (dt == 0) BY_WIDTH(float, FWD) else BY_WIDTH(bf16, FWD)
  return 0;
}
int launch_attn_bwd_f32(int dt, const void* q, const void* k, const void* v, const void* d_o, const float* lse,
                        const float* dvec, void* dq, void* dk, void* dv, int B, int S, int H, int dh, int causal, hipStream_t s) {
  if (!takes(dt, dh, q, k, v, d_o)) return 1;
#define BWD(T, W) bwd<T, W>(q, k, v, d_o, lse, dvec, dq, dk, dv, B, S, H, causal, s)
  if (dt == 0) BY_WIDTH(float, BWD) else BY_WIDTH(bf16, BWD)
  return 0;
}
