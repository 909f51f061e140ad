// Routing of the MoE half (MLP_pt of section 3.2 read as a Qwen2-MoE sparse block):
// router logits, softmax, top-k, per-expert offsets and the token permutation, the
// weighted combine, and the element-wise parts of their backward passes.
// Everything here is deterministic: integer results depend only on the logits' bits.
#include "kernels.h"
#include "operand_f32.h"
#include <initializer_list>

#define DISPATCH_DT(dt, ...)                                  \
  do {                                                        \
    if ((dt) == 0) { typedef float T; __VA_ARGS__; }          \
    else { typedef bf16 T; __VA_ARGS__; }                     \
  } while (0)

// ---------------------------------------------------------------------------------
// Router.  The logits are z = W_r (P_up_m Norm(Y1)) + b.  They are evaluated as
// (W_r P_up_m diag(gain)) Y1 / rms(Y1) with the product matrix wrp[E1, h] held in fp32 and applied to the stored Y1 with
// float32 products, so the selection depends only on the bits of Y1 and the weights, not on the rounding of the bf16
// intermediate P_up_m Norm(Y1).  Row E of wrp (optional) is the shared expert's gate vector folded the same way.
// Outputs: probs[T,E] (softmax over all experts), idx/wts[T,k] (slots by descending logit, equal logits -> lower expert
// index), gamma[T] = sigmoid(gate logit), and blk_cnt[block][E], how often the block's tokens chose each expert.
//
// One workgroup of 16 waves per block of 16 tokens.  The routing chain (this kernel, then the permutation) is latency:
// 2 MFLOP and the whole of wrp per workgroup.  The 16 x E1 logits are cut over the waves by column tile and by slices of
// h (the squares for 1/rms are summed from the same registers), added in slice order
// through LDS, and then a wave finishes one token with one lane per expert (reductions by data-parallel moves, the
// arg-max as maximum and ballot).  (32 tokens per workgroup: half the CUs, twice the matrix-core time on each.)
// ---------------------------------------------------------------------------------
#define ROUTER_TOKENS 16
#define ROUTER_WAVES 16
__host__ __device__ inline int router_slices(int tiles) { return tiles >= ROUTER_WAVES ? 1 : ROUTER_WAVES / tiles; }
// bytes of the logits, squares and counts (at most 20 KB), to a multiple of 16; the operand chunks of the waves follow
__host__ __device__ inline size_t router_lds(int E, int tiles, int ns) { return (((size_t)ns * 16 * (tiles * 16 + 1) + E) * 4 + 15) & ~(size_t)15; }

template <class T>
__global__ void __launch_bounds__(ROUTER_WAVES * 64) router_k(
    const T* __restrict__ y1, i64 ld, const float* __restrict__ wrp, const float* __restrict__ b_router,
    float* __restrict__ probs, int* __restrict__ idx, float* __restrict__ wts, float* __restrict__ gamma,
    int* __restrict__ blk_cnt, int Tn, int h, int E, int k, int has_gate, int norm_topk, float eps) {
  extern __shared__ __attribute__((aligned(16))) float sm[];
  const int E1 = E + (has_gate ? 1 : 0), tiles = (E1 + 15) >> 4, ns = router_slices(tiles), zc = tiles * 16;
  float* zpart = sm;                              // [ns][16][zc]: slice partials; slice 0 then takes the sums
  float* sspart = sm + ns * 16 * zc;              // [ns][16]
  int* cnt = (int*)(sspart + ns * 16);            // [E]
  typedef StagedOperand<T, 16> OA;
  typedef StagedOperand<float, 16> OB;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, gh = lane >> 4;
  const int t0 = blockIdx.x * ROUTER_TOKENS;
  char* lds = (char*)sm + router_lds(E, tiles, ns) + (size_t)wv * (OA::lds_bytes + OB::lds_bytes);     // the wave's operand chunks
  for (int e = threadIdx.x; e < E; e += blockDim.x) cnt[e] = 0;
  const int nchunk = (h + GKC(16) - 1) / GKC(16);
  for (int item = wv; item < tiles * ns; item += ROUTER_WAVES) {
    const int sl = item / tiles, tt = item - sl * tiles;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    float ss = 0.f;
    OA oa[1];
    OB ob[1];
    oa[0].init(y1, ld, t0, Tn, lane, lds);
    ob[0].init(wrp, h, tt * 16, E1, lane, lds + OA::lds_bytes);
    k_loop<16, 1, 1>(oa, ob, 0, h, sl, ns, nchunk, gh, [&](float (&a)[1][16], float (&b)[1][16]) {
#pragma unroll
      for (int s = 0; s < 16; s++) { acc = mfma_f32(a[0][s], b[0][s], acc); ss += a[0][s] * a[0][s]; }
    });
#pragma unroll
    for (int e = 0; e < 4; e++) zpart[(sl * 16 + gh * 4 + e) * zc + tt * 16 + (lane & 15)] = acc[e];
    ss += __shfl_xor(ss, 16, WAVE);
    ss += __shfl_xor(ss, 32, WAVE);
    if (tt == 0 && lane < 16) sspart[sl * 16 + lane] = ss;
  }
  __syncthreads();
  for (int e = threadIdx.x; e < 16 * zc; e += ROUTER_WAVES * 64) {       // the slices, added in order
    float v = 0.f;
#pragma unroll 4
    for (int s = 0; s < ns; s++) v += zpart[s * 16 * zc + e];
    zpart[e] = v;
  }
  __syncthreads();
  const int t = t0 + wv;                  // one token per wave
  if (t < Tn) {
    float ss = 0.f;
#pragma unroll 4
    for (int s = 0; s < ns; s++) ss += sspart[s * 16 + wv];
    const float r = 1.0f / sqrtf(ss / (float)h + eps);
    const float* zt = zpart + wv * zc;
    float z[4];                           // the logits of experts lane + 64 j (E <= 256)
    float mx = -INFINITY;
#pragma unroll
    for (int j = 0; j < 4; j++) {
      const int e = lane + 64 * j;
      z[j] = -INFINITY;
      if (e < E) { z[j] = zt[e] * r + (b_router ? b_router[e] : 0.f); mx = fmaxf(mx, z[j]); }
    }
    // softmax over the E routed logits
    mx = wave_max(mx);
    float p[4], sum = 0.f;
#pragma unroll
    for (int j = 0; j < 4; j++) { p[j] = lane + 64 * j < E ? __expf(z[j] - mx) : 0.f; sum += p[j]; }
    sum = wave_sum(sum);
    const float inv = 1.0f / sum;
#pragma unroll
    for (int j = 0; j < 4; j++) if (lane + 64 * j < E) probs[(i64)t * E + lane + 64 * j] = p[j] * inv;
    // top-k by k rounds of (value desc, index asc) arg-max over the experts not chosen yet.  A logit that is not a
    // number ranks as minus infinity, and a lane remembers which of its own experts are taken, so every round finds a
    // valid expert that no earlier round has chosen, whatever the logits hold: a token with a non-finite input cannot
    // disturb the tables of other tokens.
    float wsum = 0.f;
    float myw = 0.f;                      // lane s keeps the weight of slot s
    unsigned taken = 0;                   // bit j: expert lane + 64 j has been chosen
    for (int s = 0; s < k; s++) {
      float bv = -INFINITY;
#pragma unroll
      for (int j = 0; j < 4; j++) {
        const bool open = lane + 64 * j < E && !((taken >> j) & 1u);
        if (open && z[j] > bv) bv = z[j];             // (false for a NaN)
      }
      bv = wave_max(bv);
      int bi = -1;                                    // lowest index among the experts that hold the maximum
#pragma unroll
      for (int j = 0; j < 4; j++) {
        const bool open = lane + 64 * j < E && !((taken >> j) & 1u);
        const float v = (z[j] == z[j]) ? z[j] : -INFINITY;
        const unsigned long long m = __ballot(open && v == bv);
        if (bi < 0 && m) bi = 64 * j + __ffsll(m) - 1;
      }
      // (with top_k <= E at least one expert was left and the comparison is a total order, so one was found; the clamp
      // only guards the stores below)
      bi = min(max(bi, 0), E - 1);
      if ((bi & 63) == lane) taken |= 1u << (bi >> 6);
      const float pb = __expf(bv - mx) * inv;
      wsum += pb;
      if (lane == s) myw = pb;
      if (lane == 0) { idx[(i64)t * k + s] = bi; atomicAdd(&cnt[bi], 1); }
    }
    if (lane < k) wts[(i64)t * k + lane] = norm_topk ? myw / wsum : myw;
    if (has_gate && lane == 0) gamma[t] = sigmoid_f(zt[E] * r);
  }
  __syncthreads();
  for (int e = threadIdx.x; e < E; e += blockDim.x) blk_cnt[(i64)blockIdx.x * E + e] = cnt[e];
}

void launch_router(int dt, const void* y1, i64 ld, const float* wrp, const float* b_router, float* probs, int* idx,
                   float* wts, float* gamma, int* blk_cnt, int Tn, int h, int E, int k, int has_gate, int norm_topk,
                   float eps, hipStream_t s) {
  if (Tn <= 0) return;
  const int tiles = (E + (has_gate ? 1 : 0) + 15) / 16, ns = router_slices(tiles);
  const size_t smem = router_lds(E, tiles, ns) + (size_t)ROUTER_WAVES * 1024 * ((dt == 0 ? 4 : 2) + 4);
  static std::atomic<unsigned long long> attr_mask{0};
  if (attr_needed(attr_mask)) {
    (void)hipFuncSetAttribute((const void*)router_k<float>, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    (void)hipFuncSetAttribute((const void*)router_k<bf16>, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    attr_done(attr_mask);
  }
  DISPATCH_DT(dt, hipLaunchKernelGGL(router_k<T>, dim3(cdiv(Tn, ROUTER_TOKENS)), dim3(ROUTER_WAVES * 64), smem, s,
                                     (const T*)y1, ld, wrp, b_router, probs, idx, wts, gamma, blk_cnt, Tn, h, E, k,
                                     has_gate, norm_topk, eps));
}
size_t router_blocks(size_t Tn) { return (Tn + ROUTER_TOKENS - 1) / ROUTER_TOKENS; }

// ---------------------------------------------------------------------------------
// Permutation: a stable grouping of the T*k (token, slot) entries by expert.  The router kernel has counted, per block
// of 16 tokens, the entries of every expert, so a block's first row inside every expert is a column sum of that table
// and blocks need nothing of each other: one wave per block, 16 per workgroup, every workgroup adding the columns for
// itself (one workgroup that counted and placed all entries took 13.5 us at T = 2048 and 52 us at T = 8192; now 5 and
// 8 us).  Inside its block a wave hands out rows in entry order, which keeps (token, slot) order inside an expert.
// One more workgroup writes counts, offsets and the m-tile lists used by the grouped GEMMs: tile i covers rows
// [tile_m0[i], min(tile_m0[i]+bm, offsets[g+1])) of expert g = tile_group[i]; unused = -1.
// ---------------------------------------------------------------------------------
#define PERM_WAVES 16
__device__ __forceinline__ void same_expert_mask(int x, bool valid, int nbits, unsigned long long& same) {
  same = __ballot(valid);
  for (int b = 0; b < nbits; b++) {
    unsigned long long m = __ballot(valid && ((x >> b) & 1));
    same &= ((x >> b) & 1) ? m : ~m;
  }
}

__device__ __forceinline__ int wave_inclusive_scan(int v, int lane) {
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int u = __shfl_up(v, o, WAVE);
    if (lane >= o) v += u;
  }
  return v;
}
__device__ __forceinline__ int wave_sum(int v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, WAVE);
  return v;
}

__global__ void __launch_bounds__(PERM_WAVES * 64) permute_k(
    const int* __restrict__ idx, const int* __restrict__ blk_cnt, int nblk, int N, int k, int E, int epad,
    int* __restrict__ counts, int* __restrict__ offsets, int* __restrict__ row_map, int* __restrict__ inv_map,
    TileLists tl) {
  extern __shared__ int ism[];            // column sums [2][1024], next row of (wave, expert) [16][E], off[E + 1]
  int* csum = ism;
  int* next = ism + 2 * PERM_WAVES * 64;
  int* off = next + PERM_WAVES * E;
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int b0 = blockIdx.x * PERM_WAVES;           // first block of this workgroup (the last workgroup has none)
  // column sums: epad (E rounded up to a power of two) columns, 1024 / epad row lanes; those of one wave are added by
  // exchanges, so that at most 16 partial sums per column are left (with 8 experts 128 of them, read one after the other, were
  // 6 of the kernel's 10 us)
  const int cols = max(epad, 64);         // columns per row of the partial sums
  {
    const int e = threadIdx.x & (epad - 1), part = threadIdx.x / epad, parts = PERM_WAVES * 64 / epad;
    int all = 0, before = 0;
    if (e < E) {
#pragma unroll 8
      for (int b = part; b < nblk; b += parts) {
        const int c = blk_cnt[(i64)b * E + e];
        all += c;
        before += b < b0 ? c : 0;
      }
    }
    for (int o = epad; o < 64; o <<= 1) { all += __shfl_xor(all, o, WAVE); before += __shfl_xor(before, o, WAVE); }
    csum[threadIdx.x] = all;
    csum[PERM_WAVES * 64 + threadIdx.x] = before;
  }
  for (int i = threadIdx.x; i < PERM_WAVES * E; i += blockDim.x) next[i] = b0 + i / E < nblk ? blk_cnt[(i64)b0 * E + i] : 0;
  __syncthreads();
  if (threadIdx.x < E) {
    const int e = threadIdx.x;
    int all = 0, run = 0, c[PERM_WAVES];
#pragma unroll
    for (int i = 0; i < PERM_WAVES; i++) {
      const bool in = i * cols < PERM_WAVES * 64;
      all += in ? csum[i * cols + e] : 0;
      run += in ? csum[PERM_WAVES * 64 + i * cols + e] : 0;
    }
#pragma unroll
    for (int w = 0; w < PERM_WAVES; w++) c[w] = next[w * E + e];
    off[e + 1] = all;                     // totals for now
#pragma unroll
    for (int w = 0; w < PERM_WAVES; w++) { next[w * E + e] = run; run += c[w]; }
  }
  __syncthreads();
  if (wv == 0) {                          // offsets = prefix sums of the totals, 64 experts per step
    if (lane == 0) off[0] = 0;
    int carry = 0;
    for (int base = 0; base < E; base += 64) {
      const int e = base + lane;
      const int incl = carry + wave_inclusive_scan(e < E ? off[e + 1] : 0, lane);
      if (e < E) off[e + 1] = incl;
      carry = __shfl(incl, 63, WAVE);
    }
  }
  __syncthreads();
  if (blockIdx.x == gridDim.x - 1) {
    // Waves 0-2 write one tile list each, wave 3 the evenness flag, the others counts and offsets.
    if (wv < 3) {
      // tile lists: expert e owns the slots after the tiles of experts 0..e-1; slots past the last tile are marked
      // unused.  Every slot of the list is written: the fill loop runs over the count that the slots were numbered by.
      const int pass = wv;
      const int bm = tl.bm[pass], slack = tl.slack[pass], mx = tl.max_tiles[pass];
      int* tg = tl.group[pass];
      int* tm = tl.m0[pass];
      int* tf = tl.first[pass];
      int total = 0;
      for (int base = 0; base < E; base += 64) {
        const int e = base + lane;
        const int m_lo = e < E ? off[e] : 0, m_hi = e < E ? off[e + 1] : 0;
        const int mine = m_hi > m_lo ? max((m_hi - m_lo - slack + bm - 1) / bm, 1) : 0;
        const int incl = wave_inclusive_scan(mine, lane);
        const int first = total + incl - mine;
        int i = first;
        for (int m = m_lo; i < first + mine; m += bm, i++)
          if (i < mx) { tg[i] = e; tm[i] = m; tf[i] = (first << 16) | mine; }
        total += __shfl(incl, 63, WAVE);
      }
      for (int i = total + lane; i < mx; i += 64) { tg[i] = -1; tm[i] = 0; tf[i] = (i << 16) | 1; }
      if (lane == 0) tl.count[pass] = min(total, mx);
    } else if (wv == 3) {
      // Is the routing even enough for the per-expert weight-gradient launches to give each expert to two XCDs?  Then
      // experts e = 4 r + q (q = 0..3) are worked on by XCD pair q in round r, and the pairs finish together only if
      // their experts cost about the same: a tile costs a fixed part (first loads, stores: about 5 k-steps' worth) plus
      // one k-step per 64 rows of the expert.  Even = no pair more than 6 % above the mean.
      int cost[4] = {0, 0, 0, 0};
      for (int base = 0; base < E; base += 64) {
        const int e = base + lane;
        const int mine = e < E ? 5 + (off[e + 1] - off[e] + 63) / 64 : 0;
#pragma unroll
        for (int q = 0; q < 4; q++) cost[q] += wave_sum((e & 3) == q ? mine : 0);
      }
      const int tot = cost[0] + cost[1] + cost[2] + cost[3];
      const int mx = max(max(cost[0], cost[1]), max(cost[2], cost[3]));
      if (lane == 0) tl.count[3] = (E >= 8 && 400 * mx <= 106 * tot) ? 1 : 0;
    } else {
      for (int e = threadIdx.x - 256; e <= E; e += PERM_WAVES * 64 - 256) {
        offsets[e] = off[e];
        if (e < E) counts[e] = off[e + 1] - off[e];
      }
    }
    return;
  }
  if (b0 + wv >= nblk) return;            // whole wave; no barriers below
  const unsigned long long below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  int nbits = 0;
  while ((1 << nbits) < E) nbits++;
  int* mine = next + wv * E;
  const int lo = (b0 + wv) * ROUTER_TOKENS * k, hi = min(N, lo + ROUTER_TOKENS * k);
  for (int f0 = lo; f0 < hi; f0 += 64) {
    const int f = f0 + lane;
    const bool valid = f < hi;
    const int x = valid ? min(max(idx[f], 0), E - 1) : 0;    // an index outside [0, E) cannot reach the LDS tables
    unsigned long long same;
    same_expert_mask(x, valid, nbits, same);
    const int rank = __popcll(same & below);
    const int start = valid ? mine[x] : 0;  // every lane of a group reads before its leader updates
    __builtin_amdgcn_wave_barrier();
    if (valid && rank == 0) mine[x] = start + __popcll(same);
    __builtin_amdgcn_wave_barrier();
    if (valid) {
      const int pos = off[x] + start + rank;
      row_map[pos] = f;
      inv_map[f] = pos;
    }
  }
}

void launch_permute(const int* idx, const int* blk_cnt, int Tn, int k, int E, int* counts, int* offsets, int* row_map,
                    int* inv_map, const TileLists& tl, hipStream_t s) {
  const int nblk = (int)router_blocks(Tn);
  int epad = 1;
  while (epad < E) epad *= 2;
  const size_t smem = (size_t)(2 * PERM_WAVES * 64 + PERM_WAVES * E + E + 1) * sizeof(int);
  hipLaunchKernelGGL(permute_k, dim3(cdiv(nblk, PERM_WAVES) + 1), dim3(PERM_WAVES * 64), smem, s, idx, blk_cnt, nblk,
                     Tn * k, k, E, epad, counts, offsets, row_map, inv_map, tl);
}

// ---------------------------------------------------------------------------------
// Combine: rs[t] = sum_slot wts[t,slot] * yp[inv_map[t*k+slot]] + gamma[t] * ys[t], slots added
// in slot order (fixed order, no atomics).
// ---------------------------------------------------------------------------------
template <class T>
__global__ void __launch_bounds__(256) combine_k(const T* __restrict__ yp, const int* __restrict__ inv_map,
                                                 const float* __restrict__ wts, const T* __restrict__ ys,
                                                 const float* __restrict__ gamma, T* __restrict__ rs, int d, int k) {
  const int t = blockIdx.x;
  for (int c = threadIdx.x; c < d; c += 256) {
    float acc = 0.f;
    for (int s = 0; s < k; s++) {
      int pos = inv_map[(i64)t * k + s];
      acc += wts[(i64)t * k + s] * to_f(yp[(i64)pos * d + c]);
    }
    if (ys) acc += gamma[t] * to_f(ys[(i64)t * d + c]);
    rs[(i64)t * d + c] = from_f<T>(acc);
  }
}
// bf16, d % 8 == 0, 16-byte aligned rows: one lane handles 8 consecutive columns with 16-byte accesses
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
static bool vec8_ok(int dt, int d, std::initializer_list<const void*> ptrs) {
  if (dt != 1 || (d & 7)) return false;
  for (const void* q : ptrs) if ((uintptr_t)q & 15) return false;
  return true;
}
__global__ void __launch_bounds__(256) combine_v8_k(const bf16* __restrict__ yp, const int* __restrict__ inv_map,
                                                    const float* __restrict__ wts, const bf16* __restrict__ ys,
                                                    const float* __restrict__ gamma, bf16* __restrict__ rs, int d, int k) {
  const int t = blockIdx.x;
  for (int c = threadIdx.x * 8; c < d; c += 256 * 8) {
    float acc[8];
#pragma unroll
    for (int q = 0; q < 8; q++) acc[q] = 0.f;
    for (int s = 0; s < k; s++) {
      const int pos = inv_map[(i64)t * k + s];
      const float w = wts[(i64)t * k + s];
      const bf16x8_t v = *(const bf16x8_t*)(yp + (i64)pos * d + c);
#pragma unroll
      for (int q = 0; q < 8; q++) acc[q] += w * (float)v[q];
    }
    if (ys) {
      const float g = gamma[t];
      const bf16x8_t v = *(const bf16x8_t*)(ys + (i64)t * d + c);
#pragma unroll
      for (int q = 0; q < 8; q++) acc[q] += g * (float)v[q];
    }
    bf16x8_t o;
#pragma unroll
    for (int q = 0; q < 8; q++) o[q] = (__bf16)acc[q];
    *(bf16x8_t*)(rs + (i64)t * d + c) = o;
  }
}
void launch_combine(int dt, const void* yp, const int* inv_map, const float* wts, const void* ys,
                    const float* gamma, void* rs, int Tn, int d, int k, hipStream_t s) {
  if (Tn <= 0) return;
  if (vec8_ok(dt, d, {yp, ys, rs})) {
    hipLaunchKernelGGL(combine_v8_k, dim3(Tn), dim3(256), 0, s, (const bf16*)yp, inv_map, wts, (const bf16*)ys, gamma,
                       (bf16*)rs, d, k);
    return;
  }
  DISPATCH_DT(dt, hipLaunchKernelGGL(combine_k<T>, dim3(Tn), dim3(256), 0, s, (const T*)yp, inv_map, wts,
                                     (const T*)ys, gamma, (T*)rs, d, k));
}

// Combine in the half-width space of the streams (pre-merged down projections: expert outputs already have width h)
// with the coupling update of Eq. 2 / the first line of the inverse in the same pass:
//   branch[t] = sum_slot wts[t,slot] * yp[inv_map[t*k+slot]] + gamma[t] * ys[t]      (slot order, fp32)
//   dst[t] = resid[t] + sign * branch[t]   (rounded once to the stream type); tap (optional) keeps branch in fp32.
template <class T, class TS>
__global__ void __launch_bounds__(256) combine_couple_k(const T* __restrict__ yp, const int* __restrict__ inv_map,
                                                        const float* __restrict__ wts, const T* __restrict__ ys,
                                                        const float* __restrict__ gamma, const TS* resid, i64 ldr,
                                                        float sign, TS* dst, i64 ldd, float* __restrict__ tap, int h, int k) {
  const int t = blockIdx.x;
  for (int c = threadIdx.x; c < h; c += 256) {
    float acc = 0.f;
    for (int s = 0; s < k; s++) {
      int pos = inv_map[(i64)t * k + s];
      acc += wts[(i64)t * k + s] * to_f(yp[(i64)pos * h + c]);
    }
    if (ys) acc += gamma[t] * to_f(ys[(i64)t * h + c]);
    if (tap) tap[(i64)t * h + c] = acc;
    dst[(i64)t * ldd + c] = from_f<TS>(to_f(resid[(i64)t * ldr + c]) + sign * acc);   // (dst may be resid: same element)
  }
}
// bf16 branch, rows of whole groups of 4 on 8-byte (stream: 4-element) boundaries: a thread handles 4 columns, a workgroup of 256
// a row 1024 wide in one go, and the rows of all slots are asked for before the first is used (37 tokens: 10.6 -> 5.3 us, which
// were four dependent rounds of 2-byte loads)
#define COUPLE_SLOTS 4
template <class TS>
__global__ void __launch_bounds__(256) combine_couple_v4_k(const bf16* __restrict__ yp, const int* __restrict__ inv_map,
                                                           const float* __restrict__ wts, const bf16* __restrict__ ys,
                                                           const float* __restrict__ gamma, const TS* resid, i64 ldr,
                                                           float sign, TS* dst, i64 ldd, float* __restrict__ tap, int h, int k) {
  typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4_t;
  typedef __attribute__((ext_vector_type(4))) TS ts4;
  const int t = blockIdx.x;
  for (int c = threadIdx.x * 4; c < h; c += 1024) {
    const ts4 x = *(const ts4*)(resid + (i64)t * ldr + c);
    bf16x4_t y = {};
    if (ys) y = *(const bf16x4_t*)(ys + (i64)t * h + c);
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    for (int s0 = 0; s0 < k; s0 += COUPLE_SLOTS) {
      bf16x4_t v[COUPLE_SLOTS];
      float w[COUPLE_SLOTS];
#pragma unroll
      for (int s = 0; s < COUPLE_SLOTS; s++) {
        const int slot = min(s0 + s, k - 1);
        v[s] = *(const bf16x4_t*)(yp + (i64)inv_map[(i64)t * k + slot] * h + c);
        w[s] = wts[(i64)t * k + slot];
      }
#pragma unroll
      for (int s = 0; s < COUPLE_SLOTS; s++)
        if (s0 + s < k)
#pragma unroll
          for (int q = 0; q < 4; q++) acc[q] += w[s] * (float)v[s][q];
    }
    if (ys) {
      const float gm = gamma[t];
#pragma unroll
      for (int q = 0; q < 4; q++) acc[q] += gm * (float)y[q];
    }
    ts4 o;
#pragma unroll
    for (int q = 0; q < 4; q++) o[q] = (TS)((float)x[q] + sign * acc[q]);
    if (tap) *(float4*)(tap + (i64)t * h + c) = make_float4(acc[0], acc[1], acc[2], acc[3]);
    *(ts4*)(dst + (i64)t * ldd + c) = o;             // (dst may be resid: same elements)
  }
}
void launch_combine_couple(int dt, int ts, const void* yp, const int* inv_map, const float* wts, const void* ys,
                           const float* gamma, const void* resid, i64 ldr, float sign, void* dst, i64 ldd, float* tap,
                           int Tn, int h, int k, hipStream_t s) {
  if (Tn <= 0) return;
  const uintptr_t at = (uintptr_t)yp | (uintptr_t)ys, st = (uintptr_t)resid | (uintptr_t)dst;
  if (dt == 1 && !(h & 3) && !(at & 7) && !(st & (ts == 0 ? 15 : 7)) && !((ldr | ldd) & 3) && !((uintptr_t)tap & 15)) {
    if (ts == 0)
      hipLaunchKernelGGL((combine_couple_v4_k<float>), dim3(Tn), dim3(256), 0, s, (const bf16*)yp, inv_map, wts, (const bf16*)ys, gamma,
                         (const float*)resid, ldr, sign, (float*)dst, ldd, tap, h, k);
    else
      hipLaunchKernelGGL((combine_couple_v4_k<bf16>), dim3(Tn), dim3(256), 0, s, (const bf16*)yp, inv_map, wts, (const bf16*)ys, gamma,
                         (const bf16*)resid, ldr, sign, (bf16*)dst, ldd, tap, h, k);
    return;
  }
  if (dt == 0)
    hipLaunchKernelGGL((combine_couple_k<float, float>), dim3(Tn), dim3(256), 0, s, (const float*)yp, inv_map, wts,
                       (const float*)ys, gamma, (const float*)resid, ldr, sign, (float*)dst, ldd, tap, h, k);
  else if (ts == 0)
    hipLaunchKernelGGL((combine_couple_k<bf16, float>), dim3(Tn), dim3(256), 0, s, (const bf16*)yp, inv_map, wts,
                       (const bf16*)ys, gamma, (const float*)resid, ldr, sign, (float*)dst, ldd, tap, h, k);
  else
    hipLaunchKernelGGL((combine_couple_k<bf16, bf16>), dim3(Tn), dim3(256), 0, s, (const bf16*)yp, inv_map, wts,
                       (const bf16*)ys, gamma, (const bf16*)resid, ldr, sign, (bf16*)dst, ldd, tap, h, k);
}

// ---------------------------------------------------------------------------------
// Backward of the combine and of the routing weights, one workgroup per token:
//   dgamma = <drs, ys>, gate-logit gradient dzext[t,E] = dgamma*gamma*(1-gamma), dys = gamma*drs
//   dw[slot] = <drs, yp[pos]>,  dyp[pos] = wts[t,slot]*drs
// and, once a token's dw are known, softmax + top-k weights (the selection itself carries no gradient):
//   dp_sel = dw                      (or (dw - sum dw*w) / sum_sel p with renormalisation)
//   dz_j   = p_j * ([j selected] dp_j - sum_sel dp_e p_e)        for every expert j
// (a kernel of its own for the second part, and one that stacks the router rows for the GEMM that follows, were 5 us each of
// every step at any size: both are latency)
// gather.um != null: the token's row of Um goes to its experts' rows of gather.xg on the way (the operand of the gate/up weight
// gradient).  As a kernel of its own that was 3 us of the chain in small calls; from 2048 tokens on, where it ran on a helper stream, a
// step takes the same either way (this kernel 20.6 -> 28 us at 2048 tokens, 66 -> 94 at 8192, the other 16 and 50).  Bound by the rows of
// k slots, read once and written twice.  With the token's own rows read anew for every slot: 32 and 101 us.
// ---------------------------------------------------------------------------------
// dz of one token by one wave, lanes over the experts; my_dw: dw of slot `lane`, sgate: dz of the gate logit
__device__ __forceinline__ void router_bwd_token(const RouterBwd& r, const float* wts, float my_dw, float sgate, float* dzext,
                                                 int t, int k, int E1, int lane) {
  const int E = r.E;
  const float* p = r.probs + (i64)t * E;
  // slot s lives in lane s (k <= 16); sums over the slots run in slot order on every lane
  const int my_sel = lane < k ? r.idx[(i64)t * k + lane] : -1;
  const float my_w = lane < k ? wts[(i64)t * k + lane] : 0.f;
  const float my_p = lane < k ? p[my_sel] : 0.f;
  float ssum = 0.f, dww = 0.f;
  for (int s = 0; s < k; s++) { ssum += __shfl(my_p, s, WAVE); dww += __shfl(my_dw, s, WAVE) * __shfl(my_w, s, WAVE); }
  const float my_dp = r.norm_topk ? (my_dw - dww) / ssum : my_dw;
  float inner = 0.f;
  for (int s = 0; s < k; s++) inner += __shfl(my_dp, s, WAVE) * __shfl(my_p, s, WAVE);
  bf16* dzb = (bf16*)r.dzb;
  for (int j0 = 0; j0 < E; j0 += 64) {               // (every lane takes part in the exchanges)
    const int j = j0 + lane;
    float dp = 0.f;
    for (int s = 0; s < k; s++) { const int sel = __shfl(my_sel, s, WAVE); const float v = __shfl(my_dp, s, WAVE); if (sel == j) dp = v; }
    if (j < E) {
      const float dz = p[j] * (dp - inner);
      dzext[(i64)t * E1 + j] = dz;
      if (dzb) dzb[(i64)t * r.E1p + j] = (bf16)dz;
    }
  }
  // the remaining columns of the bf16 copy: the shared-gate column, zeros
  if (dzb)
    for (int j = E + lane; j < r.E1p; j += 64) dzb[(i64)t * r.E1p + j] = j < E1 ? (bf16)sgate : (bf16)0.f;
}
template <class T>
__global__ void __launch_bounds__(256) moe_bwd_rows_k(const T* __restrict__ drs, const T* __restrict__ yp,
                                                      const T* __restrict__ ys, const int* __restrict__ inv_map,
                                                      const float* __restrict__ wts, const float* __restrict__ gamma,
                                                      T* __restrict__ dyp, T* __restrict__ dys,
                                                      float* __restrict__ dzext, int Tn, int d, int k, int E1, int has_gate,
                                                      RouterBwd r, RowCopy copy, RowGather gather) {
  __shared__ float red[4];
  const int t = blockIdx.x;
  if (t >= Tn) {
    const int row = t - Tn;
    const T* sp = row < copy.rows_a ? (const T*)copy.src_a + (i64)row * d : (const T*)copy.src_b + (i64)(row - copy.rows_a) * d;
    for (int c = threadIdx.x; c < d; c += 256) ((T*)copy.dst)[(i64)row * d + c] = sp[c];
    return;
  }
  const T* dr = drs + (i64)t * d;
  float gate = 0.f;
  if (has_gate) {
    float g = gamma[t];
    float acc = 0.f;
    for (int c = threadIdx.x; c < d; c += 256) {
      float v = to_f(dr[c]);
      acc += v * to_f(ys[(i64)t * d + c]);
      dys[(i64)t * d + c] = from_f<T>(g * v);
    }
    gate = block_sum_256(acc, red) * g * (1.f - g);
    if (threadIdx.x == 0) dzext[(i64)t * E1 + (E1 - 1)] = gate;
  }
  float my_dw = 0.f;                      // dw of slot threadIdx.x (k <= 16)
  for (int s = 0; s < k; s++) {
    int pos = inv_map[(i64)t * k + s];
    float w = wts[(i64)t * k + s];
    float acc = 0.f;
    for (int c = threadIdx.x; c < d; c += 256) {
      float v = to_f(dr[c]);
      acc += v * to_f(yp[(i64)pos * d + c]);
      dyp[(i64)pos * d + c] = from_f<T>(w * v);
      if (gather.um) ((T*)gather.xg)[(i64)pos * d + c] = ((const T*)gather.um)[(i64)t * d + c];
    }
    acc = block_sum_256(acc, red);
    if ((int)threadIdx.x == s) my_dw = acc;
  }
  if (threadIdx.x < 64) router_bwd_token(r, wts, my_dw, gate, dzext, t, k, E1, threadIdx.x);
}
__global__ void __launch_bounds__(256) moe_bwd_rows_v8_k(const bf16* __restrict__ drs, const bf16* __restrict__ yp,
                                                         const bf16* __restrict__ ys, const int* __restrict__ inv_map,
                                                         const float* __restrict__ wts, const float* __restrict__ gamma,
                                                         bf16* __restrict__ dyp, bf16* __restrict__ dys,
                                                         float* __restrict__ dzext, int Tn, int d, int k,
                                                         int E1, int has_gate, RouterBwd r, RowCopy copy, int copy8, RowGather gather) {
  __shared__ float red[4];
  const int t = blockIdx.x;
  if (t >= Tn) {
    const int row = t - Tn;
    const bf16* sp = row < copy.rows_a ? (const bf16*)copy.src_a + (i64)row * d : (const bf16*)copy.src_b + (i64)(row - copy.rows_a) * d;
    bf16* dp = (bf16*)copy.dst + (i64)row * d;
    if (copy8) for (int c = threadIdx.x * 8; c < d; c += 256 * 8) *(bf16x8_t*)(dp + c) = *(const bf16x8_t*)(sp + c);
    else for (int c = threadIdx.x; c < d; c += 256) dp[c] = sp[c];
    return;
  }
  // this thread's first piece of the token's two rows, which up to 2048 wide is all of them, is read once for all slots
  const bf16 *dr = drs + (i64)t * d, *um = (const bf16*)gather.um + (i64)t * d;
  const int c0 = threadIdx.x * 8;
  bf16x8_t dr0 = {}, um0 = {};
  if (c0 < d) {
    dr0 = *(const bf16x8_t*)(dr + c0);
    if (gather.um) um0 = *(const bf16x8_t*)(um + c0);
  }
  float gate = 0.f;
  if (has_gate) {
    const float g = gamma[t];
    float acc = 0.f;
    for (int c = c0; c < d; c += 256 * 8) {
      const bf16x8_t v = c == c0 ? dr0 : *(const bf16x8_t*)(dr + c), y = *(const bf16x8_t*)(ys + (i64)t * d + c);
      bf16x8_t o;
#pragma unroll
      for (int q = 0; q < 8; q++) { acc += (float)v[q] * (float)y[q]; o[q] = (__bf16)(g * (float)v[q]); }
      *(bf16x8_t*)(dys + (i64)t * d + c) = o;
    }
    gate = block_sum_256(acc, red) * g * (1.f - g);
    if (threadIdx.x == 0) dzext[(i64)t * E1 + (E1 - 1)] = gate;
  }
  float my_dw = 0.f;                      // dw of slot threadIdx.x (k <= 16)
  for (int s = 0; s < k; s++) {
    const int pos = inv_map[(i64)t * k + s];
    const float w = wts[(i64)t * k + s];
    float acc = 0.f;
    for (int c = c0; c < d; c += 256 * 8) {
      const bf16x8_t v = c == c0 ? dr0 : *(const bf16x8_t*)(dr + c), y = *(const bf16x8_t*)(yp + (i64)pos * d + c);
      bf16x8_t o;
#pragma unroll
      for (int q = 0; q < 8; q++) { acc += (float)v[q] * (float)y[q]; o[q] = (__bf16)(w * (float)v[q]); }
      *(bf16x8_t*)(dyp + (i64)pos * d + c) = o;
      if (gather.um) *(bf16x8_t*)((bf16*)gather.xg + (i64)pos * d + c) = c == c0 ? um0 : *(const bf16x8_t*)(um + c);
    }
    acc = block_sum_256(acc, red);
    if ((int)threadIdx.x == s) my_dw = acc;
  }
  if (threadIdx.x < 64) router_bwd_token(r, wts, my_dw, gate, dzext, t, k, E1, threadIdx.x);
}
void launch_moe_bwd_rows(int dt, const void* drs, const void* yp, const void* ys, const int* inv_map,
                         const float* wts, const float* gamma, void* dyp, void* dys, float* dzext, int Tn, int d,
                         int k, int E1, int has_gate, const RouterBwd& r, const RowCopy& copy, const RowGather& gather, hipStream_t s) {
  if (Tn <= 0) return;
  const dim3 grid(Tn + copy.rows_a + copy.rows_b);
  if (vec8_ok(dt, d, {drs, yp, ys, dyp, dys, gather.um, gather.xg})) {          // (buffers of the workspace; the copied rows are the caller's weights)
    hipLaunchKernelGGL(moe_bwd_rows_v8_k, grid, dim3(256), 0, s, (const bf16*)drs, (const bf16*)yp, (const bf16*)ys,
                       inv_map, wts, gamma, (bf16*)dyp, (bf16*)dys, dzext, Tn, d, k, E1, has_gate, r, copy,
                       (int)vec8_ok(dt, d, {copy.src_a, copy.src_b, copy.dst}), gather);
    return;
  }
  DISPATCH_DT(dt, hipLaunchKernelGGL(moe_bwd_rows_k<T>, grid, dim3(256), 0, s, (const T*)drs, (const T*)yp,
                                     (const T*)ys, inv_map, wts, gamma, (T*)dyp, (T*)dys, dzext, Tn, d, k, E1,
                                     has_gate, r, copy, gather));
}

// ---------------------------------------------------------------------------------
// Gradient at the MoE input Um, all three sources added in a fixed order:
//   dum[t] = dum_sh[t] (shared expert) + sum_slot dxg[pos(t,slot)] (routed experts)
//          + sum_e dzext[t,e] * Wext[e]    (router rows, then the shared gate row)
// ---------------------------------------------------------------------------------
// dum[t] = dum_sh[t] + sum_slot dxg[pos(t,slot)] + router term, where the router term is either the
// precomputed dum_r[t] (bf16 path: a k = E1 GEMM on the matrix cores) or, when dum_r is null, is
// accumulated here from dzext and the router / shared-gate rows.
template <class T>
__global__ void __launch_bounds__(256) dum_finalize_k(const T* __restrict__ dxg, const int* __restrict__ inv_map,
                                                      const T* __restrict__ dum_sh, const T* __restrict__ dum_r,
                                                      const float* __restrict__ dzext,
                                                      const T* __restrict__ w_router, const T* __restrict__ ws_gate,
                                                      T* __restrict__ dum, int d, int k, int E, int E1) {
  extern __shared__ float dzs[];
  const int t = blockIdx.x;
  if (!dum_r) {
    for (int e = threadIdx.x; e < E1; e += 256) dzs[e] = dzext[(i64)t * E1 + e];
    __syncthreads();
  }
  for (int c = threadIdx.x; c < d; c += 256) {
    float acc = dum_sh ? to_f(dum_sh[(i64)t * d + c]) : 0.f;
    for (int s = 0; s < k; s++) acc += to_f(dxg[(i64)inv_map[(i64)t * k + s] * d + c]);
    if (dum_r) {
      acc += to_f(dum_r[(i64)t * d + c]);
    } else {
      for (int e = 0; e < E; e++) acc += dzs[e] * to_f(w_router[(i64)e * d + c]);
      if (E1 > E) acc += dzs[E] * to_f(ws_gate[c]);
    }
    dum[(i64)t * d + c] = from_f<T>(acc);
  }
}
__global__ void __launch_bounds__(256) dum_finalize_v8_k(const bf16* __restrict__ dxg, const int* __restrict__ inv_map,
                                                         const bf16* __restrict__ dum_sh, const bf16* __restrict__ dum_r,
                                                         bf16* __restrict__ dum, int d, int k) {
  const int t = blockIdx.x;
  for (int c = threadIdx.x * 8; c < d; c += 256 * 8) {
    float acc[8];
#pragma unroll
    for (int q = 0; q < 8; q++) acc[q] = 0.f;
    if (dum_sh) {
      const bf16x8_t v = *(const bf16x8_t*)(dum_sh + (i64)t * d + c);
#pragma unroll
      for (int q = 0; q < 8; q++) acc[q] = (float)v[q];
    }
    for (int s = 0; s < k; s++) {
      const bf16x8_t v = *(const bf16x8_t*)(dxg + (i64)inv_map[(i64)t * k + s] * d + c);
#pragma unroll
      for (int q = 0; q < 8; q++) acc[q] += (float)v[q];
    }
    const bf16x8_t r = *(const bf16x8_t*)(dum_r + (i64)t * d + c);
    bf16x8_t o;
#pragma unroll
    for (int q = 0; q < 8; q++) o[q] = (__bf16)(acc[q] + (float)r[q]);
    *(bf16x8_t*)(dum + (i64)t * d + c) = o;
  }
}
void launch_dum_finalize(int dt, const void* dxg, const int* inv_map, const void* dum_sh, const void* dum_r,
                         const float* dzext, const void* w_router, const void* ws_gate, void* dum, int Tn, int d,
                         int k, int E, int E1, hipStream_t s) {
  if (Tn <= 0) return;
  if (dum_r && vec8_ok(dt, d, {dxg, dum_sh, dum_r, dum})) {
    hipLaunchKernelGGL(dum_finalize_v8_k, dim3(Tn), dim3(256), 0, s, (const bf16*)dxg, inv_map, (const bf16*)dum_sh,
                       (const bf16*)dum_r, (bf16*)dum, d, k);
    return;
  }
  DISPATCH_DT(dt, hipLaunchKernelGGL(dum_finalize_k<T>, dim3(Tn), dim3(256), E1 * sizeof(float), s, (const T*)dxg,
                                     inv_map, (const T*)dum_sh, (const T*)dum_r, dzext, (const T*)w_router,
                                     (const T*)ws_gate, (T*)dum, d, k, E, E1));
}

