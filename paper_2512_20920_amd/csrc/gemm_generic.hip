// GEMM with float32 products on the matrix cores (v_mfma_f32_32x32x2_f32: every operand element enters as float32,
// bf16 ones exactly), for any shape and any of the operand layouts of GemmArgs.  It serves the float32 configuration,
// whose tolerance needs float32 products, two GEMMs around the router (folded router matrix, router weight gradient), and
// every bf16 problem whose shape the bf16 kernels do not take.
//
// These problems are small (one to a few hundred 32x32 tiles), so what bounds them is latency, not the matrix pipe: a
// workgroup owns one tile of 32 TM x 32 TN outputs and cuts the contraction among its waves (wave w takes the chunks of
// 32 k's w, w + NW, ...) and the partial tiles are added in wave order through LDS.  Inside a workgroup no two waves want the
// same element, so every wave brings its own.  Aligned float32 operands go straight into LDS of the wave (f32_tile_staged:
// whole chunks in flight, no registers, no barrier before the end); everything else goes from memory (L2) into the operand
// registers, one chunk ahead.  What a small launch is made of is its place in the chain, 3 to 5 us, so the SwiGLU formulas,
// the norm in front of a projection and the rotation behind it are part of the GEMMs (EPI), and several problems of one
// kind are one launch.  At T = 400, d = 512 (float32) a GEMM of 400 x 512 x 512 takes 4 us where the LDS-tiled vector
// kernel that it replaced took 64 us (56 workgroups, one dependent load -> LDS -> barrier chain per 16 k's).
#include "lds_load.h"
#include "operand_f32.h"
#include <type_traits>

// waves that share a contraction of k: one per chunk, at most `most`
__host__ __device__ inline int f32_k_waves(int k, int R, int most) {
  int nw = 1;
  while (nw < most && k > GKC(R) * nw) nw *= 2;
  return nw;
}

// ACT: a gate/up GEMM (32x32 tiles): columns 0-15 of a tile are gate columns n0 .., 16-31 the up columns of the same indices
// (32 of each: fewer, larger workgroups, 19 us instead of 14 for 300 tiles of k = 512)
// End of a tile: the waves' partial tiles are added and go through the epilogue.
// bx: the column tile.  EPI_NORM: sq is this lane's share of the squares of row lane & 31; x, gain, nout: the rows, the gains and
// where the normalised rows go (may be null).  The contraction has run over x g, and 1 / rms scales its sums.
template <class TC, class TS, int R, int TM, int TN, int EPI, class Acc>
__device__ __forceinline__ void f32_finish(const GemmArgs& g, TC* C, const TS* bias, float* part, const Acc (&acc)[TM][TN], int parts, int wv,
                                           int lane, int m0, int m_end, int n0, int bx = 0, float sq = 0.f, const float* x = nullptr,
                                           const float* gain = nullptr, float* nout = nullptr) {
  constexpr bool ACT = EPI & EPI_ACT, ROPE = EPI & EPI_ROPE, NORM = EPI & EPI_NORM;
  constexpr int BM = R * TM, BN = R * TN, EL = R * R / 64;   // (EL elements of a tile per lane)
  // ---- partial tiles to LDS, added in wave order by all threads, then the epilogue on whole output rows
  if (wv < parts) {
    float* mine = part + wv * (BM * BN);
#pragma unroll
    for (int i = 0; i < TM; i++)
#pragma unroll
      for (int j = 0; j < TN; j++)
#pragma unroll
        for (int e = 0; e < EL; e++) mine[(i * R + acc_row<R>(lane, e)) * BN + j * R + (lane & (R - 1))] = acc[i][j][e];
  }
  float* rows = part + parts * (BM * BN);            // NORM: the waves' squares per row
  if constexpr (NORM) {
    sq += __shfl_xor(sq, 32, WAVE);
    if (wv < parts && lane < 32) rows[wv * 32 + lane] = sq;
  }
  __syncthreads();
  auto rms_inv = [&](int r) {
    float q = 0.f;
    for (int w = 0; w < parts; w++) q += rows[w * 32 + r];
    return 1.0f / sqrtf(q / (float)g.K + g.norm_eps);
  };
  if constexpr (NORM)
    if (nout) {                                      // the column tiles of these rows share the normalised rows out
      const int items = 32 * (g.K >> 2), per = (items + (int)gridDim.x - 1) / (int)gridDim.x, end = min(items, (bx + 1) * per);
      for (int i = bx * per + (int)threadIdx.x; i < end; i += (int)blockDim.x) {
        const int r = i & 31, k = (i >> 5) * 4, m = m0 + r;
        if (m >= m_end) continue;
        const float4 v = *(const float4*)(x + (i64)m * g.lda + k), gv = *(const float4*)(gain + k);
        const float ri = rms_inv(r);
        *(float4*)(nout + (i64)m * g.K + k) = make_float4(v.x * ri * gv.x, v.y * ri * gv.y, v.z * ri * gv.z, v.w * ri * gv.w);
      }
    }
  constexpr int EPT = BM * BN / 256;                 // elements per thread
  float v[EPT];
#pragma unroll
  for (int u = 0; u < EPT; u++) v[u] = 0.f;
  if (threadIdx.x >= 256) return;
#pragma unroll 2
  for (int w = 0; w < parts; w++)
#pragma unroll
    for (int u = 0; u < EPT; u++) v[u] += part[w * (BM * BN) + threadIdx.x + u * 256];
  const TS* resid = (const TS*)g.resid;
  const TS* cscale = (const TS*)g.col_scale;
  if constexpr (NORM)
#pragma unroll
    for (int u = 0; u < EPT; u++) v[u] *= rms_inv((threadIdx.x + u * 256) / BN);
  if constexpr (ROPE) {
#pragma unroll
    for (int u = 0; u < EPT; u++) {
      const int e = threadIdx.x + u * 256, c = e % BN, m = m0 + e / BN, n = rope_tile_col(bx, c, g.rope_dh), step = g.rope_dh == 16 ? 8 : 16;
      const float own = v[u] + (bias ? to_f(bias[n]) : 0.f), other = __shfl_xor(own, step, WAVE);
      if (m >= m_end) continue;
      const bool turn = (g.rope_mask >> blockIdx.z) & 1;
      const float2 cs = turn ? ((const float2*)g.rope_cs)[(i64)(m % g.rope_S) * (g.rope_dh / 2) + (n & (g.rope_dh / 2 - 1))] : make_float2(1.f, 0.f);
      C[(i64)m * g.ldc + n] = from_f<TC>(turn ? rope_value(own, other, c & step, cs) : own);
    }
    return;
  }
  if constexpr (ACT) {                               // silu(gate) * up from the stored values, as the separate kernel
#pragma unroll
    for (int u = 0; u < EPT; u++) {
      const int e = threadIdx.x + u * 256, c = e % BN, m = m0 + e / BN, n = n0 + (c & 15);
      const TC x = from_f<TC>(v[u]);
      const float up = __shfl(to_f(x), lane | 16, WAVE);           // (a row's 32 values are in one half of a wave)
      if (m >= m_end || n >= g.act_half) continue;
      C[(i64)m * g.ldc + (c >> 4) * g.act_half + n] = x;
      if (c < 16) ((TC*)g.act_out)[(i64)m * g.ldact + n] = from_f<TC>(to_f(x) * sigmoid_f(to_f(x)) * up);
    }
    return;
  }
  if (g.dact_out) {                                  // SwiGLU's backward, from what C would have held
    const TS* gu = (const TS*)g.dact_gu;
    float ga[EPT], ua[EPT];
#pragma unroll
    for (int u = 0; u < EPT; u++) {
      const int e = threadIdx.x + u * 256, m = min(m0 + e / BN, m_end - 1), n = min(n0 + e % BN, g.N - 1);
      ga[u] = to_f(gu[(i64)m * 2 * g.N + n]);
      ua[u] = to_f(gu[(i64)m * 2 * g.N + g.N + n]);
    }
#pragma unroll
    for (int u = 0; u < EPT; u++) {
      const int e = threadIdx.x + u * 256, m = m0 + e / BN, n = n0 + e % BN;
      if (m >= m_end || n >= g.N) continue;
      float dg, du;
      swiglu_grad(to_f(from_f<TC>(v[u])), ga[u], ua[u], &dg, &du);
      TC* o = (TC*)g.dact_out + (i64)m * 2 * g.N + n;
      o[0] = from_f<TC>(dg);
      o[g.N] = from_f<TC>(du);
    }
    return;
  }
  // (loads of all elements first, from clamped positions, so that they are in flight together)
  float sc[EPT], bi[EPT], rs[EPT];
#pragma unroll
  for (int u = 0; u < EPT; u++) {
    const int e = threadIdx.x + u * 256, m = min(m0 + e / BN, m_end - 1), n = min(n0 + e % BN, g.N - 1);
    sc[u] = cscale ? to_f(cscale[n]) : 1.f;
    bi[u] = bias ? to_f(bias[n]) : 0.f;
    rs[u] = resid ? (g.resid_f32 ? ((const float*)g.resid)[(i64)m * g.ldr + n] : to_f(resid[(i64)m * g.ldr + n])) : 0.f;
  }
#pragma unroll
  for (int u = 0; u < EPT; u++) {
    const int e = threadIdx.x + u * 256, m = m0 + e / BN, n = n0 + e % BN;
    if (m >= m_end || n >= g.N) continue;
    const float x = v[u] * sc[u] + bi[u];
    if (g.tap) g.tap[(i64)m * g.ldtap + n] = x;
    TC* crow = g.c_last_row && m == g.M - 1 ? (TC*)g.c_last_row : C + (i64)m * g.ldc;
    crow[n] = from_f<TC>(resid ? rs[u] + g.resid_sign * x : x);
  }
}

template <class TA, class TB, class TC, class TS, bool AT, bool BT, int R, int TM, int TN, bool ACT>
__device__ __forceinline__ void f32_tile(const GemmArgs& g, const TA* A, const TB* Bm, TC* C, const TS* bias, int m0, int m_end,
                                         int n0, int k0, int k_end, int nw, const TA* A2, const TB* B2) {
  extern __shared__ __attribute__((aligned(16))) float part[];      // [waves][R TM][R TN]
  constexpr int EL = R * R / 64;
  const int lane = threadIdx.x & 63, gh = lane / R, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  typename AccOf<R>::type acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; i++)
#pragma unroll
    for (int j = 0; j < TN; j++)
#pragma unroll
      for (int e = 0; e < EL; e++) acc[i][j][e] = 0.f;
  const int nchunk = (k_end - k0 + GKC(R) - 1) / GKC(R), all = A2 ? 2 * nchunk : nchunk;
  const int parts = min(nw, max(all, 1));
  // this wave's chunks of one pair of operands; the second pair goes on dealing where the first ended
  auto contract = [&](const TA* pa, const TB* pb, int first) {
    if (wv >= nw || first >= nchunk) return;
    Operand<TA, AT, R> oa[TM];
    Operand<TB, BT, R> ob[TN];
#pragma unroll
    for (int i = 0; i < TM; i++) oa[i].init(pa, g.lda, m0 + R * i, m_end, lane, g.a_gather, g.gather_div, k0, (const TA*)g.a_last_row);
#pragma unroll
    for (int j = 0; j < TN; j++) {
      if (ACT) { const int up = (lane >> 4) & 1; ob[j].init(pb, g.ldb, up * (g.act_half - 16) + n0, (up + 1) * g.act_half, lane, nullptr, 1, k0); }
      else ob[j].init(pb, g.ldb, n0 + R * j, g.N, lane, nullptr, 1, k0);
    }
    k_loop<R, TM, TN>(oa, ob, k0, k_end, first, nw, nchunk, gh, [&](float (&a)[TM][16], float (&b)[TN][16]) {
#pragma unroll
      for (int s = 0; s < 16; s++)
#pragma unroll
        for (int i = 0; i < TM; i++)
#pragma unroll
          for (int j = 0; j < TN; j++) acc[i][j] = mfma_f32(a[i][s], b[j][s], acc[i][j]);
    });
  };
  contract(A, Bm, wv);
  if (A2) contract(A2, B2, (wv + nw - nchunk % nw) % nw);
  f32_finish<TC, TS, R, TM, TN, ACT ? EPI_ACT : 0>(g, C, bias, part, acc, parts, wv, lane, m0, m_end, n0);
}

// The same for float32 operands on 16-byte boundaries (see staged_ok): a wave's pieces of 32 k's go straight into LDS that no
// other wave touches, one piece in flight while the one before it is multiplied.  Loaded into registers by the lane that needs
// them, the 4 k's of a row that runs along k put every lane on a cache line of its own, which a CU's waves then fetch
// several times over (QKV of 400 tokens, d = 512: 21 us).
//  * operand with k along memory: 128-byte rows, 16-byte chunk c of row r in slot c ^ ((r >> 1) & 7);
//  * operand stored k x rows: 32 rows of 128 bytes, k in row k ^ ((k >> 2) & 1), so that the two k's (4 apart) that the halves of
//    a wave read at a time lie in different halves of the banks.
#define STAGE_F32(EPI) (8192u + ((EPI) & EPI_NORM ? 256u : 0u))     // A, B, gains
template <bool TR> struct StagedF32 {
  u32x4 d;
  unsigned off[4];
  int kc[4];                // k of this lane's share of wave-load i, relative to the piece
  unsigned ks;              // bytes per k
  // act_half > 0: see ACT; rope_dh > 0: rows in the order of rope_tile_col, tile bx
  __device__ __forceinline__ void init(const float* p, i64 ld, int r0, int r_end, int lane, const int* gather, int div, int act_half = 0,
                                       int rope_dh = 0, int bx = 0) {
    d = make_desc(p);
    const unsigned ldb = (unsigned)ld * 4u;
    ks = TR ? ldb : 4u;
#pragma unroll
    for (int i = 0; i < 4; i++) {
      if (!TR) {
        const int r = i * 8 + (lane >> 3), ch = (lane & 7) ^ ((r >> 1) & 7);
        const int row = act_half ? (r >> 4) * act_half + min(r0 + (r & 15), act_half - 1) : rope_dh ? rope_tile_col(bx, r, rope_dh) : min(r0 + r, r_end - 1);
        kc[i] = ch * 4;
        off[i] = (unsigned)(gather ? gather[row] / div : row) * ldb + (unsigned)ch * 16u;
      } else {
        const int slot = i * 8 + (lane >> 3), col = r0 + (lane & 7) * 4;
        kc[i] = slot ^ ((slot >> 2) & 1);
        off[i] = col < r_end ? (unsigned)kc[i] * ldb + (unsigned)col * 4u : OOB;
      }
    }
  }
  __device__ __forceinline__ void issue(unsigned lds, int k0, int k_end) const {
#pragma unroll
    for (int i = 0; i < 4; i++)
      load_lds_b128(d, __builtin_amdgcn_readfirstlane(lds + i * 1024u), k0 + kc[i] < k_end && off[i] != OOB ? off[i] + (unsigned)k0 * ks : OOB);
  }
  // what the lane feeds to the 16 steps: step 4 j + i takes k = 8 j + 4 (lane >> 5) + i
  __device__ __forceinline__ static void read(const unsigned char* t, int lane, float (&v)[16]) {
    const int half = lane >> 5, r = lane & 31;
#pragma unroll
    for (int j = 0; j < 4; j++) {
      if (!TR) {
        const float4 x = *(const float4*)(t + r * 128 + ((2 * j + half) ^ ((r >> 1) & 7)) * 16);
        v[4 * j] = x.x; v[4 * j + 1] = x.y; v[4 * j + 2] = x.z; v[4 * j + 3] = x.w;
      } else
#pragma unroll
        for (int i = 0; i < 4; i++) v[4 * j + i] = *(const float*)(t + ((8 * j + 4 * half + i) ^ half) * 128 + r * 4);
    }
  }
};
template <bool AT, bool BT, int EPI>
__device__ __forceinline__ void f32_tile_staged(const GemmArgs& g, const float* A, const float* Bm, float* C, const float* bias, int m0, int m_end,
                                                int n0, int k0, int k_end, int nw, const float* A2, const float* B2, int bx = 0,
                                                const float* gain = nullptr, float* nout = nullptr) {
  constexpr bool ACT = EPI & EPI_ACT, ROPE = EPI & EPI_ROPE, NORM = EPI & EPI_NORM;
  constexpr unsigned STAGE = STAGE_F32(EPI);
  extern __shared__ __attribute__((aligned(1024))) float part[];    // the waves' pieces, then their partial tiles
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  f32x16 acc[1][1] = {};
  float sq = 0.f;
  const int nchunk = (k_end - k0 + 31) / 32, all = A2 ? 2 * nchunk : nchunk;
  const int parts = min(nw, max(all, 1));
  unsigned char* mine = (unsigned char*)part + wv * STAGE;
  const unsigned lds = lds_address(part) + (unsigned)wv * STAGE;
  StagedF32<AT> oa;
  StagedF32<BT> ob;
  const bool work = wv < parts && all > 0;
  const u32x4 dg = make_desc(NORM ? gain : A);
  auto issue = [&](int c) {                          // (a piece of the second pair of operands: the same offsets)
    if (A2 && c >= nchunk) { oa.d = make_desc(A2); ob.d = make_desc(B2); c -= nchunk; }
    oa.issue(lds, k0 + c * 32, k_end);
    ob.issue(lds + 4096u, k0 + c * 32, k_end);
    if constexpr (NORM) load_lds_b32(dg, __builtin_amdgcn_readfirstlane(lds + 8192u), c * 32 + lane < k_end ? (unsigned)(c * 32 + lane) * 4u : OOB);
  };
  if (work) {
    oa.init(A, g.lda, m0, m_end, lane, AT ? nullptr : g.a_gather, g.gather_div);
    ob.init(Bm, g.ldb, n0, g.N, lane, nullptr, 1, ACT ? g.act_half : 0, ROPE ? g.rope_dh : 0, bx);
    issue(wv);
  }
  if (work)
    for (int c = wv; c < all; c += nw) {
      wait_vmcnt<0>();
      float a[16], b[16];
      StagedF32<AT>::read(mine, lane, a);
      StagedF32<BT>::read(mine + 4096, lane, b);
      if constexpr (NORM) {
#pragma unroll
        for (int j = 0; j < 4; j++) {
          const float4 gv = *(const float4*)(mine + 8192 + (8 * j + 4 * (lane >> 5)) * 4);
          const float gq[4] = {gv.x, gv.y, gv.z, gv.w};
#pragma unroll
          for (int i = 0; i < 4; i++) { sq += a[4 * j + i] * a[4 * j + i]; a[4 * j + i] *= gq[i]; }
        }
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");            // the piece is in registers: its place is free
      __builtin_amdgcn_sched_barrier(0);
      if (c + nw < all) issue(c + nw);
#pragma unroll
      for (int s = 0; s < 16; s++) acc[0][0] = mfma_f32(a[s], b[s], acc[0][0]);
    }
  __syncthreads();                                   // the partial tiles overlay the pieces
  f32_finish<float, float, 32, 1, 1, EPI>(g, C, bias, part, acc, parts, wv, lane, m0, m_end, n0, bx, sq, A, gain, nout);
}

template <class TA, class TB, class TC, class TS, bool AT, bool BT, int R, int TM, int TN, int EPI, bool STG>
__global__ void __launch_bounds__(R == 16 ? 1024 : 512) gemm_f32_k(GemmArgs g) {
  constexpr bool ACT = EPI & EPI_ACT;
  constexpr int BM = R * TM, BN = ACT ? 16 : R * TN;
  const TA *A = (const TA*)g.A, *A2 = (const TA*)g.A2;
  const TB *Bm = (const TB*)g.B, *B2 = (const TB*)g.B2;
  TC* C = (TC*)g.C;
  const TS* bias = (const TS*)g.bias;
  int m0, m_end, k0 = 0, k_end = g.K;
  if (g.group_mode == 1) {
    const int grp = g.tile_group[blockIdx.y];
    if (grp < 0) return;
    m0 = g.tile_m0[blockIdx.y];
    m_end = min(g.offsets[grp + 1], m0 + BM);
    Bm += (i64)grp * g.b_group_stride;
  } else {
    m0 = blockIdx.y * BM;
    m_end = g.M;
    if (g.group_mode == 2) {
      const int grp = blockIdx.z;
      k0 = g.offsets[grp];
      k_end = g.offsets[grp + 1];
      C += (i64)grp * g.c_group_stride;
    } else {                                         // one of several problems of one shape launched together
      if (blockIdx.z > 0) A2 = nullptr;
      if (blockIdx.z == 1) { A = (const TA*)g.subA[0]; Bm = (const TB*)g.subB[0]; C = (TC*)g.subC[0]; bias = (const TS*)g.subBias[0]; }
      if (blockIdx.z == 2) { A = (const TA*)g.subA[1]; Bm = (const TB*)g.subB[1]; C = (TC*)g.subC[1]; bias = (const TS*)g.subBias[1]; }
    }
  }
  if (g.row_skip && g.group_mode == 0) {             // nothing to do if every row of the tile is marked as finished
    int live = 0;                                    // every wave checks all rows of the tile: same answer, no LDS
    for (int r = m0 + (int)(threadIdx.x & 63); r < min(m_end, m0 + BM); r += 64) live |= g.row_skip[r] == 0;
    if (!__any(live)) return;
  }
  if constexpr (STG) {
    const float* gain = (const float*)(blockIdx.z == 0 ? g.norm_g[0] : blockIdx.z == 1 ? g.norm_g[1] : g.norm_g[2]);
    float* nout = (float*)(blockIdx.z == 0 ? g.norm_out[0] : blockIdx.z == 1 ? g.norm_out[1] : g.norm_out[2]);
    f32_tile_staged<AT, BT, EPI>(g, A, Bm, C, bias, m0, m_end, blockIdx.x * BN, k0, k_end, g.k_waves, A2, B2, blockIdx.x, gain, nout);
  }
  else f32_tile<TA, TB, TC, TS, AT, BT, R, TM, TN, ACT>(g, A, Bm, C, bias, m0, m_end, blockIdx.x * BN, k0, k_end, g.k_waves, A2, B2);
}

// The weight gradients of several dense layers as one launch, tiles numbered over the problems: alone each is a launch of one
// to a few hundred workgroups that mostly wait for their loads (ten of them at 400 tokens, d = 512: 95 us, together 48).  The sum is
// cut as in a launch of its own, so the bits are the same.
__host__ __device__ inline int batch_waves(int K, int groups) { return f32_k_waves(groups ? (K + groups - 1) / groups : K, 32, 8); }      // (as go())
template <bool STG>
__global__ void __launch_bounds__(512) gemm_f32_batch_tn_k(GemmBatch b) {
  typedef const __attribute__((address_space(4))) GemmBatch* KernArg;     // (indexed in the kernel-argument segment)
  const KernArg ka = (KernArg)__builtin_amdgcn_kernarg_segment_ptr();
  int i = 0;
  while (i + 1 < ka->n && (int)blockIdx.x >= ka->p[i + 1].tile0) i++;
  const int per = ka->p[i].tiles_m * ka->p[i].tiles_n, grp = ((int)blockIdx.x - ka->p[i].tile0) / per;
  const int local = (int)blockIdx.x - ka->p[i].tile0 - grp * per, by = local / ka->p[i].tiles_n, bx = local - by * ka->p[i].tiles_n;
  GemmArgs g;
  g.M = ka->p[i].M; g.N = ka->p[i].N; g.K = ka->p[i].K;
  g.lda = ka->p[i].lda; g.ldb = ka->p[i].ldb; g.ldc = ka->p[i].ldc;
  const float *A = (const float*)ka->p[i].A, *B = (const float*)ka->p[i].B;
  float* C = (float*)ka->p[i].C + (i64)grp * ka->p[i].c_stride;
  const int groups = ka->p[i].groups, nw = batch_waves(g.K, groups);
  const int k0 = groups ? ka->offsets[grp] : 0, k_end = groups ? ka->offsets[grp + 1] : g.K;
  if constexpr (STG) f32_tile_staged<true, true, 0>(g, A, B, C, nullptr, by * 32, g.M, bx * 32, k0, k_end, nw, nullptr, nullptr);
  else f32_tile<float, float, float, float, true, true, 32, 1, 1, false>(g, A, B, C, nullptr, by * 32, g.M, bx * 32, k0, k_end, nw, nullptr, nullptr);
}

template <class TA, class TB, class TC, class TS, bool AT, bool BT, int R, int TM, int TN, int EPI = 0, bool STG = false>
static void go_shape(const GemmArgs& g, int nw, hipStream_t s) {
  const int gy = g.group_mode == 1 ? g.max_tiles : cdiv(g.M, R * TM);
  const dim3 grid(EPI & EPI_ACT ? cdiv(g.act_half, 16) : cdiv(g.N, R * TN), gy, g.group_mode == 2 ? g.n_groups : g.group_mode == 0 ? g.n_sub : 1);
  if (grid.x == 0 || grid.y == 0 || grid.z == 0) return;
  const size_t smem = (size_t)nw * (STG ? STAGE_F32(EPI) : (R * TM) * (R * TN) * sizeof(float));
  static std::atomic<unsigned long long> attr_mask{0};
  if (smem >= 65536 && attr_needed(attr_mask)) {
    (void)hipFuncSetAttribute((const void*)gemm_f32_k<TA, TB, TC, TS, AT, BT, R, TM, TN, EPI, STG>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, STG ? 8 * STAGE_F32(EPI) : 8 * 4096 * TM * TN);
    attr_done(attr_mask);
  }
  GemmArgs a = g;
  a.k_waves = nw;
  hipLaunchKernelGGL((gemm_f32_k<TA, TB, TC, TS, AT, BT, R, TM, TN, EPI, STG>), grid, dim3(64 * (nw > 4 ? nw : 4)), smem, s, a);
}

// whether f32_tile_staged takes the problem: loads of 4 elements inside the operands, which span less than 2 GiB
static bool quads(const void* p, i64 ld, i64 rows, i64 inner) {
  return !((uintptr_t)p & 15) && !(ld & 3) && !(inner & 3) && rows * ld < (i64)1 << 29;
}
static bool staged_ok(const GemmArgs& g) {
  if (g.group_mode == 2 ? g.K <= 0 : g.M <= 0) return false;
  if (g.a_last_row || (g.a_trans && g.a_gather)) return false;
  auto a_ok = [&](const void* p) { return g.a_trans ? quads(p, g.lda, g.K, g.M) : quads(p, g.lda, g.M, g.K); };
  auto b_ok = [&](const void* p) { return g.b_trans ? quads(p, g.ldb, g.K, g.N) : quads(p, g.ldb, g.N, g.K); };
  if (!a_ok(g.A) || !b_ok(g.B) || (g.b_group_stride & 3) || (g.act_half & 3)) return false;
  if (g.A2 && (!a_ok(g.A2) || !b_ok(g.B2))) return false;
  for (int z = 1; z < g.n_sub; z++)
    if (!a_ok(g.subA[z - 1]) || !b_ok(g.subB[z - 1])) return false;
  return true;
}

template <class TA, class TB, class TC, class TS, bool AT, bool BT>
static void go(const GemmArgs& g, hipStream_t s) {
  // One wave per chunk of k, at most 8 (of a workgroup of at least 4: the epilogue wants the threads).  The cut depends
  // on k alone, so that a result has the same bits whatever else is in the launch (a product over 2 T rows and one over
  // T rows, say).  Operands that go straight into LDS are faster on 32x32 tiles at every size (us, so / 64x32 from registers:
  // 1024 x 1024 x 512 16 / 23, 2048 x 2048 x 2048 167 / 233, 4096 x 4096 x 2048 674 / 913; a step of 2048 tokens, 1024 wide,
  // 3171 / 3719).  The others take 64x32 tiles (a quarter less operand traffic per product) where they alone are 16 waves per
  // CU, else 32x32.  small_tiles (the caller's choice, since it changes the order of the sum): 16x16 tiles and up to 16 waves, for
  // the few dozen rows of the router matrices, whose 32x32 tiles would leave most CUs idle.
  const int krange = (g.group_mode == 2 ? cdiv(g.K, g.n_groups) : g.K) * (g.A2 ? 2 : 1);    // (per expert: the mean)
  if (g.small_tiles && g.group_mode == 0) {
    go_shape<TA, TB, TC, TS, AT, BT, 16, 1, 1>(g, f32_k_waves(krange, 16, 16), s);
    return;
  }
  const int nw = f32_k_waves(krange, 32, 8);
  if constexpr (std::is_same<TA, float>::value && std::is_same<TB, float>::value && !(AT && !BT))
    if (staged_ok(g)) {
      if constexpr (!AT && !BT)
      {
        if (g.act_half) { go_shape<TA, TB, TC, TS, AT, BT, 32, 1, 1, EPI_ACT, true>(g, nw, s); return; }
        if (g.norm_g[0]) { go_shape<TA, TB, TC, TS, AT, BT, 32, 1, 1, EPI_NORM, true>(g, nw, s); return; }
        if (g.rope_cs) { go_shape<TA, TB, TC, TS, AT, BT, 32, 1, 1, EPI_ROPE, true>(g, nw, s); return; }
      }
      go_shape<TA, TB, TC, TS, AT, BT, 32, 1, 1, 0, true>(g, nw, s);
      return;
    }
  if constexpr (!AT && !BT)
    if (g.act_half) { go_shape<TA, TB, TC, TS, AT, BT, 32, 1, 1, EPI_ACT>(g, nw, s); return; }
  const i64 z = g.group_mode == 2 ? g.n_groups : 1;
  if (g.group_mode != 1 && (i64)cdiv(g.M, 64) * cdiv(g.N, 32) * z * nw >= 4096) go_shape<TA, TB, TC, TS, AT, BT, 32, 2, 1>(g, nw, s);
  else go_shape<TA, TB, TC, TS, AT, BT, 32, 1, 1>(g, nw, s);
}

template <class TA, class TB, class TC, class TS>
static void go_types(const GemmArgs& g, hipStream_t s) {
  if (g.a_trans) { if (g.b_trans) go<TA, TB, TC, TS, true, true>(g, s); else go<TA, TB, TC, TS, true, false>(g, s); }
  else { if (g.b_trans) go<TA, TB, TC, TS, false, true>(g, s); else go<TA, TB, TC, TS, false, false>(g, s); }
}

int launch_gemm_generic(const GemmArgs& g, GemmTypes t, hipStream_t s) {
  if (g.group_mode == 1 && g.tile_bm != 32) return -1;
  if (g.act_half && (g.a_trans || g.b_trans || g.group_mode == 2 || g.bias || g.resid || g.tap || g.N != 2 * g.act_half)) return -1;
  if (g.norm_g[0] || g.rope_cs) {
    // norm or rotation: the staged float32 form only, with nothing else in the epilogue (and not both: no caller has that)
    if (t.ta || t.tb || t.tc || t.tside || g.a_trans || g.b_trans || g.act_half || g.dact_out || g.resid || g.tap || g.A2 || g.group_mode ||
        g.col_scale || (g.norm_g[0] && g.rope_cs) || !staged_ok(g))
      return -1;
    if (g.rope_cs && !rope_fits(g.rope_dh, g.N)) return -1;
    for (int z = 0; g.norm_g[0] && z < g.n_sub; z++)
      if (!g.norm_g[z] || ((uintptr_t)g.norm_g[z] & 15) || ((uintptr_t)g.norm_out[z] & 15)) return -1;
  }
  int key = t.ta * 8 + t.tb * 4 + t.tc * 2 + t.tside;
  switch (key) {
    case 0: go_types<float, float, float, float>(g, s); break;            // fp32 everything
    case 15: go_types<bf16, bf16, bf16, bf16>(g, s); break;               // bf16 everything
    case 13: go_types<bf16, bf16, float, bf16>(g, s); break;              // bf16 in, fp32 out (router fold)
    case 7: go_types<float, bf16, bf16, bf16>(g, s); break;               // fp32 A (router logit gradients), bf16 B/C
    case 5: go_types<float, bf16, float, bf16>(g, s); break;              // router weight gradient in float32
    default: return -1;
  }
  return 0;
}

int launch_gemm_f32_batch_tn(GemmBatch& b, hipStream_t s) {
  b.total = 0;
  int nw = 1;
  for (int i = 0; i < b.n; i++) {
    GemmProb& p = b.p[i];
    p.tile0 = b.total; p.tiles_m = cdiv(p.M, 32); p.tiles_n = cdiv(p.N, 32);
    b.total += p.tiles_m * p.tiles_n * (p.groups ? p.groups : 1);
    const int w = batch_waves(p.K, p.groups);
    if (w > nw) nw = w;
  }
  if (b.total <= 0) return 0;
  bool stg = true;
  for (int i = 0; i < b.n; i++) stg = stg && quads(b.p[i].A, b.p[i].lda, b.p[i].K, b.p[i].M) && quads(b.p[i].B, b.p[i].ldb, b.p[i].K, b.p[i].N);
  const dim3 block(64 * (nw > 4 ? nw : 4));
  if (stg) {
    static std::atomic<unsigned long long> attr_mask{0};
    if (attr_needed(attr_mask)) {
      (void)hipFuncSetAttribute((const void*)gemm_f32_batch_tn_k<true>, hipFuncAttributeMaxDynamicSharedMemorySize, 8 * 8192);
      attr_done(attr_mask);
    }
    hipLaunchKernelGGL(gemm_f32_batch_tn_k<true>, dim3(b.total), block, (size_t)nw * 8192, s, b);
  } else {
    hipLaunchKernelGGL(gemm_f32_batch_tn_k<false>, dim3(b.total), block, (size_t)nw * 4096, s, b);
  }
  return 0;
}
