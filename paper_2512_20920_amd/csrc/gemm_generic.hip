// GEMM with float32 products on the matrix cores (v_mfma_f32_32x32x2_f32: every operand element enters as float32,
// bf16 ones exactly), for any shape and any of the operand layouts of GemmArgs.  It serves the float32 configuration,
// whose tolerance needs float32 products, the three GEMMs around the router (logits, folded router matrix, router
// weight gradient), and every bf16 problem whose shape the bf16 kernels do not take.
//
// These problems are small (one to a few hundred 32x32 tiles), so what bounds them is latency, not the matrix pipe: a
// workgroup owns one tile of 32 TM x 32 TN outputs and cuts the contraction among its waves (wave w takes the chunks of
// 32 k's w, w + NW, ...), operands go from memory (L2) straight into the operand registers, two chunks ahead, and the
// waves' partial tiles are added in wave order through LDS.  No LDS staging: inside a workgroup no two waves want the
// same element.  At T = 400, d = 512 (float32) a GEMM of 400 x 512 x 512 takes 4 us where the LDS-tiled vector kernel
// that it replaced took 64 us (56 workgroups, one dependent load -> LDS -> barrier chain per 16 k's).
#include "kernels.h"

#include "operand_f32.h"

template <class TA, class TB, class TC, class TS, bool AT, bool BT, int TM, int TN>
__global__ void __launch_bounds__(TM * TN == 1 ? 512 : 256) gemm_f32_k(GemmArgs g) {
  extern __shared__ __attribute__((aligned(16))) float part[];      // [waves][32 TM][32 TN]
  constexpr int BM = 32 * TM, BN = 32 * TN;
  const TA* A = (const TA*)g.A;
  const TB* Bm = (const TB*)g.B;
  TC* C = (TC*)g.C;
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
    }
  }
  if (g.row_skip && g.group_mode == 0) {             // nothing to do if every row of the tile is marked as finished
    int live = 0;                                    // every wave checks all rows of the tile: same answer, no LDS
    for (int r = m0 + (int)(threadIdx.x & 63); r < min(m_end, m0 + BM); r += 64) live |= g.row_skip[r] == 0;
    if (!__any(live)) return;
  }
  const int n0 = blockIdx.x * BN;
  const int lane = threadIdx.x & 63, gh = lane >> 5, wv = threadIdx.x >> 6, nw = blockDim.x >> 6;
  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; i++)
#pragma unroll
    for (int j = 0; j < TN; j++)
#pragma unroll
      for (int e = 0; e < 16; e++) acc[i][j][e] = 0.f;
  const int nchunk = (k_end - k0 + GKC - 1) / GKC;
  if (wv < nchunk) {
    Operand<TA, AT> oa[TM];
    Operand<TB, BT> ob[TN];
#pragma unroll
    for (int i = 0; i < TM; i++) oa[i].init(A, g.lda, m0 + 32 * i, m_end, lane, g.a_gather, g.gather_div, k0, (const TA*)g.a_last_row);
#pragma unroll
    for (int j = 0; j < TN; j++) ob[j].init(Bm, g.ldb, n0 + 32 * j, g.N, lane, nullptr, 1, k0);
    float va[2][TM][16], vb[2][TN][16];
    auto fetch = [&](int c, float (&a)[TM][16], float (&b)[TN][16]) {
#pragma unroll
      for (int i = 0; i < TM; i++) oa[i].load(k0 + c * GKC, k_end, gh, a[i]);
#pragma unroll
      for (int j = 0; j < TN; j++) ob[j].load(k0 + c * GKC, k_end, gh, b[j]);
    };
    auto mul = [&](float (&a)[TM][16], float (&b)[TN][16]) {
#pragma unroll
      for (int s = 0; s < 16; s++)
#pragma unroll
        for (int i = 0; i < TM; i++)
#pragma unroll
          for (int j = 0; j < TN; j++) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i][s], b[j][s], acc[i][j], 0, 0, 0);
    };
    int c = wv;
    fetch(c, va[0], vb[0]);
    for (; c + nw < nchunk; c += 2 * nw) {           // one chunk in flight while the one before it is multiplied
      fetch(c + nw, va[1], vb[1]);
      mul(va[0], vb[0]);
      if (c + 2 * nw < nchunk) fetch(c + 2 * nw, va[0], vb[0]);
      mul(va[1], vb[1]);
    }
    if (c < nchunk) mul(va[0], vb[0]);
  }
  // ---- partial tiles to LDS, added in wave order by all threads, then the epilogue on whole output rows
  float* mine = part + wv * (BM * BN);
#pragma unroll
  for (int i = 0; i < TM; i++)
#pragma unroll
    for (int j = 0; j < TN; j++)
#pragma unroll
      for (int e = 0; e < 16; e++)
        mine[(i * 32 + (e >> 2) * 8 + gh * 4 + (e & 3)) * BN + j * 32 + (lane & 31)] = acc[i][j][e];
  __syncthreads();
  const TS* bias = (const TS*)g.bias;
  const TS* resid = (const TS*)g.resid;
  const TS* cscale = (const TS*)g.col_scale;
  const int parts = min(nw, max(nchunk, 1));
  for (int e = threadIdx.x; e < BM * BN; e += blockDim.x) {
    const int m = m0 + e / BN, n = n0 + e % BN;
    if (m >= m_end || n >= g.N) continue;
    float v = 0.f;
    for (int w = 0; w < parts; w++) v += part[w * (BM * BN) + e];
    if (cscale) v *= to_f(cscale[n]);
    if (bias) v += to_f(bias[n]);
    if (g.tap) g.tap[(i64)m * g.ldtap + n] = v;
    if (resid) v = (g.resid_f32 ? ((const float*)g.resid)[(i64)m * g.ldr + n] : to_f(resid[(i64)m * g.ldr + n])) + g.resid_sign * v;
    C[(i64)m * g.ldc + n] = from_f<TC>(v);
  }
}

template <class TA, class TB, class TC, class TS, bool AT, bool BT, int TM, int TN>
static void go_shape(const GemmArgs& g, int nw, hipStream_t s) {
  const int gy = g.group_mode == 1 ? g.max_tiles : cdiv(g.M, 32 * TM);
  const dim3 grid(cdiv(g.N, 32 * TN), gy, g.group_mode == 2 ? g.n_groups : 1);
  if (grid.x == 0 || grid.y == 0 || grid.z == 0) return;
  const size_t smem = (size_t)nw * 1024 * TM * TN * sizeof(float);
  static std::atomic<unsigned long long> attr_mask{0};
  if (smem > 65536 - 1024 && attr_needed(attr_mask)) {
    (void)hipFuncSetAttribute((const void*)gemm_f32_k<TA, TB, TC, TS, AT, BT, TM, TN>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, 65536);
    attr_done(attr_mask);
  }
  hipLaunchKernelGGL((gemm_f32_k<TA, TB, TC, TS, AT, BT, TM, TN>), grid, dim3(64 * nw), smem, s, g);
}

template <class TA, class TB, class TC, class TS, bool AT, bool BT>
static void go(const GemmArgs& g, hipStream_t s) {
  // 64x64 tiles of 4 waves (half the operand traffic per product) once they alone are a workgroup per CU; otherwise
  // 32x32 tiles, with as many waves as leave each two chunks of k (one to multiply, one in flight), at most 8.  Where
  // the tiles alone put more than 16 waves on a CU, further cutting of k only adds partial sums.
  const i64 z = g.group_mode == 2 ? g.n_groups : 1;
  if (g.group_mode != 1 && (i64)cdiv(g.M, 64) * cdiv(g.N, 64) * z >= 256) { go_shape<TA, TB, TC, TS, AT, BT, 2, 2>(g, 4, s); return; }
  const i64 tiles = (i64)(g.group_mode == 1 ? g.max_tiles : cdiv(g.M, 32)) * cdiv(g.N, 32) * z;
  const int krange = g.group_mode == 2 ? cdiv(g.K, g.n_groups) : g.K;    // (per expert: the mean)
  int nw = 1;
  while (nw < 8 && krange >= 4 * GKC * nw) nw *= 2;
  while (nw > 4 && tiles * nw > 8192) nw /= 2;
  go_shape<TA, TB, TC, TS, AT, BT, 1, 1>(g, nw, s);
}

template <class TA, class TB, class TC, class TS>
static void go_types(const GemmArgs& g, hipStream_t s) {
  if (g.a_trans) { if (g.b_trans) go<TA, TB, TC, TS, true, true>(g, s); else go<TA, TB, TC, TS, true, false>(g, s); }
  else { if (g.b_trans) go<TA, TB, TC, TS, false, true>(g, s); else go<TA, TB, TC, TS, false, false>(g, s); }
}

int launch_gemm_generic(const GemmArgs& g, GemmTypes t, hipStream_t s) {
  if (g.group_mode == 1 && g.tile_bm != 32) return -1;
  int key = t.ta * 8 + t.tb * 4 + t.tc * 2 + t.tside;
  switch (key) {
    case 0: go_types<float, float, float, float>(g, s); break;            // fp32 everything
    case 15: go_types<bf16, bf16, bf16, bf16>(g, s); break;               // bf16 everything
    case 13: go_types<bf16, bf16, float, bf16>(g, s); break;              // bf16 in, fp32 out (router fold)
    case 7: go_types<float, bf16, bf16, bf16>(g, s); break;               // fp32 A (router logit gradients), bf16 B/C
    case 9: go_types<bf16, float, float, bf16>(g, s); break;              // bf16 A, fp32 B/C (router logits)
    case 1: go_types<float, float, float, bf16>(g, s); break;             // router logits from float32 residual streams
    case 5: go_types<float, bf16, float, bf16>(g, s); break;              // router weight gradient in float32
    default: return -1;
  }
  return 0;
}
