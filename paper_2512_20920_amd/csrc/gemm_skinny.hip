// bf16 GEMM for few rows (short prompts, one example per step): 32 x 32 tiles, the contraction cut among the waves of a
// workgroup.
//
// With few rows a dense layer is its weight matrix read once, and what bounds it is how much of that is in flight.  The
// tile kernel walks k in one chain per tile: 128 rows x 2048 columns x k = 2048 is 32 workgroups of 128x64 with three
// k-tiles in flight each, and 32 dependent steps.  Here the same problem is 256 workgroups of 8 waves; wave w multiplies
// the 64-wide pieces w, w + 8, ... of k with two pieces of its own in flight (short k's: fewer waves and pieces, see by_k),
// and the partial tiles are added in wave order through LDS, so that a result's bits depend on k alone.
// The routed experts' GEMMs of small calls come here too, by their list of row tiles, and what would be a launch of its own
// around a small dense layer is part of it: norm of the rows, rotation, SwiGLU either way, a second pair of operands.
// Each wave stages its pieces in LDS that no other wave touches (direct loads, no barrier before the end): a fragment
// read from memory by the lane that needs it puts every lane on a cache line of its own, 94 clocks per KiB.
//  * rows x k operands: 128-byte rows, 16-byte chunk c of row r in slot c ^ ((r >> 1) & 7);
//  * B stored k x columns: 64-byte rows, transposing reads (rows 0-3 and 8-11 of a k-step cover all banks twice, the
//    least that 512 bytes can take).
// Workgroups of one XCD take a run of column tiles with the row tile fastest, so a weight line enters one L2 only.
#include "lds_load.h"
#include <type_traits>

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(8))) short s16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

// EPI: what goes with the product (EPI_ACT, EPI_ROPE, EPI_NORM, see GemmArgs); NW = waves; NS = pieces of a wave in flight; PAIR: problem 0 has a second pair of operands, its pieces follow the first's
template <bool BT, class TC, int EPI, int NW, int NS, bool PAIR, bool GRP>
__global__ void __launch_bounds__(NW * 64) gemm_skinny_k(GemmArgs g, std::conditional_t<GRP, GemmDense, char> d) {
  constexpr bool ACT = EPI & EPI_ACT, ROPE = EPI & EPI_ROPE, NORM = EPI & EPI_NORM;
  constexpr int RS = 32 + 8;                         // row stride of a partial tile (floats): rows 4 apart are 32 banks apart
  constexpr unsigned OPD = 64 * 32 * 2, STAGE = 2 * OPD + (NORM ? 256 : 0);     // LDS bytes of a piece: A, B, gains
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  const bf16* A = (const bf16*)g.A;
  const bf16* B = (const bf16*)g.B;
  TC* C = (TC*)g.C;
  const bf16* bias = (const bf16*)g.bias;
  int bx, by, m0, m_end, K = g.K, N = g.N, act_half = g.act_half;
  i64 lda = g.lda, ldb = g.ldb, ldc = g.ldc, ldact = g.ldact;
  const int* gather = g.a_gather;
  void *act_out = g.act_out, *dact_out = g.dact_out;
  const void* dact_gu = g.dact_gu;
  bool once = GRP && g.once;
  if constexpr (GRP) {
    if ((int)blockIdx.x < d.blocks) {                // the dense problem that came along
      if (!place_dense(d, (int)blockIdx.x, &bx, &by)) return;
      A = (const bf16*)d.A; B = (const bf16*)d.B; C = (TC*)d.C;
      K = d.K; N = d.N; act_half = d.act_half; lda = d.lda; ldb = d.ldb; ldc = d.ldc; ldact = d.act_half;
      gather = nullptr; act_out = d.act_out; dact_out = d.dact_out; dact_gu = d.dact_gu; once = false;
      m0 = by * 32; m_end = d.M;
    } else {                                         // routed experts: row tiles from the list, 32 high
      int bz = 0;
      if (!place_tile(1, 1, 0, g.tiles_n, 1, g.tile_count[0], g.tile_first, (int)blockIdx.x - d.blocks, &bx, &by, &bz)) return;
      const int grp = g.tile_group[by];
      if (grp < 0) return;
      m0 = g.tile_m0[by];
      m_end = min(g.offsets[grp + 1], m0 + 32);
      B += (i64)grp * g.b_group_stride;
    }
  } else {
    if (blockIdx.z == 1) { A = (const bf16*)g.subA[0]; B = (const bf16*)g.subB[0]; C = (TC*)g.subC[0]; bias = (const bf16*)g.subBias[0]; }
    if (blockIdx.z == 2) { A = (const bf16*)g.subA[1]; B = (const bf16*)g.subB[1]; C = (TC*)g.subC[1]; bias = (const bf16*)g.subBias[1]; }
    const int run = (g.tiles_n + 7) >> 3, c = (int)blockIdx.x & 7, loc = (int)blockIdx.x >> 3;
    bx = c * run + loc / g.tiles_m; by = loc % g.tiles_m;
    if (bx >= g.tiles_n) return;
    m0 = by * 32; m_end = g.M;
  }
  const int n0 = bx * (ACT ? 16 : 32), ncols = ACT ? act_half : N;
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), half = lane >> 5;
  if (!GRP && g.row_skip) {                          // every wave looks at all rows of the tile: same answer, no barrier
    const int r = m0 + (lane & 31);
    if (!__any(r < m_end && g.row_skip[r] == 0)) return;
  }
  const bool pair = PAIR && blockIdx.z == 0;
  const u32x4 da = make_desc(A), db = make_desc(B), da2 = make_desc(PAIR ? g.A2 : A), db2 = make_desc(PAIR ? g.B2 : B);
  const int np1 = (K + 63) >> 6, np = pair ? 2 * np1 : np1;
  const unsigned lda_b = (unsigned)lda * 2u, ldb_b = (unsigned)ldb * 2u;
  // where this lane's share of the four wave-loads of each operand comes from at k = 0, and which k it is (relative to
  // the piece): a load at or past K is out of range, rows and columns past the end repeat the last one or are zeros
  unsigned aoff[4], boff[4];
  int akc[4];
#pragma unroll
  for (int i = 0; i < 4; i++) {
    const int r = i * 8 + (lane >> 3), ch = (lane & 7) ^ ((r >> 1) & 7);
    akc[i] = ch * 8;
    const int row = min(m0 + r, m_end - 1);
    aoff[i] = (unsigned)(GRP && gather ? gather[row] / g.gather_div : row) * lda_b + (unsigned)ch * 16u;
    if constexpr (!BT) {
      const int col = ACT ? (r >> 4) * ncols + min(n0 + (r & 15), ncols - 1) : ROPE ? rope_tile_col(bx, r, g.rope_dh) : min(n0 + r, ncols - 1);
      boff[i] = (unsigned)col * ldb_b + (unsigned)ch * 16u;
    } else {                                         // 16 k's: lane l brings columns (l & 3) * 8 .. + 7 of row l >> 2
      const int col = n0 + (lane & 3) * 8;
      boff[i] = col < N ? (unsigned)(i * 16 + (lane >> 2)) * ldb_b + (unsigned)col * 2u : OOB;
    }
  }
  const bf16* gain = NORM ? (const bf16*)(blockIdx.z == 0 ? g.norm_g[0] : blockIdx.z == 1 ? g.norm_g[1] : g.norm_g[2]) : nullptr;
  bf16* nout = NORM ? (bf16*)(blockIdx.z == 0 ? g.norm_out[0] : blockIdx.z == 1 ? g.norm_out[1] : g.norm_out[2]) : nullptr;
  const u32x4 dg = make_desc(NORM ? gain : A);
  const unsigned my = (unsigned)wv * NS * STAGE;     // this wave's part of LDS
  const unsigned lds0 = lds_address(smem) + my;
  auto load_b = [&](u32x4 rb, unsigned lds, unsigned off) {
    if (once) load_lds_b128_once(rb, lds, off);
    else load_lds_b128(rb, lds, off);
  };
  auto issue = [&](int p, int stage) {
    const bool second = pair && p >= np1;
    const int k0 = (second ? p - np1 : p) * 64;
    const u32x4 ra = second ? da2 : da, rb = second ? db2 : db;
    const unsigned dst = lds0 + (unsigned)stage * STAGE;
    if constexpr (NORM) load_lds_b32(dg, __builtin_amdgcn_readfirstlane(dst + 2 * OPD), k0 + 2 * lane < K ? (unsigned)(k0 + 2 * lane) * 2u : OOB);
#pragma unroll
    for (int i = 0; i < 4; i++) {
      const bool in = k0 + akc[i] < K;
      load_lds_b128(ra, __builtin_amdgcn_readfirstlane(dst + i * 1024u), in ? aoff[i] + (unsigned)k0 * 2u : OOB);
      if constexpr (!BT) {
        load_b(rb, __builtin_amdgcn_readfirstlane(dst + OPD + i * 1024u), in ? boff[i] + (unsigned)k0 * 2u : OOB);
      } else {
        const bool kin = k0 + i * 16 + (lane >> 2) < K && boff[i] != OOB;
        load_b(rb, __builtin_amdgcn_readfirstlane(dst + OPD + i * 1024u), kin ? boff[i] + (unsigned)k0 * ldb_b : OOB);
      }
    }
  };
  f32x16 acc = {};

  const int fr = lane & 31, fsw = (fr >> 1) & 7;
  const unsigned tr = (unsigned)((lane >> 5) * 8 + ((lane & 15) >> 2)) * 64u + (unsigned)(((lane >> 4) & 1) * 16 + (lane & 3) * 4) * 2u;
#pragma unroll
  for (int st = 0; st < NS; st++) issue(wv + st * NW, st);          // (pieces past the end load zeros, to keep the count)
  if constexpr (NORM) {
    // every wave has its NS pieces of the rows (k <= 64 NW NS): their squares meet in LDS, then the pieces are normalised on
    // their way to the product and, by one column tile each, to memory
    float* sq = (float*)(smem + (size_t)NW * NS * STAGE);
    bf16x8 fa[NS][4];
    float ss = 0.f;
    wait_vmcnt<0>();
#pragma unroll
    for (int u = 0; u < NS; u++)
#pragma unroll
      for (int s = 0; s < 4; s++) {
        fa[u][s] = *(const bf16x8*)(smem + my + u * STAGE + (unsigned)fr * 128u + (unsigned)((2 * s + half) ^ fsw) * 16u);
#pragma unroll
        for (int i = 0; i < 8; i++) ss += (float)fa[u][s][i] * (float)fa[u][s][i];
      }
    ss += __shfl_xor(ss, 32, WAVE);
    if (half == 0) sq[wv * 32 + lane] = ss;
    __syncthreads();
    float sum = 0.f;
#pragma unroll
    for (int w = 0; w < NW; w++) sum += sq[w * 32 + fr];
    const float rinv = 1.0f / sqrtf(sum / (float)K + g.norm_eps);
#pragma unroll
    for (int u = 0; u < NS; u++) {
      const unsigned char* t = smem + my + u * STAGE;
      const int p = wv + u * NW;
      const bool keep = nout && p < np && p % g.tiles_n == bx && m0 + fr < m_end;
#pragma unroll
      for (int s = 0; s < 4; s++) {
        const bf16x8 gv = *(const bf16x8*)(t + 2 * OPD + (s * 16 + half * 8) * 2);
        const bf16x8 fb = *(const bf16x8*)(t + OPD + (unsigned)fr * 128u + (unsigned)((2 * s + half) ^ fsw) * 16u);
        bf16x8 x;
#pragma unroll
        for (int i = 0; i < 8; i++) x[i] = (__bf16)((float)fa[u][s][i] * rinv * (float)gv[i]);
        const int k = p * 64 + s * 16 + half * 8;
        if (keep && k < K) *(bf16x8*)(nout + (i64)(m0 + fr) * K + k) = x;
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, fb, acc, 0, 0, 0);
      }
    }
  } else {
    int st = 0;
    for (int p = wv; p < np; p += NW) {
      wait_vmcnt<(NS - 1) * 8>();
      const unsigned char* t = smem + my + (unsigned)st * STAGE;
      bf16x8 fa[4], fb[4];
#pragma unroll
      for (int s = 0; s < 4; s++) {
        const unsigned at = (unsigned)fr * 128u + (unsigned)((2 * s + half) ^ fsw) * 16u;
        fa[s] = *(const bf16x8*)(t + at);
        if constexpr (!BT) {
          fb[s] = *(const bf16x8*)(t + OPD + at);
        } else {
          const unsigned char* q = t + OPD + tr + s * 1024u;
          const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)q);
          const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(q + 4 * 64));
          fb[s] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
        }
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");              // the fragments are in registers: the stage is free
      __builtin_amdgcn_sched_barrier(0);
      issue(p + NS * NW, st);
      st = st + 1 == NS ? 0 : st + 1;
#pragma unroll
      for (int s = 0; s < 4; s++) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[s], fb[s], acc, 0, 0, 0);
    }
  }
  wait_vmcnt<0>();                                                  // the zero-filled loads past the end
  __syncthreads();                                   // the partial tiles overlay the stages
  float* part = (float*)smem;
#pragma unroll
  for (int e = 0; e < 16; e++) part[wv * 32 * RS + ((e >> 2) * 8 + half * 4 + (e & 3)) * RS + (lane & 31)] = acc[e];
  __syncthreads();
  const int col = (int)(threadIdx.x & 31), n = ROPE ? rope_tile_col(bx, col, g.rope_dh) : n0 + (ACT ? col & 15 : col);
  if (n >= ncols) return;                            // (ACT: a gate column and its up column both; ROPE: whole tiles)
#pragma unroll
  for (int r = (int)threadIdx.x >> 5; r < 32; r += NW * 2) {
    const int m = m0 + r;
    if (m >= m_end) break;
    float v = 0.f;
#pragma unroll
    for (int w = 0; w < NW; w++) v += part[w * 32 * RS + r * RS + col];
    if constexpr (ACT) {                             // silu(gate) * up from the rounded values, as the tile kernel
      const TC x = (TC)v;
      const float own = (float)x, up = __shfl(own, lane | 16, WAVE);
      C[(i64)m * ldc + (col >> 4) * ncols + n] = x;
      if (col < 16) ((TC*)act_out)[(i64)m * ldact + n] = (TC)(own * sigmoid_f(own) * up);
    } else if constexpr (ROPE) {
      const float own = (float)(TC)(v + (bias ? (float)bias[n] : 0.f));
      const int step = g.rope_dh == 16 ? 8 : 16, i = n & (g.rope_dh / 2 - 1);
      const float other = __shfl_xor(own, step, WAVE);
      const bool turn = (g.rope_mask >> blockIdx.z) & 1;
      const float2 cs = turn ? ((const float2*)g.rope_cs)[(i64)(m % g.rope_S) * (g.rope_dh / 2) + i] : make_float2(1.f, 0.f);
      C[(i64)m * ldc + n] = (TC)(turn ? rope_value(own, other, col & step, cs) : own);
    } else if (dact_out) {                         // SwiGLU's backward, from what C would have held
      const bf16* gu = (const bf16*)dact_gu + (i64)m * 2 * N + n;
      float dg, du;
      swiglu_grad((float)(TC)v, (float)gu[0], (float)gu[N], &dg, &du);
      TC* out = (TC*)dact_out + (i64)m * 2 * N + n;
      out[0] = (TC)dg;
      out[N] = (TC)du;
    } else {
      float o = v + (bias ? (float)bias[n] : 0.f);
      if (g.tap) g.tap[(i64)m * g.ldtap + n] = o;
      if (g.resid) {
        const i64 at = (i64)m * g.ldr + n;
        o = (g.resid_f32 ? ((const float*)g.resid)[at] : (float)((const bf16*)g.resid)[at]) + g.resid_sign * o;
      }
      C[(i64)m * ldc + n] = (TC)o;
    }
  }
}

template <bool BT, class TC, int EPI, int NW, int NS, bool PAIR = false, bool GRP = false>
static void go(GemmArgs g, hipStream_t s) {
  g.tiles_m = GRP ? g.max_tiles : cdiv(g.M, 32);
  g.tiles_n = EPI & EPI_ACT ? cdiv(g.act_half, 16) : cdiv(g.N, 32);
  constexpr size_t part = (size_t)NW * 32 * 40 * 4, bufs = (size_t)NW * NS * (2 * 64 * 32 * 2 + (EPI & EPI_NORM ? 256 : 0)) + (EPI & EPI_NORM ? NW * 128 : 0);
  constexpr size_t smem = part > bufs ? part : bufs;
  static_assert(smem <= 160 * 1024, "LDS of a CU");
  static std::atomic<unsigned long long> attr_mask{0};
  if (attr_needed(attr_mask)) {
    (void)hipFuncSetAttribute((const void*)gemm_skinny_k<BT, TC, EPI, NW, NS, PAIR, GRP>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    attr_done(attr_mask);
  }
  if constexpr (GRP) {
    GemmDense d;
    if (g.co) { d = *g.co; place_dense_grid(d, EPI & EPI_ACT ? 16 : 32); }
    hipLaunchKernelGGL((gemm_skinny_k<BT, TC, EPI, NW, NS, PAIR, true>), dim3(d.blocks + g.tiles_n * g.tiles_m), dim3(NW * 64), smem, s, g, d);
  } else {
    hipLaunchKernelGGL((gemm_skinny_k<BT, TC, EPI, NW, NS, PAIR, false>), dim3(8 * cdiv(g.tiles_n, 8) * g.tiles_m, 1, g.n_sub), dim3(NW * 64), smem, s, g, '\0');
  }
}

// Pieces in flight are LDS, and LDS decides how many workgroups share a CU.  Up to 4 pieces there are 4 waves with one each
// (32 KiB, four workgroups), up to 8 pieces 8 waves (64 KiB, two).  With more k a wave has two in flight (128 KiB) where
// every workgroup has a CU to itself anyway; a larger launch gains more from a second workgroup.
template <bool BT, class TC, int EPI, bool PAIR = false, bool GRP = false>
static void by_k(const GemmArgs& g, hipStream_t s) {
  const int k = PAIR ? 2 * g.K : g.K;
  if (k <= 256) go<BT, TC, EPI, 4, 1, PAIR, GRP>(g, s);
  else if (k <= 512 || (!(EPI & EPI_NORM) && (i64)(GRP ? g.max_tiles : cdiv(g.M, 32)) * cdiv(g.N, 32) * g.n_sub > 256)) go<BT, TC, EPI, 8, 1, PAIR, GRP>(g, s);
  else go<BT, TC, EPI, 8, 2, PAIR, GRP>(g, s);
}

void launch_gemm_skinny(const GemmArgs& g, int out_f32, hipStream_t s) {
  if (g.group_mode == 1) {                           // (bf16 results, launch_gemm_mfma)
    if (g.act_half) by_k<false, bf16, EPI_ACT, false, true>(g, s);
    else if (g.b_trans) by_k<true, bf16, 0, false, true>(g, s);
    else by_k<false, bf16, 0, false, true>(g, s);
    return;
  }
  // (launch_gemm_mfma admits a second pair of operands with b_trans, norm and rotation without, all with bf16 results)
  if (g.act_half) { if (out_f32) by_k<false, float, EPI_ACT>(g, s); else by_k<false, bf16, EPI_ACT>(g, s); }
  else if (g.A2) by_k<true, bf16, 0, true>(g, s);
  else if (g.b_trans) { if (out_f32) by_k<true, float, 0>(g, s); else by_k<true, bf16, 0>(g, s); }
  else if (g.norm_g[0] && g.rope_cs) by_k<false, bf16, EPI_NORM | EPI_ROPE>(g, s);
  else if (g.norm_g[0]) by_k<false, bf16, EPI_NORM>(g, s);
  else if (g.rope_cs) by_k<false, bf16, EPI_ROPE>(g, s);
  else { if (out_f32) by_k<false, float, 0>(g, s); else by_k<false, bf16, 0>(g, s); }
}
