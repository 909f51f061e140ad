// The routed experts' GEMMs where an expert has few rows: up to 32 rows x 64 columns per workgroup, the contraction cut among
// its four waves.
//
// With a few rows per expert a launch is the weights of the experts reached, read once, and the time is how steadily they come.
// The 128x256 tile asks for 32 KiB per k-tile and then waits for all of it at a barrier, one workgroup to a CU, with the MFMAs and
// LDS reads of 128 rows (most of them empty) in between: 5.3 TB/s.  Here a wave has one piece of 64 k's (B 8 KiB, A 4 KiB) on its
// way at a time, waits for nobody before the end, and twelve waves of three workgroups share a CU, so that some piece is always
// being asked for: 6.2 TB/s, where the same reads without arithmetic reach 6.9.  Rows past an expert's end are not read at all.
// Measured, us per launch, 128x256 tiles / this, Qwen shape (8 rows per expert): gate/up (692 MB) 131 / 111, down 59 / 56, dHh
// 71 / 64; half as wide with merged weights (37 tokens): 72 / 53, 30 / 29; 20 rows: 138 / 122, 62 / 59, 72 / 72.
// (32 columns per workgroup: 109, 57, and data gradients, whose lines are then shared by two tiles, 85; 128 columns 122 to 132, 57,
// 63 to 71; two waves 127, 58, 65; six 116, 62, 68; eight 127, 69, 74; two pieces per wave in flight 126, 70, 75; 64 rows 124, 65, 70.)
// The partial tiles are added in wave order through LDS, so that a result's bits depend on k alone.
#include "operand_bf16.h"

#define STREAM_WAVES 4
#define PIECE 4096u                  // LDS bytes of 64 k's of 32 rows or columns

// A piece of a wave: A, then B's two blocks of 32 columns (ACT: 32 gate columns and the up columns of the same indices)
template <bool BT, bool ACT>
__global__ void __launch_bounds__(STREAM_WAVES * 64) expert_stream_k(GemmArgs g, GemmDense d) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  int bx, by, m0, m_end, K = g.K, N = g.N, act_half = g.act_half;
  i64 lda = g.lda, ldb = g.ldb, ldc = g.ldc, ldact = g.ldact;
  const bf16 *A = (const bf16*)g.A, *B = (const bf16*)g.B;
  bf16* C = (bf16*)g.C;
  const int* gather = g.a_gather;
  void *act_out = g.act_out, *dact_out = g.dact_out;
  const void* dact_gu = g.dact_gu;
  bool once = g.once;
  if ((int)blockIdx.x < d.blocks) {                  // the dense problem that came along
    if (!place_dense(d, (int)blockIdx.x, &bx, &by)) return;
    A = (const bf16*)d.A; B = (const bf16*)d.B; C = (bf16*)d.C;
    K = d.K; N = d.N; act_half = d.act_half; lda = d.lda; ldb = d.ldb; ldc = d.ldc; ldact = d.act_half;
    gather = nullptr; act_out = d.act_out; dact_out = d.dact_out; dact_gu = d.dact_gu; once = false;
    m0 = by * 32; m_end = min(d.M, m0 + 32);
  } else {
    int bz = 0;
    if (!place_tile(1, 1, 0, g.tiles_n, 1, g.tile_count[0], g.tile_first, (int)blockIdx.x - d.blocks, &bx, &by, &bz)) return;
    const int grp = g.tile_group[by];
    if (grp < 0) return;
    m0 = g.tile_m0[by];
    m_end = min(g.offsets[grp + 1], m0 + 32);
    B += (i64)grp * g.b_group_stride;
  }
  const int n0 = bx * (ACT ? 32 : 64), ncols = ACT ? act_half : N;
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const u32x4 da = make_desc(A), db = make_desc(B);
  const unsigned lda_b = (unsigned)lda * 2u, ldb_b = (unsigned)ldb * 2u, bstep = BT ? 64u * ldb_b : 128u;
  const int np = (K + 63) >> 6;
  // this lane's share of the wave-loads at k = 0; kc: its k relative to the piece (the contraction ends inside the last one)
  unsigned aoff[4], boff[8];
#pragma unroll
  for (int i = 0; i < 4; i++) {
    int in;
    chunk_source<false, 32>(i * 64 + lane, m0, m_end, lda_b, 0, 1 << 30, gather, g.gather_div, &aoff[i], &in);
    if (!in) aoff[i] = OOB;
  }
#pragma unroll
  for (int i = 0; i < 8; i++) {
    int in;
    if constexpr (ACT) chunk_source_gate_up(i * 64 + lane, n0, ncols, ldb_b, 0, 1 << 30, &boff[i], &in);
    else chunk_source<BT, 64>(i * 64 + lane, n0, ncols, ldb_b, 0, 1 << 30, nullptr, 1, &boff[i], &in);
    if (!in) boff[i] = OOB;
  }
  const unsigned char* mine = smem + (unsigned)wv * 3 * PIECE;
  const unsigned lds = lds_address(mine);
  auto issue = [&](int p) {                          // (pieces past the end load zeros)
    const int krem = K - p * 64;
#pragma unroll
    for (int i = 0; i < 4; i++) {
      const int pos = i * 64 + lane, kc = ((pos & 7) ^ ((pos >> 4) & 7)) << 3;
      load_lds_b128(da, __builtin_amdgcn_readfirstlane(lds + i * 1024u), kc < krem && aoff[i] != OOB ? aoff[i] + (unsigned)p * 128u : OOB);
    }
#pragma unroll
    for (int i = 0; i < 8; i++) {
      const int pos = i * 64 + lane, kc = BT ? pos >> 3 : ((pos & 7) ^ ((pos >> 4) & 7)) << 3;
      const unsigned off = kc < krem && boff[i] != OOB ? boff[i] + (unsigned)p * bstep : OOB;
      if (once) load_lds_b128_once(db, __builtin_amdgcn_readfirstlane(lds + PIECE + i * 1024u), off);
      else load_lds_b128(db, __builtin_amdgcn_readfirstlane(lds + PIECE + i * 1024u), off);
    }
  };
  f32x16 acc[2] = {};
  const unsigned fba = frag_base<false, 32>(0, lane);
  unsigned fbb[2];
#pragma unroll
  for (int j = 0; j < 2; j++) fbb[j] = PIECE + frag_base<BT, 64>(j * 32, lane);
  issue(wv);
  for (int p = wv; p < np; p += STREAM_WAVES) {
    wait_vmcnt<0>();
    bf16x8 fa[4], fb[4][2];
#pragma unroll
    for (int kk = 0; kk < 4; kk++) {
      fa[kk] = load_frag<false, 32>(mine, fba, 0, kk, lane);
#pragma unroll
      for (int j = 0; j < 2; j++) fb[kk][j] = load_frag<BT, 64>(mine, fbb[j], j * 32, kk, lane);
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");              // the fragments are in registers: the piece's place is free
    __builtin_amdgcn_sched_barrier(0);
    issue(p + STREAM_WAVES);
#pragma unroll
    for (int kk = 0; kk < 4; kk++)
#pragma unroll
      for (int j = 0; j < 2; j++) acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[kk], fb[kk][j], acc[j], 0, 0, 0);
  }
  wait_vmcnt<0>();                                   // the zero-filled loads past the end
  __syncthreads();                                   // the partial tiles overlay the pieces
  // [waves][32][64]; a row's halves change places every four rows, so that the lanes of a write meet all banks
  float* part = (float*)smem;
#pragma unroll
  for (int j = 0; j < 2; j++)
#pragma unroll
    for (int e = 0; e < 16; e++) {
      const int r = (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3);
      part[(wv * 32 + r) * 64 + ((j * 32 + (lane & 31)) ^ ((r & 4) << 3))] = acc[j][e];
    }
  __syncthreads();
  auto sum = [&](int r, int c) {
    float v = 0.f;
#pragma unroll
    for (int w = 0; w < STREAM_WAVES; w++) v += part[(w * 32 + r) * 64 + (c ^ ((r & 4) << 3))];
    return v;
  };
  constexpr int CW = ACT ? 32 : 64;                  // columns that a row of threads shares out
  const int c = (int)threadIdx.x % CW, n = n0 + c;
  if (n >= ncols) return;
#pragma unroll 4
  for (int r = (int)threadIdx.x / CW; r < 32; r += STREAM_WAVES * 64 / CW) {
    const int m = m0 + r;
    if (m >= m_end) break;
    const bf16 x = (bf16)sum(r, c);
    if constexpr (ACT) {                             // silu(gate) * up from the rounded values, as the other kernels
      const bf16 u = (bf16)sum(r, c + 32);
      C[(i64)m * ldc + n] = x;
      C[(i64)m * ldc + ncols + n] = u;
      ((bf16*)act_out)[(i64)m * ldact + n] = (bf16)((float)x * sigmoid_f((float)x) * (float)u);
    } else if (dact_out) {                         // SwiGLU's backward, from what C would have held
      const bf16* gu = (const bf16*)dact_gu + (i64)m * 2 * N + n;
      float dg, du;
      swiglu_grad((float)x, (float)gu[0], (float)gu[N], &dg, &du);
      bf16* out = (bf16*)dact_out + (i64)m * 2 * N + n;
      out[0] = (bf16)dg;
      out[N] = (bf16)du;
    } else C[(i64)m * ldc + n] = x;
  }
}

template <bool BT, bool ACT>
static void go(GemmArgs g, hipStream_t s) {
  g.tiles_m = g.max_tiles;
  g.tiles_n = ACT ? cdiv(g.act_half, 32) : cdiv(g.N, 64);
  constexpr size_t smem = STREAM_WAVES * 3 * PIECE;          // (the partial tiles take two thirds of it)
  GemmDense d;
  if (g.co) { d = *g.co; place_dense_grid(d, ACT ? 32 : 64); }
  hipLaunchKernelGGL((expert_stream_k<BT, ACT>), dim3(d.blocks + g.tiles_n * g.tiles_m), dim3(STREAM_WAVES * 64), smem, s, g, d);
}
void launch_gemm_experts(const GemmArgs& g, hipStream_t s) {
  if (g.act_half) go<false, true>(g, s);
  else if (g.b_trans) go<true, false>(g, s);
  else go<false, false>(g, s);
}
