// bf16 GEMM on the gfx950 matrix cores (v_mfma_f32_32x32x16_bf16, fp32 accumulation) for
// every dense contraction of the block: adapters, Q/K/V/O projections, shared expert,
// grouped routed experts (forward, data gradient, weight gradient).
//
// Workgroup = NW waves laid out WGM x (NW / WGM) over a BM x BN tile, k-step 64 (128 bytes per
// row), NS LDS stages.  Operand tiles go from global memory straight into LDS
// (buffer_load_dwordx4 ... lds: lane l of a wave-load lands at M0 + 16*l), NS-1 k-tiles ahead of
// the one being multiplied, and the loads of the next tile are issued between the MFMA groups of
// the current one, so that the load path and the matrix pipe run together instead of in turns.
// There is no register staging and no LDS store instruction.
//
// How operand tiles lie in LDS: operand_bf16.h.
#include "operand_bf16.h"
#include <math.h>
#include <stdlib.h>

// Every matrix handed to this kernel spans less than 2 GiB from its base (checked on the host): the offset OOB stands for
// "outside the k range / past the last row".
#define PHASED 0          // (as the number of LDS stages: the 256x256 tile in phases)

// Two neighbouring lanes (columns n, n+1) hold values x0, x1 of rows r, r+1.  After the swap the even lane holds row r
// and the odd lane row r+1, each as (left column, right column): one 4-byte store of two 2-byte results per lane.
// Both lanes of a pair must be active.
__device__ __forceinline__ void pair_rows(bool odd, float x0, float x1, float* left, float* right) {
  const float send = odd ? x0 : x1;
  const float recv = __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, send), 0xB1, 0xf, 0xf, false));
  *left = odd ? recv : x0;
  *right = odd ? x1 : recv;
}

typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
__device__ __forceinline__ bf16x2 pair_rows_bf16(bool odd, float x0, float x1) {
  float l, r;
  pair_rows(odd, x0, x1, &l, &r);
  bf16x2 w;
  w[0] = (__bf16)l; w[1] = (__bf16)r;
  return w;
}

// a plain result that can be stored 16 bytes at a time (widths of this layout are multiples of 8)
__device__ __forceinline__ bool whole_lines(const GemmArgs& g, const void* C, const void* bias) {
  return !bias && !g.resid && !g.tap && !(g.ldc & 7) && !((uintptr_t)C & 15);
}

// Epilogue of one output tile.  rb, cb: first row (column) of the wave's 32-row (32-column) blocks inside the tile;
// act_col: with the SwiGLU epilogue, the wave's first gate column inside the tile's BN / 2.
// KIND: 0 = whatever the arguments ask for; the routed experts' 320-row tiles, whose registers are short: 1 = plain store only, 2 = SwiGLU only
template <int BM, int BN, bool AT, bool BT, class TC, int TE, int TN, int KIND = 0>
__device__ __forceinline__ void gemm_epilogue(const GemmArgs& g, TC* C, const void* bias_ptr, int bx, int m0, int m_end,
                                              const int (&rb)[TE], const int (&cb)[TN], int act_col, f32x16 (&acc)[TE][TN]) {
  const int n0 = bx * BN, lane = threadIdx.x & 63;
  // ---- epilogue: lane holds column n = lane & 31 and rows (e>>2)*8 + (lane>>5)*4 + (e&3)
  if (KIND == 2 || (KIND == 0 && g.act_half)) {
    // gate/up GEMM with the SwiGLU epilogue: this wave's first 32-column block is gate columns, its second the up
    // columns of the same indices.  Both go to C (the backward pass needs them), and silu(gate) * up, from the
    // rounded values, to act_out.
    if constexpr (!AT && !BT && TN == 2) {
      TC* H = (TC*)g.act_out;
      const int half = g.act_half;
      const int col = bx * (BN / 2) + act_col + (lane & 31);
      if constexpr (sizeof(TC) == 2) {
        // pairs of lanes store two columns of one row each (see the plain store below); rows past the end are masked
        // per lane after the swap, columns per pair (the width is even)
        if (!(g.ldc & 1) && !(g.ldact & 1) && !(half & 1) && !((uintptr_t)C & 3) && !((uintptr_t)H & 3) && !g.no_packed_stores) {
          const bool odd = lane & 1;
          const int colp = col - (odd ? 1 : 0);
          typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_v;
          if (colp < half) {
#pragma unroll
            for (int i = 0; i < TE; i++)
#pragma unroll
              for (int e = 0; e < 16; e += 2) {
                const int m = m0 + rb[i] + (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3) + (odd ? 1 : 0);
                float gq[2], uq[2], hq[2];
#pragma unroll
                for (int p = 0; p < 2; p++) {
                  const TC gb = (TC)acc[i][0][e + p], ub = (TC)acc[i][1][e + p];
                  gq[p] = (float)gb; uq[p] = (float)ub;
                  hq[p] = (float)(TC)(gq[p] * sigmoid_f(gq[p]) * uq[p]);
                }
                float l, r;
                bf16x2_v wg, wu, wh;
                pair_rows(odd, gq[0], gq[1], &l, &r); wg[0] = (__bf16)l; wg[1] = (__bf16)r;
                pair_rows(odd, uq[0], uq[1], &l, &r); wu[0] = (__bf16)l; wu[1] = (__bf16)r;
                pair_rows(odd, hq[0], hq[1], &l, &r); wh[0] = (__bf16)l; wh[1] = (__bf16)r;
                if (m < m_end) {
                  *(bf16x2_v*)(C + (i64)m * g.ldc + colp) = wg;
                  *(bf16x2_v*)(C + (i64)m * g.ldc + half + colp) = wu;
                  *(bf16x2_v*)(H + (i64)m * g.ldact + colp) = wh;
                }
              }
          }
          return;
        }
      }
      if (col < half) {
#pragma unroll
        for (int i = 0; i < TE; i++)
#pragma unroll
          for (int e = 0; e < 16; e++) {
            const int m = m0 + rb[i] + (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3);
            if (m < m_end) {
              const TC gb = (TC)acc[i][0][e], ub = (TC)acc[i][1][e];
              const float gv = (float)gb;
              C[(i64)m * g.ldc + col] = gb;
              C[(i64)m * g.ldc + half + col] = ub;
              H[(i64)m * g.ldact + col] = (TC)(gv * sigmoid_f(gv) * (float)ub);
            }
          }
      }
    }
    return;
  }
  if constexpr (KIND == 2) return;
  const bf16* bias = (const bf16*)bias_ptr;
  const bf16* resid = (const bf16*)g.resid;
  if (KIND == 1 || (!bias && !g.tap && !resid)) {
    // plain store (most projections, data gradients, weight gradients in float32 and those in bf16 that do not leave through
    // LDS, see gemm_tile): no per-element epilogue work
    // the column blocks of one row are stored back to back, so that the 64-byte pieces of a line reach L2 together and
    // are merged there.  (Through LDS in whole lines, as the bf16 weight gradients go: no faster for stores that stay in L2.)
    const bool full = (m0 + BM <= m_end) && (n0 + BN <= g.N);
    auto put = [](auto v, auto* p) {                 // (weight gradients go past the caches, see GemmArgs::once)
      if constexpr (AT && BT) __builtin_nontemporal_store(v, p);
      else *p = v;
    };
    if constexpr (sizeof(TC) == 2) {
      // Whole tiles of 2-byte results: neighbouring lanes hold neighbouring columns of the same rows, so a pair of
      // lanes swaps one value per two rows (the even lane gives its value of the odd row and gets the neighbour's
      // value of the even row) and each lane stores 4 bytes, two columns of one row: half as many store
      // instructions, and the stores of a tile are bound by their number (measured on the weight gradients when they
      // came here: 10 %, 1-2 % of a step).  Going on to a 4x4 transpose inside a quad and 8-byte stores is slower than no packing at
      // all: one instruction then touches eight rows.
      if (full && !(g.ldc & 1) && !((uintptr_t)C & 3) && !g.no_packed_stores) {
        const bool odd = lane & 1;
        typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_v;
#pragma unroll
        for (int i = 0; i < TE; i++) {
          // even lane: row of element e, its own column; odd lane: the row below, the column to its left
          TC* cp = C + (i64)(m0 + rb[i] + (lane >> 5) * 4 + (odd ? 1 : 0)) * g.ldc + n0 + (lane & 31) - (odd ? 1 : 0);
#pragma unroll
          for (int e = 0; e < 16; e += 2) {
            const int dm = (e >> 2) * 8 + (e & 3);
#pragma unroll
            for (int j = 0; j < TN; j++) {
              float l, r;
              pair_rows(odd, acc[i][j][e], acc[i][j][e + 1], &l, &r);
              bf16x2_v w;
              w[0] = (__bf16)l; w[1] = (__bf16)r;
              put(w, (bf16x2_v*)(cp + (i64)dm * g.ldc + cb[j]));
            }
          }
        }
        return;
      }
    }
#pragma unroll
    for (int i = 0; i < TE; i++) {
      TC* cp = C + (i64)(m0 + rb[i] + (lane >> 5) * 4) * g.ldc + n0 + (lane & 31);
#pragma unroll
      for (int e = 0; e < 16; e++) {
        const int dm = (e >> 2) * 8 + (e & 3);
        const bool row_ok = full || (m0 + rb[i] + (lane >> 5) * 4 + dm < m_end);
#pragma unroll
        for (int j = 0; j < TN; j++)
          if (row_ok && (full || n0 + cb[j] + (lane & 31) < g.N)) put((TC)acc[i][j][e], cp + (i64)dm * g.ldc + cb[j]);
      }
    }
    return;
  }
  if constexpr (KIND == 0) {
  // Two phases per 32-column block: every load (bias, residual) and all arithmetic on loaded values
  // first, then nothing but stores.  On this ISA one counter tracks loads and stores, and where a store may or may
  // not have been issued (rows and columns past the problem's edge are masked per lane) the compiler can only wait
  // for "everything": a use of a loaded value between two stores then waits for the earlier store to complete, and
  // the 16 * TE * TN stores of a lane run one after the other (the coupling GEMMs with a residual operand took
  // twice as long as the same GEMM with a plain store).  So loads are never masked (indices past the edge are
  // clamped to the last valid row / column instead), the finished values are pinned in registers before the first
  // store (the empty asm keeps the compiler from sinking the arithmetic into the masked store blocks), and the
  // store phase has nothing to wait for.  The residual operand may be the output itself (in-place coupling update):
  // it either is C, element for element, or does not overlap it, and each lane reads its elements before it writes.
  constexpr int GI = 1;                              // 32-row blocks whose loads are issued together (more would spill at TE = 2)
  const bool full = (m0 + BM <= m_end) && (n0 + BN <= g.N);
  const int m_last = m_end - 1, n_last = g.N - 1;
  auto row_of = [&](int i, int e) { return m0 + rb[i] + (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3); };
#pragma unroll
  for (int j = 0; j < TN; j++) {
    const int n = n0 + cb[j] + (lane & 31);
    const bool n_ok = full || n < g.N;
    const int nn = min(n, n_last);
    const float bv = bias ? (float)bias[nn] : 0.f;
#pragma unroll
    for (int i0 = 0; i0 < TE; i0 += GI) {
      // ---- phase 1: loads and arithmetic
      float rv[GI][16];
      if (resid) {
        if (g.resid_f32) {
#pragma unroll
          for (int ii = 0; ii < GI; ii++)
#pragma unroll
            for (int e = 0; e < 16; e++)
              rv[ii][e] = ((const float*)g.resid)[(i64)min(row_of(i0 + ii, e), m_last) * g.ldr + nn];
        } else {
#pragma unroll
          for (int ii = 0; ii < GI; ii++)
#pragma unroll
            for (int e = 0; e < 16; e++) rv[ii][e] = (float)resid[(i64)min(row_of(i0 + ii, e), m_last) * g.ldr + nn];
        }
      } else {
#pragma unroll
        for (int ii = 0; ii < GI; ii++)
#pragma unroll
          for (int e = 0; e < 16; e++) rv[ii][e] = 0.f;
      }
#pragma unroll
      for (int ii = 0; ii < GI; ii++)
#pragma unroll
        for (int e = 0; e < 16; e++) {
          float v = acc[i0 + ii][j][e] + bv;                   // the value the tap records
          float o = resid ? rv[ii][e] + g.resid_sign * v : v;
          asm volatile("" : "+v"(v), "+v"(o));
          acc[i0 + ii][j][e] = v;
          rv[ii][e] = o;
        }
      // ---- phase 2: stores
      if constexpr (sizeof(TC) == 2) {
        // two columns of one row per lane (see the plain store above); the swap runs on every lane, the masks after it
        if (!g.tap && !(g.ldc & 1) && !(g.N & 1) && !((uintptr_t)C & 3) && !g.no_packed_stores) {
          const bool odd = lane & 1;
          typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_v;
#pragma unroll
          for (int ii = 0; ii < GI; ii++)
#pragma unroll
            for (int e = 0; e < 16; e += 2) {
              float l, r;
              pair_rows(odd, rv[ii][e], rv[ii][e + 1], &l, &r);
              bf16x2_v w;
              w[0] = (__bf16)l; w[1] = (__bf16)r;
              const int m = row_of(i0 + ii, e) + (odd ? 1 : 0);
              if (n_ok && (full || m < m_end)) *(bf16x2_v*)(C + (i64)m * g.ldc + n - (odd ? 1 : 0)) = w;
            }
          continue;
        }
      }
#pragma unroll
      for (int ii = 0; ii < GI; ii++)
#pragma unroll
        for (int e = 0; e < 16; e++) {
          const int m = row_of(i0 + ii, e);
          if (n_ok && (full || m < m_end)) {
            if (g.tap) g.tap[(i64)m * g.ldtap + n] = acc[i0 + ii][j][e];
            C[(i64)m * g.ldc + n] = (TC)rv[ii][e];
          }
        }
    }
  }
  }
}

// One output tile; TE = 32-row blocks per wave.
template <int BM, int BN, int WGM, bool AT, bool BT, class TC, int NW, int NS, int TE, int KB = BK, bool ONCE = false>
__device__ __forceinline__ void gemm_tile(const GemmArgs& g, const bf16* A, const bf16* Bm, TC* C, const void* bias_ptr,
                                          int bx, int bz, int m0, int m_end, int k0, int k_end, int rot_seed) {
  constexpr int WGN = NW / WGM;                      // waves along n
  constexpr int WM = BM / WGM, WN = BN / WGN, TN = WN / 32;
  // KB: elements of k per LDS stage (64; 32 for the per-expert weight gradients, whose k range is a few dozen rows)
  constexpr int STAGE = (BM + BN) * KB * 2;          // bytes of one LDS stage: A tile, then B tile
  constexpr int ALOADS = BM * KB / 512;              // wave-loads (1 KiB) of the A tile
  constexpr int LPW = (BM + BN) * KB / 512 / NW;     // wave-loads per wave per stage
  constexpr int KS = KB / 16;                        // MFMA k-steps per stage
  static_assert(WM % 32 == 0 && WN % 32 == 0, "wave tile must be made of 32x32 blocks");
  static_assert(((BM + BN) * KB) % (512 * NW) == 0 && (BM * KB) % 512 == 0 && LPW % KS == 0 || KB == BK, "wave-loads must divide evenly");
  static_assert((BM + BN) % (8 * NW) == 0 && BM % 8 == 0, "wave-loads must divide evenly");
  static_assert(KB == BK || (AT && BT), "a shorter k-tile only for operands stored k x rows");
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  const int n0 = bx * BN;
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = (wv / WGN) * WM, wn = (wv % WGN) * WN;
  const int krange = k_end - k0;
  const int nk = (krange + KB - 1) / KB;

  // ---- this wave's loads: wave-load j = wv*LPW + i fills LDS chunks [64 j, 64 j + 64) of a stage; the first
  // BM/8 wave-loads are the A tile, the rest the B tile
  const u32x4 da = make_desc(A), db = make_desc(Bm);
  const unsigned lda_b = (unsigned)g.lda * 2u, ldb_b = (unsigned)g.ldb * 2u;
  const unsigned kstep_a = AT ? KB * lda_b : KB * 2u, kstep_b = BT ? KB * ldb_b : KB * 2u;
  unsigned base[LPW];
  int ntile[LPW];
#pragma unroll
  for (int i = 0; i < LPW; i++) {
    const int j = wv * LPW + i;
    if (j < ALOADS) chunk_source<AT, BM, KB>(j * 64 + lane, m0, m_end, lda_b, k0, krange, g.a_gather, g.gather_div, &base[i], &ntile[i]);
    else if (!AT && !BT && TN == 2 && g.act_half)
      chunk_source_gate_up((j - ALOADS) * 64 + lane, bx * (BN / 2), g.act_half, ldb_b, k0, krange, &base[i], &ntile[i]);
    else chunk_source<BT, BN, KB>((j - ALOADS) * 64 + lane, n0, g.N, ldb_b, k0, krange, nullptr, 1, &base[i], &ntile[i]);
  }
  const unsigned lds0 = lds_address(smem);
  const unsigned lw = __builtin_amdgcn_readfirstlane(lds0 + (unsigned)wv * LPW * 1024u);
  // The k-tiles are walked from a start that differs from workgroup to workgroup (and wraps around): workgroups
  // that stream weights from HBM otherwise all ask for the same address bits above the cache-line offset at the
  // same time (every tile row starts a multiple of 4 KiB from its operand's base), which lands on a few memory
  // channels at a time; staggered starts spread the requests over all of them.  The sum over k is the same set of
  // products in a rotated, per-tile fixed order.
  const int rot = __builtin_amdgcn_readfirstlane(nk > 0 ? rot_seed % nk : 0);
  auto issue = [&](int kt, int i) {                  // wave-load i of the kt-th k-tile walked, into stage kt % NS
    const bool isA = (wv * LPW + i) < ALOADS;        // wave-uniform
    const int kr = kt + rot >= nk ? kt + rot - nk : kt + rot;
    const unsigned off = (kt < nk && kr < ntile[i]) ? base[i] + (unsigned)kr * (isA ? kstep_a : kstep_b) : OOB;
    const unsigned dst = lw + (unsigned)(kt % NS) * STAGE + i * 1024;
    if (ONCE && !isA) load_lds_b128_once(db, dst, off);
    else load_lds_b128(isA ? da : db, dst, off);
  };

  f32x16 acc[TE][TN];
#pragma unroll
  for (int i = 0; i < TE; i++)
#pragma unroll
    for (int j = 0; j < TN; j++)
#pragma unroll
      for (int e = 0; e < 16; e++) acc[i][j][e] = 0.f;
  unsigned fba[TE], fbb[TN];
#pragma unroll
  for (int i = 0; i < TE; i++) fba[i] = frag_base<AT, BM>(wm + i * 32, lane);
#pragma unroll
  for (int j = 0; j < TN; j++) fbb[j] = BM * KB * 2u + frag_base<BT, BN>(wn + j * 32, lane);

  // ---- pipeline: tiles kt+1 .. kt+NS-1 are in flight while tile kt is multiplied.  A tile past the end of the
  // k range is loaded as zeros (OOB), so every iteration issues the same number of loads and the wait count
  // below is a constant.
#pragma unroll
  for (int p = 0; p < NS - 1; p++)
#pragma unroll
    for (int i = 0; i < LPW; i++) issue(p, i);
  for (int kt = 0; kt < nk; kt++) {
    wait_vmcnt<LPW * (NS - 2)>();                    // this wave's share of tile kt has landed in LDS
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // and its LDS reads of tile kt-1 have returned
    __builtin_amdgcn_s_barrier();                    // ... for every wave: stage (kt-1) % NS may be overwritten
    const unsigned char* st = smem + (kt % NS) * STAGE;
    // fragments of k-step kk+1 are fetched from LDS, and a share of the loads of tile kt+NS-1 issued, while the
    // MFMAs of k-step kk run
    bf16x8 fa[2][TE], fb[2][TN];
#pragma unroll
    for (int i = 0; i < TE; i++) fa[0][i] = load_frag<AT, BM>(st, fba[i], wm + i * 32, 0, lane);
#pragma unroll
    for (int j = 0; j < TN; j++) fb[0][j] = load_frag<BT, BN>(st, fbb[j], wn + j * 32, 0, lane);
#pragma unroll
    for (int kk = 0; kk < KS; kk++) {
#pragma unroll
      for (int i = kk * LPW / KS; i < (kk + 1) * LPW / KS; i++) issue(kt + NS - 1, i);
      if (kk + 1 < KS) {
#pragma unroll
        for (int i = 0; i < TE; i++) fa[(kk + 1) & 1][i] = load_frag<AT, BM>(st, fba[i], wm + i * 32, kk + 1, lane);
#pragma unroll
        for (int j = 0; j < TN; j++) fb[(kk + 1) & 1][j] = load_frag<BT, BN>(st, fbb[j], wn + j * 32, kk + 1, lane);
      }
#pragma unroll
      for (int i = 0; i < TE; i++)
#pragma unroll
        for (int j = 0; j < TN; j++)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[kk & 1][i], fb[kk & 1][j], acc[i][j], 0, 0, 0);
    }
  }
  wait_vmcnt<0>();                                   // the zero-filled loads past the last tile

  // Weight gradients go out in whole lines: through LDS (every wave its own rows of 128 bytes), 16 bytes per lane.  Stores
  // past the caches are not merged on the way (see GemmArgs::once), and in pieces of 64 bytes they were what bound these
  // kernels: 8 rows per expert 96 and 191 us; a step of 128 tokens 1176 -> 1130 us, of 512 1514 -> 1475, 4 x 512
  // 2749 -> 2705, 4 blocks of 1024 7873 -> 7704, 8 experts of 14336, 60 tokens, 2683 -> 2529.
  // (Tiles whose waves are 32 columns wide, for small gradients, store 64 bytes at a time from the registers.  Two waves' halves put
  // together, past the caches or not, took the same time: 512-wide block, 400 tokens 323 us per step in all four forms, 1500 tokens
  // 451 to 454, with a kernel that reads the gradients behind it 338 and 471.  The same for buffers that are not 16-byte aligned:
  // 512 tokens at the Qwen shape 1676 us past the caches, 1680 through them.)
  if constexpr (AT && BT && sizeof(TC) == 2 && TN == 2 && (unsigned)NW * TE * 32 * 128 <= NS * STAGE) {
    if (whole_lines(g, C, bias_ptr)) {
      const int mw = m0 + wm, nw = n0 + wn + (lane & 7) * 8;
      unsigned char* own = smem + (unsigned)wv * (TE * 32 * 128);
      const int lr = (lane >> 5) * 4 + (lane & 1), lc = ((lane & 31) & ~1) * 2;
      __syncthreads();                               // every wave is done with the stages
#pragma unroll
      for (int i = 0; i < TE; i++)
#pragma unroll
        for (int e = 0; e < 16; e += 2)
#pragma unroll
          for (int j = 0; j < TN; j++)
            *(bf16x2*)(own + (i * 32 + (e >> 2) * 8 + (e & 3) + lr) * 128 + j * 64 + lc) = pair_rows_bf16(lane & 1, acc[i][j][e], acc[i][j][e + 1]);
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      TC* cp = C + (i64)(mw + (lane >> 3)) * g.ldc + nw;
#pragma unroll
      for (int t = 0; t < TE * 4; t++)               // (the width is a multiple of 8)
        if (mw + t * 8 + (lane >> 3) < m_end && nw < g.N)
          __builtin_nontemporal_store(*(const u32x4*)(own + t * 1024 + lane * 16), (u32x4*)(cp + (i64)t * 8 * g.ldc));
      return;
    }
  }
  int rb[TE], cb[TN];
#pragma unroll
  for (int i = 0; i < TE; i++) rb[i] = wm + i * 32;
#pragma unroll
  for (int j = 0; j < TN; j++) cb[j] = wn + j * 32;
  gemm_epilogue<BM, BN, AT, BT, TC, TE, TN>(g, C, bias_ptr, bx, m0, m_end, rb, cb, (wn >> 6) * 32, acc);
}

// ---- 256x256 tile in phases ------------------------------------------------------------------------------------------
// The plain loop above waits once per k-tile for everything it has asked for; with 64 KiB per stage only two stages fit,
// so the last loads of a k-tile are issued right before the wait for them and their latency (1300-2200 clocks) is in the
// open.  Here a k-tile is two phases, the upper and the lower half of the tile's rows, and LDS holds two k-tiles as half
// tiles of 16 KiB (A0 A1: 128 rows each, B0 B1: 128 columns each):
//   phase 0: read A0 B0 B1, multiply A0 x (B0 B1), ask for A1 of k-tile t + 1
//   phase 1: read A1,       multiply A1 x (B0 B1), ask for A0 B0 B1 of k-tile t + 2
// (8 waves as 2 x 4, a wave owns 64 rows x 2 x 32 columns of each half).  Every load has three phases to arrive and a wait
// never asks for the youngest four half tiles.
// The two waves of a SIMD run half a phase apart: while one multiplies (16 MFMAs), the other reads its next fragments and
// issues loads; a barrier at each half phase keeps them so.  Measured, 8192 x 2048 with k = 2048 / 4096: 81 -> 61 / 153 ->
// 108 us, i.e. 1.47 us per k-tile (1.46 PFLOP/s) once running; with all-zero operands 0.99 us (2.2 PFLOP/s, 86 % of the
// pipe), so what is left is the power limit, and 13 us of launch, first loads and 33 MB of results.
// (Four phases of 8 MFMAs: 5 % slower, the barriers; all eight waves in step: 25 % slower; one wave per SIMD with 128 x 128
// outputs, a third less LDS traffic: 6-15 % slower, its loads hold up its own MFMAs.)
//
// TE = 5: 320 rows, for an expert's last tile (expert_rows_c): a third phase reads A2 (64 rows, 32 per wave) and multiplies it by
// the same B, 8 MFMAs more for the half that 64 rows would otherwise be a tile of their own for.  Loads: A2 of k-tile t + 1 in phase 0,
// A0 B0 B1 of t + 2 in phase 1, A1 of t + 2 in phase 2.  251 to 256 registers, so its kernels have one epilogue each (KIND).
//
// What the barriers guarantee (segment n lies between barriers n and n+1; waves 0-3 read fragments of phase p in segment
// 2p and multiply in 2p+1, waves 4-7 one segment later):
//  * at the end of a read segment a wave waits for all but its youngest 8 loads (TE = 5: 10, 15, 11 by phase), which covers the half tiles that the next
//    phase reads; the first reader comes after a barrier that everybody passes after that wait;
//  * a wave has its fragments in registers when its read segment ends (lgkmcnt(0)), so those of phase p have been read by
//    everybody before segment 2p+2, and the first load into their half tile is issued in segment 2p+2 (phase p+1) or later.
template <bool AT, bool BT, class TC, int TE = 4, int KIND = 0>
__device__ __forceinline__ void gemm_tile_phased(const GemmArgs& g, const bf16* A, const bf16* Bm, TC* C, const void* bias_ptr,
                                                 int bx, int m0, int m_end, int k0, int k_end) {
  constexpr bool TALL = TE == 5;                     // 320 rows
  static_assert(TE == 4 || (TALL && !AT), "A2 is laid out rows x k");
  constexpr unsigned HALF = 128 * BK * 2, STAGE = 4 * HALF + (TALL ? HALF / 2 : 0);       // A0 A1 B0 B1 (A2)
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  const int n0 = bx * 256;
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = (wv >> 2) * 64, wn = (wv & 3) * 32;              // inside a half
  const int krange = k_end - k0;
  const int nk = (krange + BK - 1) / BK;
  const u32x4 da = make_desc(A), db = make_desc(Bm);
  const unsigned lda_b = (unsigned)g.lda * 2u, ldb_b = (unsigned)g.ldb * 2u;
  const unsigned kstep_a = AT ? BK * lda_b : BK * 2u, kstep_b = BT ? BK * ldb_b : BK * 2u;
  // wave-loads 2 wv and 2 wv + 1 of each half tile.  A row (column) past the end has an offset out of range for good; k's
  // past the end can only be in the last k-tile.
  unsigned base[4][2];
#pragma unroll
  for (int h = 0; h < 2; h++)
#pragma unroll
    for (int i = 0; i < 2; i++) {
      const int pos = (wv * 2 + i) * 64 + lane;
      int in;
      chunk_source<AT, 128>(pos, m0 + h * 128, m_end, lda_b, k0, 1 << 30, g.a_gather, g.gather_div, &base[h][i], &in);
      if (!in) base[h][i] = OOB;
      // (SwiGLU epilogue: B0 holds gate columns, B1 the up columns of the same indices)
      const int r0 = !BT && g.act_half ? h * g.act_half + bx * 128 : n0 + h * 128;
      const int lim = !BT && g.act_half ? (h + 1) * g.act_half : g.N;
      chunk_source<BT, 128>(pos, r0, lim, ldb_b, k0, 1 << 30, nullptr, 1, &base[2 + h][i], &in);
      if (!in) base[2 + h][i] = OOB;
    }
  unsigned base2 = OOB;                              // A2: 64 rows, a wave-load per wave
  if constexpr (TALL) {
    int in;
    chunk_source<false, 64>(wv * 64 + lane, m0 + 256, m_end, lda_b, k0, 1 << 30, g.a_gather, g.gather_div, &base2, &in);
    if (!in) base2 = OOB;
  }
  const unsigned lds0 = lds_address(smem);
  const unsigned lw = __builtin_amdgcn_readfirstlane(lds0 + (unsigned)wv * 2048u);
  const int kfull = krange / BK;                     // whole k-tiles
  auto issue = [&](int kt, int hf) {                 // this wave's part of half tile hf (A0 A1 B0 B1) of k-tile kt
    const unsigned soff = (unsigned)kt * (hf < 2 ? kstep_a : kstep_b), dst = lw + (unsigned)(kt & 1) * STAGE + hf * HALF;
    if (kt < kfull) {
#pragma unroll
      for (int i = 0; i < 2; i++) load_lds_b128_s(hf < 2 ? da : db, dst + i * 1024, base[hf][i], soff);
    } else {
      const int krem = krange - kt * BK;
#pragma unroll
      for (int i = 0; i < 2; i++) {
        const int pos = (wv * 2 + i) * 64 + lane;
        const bool in = (hf < 2 ? AT : BT) ? pos / 16 < krem : (((pos & 7) ^ ((pos >> 4) & 7)) << 3) < krem;
        load_lds_b128_s(hf < 2 ? da : db, dst + i * 1024, in ? base[hf][i] : OOB, soff);
      }
    }
  };
  auto issue_a2 = [&](int kt) {
    const int pos = wv * 64 + lane;
    const bool in = (((pos & 7) ^ ((pos >> 4) & 7)) << 3) < krange - kt * BK;
    load_lds_b128_s(da, __builtin_amdgcn_readfirstlane(lds0 + (unsigned)(kt & 1) * STAGE + 4 * HALF + (unsigned)wv * 1024u), in ? base2 : OOB, (unsigned)kt * kstep_a);
  };
  f32x16 acc[TE][2];
#pragma unroll
  for (int i = 0; i < TE; i++)
#pragma unroll
    for (int j = 0; j < 2; j++)
#pragma unroll
      for (int e = 0; e < 16; e++) acc[i][j][e] = 0.f;
  unsigned fba[2], fbb;
#pragma unroll
  for (int i = 0; i < 2; i++) fba[i] = frag_base<AT, 128>(wm + i * 32, lane);
  fbb = frag_base<BT, 128>(wn, lane);
  const int wm2 = (wv >> 2) * 32;
  const unsigned fba2 = frag_base<false, 64>(wm2, lane);

  auto issue3 = [&](int kt) { issue(kt, 0); issue(kt, 2); issue(kt, 3); };
  issue3(0); issue(0, 1);
  if constexpr (TALL) issue_a2(0);
  issue3(1);
  if constexpr (TALL) issue(1, 1);
  wait_vmcnt<TALL ? 11 : 8>();                                   // A0 B0 B1 of k-tile 0
  __builtin_amdgcn_s_barrier();
  if (wv >= 4) __builtin_amdgcn_s_barrier();         // waves 4-7 half a phase behind
  // a tile with no row in its lower half (the last one of an expert, often) does only its loads (out of range, to keep
  // the counts) and barriers in phase 1
  const bool lower = m_end - m0 > 128;
  bf16x8 fa[2][4], fb[2][4];
  for (int kt = 0; kt < nk; kt++) {
    const unsigned char* st = smem + (unsigned)(kt & 1) * STAGE;
#pragma unroll
    for (int p = 0; p < 2; p++) {
      // ---- read this phase's new fragments, ask for the half tiles whose places are free
      if (p == 0 || lower)
#pragma unroll
      for (int kk = 0; kk < 4; kk++) {
#pragma unroll
        for (int i = 0; i < 2; i++) fa[i][kk] = load_frag<AT, 128>(st + p * HALF, fba[i], wm + i * 32, kk, lane);
        if (p == 0)
#pragma unroll
          for (int j = 0; j < 2; j++) fb[j][kk] = load_frag<BT, 128>(st + (2 + j) * HALF, fbb, wn, kk, lane);
      }
      if constexpr (!TALL) {
        if (p == 0) issue(kt + 1, 1); else issue3(kt + 2);
        wait_vmcnt<8>();
      } else if (p == 0) {
        issue_a2(kt + 1);
        wait_vmcnt<10>();
      } else {
        issue3(kt + 2);
        wait_vmcnt<15>();
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
      // ---- multiply
      __builtin_amdgcn_s_setprio(1);
      if (p == 0 || lower)
#pragma unroll
      for (int kk = 0; kk < 4; kk++)
#pragma unroll
        for (int i = 0; i < 2; i++)
#pragma unroll
          for (int j = 0; j < 2; j++)
            acc[p * 2 + i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i][kk], fb[j][kk], acc[p * 2 + i][j], 0, 0, 0);
      __builtin_amdgcn_s_setprio(0);
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
    }
    if constexpr (TALL) {                            // phase 2
#pragma unroll
      for (int kk = 0; kk < 4; kk++) fa[0][kk] = load_frag<false, 64>(st + 4 * HALF, fba2, wm2, kk, lane);
      issue(kt + 2, 1);
      wait_vmcnt<11>();
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_setprio(1);
#pragma unroll
      for (int kk = 0; kk < 4; kk++)
#pragma unroll
        for (int j = 0; j < 2; j++) acc[TE - 1][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[0][kk], fb[j][kk], acc[TE - 1][j], 0, 0, 0);
      __builtin_amdgcn_s_setprio(0);
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
    }
  }
  if (wv < 4) __builtin_amdgcn_s_barrier();
  wait_vmcnt<0>();                                   // the zero-filled loads past the last k-tile
  int rb[TE], cb[2];
  if constexpr (TALL) rb[TE - 1] = 256 + wm2;
#pragma unroll
  for (int i = 0; i < 4; i++) rb[i] = (i >> 1) * 128 + wm + (i & 1) * 32;
  cb[0] = wn; cb[1] = 128 + wn;
  // weight gradients in whole lines, as above; a wave's columns are 64 bytes here and 64 there, so the tile is put together
  // first.  (Rows are 512 bytes apart: the 16-byte chunk moves with the row, so that a write meets no bank twice.)
  if constexpr (AT && BT && sizeof(TC) == 2) {
    if (whole_lines(g, C, bias_ptr)) {
      auto at = [&](int row, int byte) { return smem + row * 512 + ((unsigned)byte ^ ((unsigned)(row & 1) * 64u + (unsigned)((row >> 2) & 1) * 128u)); };
      __syncthreads();
#pragma unroll
      for (int i = 0; i < 4; i++)
#pragma unroll
        for (int e = 0; e < 16; e += 2)
#pragma unroll
          for (int j = 0; j < 2; j++)
            *(bf16x2*)at(rb[i] + (e >> 2) * 8 + (e & 3) + (lane >> 5) * 4 + (lane & 1), cb[j] * 2 + ((lane & 31) & ~1) * 2) =
                pair_rows_bf16(lane & 1, acc[i][j][e], acc[i][j][e + 1]);
      __syncthreads();
      const int n = bx * 256 + (lane & 31) * 8;
#pragma unroll
      for (int t = 0; t < 16; t++) {
        const int row = wv * 32 + t * 2 + (lane >> 5);
        if (m0 + row < m_end && n < g.N)
          __builtin_nontemporal_store(*(const u32x4*)at(row, (lane & 31) * 16), (u32x4*)(C + (i64)(m0 + row) * g.ldc + n));
      }
      return;
    }
  }
  gemm_epilogue<TE * 64, 256, AT, BT, TC, TE, 2, KIND>(g, C, bias_ptr, bx, m0, m_end, rb, cb, wn, acc);
}

template <int BM, int BN, int WGM, bool AT, bool BT, class TC, int NW, int NS, int KB = BK, bool ONCE = false>
__global__ void __launch_bounds__(NW * 64) gemm_mfma_k(GemmArgs g) {
  constexpr int TM = BM / WGM / 32;
  const bf16* A = (const bf16*)g.A;
  const bf16* Bm = (const bf16*)g.B;
  TC* C = (TC*)g.C;
  const void* bias = g.bias;
  // ---- which tile this workgroup computes (plain 2-D grid, or the XCD-aware placement of a 1-D grid)
  int bx = blockIdx.x, by = blockIdx.y, bz = blockIdx.z;
  if (g.xcd_m != 0 && !place_tile(g.group_mode, g.xcd_m, g.tiles_m, g.tiles_n, g.n_groups,
                                  g.group_mode == 0 ? 0 : g.tile_count[0], g.tile_first, (int)blockIdx.x, &bx, &by, &bz))
    return;
  int m0, m_end, k0 = 0, k_end = g.K, rot_seed = 0;
  if (g.group_mode == 1) {
    if (!BT) rot_seed = by;     // per row tile (weights with k as the slow index are spread by their column tile already)
    int ti = by;
    int grp = g.tile_group[ti];
    if (grp < 0) return;
    m0 = g.tile_m0[ti];
    m_end = min(g.offsets[grp + 1], m0 + BM);
    Bm += (i64)grp * g.b_group_stride;
  } else {
    m0 = by * BM;
    m_end = g.M;
    if (g.group_mode == 2) {
      int grp = bz;
      k0 = g.offsets[grp];
      k_end = g.offsets[grp + 1];
      C += (i64)grp * g.c_group_stride;
    } else if (g.n_sub > 1 && bz > 0) {              // one of several problems of one shape launched together
      // (constant indices: the argument block stays in scalar registers)
      if (bz == 1) { A = (const bf16*)g.subA[0]; Bm = (const bf16*)g.subB[0]; C = (TC*)g.subC[0]; bias = g.subBias[0]; }
      else { A = (const bf16*)g.subA[1]; Bm = (const bf16*)g.subB[1]; C = (TC*)g.subC[1]; bias = g.subBias[1]; }
    }
  }
  if (g.row_skip && g.group_mode == 0) {             // nothing to do if every row of the tile is marked as finished
    // every wave looks at all rows of the tile itself and reaches the same answer: no LDS, no barrier (a block-wide
    // vote adds 1 KiB of static LDS in front of the stages, which a tile that uses all 160 KiB for them cannot afford)
    int live = 0;
    for (int r = m0 + (int)(threadIdx.x & 63); r < min(m_end, m0 + BM); r += 64) live |= g.row_skip[r] == 0;
    if (!__any(live)) return;
  }
  if constexpr (NS == PHASED) gemm_tile_phased<AT, BT, TC>(g, A, Bm, C, bias, bx, m0, m_end, k0, k_end);
  else gemm_tile<BM, BN, WGM, AT, BT, TC, NW, NS, TM, KB, ONCE>(g, A, Bm, C, bias, bx, bz, m0, m_end, k0, k_end, rot_seed);
}

// The routed experts' 256x256 tiles where an expert's last one may have up to 320 rows (list c, expert_rows_c)
template <bool BT, bool ACT>
__global__ void __launch_bounds__(512) expert_tall_k(GemmArgs g) {
  int bx, by, bz = 0;
  if (!place_tile(1, 1, 0, g.tiles_n, 1, g.tile_count[0], g.tile_first, (int)blockIdx.x, &bx, &by, &bz)) return;
  const int grp = g.tile_group[by];
  if (grp < 0) return;
  const int m0 = g.tile_m0[by], rows_end = g.offsets[grp + 1];
  const bf16* B = (const bf16*)g.B + (i64)grp * g.b_group_stride;
  if (rows_end - m0 > 256 && rows_end - m0 <= 320) gemm_tile_phased<false, BT, bf16, 5, ACT ? 2 : 1>(g, (const bf16*)g.A, B, (bf16*)g.C, nullptr, bx, m0, rows_end, 0, g.K);
  else gemm_tile_phased<false, BT, bf16, 4, ACT ? 2 : 1>(g, (const bf16*)g.A, B, (bf16*)g.C, nullptr, bx, m0, min(rows_end, m0 + 256), 0, g.K);
}
template <bool BT, bool ACT>
static void go_tall(GemmArgs g, hipStream_t s) {
  g.tiles_n = ACT ? cdiv(g.act_half, 128) : cdiv(g.N, 256);
  g.tiles_m = g.max_tiles;
  constexpr size_t smem = 2 * (320 + 256) * BK * 2;
  static std::atomic<unsigned long long> attr_mask{0};
  if (attr_needed(attr_mask)) {
    (void)hipFuncSetAttribute((const void*)expert_tall_k<BT, ACT>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    attr_done(attr_mask);
  }
  hipLaunchKernelGGL((expert_tall_k<BT, ACT>), dim3(g.tiles_n * g.tiles_m), dim3(512), smem, s, g);
}

// REVFFN_XCD (tuning aid): 0 = plain 2-D grids, tiles land on the XCDs round-robin
static int xcd_enabled() {
  static int v = -1;
  if (v < 0) { const char* e = getenv("REVFFN_XCD"); v = e ? atoi(e) : 1; }
  return v;
}

template <int BM, int BN, int WGM, bool AT, bool BT, class TC, int NW, int NS, int KB = BK, bool ONCE = false>
static void go(const GemmArgs& g0, hipStream_t s) {
  GemmArgs g = g0;
  { static int off = -1; if (off < 0) { const char* e = getenv("REVFFN_NO_PACKED_STORES"); off = e ? atoi(e) : 0; } g.no_packed_stores = off; }
  g.tiles_n = g.act_half ? cdiv(g.act_half, BN / 2) : cdiv(g.N, BN);
  g.tiles_m = g.group_mode == 1 ? g.max_tiles : cdiv(g.M, BM);
  const int zdim = g.group_mode == 2 ? g.n_groups : (g.group_mode == 0 ? g.n_sub : 1);
  if (g.tiles_n <= 0 || g.tiles_m <= 0 || zdim <= 0) return;
  dim3 grid(g.tiles_n, g.tiles_m, zdim);
  g.xcd_m = 0;
  if (xcd_enabled()) {
    if (g.group_mode == 1) {
      if (g.tile_count) { g.xcd_m = 1; grid = dim3(g.tiles_n * g.tiles_m, 1, 1); }
    } else if (g.group_mode == 2) {
      // two XCDs per expert while the routing is even (decided on the device, by the permutation kernel): 3.1x fewer
      // operand bytes cross the fabric and these kernels are 6.5 % faster; whole experts per XCD fetch even less
      // but leave XCDs idle, four XCDs per expert split 1408 columns unevenly (both measured slower)
      if (g.tile_count) { g.xcd_m = 2; grid = dim3((unsigned)wgrad_grid_x(2, g.tiles_m, g.tiles_n, g.n_groups), 1, 1); }
    } else if ((i64)g.tiles_n * g.tiles_m >= 64) {
      g.xcd_m = pick_xcd_m(g.tiles_m, g.tiles_n, BM, BN);
      grid = dim3(dense_grid_x(g.xcd_m, g.tiles_m, g.tiles_n), 1, zdim);
    }
  }
  constexpr size_t smem = (size_t)(NS == PHASED ? 2 : NS) * (BM + BN) * KB * 2;
  static_assert(smem <= 160 * 1024, "LDS stages exceed the CU's 160 KiB");
  static std::atomic<unsigned long long> attr_mask{0};
  if (attr_needed(attr_mask)) {
    (void)hipFuncSetAttribute((const void*)gemm_mfma_k<BM, BN, WGM, AT, BT, TC, NW, NS, KB, ONCE>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    attr_done(attr_mask);
  }
  hipLaunchKernelGGL((gemm_mfma_k<BM, BN, WGM, AT, BT, TC, NW, NS, KB, ONCE>), grid, dim3(NW * 64), smem, s, g);
}

// The tile shapes: 256x128 and 128x256 (8 waves, one workgroup per CU), 256x256 (2 stages), 128x128 (8 waves of 32x64,
// 4 stages: with one workgroup per CU, two waves per SIMD hide each other's LDS and barrier waits; 10-17 % faster than
// 4 waves of 64x64 on the 2048^3 projections) and 128x64 (8 waves of 32x32, two workgroups per CU; 1.5 % of a step
// over 4 waves of 64x32, measured on one box with both builds).  64x64 (4 waves of 32x32, 4 stages) and 128x64 with a fourth
// stage for narrow results, 256x256 with 4 stages of 32 rows for per-expert weight gradients: see pick_tile.
template <bool AT, bool BT, class TC> static void go_256x128(const GemmArgs& g, hipStream_t s) { go<256, 128, 4, AT, BT, TC, 8, 3>(g, s); }
template <bool AT, bool BT, class TC> static void go_256x256(const GemmArgs& g, hipStream_t s) { go<256, 256, 2, AT, BT, TC, 8, PHASED>(g, s); }
template <bool AT, bool BT, class TC> static void go_128x128(const GemmArgs& g, hipStream_t s) { go<128, 128, 4, AT, BT, TC, 8, 4>(g, s); }
template <bool AT, bool BT, class TC> static void go_128x256(const GemmArgs& g, hipStream_t s) { go<128, 256, 2, AT, BT, TC, 8, 3>(g, s); }
template <bool AT, bool BT, class TC> static void go_128x64(const GemmArgs& g, hipStream_t s) { go<128, 64, 4, AT, BT, TC, 8, 3>(g, s); }
// 160x256 for the routed experts' forward GEMMs where one 160-row tile holds a typical expert: 4 waves side by side,
// each 160 rows x 64 columns (a gate and an up block for the SwiGLU epilogue), one wave per SIMD, 3 stages of 52 KiB
template <bool AT, bool BT, class TC> static void go_160x256(const GemmArgs& g, hipStream_t s) { go<160, 256, 1, AT, BT, TC, 4, 3>(g, s); }

template <bool AT, bool BT, class TC>
static void pick_tile(const GemmArgs& g, hipStream_t s) {
  // Dense problems: the tile whose rounds of workgroups over the 256 CUs cost least.  One tile of 256x128 takes about
  // 1.85 times, one of 256x256 (in phases) about 2.6 times as long as one of 128x128 (measured at 1024 to
  // 8192 tokens: larger tiles do more work per loaded byte, but a last, partly filled round costs a whole tile's time).
  auto dense_choice = [&]() {
    const int z = g.n_sub;
    // (a launch that runs beside others on a helper stream fills only the CUs it needs: its cost is its tile count.
    // Not for a problem of fewer than 128 of the largest tiles: on a fraction of the CUs it takes several times as
    // long, and helper streams are chains too -- 32-tile weight gradients at the end of a call were the last thing
    // running, on an eighth of the chip.)
    const bool bulk = g.bulk && (i64)cdiv(g.M, 256) * cdiv(g.N, 256) * z >= 128;
    auto rounds = [&](int bm, int bn) {
      const i64 tiles = (i64)cdiv(g.M, bm) * cdiv(g.N, bn) * z;
      return bulk ? (double)tiles / 256.0 : (double)cdiv(tiles, 256);
    };
    const double c2 = rounds(128, 128), c3 = 1.85 * rounds(256, 128), c4 = 2.6 * rounds(256, 256);
    return (c4 < c3 && c4 < c2) ? 4 : (c3 < c2 ? 3 : 2);
  };
  if (g.act_half && g.group_mode == 0) {
    // SwiGLU epilogue: only tiles whose waves are 64 columns wide (a gate and an up block)
    switch (g.force_tile >= 2 ? g.force_tile : dense_choice()) {
      case 4: go_256x256<AT, BT, TC>(g, s); break;
      case 3: go_256x128<AT, BT, TC>(g, s); break;
      default: go_128x128<AT, BT, TC>(g, s);
    }
    return;
  }
  if (g.group_mode != 1 && g.force_tile) {           // a unit test asks for one of the shapes (dense problems)
    switch (g.force_tile) {
      case 1: go_128x64<AT, BT, TC>(g, s); return;
      case 2: go_128x128<AT, BT, TC>(g, s); return;
      case 3: go_256x128<AT, BT, TC>(g, s); return;
      case 4:
        go_256x256<AT, BT, TC>(g, s);
        return;
    }
  }
  if (g.group_mode == 1) {
    // expert tiles.  Skipping the MFMAs of the 32-row blocks past an expert's end (waves spanning all rows, a loop
    // specialised per block count) measured no gain, and neither did a fifth LDS stage.
    if constexpr (!AT) {
      if constexpr (!BT) { if (g.tile_bm == 160) { go_160x256<AT, BT, TC>(g, s); return; } }
      if (g.tile_bm == 256 && g.tile_bn == 256) go_256x256<AT, BT, TC>(g, s);
      else if (g.tile_bm == 256) go_256x128<AT, BT, TC>(g, s);
      else if (g.tile_bn == 256 && g.once) go<128, 256, 2, AT, BT, TC, 8, 3, BK, true>(g, s);   // (a kernel of its own: a branch costs 1 % of a skewed 2 x 2048 step)
      else if (g.tile_bn == 256) go_128x256<AT, BT, TC>(g, s);
      else go_128x128<AT, BT, TC>(g, s);
    }
    return;
  }
  if (g.group_mode == 2) {
    // per-expert weight gradients: the k range is one expert's rows, a few k-tiles only, so a workgroup is mostly
    // fixed cost (start-up, first load latency) and output stores, none of which overlap on a CU that holds one
    // workgroup.  The largest tile, 256x256 (2 stages), spreads the fixed cost over the most output: 12 % faster than
    // 256x128 on these kernels and 1-1.6 % of a step, even where the last tile column is half empty (N = 1408).
    // Smaller tiles with two workgroups per CU (128x128 with 2 stages, 4 or 8 waves) were up to 7 % faster than
    // 256x128 alone but slower inside the step, next to the data-gradient chain on the main stream; a persistent
    // form of 256x128 (a workgroup walks over tiles and issues the next tile's first loads before it stores the
    // finished one) was 5 % faster alone and 3 % of a step slower.
    // With k-tiles of 32 rows (4 stages of 32 KiB) an expert of 137 rows is 5 k-tiles instead of 3 of 64 (17 % fewer
    // multiplied zero rows), and all but the last are in flight at once: these kernels 10 % faster, a step 1.1 %.
    // (5 stages: 8 % slower again; 3: the same.)
    // (The tile in phases is 6-25 % slower here at 8 to 546 rows per expert.)
    // All that holds from about one such tile per CU on.  With fewer (small blocks) 128x64 tiles put eight times the CUs to
    // work: a 512-wide block of 12 experts (48 and 24 tiles), 400 tokens 354 -> 344 us per step, 1536 tokens 518 -> 499.
    if constexpr (AT && BT) {
      if ((i64)cdiv(g.M, 256) * cdiv(g.N, 256) * g.n_groups <= 256) go_128x64<AT, BT, TC>(g, s);
      else go<256, 256, 2, AT, BT, TC, 8, 4, 32>(g, s);
      return;
    }
    return;                                            // (launch_gemm_mfma admits this mode for that layout only)
  }
  // below ~200 tiles of 128x128: 128x64 (two workgroups per CU)
  const i64 t128 = (i64)cdiv(g.M, 128) * cdiv(g.N, 128) * g.n_sub;
  if (t128 < 200 && g.N >= 128) {
    // With a CU per workgroup a fourth stage (a third k-tile in flight) is free: 1024 rows, 2048 outputs, k = 2048: 17.0 -> 16.0 us,
    // data gradient 19.1 -> 18.0; 700 rows 15.9 -> 14.8, 18.3 -> 16.4 (fifth and sixth: no change).  Half as many workgroups
    // as CUs: half as large tiles (1024 outputs: 19.1 -> 15.4 us, 17.2 with a fourth stage alone).
    const i64 t64 = (i64)cdiv(g.M, 128) * cdiv(g.N, 64) * g.n_sub;
    if (t64 <= 128) go<64, 64, 2, AT, BT, TC, 4, 4>(g, s);
    else if (t64 <= 256) go<128, 64, 4, AT, BT, TC, 8, 4>(g, s);
    else go_128x64<AT, BT, TC>(g, s);
    return;
  }
  switch (dense_choice()) {
    case 4:
      go_256x256<AT, BT, TC>(g, s);
      break;
    case 3:
      // (the same tile count either way; with k contiguous in both operands the wide tile measured 1-4 % faster)
      if (!AT && !BT && g.N % 256 == 0) go_128x256<AT, BT, TC>(g, s);
      else go_256x128<AT, BT, TC>(g, s);
      break;
    default: go_128x128<AT, BT, TC>(g, s);
  }
}

// ---- several weight gradients as one launch ------------------------------------------------------------------------
// The dense layers' weight gradients (4 to 10 per call, K = tokens) are leaves of the computation, so they can wait for
// each other and share the rounds of workgroups: alone a 2048 x 2048 result is 64 tiles of 256x256 for 256 CUs, so each
// ran on smaller, dearer tiles, and every launch had a last round of its own.
// Tiles are numbered over the problems, inside a problem in bands of 4 tile rows with the row fastest; XCD c takes one
// consecutive run of them, so that what it holds in its L2 at a time is a 4 x 8 block of one problem.
template <int BM, int BN, int WGM, class TC, int NW, int NS, int KB>
__global__ void __launch_bounds__(NW * 64) gemm_batch_tn_k(GemmBatch b) {
  typedef const __attribute__((address_space(4))) GemmBatch* KernArg;     // (indexed in the kernel-argument segment, where
  const KernArg ka = (KernArg)__builtin_amdgcn_kernarg_segment_ptr();     // a copy by value would go through scratch)
  const int total = ka->total, n = ka->n;
  const int c = (int)blockIdx.x & 7, loc = (int)blockIdx.x >> 3, q = total >> 3, r = total & 7;
  if (loc >= q + (c < r ? 1 : 0)) return;
  // (with experts among the problems, whose contractions are a fraction as long, a run each would leave XCDs idle: round-robin)
  const int id = ka->spread ? (int)blockIdx.x : c * q + (c < r ? c : r) + loc;
  if (id >= total) return;
  int i = 0;
  while (i + 1 < n && id >= ka->p[i + 1].tile0) i++;
  const int tm = ka->p[i].tiles_m, tn = ka->p[i].tiles_n;
  const int per = tm * tn, grp = (id - ka->p[i].tile0) / per;
  const int local = id - ka->p[i].tile0 - grp * per, band = local / (4 * tn), rem = local - band * 4 * tn;
  const int bh = tm - band * 4 < 4 ? tm - band * 4 : 4;
  const int bx = rem / bh, by = band * 4 + rem - bx * bh;
  GemmArgs g;
  g.M = ka->p[i].M; g.N = ka->p[i].N; g.K = ka->p[i].K;
  g.lda = ka->p[i].lda; g.ldb = ka->p[i].ldb; g.ldc = ka->p[i].ldc;
  const bf16 *A = (const bf16*)ka->p[i].A, *B = (const bf16*)ka->p[i].B;
  TC* C = (TC*)ka->p[i].C + (i64)grp * ka->p[i].c_stride;
  const bool grouped = ka->p[i].groups > 0;
  const int k0 = grouped ? ka->offsets[grp] : 0, k_end = grouped ? ka->offsets[grp + 1] : g.K;
  if constexpr (NS == PHASED) gemm_tile_phased<true, true, TC>(g, A, B, C, nullptr, bx, by * BM, g.M, k0, k_end);
  else gemm_tile<BM, BN, WGM, true, true, TC, NW, NS, BM / WGM / 32, KB>(g, A, B, C, nullptr, bx, 0, by * BM, g.M, k0, k_end, 0);
}
template <int BM, int BN, int WGM, class TC, int NW, int NS, int KB = BK>
static void go_batch(GemmBatch& b, hipStream_t s) {
  b.total = 0;
  for (int i = 0; i < b.n; i++) {
    GemmProb& p = b.p[i];
    p.tile0 = b.total; p.tiles_m = cdiv(p.M, BM); p.tiles_n = cdiv(p.N, BN);
    b.total += p.tiles_m * p.tiles_n * (p.groups ? p.groups : 1);
  }
  constexpr size_t smem = (size_t)(NS == PHASED ? 2 : NS) * (BM + BN) * KB * 2;
  static std::atomic<unsigned long long> attr_mask{0};
  if (attr_needed(attr_mask)) {
    (void)hipFuncSetAttribute((const void*)gemm_batch_tn_k<BM, BN, WGM, TC, NW, NS, KB>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    attr_done(attr_mask);
  }
  if (b.total > 0)
    hipLaunchKernelGGL((gemm_batch_tn_k<BM, BN, WGM, TC, NW, NS, KB>), dim3(cdiv(b.total, 8) * 8), dim3(NW * 64), smem, s, b);
}
template <class TC> static void pick_batch_tile(GemmBatch& b, bool bulk, hipStream_t s) {
  // the same costs per tile as for a single problem (pick_tile), over the tiles of all problems
  double t64 = 0, t128 = 0, t256x128 = 0, t256 = 0;
  bool experts = false;
  for (int i = 0; i < b.n; i++) {
    experts = experts || b.p[i].groups;
    const double n = b.p[i].groups ? b.p[i].groups : 1;
    t64 += n * cdiv(b.p[i].M, 128) * cdiv(b.p[i].N, 64);
    t128 += n * cdiv(b.p[i].M, 128) * cdiv(b.p[i].N, 128);
    t256x128 += n * cdiv(b.p[i].M, 256) * cdiv(b.p[i].N, 128);
    t256 += n * cdiv(b.p[i].M, 256) * cdiv(b.p[i].N, 256);
  }
  auto rounds = [&](double t) { return bulk && t256 >= 128 ? t / 256.0 : ceil(t / 256.0); };
  const double c2 = rounds(t128), c3 = 1.85 * rounds(t256x128), c4 = 2.6 * rounds(t256);
  b.spread = experts;
  if (experts) go_batch<128, 64, 4, TC, 8, 3>(b, s);                   // (what they take alone at these sizes, see pick_tile)
  else if (c4 < c2 && c4 < c3) go_batch<256, 256, 2, TC, 8, PHASED>(b, s);
  else if (c3 < c2) go_batch<256, 128, 4, TC, 8, 3>(b, s);
  else if (t128 >= 200) go_batch<128, 128, 4, TC, 8, 4>(b, s);
  else go_batch<128, 64, 4, TC, 8, 3>(b, s);
}
static bool aligned16(const void* p) { return ((uintptr_t)p & 15) == 0; }

// norm and rotation: rows of 16-byte pieces, whole tiles of heads, and nothing else in the epilogue
static bool norm_rope_ok(const GemmArgs& g, bool f32out) {
  if (!g.norm_g[0] && !g.rope_cs) return true;
  if (f32out || g.b_trans || g.act_half || g.resid || g.tap || g.group_mode != 0) return false;
  if (g.rope_cs && !rope_fits(g.rope_dh, g.N)) return false;
  if (g.norm_g[0] && g.K > 1024) return false;             // (a workgroup's pieces of the rows are in LDS all at once)
  for (int z = 0; g.norm_g[0] && z < g.n_sub; z++)
    if (!g.norm_g[z] || !aligned16(g.norm_g[z]) || !aligned16(g.norm_out[z])) return false;
  return true;
}

int launch_gemm_mfma(const GemmArgs& g, GemmTypes t, hipStream_t s) {
  if (t.ta != 1 || t.tb != 1 || t.tside != 1) return 1;
  if (!aligned16(g.A) || !aligned16(g.B) || (g.lda & 7) || (g.ldb & 7)) return 1;
  if ((g.b_group_stride & 7) || (g.c_group_stride & 7)) return 1;
  if (!g.a_trans && (g.K & 7)) return 1;
  if (!g.b_trans && (g.K & 7)) return 1;
  if (g.a_trans && (g.M & 7)) return 1;
  if (g.b_trans && (g.N & 7)) return 1;
  if (g.a_trans && !g.b_trans) return 1;                 // layout not used by the block
  if (g.group_mode == 2 && !(g.a_trans && g.b_trans)) return 1;
  if (g.group_mode == 1 && (g.a_trans || (g.tile_bm != 128 && !(g.few_rows && g.tile_bm == 32 && t.tc == 1) && g.tile_bm != 256 && !(g.tile_bm == 320 && t.tc == 1) && !(g.tile_bm == 160 && !g.b_trans && g.tile_bn == 256)))) return 1;
  if (g.a_gather && g.a_trans) return 1;
  if (g.group_mode != 1 && g.M <= 0) return 1;
  if (g.n_sub < 1 || g.n_sub > 3 || (g.n_sub > 1 && (g.group_mode != 0 || g.resid || g.tap || g.act_half))) return 1;
  for (int z = 1; z < g.n_sub; z++)
    if (!g.subA[z - 1] || !g.subB[z - 1] || !g.subC[z - 1] || !aligned16(g.subA[z - 1]) || !aligned16(g.subB[z - 1])) return 1;
  if (g.col_scale) return 1;                             // (the generic kernel's epilogue only)
  if (g.act_half) {
    if (g.a_trans || g.b_trans || g.group_mode == 2 || g.bias || g.resid || g.tap || !g.act_out) return 1;
    if (g.N != 2 * g.act_half) return 1;
  }
  // every operand must span less than 2 GiB from its base (32-bit buffer offsets)
  {
    const i64 lim = (i64)1 << 30;                        // elements
    i64 a_rows = g.a_trans ? g.K : g.M, b_rows = g.b_trans ? g.K : g.N;
    if (a_rows * g.lda >= lim || b_rows * g.ldb >= lim) return 1;
  }
  const bool f32out = t.tc == 0;
  if (!norm_rope_ok(g, f32out)) return 1;
  if (g.A2 && (!aligned16(g.A2) || !aligned16(g.B2) || !g.b_trans || f32out)) return 1;
  if (g.group_mode == 1 && g.tile_bm == 320) {
    if (g.act_half) go_tall<false, true>(g, s); else if (g.b_trans) go_tall<true, false>(g, s); else go_tall<false, false>(g, s);
    return 0;
  }
  if (g.few_rows && g.group_mode == 1 && g.stream) { launch_gemm_experts(g, s); return 0; }
  if (g.few_rows && !g.a_trans && !g.force_tile && (g.group_mode == 1 || (g.group_mode == 0 && !g.a_gather))) {
    launch_gemm_skinny(g, f32out, s);
    return 0;
  }
  if (g.A2 || g.dact_out || g.norm_g[0] || g.rope_cs) return 1;
  if (!g.a_trans && !g.b_trans) {
    if (f32out) pick_tile<false, false, float>(g, s); else pick_tile<false, false, bf16>(g, s);
  } else if (!g.a_trans && g.b_trans) {
    if (f32out) pick_tile<false, true, float>(g, s); else pick_tile<false, true, bf16>(g, s);
  } else {
    if (f32out) pick_tile<true, true, float>(g, s); else pick_tile<true, true, bf16>(g, s);
  }
  return 0;
}

int launch_gemm_batch_tn(GemmBatch& b, int out_f32, int bulk, hipStream_t s) {
  for (int i = 0; i < b.n; i++) {
    const GemmProb& p = b.p[i];
    if (!aligned16(p.A) || !aligned16(p.B) || (p.lda & 7) || (p.ldb & 7) || (p.M & 7) || (p.N & 7) || (p.c_stride & 7) || p.M <= 0) return 1;
    if ((i64)p.K * p.lda >= (i64)1 << 30 || (i64)p.K * p.ldb >= (i64)1 << 30) return 1;
  }
  if (b.n == 0) return 0;
  if (out_f32) pick_batch_tile<float>(b, bulk, s); else pick_batch_tile<bf16>(b, bulk, s);
  return 0;
}
