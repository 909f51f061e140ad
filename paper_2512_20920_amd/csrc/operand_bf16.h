// Operand tiles of the bf16 matrix-core kernels in LDS: where each 16-byte chunk of a direct load comes from, and how the
// fragments of v_mfma_f32_32x32x16_bf16 are read back.
//
// A wave-load fills 1 KiB of LDS in lane order, so bank-conflict-free fragment reads cannot come from row padding; each lane
// instead fetches the 16-byte chunk that belongs in its slot under an XOR swizzle:
//  * operand with the contraction index contiguous in memory ("rows x k"): LDS row = 128 bytes =
//    8 chunks, chunk c of row r sits in slot c ^ ((r >> 1) & 7); fragments are 16-byte reads;
//  * operand with the contraction index as the slow one ("k x rows", the transposed layouts of
//    the data- and weight-gradient GEMMs): kept as stored, LDS row k = ROWS*2 bytes, and the
//    64-byte group G of row k sits in group G ^ (k & 3) (ROWS = 64: G ^ ((k >> 1) & 1)); fragments
//    come from the transposing read ds_read_b64_tr_b16, whose lane mapping is: inside each block
//    of 16 lanes, lane j receives element (j & 3) of the 8-byte words addressed by lanes
//    4*e + (j >> 2), e = 0..3.
#pragma once
#include "lds_load.h"

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(8))) short s16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

#define BK 64

// Where the 16-byte chunk at LDS position `pos` (in chunks, lane order of the wave-loads) of one operand tile
// comes from: byte offset of that chunk at k-tile 0 relative to the operand base, and the number of k-tiles for
// which it lies inside the k range (0 = never: a row past the limit).  krange = elements of the k range.
template <bool TR, int ROWS, int KB = BK>
__device__ __forceinline__ void chunk_source(int pos, int row0, int row_lim, unsigned ld_bytes, int k0, int krange,
                                             const int* gather, int div, unsigned* base, int* ntiles) {
  static_assert(KB == BK || TR, "rows x k tiles are laid out for 128-byte rows");
  if (!TR) {
    const int r = pos >> 3, slot = pos & 7;
    const int c = slot ^ ((r >> 1) & 7);                          // k-chunk of row r that lives in this slot
    int row = row0 + r;
    const bool in = row < row_lim;
    if (!in) row = row_lim - 1;
    const unsigned rr = gather ? (unsigned)(gather[row] / div) : (unsigned)row;
    *base = rr * ld_bytes + (unsigned)(k0 + c * 8) * 2u;
    *ntiles = in ? (krange - c * 8 + BK - 1) / BK : 0;
  } else {
    constexpr int CPR = ROWS / 8;                                 // chunks per LDS row (one k)
    const int kr = pos / CPR, slot = pos % CPR;
    const int gsw = (CPR >= 16) ? (kr & 3) : ((kr >> 1) & 1);
    const int c = (((slot >> 2) ^ gsw) << 2) | (slot & 3);        // 8-element column chunk that lives in this slot
    const int col = row0 + c * 8;
    *base = (unsigned)(k0 + kr) * ld_bytes + (unsigned)col * 2u;
    *ntiles = col < row_lim ? (krange - kr + KB - 1) / KB : 0;
  }
}

// The same for the weight tile of a gate/up GEMM with the SwiGLU epilogue: LDS row r of the tile holds weight row
// (r>>5 & 1) * half + col0 + (r>>6) * 32 + (r & 31), i.e. each wave's 64 rows are 32 gate rows and the 32 up rows of
// the same columns col0 + 32 w .. + 31 (col0 = first gate column of the tile; columns >= half are zeros).
__device__ __forceinline__ void chunk_source_gate_up(int pos, int col0, int half, unsigned ld_bytes, int k0, int krange,
                                                     unsigned* base, int* ntiles) {
  const int r = pos >> 3, slot = pos & 7;
  const int c = slot ^ ((r >> 1) & 7);
  int col = col0 + (r >> 6) * 32 + (r & 31);
  const bool in = col < half;
  if (!in) col = half - 1;
  const unsigned row = (unsigned)(((r >> 5) & 1) * half + col);
  *base = row * ld_bytes + (unsigned)(k0 + c * 8) * 2u;
  *ntiles = in ? (krange - c * 8 + BK - 1) / BK : 0;
}

// Per-lane LDS byte offset (inside the operand's tile, k-step kk = 0) of the MFMA fragment rows r0..r0+31:
// lane (r = lane & 31, g = lane >> 5) holds k = 16*kk + 8*g .. +7 of row r0 + r.
template <bool TR, int ROWS>
__device__ __forceinline__ unsigned frag_base(int r0, int lane) {
  if (!TR) return (unsigned)(r0 + (lane & 31)) * 128u;
  const int blk = lane >> 4, i = lane & 15;
  const int kr = (blk >> 1) * 8 + (i >> 2);
  const int col = r0 + (blk & 1) * 16 + (i & 3) * 4;
  constexpr int CPR = ROWS / 8;
  const int c = col >> 3;
  const int gsw = (CPR >= 16) ? (kr & 3) : ((kr >> 1) & 1);       // unchanged by + 4, + 8, + 16*kk
  const int slot = (((c >> 2) ^ gsw) << 2) | (c & 3);
  return (unsigned)kr * (ROWS * 2u) + (unsigned)slot * 16u + (unsigned)(col & 7) * 2u;
}
template <bool TR, int ROWS>
__device__ __forceinline__ bf16x8 load_frag(const unsigned char* tile, unsigned fb, int r0, int kk, int lane) {
  if (!TR) {
    const int sw = ((r0 + (lane & 31)) >> 1) & 7;
    return *(const bf16x8*)(tile + fb + ((((kk * 2) + (lane >> 5)) ^ sw) << 4));
  } else {
    const unsigned char* p = tile + fb + kk * 16 * (ROWS * 2);
    s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p));
    s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + 4 * (ROWS * 2)));
    s16x8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, v);
  }
}
