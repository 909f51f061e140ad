// Flash-style attention on the gfx950 matrix cores (bf16, head_dim 128, fp32 online softmax)
// for the cross-branch attention of Eq. 1: queries from stream 1, keys/values from stream 2.
//
// Layout: q,k,v,o,do,dq,dk,dv are [T, H*128] token-major, head hh in columns hh*128...
// All kernels work on TRANSPOSED score tiles S^T[key, query] = K Q^T, so that in the
// MFMA result layout a lane owns one query (forward, dQ) or one key (dK/dV) column: softmax
// statistics and accumulator rescaling stay inside a lane, and the probability tile is
// already in the operand layout of the second product.  The operand that has to be read
// against its storage order (V^T, K^T, Q^T, dO^T) comes from LDS through the transposing
// read ds_read_b64_tr_b16.
#include "lds_load.h"

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

#define DH 128
#define BKV 64            // rows of the tile that is streamed through LDS
#define LOG2E 1.4426950408889634f
#define LN2 0.6931471805599453f

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// elements 8c..8c+7 of an accumulator tile as a bf16 operand fragment
__device__ __forceinline__ bf16x8 acc_to_frag(const f32x16& a, int c) {
  bf16x8 r;
#pragma unroll
  for (int u = 0; u < 8; u++) r[u] = (__bf16)a[8 * c + u];
  return r;
}

// Rows of one (batch, head) slice [S, DH], row stride ld.  Tiles of them are brought by range-checked buffer loads: the
// descriptor ends at the last byte of row S - 1, so a row past the end is out of range and reads as zeros with no branch and
// no traffic, and the address is one 32-bit offset per lane.
struct RowSlice { __amdgpu_buffer_rsrc_t rs; unsigned ldb; };    // ldb = row stride in bytes
__device__ __forceinline__ RowSlice row_slice(const bf16* base, i64 ld, int S) {
  RowSlice r;
  r.rs = __builtin_amdgcn_make_buffer_rsrc((void*)base, (short)0, (int)(((i64)S - 1) * ld * 2 + DH * 2), 0x00020000);
  r.ldb = (unsigned)(ld * 2);
  return r;
}

// Which tile a workgroup takes (1-D grid of tiles x B x H workgroups; tile 0 has the most work when causal).  Heads are the
// fastest index, so that an XCD (id & 7) keeps to H / 8 heads, then batches, so that long tiles of all batches come first
// (a 3-D grid with the batch slowest: 2 x 2048 tokens, 16 heads, forward and dQ 78 and 111 us, 65 and 98 like this).  Two
// workgroups fit on a CU: where the whole grid is resident at once, workgroups i and i + 256 share one, so the second 256
// run from short to long (forward, dQ, dK/dV: 65, 98, 137 -> 63, 95, 134).
__device__ __forceinline__ void place(int H, int B, int tiles, int per_cu, int* t, int* hh, int* b) {
  const int rows = tiles * B, first = 256 / H;
  int row = (int)blockIdx.x / H;
  *hh = (int)blockIdx.x - row * H;
  if (per_cu == 2 && (int)gridDim.x <= 512 && row >= first) row = rows - 1 - (row - first);
  *t = row / B;
  *b = row - *t * B;
}

// ------------------------------------------------------------------------------------
// Tiles of 64 rows that are read both ways (16-byte fragments of 32 rows, and transposed).  They are loaded straight into
// LDS, without padding, so the layout is a swizzle of the 16-byte chunks of a 256-byte row: chunk c of row r lies in place
// c ^ swz(r).  Sixteen consecutive rows have sixteen different swz, so a fragment read meets every bank once; the four
// rows of a transposing read differ in the upper two bits, i.e. in which quarter of the banks their 64 bytes fall.
// ------------------------------------------------------------------------------------
__device__ __forceinline__ int swz(int r) { return ((r & 3) << 2) | ((r >> 2) & 3); }
// 16 rows (4 wave-loads) of the slice, from row0 on, to LDS at dst.  What does not change from tile to tile is worked out once and
// takes two registers: swz(4 i + (lane >> 4)) = swz(lane >> 4) ^ i.
struct RowOffset { unsigned row, chunk; };
__device__ __forceinline__ RowOffset row_offset(const RowSlice& sl, int row0, int lane) {
  return {(unsigned)(row0 + (lane >> 4)) * sl.ldb, (unsigned)((lane & 15) ^ swz(lane >> 4)) * 16u};
}
__device__ __forceinline__ void load_rows16_lds(const RowSlice& sl, RowOffset at, int row0, unsigned dst) {
  asm volatile("" : "+v"(at.row), "+v"(at.chunk));  // (the sums below are not worth a register each from tile to tile)
#pragma unroll
  for (int i = 0; i < 4; i++)
    load_lds_b128(sl.rs, __builtin_amdgcn_readfirstlane(dst + i * 1024u),
                  at.row + (at.chunk ^ (i * 16u)) + __builtin_amdgcn_readfirstlane((unsigned)(row0 + i * 4) * sl.ldb));
}
// 64 floats (the lane number is asked for here: spilled, it would come back through a wait for all loads on their way)
__device__ __forceinline__ void load_stats64_lds(__amdgpu_buffer_rsrc_t rs, int row0, unsigned dst) {
  unsigned none = 0;
  asm volatile("" : "+v"(none));
  const int lane = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, none));
  load_lds_b32(rs, __builtin_amdgcn_readfirstlane(dst), (unsigned)(row0 + lane) * 4u);
}
// per-lane byte offsets: 16-byte fragments of rows lane & 31 (k-step kk: ^ kk * 32), transposed ones (column block: ^ dtile * 64)
__device__ __forceinline__ unsigned swz_row_base(int lane) { return (unsigned)(lane & 31) * 256u + (unsigned)((lane >> 5) ^ swz(lane & 15)) * 16u; }
__device__ __forceinline__ unsigned swz_col_base(int lane) {
  const int blk = lane >> 4, i16 = lane & 15, row = 4 * (blk >> 1) + (i16 >> 2), c = 2 * (blk & 1) + ((i16 & 3) >> 1);
  return (unsigned)row * 256u + (unsigned)(c ^ swz(row)) * 16u + (unsigned)(i16 & 1) * 8u;
}
// Transposed fragment for a product whose contraction runs over the tile's rows: operand row (MFMA row index) = tile column
// dtile * 32 + (lane & 31); the 8 contraction slots u = 4 * jp + i of half g = lane >> 5 are tile rows rb + 8 * jp + 4 * g + i.
// This matches a probability or score tile taken straight from the accumulator layout of a 32x32 MFMA (elements 8c..8c+7).
__device__ __forceinline__ bf16x8 swz_cols(const unsigned char* tile, unsigned base, int rb, int dtile) {
  const unsigned at = base ^ (unsigned)(dtile * 64);
  s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(tile + rb * 256 + at));
  s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(tile + rb * 256 + 2048 + (at ^ 32u)));     // rows + 8
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// one row of 128 as operand fragments of a product over the head width; rows past the end are zeros
__device__ __forceinline__ void load_frags(const bf16* base, i64 ld, int row, int S, int g, bf16x8 (&f)[8]) {
#pragma unroll
  for (int kk = 0; kk < 8; kk++) {
    uint4 t = make_uint4(0, 0, 0, 0);
    if (row < S) t = *(const uint4*)(base + (i64)row * ld + kk * 16 + g * 8);
    f[kk] = __builtin_bit_cast(bf16x8, t);
  }
}
// the compiler's own wait for fragments just loaded belongs here: inside the loop it would wait for every tile on its way too
__device__ __forceinline__ void arrived(bf16x8 (&f)[8]) {
#pragma unroll
  for (int kk = 0; kk < 8; kk++) asm volatile("" : "+v"(f[kk]));
}

// ------------------------------------------------------------------------------------
// Forward.  Workgroup = 128 queries of one (batch, head), wave = 32 queries; keys/values streamed in tiles of 64, straight into
// LDS, K two tiles ahead and V one.  An iteration is two phases with a barrier behind each.  In the first a wave multiplies:
// scores of the next tile from key fragments that are in registers already, then P V of this one, the value fragments read 16
// rows ahead; half of the tile's exponentials go between the former.  In the second it takes the maximum and the other half of
// the exponentials, and reads the next key fragments meanwhile, so that LDS is busy in both phases.
// GROUPS = 1: 4 waves, two workgroups on a CU.  GROUPS = 2: two groups of 4 waves with the same queries, group 0 on the even
// tiles and group 1 on the odd ones, half an iteration apart (one wave of each on a SIMD: one multiplies while the other
// doesn't); their partial results meet in LDS at the end.  two_groups() has the rule.
// Where the grid is large (8192 tokens, 16 heads): 0.97 PFLOP/s on random values, the matrix pipe busy half of the time at 80 % of its
// nominal rate.  Power has a part in the rate (a third more on zeros), the idle half is the maximum, half of the exponentials and
// the barriers, which the other workgroup's products only partly cover.
// Against tiles staged through registers and fragments read just before use, us: 1 x 8192 332 -> 284, 1 x 4096 109 -> 84, 2 x 2048
// 59 -> 51, 4 x 512 20.1 -> 17.8, 64 x 128 32.1 -> 31.5.
// ------------------------------------------------------------------------------------
#define KV_TILE 16384u                            // 64 rows x 256 bytes, swizzled
#define FWD_SMEM(GROUPS) ((GROUPS) * 4 * KV_TILE) // two stages of K and V per group; the partial results at the end
__device__ __forceinline__ void phase_end() {     // reads of this phase have returned, then everybody's
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" ::: "memory");
}
__device__ __forceinline__ float both_halves_max(float x) {       // of lane l and lane l ^ 32
  const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, x), __builtin_bit_cast(unsigned, x), false, false);
  return fmaxf(__builtin_bit_cast(float, (unsigned)r[0]), __builtin_bit_cast(float, (unsigned)r[1]));
}
__device__ __forceinline__ float both_halves_sum(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, x), __builtin_bit_cast(unsigned, x), false, false);
  return __builtin_bit_cast(float, (unsigned)r[0]) + __builtin_bit_cast(float, (unsigned)r[1]);
}
// one row of 128, times f
__device__ __forceinline__ void store_cols(bf16* row, const f32x16 (&acc)[4], float f, int g) {
#pragma unroll
  for (int d = 0; d < 4; d++)
#pragma unroll
    for (int e = 0; e < 4; e++) {
      bf16x4 r;
#pragma unroll
      for (int i = 0; i < 4; i++) r[i] = (__bf16)(acc[d][e * 4 + i] * f);
      *(bf16x4*)(row + d * 32 + e * 8 + g * 4) = r;
    }
}
// acc^T[column, lane] += tile^T p for a tile of 64 rows, the next 16 rows' fragments read while this one's are multiplied; first:
// the fragments of the first 16 rows
__device__ __forceinline__ void read_cols(bf16x8 (&f)[4], const unsigned char* tile, unsigned cbase, int c) {
#pragma unroll
  for (int dtile = 0; dtile < 4; dtile++) f[dtile] = swz_cols(tile, cbase, c * 16, dtile);
}
__device__ __forceinline__ void cols_times64(f32x16 (&acc)[4], const unsigned char* tile, unsigned cbase, const bf16x8 (&p)[4], bf16x8 (&first)[4]) {
  bf16x8 f[2][4];
#pragma unroll
  for (int dtile = 0; dtile < 4; dtile++) f[0][dtile] = first[dtile];
#pragma unroll
  for (int c = 0; c < 4; c++) {
    if (c < 3) read_cols(f[(c + 1) & 1], tile, cbase, c + 1);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int dtile = 0; dtile < 4; dtile++) acc[dtile] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[c & 1][dtile], p[c], acc[dtile], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  }
}
template <int GROUPS>
__global__ void __launch_bounds__(256 * GROUPS, 2) flash_fwd_k(const bf16* __restrict__ q, const bf16* __restrict__ k,
                                                   const bf16* __restrict__ v, bf16* __restrict__ o,
                                                   float* __restrict__ lse, int B, int S, int H, int causal, float scale,
                                                   const unsigned char* __restrict__ row_skip) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem_raw[];
  int qt, hh, b;
  place(H, B, (S + 127) / 128, 3 - GROUPS, &qt, &hh, &b);
  qt = (S + 127) / 128 - 1 - qt;            // late query tiles are the long ones
  if (row_skip) {                           // every query of the tile is a finished row of the inverse's iteration
    int live = 0;                           // every wave checks all 128 rows of the tile: same answer, no LDS
    for (int r = qt * 128 + (int)(threadIdx.x & 63); r < min(S, qt * 128 + 128); r += 64) live |= row_skip[(i64)b * S + r] == 0;
    if (!__any(live)) return;
  }
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), g = lane >> 5;
  const int grp = GROUPS == 2 ? wave >> 2 : 0, wv = wave & 3;
  const i64 ld = (i64)H * DH, boff = (i64)b * S * ld + hh * DH;
  const int q0 = qt * 128, qw = q0 + wv * 32;
  const int myq = qw + (lane & 31);
  const float sl2 = scale * LOG2E;
  const int nt = ((causal ? min(S, q0 + 128) : S) + BKV - 1) / BKV, ni = (nt + GROUPS - 1) / GROUPS;
  const int none = S;                               // (a tile that is not there: rows past the end, zeros without traffic)

  bf16x8 qf[8];
  load_frags(q + boff, ld, myq, S, g, qf);
  const RowSlice slK = row_slice(k + boff, ld, S), slV = row_slice(v + boff, ld, S);
  const unsigned char* tiles = smem_raw + (unsigned)grp * 4 * KV_TILE;      // K, V, K, V
  const unsigned lds0 = lds_address(smem_raw) + (unsigned)grp * 4 * KV_TILE + (unsigned)wv * 4096u;
  const RowOffset off = row_offset(slK, wv * 16, lane);
  auto issue = [&](const RowSlice& sl, int i, unsigned which) {           // 16 of tile i's rows
    const int t = GROUPS * i + grp;
    load_rows16_lds(sl, off, t < nt ? t * BKV : none, lds0 + ((unsigned)(i & 1) * 2 + which) * KV_TILE);
  };
  auto live = [&](int i) { const int t = GROUPS * i + grp; return t < nt && (!causal || t * BKV <= qw + 31); };   // some key to see
  const unsigned rbase = swz_row_base(lane), cbase = swz_col_base(lane);
  f32x16 oacc[4] = {}, s[2];
  bf16x8 kf[16], pf[4];
  float m = -INFINITY, l = 0.f;
  auto read_k = [&](int i, int from) {              // half of K of tile i
    const unsigned char* cK = tiles + (unsigned)(i & 1) * 2 * KV_TILE;
#pragma unroll
    for (int kk = from; kk < from + 4; kk++)
#pragma unroll
      for (int j = 0; j < 2; j++) kf[kk * 2 + j] = *(const bf16x8*)(cK + j * 8192 + (rbase ^ (unsigned)(kk * 32)));
  };
  auto times_q = [&]() {
    s[0] = f32x16{};
    s[1] = f32x16{};
#pragma unroll
    for (int kk = 0; kk < 8; kk++)
#pragma unroll
      for (int j = 0; j < 2; j++) s[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[kk * 2 + j], qf[kk], s[j], 0, 0, 0);
  };
  // In the order of the loop below (keys of a tile before the values of the one before it), so that each wait counts what is younger
  // than the tile it is for.  (The compiler's wait for Q, which doesn't count these loads, lets them all arrive today; nothing relies on it.)
  issue(slK, 0, 0); issue(slK, 1, 0); issue(slV, 0, 1);
  arrived(qf);
  wait_vmcnt<8>();                                  // the first keys
  phase_end();
  if (GROUPS == 2 && grp == 1) phase_end();                        // half an iteration behind
  read_k(0, 0);
  read_k(0, 4);
  times_q();
  wait_vmcnt<4>();                                  // K of tile 1 is there, V of tile 0 may be on its way
  phase_end();
  // keys past the sequence end or after the query
  auto mask = [&](int i) {
    const int seen = (causal ? min(myq, S - 1) : S - 1) - (GROUPS * i + grp) * BKV - g * 4;
#pragma unroll
    for (int j = 0; j < 2; j++)
#pragma unroll
      for (int e = 0; e < 16; e++)
        if (j * 32 + (e >> 2) * 8 + (e & 3) > seen) s[j][e] = -INFINITY;
  };
  // half of a tile's probabilities, and their part of the sum (of this half's keys; the halves meet at the end)
  float ms = 0.f;
  auto exponentials = [&](f32x16 x, int h) {
    float rs[2] = {};
#pragma unroll
    for (int e = 0; e < 16; e++) {
      x[e] = fast_exp2(fmaf(x[e], sl2, -ms));
      rs[e & 1] += x[e];
    }
    l += rs[0] + rs[1];
    pf[h * 2] = acc_to_frag(x, 0);
    pf[h * 2 + 1] = acc_to_frag(x, 1);
  };
  // the keys read in the phase before and the values just read make room
  auto softmax = [&](int i) {
    issue(slK, i + 2, 0);
    issue(slV, i + 1, 1);
    read_k(i + 1, 0);
    float mx[4] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
#pragma unroll
    for (int e = 0; e < 32; e += 2) mx[(e >> 1) & 3] = fmaxf(fmaxf(mx[(e >> 1) & 3], s[e >> 4][e & 15]), s[e >> 4][(e & 15) + 1]);
    const float mn = fmaxf(m, both_halves_max(fmaxf(fmaxf(mx[0], mx[1]), fmaxf(mx[2], mx[3]))) * sl2);
    // the accumulator is rescaled only when some query of the wave has raised its maximum.  (Letting it lag by up to 2^8 saves a
    // part of that, but the largest probabilities are then no longer exactly 1: O's error against 64 bits 1.82e-3 -> 2.12e-3.)
    if (__any(mn > m)) {
      const float alpha = fast_exp2(m - (mn == -INFINITY ? 0.f : mn));
      l *= alpha;
#pragma unroll
      for (int d = 0; d < 4; d++) oacc[d] *= alpha;
      m = mn;
    }
    read_k(i + 1, 4);
    ms = m == -INFINITY ? 0.f : m;
    exponentials(s[0], 0);
    wait_vmcnt<8>();                                // V of i is there
    phase_end();
  };
  for (int i = 0; i + 1 < ni; i++) {
    if (GROUPS == 1 && i + 2 == ni) mask(i);
    softmax(i);
    __builtin_amdgcn_s_setprio(1);
    const f32x16 rest = s[1];
    const unsigned char* cV = tiles + ((unsigned)(i & 1) * 2 + 1) * KV_TILE;
    bf16x8 vf[4];
    times_q();
    exponentials(rest, 1);
    read_cols(vf, cV, cbase, 0);
    __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
#pragma unroll
    for (int j = 0; j < 14; j++) {
      __builtin_amdgcn_sched_group_barrier(0x002, 5, 0);
      if (j >= 6) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    cols_times64(oacc, cV, cbase, pf, vf);          // O^T[dh, q] += V^T[dh, kv] P^T[kv, q]
    __builtin_amdgcn_s_setprio(0);
    wait_vmcnt<4>();                                // K of i + 2 is there
    phase_end();
  }
  mask(ni - 1);                                     // only the last 128 keys can hold some that are not to be seen
  softmax(ni - 1);
  exponentials(s[1], 1);
  if (live(ni - 1)) {
    const unsigned char* cV = tiles + ((unsigned)((ni - 1) & 1) * 2 + 1) * KV_TILE;
    bf16x8 vf[4];
    read_cols(vf, cV, cbase, 0);
    cols_times64(oacc, cV, cbase, pf, vf);
  }
  if (GROUPS == 2 && grp == 0) phase_end();
  wait_vmcnt<0>();                                  // the zero-filled loads past the last tile
  phase_end();
  l = both_halves_sum(l);
  if constexpr (GROUPS == 1) {
    if (myq < S) {
      const float inv = 1.0f / l;
      store_cols(o + boff + (i64)myq * ld, oacc, inv, g);
      if (g == 0) lse[((i64)b * H + hh) * S + myq] = (m + __log2f(l)) * LN2;
    }
    return;
  }
  // each group takes half of the columns of both
  float4* part = (float4*)smem_raw;                 // [wave][8][lane], then statistics
  float2* stats = (float2*)(smem_raw + 8 * 8192);
  // element e of accumulator d of this group's half, of the other one's
  auto half = [&](int theirs, int d, int e) { return grp == theirs ? oacc[d][e] : oacc[2 + d][e]; };
#pragma unroll
  for (int d = 0; d < 2; d++)
#pragma unroll
    for (int e = 0; e < 4; e++) part[(wave * 8 + d * 4 + e) * 64 + lane] = make_float4(half(1, d, e * 4), half(1, d, e * 4 + 1), half(1, d, e * 4 + 2), half(1, d, e * 4 + 3));
  if (g == 0) stats[wave * 32 + lane] = make_float2(m, l);
  __syncthreads();
  const float2 other = stats[(wave ^ 4) * 32 + (lane & 31)];
  const float M = fmaxf(m, other.x), Ms = M == -INFINITY ? 0.f : M;
  float w = fast_exp2(m - Ms), w2 = fast_exp2(other.x - Ms);
  const float tot = grp == 0 ? w * l + w2 * other.y : w2 * other.y + w * l;
  const float inv = 1.0f / tot;
  w *= inv;
  w2 *= inv;
  if (myq < S) {
    bf16* op = o + boff + (i64)myq * ld + grp * 64;
#pragma unroll
    for (int d = 0; d < 2; d++)
#pragma unroll
      for (int e = 0; e < 4; e++) {
        const float4 p = part[((wave ^ 4) * 8 + d * 4 + e) * 64 + lane];
        bf16x4 r;
        r[0] = (__bf16)(half(0, d, e * 4) * w + p.x * w2);
        r[1] = (__bf16)(half(0, d, e * 4 + 1) * w + p.y * w2);
        r[2] = (__bf16)(half(0, d, e * 4 + 2) * w + p.z * w2);
        r[3] = (__bf16)(half(0, d, e * 4 + 3) * w + p.w * w2);
        *(bf16x4*)(op + d * 32 + e * 8 + g * 4) = r;
      }
    if (wave < 4 && g == 0) lse[((i64)b * H + hh) * S + myq] = (M + __log2f(tot)) * LN2;
  }
}

// ------------------------------------------------------------------------------------
// Backward, part 1: dQ, and D = <o, dO> of the rows.  The forward kernel's scheme with 4 waves.  Per tile:
//   S^T = K Q^T,  P^T = exp(S^T*scale - lse),  dP^T = V dO^T,  dS^T = P^T (dP^T - D),
//   dQ^T += K^T dS^T,  times scale at the end.
// Three products against one exponential: the matrix pipe is busy 63 % of the time at 8192 tokens; fragments are read one step ahead of theirs.  The keys of
// a tile are read once more in the phase after, so they have three stages.  Against tiles staged through registers and a
// kernel of its own for D, us, 16 heads: 1 x 8192 475 -> 355, 2 x 2048 108 -> 72, 4 x 512 32 -> 21.
// ------------------------------------------------------------------------------------
#define DQ_SMEM (5 * KV_TILE)                     // three stages of K, two of V
__global__ void __launch_bounds__(256, 2) flash_bwd_dq_k(const bf16* __restrict__ q, const bf16* __restrict__ k,
                                                      const bf16* __restrict__ v, const bf16* __restrict__ o, const bf16* __restrict__ d_o,
                                                      const float* __restrict__ lse, float* __restrict__ dvec,
                                                      bf16* __restrict__ dq, int B, int S, int H, int causal, float scale) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem_raw[];
  int qt, hh, b;
  place(H, B, (S + 127) / 128, 2, &qt, &hh, &b);
  qt = (S + 127) / 128 - 1 - qt;
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), g = lane >> 5;
  const i64 ld = (i64)H * DH, boff = (i64)b * S * ld + hh * DH;
  const int q0 = qt * 128, qw = q0 + wv * 32;
  const int myq = qw + (lane & 31);
  const float sl2 = scale * LOG2E;
  const int nt = ((causal ? min(S, q0 + 128) : S) + BKV - 1) / BKV;
  const int none = S;

  bf16x8 qf[8], dof[8];
  load_frags(q + boff, ld, myq, S, g, qf);
  load_frags(d_o + boff, ld, myq, S, g, dof);
  float mylse = (myq < S) ? lse[((i64)b * H + hh) * S + myq] * LOG2E : 0.f;
  // D = <o, dO> of the row, for the kernel behind this one too
  float myD = 0.f;
  {
    bf16x8 of[8];
    load_frags(o + boff, ld, myq, S, g, of);
#pragma unroll
    for (int kk = 0; kk < 8; kk++)
#pragma unroll
      for (int u = 0; u < 8; u++) myD = fmaf((float)of[kk][u], (float)dof[kk][u], myD);
    myD = both_halves_sum(myD);
    if (g == 0 && myq < S) dvec[((i64)b * H + hh) * S + myq] = myD;
  }
  const RowSlice slK = row_slice(k + boff, ld, S), slV = row_slice(v + boff, ld, S);
  const unsigned lds0 = lds_address(smem_raw) + (unsigned)wv * 4096u;
  const RowOffset off = row_offset(slK, wv * 16, lane);
  auto issue = [&](const RowSlice& sl, int i, unsigned stage) {           // 16 of tile i's rows; stages K, K, K, V, V
    load_rows16_lds(sl, off, i < nt ? i * BKV : none, lds0 + stage * KV_TILE);
  };
  const unsigned rbase = swz_row_base(lane), cbase = swz_col_base(lane);
  f32x16 acc[4] = {}, s[2], dp[2];
  bf16x8 dsf[4], first[4];
  bf16x8 fr[2][4];
  auto read_kv = [&](bf16x8 (&f)[4], int i, unsigned stage, int kk) {
    const unsigned char* cK = smem_raw + stage * KV_TILE;
    const unsigned char* cV = smem_raw + (3u + (unsigned)(i & 1)) * KV_TILE;
    const unsigned at = rbase ^ (unsigned)(kk * 32);
    f[0] = *(const bf16x8*)(cK + at);
    f[1] = *(const bf16x8*)(cV + at);
    f[2] = *(const bf16x8*)(cK + 8192 + at);
    f[3] = *(const bf16x8*)(cV + 8192 + at);
  };
  auto times_q = [&](int i, unsigned stage) {       // (after read_kv(fr[0], i, stage, 0))
#pragma unroll
    for (int j = 0; j < 2; j++) { s[j] = f32x16{}; dp[j] = f32x16{}; }
#pragma unroll
    for (int kk = 0; kk < 8; kk++) {
      if (kk < 7) read_kv(fr[(kk + 1) & 1], i, stage, kk + 1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < 2; j++) {
        s[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[kk & 1][j * 2], qf[kk], s[j], 0, 0, 0);
        dp[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[kk & 1][j * 2 + 1], dof[kk], dp[j], 0, 0, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  issue(slK, 0, 0); issue(slV, 0, 3); issue(slK, 1, 1); issue(slV, 1, 4);
  arrived(qf);
  arrived(dof);
  asm volatile("" : "+v"(mylse), "+v"(myD));
  wait_vmcnt<8>();
  phase_end();
  unsigned before = 2, now = 0;                     // places of K of the last iteration and this one
  read_kv(fr[0], 0, 0, 0);
  times_q(0, 0);
  phase_end();
  // keys past the sequence end or after the query
  auto mask = [&](int i) {
    const int seen = (causal ? min(myq, S - 1) : S - 1) - i * BKV - g * 4;
#pragma unroll
    for (int j = 0; j < 2; j++)
#pragma unroll
      for (int e = 0; e < 16; e++)
        if (j * 32 + (e >> 2) * 8 + (e & 3) > seen) s[j][e] = -INFINITY;
  };
  // the values just read and the keys read for the second time make room
  auto probabilities = [&](int i) {
    issue(slK, i + 2, before);
    issue(slV, i + 2, 3u + (unsigned)(i & 1));
#pragma unroll
    for (int j = 0; j < 2; j++)
#pragma unroll
      for (int e = 0; e < 16; e++) s[j][e] = fast_exp2(fmaf(s[j][e], sl2, -mylse)) * (dp[j][e] - myD);
#pragma unroll
    for (int c = 0; c < 4; c++) dsf[c] = acc_to_frag(s[c >> 1], c & 1);
    read_cols(first, smem_raw + now * KV_TILE, cbase, 0);
    const unsigned next = 3u - before - now;
    before = now;
    now = next;
    wait_vmcnt<8>();                                // K and V of i + 1 are there
    phase_end();
  };
  for (int i = 0; i + 1 < nt; i++) {
    if (i + 2 == nt) mask(i);
    probabilities(i);
    __builtin_amdgcn_s_setprio(1);
    read_kv(fr[0], i + 1, now, 0);
    cols_times64(acc, smem_raw + before * KV_TILE, cbase, dsf, first);
    times_q(i + 1, now);
    __builtin_amdgcn_s_setprio(0);
    phase_end();
  }
  mask(nt - 1);                                     // only the last 128 keys can hold some that are not to be seen
  probabilities(nt - 1);
  if (!causal || (nt - 1) * BKV <= qw + 31) cols_times64(acc, smem_raw + before * KV_TILE, cbase, dsf, first);
  wait_vmcnt<0>();                                  // the zero-filled loads past the last tile
  if (myq < S) store_cols(dq + boff + (i64)myq * ld, acc, scale, g);
}

// ------------------------------------------------------------------------------------
// Backward, part 2: dK and dV.  Workgroup = 128 keys, wave = 32 keys (one per lane column);
// queries (with dO, lse, D) streamed in tiles of 64, starting at the diagonal when causal.
//   S = Q K^T,  P = exp(S*scale - lse),  dP = dO V^T,  dS = P (dP - D),
//   dV^T += dO^T P,   dK^T += Q^T dS,  times scale at the end.
// Four products against one exponential: the matrix pipe is busy 52 % of the time at 8192 tokens.  Accumulators and the wave's K and V take 192 registers, so with
// the queries of a tile worked on QB = 1 block of 32 at a time two workgroups fit on a CU, and one wave's exponentials run beside
// the other's products.  A grid that has one workgroup per CU at most gains nothing from that; there QB = 2, 64 queries at a time,
// leaves more to overlap inside the wave.  All of the backward pass, us, 16 heads, QB = 1 -> 2: 4 x 512 50.1 -> 49.1, 1 x 2048 128.9
// -> 126.2, 2 x 2048 158 -> 172, 1 x 8192 918 -> 962.  Both add the queries in the same order, so the results have the same bits.
// Fragments are read one step ahead of their products, addresses are worked out where they are used, and nothing is spilled inside
// the loop (a register that is comes back through a wait for every tile on its way): the backward pass with dQ's part 1 x 8192
// 1074 -> 897 us, 2 x 2048 227 -> 156, 4 x 512 70 -> 48.
// ------------------------------------------------------------------------------------
#define DKV_STAGE (2 * 64 * 256 + 2 * 256)      // Q, dO, lse, D
template <int QB>
__global__ void __launch_bounds__(256, QB == 1 ? 2 : 1) flash_bwd_dkv_k(const bf16* __restrict__ q, const bf16* __restrict__ k,
                                                       const bf16* __restrict__ v, const bf16* __restrict__ d_o,
                                                       const float* __restrict__ lse, const float* __restrict__ dvec,
                                                       bf16* __restrict__ dk, bf16* __restrict__ dv, int B, int S, int H,
                                                       int causal, float scale) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem_raw[];      // 2 stages
  int kt, hh, b;
  place(H, B, (S + 127) / 128, 2, &kt, &hh, &b);       // early key tiles see the most queries
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), g = lane >> 5;
  const i64 ld = (i64)H * DH;
  const i64 boff = (i64)b * S * ld + hh * DH;
  const i64 soff = ((i64)b * H + hh) * S;
  const int k0 = kt * 128, kw = k0 + wv * 32;
  const int mykv = kw + (lane & 31);
  const float sl2 = scale * LOG2E;

  bf16x8 kf[8], vf[8];
#pragma unroll
  for (int kk = 0; kk < 8; kk++) {
    uint4 t = make_uint4(0, 0, 0, 0), u = make_uint4(0, 0, 0, 0);
    if (mykv < S) {
      t = *(const uint4*)(k + boff + (i64)mykv * ld + kk * 16 + g * 8);
      u = *(const uint4*)(v + boff + (i64)mykv * ld + kk * 16 + g * 8);
    }
    kf[kk] = __builtin_bit_cast(bf16x8, t);
    vf[kk] = __builtin_bit_cast(bf16x8, u);
  }
  const int t_lo = causal ? k0 / BKV : 0;
  const int nt = (S + BKV - 1) / BKV;

  f32x16 dkacc[4], dvacc[4];
#pragma unroll
  for (int i = 0; i < 4; i++)
#pragma unroll
    for (int e = 0; e < 16; e++) { dkacc[i][e] = 0.f; dvacc[i][e] = 0.f; }

  const RowSlice slQ = row_slice(q + boff, ld, S), slO = row_slice(d_o + boff, ld, S);
  const __amdgpu_buffer_rsrc_t rsL = __builtin_amdgcn_make_buffer_rsrc((void*)(lse + soff), (short)0, S * 4, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsD = __builtin_amdgcn_make_buffer_rsrc((void*)(dvec + soff), (short)0, S * 4, 0x00020000);
  const unsigned lds0 = lds_address(smem_raw);
  // rows past the end are zeros throughout: whatever their probabilities, they add Q = dO = 0
  const RowOffset off = row_offset(slQ, wv * 16, lane);
  auto issue = [&](int t, int stage) {
    const unsigned dst = lds0 + (unsigned)stage * DKV_STAGE;
    load_rows16_lds(slQ, off, t * BKV, dst + wv * 4096u);
    load_rows16_lds(slO, off, t * BKV, dst + 16384u + wv * 4096u);
    if (wv == 0) load_stats64_lds(rsL, t * BKV, dst + 32768u);
    if (wv == 1) load_stats64_lds(rsD, t * BKV, dst + 32768u + 256u);
  };
  const unsigned rbase = swz_row_base(lane), cbase = swz_col_base(lane);
  issue(t_lo, 0);
  arrived(kf);
  arrived(vf);
  wait_vmcnt<0>();
  __syncthreads();
  for (int t = t_lo; t < nt; t++) {
    const int cur = (t - t_lo) & 1, q0 = t * BKV;
    if (t + 1 < nt) issue(t + 1, cur ^ 1);
    const unsigned char* cQ = smem_raw + cur * DKV_STAGE;
    const unsigned char* cO = cQ + 16384;
    const float* cL = (const float*)(cQ + 32768);
    const float* cD = cL + 64;
#pragma unroll 1
    for (int j0 = 0; j0 < 2; j0 += QB) {
      if (causal && q0 + (j0 + QB) * 32 - 1 < kw) continue;    // no query of the block can see a key of this wave
      // (addresses are worked out where they are used: kept for all k-steps they cost the registers that are short here)
      unsigned rb = rbase + (unsigned)(j0 * 8192), cb = cbase;
      asm volatile("" : "+v"(rb), "+v"(cb));
      f32x16 s[QB], dp[QB];
      bf16x8 f[2][QB * 2];
      auto read_rows = [&](bf16x8 (&x)[QB * 2], int kk) {
#pragma unroll
        for (int j = 0; j < QB; j++) {
          const unsigned at = (unsigned)(j * 8192) + (rb ^ (unsigned)(kk * 32));
          x[j * 2] = *(const bf16x8*)(cQ + at);
          x[j * 2 + 1] = *(const bf16x8*)(cO + at);
        }
      };
#pragma unroll
      for (int j = 0; j < QB; j++) { s[j] = f32x16{}; dp[j] = f32x16{}; }
      read_rows(f[0], 0);
#pragma unroll
      for (int kk = 0; kk < 8; kk++) {
        if (kk < 7) read_rows(f[(kk + 1) & 1], kk + 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < QB; j++) {
          s[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[kk & 1][j * 2], kf[kk], s[j], 0, 0, 0);
          dp[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[kk & 1][j * 2 + 1], vf[kk], dp[j], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      bf16x8 pf[QB * 2], dsf[QB * 2];
#pragma unroll
      for (int j = 0; j < QB; j++) {
#pragma unroll
        for (int eb = 0; eb < 4; eb++) {
          const float4 l4 = *(const float4*)(cL + (j0 + j) * 32 + eb * 8 + g * 4);   // 4 consecutive query rows inside the tile
          const float lv[4] = {l4.x, l4.y, l4.z, l4.w};
#pragma unroll
          for (int i = 0; i < 4; i++) s[j][eb * 4 + i] = fast_exp2(s[j][eb * 4 + i] * sl2 - lv[i] * LOG2E);      // P
        }
        const int before = mykv - q0 - (j0 + j) * 32 - g * 4;         // queries that precede this lane's key
        if (causal && q0 + (j0 + j) * 32 < kw + 31) {
#pragma unroll
          for (int e = 0; e < 16; e++)
            if ((e >> 2) * 8 + (e & 3) < before) s[j][e] = 0.f;
        }
#pragma unroll
        for (int eb = 0; eb < 4; eb++) {
          const float4 d4 = *(const float4*)(cD + (j0 + j) * 32 + eb * 8 + g * 4);
          const float dv4[4] = {d4.x, d4.y, d4.z, d4.w};
#pragma unroll
          for (int i = 0; i < 4; i++) dp[j][eb * 4 + i] = s[j][eb * 4 + i] * (dp[j][eb * 4 + i] - dv4[i]);     // dS, without scale
        }
#pragma unroll
        for (int c = 0; c < 2; c++) { pf[j * 2 + c] = acc_to_frag(s[j], c); dsf[j * 2 + c] = acc_to_frag(dp[j], c); }
      }
      // dO^T P and Q^T dS by turns, 16 queries each, the next fragments read while these are multiplied
      bf16x8 x[2][4];
      read_cols(x[0], cO + j0 * 8192, cb, 0);
#pragma unroll
      for (int c = 0; c < QB * 4; c++) {
        if (c + 1 < QB * 4) read_cols(x[(c + 1) & 1], (c & 1 ? cO : cQ) + j0 * 8192, cb, (c + 1) >> 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int d = 0; d < 4; d++) {
          if (c & 1) dkacc[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[c & 1][d], dsf[c >> 1], dkacc[d], 0, 0, 0);
          else dvacc[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[c & 1][d], pf[c >> 1], dvacc[d], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    // this wave's part of the next tile has landed, and its reads of this one have returned
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __syncthreads();
  }
  if (mykv < S) {
    store_cols(dk + boff + (i64)mykv * ld, dkacc, scale, g);
    store_cols(dv + boff + (i64)mykv * ld, dvacc, 1.0f, g);
  }
}

// ------------------------------------------------------------------------------------
// Short sequences.  With 128 queries (keys) per workgroup a short sequence leaves most CUs idle or gives each one chain over
// all its key tiles: one wave per SIMD whose products, exponentials and loads follow each other.  Here a workgroup is 32
// queries (keys) and its 4 waves share the keys (queries) out, tile w, w + 4, .. of 32, each in LDS of its own that no other
// wave touches, so nothing waits at a barrier until the waves' partial results meet in LDS in wave order; fragments are read ahead
// of their products as above (2 x 1024 tokens, 16 heads, backward 80 -> 72 us, 1 x 1024 forward 18.2 -> 16.8).  A wave's two
// tiles (K and V, or Q and dO) are 16 KiB, two workgroups share a CU.  Every wave loads its tiles itself, four times the
// traffic of the kernels above, which is what bounds this form once it fills the chip.  dQ and dK/dV are one launch.
// ------------------------------------------------------------------------------------
#define SHORT_TILE 8192u                          // 32 rows x 256 bytes, swizzled
#define SHORT_SMEM (4 * 2 * SHORT_TILE + 2048)    // the waves' tiles (then their partial results), then statistics
__device__ __forceinline__ void load_rows32_lds(const RowSlice& sl, RowOffset at, int row0, unsigned dst) {
  load_rows16_lds(sl, at, row0, dst);
  load_rows16_lds(sl, at, row0 + 16, dst + 4096u);
}
// tile rows x fragments: element e of lane l is tile row (e >> 2) * 8 + (l >> 5) * 4 + (e & 3), column l & 31
__device__ __forceinline__ f32x16 rows_times(const unsigned char* tile, unsigned rbase, const bf16x8 (&f)[8]) {
  f32x16 a = {};
  bf16x8 x[8];
#pragma unroll
  for (int kk = 0; kk < 8; kk++) x[kk] = *(const bf16x8*)(tile + (rbase ^ (unsigned)(kk * 32)));
  __builtin_amdgcn_sched_barrier(0);                // (or each product would wait for a read of its own)
#pragma unroll
  for (int kk = 0; kk < 8; kk++) a = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[kk], f[kk], a, 0, 0, 0);
  return a;
}
// two of them, the next fragments read while these are multiplied
__device__ __forceinline__ void rows_times2(f32x16& a, f32x16& b, const unsigned char* ta, const unsigned char* tb, unsigned rbase,
                                            const bf16x8 (&fa)[8], const bf16x8 (&fb)[8]) {
  asm volatile("" : "+v"(rbase));                   // (eight addresses kept from tile to tile cost the registers that are short)
  bf16x8 x[2][2];
  auto read = [&](bf16x8 (&y)[2], int kk) {
    y[0] = *(const bf16x8*)(ta + (rbase ^ (unsigned)(kk * 32)));
    y[1] = *(const bf16x8*)(tb + (rbase ^ (unsigned)(kk * 32)));
  };
  a = f32x16{};
  b = f32x16{};
  read(x[0], 0);
#pragma unroll
  for (int kk = 0; kk < 8; kk++) {
    if (kk < 7) read(x[(kk + 1) & 1], kk + 1);
    __builtin_amdgcn_sched_barrier(0);
    a = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[kk & 1][0], fa[kk], a, 0, 0, 0);
    b = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[kk & 1][1], fb[kk], b, 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  }
}
// acc^T[column, lane] += tile^T p for a tile of 32 rows
__device__ __forceinline__ void cols_times(f32x16 (&acc)[4], const unsigned char* tile, unsigned cbase, const f32x16& p) {
  bf16x8 x[2][4];
#pragma unroll
  for (int c = 0; c < 2; c++) read_cols(x[c], tile, cbase, c);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int c = 0; c < 2; c++) {
    const bf16x8 f = acc_to_frag(p, c);
#pragma unroll
    for (int dtile = 0; dtile < 4; dtile++) acc[dtile] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[c][dtile], f, acc[dtile], 0, 0, 0);
  }
}
// a += ta^T pa and b += tb^T pb by turns, 16 rows each, the next fragments read while these are multiplied
__device__ __forceinline__ void cols_times2(f32x16 (&a)[4], f32x16 (&b)[4], const unsigned char* ta, const unsigned char* tb, unsigned cbase,
                                            const bf16x8 (&pa)[2], const bf16x8 (&pb)[2]) {
  asm volatile("" : "+v"(cbase));
  bf16x8 x[2][4];
  read_cols(x[0], ta, cbase, 0);
#pragma unroll
  for (int c = 0; c < 4; c++) {
    if (c < 3) read_cols(x[(c + 1) & 1], c & 1 ? ta : tb, cbase, (c + 1) >> 1);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int d = 0; d < 4; d++) {
      if (c & 1) b[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[c & 1][d], pb[c >> 1], b[d], 0, 0, 0);
      else a[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[c & 1][d], pa[c >> 1], a[d], 0, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
}
// a wave's partial result to its 16 KiB: [column 128][row 32]
__device__ __forceinline__ void put_partial(float* mine, const f32x16 (&acc)[4], int lane) {
#pragma unroll
  for (int dtile = 0; dtile < 4; dtile++)
#pragma unroll
    for (int e = 0; e < 16; e++) mine[(dtile * 32 + (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3)) * 32 + (lane & 31)] = acc[dtile][e];
}
// the sum of the four, weighted (w), to row threadIdx.x & 31, 16 columns of it per thread
__device__ __forceinline__ void store_partials(const float* part, const float (&w)[4], bf16* row, bool in) {
  const int r = threadIdx.x & 31, c0 = (int)(threadIdx.x >> 5) * 16;
  bf16x8 o[2];
#pragma unroll
  for (int i = 0; i < 16; i++) {
    float v = 0.f;
#pragma unroll
    for (int j = 0; j < 4; j++) v += w[j] * part[j * 4096 + (c0 + i) * 32 + r];
    o[i >> 3][i & 7] = (__bf16)v;
  }
  if (in) { *(bf16x8*)(row + c0) = o[0]; *(bf16x8*)(row + c0 + 8) = o[1]; }
}

__global__ void __launch_bounds__(256, 2) flash_fwd_short_k(const bf16* __restrict__ q, const bf16* __restrict__ k,
                                                            const bf16* __restrict__ v, bf16* __restrict__ o, float* __restrict__ lse,
                                                            int B, int S, int H, int causal, float scale,
                                                            const unsigned char* __restrict__ row_skip) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem_raw[];
  const int tiles = (S + 31) / 32, row = (int)blockIdx.x / H, hh = (int)blockIdx.x - row * H, b = row % B;
  const int q0 = (tiles - 1 - row / B) * 32;        // late query tiles are the long ones
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), g = lane >> 5, myq = q0 + (lane & 31);
  if (row_skip && !__any(myq < S && row_skip[(i64)b * S + myq] == 0)) return;      // (the same answer in every wave)
  const i64 ld = (i64)H * DH, boff = (i64)b * S * ld + hh * DH;
  const RowSlice slK = row_slice(k + boff, ld, S), slV = row_slice(v + boff, ld, S);
  const RowOffset off = row_offset(slK, 0, lane);
  unsigned char* tK = smem_raw + wv * 2 * SHORT_TILE;
  const unsigned aK = lds_address(smem_raw) + (unsigned)wv * 2 * SHORT_TILE, aV = aK + SHORT_TILE;
  const int nt = ((causal ? min(S, q0 + 32) : S) + 31) / 32;
  const int none = tiles * 32;                      // (a tile that is not there: rows past the end, zeros without traffic)
  load_rows32_lds(slK, off, wv < nt ? wv * 32 : none, aK);
  load_rows32_lds(slV, off, wv < nt ? wv * 32 : none, aV);
  bf16x8 qf[8];
  load_frags(q + boff, ld, myq, S, g, qf);
  arrived(qf);
  const unsigned rbase = swz_row_base(lane), cbase = swz_col_base(lane);
  const float sl2 = scale * LOG2E;
  f32x16 acc[4] = {};
  float m = -INFINITY, l = 0.f;
  for (int t = wv; t < nt; t += 4) {
    const int kv0 = t * 32, next = t + 4 < nt ? kv0 + 128 : none;
    // (the fragments of Q were asked for after the first tile: nothing may be outstanding the first time)
    if (t == wv) wait_vmcnt<0>(); else wait_vmcnt<8>();
    f32x16 s = rows_times(tK, rbase, qf);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    load_rows32_lds(slK, off, next, aK);
    float mx = -INFINITY;
    const bool need_mask = kv0 + 32 > S || (causal && kv0 + 31 > q0);
#pragma unroll
    for (int e = 0; e < 16; e++) {
      const int kv = kv0 + (e >> 2) * 8 + g * 4 + (e & 3);
      float sv = s[e] * sl2;
      if (need_mask && (kv >= S || (causal && kv > myq))) sv = -INFINITY;
      s[e] = sv;
      mx = fmaxf(mx, sv);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 32, WAVE));
    const float mn = fmaxf(m, mx), ms = mn == -INFINITY ? 0.f : mn;
    float rs = 0.f;
#pragma unroll
    for (int e = 0; e < 16; e++) { s[e] = fast_exp2(s[e] - ms); rs += s[e]; }
    rs += __shfl_xor(rs, 32, WAVE);
    if (__any(mn > m)) {
      const float alpha = fast_exp2(m - ms);
      l *= alpha;
#pragma unroll
      for (int i = 0; i < 4; i++) acc[i] *= alpha;
    }
    l += rs;
    m = mn;
    wait_vmcnt<8>();                                // V; the next K may be on its way
    cols_times(acc, tK + SHORT_TILE, cbase, s);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    load_rows32_lds(slV, off, next, aV);
  }
  wait_vmcnt<0>();
  float* stats = (float*)(smem_raw + 8 * SHORT_TILE);
  put_partial((float*)tK, acc, lane);
  if (g == 0) { stats[wv * 64 + lane] = m; stats[wv * 64 + 32 + lane] = l; }
  __syncthreads();
  const int r = threadIdx.x & 31;
  float M = -INFINITY, w[4], tot = 0.f;
#pragma unroll
  for (int j = 0; j < 4; j++) M = fmaxf(M, stats[j * 64 + r]);
  const float Ms = M == -INFINITY ? 0.f : M;
#pragma unroll
  for (int j = 0; j < 4; j++) { w[j] = fast_exp2(stats[j * 64 + r] - Ms); tot += w[j] * stats[j * 64 + 32 + r]; }
  const float inv = 1.0f / tot;
#pragma unroll
  for (int j = 0; j < 4; j++) w[j] *= inv;
  store_partials((const float*)smem_raw, w, o + boff + (i64)(q0 + r) * ld, q0 + r < S);
  if (threadIdx.x < 32 && q0 + r < S) lse[((i64)b * H + hh) * S + q0 + r] = (M + __log2f(tot)) * LN2;
}

// dQ of 32 queries
__device__ __forceinline__ void short_dq(unsigned char* smem_raw, int tile, int b, int hh, const bf16* q, const bf16* k, const bf16* v,
                                         const bf16* d_o, const float* lse, const float* dvec, bf16* dq, int S, int H, int causal, float scale) {
  const int q0 = ((S + 31) / 32 - 1 - tile) * 32;
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), g = lane >> 5, myq = q0 + (lane & 31);
  const i64 ld = (i64)H * DH, boff = (i64)b * S * ld + hh * DH, soff = ((i64)b * H + hh) * S;
  const RowSlice slK = row_slice(k + boff, ld, S), slV = row_slice(v + boff, ld, S);
  const RowOffset off = row_offset(slK, 0, lane);
  unsigned char* tK = smem_raw + wv * 2 * SHORT_TILE;
  const unsigned aK = lds_address(smem_raw) + (unsigned)wv * 2 * SHORT_TILE, aV = aK + SHORT_TILE;
  const int nt = ((causal ? min(S, q0 + 32) : S) + 31) / 32;
  if (wv < nt) {
    load_rows32_lds(slV, off, wv * 32, aV);
    load_rows32_lds(slK, off, wv * 32, aK);
  }
  bf16x8 qf[8], dof[8];
  load_frags(q + boff, ld, myq, S, g, qf);
  load_frags(d_o + boff, ld, myq, S, g, dof);
  float L = myq < S ? lse[soff + myq] * LOG2E : 0.f, D = myq < S ? dvec[soff + myq] : 0.f;
  arrived(qf);
  arrived(dof);
  asm volatile("" : "+v"(L), "+v"(D));
  const unsigned rbase = swz_row_base(lane), cbase = swz_col_base(lane);
  const float sl2 = scale * LOG2E;
  f32x16 acc[4] = {};
  for (int t = wv; t < nt; t += 4) {
    const int kv0 = t * 32;
    wait_vmcnt<0>();
    f32x16 dp, s;
    rows_times2(dp, s, tK + SHORT_TILE, tK, rbase, dof, qf);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    if (t + 4 < nt) load_rows32_lds(slV, off, kv0 + 128, aV);
    const bool need_mask = kv0 + 32 > S || (causal && kv0 + 31 > q0);
#pragma unroll
    for (int e = 0; e < 16; e++) {
      const int kv = kv0 + (e >> 2) * 8 + g * 4 + (e & 3);
      float p = fast_exp2(s[e] * sl2 - L);
      if (need_mask && (kv >= S || (causal && kv > myq))) p = 0.f;
      s[e] = p * (dp[e] - D) * scale;
    }
    cols_times(acc, tK, cbase, s);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    if (t + 4 < nt) load_rows32_lds(slK, off, kv0 + 128, aK);
  }
  put_partial((float*)tK, acc, lane);
  __syncthreads();
  const float w[4] = {1.f, 1.f, 1.f, 1.f};
  const int r = threadIdx.x & 31;
  store_partials((const float*)smem_raw, w, dq + boff + (i64)(q0 + r) * ld, q0 + r < S);
}
// dK, dV of 32 keys
__device__ __forceinline__ void short_dkv(unsigned char* smem_raw, int tile, int b, int hh, const bf16* q, const bf16* k, const bf16* v,
                                          const bf16* d_o, const float* lse, const float* dvec, bf16* dk, bf16* dv, int S, int H,
                                          int causal, float scale) {
  const int k0 = tile * 32, nt = (S + 31) / 32;     // early key tiles see the most queries
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), g = lane >> 5, mykv = k0 + (lane & 31);
  const i64 ld = (i64)H * DH, boff = (i64)b * S * ld + hh * DH, soff = ((i64)b * H + hh) * S;
  const RowSlice slQ = row_slice(q + boff, ld, S), slO = row_slice(d_o + boff, ld, S);
  const RowOffset off = row_offset(slQ, 0, lane);
  const __amdgpu_buffer_rsrc_t rsL = __builtin_amdgcn_make_buffer_rsrc((void*)(lse + soff), (short)0, S * 4, 0x00020000);
  const __amdgpu_buffer_rsrc_t rsD = __builtin_amdgcn_make_buffer_rsrc((void*)(dvec + soff), (short)0, S * 4, 0x00020000);
  unsigned char* tQ = smem_raw + wv * 2 * SHORT_TILE;
  const unsigned aQ = lds_address(smem_raw) + (unsigned)wv * 2 * SHORT_TILE, aO = aQ + SHORT_TILE;
  // statistics of the tile, lse and D (a load brings 64, of which 32 are used)
  float* st = (float*)(smem_raw + 8 * SHORT_TILE) + wv * 128;
  const unsigned aS = lds_address(smem_raw) + 8 * SHORT_TILE + (unsigned)wv * 512u;
  auto stats = [&](int row0) {
    load_stats64_lds(rsL, row0, aS);
    load_stats64_lds(rsD, row0, aS + 256u);
  };
  const int t0 = (causal ? tile : 0) + wv;
  if (t0 < nt) {
    load_rows32_lds(slQ, off, t0 * 32, aQ);
    load_rows32_lds(slO, off, t0 * 32, aO);
    stats(t0 * 32);
  }
  bf16x8 kf[8], vf[8];
  load_frags(k + boff, ld, mykv, S, g, kf);
  load_frags(v + boff, ld, mykv, S, g, vf);
  arrived(kf);
  arrived(vf);
  const unsigned rbase = swz_row_base(lane), cbase = swz_col_base(lane);
  const float sl2 = scale * LOG2E;
  f32x16 dka[4] = {}, dva[4] = {};
  for (int t = t0; t < nt; t += 4) {
    const int q0 = t * 32;
    wait_vmcnt<0>();
    f32x16 s, dp;
    rows_times2(s, dp, tQ, tQ + SHORT_TILE, rbase, kf, vf);
    const bool need_mask = causal && q0 < k0 + 31;
#pragma unroll
    for (int eb = 0; eb < 4; eb++) {
      const int r0 = eb * 8 + g * 4;
      const float4 l4 = *(const float4*)(st + r0), d4 = *(const float4*)(st + 64 + r0);
      const float lv[4] = {l4.x, l4.y, l4.z, l4.w}, dv4[4] = {d4.x, d4.y, d4.z, d4.w};
#pragma unroll
      for (int i = 0; i < 4; i++) {
        const int e = eb * 4 + i;
        float p = fast_exp2(s[e] * sl2 - lv[i] * LOG2E);
        if (need_mask && mykv > q0 + r0 + i) p = 0.f;
        dp[e] = p * (dp[e] - dv4[i]) * scale;
        s[e] = p;
      }
    }
    bf16x8 pf[2], dsf[2];
#pragma unroll
    for (int c = 0; c < 2; c++) { pf[c] = acc_to_frag(s, c); dsf[c] = acc_to_frag(dp, c); }
    cols_times2(dva, dka, tQ + SHORT_TILE, tQ, cbase, pf, dsf);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    if (t + 4 < nt) {
      load_rows32_lds(slQ, off, q0 + 128, aQ);
      load_rows32_lds(slO, off, q0 + 128, aO);
      stats(q0 + 128);
    }
  }
  const float w[4] = {1.f, 1.f, 1.f, 1.f};
  const int r = threadIdx.x & 31;
  const i64 at = boff + (i64)(k0 + r) * ld;
  put_partial((float*)tQ, dka, lane);
  __syncthreads();
  store_partials((const float*)smem_raw, w, dk + at, k0 + r < S);
  __syncthreads();
  put_partial((float*)tQ, dva, lane);
  __syncthreads();
  store_partials((const float*)smem_raw, w, dv + at, k0 + r < S);
}
// D = <o, dO> of each row, 16 bytes per lane and 16 lanes per row
__global__ void __launch_bounds__(256) flash_dvec_k(const bf16* __restrict__ o, const bf16* __restrict__ d_o, float* __restrict__ dvec, int S, int H,
                                                    i64 rows) {
  const i64 r = (i64)blockIdx.x * 16 + (threadIdx.x >> 4);
  if (r >= rows) return;
  const int c = (threadIdx.x & 15) * 8;
  const bf16x8 a = *(const bf16x8*)(o + r * DH + c), d = *(const bf16x8*)(d_o + r * DH + c);
  float acc = 0.f;
#pragma unroll
  for (int u = 0; u < 8; u++) acc = fmaf((float)a[u], (float)d[u], acc);
#pragma unroll
  for (int x = 8; x; x >>= 1) acc += __shfl_xor(acc, x, WAVE);
  if (c == 0) {
    const i64 t = r / H, b = t / S;
    dvec[(b * H + (r - t * H)) * S + (t - b * S)] = acc;
  }
}
// rows of H workgroups, by turns dK/dV and dQ, long tiles first in both
__global__ void __launch_bounds__(256, 2) flash_bwd_short_k(const bf16* __restrict__ q, const bf16* __restrict__ k, const bf16* __restrict__ v,
                                                            const bf16* __restrict__ d_o, const float* __restrict__ lse,
                                                            const float* __restrict__ dvec, bf16* __restrict__ dq, bf16* __restrict__ dk,
                                                            bf16* __restrict__ dv, int B, int S, int H, int causal, float scale) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem_raw[];
  const int row = (int)blockIdx.x / H, hh = (int)blockIdx.x - row * H, tile = (row >> 1) / B, b = (row >> 1) - tile * B;
  if (row & 1) short_dq(smem_raw, tile, b, hh, q, k, v, d_o, lse, dvec, dq, S, H, causal, scale);
  else short_dkv(smem_raw, tile, b, hh, q, k, v, d_o, lse, dvec, dk, dv, S, H, causal, scale);
}

// Which form a problem takes.  Measured, us, forward / all of the backward pass, 128 queries per workgroup -> 32:
//   16 heads: 1 x 256 10.8 / 29 -> 7.9 / 13    1 x 512 15.0 / 42 -> 10.1 / 19    2 x 400 13.0 / 38 -> 11.5 / 27    3 x 333 12.3 / 36 -> 13.0 / 30
//             2 x 512 15.5 / 43 -> 12.0 / 30   1 x 1024 20.4 / 70 -> 16.4 / 41   1 x 1536 28.6 / 97 -> 26.1 / 69   2 x 1024 23.1 / 72 -> 27.0 / 72
//             1 x 2048 36 / 125 -> 39.5 / 105
//   8 heads: 1 x 2048 31.5 / 122 -> 26.4 / 56    4 heads: 4 x 1024 19.9 / 68 -> 16.3 / 42    32 heads: 1 x 1024 21.7 / 72 -> 26.2 / 67
// Alone 32 queries pay further up than inside a step, where the attention shares the chip with the experts' weight gradients and
// the CU time counts, of which they take more.  16 heads, us per step, 128 queries always -> 32 at both: 1 x 512 1486.6 -> 1487.4,
// 1 x 1024 1872 -> 1886, 1 x 1600 2280 -> 2324, 1 x 2048 2813 -> 2891; adapters only, with little beside the attention, 3 x 333
// 1578 -> 1573; merged passes, forward only, 1 x 512 472 -> 465, 1 x 1024 535.5 -> 529.8, 1 x 2048 792 -> 807; 4 heads, 2 x 1024
// 566 -> 518.  So the line is at 1024 tokens of 16 heads, from 1024 positions on at 1536, with more than 16 heads counted as 18.
// Backward at 1280 instead: all gradients 1 x 1300 2220 -> 2205, 1 x 1536 2354 -> 2336, but adapters only 1853 -> 1872, 1934 -> 1953, and a
// block of 8 experts of 704, 16 heads, 1 x 1400 1079 -> 1087, its adapters only 950 -> 976.
// From 1024 positions on fewer heads than 16 count as they are: alone, forward / backward, 9 heads, 1 x 1400 26.2 / 89 -> 21.0 / 39, 12,
// 1 x 1700 29.7 / 105 -> 25.5 / 63, 5, 2 x 2048 34.7 / 122 -> 28.1 / 68; a step of the block of 8 experts, counted as 16 -> as they are, 9
// heads, 1 x 1400 745 -> 698, 12, 1 x 1700 974 -> 940, of 32 experts of 1024, 12, 1 x 1700 1356 -> 1342.  Below that they count coarsely
// (5 heads as 8, 9 as 16): a call on 40 heads of 5 x 300 tokens, which takes 128 queries, and one on a quarter of them give the
// same bits that way.
// Many heads fill the chip with few tokens, so from there on a second line bounds tokens x heads, in tokens of 16 heads (work).
// Measured, us, two forward passes and a backward one, 128 queries -> 32 (heads, tokens: work):
//   24, 1 x 1024: 1536 115 -> 96    32, 1 x 1024: 2048 117 -> 116    40, 1 x 1024: 2560 131 -> 147    48, 1 x 1024: 3072 139 -> 169
//   32, 1 x 512: 1024 74 -> 52    48, 1 x 512: 1536 77 -> 76    64, 1 x 512: 2048 78 -> 88    48, 2 x 451: 2706 88 -> 123    128, 1 x 512: 4096 101 -> 172
//   32, 2 x 256: 1024 52 -> 43    32, 3 x 256: 1536 54 -> 64    64, 4 x 256: 4096 91 -> 151
//   64, 2 x 128: 1024 41 -> 40    40, 4 x 128: 1280 43 -> 54    64, 4 x 128: 2048 49 -> 70
//   32, 4 x 64: 512 31 -> 29    40, 4 x 64: 640 31 -> 35    64, 8 x 64: 2048 42 -> 67
// By time alone it would lie at 2048 from 1024 positions on, 1536 from 448, 1024 from 128 and 512 below.  It lies where the kernels
// before these had it, because of what it decides besides:
// The two forms add in different orders.  A call on some of the heads takes the short form wherever the call on all of them does,
// and gives the same bits then; where all of them take the long form, some alone need not.  A lower line would take that from calls
// that have it.  Two groups of waves add in yet another order.
static bool short_sequence(int B, int S, int H) {
  const i64 tokens = (i64)B * S, heads = H > 16 ? 18 : S >= 1024 ? H : H > 8 ? 16 : H > 4 ? 8 : 4, load = tokens * heads / 16;
  if (S > 2048 || load > (S >= 1024 ? 1536 : 1024)) return false;
  return H <= 16 || tokens * H <= 16 * (S >= 448 ? 2752 : S >= 256 ? 1856 : S >= 128 ? 1344 : 768);
}

// One or two groups of waves per workgroup of the forward kernel.  One lets two workgroups share a CU, which keeps both busy
// where there are enough of them; two halve the chain of tiles, which is what counts where the workgroups are few or the longest
// ones run on alone.  Measured, us, 16 heads, causal, one group -> two (workgroups):
//   4 x 512 (256) 17.9 -> 17.6    8 x 256 (256) 12.5 -> 13.1    5 x 400 (320) 15.2 -> 21.5    2 x 1100 (288) 28.3 -> 23.8
//   3 x 1024 (384) 28.6 -> 30.1   2 x 1300 (352) 32.6 -> 29.3   2 x 1700 (448) 41.8 -> 40.1   2 x 2048 (512) 51.3 -> 50.1
//   2 x 2300 (576) 63.4 -> 67.0   1 x 2500 (320) 54.0 -> 43.7   1 x 4096 (512) 93.2 -> 85.2   1 x 5600 (704) 154 -> 159
//   8 heads: 1 x 8192 (512) 175 -> 154    32 heads: 1 x 2500 (640) 71.4 -> 77.5
// Workgroups of two leave no room beside them, so where both take about the same time other streams' kernels decide for one
// (2 x 2048: a step 0.7 % faster with one); dQ, which runs beside the experts' gradients, gains only alone (1 x 4096 355 -> 338
// us, a step 0.5 % slower) and has one.
static bool two_groups(int B, int S, int H) {
  const i64 tiles = cdiv(S, 128), workgroups = tiles * B * H;
  return tiles >= 8 && workgroups <= 256 + 10 * tiles;
}

int launch_attn_fwd_flash(const void* q, const void* k, const void* v, void* o, float* lse, int B, int S, int H,
                          int dh, int causal, hipStream_t s, const unsigned char* row_skip) {
  if (dh != DH || B <= 0 || S <= 0) return 1;
  if ((i64)S * H * DH * 2 >= ((i64)1 << 31)) return 1;      // one sequence of one tensor is addressed with 32-bit offsets
  if (((uintptr_t)q | (uintptr_t)k | (uintptr_t)v | (uintptr_t)o) & 15) return 1;
  if (short_sequence(B, S, H)) {
    static std::atomic<unsigned long long> attr_mask{0};
    if (attr_needed(attr_mask)) {
      (void)hipFuncSetAttribute((const void*)flash_fwd_short_k, hipFuncAttributeMaxDynamicSharedMemorySize, SHORT_SMEM);
      attr_done(attr_mask);
    }
    hipLaunchKernelGGL(flash_fwd_short_k, dim3((unsigned)((i64)H * cdiv(S, 32) * B)), dim3(256), SHORT_SMEM, s, (const bf16*)q, (const bf16*)k,
                       (const bf16*)v, (bf16*)o, lse, B, S, H, causal, 1.0f / sqrtf((float)dh), row_skip);
    return 0;
  }
  static std::atomic<unsigned long long> attr_mask{0};
  if (attr_needed(attr_mask)) {
    (void)hipFuncSetAttribute((const void*)flash_fwd_k<1>, hipFuncAttributeMaxDynamicSharedMemorySize, FWD_SMEM(1));
    (void)hipFuncSetAttribute((const void*)flash_fwd_k<2>, hipFuncAttributeMaxDynamicSharedMemorySize, FWD_SMEM(2));
    attr_done(attr_mask);
  }
  const int groups = two_groups(B, S, H) ? 2 : 1;
  hipLaunchKernelGGL(groups == 2 ? flash_fwd_k<2> : flash_fwd_k<1>, dim3((unsigned)((i64)H * cdiv(S, 128) * B)), dim3(256 * groups), FWD_SMEM(groups), s,
                     (const bf16*)q, (const bf16*)k, (const bf16*)v, (bf16*)o, lse, B, S, H, causal, 1.0f / sqrtf((float)dh), row_skip);
  return 0;
}

int launch_attn_bwd_flash(const void* q, const void* k, const void* v, const void* o, const void* d_o,
                          const float* lse, float* dvec, void* dq, void* dk, void* dv, int B, int S, int H, int dh,
                          int causal, hipStream_t s) {
  if (dh != DH || B <= 0 || S <= 0) return 1;
  if ((i64)S * H * DH * 2 >= ((i64)1 << 31)) return 1;      // one sequence of one tensor is addressed with 32-bit offsets
  if (((uintptr_t)q | (uintptr_t)k | (uintptr_t)v | (uintptr_t)o | (uintptr_t)d_o | (uintptr_t)dq | (uintptr_t)dk |
       (uintptr_t)dv) & 15)
    return 1;
  const float scale = 1.0f / sqrtf((float)dh);
  if (short_sequence(B, S, H)) {
    const i64 rows = (i64)B * S * H;
    hipLaunchKernelGGL(flash_dvec_k, dim3((unsigned)cdiv(rows, 16)), dim3(256), 0, s, (const bf16*)o, (const bf16*)d_o, dvec, S, H, rows);
    static std::atomic<unsigned long long> attr_mask{0};
    if (attr_needed(attr_mask)) {
      (void)hipFuncSetAttribute((const void*)flash_bwd_short_k, hipFuncAttributeMaxDynamicSharedMemorySize, SHORT_SMEM);
      attr_done(attr_mask);
    }
    hipLaunchKernelGGL(flash_bwd_short_k, dim3((unsigned)((i64)2 * H * cdiv(S, 32) * B)), dim3(256), SHORT_SMEM, s, (const bf16*)q, (const bf16*)k,
                       (const bf16*)v, (const bf16*)d_o, lse, dvec, (bf16*)dq, (bf16*)dk, (bf16*)dv, B, S, H, causal, scale);
    return 0;
  }
  size_t sm2 = 2 * DKV_STAGE;
  static std::atomic<unsigned long long> attr_mask{0};
  if (attr_needed(attr_mask)) {
    (void)hipFuncSetAttribute((const void*)flash_bwd_dq_k, hipFuncAttributeMaxDynamicSharedMemorySize, DQ_SMEM);
    (void)hipFuncSetAttribute((const void*)flash_bwd_dkv_k<1>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sm2);
    (void)hipFuncSetAttribute((const void*)flash_bwd_dkv_k<2>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)sm2);
    attr_done(attr_mask);
  }
  dim3 grid((unsigned)((i64)H * cdiv(S, 128) * B));
  hipLaunchKernelGGL(flash_bwd_dq_k, grid, dim3(256), DQ_SMEM, s, (const bf16*)q, (const bf16*)k,
                     (const bf16*)v, (const bf16*)o, (const bf16*)d_o, lse, dvec, (bf16*)dq, B, S, H, causal, scale);
  if (grid.x <= 256)         // one workgroup on a CU at most
    hipLaunchKernelGGL(flash_bwd_dkv_k<2>, grid, dim3(256), sm2, s, (const bf16*)q, (const bf16*)k, (const bf16*)v,
                       (const bf16*)d_o, lse, dvec, (bf16*)dk, (bf16*)dv, B, S, H, causal, scale);
  else
    hipLaunchKernelGGL(flash_bwd_dkv_k<1>, grid, dim3(256), sm2, s, (const bf16*)q, (const bf16*)k, (const bf16*)v,
                       (const bf16*)d_o, lse, dvec, (bf16*)dk, (bf16*)dv, B, S, H, causal, scale);
  return 0;
}
