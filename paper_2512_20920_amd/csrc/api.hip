// C ABI of the RevFFN block: argument validation, workspace, and the sequence of kernel
// launches for forward (Eq. 1-2), inverse (the display under them) and backward.
// No device synchronisation and no allocation happens outside create/destroy.
#include "../../include/revffn.h"
#include "kernels.h"

#include <math.h>
#include <mutex>
#include <new>
#include <stdlib.h>
#include <string.h>
#include <vector>

namespace {

struct Carver {            // hands out 256-byte aligned slices of one allocation (or just counts)
  char* base = nullptr;
  size_t off = 0;
  void* take(size_t bytes) {
    size_t a = (off + 255) & ~(size_t)255;
    off = a + bytes;
    return base ? (void*)(base + a) : nullptr;
  }
};

}  // namespace

// Kernel families of the per-launch timing.  The expert GEMMs (one weight matrix per expert, streamed once: bound by
// HBM) are kept apart from the dense GEMMs of the same operand layout (bound by the matrix cores).
enum { KID_GEMM_NT = 0, KID_GEMM_NN, KID_GEMM_TN, KID_GEMM_GENERIC, KID_ATTN_FWD_FLASH, KID_ATTN_BWD_FLASH,
       KID_ATTN_FWD_GENERIC, KID_ATTN_BWD_GENERIC, KID_GEMM_NT_EXPERTS, KID_GEMM_NN_EXPERTS, KID_GEMM_TN_EXPERTS,
       // the memory-bound kernels: algorithmic bytes only (every input read once, every output written once; the families
       // router_bwd and gather_rows are part of moe_bwd_rows now and keep their places in the list)
       KID_RMSNORM_FWD, KID_RMSNORM_BWD, KID_ROPE, KID_ROUTER, KID_PERMUTE, KID_COMBINE, KID_MOE_BWD_ROWS,
       KID_ROUTER_BWD, KID_DUM_FINALIZE, KID_SWIGLU_BWD, KID_COLSUM, KID_GATHER_ROWS, KID_COPY_ROWS,
       KID_COUNT };
static const char* const kid_names[KID_COUNT] = {"gemm_mfma_nt", "gemm_mfma_nn", "gemm_mfma_tn", "gemm_generic",
                                                 "attn_fwd_flash", "attn_bwd_flash", "attn_fwd_generic",
                                                 "attn_bwd_generic", "gemm_mfma_nt_experts", "gemm_mfma_nn_experts",
                                                 "gemm_mfma_tn_experts",
                                                 "rmsnorm_fwd", "rmsnorm_bwd", "rope", "router", "permute", "combine",
                                                 "moe_bwd_rows", "router_bwd", "dum_finalize", "swiglu_bwd", "colsum",
                                                 "gather_rows", "copy_rows"};
struct ProfRec { int kid; hipEvent_t a, b; double flops, bytes; };

struct revffn_ctx {
  bool prof_on = false;
  std::vector<ProfRec>* prof = nullptr;        // launches recorded since profiling was switched on
  std::vector<hipEvent_t>* ev_pool = nullptr;  // recycled events
  revffn_config cfg;
  int dt, es;                 // element type / size of weights, activations and gradients
  int sdt, ses;               // element type / size of the residual streams x1, x2, y1, y2 (float32 with fp32_streams)
  int gdt, ges;               // element type / size of the weight gradients (float32 with fp32_grads)
  int maxT;
  int mode = 0;               // 0 auto, 1 generic kernels only
  int taps = 0;
  int device = 0;
  void* slab = nullptr;
  size_t slab_bytes = 0;
  // helper streams for independent branches of one call: 0 beside the MoE half (the shared expert, the first query side;
  // going back also the weight gradients), 1 the attention half of a sweep step
  hipStream_t side[2] = {nullptr, nullptr};
  std::vector<hipEvent_t>* sync_ev = nullptr;  // ring of timing-free events for fork/join
  size_t sync_next = 0;
  bool use_streams = true;
  bool par = false;           // this call spreads independent branches over the helper streams (see fork_pays)
  int lastT = 0;
  bool small = false;         // this call is too small for helper streams, whatever the switches say (see fork_pays)
  i64 call_T = 0;             // tokens of the current call
  int lastT_rows = 0;         // lastT * top_k: permuted rows of the current routing
  // attention half
  void *n12, *U12, *Q, *K, *V, *O, *AO;
  float* lse;
  // moe half
  void *n3, *Um;
  float *wrp, *probs, *gamma, *wts;
  int *idx, *counts, *offsets, *row_map, *inv_map;
  int *tg_a, *tm_a, *tg_b, *tm_b, *tf_a, *tf_b, *tg_c, *tm_c, *tf_c;
  int max_tiles_a, max_tiles_b, max_tiles_c;
  int expert_width = 0;       // width of the routed experts' inputs and outputs: d_model, half of it with merged weights
  int bm_b = 128;             // height of the tiles in list b for the routing in the workspace: 128, or 160 (see expert_rows_b)
  int bm_c = 256;             // height of the tiles in list c: 256, or 320 (see expert_rows_c)
  int bm_c_kernel = 256;      // the height that experts_in_phases goes by: no call's, so that all calls get the same kernels
  int expert_nt = 0, expert_nn = 0;
  bool no_fused_swiglu = false; // REVFFN_NO_FUSED_SWIGLU (tuning aid): SwiGLU as a kernel of its own after the gate/up GEMM
  int expert_tile = 0;        // m-tile height of the MFMA expert GEMMs forced to 128 or 256 (REVFFN_EXPERT_TILE), 0 = by rows per expert
  int* tile_cnt;              // tiles in use of the three lists, then the flag that the routing is even
  void *Xg, *GU, *Hh, *Yp, *GUs, *Hs, *Ys, *RS;
  float *tapA, *tapM;
  void *y1c, *xtmp;
  float* resid_dev;
  // tolerance-driven inverse: > 0 = every block of rows iterates until its max|x_n - x_(n-1)| <= inv_tol, at most
  // inv_max_iters times; inv_block = positions per block inside a sequence (0 = one block for the whole call).
  // The decision is taken on the device (conv_* kernels); conv holds its state.
  float inv_tol = 0.f;
  int inv_max_iters = 0;
  int inv_block = 0;
  ConvState conv;
  size_t conv_zero_words = 0;                     // 32-bit words from conv.row_done on that start every inverse at zero
  int conv_last_nblk = 0;
  // backward
  void *dRS, *dYp, *dYs, *dHs, *dGUs, *dUm_sh, *dHh, *dGU, *dXg, *dUm, *dn3, *g1;
  float *dzext, *rinv, *rinv3, *partial;
  int* ticket;                // of the column sums
  int* blk_cnt;                     // entries per token block and expert, from the router kernel to the permutation
  // the workspace still holds every activation of this revffn_forward call (stored-activation backward)
  const void *fwd_x1 = nullptr, *fwd_x2 = nullptr, *fwd_y1 = nullptr;
  int fwd_B = 0, fwd_S = 0;
  i64 fwd_ld = 0;
  void* wr_ext;               // [E1p, d]: router rows, shared-gate row, zero rows up to a multiple of 8
  void *dzb, *dUm_r;          // bf16 logit gradients [T, E1p] and the router term of dUm [T, d]
  void *dAO, *dO, *dQ, *dK, *dV, *dU12, *dn12;
  float* dvec;
  float* rope_cs;
};

namespace {

const int BM_A = 32;    // m-tile height of the generic grouped GEMM
const int BM_B = 128;   // m-tile heights of the MFMA grouped GEMM (list b is built 160 rows high instead where that
const int BM_C = 256;   // holds a typical expert, see expert_rows_b)
const int BM_B_MID = 160;
const int BM_C_TALL = 320;      // list c where the last tile of an expert may be this high (expert_rows_c)

int check_cfg(const revffn_config* c) {
  if (!c) return REVFFN_ENULL;
  if (c->d_model < 2 || (c->d_model & 1)) return REVFFN_EINVAL;
  if (c->n_heads < 1 || c->head_dim < 2 || (c->head_dim & 1) || c->head_dim > 1024) return REVFFN_EINVAL;
  if ((long long)c->n_heads * c->head_dim != c->d_model) return REVFFN_EINVAL;
  if (c->n_experts < 1 || c->n_experts > 256) return REVFFN_EINVAL;
  if (c->top_k < 1 || c->top_k > c->n_experts || c->top_k > 16) return REVFFN_EINVAL;
  if (c->d_expert < 1 || c->d_shared < 0) return REVFFN_EINVAL;
  if (c->dtype != REVFFN_F32 && c->dtype != REVFFN_BF16) return REVFFN_EINVAL;
  if (c->fp32_streams != 0 && c->fp32_streams != 1) return REVFFN_EINVAL;
  if (c->symmetric != 0 && c->symmetric != 1) return REVFFN_EINVAL;
  if (c->fp32_grads != 0 && c->fp32_grads != 1) return REVFFN_EINVAL;
  if (c->n_inv_iters < 0 || c->n_inv_iters > 1024) return REVFFN_EINVAL;
  if (!(c->rms_eps >= 0.f) || !(c->rope_theta > 0.f)) return REVFFN_EINVAL;
  return REVFFN_OK;
}

// Lays out every workspace buffer; with c->slab == nullptr it only measures.
size_t carve(revffn_ctx* c, char* base) {
  const revffn_config& f = c->cfg;
  const size_t T = (size_t)c->maxT, d = f.d_model, h = d / 2, E = f.n_experts, k = f.top_k, I = f.d_expert,
               Is = f.d_shared, N = T * k, es = c->es, H = f.n_heads;
  const size_t E1 = E + (Is ? 1 : 0);
  Carver cv;
  cv.base = base;
  c->n12 = cv.take(2 * T * h * es);
  c->U12 = cv.take(2 * T * d * es);
  c->Q = cv.take(T * d * es);
  c->K = cv.take(T * d * es);
  c->V = cv.take(T * d * es);
  c->O = cv.take(T * d * es);
  c->AO = cv.take(T * d * es);
  c->lse = (float*)cv.take(T * H * 4);
  c->n3 = cv.take(T * h * es);
  c->Um = cv.take(T * d * es);
  c->wrp = (float*)cv.take(E1 * h * 4);
  c->probs = (float*)cv.take(T * E * 4);
  c->gamma = (float*)cv.take(T * 4);
  c->wts = (float*)cv.take(N * 4);
  c->idx = (int*)cv.take(N * 4);
  c->counts = (int*)cv.take(E * 4);
  c->offsets = (int*)cv.take((E + 1) * 4);
  c->row_map = (int*)cv.take(N * 4);
  c->inv_map = (int*)cv.take(N * 4);
  c->max_tiles_a = (int)(N / BM_A + E + 1);
  c->max_tiles_b = (int)(N / BM_B + E + 1);
  c->tg_a = (int*)cv.take(c->max_tiles_a * 4);
  c->tm_a = (int*)cv.take(c->max_tiles_a * 4);
  c->tg_b = (int*)cv.take(c->max_tiles_b * 4);
  c->tm_b = (int*)cv.take(c->max_tiles_b * 4);
  c->max_tiles_c = (int)(N / BM_C + E + 1);
  c->tg_c = (int*)cv.take(c->max_tiles_c * 4);
  c->tm_c = (int*)cv.take(c->max_tiles_c * 4);
  c->tf_c = (int*)cv.take(c->max_tiles_c * 4);
  c->tile_cnt = (int*)cv.take(4 * 4);
  c->tf_a = (int*)cv.take(c->max_tiles_a * 4);
  c->tf_b = (int*)cv.take(c->max_tiles_b * 4);
  c->Xg = cv.take(N * d * es);
  c->GU = cv.take(N * 2 * I * es);
  c->Hh = cv.take(N * I * es);
  c->Yp = cv.take(N * d * es);
  c->GUs = Is ? cv.take(T * 2 * Is * es) : nullptr;
  c->Hs = Is ? cv.take(T * Is * es) : nullptr;
  c->Ys = Is ? cv.take(T * d * es) : nullptr;
  c->RS = cv.take(T * d * es);
  c->tapA = (float*)cv.take(T * h * 4);
  c->tapM = (float*)cv.take(T * h * 4);
  c->y1c = cv.take(T * h * c->ses);
  c->xtmp = cv.take(T * h * c->ses);
  c->resid_dev = (float*)cv.take(256);
  const size_t colsums = 3 * d + 3 * h + E;      // at most this many columns are summed in a call
  {
    // state of the device-side stopping rule: the four arrays that start every inverse at zero are contiguous
    const size_t Tp = (T + 3) & ~(size_t)3;
    char* z = (char*)cv.take(Tp * (1 + 1 + 4 + 4));
    c->conv.row_done = (unsigned char*)z;
    c->conv.blk_done = (unsigned char*)(base ? z + Tp : nullptr);
    c->conv.blk_bits = (unsigned*)(base ? z + 2 * Tp : nullptr);
    c->conv.blk_iters = (int*)(base ? z + 6 * Tp : nullptr);
    c->conv_zero_words = Tp * 10 / 4;
    c->conv.blk_res = (float*)cv.take(Tp * 4);
    c->conv.stats = (int*)cv.take(256);
    c->ticket = (int*)cv.take(colsum_tickets(colsums) * 4);       // (behind the statistics: cleared together)
  }
  c->dRS = cv.take(T * d * es);
  c->dYp = cv.take(N * d * es);
  c->dYs = Is ? cv.take(T * d * es) : nullptr;
  c->dHs = Is ? cv.take(T * Is * es) : nullptr;
  c->dGUs = Is ? cv.take(T * 2 * Is * es) : nullptr;
  c->dUm_sh = Is ? cv.take(T * d * es) : nullptr;
  c->dHh = cv.take(N * I * es);
  c->dGU = cv.take(N * 2 * I * es);
  c->dXg = cv.take(N * d * es);
  c->dUm = cv.take(T * d * es);
  c->dn3 = cv.take(T * h * es);
  c->g1 = cv.take(T * h * es);
  c->dzext = (float*)cv.take(T * E1 * 4);
  const size_t E1p = (E1 + 7) / 8 * 8;
  c->wr_ext = cv.take(E1p * d * es);
  c->dzb = cv.take(T * E1p * 2);
  c->dUm_r = cv.take(T * d * es);
  c->blk_cnt = (int*)cv.take(router_blocks(T) * E * 4);
  c->rinv = (float*)cv.take(2 * T * 4);
  c->rinv3 = (float*)cv.take(T * 4);
  c->partial = (float*)cv.take(colsum_partial_floats(colsums) * 4);
  c->dAO = cv.take(T * d * es);
  c->dO = cv.take(T * d * es);
  c->dQ = cv.take(T * d * es);
  c->dK = cv.take(T * d * es);
  c->dV = cv.take(T * d * es);
  c->dU12 = cv.take(2 * T * d * es);
  c->dn12 = cv.take(2 * T * h * es);
  c->dvec = (float*)cv.take(T * H * 4);
  c->rope_cs = (float*)cv.take(T * (f.head_dim / 2) * 8);
  return cv.off + 256;
}

inline char* at(void* p, size_t elems, int es) { return (char*)p + elems * (size_t)es; }
inline const char* at(const void* p, size_t elems, int es) { return (const char*)p + elems * (size_t)es; }

// ---- GEMM shorthands --------------------------------------------------------------
// C[M,N] = A[M,K] . W^T, W row-major [N,K]
GemmArgs nt(const void* A, i64 lda, const void* W, i64 ldw, void* C, i64 ldc, int M, int N, int K) {
  GemmArgs g;
  g.A = A; g.lda = lda; g.B = W; g.ldb = ldw; g.C = C; g.ldc = ldc; g.M = M; g.N = N; g.K = K;
  return g;
}
// C[M,N] = A[M,K] . W, W row-major [K,N]
GemmArgs nn(const void* A, i64 lda, const void* W, i64 ldw, void* C, i64 ldc, int M, int N, int K) {
  GemmArgs g = nt(A, lda, W, ldw, C, ldc, M, N, K);
  g.b_trans = 1;
  return g;
}
// C[M,N] = A^T . Bm, A row-major [K,M], Bm row-major [K,N]
GemmArgs tn(const void* A, i64 lda, const void* Bm, i64 ldb, void* C, i64 ldc, int M, int N, int K) {
  GemmArgs g = nt(A, lda, Bm, ldb, C, ldc, M, N, K);
  g.a_trans = 1;
  g.b_trans = 1;
  return g;
}

// ---- optional per-kernel timing with HIP events on the launch stream -----------------
hipEvent_t prof_event(revffn_ctx* c) {
  hipEvent_t e = nullptr;
  if (!c->ev_pool->empty()) { e = c->ev_pool->back(); c->ev_pool->pop_back(); }
  else (void)hipEventCreate(&e);
  return e;
}
struct ProfScope {
  revffn_ctx* c; hipStream_t s; ProfRec r; bool on;
  ProfScope(revffn_ctx* c_, hipStream_t s_, double flops, double bytes) : c(c_), s(s_), on(c_->prof_on) {
    if (!on) return;
    r.kid = -1; r.flops = flops; r.bytes = bytes; r.a = prof_event(c); r.b = prof_event(c);
    (void)hipEventRecord(r.a, s);
  }
  void done(int kid) {
    if (!on) return;
    r.kid = kid;
    (void)hipEventRecord(r.b, s);
    c->prof->push_back(r);
  }
};

// algorithmic work of one GEMM launch: 2*M*N*K flops; every operand and the result moved once
void gemm_work(const revffn_ctx* c, const GemmArgs& g, int ta, int tb, int tc, double* flops, double* bytes) {
  const double ea = ta ? 2 : 4, eb = tb ? 2 : 4, ec = tc ? 2 : 4;
  double M = g.M, N = g.N, K = g.K, G = g.n_groups;
  if (g.group_mode == 1) { *flops = 2 * M * N * K; *bytes = M * K * ea + G * N * K * eb + M * N * ec; }
  else if (g.group_mode == 2) { double R = K;                                     // rows summed over groups
    *flops = 2 * M * N * R; *bytes = R * M * ea + R * N * eb + G * M * N * ec; }
  else { if (g.A2) K *= 2; *flops = 2 * M * N * K; *bytes = M * K * ea + N * K * eb + M * N * ec; }
  if (g.resid) *bytes += M * N * (g.resid_f32 ? 4 : c->es);
  if (g.act_half) *bytes += M * (double)g.act_half * ec;
}

// a layer's GEMM over the rows of the call (one or both streams), few enough for the kernel of that name, or with a second pair of
// operands, which no other takes
bool few_rows(const revffn_ctx* c, const GemmArgs& g) {
  return g.group_mode == 0 && !g.a_trans && (g.A2 || (g.M <= 2 * c->call_T && gemm_few_rows(c->call_T, g.N)));
}

// Up to this mean of rows per expert nearly all experts fit in one tile of 128 rows
constexpr i64 ROWS_ONE_TILE = 118;
// the routed experts' weights are more than the memory-side cache keeps from one pass over them to the next
// (of the experts that the rows reach; merged weights are half as wide, and a few tokens' experts of them do stay: Qwen shape,
// 4, 5, 6, 7 tokens, past the caches / through them, 176, 193, 207, 211 / 167, 183, 192, 202 us per forward and inverse pass,
// 8 tokens (277 MB) 220 / 221, 12 245 / 259)
bool experts_pass_through(const revffn_ctx* c, i64 rows) {
  const revffn_config& f = c->cfg;
  return 3.0 * (double)(rows < f.n_experts ? rows : f.n_experts) * f.d_expert * c->expert_width * c->es >= (double)(1 << 28);
}

// the most row tiles of 32 that `rows` rows of E experts make
i64 row_tiles32(i64 rows, i64 E) { return rows < rows / 32 + E ? rows : rows / 32 + E; }
// Which kernel takes a GEMM of the routed experts (of N outputs, a contraction of K) for `rows` permuted rows: 0 one of the tile
// kernels, 1 the one for few rows (gemm_skinny.hip), 2 the one for weights that come from memory (gemm_experts.hip)
int experts_kernel(const revffn_ctx* c, i64 rows, i64 N, i64 K, bool b_trans) {
  const i64 E = c->cfg.n_experts;
  // Small problems are latency: 32x32 tiles with k cut among the waves, up to about as many as the chip holds at once.
  // Measured, us per pass: a 512-wide block of 12 experts, 400 tokens (294 to 784 tiles) 420 -> 392, 1536 tokens (at most 936
  // of 2496: 595 -> 585; all of them 597); 256 wide, 15 experts, 753 tokens, k = 256: 872 tiles 460 -> 448, 1308 -> 440.
  // One token of merged Qwen weights (352) 199 -> 153.
  const i64 tiles32 = row_tiles32(rows, E) * ((N + 31) / 32);
  const bool past = experts_pass_through(c, rows);
  // (A row or two per expert, and weights that stay in the caches: merged, 4 tokens 170, in the kernel below 180.)
  if (tiles32 <= (K <= 256 ? 1600 : 1000) || (!past && rows <= 2 * E && K <= 4096 && tiles32 <= 6000)) return 1;
  // Above that, as long as nearly every expert fits in one row tile: see gemm_experts.hip.  Old / new, us per pass at the Qwen
  // shape: 16 tokens 925 / 895, 64 1050 / 993, 128 1105 / 1067, 240 (16 rows) 1284 / 1240, merged 37 tokens 323 / 294, 200 378 / 350;
  // 8 experts of 14336, 64 tokens 2416 / 2317, 80 (20 rows) 2505 / 2575 (experts of two tiles are read twice); 260 tokens
  // 1240 / 1337 (its workgroups leave no room for the shared expert's larger tiles beside them).  Data gradients with k long (dXg)
  // are faster on 128x256 tiles, whose lines are 512 bytes: 64 tokens 108 / 116 us alone; with a row or two per expert 20 tokens
  // 101 / 93 alone, but a step of 16, 25, 30 tokens 912, 894, 980 / 997, 972, 1085 (with a k as long its weights do not go past the
  // caches, see below, and it runs beside the weight gradients).  The rule looks at the mean.  Skewed, the hottest expert 8 times the mean, a step of 64, 128, 200, 240 tokens
  // 986, 1090, 1171, 1194 / 929, 1053, 1166, 1202, merged 37, 128, 240 285, 339, 386 / 251, 311, 364.
  if (rows <= 16 * E && (!b_trans || K <= 2048)) return 2;
  return 0;
}

// Which tile a forward GEMM of the routed experts takes beyond few rows, for `rows` permuted rows, N outputs and last tiles of up to
// bm_c rows: 256 (320) rows in phases where their rounds over the 256 CUs cost less than those of 128x256, a tile of 256
// rows (with both phases at work) 1.8 times as much.  The two add in different orders, and the calls on one block promise each other's
// bits, so the answer must not depend on the call (bm_c_kernel).  128x256 / this, us per launch, gate/up and down: 173 rows 241, 115 /
// 220, 102   200: a step 3750 / 3680   273: 285, 151 / 248, 120   347: 306, 160 / 321, 175 (two tiles of which one is
// mostly empty; the rule stays)   546: 495, 245 / 436, 206   8 experts of 14336, 175: down 221 / 316 (half the CUs; stays)
bool experts_in_phases(i64 rows, i64 E, i64 N, int bm_c) {
  const i64 mean = (rows + E - 1) / E, cols = (N + 255) / 256;
  auto rounds = [&](i64 tiles) { return (double)((E * tiles * cols + 255) / 256); };
  const i64 nt = mean <= bm_c ? 1 : (mean - (bm_c - BM_C) + BM_C - 1) / BM_C, last = mean - (nt - 1) * BM_C;
  const double tile = 1.8 * ((nt - 1) + (last > 256 ? 1.25 : last > 128 ? 1.0 : 0.55)) / nt;
  return rows > 152 * E && tile * rounds(nt) < rounds((mean + 127) / 128);
}

// Whether the shared expert's GEMM `d` goes into the launch of the routed experts' one `g`.  In calls that the kernels for few rows take,
// a launch of its own is its place in the chain or, on a helper stream, a fork and a join of it, 13 us.
bool rides(const revffn_ctx* c, const GemmArgs& g, const GemmArgs& d) {
  if (c->dt != 1 || c->mode != 0 || c->expert_tile || c->expert_nt || c->expert_nn) return false;
  if (!experts_kernel(c, c->lastT_rows, g.N, g.K, g.b_trans)) return false;
  auto ok = [&](const GemmArgs& x) {                 // what launch_gemm_mfma asks for
    return !(((uintptr_t)x.A | (uintptr_t)x.B) & 15) && !((x.lda | x.ldb | x.K) & 7) && (!x.b_trans || !(x.N & 7)) && !(x.b_group_stride & 7) &&
           x.M * x.lda < (i64)1 << 30 && (x.b_trans ? x.K : x.N) * x.ldb < (i64)1 << 30;
  };
  return ok(g) && ok(d);
}

// the dense problem that came along with the routed experts' (GemmDense), as a launch of its own
GemmArgs alone(const GemmDense& d, int b_trans) {
  GemmArgs g;
  g.A = d.A; g.lda = d.lda; g.B = d.B; g.ldb = d.ldb; g.C = d.C; g.ldc = d.ldc; g.M = d.M; g.N = d.N; g.K = d.K; g.b_trans = b_trans;
  g.act_out = d.act_out; g.ldact = g.act_half = d.act_half;
  g.dact_gu = d.dact_gu; g.dact_out = d.dact_out;
  return g;
}
GemmDense along(const GemmArgs& g) {
  GemmDense d;
  d.A = g.A; d.B = g.B; d.C = g.C; d.M = g.M; d.N = g.N; d.K = g.K; d.lda = (int)g.lda; d.ldb = (int)g.ldb; d.ldc = (int)g.ldc;
  d.act_out = g.act_out; d.act_half = g.act_half;
  d.dact_gu = g.dact_gu; d.dact_out = g.dact_out;
  return d;
}

int run_gemm(revffn_ctx* c, GemmArgs g, int ta, int tb, int tc, hipStream_t s) {
  g.few_rows = few_rows(c, g);
  GemmTypes t{ta, tb, tc, c->dt};
  double fl = 0, by = 0;
  if (c->prof_on) {
    gemm_work(c, g, ta, tb, tc, &fl, &by);
    if (g.co) {
      double f1, b1;
      gemm_work(c, alone(*g.co, g.b_trans), ta, tb, tc, &f1, &b1);
      fl += f1; by += b1;
    }
  }
  ProfScope ps(c, s, fl, by);
  // A gate/up GEMM asks for silu(gate) * up beside its output, a data gradient at that product for the gradients at gate and
  // up instead of its output.  A kernel that cannot do so in its epilogue is followed by one that reads the output back.
  void *act_out = g.act_out, *dact_out = g.dact_out;
  const int act_half = g.act_half;
  const i64 out_rows = g.group_mode == 1 ? c->lastT_rows : g.M;
  GemmDense co;
  if (g.co) co = *g.co;
  const GemmDense co_asked = co;
  if (c->no_fused_swiglu) { g.act_out = co.act_out = nullptr; g.act_half = co.act_half = 0; g.dact_out = co.dact_out = nullptr; }
  const bool has_co = g.co != nullptr;
  if (has_co) g.co = &co;
  // co_in: the problem that comes along was in the launch; otherwise it gets one of its own, whichever kernel that was
  auto finish = [&](bool co_in) -> int {
    if (has_co && !co_in) {
      const int e = run_gemm(c, alone(co_asked, g.b_trans), ta, tb, tc, s);
      if (e) return e;
      co = co_asked;
    }
    if (co_asked.act_half && !co.act_half) launch_swiglu_fwd(c->dt, co.C, co_asked.act_out, co.M, co_asked.act_half, s);
    if (co_asked.dact_out && !co.dact_out) launch_swiglu_bwd(c->dt, co.C, co.dact_gu, co_asked.dact_out, co.M, co.N, s);
    if (act_half && !g.act_half) launch_swiglu_fwd(c->dt, g.C, act_out, out_rows, act_half, s);
    if (dact_out && !g.dact_out) {
      ProfScope q(c, s, 0, 5.0 * out_rows * g.N * c->es);
      launch_swiglu_bwd(c->dt, g.C, g.dact_gu, dact_out, out_rows, g.N, s);
      q.done(KID_SWIGLU_BWD);
    }
    return 0;
  };
  if (c->dt == 1 && c->mode == 0 && ta == 1 && tb == 1) {
    if (g.group_mode == 1) {
      // Expert tiles stream weights that nothing else reads, so with few rows per expert what counts is weight bytes in
      // flight per CU: a 128x256 tile (3 stages) keeps 64 KiB of them in flight, the other shapes half of that.  With
      // many rows the matrix pipe counts: 256x256 in phases.  Measured, us per launch (mean rows per expert):
      //   forward gate/up      68: 146 (128x256), 183 (256x256)   137: 191 (160x256, see expert_rows_b), 210   273: 276, 291
      //                        546: 495, 453      512 of width 14336: 1133, 1004
      //   data gradient dXg    68: 142, 182    137: 218 (256x128), 195    273: 268, 240    546: 454, 417
      //   data gradient dHh    137: 119, 127 (1408 columns: the sixth column of tiles is half empty)    546: 254, 247
      // Shapes: 1 = 128x128, 2 = 256x128, 3 = 128x256 (160x256 where list b was built that high), 4 = 256x256
      // (REVFFN_EXPERT_NT / REVFFN_EXPERT_NN force one).
      // Data gradients on 128x256 as long as one such tile holds an expert, if the weights go past the caches (see GemmArgs::once);
      // through them up to 96 rows.  Line at 96 / 118, us per step: 1450 tokens (97 rows) 2376, 2281   1600: 2386, 2318
      // 1750: 2558, 2521   8 experts of 14336, 430 tokens (107 rows): 3564, 3447;  at 60: 1024 tokens 4 % slower.
      const i64 rows = c->lastT_rows, E = c->cfg.n_experts;
      const bool past = experts_pass_through(c, rows);
      const i64 one_tile = (past ? ROWS_ONE_TILE : 96) * E;
      int shape = g.b_trans ? c->expert_nn : c->expert_nt;
      if (c->expert_tile) shape = c->expert_tile == 256 ? 2 : 1;
      const bool forced = shape != 0;
      if (!forced) {
        if (!g.b_trans) {
          shape = experts_in_phases(rows, E, g.act_half ? 2 * g.act_half : g.N, c->bm_c_kernel) ? 4 : 3;
        }
        else if (rows > 192 * E || (rows > one_tile && g.N % 256 == 0)) shape = 4;
        else shape = rows > one_tile ? 2 : 3;
      }
      const int few = forced ? 0 : experts_kernel(c, rows, g.N, g.K, g.b_trans);
      g.few_rows = few != 0;
      g.stream = few == 2;
      bool tall = shape == 2 || shape == 4;
      g.tile_bn = shape >= 3 ? 256 : 128;
      const bool mid = c->bm_b == BM_B_MID;              // list b holds 160-row tiles: for the 160x256 forward kernel only
      if (mid && !tall) { if (g.b_trans) tall = true; else g.tile_bn = 256; }
      if (tall && g.b_trans && shape != 4) g.tile_bn = 128;
      if (g.few_rows) {
        g.tile_group = c->tg_a; g.tile_m0 = c->tm_a; g.max_tiles = (int)row_tiles32(rows, E); g.tile_bm = BM_A; g.tile_count = c->tile_cnt; g.tile_first = c->tf_a;
        // (Weights past the caches, see GemmArgs::once; with k as the slow index a line belongs to two tiles, which does not pay
        // where k is long.  Through / past, us: 8, 16, 25 tokens at the Qwen shape 862, 1005, 1107 / 816, 972, 1043;
        // merged 16, 29 tokens 300, 344 / 280, 318; 8 experts of 14336, 8 tokens, the forward layout only / both 2589 / 2629.  An expert of
        // several row tiles is then fetched once for each, which still pays skewed as above: 64, 128, 240 tokens 1038, 1178, 1308 / 929,
        // 1053, 1202.)
        g.once = rows <= 16 * E && (!g.b_trans || g.K <= 2048) && past;
      } else if (tall) {
        g.tile_group = c->tg_c; g.tile_m0 = c->tm_c; g.max_tiles = c->max_tiles_c; g.tile_bm = c->bm_c; g.tile_count = c->tile_cnt + 2;
        if (c->max_tiles_c < 32768) g.tile_first = c->tf_c;      // (the packed entry holds 15 + 16 bits)
      } else {
        g.tile_group = c->tg_b; g.tile_m0 = c->tm_b; g.max_tiles = c->max_tiles_b; g.tile_bm = c->bm_b; g.tile_count = c->tile_cnt + 1;
        if (c->max_tiles_b < 32768) g.tile_first = c->tf_b;
        g.once = rows <= ROWS_ONE_TILE * E && past;
      }
    }
    if (!g.few_rows) g.dact_out = nullptr;
    if (launch_gemm_mfma(g, t, s) == 0) {
      if (g.group_mode) ps.done(g.a_trans ? KID_GEMM_TN_EXPERTS : (g.b_trans ? KID_GEMM_NN_EXPERTS : KID_GEMM_NT_EXPERTS));
      else ps.done(g.a_trans ? KID_GEMM_TN : (g.b_trans ? KID_GEMM_NN : KID_GEMM_NT));
      return finish(g.group_mode == 1 && g.few_rows);            // (the kernels that take a second problem)
    }
  }
  if (g.group_mode == 1) { g.tile_group = c->tg_a; g.tile_m0 = c->tm_a; g.max_tiles = c->max_tiles_a; g.tile_bm = BM_A; g.tile_count = c->tile_cnt; }
  if (!c->no_fused_swiglu) g.dact_out = dact_out;
  int e = launch_gemm_generic(g, t, s) == 0 ? 0 : REVFFN_EUNSUPPORTED;
  ps.done(KID_GEMM_GENERIC);
  return e ? e : finish(false);
}
int run_gemm(revffn_ctx* c, const GemmArgs& g, hipStream_t s) { return run_gemm(c, g, c->dt, c->dt, c->dt, s); }
// a GEMM whose result is a weight gradient: written in the gradient dtype (float32 with fp32_grads)
// (weight gradients run on helper streams beside the data-gradient chain: the tile with the least CU-time, see
// GemmArgs::bulk; measured 1.3 % of a headline step with the shared expert's forward GEMMs treated the same way)
int run_wgrad(revffn_ctx* c, const GemmArgs& g0, hipStream_t s) {
  GemmArgs g = g0;
  g.bulk = c->par;
  return run_gemm(c, g, c->dt, c->dt, c->gdt, s);
}

// ---- the memory-bound kernels, timed like the GEMMs when profiling is on: algorithmic bytes = every input read
// once and every output written once (index arrays and per-row scalars included, gains and tables left out)
inline double esz(int dt) { return dt ? 2.0 : 4.0; }
void p_rmsnorm_fwd(revffn_ctx* c, int dt, int tx, const void* x, i64 ldx, const void* g, void* out, i64 ldo, int rows,
                   int h, float eps, hipStream_t s, const unsigned char* skip = nullptr, const void* x2 = nullptr,
                   const void* g2 = nullptr, void* out2 = nullptr) {
  ProfScope ps(c, s, 0, (x2 ? 2.0 : 1.0) * rows * h * (esz(tx) + esz(dt)));
  launch_rmsnorm_fwd(dt, tx, x, ldx, g, out, ldo, rows, h, eps, s, skip, x2, g2, out2);
  ps.done(KID_RMSNORM_FWD);
}
void p_rmsnorm_bwd(revffn_ctx* c, int dt, int tx, const NormBwd& p, const NormBwd* p2, i64 ldd, i64 ldx, i64 ldo, int rows, int h,
                   float eps, hipStream_t s) {
  ProfScope ps(c, s, 0, (p2 ? 2.0 : 1.0) * ((double)rows * h * (esz(tx) + (p.base ? 3 : 2) * esz(dt)) + rows * 4.0));
  launch_rmsnorm_bwd(dt, tx, p, p2, ldd, ldx, ldo, rows, h, eps, s);
  ps.done(KID_RMSNORM_BWD);
}
void p_rope(revffn_ctx* c, int dt, void* buf, const float* cs, int T, int S, int H, int dh, float sign, hipStream_t s,
            void* buf2 = nullptr, const unsigned char* skip = nullptr) {
  ProfScope ps(c, s, 0, (buf2 ? 2.0 : 1.0) * 2.0 * T * H * dh * esz(dt));
  launch_rope(dt, buf, cs, T, S, H, dh, sign, s, buf2, skip);
  ps.done(KID_ROPE);
}
// the routing chain: logits, softmax and selection, then the permutation
void p_routing(revffn_ctx* c, const void* y1, i64 ld, const float* wrp, const float* b_router, int T, hipStream_t s) {
  const revffn_config& f = c->cfg;
  const int h = f.d_model / 2, E = f.n_experts, k = f.top_k, gate = f.d_shared ? 1 : 0;
  {
    ProfScope ps(c, s, 0, (double)T * (h * esz(c->sdt) + E * 4 + k * 8 + gate * 4) + (double)(E + gate) * h * 4);
    launch_router(c->sdt, y1, ld, wrp, b_router, c->probs, c->idx, c->wts, c->gamma, c->blk_cnt, T, h, E, k, gate,
                  f.norm_topk_prob, f.rms_eps, s);
    ps.done(KID_ROUTER);
  }
  TileLists tl{{c->tg_a, c->tg_b, c->tg_c}, {c->tm_a, c->tm_b, c->tm_c}, {c->tf_a, c->tf_b, c->tf_c},
               {c->max_tiles_a, c->max_tiles_b, c->max_tiles_c}, {BM_A, c->bm_b, BM_C}, c->tile_cnt, {0, 0, c->bm_c - BM_C}};
  ProfScope ps(c, s, 0, (double)T * k * 4 * 3);                    // idx read, row_map and inv_map written
  launch_permute(c->idx, c->blk_cnt, T, k, E, c->counts, c->offsets, c->row_map, c->inv_map, tl, s);
  ps.done(KID_PERMUTE);
}
void p_combine(revffn_ctx* c, int dt, const void* yp, const int* inv_map, const float* wts, const void* ys,
               const float* gamma, void* rs, int T, int d, int k, hipStream_t s) {
  ProfScope ps(c, s, 0, (double)T * d * esz(dt) * (k + (ys ? 2 : 1)) + (double)T * k * 8);
  launch_combine(dt, yp, inv_map, wts, ys, gamma, rs, T, d, k, s);
  ps.done(KID_COMBINE);
}
void p_moe_bwd_rows(revffn_ctx* c, int dt, const void* drs, const void* yp, const void* ys, const int* inv_map,
                    const float* wts, const float* gamma, void* dyp, void* dys, float* dzext, int T, int d,
                    int k, int E1, int has_gate, const RouterBwd& r, const RowCopy& copy, const RowGather& gather, hipStream_t s) {
  ProfScope ps(c, s, 0, (double)T * d * esz(dt) * (1 + 2 * k + (has_gate ? 2 : 0)) + 2.0 * (copy.rows_a + copy.rows_b) * d * esz(dt) + (gather.um ? (double)T * d * esz(dt) * (1 + k) : 0.0) +
                        (double)T * (r.E * 8.0 + k * 12.0 + (r.dzb ? r.E1p * 2.0 : 0.0)));
  launch_moe_bwd_rows(dt, drs, yp, ys, inv_map, wts, gamma, dyp, dys, dzext, T, d, k, E1, has_gate, r, copy, gather, s);
  ps.done(KID_MOE_BWD_ROWS);
}
void p_dum_finalize(revffn_ctx* c, int dt, const void* dxg, const int* inv_map, const void* dum_sh, const void* dum_r,
                    const float* dzext, const void* w_router, const void* ws_gate, void* dum, int T, int d, int k, int E,
                    int E1, hipStream_t s) {
  ProfScope ps(c, s, 0, (double)T * d * esz(dt) * (k + 1 + (dum_sh ? 1 : 0) + (dum_r ? 1 : 0)) + (double)T * k * 4);
  launch_dum_finalize(dt, dxg, inv_map, dum_sh, dum_r, dzext, w_router, ws_gate, dum, T, d, k, E, E1, s);
  ps.done(KID_DUM_FINALIZE);
}
void add_colsum(ColsumBatch& q, int ta, const void* a, i64 lda, int tb, const void* b, i64 ldb,
                const float* sc, int tout, void* out, int rows, int cols) {
  if (!out) return;
  q.p[q.n++] = Colsum{a, b, sc, out, lda, ldb, rows, cols, ta == 0, tb == 0, tout == 0, 0};
}
void p_colsum_batch(revffn_ctx* c, ColsumBatch& q, hipStream_t s) {
  if (!q.n) return;
  double by = 0;
  for (int i = 0; i < q.n; i++)
    by += (double)q.p[i].rows * (q.p[i].cols * ((q.p[i].a_f32 ? 4.0 : 2.0) + (q.p[i].b ? (q.p[i].b_f32 ? 4.0 : 2.0) : 0.0)) + (q.p[i].sc ? 4.0 : 0.0));
  ProfScope ps(c, s, 0, by);
  launch_colsum_batch(q, c->partial, c->ticket, s);
  ps.done(KID_COLSUM);
}
void p_copy_rows(revffn_ctx* c, int dt, const void* src, i64 lds_, void* dst, i64 ldd, int rows, int cols, hipStream_t s) {
  ProfScope ps(c, s, 0, 2.0 * rows * cols * esz(dt));
  launch_copy_rows(dt, src, lds_, dst, ldd, rows, cols, s);
  ps.done(KID_COPY_ROWS);
}

// n <= 3 dense GEMMs of one shape, layout and strides as ONE launch of the matrix-core kernel (the 2048-wide
// projections are one round of workgroups each: together they fill the chip for several rounds), or of the float32 one;
// bf16 problems that the former does not take run one after the other.  tc: element type of the results.
int run_gemm_multi(revffn_ctx* c, const GemmArgs* subs, int n, int tc, hipStream_t s) {
  if (n <= 0) return 0;
  if (n > 1) {
    GemmArgs g = subs[0];
    g.n_sub = n;
    g.few_rows = few_rows(c, g);
    for (int z = 1; z < n; z++) {
      g.subA[z - 1] = subs[z].A; g.subB[z - 1] = subs[z].B; g.subC[z - 1] = subs[z].C; g.subBias[z - 1] = subs[z].bias;
    }
    GemmTypes t{c->dt, c->dt, tc, c->dt};
    double fl = 0, by = 0;
    if (c->prof_on)
      for (int z = 0; z < n; z++) {
        double f1, b1;
        gemm_work(c, subs[z], c->dt, c->dt, tc, &f1, &b1);
        fl += f1; by += b1;
      }
    ProfScope ps(c, s, fl, by);
    if (c->dt == 1 && c->mode == 0) {
      if (launch_gemm_mfma(g, t, s) == 0) {
        ps.done(g.a_trans ? KID_GEMM_TN : (g.b_trans ? KID_GEMM_NN : KID_GEMM_NT));
        return 0;
      }
    } else if (launch_gemm_generic(g, t, s) == 0) {
      ps.done(KID_GEMM_GENERIC);
      return 0;
    }
  }
  for (int z = 0; z < n; z++) {
    int e = run_gemm(c, subs[z], c->dt, c->dt, tc, s);
    if (e) return e;
  }
  return 0;
}

// whether a layer of N outputs may take norm or rotation along (a rule on the call and the layer, as gemm_few_rows)
bool norms_in_gemm(const revffn_ctx* c, i64 N) { return c->dt == 0 || (c->mode == 0 && gemm_few_rows(c->call_T, N)); }

// One to three problems of one shape with the norm of A's rows (rows that suit, see suit_rows) or the rotation of the outputs in the
// same launch, where the kernel for small problems takes them; 1: nothing launched.
int run_gemm_small(revffn_ctx* c, const GemmArgs* subs, int n, hipStream_t s) {
  GemmArgs g = subs[0];
  if (!norms_in_gemm(c, g.N)) return 1;
  g.n_sub = n;
  g.few_rows = 1;
  for (int z = 1; z < n; z++) {
    if (subs[z].lda != g.lda) return 1;
    g.subA[z - 1] = subs[z].A; g.subB[z - 1] = subs[z].B; g.subC[z - 1] = subs[z].C; g.subBias[z - 1] = subs[z].bias;
    g.norm_g[z] = subs[z].norm_g[0]; g.norm_out[z] = subs[z].norm_out[0];
  }
  double fl = 0, by = 0;
  if (c->prof_on) { gemm_work(c, subs[0], c->dt, c->dt, c->dt, &fl, &by); fl *= n; by *= n; }
  const GemmTypes t{c->dt, c->dt, c->dt, c->dt};
  ProfScope ps(c, s, fl, by);
  if (c->dt == 1 ? launch_gemm_mfma(g, t, s) : launch_gemm_generic(g, t, s)) return 1;
  ps.done(c->dt == 1 ? KID_GEMM_NT : KID_GEMM_GENERIC);
  return 0;
}

// the weight gradients of several dense layers as one launch; where the bf16 kernel does not take them they run one after
// the other
int run_wgrad_batch(revffn_ctx* c, const GemmArgs* subs, int n, bool bulk, hipStream_t s) {
  if (n <= 0) return 0;
  const bool f32 = c->dt == 0 && c->gdt == 0;
  if (f32 || (c->dt == 1 && c->mode == 0)) {
    GemmBatch b;
    double fl = 0, by = 0;
    for (int j = 0; j < 2 * n; j++) {                // (the long contractions of the dense layers first)
      const GemmArgs& g = subs[j % n];
      if ((g.group_mode == 2) != (j >= n)) continue;
      GemmProb p{g.A, g.B, g.C, g.M, g.N, g.K, (int)g.lda, (int)g.ldb, (int)g.ldc, 0, 0, 0};
      if (g.group_mode == 2) { p.groups = g.n_groups; b.offsets = g.offsets; p.c_stride = g.c_group_stride; }
      b.p[b.n++] = p;
      double f1, b1;
      if (c->prof_on) { gemm_work(c, g, c->dt, c->dt, c->gdt, &f1, &b1); fl += f1; by += b1; }
    }
    ProfScope ps(c, s, fl, by);
    if (f32 ? launch_gemm_f32_batch_tn(b, s) == 0 : launch_gemm_batch_tn(b, c->gdt == 0, bulk, s) == 0) { ps.done(f32 ? KID_GEMM_GENERIC : KID_GEMM_TN); return 0; }
  }
  for (int i = 0; i < n; i++) {
    int e = run_gemm(c, subs[i], c->dt, c->dt, c->gdt, s);
    if (e) return e;
  }
  return 0;
}

#define TRY(x) do { int _e = (x); if (_e) return _e; } while (0)

// ---- fork / join between the caller's stream and the context's helper streams ----------
// Independent branches of one call run on helper streams of default priority, so that launches that do not fill the
// chip overlap: the shared expert next to the routed experts, the rebuilding of X1^ and the attention half's
// recomputation next to the MoE half's backward pass, the MoE half's weight gradients next to the attention half's
// backward pass.  Recording an event and making another stream wait for it costs the host 13 us (a launch: 3 us), so
// there are eleven such edges in a training step, between long branches only, and none at all in a call so small that the
// host would be what the GPU waits for: below about 8 us per evaluation of the block at the rates below, which a call of a
// few hundred tokens of a 512-wide block reaches.  One stream / helper streams, us per step: 512 wide, 12 experts, 400
// tokens (5.6) 324 to 350 / 340 and up to 440 where the host is slow, 800 (9.0) 436 / 405, 1200 (12) 511 / 484, 1536 532 / 506,
// float32, 60 (8.0) 400 / 393, 200 460 / 453, 400 541 / 508; 256 wide, 753 (5.9) 400 / 400, 1400 (9.3) 550 / 496, 2000 690 / 653;
// one token at the Qwen shape (38) 617 / 527.  A merged pass is little more than its experts, with one fork in it: one token
// 149 / 180, 4 tokens (64) 178 / 180, 37 tokens 354 / 337: there the line is at 60.
constexpr double FORK_PAYS = 8e-6, FORK_PAYS_MERGED = 60e-6;
bool fork_pays(const revffn_ctx* c, i64 T, double line) {
  const revffn_config& f = c->cfg;
  const double d = f.d_model, dense = 6 * d * d + 3 * d * f.d_shared, per_expert = 3 * d * f.d_expert;
  const double hit = (double)T * f.top_k < f.n_experts ? (double)T * f.top_k : f.n_experts;
  const double weights = (dense + hit * per_expert) * c->es, flops = 2.0 * T * (dense + f.top_k * per_expert);
  return weights / 5e12 + flops / (c->dt == 1 ? 7e14 : 1e14) > line;
}
hipEvent_t next_sync(revffn_ctx* c) {
  hipEvent_t e = (*c->sync_ev)[c->sync_next % c->sync_ev->size()];
  c->sync_next++;
  return e;
}
// stream `to` waits for everything enqueued so far on `from`
void after(revffn_ctx* c, hipStream_t from, hipStream_t to) {
  if (from == to) return;
  hipEvent_t e = next_sync(c);
  (void)hipEventRecord(e, from);
  (void)hipStreamWaitEvent(to, e, 0);
}
// helper stream i, or the main stream when helper streams are switched off
hipStream_t side(revffn_ctx* c, hipStream_t main, int i) { return c->par ? c->side[i] : main; }

// ---- attention half ---------------------------------------------------------------
// The GEMMs that take the norm of their rows along read them 16 bytes at a time, and add in another order than the norm kernel.
// Which of the two runs may follow from the call and the layer only, never from where the caller's rows lie (a call in place works
// from a dense copy of Y1, and promises the bits of the calls that do not): rows whose base or stride does not suit are copied to
// `dense` ([T, h], of a backward buffer that is idle until every use of the copy is done) first.
void suit_rows(revffn_ctx* c, const void** x, i64* ldx, void* dense, int T, hipStream_t s) {
  const int h = c->cfg.d_model / 2, piece = 16 / c->es;
  if (h % piece || (!((uintptr_t)*x & 15) && *ldx % piece == 0 && (i64)T * *ldx * c->es < (i64)1 << 31)) return;
  p_copy_rows(c, c->dt, *x, *ldx, dense, h, T, h, s);
  *x = dense;
  *ldx = h;
}
// U = Norm(x) . P_up^T for one stream or both (U and the normalised rows of the second behind those of the first).
// skip (may be null): rows marked there are finished rows of the inverse's iteration and are left alone.
struct NormUp { const void* x; i64 ldx; const void* gain; void *nout, *U, *dense; };
int norm_up(revffn_ctx* c, const NormUp* streams, int n, const void* pup, int T, hipStream_t s, const unsigned char* skip = nullptr) {
  const revffn_config& f = c->cfg;
  const int d = f.d_model, h = d / 2, dt = c->dt;
  NormUp p[2] = {streams[0], streams[n - 1]};
  if (c->sdt == dt && norms_in_gemm(c, d))
    for (int i = 0; i < n; i++) suit_rows(c, &p[i].x, &p[i].ldx, p[i].dense, T, s);
  if (n == 2 && p[0].ldx != p[1].ldx) {
    TRY(norm_up(c, p, 1, pup, T, s, skip));
    return norm_up(c, p + 1, 1, pup, T, s, skip);
  }
  if (c->sdt == dt) {
    GemmArgs g[2];
    for (int i = 0; i < n; i++) {
      g[i] = nt(p[i].x, p[i].ldx, pup, h, p[i].U, d, T, d, h);
      g[i].row_skip = skip;
      g[i].norm_g[0] = p[i].gain; g[i].norm_out[0] = p[i].nout; g[i].norm_eps = f.rms_eps;
    }
    if (run_gemm_small(c, g, n, s) == 0) return 0;
  }
  p_rmsnorm_fwd(c, dt, c->sdt, p[0].x, p[0].ldx, p[0].gain, p[0].nout, h, T, h, f.rms_eps, s, skip, n == 2 ? p[1].x : nullptr,
                n == 2 ? p[1].gain : nullptr, n == 2 ? p[1].nout : nullptr);
  GemmArgs g = nt(p[0].nout, h, pup, h, p[0].U, d, n * T, d, h);       // the same P_up serves both streams: stacked rows
  g.row_skip = skip;
  return run_gemm(c, g, s);
}
// n <= 3 projections of one shape, the outputs of the first n_rot rotated
int project(revffn_ctx* c, GemmArgs* q, int n, int n_rot, int T, int S, hipStream_t s, const unsigned char* skip = nullptr) {
  const revffn_config& f = c->cfg;
  if (!f.use_rope) n_rot = 0;
  if (n_rot) {
    GemmArgs& g = q[0];
    g.rope_cs = c->rope_cs; g.rope_S = S; g.rope_dh = f.head_dim; g.rope_mask = (1 << n_rot) - 1;
    if (run_gemm_small(c, q, n, s) == 0) return 0;
    g.rope_cs = nullptr;
  }
  TRY(run_gemm_multi(c, q, n, c->dt, s));
  if (n_rot) p_rope(c, c->dt, q[0].C, c->rope_cs, T, S, f.n_heads, f.head_dim, 1.f, s, n_rot == 2 ? q[1].C : nullptr, skip);
  return 0;
}
// Query side of the attention half at x1: n12[0:T], U12[0:T], Q.
int attn_q(revffn_ctx* c, const revffn_weights* w, const void* x1, i64 ld1, int B, int S, hipStream_t s,
           const unsigned char* skip = nullptr) {
  const int T = B * S, d = c->cfg.d_model;
  const NormUp nu{x1, ld1, w->norm_a1, c->n12, c->U12, c->dn12};
  TRY(norm_up(c, &nu, 1, w->pup_a, T, s, skip));
  GemmArgs gq = nt(c->U12, d, w->wq, d, c->Q, d, T, d, d);
  gq.bias = w->bq;
  gq.row_skip = skip;
  return project(c, &gq, 1, 1, T, S, s, skip);
}
// Recomputes n12, U12, Q, (K, V), O, lse, AO at streams (x1, x2).  q_done: attn_q(x1) has been enqueued already.
int attn_acts(revffn_ctx* c, const revffn_weights* w, const void* x1, i64 ld1, const void* x2, i64 ld2, int B, int S,
              bool do_kv, hipStream_t s, bool q_done = false, const unsigned char* skip = nullptr) {
  const revffn_config& f = c->cfg;
  const int T = B * S, d = f.d_model, h = d / 2, es = c->es, dt = c->dt;
  void* U2 = at(c->U12, (size_t)T * d, es);
  // queries (which the comparison block takes from stream 2 as well), keys and values: up to three problems of one shape
  GemmArgs q3[3] = {nt(f.symmetric ? U2 : c->U12, d, w->wq, d, c->Q, d, T, d, d), nt(U2, d, w->wk, d, c->K, d, T, d, d),
                    nt(U2, d, w->wv, d, c->V, d, T, d, d)};
  q3[0].bias = w->bq; q3[1].bias = w->bk; q3[2].bias = w->bv;
  const NormUp nu[2] = {{x1, ld1, w->norm_a1, c->n12, c->U12, c->dn12},
                        {x2, ld2, w->norm_a2, at(c->n12, (size_t)T * h, es), U2, at(c->dn12, (size_t)T * h, es)}};
  if (f.symmetric) {                                    // n2, U2 keep their places in the second halves of n12, U12
    TRY(norm_up(c, nu + 1, 1, w->pup_a, T, s));
    TRY(project(c, q3, 3, 2, T, S, s));
  } else if (!do_kv) {
    if (!q_done) TRY(attn_q(c, w, x1, ld1, B, S, s, skip));          // a later iterate of the inverse: query side only
  } else if (q_done) {                                 // (the query side was enqueued earlier)
    TRY(norm_up(c, nu + 1, 1, w->pup_a, T, s));
    TRY(project(c, q3 + 1, 2, 1, T, S, s));
  } else {
    TRY(norm_up(c, nu, 2, w->pup_a, T, s));
    TRY(project(c, q3, 3, 2, T, S, s));
  }
  {
    // algorithmic work of the attention core: QK^T and PV, halved by the causal mask
    double fl = 4.0 * B * (double)S * S * d * (f.causal ? 0.5 : 1.0), by = 4.0 * T * d * es;
    ProfScope ps(c, s, fl, by);
    bool done = false;
    if (dt == 1 && c->mode == 0)
      done = launch_attn_fwd_flash(c->Q, c->K, c->V, c->O, c->lse, B, S, f.n_heads, f.head_dim, f.causal, s, skip) == 0;
    if (!done) launch_attn_fwd_generic(dt, c->Q, c->K, c->V, c->O, c->lse, B, S, f.n_heads, f.head_dim, f.causal, s, skip);
    ps.done(done ? KID_ATTN_FWD_FLASH : KID_ATTN_FWD_GENERIC);
  }
  GemmArgs go = nt(c->O, d, w->wo, d, c->AO, d, T, d, d);
  go.row_skip = skip;
  TRY(run_gemm(c, go, s));
  return 0;
}
// dst = resid + sign * P_dn_a(AO)     (Eq. 1 and the second line of the inverse)
int attn_out(revffn_ctx* c, const revffn_weights* w, const void* resid, i64 ldr, float sign, void* dst, i64 ldd,
             int T, hipStream_t s, const unsigned char* skip = nullptr) {
  const int d = c->cfg.d_model, h = d / 2;
  GemmArgs g = nt(c->AO, d, w->pdn_a, d, dst, ldd, T, h, d);
  g.row_skip = skip;
  g.resid = resid; g.ldr = ldr; g.resid_sign = sign; g.resid_f32 = c->sdt == REVFFN_F32;
  if (c->taps) { g.tap = c->tapA; g.ldtap = h; }
  return run_gemm(c, g, c->dt, c->dt, c->sdt, s);
}

// ---- MoE half ---------------------------------------------------------------------
// Folded fp32 router matrix wrp = [W_r ; w_shared_gate] . P_up_m . diag(gain), into dst.
void router_fold(revffn_ctx* c, const revffn_weights* w, float* dst, hipStream_t s) {
  const revffn_config& f = c->cfg;
  const int d = f.d_model, h = d / 2, E = f.n_experts, Is = f.d_shared, dt = c->dt;
  GemmArgs a = nn(w->w_router, d, w->pup_m, h, dst, h, E + (Is ? 1 : 0), h, d);
  if (Is) a.a_last_row = w->ws_gate;      // the shared expert's gate vector is the last row
  a.col_scale = w->norm_m;
  a.small_tiles = 1;
  (void)launch_gemm_generic(a, GemmTypes{dt, dt, 0, dt}, s);
}

// Height of the tiles in list b (the routed experts' forward GEMMs) for N permuted rows over E experts.  An expert's
// rows are padded to whole tiles, its weight tile is fetched once per row tile, and with top-k of many small experts
// the mean expert (Qwen shape at 2048 tokens: 137 rows, standard deviation 12) is just above one 128-row tile: 77 %
// of the experts then take two tiles, the second nearly empty.  Tiles 160 rows high hold such experts in one (the
// forward kernels 7.5 % faster).  Only when the mean lies where that pays; a pure function of (N, E), so every call
// that reuses a routing sees the height its lists were built with.
static int expert_rows_b(const revffn_ctx* c, i64 N, i64 E) {
  if (c->expert_tile || c->expert_nt || c->expert_nn) return BM_B;          // a forced shape (tuning aid) keeps 128
  return (N > ROWS_ONE_TILE * E && N <= 152 * E) ? BM_B_MID : BM_B;
}

// The same for list c, whose tiles are 256 rows high: where the mean is a little more than a multiple of that, the last tile of
// an expert takes up to 64 rows more (320), instead of a tile of its own for them that costs more than half of a full one (the
// results' bits are the same either way).  Us per launch, gate/up, down, dHh, dXg: 8 experts of 14336, 512 rows 1075, 635,
// 513, 1250 / 910, 418, 517, 834 (320 tiles are two rounds of 256 CUs, 256 one); Qwen shape, 546 rows 464, 227, 245, 415 / 436, 206, 208, 367.
// A step: 2 x 1024 tokens of the former 9030 -> 8340, 1200 6330 -> 5720, Qwen shape 4096 4860 -> 4645, 4600 5410 -> 5230, 8192 9390 -> 9210.
// Not where a tile more per expert still is one round of CUs that takes most of them: then the taller tile only makes that round
// longer.  By dXg's grid with that tile, as long as gate/up's is one round too; a step, us, 256 rows / up to 320, 275 rows unless said:
// 192 (8 experts, 3072 wide) 1409 / 1449, 192 (8, 2048 wide, 520 rows) 1479 / 1491, 256 (8, 4096 wide) 2072 / 2121, 256 (16, 2048 wide)
// 1519 / 1554; but 128 (8, 2048 wide) 976 / 962, 144 (12, 1536 wide) 762 / 756, 384 (16, 3072 wide) 2449 / 2431, 256 with a gate/up
// of 352 (8, 4096 wide, experts of 2816) 2854 / 2734.  That is a fused step with helper streams.  On one stream,
// in a forward call (whose lists the backward of stored activations uses) and where a backward call evaluates the half itself
// (`plain`), any one round is better without: forward and stored backward, 8 experts of 1408, 512 wide, 264 and 326 rows 383 / 398,
// 401 / 423, 2048 wide, 296 and 326 rows 796 / 838, 825 / 878, of 704, 264 and 326 rows 680 / 702, 754 / 782; three separate calls, of 1408,
// 2048 wide 1285 / 1327, 1318 / 1372.
static int expert_rows_c(const revffn_ctx* c, i64 N, i64 E, bool plain) {
  if (c->expert_tile || c->expert_nt || c->expert_nn) return BM_C;
  const i64 mean = (N + E - 1) / E, over = mean % BM_C;
  if (mean < 240 || (over > 72 && over < 240)) return BM_C;
  const i64 tiles = ((mean + 16) / BM_C + 1) * E, dxg = tiles * cdiv(c->expert_width, 256), gate_up = tiles * cdiv(c->cfg.d_expert, 128);
  const bool one_round = dxg <= 256 && gate_up <= 256;
  return one_round && (plain || dxg > 160) ? BM_C : BM_C_TALL;
}

// the geometry of the routing that an evaluation of the MoE half is about to make; width: of the routed experts' inputs and outputs;
// plain: not in an inversion
void moe_begin(revffn_ctx* c, int T, int width, bool plain) {
  c->lastT = T;
  c->lastT_rows = T * c->cfg.top_k;
  c->expert_width = width;
  c->bm_b = expert_rows_b(c, c->lastT_rows, c->cfg.n_experts);
  c->bm_c = expert_rows_c(c, c->lastT_rows, c->cfg.n_experts, plain || !c->par);
  c->bm_c_kernel = expert_rows_c(c, c->lastT_rows, c->cfg.n_experts, false);
}

// The four GEMMs of the MoE half on inputs and outputs `width` wide (d_model; half of it with merged weights)
void moe_gemms(revffn_ctx* c, const void* w_gu, const void* w_dn, const void* ws_gu, const void* ws_dn, const void* in, int width, int T,
               GemmArgs* g1, GemmArgs* g2, GemmArgs* gs, GemmArgs* gd) {
  const revffn_config& f = c->cfg;
  const int E = f.n_experts, k = f.top_k, I = f.d_expert, Is = f.d_shared, N = T * k;
  *g1 = nt(in, width, w_gu, width, c->GU, 2 * I, N, 2 * I, width);
  g1->group_mode = 1; g1->n_groups = E; g1->offsets = c->offsets; g1->b_group_stride = (i64)2 * I * width;
  g1->a_gather = c->row_map; g1->gather_div = k;
  g1->act_out = c->Hh; g1->ldact = I; g1->act_half = I;          // Hh = silu(gate) * up with the GEMM
  *g2 = nt(c->Hh, I, w_dn, I, c->Yp, width, N, width, I);
  g2->group_mode = 1; g2->n_groups = E; g2->offsets = c->offsets; g2->b_group_stride = (i64)width * I;
  if (!Is) return;
  *gs = nt(in, width, ws_gu, width, c->GUs, 2 * Is, T, 2 * Is, width);
  gs->act_out = c->Hs; gs->ldact = Is; gs->act_half = Is;        // Hs = silu(gate) * up with the GEMM
  gs->bulk = c->par;                                  // beside the routed experts' GEMMs
  *gd = nt(c->Hs, Is, ws_dn, Is, c->Ys, width, T, width, Is);
  gd->bulk = gs->bulk;
}
// Which of the shared expert's forward GEMMs go along with the routed experts': both, or where the call has one stream anyway
// either.  Not in training steps that have helper streams, where the first query side shares the fork and larger tiles run beside the
// routing chain: with them along, 64 tokens at the Qwen shape 992 -> 1007 us, 128 1067 -> 1105, 160 1118 -> 1156.
// A 512-wide block, 400 tokens, 323 -> 298 us (the backward's two as well); merged Qwen weights, 1 token 145 -> 125, 37 295 -> 274, 240 353 -> 351.
// Up to a size: these kernels' tiles load twice and more of what larger ones do per product, which a wide shared expert beside narrow
// routed ones makes the larger part of the launch.  Alone -> along, us:
//   one stream, tiles of 32x32 of its gate/up GEMM: 128 wide, a step of 2048 tokens, 1920 469.6 -> 465.2,
//   2880 476.8 -> 475.4, 3840 481 -> 487, 5760 500 -> 510; merged, 1920 182.5 -> 178.7, 2880 185.3 -> 186.2, 5760 196.6 -> 206.1; 256 wide,
//   2250 147.7 -> 143.0, 3125 147.1 -> 148.1; 512 wide, 2000 123.5 -> 121.0, 2880 167.4 -> 169.1, 5760 177 -> 189
//   one stream, merged, down, row tiles of 32 x outputs x k: 128 wide, 11e6 234 -> 222, 512 wide, 24e6 183 -> 177, 768 wide, 35e6 206 -> 210
//   helper streams, merged, the same of gate/up: up to 8 row tiles 46e6 (60 experts) 325 -> 312, 92e6 357 -> 352, (128 experts)
//   46e6 427 -> 412, 58e6 484 -> 486; more of them: 24e6 203 -> 204, 35e6 190 -> 205, 46e6 617 -> 628, 47e6 209 -> 225, 92e6 622 -> 648,
//   94e6 226 -> 273, 173e6 564 -> 607
struct Riders { bool gate_up = false, down = false; GemmDense d1, d2; bool both() const { return gate_up && down; } };
Riders riders(const revffn_ctx* c, const GemmArgs& g1, const GemmArgs& g2, const GemmArgs& gs, const GemmArgs& gd) {
  Riders r;
  const bool merged = c->expert_width != c->cfg.d_model;
  if (!c->cfg.d_shared || (!c->small && !merged)) return r;
  r.gate_up = rides(c, g1, gs);
  r.down = rides(c, g2, gd);
  const i64 row_tiles = cdiv(gs.M, 32);
  const double most = 28e6;                          // (row tiles x outputs x k)
  if (c->small) {
    r.gate_up = r.gate_up && row_tiles * cdiv(gs.N, 32) <= 2560;
    r.down = r.down && (double)row_tiles * gd.N * gd.K <= most;
  } else if (!r.both() || (row_tiles > 8 && (double)row_tiles * gs.N * gs.K > most)) r.gate_up = r.down = false;
  r.d1 = along(gs);
  r.d2 = along(gd);
  return r;
}

// Recomputes n3, Um, routing, GU, Hh, Yp, shared expert and RS at y1.  q_x1 != null: the query side of the attention
// half at q_x1 (which must not depend on this MoE evaluation) is enqueued beside it and done when s goes on.
int moe_acts(revffn_ctx* c, const revffn_weights* w, const void* y1, i64 ld, int T, hipStream_t s,
             const void* q_x1 = nullptr, i64 q_ld = 0, int qB = 0, int qS = 0, const unsigned char* q_skip = nullptr, bool plain = false) {
  const revffn_config& f = c->cfg;
  const int d = f.d_model, k = f.top_k, Is = f.d_shared, dt = c->dt;
  moe_begin(c, T, d, plain);
  // The norm and the up-projection come first, then one fork (if there is work for it): the first query side and the shared expert
  // (which needs Um only) run beside the routing chain and the routed experts, and join where the results are combined.  An edge costs
  // the chain of launches more than the 6 us of the up-projection in front of the routing chain: with the routing chain
  // on a helper stream instead (two forks, two joins) a step of 128 tokens took 1412 us, now 1391; 300 tokens 1646 and
  // 1628, 4 x 512 2831 and 2809, four blocks of 1024 8421 and 8358; 20, 3000, 8192 tokens and few large experts within 1 %.
  const NormUp nu{y1, ld, w->norm_m, c->n3, c->Um, c->dn3};
  TRY(norm_up(c, &nu, 1, w->pup_m, T, s));
  // routed experts: GU = Xg . Wgu_e^T (rows gathered from Um through row_map), SwiGLU, Yp = Hh . Wd_e^T
  GemmArgs g1, g2, gs, gd;
  moe_gemms(c, w->w_gate_up, w->w_down, w->ws_gate_up, w->ws_down, c->Um, d, T, &g1, &g2, &gs, &gd);
  const Riders ride = riders(c, g1, g2, gs, gd);
  if (ride.gate_up) g1.co = &ride.d1;
  if (ride.down) g2.co = &ride.d2;
  const bool forks = q_x1 || (Is && !ride.both());
  hipStream_t s0 = side(c, s, 0);
  if (forks) after(c, s, s0);
  if (q_x1) TRY(attn_q(c, w, q_x1, q_ld, qB, qS, s0, q_skip));
  if (Is && !ride.gate_up) TRY(run_gemm(c, gs, s0));
  if (Is && !ride.down && !ride.gate_up) TRY(run_gemm(c, gd, s0));
  router_fold(c, w, c->wrp, s);
  p_routing(c, y1, ld, c->wrp, w->b_router, T, s);
  TRY(run_gemm(c, g1, s));
  if (Is && !ride.down && ride.gate_up) TRY(run_gemm(c, gd, s));
  TRY(run_gemm(c, g2, s));
  if (forks) after(c, s0, s);
  p_combine(c, dt, c->Yp, c->inv_map, c->wts, Is ? c->Ys : nullptr, c->gamma, c->RS, T, d, k, s);
  return 0;
}
// dst = resid + sign * P_dn_m(RS)     (Eq. 2 and the first line of the inverse)
int moe_out(revffn_ctx* c, const revffn_weights* w, const void* resid, i64 ldr, float sign, void* dst, i64 ldd,
            int T, hipStream_t s) {
  const int d = c->cfg.d_model, h = d / 2;
  GemmArgs g = nt(c->RS, d, w->pdn_m, d, dst, ldd, T, h, d);
  g.resid = resid; g.ldr = ldr; g.resid_sign = sign; g.resid_f32 = c->sdt == REVFFN_F32;
  if (c->taps) { g.tap = c->tapM; g.ldtap = h; }
  return run_gemm(c, g, c->dt, c->dt, c->sdt, s);
}

// End of an entry point: a call that failed half way (REVFFN_EHIP / EUNSUPPORTED from a launch) may have forked work
// onto the helper streams; the caller's stream is made to wait for them, so that whatever was enqueued is ordered
// before the caller's next work.
int finish(revffn_ctx* c, hipStream_t s, int e) {
  if (e && c && c->par)
    for (int i = 0; i < 2; i++) after(c, c->side[i], s);
  return e;
}

// ---- pre-merged adapters (section 3.2: Attn(.) = P_dn(Attn_pt(P_up .)), MLP(.) = P_dn(MLP_pt(P_up .))) ------------
// With static weights the products W . P_up and P_dn . W can be formed once; the forward and inverse passes then
// work on half-width inputs and outputs: no adapter GEMMs, Q/K/V projections and expert gate-up GEMMs with half the
// contraction length, expert down GEMMs with half the output width, and half the expert weight bytes to stream.
int merge_impl(revffn_ctx* c, const revffn_weights* w, const revffn_merged* m, hipStream_t s) {
  const revffn_config& f = c->cfg;
  const int d = f.d_model, h = d / 2, E = f.n_experts, I = f.d_expert, Is = f.d_shared, es = c->es;
  GemmArgs q3[3] = {nn(w->wq, d, w->pup_a, h, m->wq, h, d, h, d), nn(w->wk, d, w->pup_a, h, m->wk, h, d, h, d),
                    nn(w->wv, d, w->pup_a, h, m->wv, h, d, h, d)};
  TRY(run_gemm_multi(c, q3, 3, c->dt, s));
  TRY(run_gemm(c, nn(w->pdn_a, d, w->wo, d, m->wo, d, h, d, d), s));
  {
    // every expert's gate-up rows at once: [E * 2I, d] . [d, h]; in slices that keep 32-bit operand offsets valid
    const i64 rows = (i64)E * 2 * I, step = ((i64)1 << 29) / d;
    for (i64 r0 = 0; r0 < rows; r0 += step) {
      const int mrows = (int)((rows - r0) < step ? (rows - r0) : step);
      TRY(run_gemm(c, nn(at(w->w_gate_up, (size_t)r0 * d, es), d, w->pup_m, h, at(m->w_gate_up, (size_t)r0 * h, es), h, mrows, h, d), s));
    }
  }
  for (int e = 0; e < E; e++)
    TRY(run_gemm(c, nn(w->pdn_m, d, at(w->w_down, (size_t)e * d * I, es), I, at(m->w_down, (size_t)e * h * I, es), I, h, I, d), s));
  if (Is) {
    TRY(run_gemm(c, nn(w->ws_gate_up, d, w->pup_m, h, m->ws_gate_up, h, 2 * Is, h, d), s));
    TRY(run_gemm(c, nn(w->pdn_m, d, w->ws_down, Is, m->ws_down, Is, h, Is, d), s));
  }
  router_fold(c, w, m->w_router, s);
  return 0;
}

// n12, Q, (K, V), O, lse at streams (x1, x2) from merged projections.  do_kv = false: the query side only (a later
// iterate of the inverse).
int attn_acts_merged(revffn_ctx* c, const revffn_weights* w, const revffn_merged* m, const void* x1, i64 ld1,
                     const void* x2, i64 ld2, int B, int S, bool do_kv, hipStream_t s) {
  const revffn_config& f = c->cfg;
  const int T = B * S, d = f.d_model, h = d / 2, es = c->es, dt = c->dt;
  void* n2 = at(c->n12, (size_t)T * h, es);
  const int n = do_kv ? 3 : 1;
  GemmArgs q3[3] = {nt(c->n12, h, m->wq, h, c->Q, d, T, d, h), nt(n2, h, m->wk, h, c->K, d, T, d, h), nt(n2, h, m->wv, h, c->V, d, T, d, h)};
  q3[0].bias = w->bq; q3[1].bias = w->bk; q3[2].bias = w->bv;
  bool done = false;
  // few tokens: norms, projections and rotation as one launch (two if the strides differ).  Rows wider than 512 take a workgroup's
  // CU for itself there, which pays in one round of workgroups only.
  if (c->sdt == dt && f.use_rope && (h <= 512 || (i64)cdiv(T, 32) * cdiv(d, 32) * 3 <= 256)) {
    GemmArgs q[3] = {q3[0], q3[1], q3[2]};
    if (norms_in_gemm(c, d)) {
      suit_rows(c, &x1, &ld1, c->dn12, T, s);
      if (do_kv) suit_rows(c, &x2, &ld2, at(c->dn12, (size_t)T * h, es), T, s);
    }
    for (int i = 0; i < n; i++) {
      q[i].A = i ? x2 : x1; q[i].lda = i ? ld2 : ld1;
      q[i].norm_g[0] = i ? w->norm_a2 : w->norm_a1; q[i].norm_eps = f.rms_eps;
      q[i].rope_cs = c->rope_cs; q[i].rope_S = S; q[i].rope_dh = f.head_dim;
    }
    q[0].rope_mask = 3; q[1].rope_mask = 1;
    if (n == 1 || ld1 == ld2) done = run_gemm_small(c, q, n, s) == 0;
    else done = run_gemm_small(c, q, 1, s) == 0 && run_gemm_small(c, q + 1, 2, s) == 0;
  }
  if (!done) {
    if (do_kv && ld1 == ld2) p_rmsnorm_fwd(c, dt, c->sdt, x1, ld1, w->norm_a1, c->n12, h, T, h, f.rms_eps, s, nullptr, x2, w->norm_a2, n2);
    else {
      p_rmsnorm_fwd(c, dt, c->sdt, x1, ld1, w->norm_a1, c->n12, h, T, h, f.rms_eps, s);
      if (do_kv) p_rmsnorm_fwd(c, dt, c->sdt, x2, ld2, w->norm_a2, n2, h, T, h, f.rms_eps, s);
    }
    TRY(project(c, q3, n, do_kv ? 2 : 1, T, S, s));
  }
  double fl = 4.0 * B * (double)S * S * d * (f.causal ? 0.5 : 1.0), by = 4.0 * T * d * es;
  ProfScope ps(c, s, fl, by);
  done = false;
  if (dt == 1 && c->mode == 0)
    done = launch_attn_fwd_flash(c->Q, c->K, c->V, c->O, c->lse, B, S, f.n_heads, f.head_dim, f.causal, s) == 0;
  if (!done) launch_attn_fwd_generic(dt, c->Q, c->K, c->V, c->O, c->lse, B, S, f.n_heads, f.head_dim, f.causal, s);
  ps.done(done ? KID_ATTN_FWD_FLASH : KID_ATTN_FWD_GENERIC);
  return 0;
}
// dst = resid + sign * O . (P_dn_a Wo)^T
int attn_out_merged(revffn_ctx* c, const revffn_merged* m, const void* resid, i64 ldr, float sign, void* dst, i64 ldd,
                    int T, hipStream_t s) {
  const int d = c->cfg.d_model, h = d / 2;
  GemmArgs g = nt(c->O, d, m->wo, d, dst, ldd, T, h, d);
  g.resid = resid; g.ldr = ldr; g.resid_sign = sign; g.resid_f32 = c->sdt == REVFFN_F32;
  if (c->taps) { g.tap = c->tapA; g.ldtap = h; }
  return run_gemm(c, g, c->dt, c->dt, c->sdt, s);
}
// dst = resid + sign * MoE branch at y1, everything from merged weights (routing from the stored fp32 fold)
int moe_merged(revffn_ctx* c, const revffn_weights* w, const revffn_merged* m, const void* y1, i64 ld, const void* resid,
               i64 ldr, float sign, void* dst, i64 ldd, int T, hipStream_t s) {
  const revffn_config& f = c->cfg;
  const int h = f.d_model / 2, k = f.top_k, Is = f.d_shared, dt = c->dt;
  moe_begin(c, T, h, true);
  hipStream_t s0 = side(c, s, 0);
  p_rmsnorm_fwd(c, dt, c->sdt, y1, ld, w->norm_m, c->n3, h, T, h, f.rms_eps, s);
  GemmArgs g1, g2, gs, gd;
  moe_gemms(c, m->w_gate_up, m->w_down, m->ws_gate_up, m->ws_down, c->n3, h, T, &g1, &g2, &gs, &gd);
  const Riders ride = riders(c, g1, g2, gs, gd);
  if (ride.gate_up) g1.co = &ride.d1;
  if (ride.down) g2.co = &ride.d2;
  const bool forks = Is && !ride.both();
  if (forks) after(c, s, s0);
  if (Is && !ride.gate_up) TRY(run_gemm(c, gs, s0));
  if (Is && !ride.down && !ride.gate_up) TRY(run_gemm(c, gd, s0));
  p_routing(c, y1, ld, m->w_router, w->b_router, T, s);
  TRY(run_gemm(c, g1, s));
  if (Is && !ride.down && ride.gate_up) TRY(run_gemm(c, gd, s));
  TRY(run_gemm(c, g2, s));
  if (forks) after(c, s0, s);
  {
    ProfScope ps(c, s, 0, (double)T * h * esz(dt) * (k + (Is ? 1 : 0)) + 2.0 * T * h * esz(c->sdt));
    launch_combine_couple(dt, c->sdt, c->Yp, c->inv_map, c->wts, Is ? c->Ys : nullptr, c->gamma, resid, ldr, sign, dst, ldd,
                          c->taps ? c->tapM : nullptr, T, h, k, s);
    ps.done(KID_COMBINE);
  }
  return 0;
}
int check_merged(const revffn_ctx* c, const revffn_merged* m) {
  if (!m) return REVFFN_ENULL;
  if (c->cfg.symmetric) return REVFFN_EUNSUPPORTED;
  if (!m->wq || !m->wk || !m->wv || !m->wo || !m->w_gate_up || !m->w_down || !m->w_router) return REVFFN_ENULL;
  if (c->cfg.d_shared && (!m->ws_gate_up || !m->ws_down)) return REVFFN_ENULL;
  return 0;
}

int check_call(revffn_ctx* c, const revffn_weights* w, int B, int S, i64 ld, double fork_line = FORK_PAYS) {
  if (!c || !w) return REVFFN_ENULL;
  c->fwd_x1 = nullptr;                    // any call invalidates the activations a forward call left behind
  if (B < 1 || S < 1) return REVFFN_ESHAPE;
  if ((i64)B * S > c->maxT) return REVFFN_ESHAPE;
  if (ld < c->cfg.d_model / 2) return REVFFN_ESHAPE;
  c->call_T = (i64)B * S;
  c->small = !fork_pays(c, (i64)B * S, fork_line);
  c->par = c->use_streams && !c->small;
  if (!w->norm_a1 || !w->norm_a2 || !w->norm_m || !w->pup_a || !w->pdn_a || !w->pup_m || !w->pdn_m || !w->wq ||
      !w->wk || !w->wv || !w->wo || !w->w_router || !w->w_gate_up || !w->w_down)
    return REVFFN_ENULL;
  if (c->cfg.d_shared && (!w->ws_gate_up || !w->ws_down || !w->ws_gate)) return REVFFN_ENULL;
  return 0;
}

int forward_impl(revffn_ctx* c, const revffn_weights* w, const void* x1, const void* x2, void* y1, void* y2, int B,
                 int S, i64 ld, hipStream_t s) {
  const int T = B * S;
  TRY(attn_acts(c, w, x1, ld, x2, ld, B, S, true, s));
  TRY(attn_out(c, w, x1, ld, 1.f, y1, ld, T, s));                 // Eq. 1
  TRY(moe_acts(c, w, y1, ld, T, s, nullptr, 0, 0, 0, nullptr, true));
  TRY(moe_out(c, w, x2, ld, 1.f, y2, ld, T, s));                  // Eq. 2
  return 0;
}

// y1k/ldk: where the exact Y1 stays readable during and after the call (== y1 unless in place)
int inverse_impl(revffn_ctx* c, const revffn_weights* w, const void* y1, const void* y2, void* x1, void* x2, int B,
                 int S, i64 ld, float* residual, hipStream_t s, const void** y1_kept, i64* ld_kept,
                 hipStream_t s_attn = nullptr, hipStream_t* s_attn_used = nullptr) {
  const int T = B * S, h = c->cfg.d_model / 2;
  const bool sym = c->cfg.symmetric != 0;  // closed-form inverse: one evaluation of the branch at X2^, no iteration
  const bool conv = !sym && c->inv_tol > 0.f;      // stop on the residual instead of after a fixed count
  const int n = sym ? 1 : conv ? c->inv_max_iters : c->cfg.n_inv_iters;
  const void* y1k = y1;
  i64 ldk = ld;
  if (x1 == y1 && (n >= 1)) {             // in place: Y1 is needed after x1 starts being overwritten
    p_copy_rows(c, c->sdt, y1, ld, c->y1c, h, T, h, s);
    y1k = c->y1c;
    ldk = h;
  }
  const unsigned char* skip = nullptr;
  if (conv) {
    // the stopping rule runs on the device: row marks, per-block residuals and counts start at zero (a fill kernel,
    // so that the call can be captured into a graph)
    c->conv.S = S;
    c->conv.bp = c->inv_block;
    c->conv.nj = c->inv_block > 0 ? (S + c->inv_block - 1) / c->inv_block : 1;
    c->conv.nblk = c->inv_block > 0 ? B * c->conv.nj : 1;
    c->conv_last_nblk = c->conv.nblk;
    launch_fill_u32((uint32_t*)c->conv.row_done, 0, (int)c->conv_zero_words, s);
    skip = c->conv.row_done;
  }
  // the first fixed-point iterate is Y1 itself, so its query side does not wait for X2^: it runs beside the routing
  // chain.  On one stream there is nothing to fill, and both streams' norms, projections and rotations are a launch each
  // instead of two (a step of a 512-wide block of 400 tokens: 455 -> 446 us).
  const bool q_early = n >= 1 && !sym && c->par;
  TRY(moe_acts(c, w, y1k, ldk, T, s, q_early ? y1k : nullptr, ldk, B, S, skip));
  TRY(moe_out(c, w, y2, ld, -1.f, x2, ld, T, s));                 // X2^ = Y2 - MoE branch(Y1)
  if (n == 0) {
    if (x1 != y1) p_copy_rows(c, c->sdt, y1, ld, x1, ld, T, h, s);
    if (residual) launch_fill_u32((uint32_t*)residual, 0, 1, s);
  }
  // The iteration needs X2^ and nothing else of the MoE half.  A caller that goes on with work that does not need X1^
  // (the fused sweep step: the MoE half's backward pass) hands over a stream of its own for it and joins that stream
  // itself, where X1^ is first needed.
  hipStream_t sa = s;
  if (s_attn && c->par && n >= 1) { sa = s_attn; after(c, s, sa); }
  if (s_attn_used) *s_attn_used = sa;     // == s: nothing was left on another stream
  for (int it = 1; it <= n; it++) {
    const void* xin = (it == 1) ? y1k : x1;                       // iterate, started at Y1
    i64 ldin = (it == 1) ? ldk : ld;
    TRY(attn_acts(c, w, xin, ldin, x2, ld, B, S, it == 1, sa, it == 1 && q_early, skip));   // K, V depend on X2^ only: once
    if (sym && residual) launch_fill_u32((uint32_t*)residual, 0, 1, sa);    // nothing is iterated: residual 0
    if (conv) {
      // every iteration up to the cap is enqueued; workgroups whose rows have all met the tolerance exit at once,
      // and the update below touches the other rows only.  The host takes no part in the decision.
      TRY(attn_out(c, w, y1k, ldk, -1.f, c->xtmp, h, T, sa, skip));
      launch_conv_update(c->sdt, c->xtmp, h, xin, ldin, x1, ld, c->conv, T, h, sa);
      launch_conv_decide(c->conv, T, c->inv_tol, it, sa);
    } else if (!sym && it == n && residual) {
      TRY(attn_out(c, w, y1k, ldk, -1.f, c->xtmp, h, T, sa));
      launch_fill_u32((uint32_t*)residual, 0, 1, sa);
      launch_absdiff_max_copy(c->sdt, c->xtmp, h, xin, ldin, x1, ld, residual, T, h, sa);
    } else {
      TRY(attn_out(c, w, y1k, ldk, -1.f, x1, ld, T, sa));         // x <- Y1 - attention branch(x, X2^)
    }
  }
  if (conv) launch_conv_finalize(c->conv, residual, sa);
  if (y1_kept) { *y1_kept = y1k; *ld_kept = ldk; }
  return 0;
}

void* gfield(const revffn_grads* g, size_t off) { return g ? *(void* const*)((const char*)g + off) : nullptr; }
#define GF(name) gfield(g, offsetof(revffn_grads, name))

int backward_impl(revffn_ctx* c, const revffn_weights* w, const void* x1, const void* x2, const void* y1, i64 ldy,
                  const void* dy1, const void* dy2, void* dx1, void* dx2, const revffn_grads* g, int B, int S,
                  i64 ld, bool reuse_moe, bool reuse_kv, hipStream_t s, bool reuse_attn = false,
                  hipStream_t s_attn = nullptr) {
  const revffn_config& f = c->cfg;
  const int T = B * S, d = f.d_model, h = d / 2, E = f.n_experts, k = f.top_k, I = f.d_expert, Is = f.d_shared;
  const int N = T * k, E1 = E + (Is ? 1 : 0), dt = c->dt, es = c->es;
  // ---- recompute the attention half at (x1, x2)
  // (K, V and the normalised, lifted X2 are still those of the inverse when it ran in the same call: same X2 bits)
  // The MoE half's backward pass needs dY2, Y1 and the MoE activations only; the attention half is recomputed beside
  // it on a stream of its own (sa) and joined where its activations are first used.  (With y1 == NULL the MoE half
  // needs the recomputed Y1 first: one stream.)  s_attn: the stream the caller's inverse left X1^ on.
  hipStream_t sa = s;
  if (y1 && c->par && !reuse_attn) {
    sa = s_attn ? s_attn : c->side[1];
    if (!s_attn) after(c, s, sa);
  } else if (s_attn && s_attn != s) {
    after(c, s_attn, s);                  // no overlap in this call: X1^ is needed on s from here on
  }
  if (!reuse_attn) TRY(attn_acts(c, w, x1, ld, x2, ld, B, S, !reuse_kv, sa));
  if (!y1) {
    TRY(attn_out(c, w, x1, ld, 1.f, c->y1c, h, T, s));
    y1 = c->y1c;
    ldy = h;
    reuse_moe = false;
  }
  // ---- recompute the MoE half at the exact y1
  if (!reuse_moe) TRY(moe_acts(c, w, y1, ldy, T, s, nullptr, 0, 0, 0, nullptr, true));
  // ---- MoE half backward: Y2 = X2 + P_dn_m(RS)
  // Weight gradients are leaves of the computation.  With helper streams they run on sw, the experts' next to the data
  // gradients of the experts, the dense layers' known before the attention core's backward pass as one launch next to
  // that, so that each launch's last, partly filled round of workgroups is filled by the other stream; the rest, or
  // without helper streams all of the dense ones, are one launch near the end.  The column sums (bias and gain
  // gradients) are one launch at the end.
  hipStream_t sw = side(c, s, 0);
  GemmArgs wg[GEMM_BATCH];
  int nwg = 0;
  bool sw_used = false;
  auto to_sw = [&]() { after(c, s, sw); sw_used = true; };      // sw may use what s has computed so far
  // In calls too small for helper streams the experts' weight gradients wait for the dense layers' launch, where they are fewer than the tiles
  // that suit larger ones (see pick_tile).  512 wide, 12 experts, 400 tokens 297 -> 286 us per step, 256 wide, 753 tokens 375 -> 361, float32,
  // 64 tokens 253 -> 245.
  // (Only widths of whole 16-byte pieces: for one problem of another that launch refuses all of them, or in float32 takes them through
  // slower loads.  512 wide, 12 experts of 196, 400 tokens 379 us with the experts among them, 336 without.)
  const bool batched = c->small && (i64)cdiv(d, 256) * cdiv(2 * I, 256) * E <= 256 && I % (16 / c->es) == 0;
  ColsumBatch cs;
  TRY(run_gemm(c, nn(dy2, ld, w->pdn_m, d, c->dRS, d, T, d, h), s));
  // (for the matrix-core router GEMM below: the logit gradients also in bf16, and the router rows stacked, dz . [W_r ; w_gate ; 0])
  const bool dz_bf16 = dt == 1 && c->mode == 0;
  const int E1p = (E1 + 7) / 8 * 8;
  const RouterBwd rb{c->probs, c->idx, E, f.norm_topk_prob, dz_bf16 ? c->dzb : nullptr, E1p};
  // Xg, the permuted rows of Um: for the gate/up weight gradient
  const RowGather rg{GF(w_gate_up) ? c->Um : nullptr, c->Xg};
  const RowCopy rc{w->w_router, Is ? w->ws_gate : w->w_router, c->wr_ext, dz_bf16 ? E : 0, dz_bf16 && Is ? 1 : 0};
  p_moe_bwd_rows(c, dt, c->dRS, c->Yp, c->Ys, c->inv_map, c->wts, c->gamma, c->dYp, c->dYs, c->dzext, T, d, k, E1, Is ? 1 : 0, rb, rc, rg, s);
  // The shared expert's data gradients go in front of the weight gradients on sw: a stream of their own is one more edge in
  // the chain, and one more hardware queue (see the streams' creation).  Own stream / sw: 128 tokens 1386 / 1370 us,
  // 3 x 333, adapters only, 1633 / 1626, skewed 2 x 2048 4553 / 4580, four blocks of 1024 8302 / 8255, others within 1 %.
  hipEvent_t shared_done = nullptr;
  GemmArgs a1 = nn(c->dYp, d, w->w_down, I, c->dHh, I, N, I, d);           // dHh = dYp . Wd_e
  a1.group_mode = 1; a1.n_groups = E; a1.offsets = c->offsets; a1.b_group_stride = (i64)d * I;
  a1.dact_gu = c->GU; a1.dact_out = c->dGU;
  GemmArgs a2 = nn(c->dGU, 2 * I, w->w_gate_up, d, c->dXg, d, N, d, 2 * I);          // dXg = dGU . Wgu_e
  a2.group_mode = 1; a2.n_groups = E; a2.offsets = c->offsets; a2.b_group_stride = (i64)2 * I * d;
  GemmDense d1, d2;
  if (Is) {
    GemmArgs dh = nn(c->dYs, d, w->ws_down, Is, c->dHs, Is, T, Is, d);
    dh.dact_gu = c->GUs; dh.dact_out = c->dGUs;
    const GemmArgs du = nn(c->dGUs, 2 * Is, w->ws_gate_up, d, c->dUm_sh, d, T, d, 2 * Is);
    d1 = along(dh);
    d2 = along(du);
    if (c->small && rides(c, a1, dh)) a1.co = &d1;                         // (see riders)
    if (a1.co && rides(c, a2, du)) a2.co = &d2;
    after(c, s, sw);
    if (!a1.co) {
      TRY(run_gemm(c, dh, sw));
      TRY(run_gemm(c, du, sw));
    }
    if (sw != s) { shared_done = next_sync(c); (void)hipEventRecord(shared_done, sw); }
    if (GF(ws_down)) wg[nwg++] = tn(c->dYs, d, c->Hs, Is, GF(ws_down), Is, d, Is, T);
    if (GF(ws_gate_up)) wg[nwg++] = tn(c->dGUs, 2 * Is, c->Um, d, GF(ws_gate_up), d, 2 * Is, d, T);
  }
  {
    if (GF(w_down)) {
      if (!Is) to_sw();                                                    // (else sw has waited for dYp already)
      sw_used = true;
      GemmArgs b = tn(c->dYp, d, c->Hh, I, GF(w_down), I, d, I, N);        // dWd_e = dYp_e^T . Hh_e
      b.group_mode = 2; b.n_groups = E; b.offsets = c->offsets; b.tile_count = c->tile_cnt + 3; b.c_group_stride = (i64)d * I;
      if (batched) wg[nwg++] = b;
      else TRY(run_wgrad(c, b, sw));
    }
    TRY(run_gemm(c, a1, s));
    if (a1.co && !a2.co) TRY(run_gemm(c, nn(c->dGUs, 2 * Is, w->ws_gate_up, d, c->dUm_sh, d, T, d, 2 * Is), s));
    if (GF(w_gate_up)) {
      // dWgu_e = dGU_e^T . Xg_e
      to_sw();
      GemmArgs b = tn(c->dGU, 2 * I, c->Xg, d, GF(w_gate_up), d, 2 * I, d, N);
      b.group_mode = 2; b.n_groups = E; b.offsets = c->offsets; b.tile_count = c->tile_cnt + 3; b.c_group_stride = (i64)2 * I * d;
      if (batched) wg[nwg++] = b;
      else TRY(run_wgrad(c, b, sw));
    }
    TRY(run_gemm(c, a2, s));
  }
  if (g && g->b_router) add_colsum(cs, 0, c->dzext, E1, 0, nullptr, 0, nullptr, 0, g->b_router, T, E);
  const void* dum_r = nullptr;
  if (dz_bf16) {
    // router term of dUm on the matrix cores, contraction over E1p
    GemmArgs a = nn(c->dzb, E1p, c->wr_ext, d, c->dUm_r, d, T, d, E1p);
    GemmTypes tt{1, 1, 1, 1};
    if (launch_gemm_mfma(a, tt, s) == 0) dum_r = c->dUm_r;
  }
  if (shared_done) (void)hipStreamWaitEvent(s, shared_done, 0);
  p_dum_finalize(c, dt, c->dXg, c->inv_map, Is ? c->dUm_sh : nullptr, dum_r, c->dzext, w->w_router, w->ws_gate,
                      c->dUm, T, d, k, E, E1, s);
  if (GF(pup_m)) wg[nwg++] = tn(c->dUm, d, c->n3, h, GF(pup_m), h, d, h, T);
  TRY(run_gemm(c, nn(c->dUm, d, w->pup_m, h, c->dn3, h, T, h, d), s));
  // g1 = dY1 + Norm'(dn3): total gradient at Y1
  p_rmsnorm_bwd(c, dt, c->sdt, NormBwd{c->dn3, y1, w->norm_m, dy1, ld, c->g1, c->rinv3}, nullptr, h, ldy, h, T, h, f.rms_eps, s);
  add_colsum(cs, c->sdt, y1, ldy, dt, c->dn3, h, c->rinv3, c->gdt, GF(norm_m), T, h);
  // ---- attention half backward: Y1 = X1 + P_dn_a(AO)
  if (sa != s) after(c, sa, s);           // the recomputed attention activations (and X1^ of a fused call)
  if (GF(pdn_m)) wg[nwg++] = tn(dy2, ld, c->RS, d, GF(pdn_m), d, h, d, T);
  if (GF(pdn_a)) wg[nwg++] = tn(c->g1, h, c->AO, d, GF(pdn_a), d, h, d, T);
  TRY(run_gemm(c, nn(c->g1, h, w->pdn_a, d, c->dAO, d, T, d, h), s));
  if (GF(wo)) wg[nwg++] = tn(c->dAO, d, c->O, d, GF(wo), d, d, d, T);
  {
    const bool router_w = GF(w_router) != nullptr, gate_w = Is && GF(ws_gate);
    if (router_w || gate_w || (c->par && nwg)) to_sw();
    if (router_w || gate_w) {
      // [dW_r ; dw_shared_gate] = dzext^T . Um in one fp32-A GEMM (the gate row alone if that is all that is wanted)
      GemmArgs a = router_w ? tn(c->dzext, E1, c->Um, d, GF(w_router), d, gate_w ? E1 : E, d, T)
                            : tn(c->dzext + E, E1, c->Um, d, GF(ws_gate), d, 1, d, T);
      if (router_w && gate_w) a.c_last_row = GF(ws_gate);
      a.small_tiles = 1;
      GemmTypes t{0, dt, c->gdt, dt};
      if (launch_gemm_generic(a, t, sw)) return REVFFN_EUNSUPPORTED;
    }
    if (c->par) { TRY(run_wgrad_batch(c, wg, nwg, true, sw)); nwg = 0; }
  }
  TRY(run_gemm(c, nn(c->dAO, d, w->wo, d, c->dO, d, T, d, d), s));
  {
    // five S x S x dh products (scores, dP, dV, dQ, dK), halved by the causal mask
    double fl = 10.0 * B * (double)S * S * d * (f.causal ? 0.5 : 1.0), by = 8.0 * T * d * es;
    ProfScope ps(c, s, fl, by);
    bool done = false;
    if (dt == 1 && c->mode == 0)
      done = launch_attn_bwd_flash(c->Q, c->K, c->V, c->O, c->dO, c->lse, c->dvec, c->dQ, c->dK, c->dV, B, S,
                                   f.n_heads, f.head_dim, f.causal, s) == 0;
    if (!done)
      launch_attn_bwd_generic(dt, c->Q, c->K, c->V, c->O, c->dO, c->lse, c->dvec, c->dQ, c->dK, c->dV, B, S,
                              f.n_heads, f.head_dim, f.causal, s);
    ps.done(done ? KID_ATTN_BWD_FLASH : KID_ATTN_BWD_GENERIC);
  }
  if (f.use_rope) {
    p_rope(c, dt, c->dQ, c->rope_cs, T, S, f.n_heads, f.head_dim, -1.f, s, c->dK);   // both in one launch
  }
  const void* U1 = c->U12;
  const void* U2 = at(c->U12, (size_t)T * d, es);
  void* dU1 = c->dU12;
  void* dU2 = at(c->dU12, (size_t)T * d, es);
  const bool sym = f.symmetric != 0;
  if (GF(wq)) wg[nwg++] = tn(c->dQ, d, sym ? U2 : U1, d, GF(wq), d, d, d, T);
  if (GF(wk)) wg[nwg++] = tn(c->dK, d, U2, d, GF(wk), d, d, d, T);
  if (GF(wv)) wg[nwg++] = tn(c->dV, d, U2, d, GF(wv), d, d, d, T);
  if (w->bq) add_colsum(cs, dt, c->dQ, d, dt, nullptr, 0, nullptr, c->gdt, GF(bq), T, d);
  if (w->bk) add_colsum(cs, dt, c->dK, d, dt, nullptr, 0, nullptr, c->gdt, GF(bk), T, d);
  if (w->bv) add_colsum(cs, dt, c->dV, d, dt, nullptr, 0, nullptr, c->gdt, GF(bv), T, d);
  // dU2 = dK . Wk + dV . Wv: one contraction over both where the kernel takes two pairs of operands (then in one launch with
  // dU1 = dQ . Wq), else one after the other, with the first product rounded in between
  const bool pairs = dt == 0 || c->mode == 1 || gemm_pairs(T, d);
  GemmArgs du[2] = {nn(c->dK, d, w->wk, d, dU2, d, T, d, d), nn(c->dQ, d, w->wq, d, dU1, d, T, d, d)};
  if (pairs) {
    du[0].A2 = c->dV; du[0].B2 = w->wv;
    TRY(run_gemm_multi(c, du, sym ? 1 : 2, dt, s));
  } else {
    TRY(run_gemm(c, du[0], s));
    GemmArgs a = nn(c->dV, d, w->wv, d, dU2, d, T, d, d);        // dU2 += dV . Wv
    a.resid = dU2; a.ldr = d; a.resid_sign = 1.f;
    TRY(run_gemm(c, a, s));
  }
  // sw's weight gradients read dy2, which dx2, written below, may alias
  auto before_dx2 = [&]() { if (sw_used && dx2 == dy2) { after(c, sw, s); sw_used = false; } };
  void* n2 = at(c->n12, (size_t)T * h, es);
  void* dn2 = at(c->dn12, (size_t)T * h, es);
  if (sym) {
    // the query path ends in stream 2 too: dU2 += dQ . Wq; stream 1 only carries the residual path
    GemmArgs a = nn(c->dQ, d, w->wq, d, dU2, d, T, d, d);
    a.resid = dU2; a.ldr = d; a.resid_sign = 1.f;
    TRY(run_gemm(c, a, s));
    if (GF(pup_a)) wg[nwg++] = tn(dU2, d, n2, h, GF(pup_a), h, d, h, T);
    TRY(run_gemm(c, nn(dU2, d, w->pup_a, h, dn2, h, T, h, d), s));
    TRY(run_wgrad_batch(c, wg, nwg, false, s));
    before_dx2();
    p_rmsnorm_bwd(c, dt, c->sdt, NormBwd{dn2, x2, w->norm_a2, dy2, ld, dx2, c->rinv + T}, nullptr, h, ld, ld, T, h, f.rms_eps, s);
    p_copy_rows(c, dt, c->g1, h, dx1, ld, T, h, s);              // dX1 = total gradient at Y1
    if (GF(norm_a1)) launch_zero(c->gdt, GF(norm_a1), h, s);           // stream 1 is not normalised in this block
  } else {
    if (!pairs) TRY(run_gemm(c, du[1], s));
    if (GF(pup_a)) wg[nwg++] = tn(c->dU12, d, c->n12, h, GF(pup_a), h, d, h, 2 * T);
    TRY(run_gemm(c, nn(c->dU12, d, w->pup_a, h, c->dn12, h, 2 * T, h, d), s));
    TRY(run_wgrad_batch(c, wg, nwg, false, s));
    before_dx2();
    // dX1 = g1 + Norm'(dn1);  dX2 = dY2 + Norm'(dn2)
    const NormBwd nb2{dn2, x2, w->norm_a2, dy2, ld, dx2, c->rinv + T};
    p_rmsnorm_bwd(c, dt, c->sdt, NormBwd{c->dn12, x1, w->norm_a1, c->g1, h, dx1, c->rinv}, &nb2, h, ld, ld, T, h, f.rms_eps, s);
    add_colsum(cs, c->sdt, x1, ld, dt, c->dn12, h, c->rinv, c->gdt, GF(norm_a1), T, h);
  }
  add_colsum(cs, c->sdt, x2, ld, dt, dn2, h, c->rinv + T, c->gdt, GF(norm_a2), T, h);
  p_colsum_batch(c, cs, s);
  if (sw_used) after(c, sw, s);          // every weight gradient is complete for the caller's stream
  return 0;
}

}  // namespace

// ====================================================================================
extern "C" {

size_t revffn_workspace_bytes(const revffn_config* cfg, int32_t max_B, int32_t max_S) {
  if (check_cfg(cfg) || max_B < 1 || max_S < 1 || (long long)max_B * max_S > (1 << 24)) return 0;
  revffn_ctx tmp;
  tmp.cfg = *cfg;
  tmp.dt = cfg->dtype;
  tmp.es = cfg->dtype == REVFFN_BF16 ? 2 : 4;
  tmp.sdt = cfg->fp32_streams ? REVFFN_F32 : cfg->dtype;
  tmp.ses = tmp.sdt == REVFFN_BF16 ? 2 : 4;
  tmp.gdt = cfg->fp32_grads ? REVFFN_F32 : cfg->dtype;
  tmp.ges = tmp.gdt == REVFFN_BF16 ? 2 : 4;
  tmp.maxT = max_B * max_S;
  return carve(&tmp, nullptr);
}

void revffn_destroy(revffn_ctx* c);

int revffn_create(revffn_ctx** out, const revffn_config* cfg, int32_t max_B, int32_t max_S) {
  if (!out) return REVFFN_ENULL;
  *out = nullptr;
  int e = check_cfg(cfg);
  if (e) return e;
  if (max_B < 1 || max_S < 1 || (long long)max_B * max_S > (1 << 24)) return REVFFN_ESHAPE;
  revffn_ctx* c = new (std::nothrow) revffn_ctx;
  if (!c) return REVFFN_EWORKSPACE;
  memset(c, 0, sizeof(*c));
  c->prof = new (std::nothrow) std::vector<ProfRec>();
  c->ev_pool = new (std::nothrow) std::vector<hipEvent_t>();
  if (!c->prof || !c->ev_pool) { delete c->prof; delete c->ev_pool; delete c; return REVFFN_EWORKSPACE; }
  c->cfg = *cfg;
  c->dt = cfg->dtype;
  c->es = cfg->dtype == REVFFN_BF16 ? 2 : 4;
  c->sdt = cfg->fp32_streams ? REVFFN_F32 : cfg->dtype;
  c->ses = c->sdt == REVFFN_BF16 ? 2 : 4;
  c->gdt = cfg->fp32_grads ? REVFFN_F32 : cfg->dtype;
  c->ges = c->gdt == REVFFN_BF16 ? 2 : 4;
  c->maxT = max_B * max_S;
  c->slab_bytes = carve(c, nullptr);
  if (hipGetDevice(&c->device) != hipSuccess) { delete c->prof; delete c->ev_pool; delete c; return REVFFN_EHIP; }
  if (hipMalloc(&c->slab, c->slab_bytes) != hipSuccess) {
    (void)hipGetLastError();
    delete c->prof; delete c->ev_pool; delete c;
    return REVFFN_EWORKSPACE;
  }
  carve(c, (char*)c->slab);
  (void)hipMemset(c->wr_ext, 0, (size_t)((c->cfg.n_experts + (c->cfg.d_shared ? 1 : 0) + 7) / 8 * 8) * c->cfg.d_model * c->es);
  const size_t ticket_bytes = colsum_tickets((size_t)9 * (cfg->d_model / 2) + cfg->n_experts) * 4;
  (void)hipMemset(c->conv.stats, 0, (size_t)((char*)c->ticket - (char*)c->conv.stats) + ticket_bytes);
  c->use_streams = getenv("REVFFN_NO_STREAMS") == nullptr;
  { const char* e = getenv("REVFFN_EXPERT_TILE"); if (e && (atoi(e) == 256 || atoi(e) == 128)) c->expert_tile = atoi(e); }
  { const char* e = getenv("REVFFN_NO_FUSED_SWIGLU"); c->no_fused_swiglu = e && atoi(e) != 0; }
  { const char* e = getenv("REVFFN_EXPERT_NT"); if (e && atoi(e) >= 1 && atoi(e) <= 4) c->expert_nt = atoi(e); }
  { const char* e = getenv("REVFFN_EXPERT_NN"); if (e && atoi(e) >= 1 && atoi(e) <= 4) c->expert_nn = atoi(e); }
  c->sync_ev = new (std::nothrow) std::vector<hipEvent_t>();
  bool ok = c->sync_ev != nullptr;
  // Two streams: a process has four hardware queues by default, streams beyond them share one, and work of streams that share
  // runs one after the other.  With four helper streams two of them (of a second context even the caller's and one of them)
  // did: a step of 300 tokens 1627 us, of 512 1790, of 3 x 333 without block gradients 1713; with two 1520, 1687, 1625.
  for (int i = 0; ok && i < 2; i++) ok = hipStreamCreateWithFlags(&c->side[i], hipStreamNonBlocking) == hipSuccess;
  for (int i = 0; ok && i < 96; i++) {
    hipEvent_t e;
    ok = hipEventCreateWithFlags(&e, hipEventDisableTiming) == hipSuccess;
    if (ok) c->sync_ev->push_back(e);
  }
  if (!ok) { revffn_destroy(c); return REVFFN_EHIP; }
  // rotary table: cs[s][i] = (cos, sin)(s * theta^(-2i/dh)), built in double precision on the host.  One entry per
  // position a call may use: a call may put all maxT tokens into one sequence.
  const int half = cfg->head_dim / 2;
  std::vector<float> tab;
  try { tab.resize((size_t)c->maxT * half * 2); } catch (...) { revffn_destroy(c); return REVFFN_EWORKSPACE; }
  for (int sp = 0; sp < c->maxT; sp++)
    for (int i = 0; i < half; i++) {
      double ang = (double)sp * pow((double)cfg->rope_theta, -2.0 * i / (double)cfg->head_dim);
      tab[((size_t)sp * half + i) * 2 + 0] = (float)cos(ang);
      tab[((size_t)sp * half + i) * 2 + 1] = (float)sin(ang);
    }
  if (hipMemcpy(c->rope_cs, tab.data(), tab.size() * 4, hipMemcpyHostToDevice) != hipSuccess) {
    revffn_destroy(c);                      // streams, events and the workspace go with it
    return REVFFN_EHIP;
  }
  *out = c;
  return REVFFN_OK;
}

static void prof_clear(revffn_ctx* c) {
  for (auto& r : *c->prof) { c->ev_pool->push_back(r.a); c->ev_pool->push_back(r.b); }
  c->prof->clear();
}

void revffn_destroy(revffn_ctx* c) {
  if (!c) return;
  (void)hipDeviceSynchronize();          // helper streams may still hold work of the last call
  if (c->prof) {
    prof_clear(c);
    for (hipEvent_t e : *c->ev_pool) (void)hipEventDestroy(e);
    delete c->prof;
    delete c->ev_pool;
  }
  if (c->sync_ev) {
    for (hipEvent_t e : *c->sync_ev) (void)hipEventDestroy(e);
    delete c->sync_ev;
  }
  for (int i = 0; i < 2; i++) if (c->side[i]) (void)hipStreamDestroy(c->side[i]);
  if (c->slab) (void)hipFree(c->slab);
  delete c;
}

int revffn_profile_enable(revffn_ctx* c, int32_t on) {
  if (!c) return REVFFN_ENULL;
  prof_clear(c);
  c->prof_on = on != 0;
  return 0;
}

int revffn_profile_read(revffn_ctx* c, int32_t kid, double* ms_total, int64_t* launches, double* flops,
                        double* bytes) {
  if (!c) return REVFFN_ENULL;
  if (kid < 0 || kid >= KID_COUNT) return REVFFN_EINVAL;
  double ms = 0, fl = 0, by = 0;
  int64_t n = 0;
  for (auto& r : *c->prof) {
    if (r.kid != kid) continue;
    if (hipEventSynchronize(r.b) != hipSuccess) return REVFFN_EHIP;
    float t = 0.f;
    if (hipEventElapsedTime(&t, r.a, r.b) != hipSuccess) return REVFFN_EHIP;
    ms += t; fl += r.flops; by += r.bytes; n++;
  }
  if (ms_total) *ms_total = ms;
  if (launches) *launches = n;
  if (flops) *flops = fl;
  if (bytes) *bytes = by;
  return 0;
}

const char* revffn_profile_kernel_name(int32_t kid) {
  return (kid >= 0 && kid < KID_COUNT) ? kid_names[kid] : nullptr;
}

int revffn_set_inv_iters(revffn_ctx* c, int32_t n) {
  if (!c) return REVFFN_ENULL;
  if (n < 0 || n > 1024) return REVFFN_EINVAL;
  c->cfg.n_inv_iters = n;
  return 0;
}
int revffn_set_inverse_tolerance_blocked(revffn_ctx* c, float tol, int32_t max_iters, int32_t block_positions) {
  if (!c) return REVFFN_ENULL;
  if (!(tol >= 0.f) || (tol > 0.f && (max_iters < 1 || max_iters > 1024)) || block_positions < 0) return REVFFN_EINVAL;
  if (hipDeviceSynchronize() != hipSuccess) return REVFFN_EHIP;            // earlier inverses still update the statistics
  if (hipMemset(c->conv.stats, 0, 4 * sizeof(int)) != hipSuccess) return REVFFN_EHIP;
  c->inv_tol = tol;
  c->inv_max_iters = tol > 0.f ? max_iters : 0;
  c->inv_block = tol > 0.f ? block_positions : 0;
  c->conv_last_nblk = 0;
  return 0;
}
int revffn_set_inverse_tolerance(revffn_ctx* c, float tol, int32_t max_iters) {
  return revffn_set_inverse_tolerance_blocked(c, tol, max_iters, 0);
}
int revffn_get_inverse_stats(revffn_ctx* c, int64_t* calls, int64_t* iters_total, int32_t* last_iters,
                             float* last_residual) {
  if (!c) return REVFFN_ENULL;
  int st[4] = {0, 0, 0, 0};
  if (c->inv_tol > 0.f) {
    if (hipDeviceSynchronize() != hipSuccess) return REVFFN_EHIP;
    if (hipMemcpy(st, c->conv.stats, sizeof(st), hipMemcpyDeviceToHost) != hipSuccess) return REVFFN_EHIP;
  }
  float r;
  memcpy(&r, &st[3], sizeof(r));
  if (calls) *calls = st[0];
  if (iters_total) *iters_total = st[1];
  if (last_iters) *last_iters = st[2];
  if (last_residual) *last_residual = r;
  return 0;
}
int revffn_get_inverse_blocks(revffn_ctx* c, int32_t* iters, float* residuals, int32_t cap, int32_t* n_blocks) {
  if (!c) return REVFFN_ENULL;
  if (cap < 0) return REVFFN_EINVAL;
  const int n = c->inv_tol > 0.f ? c->conv_last_nblk : 0;
  if (n_blocks) *n_blocks = n;
  const int m = n < cap ? n : cap;
  if (m == 0) return 0;
  if (hipDeviceSynchronize() != hipSuccess) return REVFFN_EHIP;
  if (iters && hipMemcpy(iters, c->conv.blk_iters, (size_t)m * 4, hipMemcpyDeviceToHost) != hipSuccess) return REVFFN_EHIP;
  if (residuals && hipMemcpy(residuals, c->conv.blk_res, (size_t)m * 4, hipMemcpyDeviceToHost) != hipSuccess) return REVFFN_EHIP;
  return 0;
}
int revffn_enable_taps(revffn_ctx* c, int32_t on) {
  if (!c) return REVFFN_ENULL;
  c->taps = on ? 1 : 0;
  return 0;
}
int revffn_set_kernel_mode(revffn_ctx* c, int32_t mode) {
  if (!c) return REVFFN_ENULL;
  if (mode != 0 && mode != 1) return REVFFN_EINVAL;
  c->mode = mode;
  return 0;
}

int revffn_op_tile_placement(int32_t group_mode, int32_t tiles_m, int32_t tiles_n, int32_t bm, int32_t bn,
                             int32_t n_groups, const int32_t* tile_first, int32_t n_used, int32_t* out,
                             int32_t max_wg) {
  if (group_mode < 0 || group_mode > 2 || tiles_m < 1 || tiles_n < 1 || bm < 1 || bn < 1 || !out) return REVFFN_EINVAL;
  if (group_mode == 1 && (n_used < 0 || n_used > tiles_m)) return REVFFN_EINVAL;
  if (group_mode == 2 && n_groups < 1) return REVFFN_EINVAL;
  int xcd_m = 1;
  long long grid;
  if (group_mode == 0) { xcd_m = pick_xcd_m(tiles_m, tiles_n, bm, bn); grid = dense_grid_x(xcd_m, tiles_m, tiles_n); }
  else if (group_mode == 1) grid = (long long)tiles_n * tiles_m;
  else { xcd_m = 2; grid = wgrad_grid_x(xcd_m, tiles_m, tiles_n, n_groups); }
  if (grid > max_wg) return REVFFN_EINVAL;
  for (int i = 0; i < (int)grid; i++) {
    int bx = -1, by = -1, bz = 0;
    if (!place_tile(group_mode, xcd_m, tiles_m, tiles_n, n_groups, n_used, tile_first, i, &bx, &by, &bz)) bx = by = bz = -1;
    out[3 * i] = bx; out[3 * i + 1] = by; out[3 * i + 2] = bz;
  }
  return (int)grid;
}

int revffn_set_helper_streams(revffn_ctx* c, int32_t on) {
  if (!c) return REVFFN_ENULL;
  c->use_streams = on != 0;
  return 0;
}

int revffn_forward(revffn_ctx* c, const revffn_weights* w, const void* x1, const void* x2, void* y1, void* y2,
                   int32_t B, int32_t S, int64_t ld, void* stream) {
  TRY(check_call(c, w, B, S, ld));
  if (!x1 || !x2 || !y1 || !y2) return REVFFN_ENULL;
  TRY(finish(c, (hipStream_t)stream, forward_impl(c, w, x1, x2, y1, y2, B, S, ld, (hipStream_t)stream)));
  if (x1 != y1 && x2 != y2) { c->fwd_x1 = x1; c->fwd_x2 = x2; c->fwd_y1 = y1; c->fwd_B = B; c->fwd_S = S; c->fwd_ld = ld; }
  return 0;
}

int revffn_backward_stored(revffn_ctx* c, const revffn_weights* w, const void* x1, const void* x2, const void* y1,
                           const void* dy1, const void* dy2, void* dx1, void* dx2, const revffn_grads* g, int32_t B,
                           int32_t S, int64_t ld, void* stream) {
  if (!c) return REVFFN_ENULL;
  const bool match = c->fwd_x1 && c->fwd_x1 == x1 && c->fwd_x2 == x2 && c->fwd_y1 == y1 && c->fwd_B == B &&
                     c->fwd_S == S && c->fwd_ld == ld;
  TRY(check_call(c, w, B, S, ld));        // (also drops the stored state: it serves one backward call)
  if (!x1 || !x2 || !y1 || !dy1 || !dy2 || !dx1 || !dx2) return REVFFN_ENULL;
  if (!match) return REVFFN_EINVAL;
  if (dx1 == x1 || dx1 == x2 || dx2 == x1 || dx2 == x2 || dx1 == y1 || dx2 == y1) return REVFFN_EINVAL;
  return finish(c, (hipStream_t)stream,
                backward_impl(c, w, x1, x2, y1, ld, dy1, dy2, dx1, dx2, g, B, S, ld, true, true, (hipStream_t)stream, true));
}

int revffn_inverse(revffn_ctx* c, const revffn_weights* w, const void* y1, const void* y2, void* x1, void* x2,
                   int32_t B, int32_t S, int64_t ld, float* residual, void* stream) {
  TRY(check_call(c, w, B, S, ld));
  if (!x1 || !x2 || !y1 || !y2) return REVFFN_ENULL;
  return finish(c, (hipStream_t)stream,
                inverse_impl(c, w, y1, y2, x1, x2, B, S, ld, residual, (hipStream_t)stream, nullptr, nullptr));
}

int revffn_backward(revffn_ctx* c, const revffn_weights* w, const void* x1, const void* x2, const void* y1,
                    const void* dy1, const void* dy2, void* dx1, void* dx2, const revffn_grads* g, int32_t B,
                    int32_t S, int64_t ld, void* stream) {
  TRY(check_call(c, w, B, S, ld));
  if (!x1 || !x2 || !dy1 || !dy2 || !dx1 || !dx2) return REVFFN_ENULL;
  return finish(c, (hipStream_t)stream,
                backward_impl(c, w, x1, x2, y1, ld, dy1, dy2, dx1, dx2, g, B, S, ld, false, false, (hipStream_t)stream));
}

int revffn_inverse_backward(revffn_ctx* c, const revffn_weights* w, const void* y1, const void* y2, void* x1, void* x2,
                            const void* dy1, const void* dy2, void* dx1, void* dx2, const revffn_grads* g, int32_t B,
                            int32_t S, int64_t ld, float* residual, void* stream) {
  TRY(check_call(c, w, B, S, ld));
  if (!y1 || !y2 || !x1 || !x2 || !dy1 || !dy2 || !dx1 || !dx2) return REVFFN_ENULL;
  hipStream_t s = (hipStream_t)stream;
  const void* y1k = nullptr;
  i64 ldk = 0;
  hipStream_t sa = s;                     // the stream the inverse leaves X1^ on (helper stream 1 beside the MoE backward pass)
  TRY(finish(c, s, inverse_impl(c, w, y1, y2, x1, x2, B, S, ld, residual, s, &y1k, &ldk, c->side[1], &sa)));
  return finish(c, s, backward_impl(c, w, x1, x2, y1k, ldk, dy1, dy2, dx1, dx2, g, B, S, ld, true, c->cfg.n_inv_iters >= 1, s,
                                    false, sa == s ? nullptr : sa));
}

int revffn_merge_adapters(revffn_ctx* c, const revffn_weights* w, const revffn_merged* m, void* stream) {
  TRY(check_call(c, w, 1, 1, c ? c->cfg.d_model / 2 : 0));
  TRY(check_merged(c, m));
  return finish(c, (hipStream_t)stream, merge_impl(c, w, m, (hipStream_t)stream));
}

int revffn_forward_merged(revffn_ctx* c, const revffn_weights* w, const revffn_merged* m, const void* x1, const void* x2,
                          void* y1, void* y2, int32_t B, int32_t S, int64_t ld, void* stream) {
  TRY(check_call(c, w, B, S, ld, FORK_PAYS_MERGED));
  TRY(check_merged(c, m));
  if (!x1 || !x2 || !y1 || !y2) return REVFFN_ENULL;
  hipStream_t s = (hipStream_t)stream;
  const int T = B * S;
  TRY(finish(c, s, attn_acts_merged(c, w, m, x1, ld, x2, ld, B, S, true, s)));
  TRY(finish(c, s, attn_out_merged(c, m, x1, ld, 1.f, y1, ld, T, s)));                 // Eq. 1
  return finish(c, s, moe_merged(c, w, m, y1, ld, x2, ld, 1.f, y2, ld, T, s));         // Eq. 2
}

int revffn_inverse_merged(revffn_ctx* c, const revffn_weights* w, const revffn_merged* m, const void* y1, const void* y2,
                          void* x1, void* x2, int32_t B, int32_t S, int64_t ld, float* residual, void* stream) {
  TRY(check_call(c, w, B, S, ld, FORK_PAYS_MERGED));
  TRY(check_merged(c, m));
  if (!x1 || !x2 || !y1 || !y2) return REVFFN_ENULL;
  hipStream_t s = (hipStream_t)stream;
  const int T = B * S, h = c->cfg.d_model / 2, n = c->cfg.n_inv_iters;
  const void* y1k = y1;
  i64 ldk = ld;
  if (x1 == y1 && n >= 1) {               // in place: Y1 is needed after x1 starts being overwritten
    p_copy_rows(c, c->sdt, y1, ld, c->y1c, h, T, h, s);
    y1k = c->y1c;
    ldk = h;
  }
  TRY(finish(c, s, moe_merged(c, w, m, y1k, ldk, y2, ld, -1.f, x2, ld, T, s)));        // X2^ = Y2 - MoE branch(Y1)
  if (n == 0) {
    if (x1 != y1) p_copy_rows(c, c->sdt, y1, ld, x1, ld, T, h, s);
    if (residual) launch_fill_u32((uint32_t*)residual, 0, 1, s);
  }
  for (int it = 1; it <= n; it++) {
    const void* xin = (it == 1) ? y1k : x1;
    const i64 ldin = (it == 1) ? ldk : ld;
    TRY(finish(c, s, attn_acts_merged(c, w, m, xin, ldin, x2, ld, B, S, it == 1, s)));  // K, V depend on X2^ only: once
    if (it == n && residual) {
      TRY(finish(c, s, attn_out_merged(c, m, y1k, ldk, -1.f, c->xtmp, h, T, s)));
      launch_fill_u32((uint32_t*)residual, 0, 1, s);
      launch_absdiff_max_copy(c->sdt, c->xtmp, h, xin, ldin, x1, ld, residual, T, h, s);
    } else {
      TRY(finish(c, s, attn_out_merged(c, m, y1k, ldk, -1.f, x1, ld, T, s)));          // x <- Y1 - attention branch(x, X2^)
    }
  }
  return 0;
}

int revffn_stack_forward(revffn_ctx* c, const revffn_weights* w, int32_t n_blocks, const void* x1, const void* x2,
                         void* y1, void* y2, int32_t B, int32_t S, int64_t ld, void* stream) {
  if (n_blocks < 1) return REVFFN_EINVAL;
  if (!c || !w) return REVFFN_ENULL;
  for (int l = 0; l < n_blocks; l++) TRY(check_call(c, w + l, B, S, ld));
  if (!x1 || !x2 || !y1 || !y2) return REVFFN_ENULL;
  for (int l = 0; l < n_blocks; l++) {
    TRY(finish(c, (hipStream_t)stream, forward_impl(c, w + l, l == 0 ? x1 : y1, l == 0 ? x2 : y2, y1, y2, B, S, ld, (hipStream_t)stream)));
  }
  return 0;
}

int revffn_stack_backward(revffn_ctx* c, const revffn_weights* w, const revffn_grads* g, int32_t n_blocks, void* y1,
                          void* y2, void* dy1, void* dy2, int32_t B, int32_t S, int64_t ld, void* stream) {
  if (n_blocks < 1) return REVFFN_EINVAL;
  if (!c || !w) return REVFFN_ENULL;
  for (int l = 0; l < n_blocks; l++) TRY(check_call(c, w + l, B, S, ld));
  if (!y1 || !y2 || !dy1 || !dy2) return REVFFN_ENULL;
  hipStream_t s = (hipStream_t)stream;
  for (int l = n_blocks - 1; l >= 0; l--) {
    // rebuild this block's input in place; the exact Y1 survives in the workspace copy, and the MoE
    // activations computed at it by the inverse are reused by the backward pass
    const void* y1k = nullptr;
    i64 ldk = 0;
    hipStream_t sa = s;
    TRY(finish(c, s, inverse_impl(c, w + l, y1, y2, y1, y2, B, S, ld, nullptr, s, &y1k, &ldk, c->side[1], &sa)));
    TRY(finish(c, s, backward_impl(c, w + l, y1, y2, y1k, ldk, dy1, dy2, dy1, dy2, g ? g + l : nullptr, B, S, ld, true, c->cfg.n_inv_iters >= 1, s,
                                   false, sa == s ? nullptr : sa)));
  }
  return 0;
}

int revffn_get_routing(revffn_ctx* c, int32_t* idx, float* wts, int32_t* counts, int32_t* offsets, int32_t* row_map,
                       void* stream) {
  if (!c) return REVFFN_ENULL;
  if (c->lastT <= 0) return REVFFN_EINVAL;
  hipStream_t s = (hipStream_t)stream;
  const size_t N = (size_t)c->lastT * c->cfg.top_k, E = c->cfg.n_experts;
  hipError_t e = hipSuccess;
  if (idx && e == hipSuccess) e = hipMemcpyAsync(idx, c->idx, N * 4, hipMemcpyDeviceToDevice, s);
  if (wts && e == hipSuccess) e = hipMemcpyAsync(wts, c->wts, N * 4, hipMemcpyDeviceToDevice, s);
  if (counts && e == hipSuccess) e = hipMemcpyAsync(counts, c->counts, E * 4, hipMemcpyDeviceToDevice, s);
  if (offsets && e == hipSuccess) e = hipMemcpyAsync(offsets, c->offsets, (E + 1) * 4, hipMemcpyDeviceToDevice, s);
  if (row_map && e == hipSuccess) e = hipMemcpyAsync(row_map, c->row_map, N * 4, hipMemcpyDeviceToDevice, s);
  return e == hipSuccess ? 0 : REVFFN_EHIP;
}

int revffn_get_branch(revffn_ctx* c, int32_t which, float* dst, void* stream) {
  if (!c || !dst) return REVFFN_ENULL;
  if (!c->taps || c->lastT <= 0 || (which != 0 && which != 1)) return REVFFN_EINVAL;
  size_t bytes = (size_t)c->lastT * (c->cfg.d_model / 2) * 4;
  hipError_t e = hipMemcpyAsync(dst, which == 0 ? c->tapA : c->tapM, bytes, hipMemcpyDeviceToDevice, (hipStream_t)stream);
  return e == hipSuccess ? 0 : REVFFN_EHIP;
}

int revffn_op_gemm(int32_t dtype, int32_t kernel_mode, const void* a, const void* b, void* c, int32_t M, int32_t N,
                   int32_t K, int64_t lda, int64_t ldb, int64_t ldc, int32_t a_trans, int32_t b_trans,
                   int32_t out_f32, void* stream) {
  const int tile = kernel_mode >> 8;       // bits 8 and up: MFMA tile shape to force (1..4), 0 = chosen by size
  kernel_mode &= 0xff;
  if ((dtype != 0 && dtype != 1) || kernel_mode < 0 || kernel_mode > 2 || tile < 0 || tile > 4 || !a || !b || !c ||
      M < 1 || N < 1 || K < 0)
    return REVFFN_EINVAL;
  GemmArgs g = nt(a, lda, b, ldb, c, ldc, M, N, K);
  g.force_tile = tile;
  g.few_rows = gemm_few_rows(M, N);
  g.a_trans = a_trans ? 1 : 0;
  g.b_trans = b_trans ? 1 : 0;
  GemmTypes t{dtype, dtype, out_f32 ? 0 : dtype, dtype};
  if (dtype == 1 && kernel_mode != 1 && launch_gemm_mfma(g, t, (hipStream_t)stream) == 0) return 0;
  if (kernel_mode == 2) return REVFFN_EUNSUPPORTED;
  return launch_gemm_generic(g, t, (hipStream_t)stream) == 0 ? 0 : REVFFN_EUNSUPPORTED;
}

int revffn_op_attention_fwd(int32_t dtype, int32_t kernel_mode, const void* q, const void* k, const void* v, void* o,
                            float* lse, int32_t B, int32_t S, int32_t H, int32_t dh, int32_t causal, void* stream) {
  if ((dtype != 0 && dtype != 1) || kernel_mode < 0 || kernel_mode > 2 || !q || !k || !v || !o || !lse || B < 1 ||
      S < 1 || H < 1 || dh < 2 || dh > 1024)
    return REVFFN_EINVAL;
  hipStream_t s = (hipStream_t)stream;
  if (dtype == 1 && kernel_mode != 1 && launch_attn_fwd_flash(q, k, v, o, lse, B, S, H, dh, causal, s) == 0) return 0;
  if (kernel_mode == 2) return REVFFN_EUNSUPPORTED;
  launch_attn_fwd_generic(dtype, q, k, v, o, lse, B, S, H, dh, causal, s);
  return 0;
}

int revffn_op_attention_bwd(int32_t dtype, int32_t kernel_mode, const void* q, const void* k, const void* v,
                            const void* o, const void* d_o, const float* lse, float* dvec, void* dq, void* dk, void* dv,
                            int32_t B, int32_t S, int32_t H, int32_t dh, int32_t causal, void* stream) {
  if ((dtype != 0 && dtype != 1) || kernel_mode < 0 || kernel_mode > 2 || !q || !k || !v || !o || !d_o || !lse ||
      !dvec || !dq || !dk || !dv || B < 1 || S < 1 || H < 1 || dh < 2 || dh > 1024)
    return REVFFN_EINVAL;
  hipStream_t s = (hipStream_t)stream;
  if (dtype == 1 && kernel_mode != 1 &&
      launch_attn_bwd_flash(q, k, v, o, d_o, lse, dvec, dq, dk, dv, B, S, H, dh, causal, s) == 0)
    return 0;
  if (kernel_mode == 2) return REVFFN_EUNSUPPORTED;
  launch_attn_bwd_generic(dtype, q, k, v, o, d_o, lse, dvec, dq, dk, dv, B, S, H, dh, causal, s);
  return 0;
}

// ---- the entry point that allocates nothing -----------------------------------------------------------------
// The row-dot scratch of the attention backward (D[b, head, s] = <dO, O>, float) lives in a file-scope device array
// instead of a caller buffer.  In host code the array's name is only a handle: the device address is looked up once
// per device with hipGetSymbolAddress and kept, and only that pointer is ever handed to a kernel.
#define REVFFN_NOALLOC_MAX_ROWS (1 << 20)
static __device__ __align__(256) float scratch[REVFFN_NOALLOC_MAX_ROWS];
#define REVFFN_MAX_DEVICES 64
static float* scratch_ptr[REVFFN_MAX_DEVICES];          // per device: address of that device's copy of `scratch`
static std::mutex scratch_mu;

int revffn_op_attention_bwd_noalloc(int32_t dtype, int32_t kernel_mode, const void* q, const void* k, const void* v,
                                    const void* o, const void* d_o, const float* lse, void* dq, void* dk, void* dv,
                                    int32_t B, int32_t S, int32_t H, int32_t dh, int32_t causal, void* stream) {
  if ((dtype != 0 && dtype != 1) || kernel_mode < 0 || kernel_mode > 2 || !q || !k || !v || !o || !d_o || !lse ||
      !dq || !dk || !dv || B < 1 || S < 1 || H < 1 || dh < 2 || dh > 1024)
    return REVFFN_EINVAL;
  if ((long long)B * H * S > REVFFN_NOALLOC_MAX_ROWS) return REVFFN_ESHAPE;   // beyond the static scratch
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess) return REVFFN_EHIP;
  if (dev < 0 || dev >= REVFFN_MAX_DEVICES) return REVFFN_EUNSUPPORTED;
  float* dvec;
  {
    std::lock_guard<std::mutex> lock(scratch_mu);
    if (!scratch_ptr[dev]) {
      void* p = nullptr;
      if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) { (void)hipGetLastError(); return REVFFN_EHIP; }
      scratch_ptr[dev] = (float*)p;
    }
    dvec = scratch_ptr[dev];
  }
  // every element of dvec that the kernels read is written first by the row-dot kernel of the same call, so nothing
  // of an earlier call's contents needs clearing
  return revffn_op_attention_bwd(dtype, kernel_mode, q, k, v, o, d_o, lse, dvec, dq, dk, dv, B, S, H, dh, causal, stream);
}

const char* revffn_strerror(int code) {
  switch (code) {
    case REVFFN_OK: return "ok";
    case REVFFN_EINVAL: return "invalid configuration value";
    case REVFFN_ESHAPE: return "batch, sequence length or row stride out of range for this context";
    case REVFFN_ENULL: return "required pointer is NULL";
    case REVFFN_EWORKSPACE: return "workspace allocation failed";
    case REVFFN_EHIP: return "HIP runtime call failed";
    case REVFFN_EUNSUPPORTED: return "request not implemented by this build";
    default: return "unknown error";
  }
}

}  // extern "C"
