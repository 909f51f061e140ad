// Memory-bound kernels of the RevFFN block: RMSNorm (Norm of Eq. 1-2) forward and
// backward, rotary encoding, SwiGLU, row gathers/copies, deterministic column sums.
#include "kernels.h"
#include <initializer_list>

#define DISPATCH_DT(dt, ...)                                  \
  do {                                                        \
    if ((dt) == 0) { typedef float T; __VA_ARGS__; }          \
    else { typedef bf16 T; __VA_ARGS__; }                     \
  } while (0)

// element types of gains and results and of the rows, and columns per lane, of the norm kernels
#define BY_NORM_TYPES(call)                                       \
  do {                                                            \
    if (dt == 0) call(float, float, 1);                           \
    else if (tx == 0) { if (h & 7) call(bf16, float, 1); else call(bf16, float, 8); } \
    else if (h & 7) call(bf16, bf16, 1);                          \
    else call(bf16, bf16, 8);                                     \
  } while (0)

// ---------------------------------------------------------------------------------
// RMSNorm forward: one wave per token row.
// ---------------------------------------------------------------------------------
// (blockIdx.y == 1: the second problem of the launch, same shape: x2, g2, out2)
// A lane takes V neighbouring columns at a time: 8 in bf16 rows of whole groups of 8, the order in which the form with 16-byte
// accesses below adds, so that the result does not depend on the rows' addresses; else 1.
template <class T, class TX, int V>
__global__ void __launch_bounds__(256) rmsnorm_fwd_k(const TX* __restrict__ x, i64 ldx, const T* __restrict__ g,
                                                     T* __restrict__ out, i64 ldo, int rows, int h, float eps,
                                                     const unsigned char* __restrict__ row_skip,
                                                     const TX* __restrict__ x2, const T* __restrict__ g2, T* __restrict__ out2) {
  int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  int lane = threadIdx.x & 63;
  if (row >= rows || (row_skip && row_skip[row])) return;
  if (blockIdx.y) { x = x2; g = g2; out = out2; }
  const TX* xr = x + (i64)row * ldx;
  float ss = 0.f;
  for (int j0 = lane * V; j0 < h; j0 += 64 * V)
#pragma unroll
    for (int j = j0; j < j0 + V; j++) { float v = to_f(xr[j]); ss += v * v; }
  ss = wave_sum(ss);
  float r = 1.0f / sqrtf(ss / (float)h + eps);
  T* orow = out + (i64)row * ldo;
  for (int j = lane; j < h; j += 64) orow[j] = from_f<T>(to_f(xr[j]) * r * to_f(g[j]));
}

// bf16 rows of h % 8 == 0 elements at 16-byte aligned addresses: 16-byte accesses, 8 elements per lane
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_v;
static bool rows_vec8(int dt, int h, std::initializer_list<const void*> ptrs, std::initializer_list<i64> lds) {
  if (dt != 1 || (h & 7)) return false;
  for (const void* q : ptrs) if ((uintptr_t)q & 15) return false;
  for (i64 l : lds) if (l & 7) return false;
  return true;
}
// 8 consecutive elements of a bf16 or float32 row as floats (float32 rows: two 16-byte loads; p 16-byte aligned)
struct f32x8 { float v[8]; };
__device__ __forceinline__ f32x8 load8(const bf16* p) {
  const bf16x8_v t = *(const bf16x8_v*)p;
  f32x8 o;
#pragma unroll
  for (int q = 0; q < 8; q++) o.v[q] = (float)t[q];
  return o;
}
__device__ __forceinline__ f32x8 load8(const float* p) {
  const float4 a = *(const float4*)p, b = *(const float4*)(p + 4);
  return f32x8{{a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w}};
}
template <class TX>
__global__ void __launch_bounds__(256) rmsnorm_fwd_v8_k(const TX* __restrict__ x, i64 ldx, const bf16* __restrict__ g,
                                                        bf16* __restrict__ out, i64 ldo, int rows, int h, float eps,
                                                        const unsigned char* __restrict__ row_skip,
                                                        const TX* __restrict__ x2, const bf16* __restrict__ g2,
                                                        bf16* __restrict__ out2) {
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (row >= rows || (row_skip && row_skip[row])) return;
  if (blockIdx.y) { x = x2; g = g2; out = out2; }
  const TX* xr = x + (i64)row * ldx;
  float ss = 0.f;
  for (int j = lane * 8; j < h; j += 512) {
    const f32x8 v = load8(xr + j);
#pragma unroll
    for (int q = 0; q < 8; q++) ss += v.v[q] * v.v[q];
  }
  ss = wave_sum(ss);
  const float r = 1.0f / sqrtf(ss / (float)h + eps);
  bf16* orow = out + (i64)row * ldo;
  for (int j = lane * 8; j < h; j += 512) {
    const f32x8 v = load8(xr + j);
    const bf16x8_v gv = *(const bf16x8_v*)(g + j);
    bf16x8_v o;
#pragma unroll
    for (int q = 0; q < 8; q++) o[q] = (__bf16)(v.v[q] * r * (float)gv[q]);
    *(bf16x8_v*)(orow + j) = o;
  }
}

void launch_rmsnorm_fwd(int dt, int tx, const void* x, i64 ldx, const void* g, void* out, i64 ldo, int rows, int h,
                        float eps, hipStream_t s, const unsigned char* row_skip, const void* x2, const void* g2,
                        void* out2) {
  if (rows <= 0) return;
  const dim3 grid(cdiv(rows, 4), x2 ? 2 : 1), block(256);
  if (rows_vec8(dt, h, {x, g, out, x2, g2, out2}, {ldx, ldo})) {
    if (tx == 0)
      hipLaunchKernelGGL(rmsnorm_fwd_v8_k<float>, grid, block, 0, s, (const float*)x, ldx, (const bf16*)g, (bf16*)out,
                         ldo, rows, h, eps, row_skip, (const float*)x2, (const bf16*)g2, (bf16*)out2);
    else
      hipLaunchKernelGGL(rmsnorm_fwd_v8_k<bf16>, grid, block, 0, s, (const bf16*)x, ldx, (const bf16*)g, (bf16*)out,
                         ldo, rows, h, eps, row_skip, (const bf16*)x2, (const bf16*)g2, (bf16*)out2);
    return;
  }
#define NORM_FWD(T, TX, V) hipLaunchKernelGGL((rmsnorm_fwd_k<T, TX, V>), grid, block, 0, s, (const TX*)x, ldx, (const T*)g, (T*)out, \
                                              ldo, rows, h, eps, row_skip, (const TX*)x2, (const T*)g2, (T*)out2)
  BY_NORM_TYPES(NORM_FWD);
}

// RMSNorm backward for the input:  dx = r*(g.dy) - x*r^3*mean_j(x_j g_j dy_j), plus an
// optional base term (the residual path of Eq. 1-2).  1/rms is kept per row.
// (blockIdx.y == 1: the second problem of the launch, same rows, width and strides but for the base's; V as above)
template <class T, class TX, int V>
__global__ void __launch_bounds__(256) rmsnorm_bwd_k(NormBwd p, NormBwd p2, i64 ldd, i64 ldx, i64 ldo, int rows, int h, float eps) {
  int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  int lane = threadIdx.x & 63;
  if (row >= rows) return;
  if (blockIdx.y) p = p2;
  const TX* xr = (const TX*)p.x + (i64)row * ldx;
  const T* dr = (const T*)p.dy + (i64)row * ldd;
  const T *g = (const T*)p.g, *base = (const T*)p.base;
  T* dx = (T*)p.dx;
  float ss = 0.f, sd = 0.f;
  for (int j0 = lane * V; j0 < h; j0 += 64 * V)
#pragma unroll
    for (int j = j0; j < j0 + V; j++) {
      float v = to_f(xr[j]);
      ss += v * v;
      sd += v * to_f(g[j]) * to_f(dr[j]);
    }
  ss = wave_sum(ss);
  sd = wave_sum(sd);
  float r = 1.0f / sqrtf(ss / (float)h + eps);
  float c = r * r * r * sd / (float)h;
  if (lane == 0) p.rinv[row] = r;
  for (int j = lane; j < h; j += 64) {
    float v = r * to_f(g[j]) * to_f(dr[j]) - to_f(xr[j]) * c;
    if (base) v += to_f(base[(i64)row * p.ldb + j]);
    dx[(i64)row * ldo + j] = from_f<T>(v);
  }
}

template <class TX>
__global__ void __launch_bounds__(256) rmsnorm_bwd_v8_k(NormBwd p, NormBwd p2, i64 ldd, i64 ldx, i64 ldo, int rows, int h, float eps) {
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (row >= rows) return;
  if (blockIdx.y) p = p2;
  const TX* xr = (const TX*)p.x + (i64)row * ldx;
  const bf16* dr = (const bf16*)p.dy + (i64)row * ldd;
  const bf16 *g = (const bf16*)p.g, *base = (const bf16*)p.base;
  bf16* dx = (bf16*)p.dx;
  float ss = 0.f, sd = 0.f;
  for (int j = lane * 8; j < h; j += 512) {
    const f32x8 v = load8(xr + j);
    const bf16x8_v gv = *(const bf16x8_v*)(g + j), d = *(const bf16x8_v*)(dr + j);
#pragma unroll
    for (int q = 0; q < 8; q++) { ss += v.v[q] * v.v[q]; sd += v.v[q] * (float)gv[q] * (float)d[q]; }
  }
  ss = wave_sum(ss);
  sd = wave_sum(sd);
  const float r = 1.0f / sqrtf(ss / (float)h + eps);
  const float c = r * r * r * sd / (float)h;
  if (lane == 0) p.rinv[row] = r;
  for (int j = lane * 8; j < h; j += 512) {
    // (dx may alias base or dy: every lane reads its 8 elements of all inputs before it writes them)
    const f32x8 v = load8(xr + j);
    const bf16x8_v gv = *(const bf16x8_v*)(g + j), d = *(const bf16x8_v*)(dr + j);
    bf16x8_v b;
    if (base) b = *(const bf16x8_v*)(base + (i64)row * p.ldb + j);
    bf16x8_v o;
#pragma unroll
    for (int q = 0; q < 8; q++) {
      float t = r * (float)gv[q] * (float)d[q] - v.v[q] * c;
      if (base) t += (float)b[q];
      o[q] = (__bf16)t;
    }
    *(bf16x8_v*)(dx + (i64)row * ldo + j) = o;
  }
}

void launch_rmsnorm_bwd(int dt, int tx, const NormBwd& p, const NormBwd* p2, i64 ldd, i64 ldx, i64 ldo, int rows, int h, float eps,
                        hipStream_t s) {
  if (rows <= 0) return;
  const dim3 grid(cdiv(rows, 4), p2 ? 2 : 1), block(256);
  const NormBwd q = p2 ? *p2 : p;
  if (rows_vec8(dt, h, {p.dy, p.x, p.g, p.base, p.dx, q.dy, q.x, q.g, q.base, q.dx}, {ldd, ldx, p.ldb, q.ldb, ldo})) {
    if (tx == 0) hipLaunchKernelGGL(rmsnorm_bwd_v8_k<float>, grid, block, 0, s, p, q, ldd, ldx, ldo, rows, h, eps);
    else hipLaunchKernelGGL(rmsnorm_bwd_v8_k<bf16>, grid, block, 0, s, p, q, ldd, ldx, ldo, rows, h, eps);
    return;
  }
#define NORM_BWD(T, TX, V) hipLaunchKernelGGL((rmsnorm_bwd_k<T, TX, V>), grid, block, 0, s, p, q, ldd, ldx, ldo, rows, h, eps)
  BY_NORM_TYPES(NORM_BWD);
}

// ---------------------------------------------------------------------------------
// Deterministic column sums (gain, bias and router-bias gradients), all of a call in one launch.  A workgroup adds one
// chunk of rows of 256 columns (a thread owns 8 adjacent columns and every 8th row) and leaves the chunk's sums in
// `partial`; the last workgroup of those columns to finish, told by a ticket, adds the chunks in index order, so the
// result does not depend on which one that is.  Latency-bound (8-25 MB in all): one launch instead of four pairs.
// ---------------------------------------------------------------------------------
#define COLSUM_CHUNKS 32
__host__ __device__ inline int colsum_chunk_rows(int rows) { const int c = (rows + COLSUM_CHUNKS - 1) / COLSUM_CHUNKS; return c < 32 ? 32 : c; }
size_t colsum_tickets(size_t cols_sum) { return (cols_sum + 255) / 256 + COLSUM_MAX; }
size_t colsum_partial_floats(size_t cols_sum) { return colsum_tickets(cols_sum) * (COLSUM_CHUNKS + 1) * 256; }

// 8 consecutive elements from column c on, of which those below cols exist; vec: all 8 at once
__device__ __forceinline__ f32x8 colsum_load(const void* p, bool f32, i64 off, int n, bool vec) {
  f32x8 o;
  if (vec) return f32 ? load8((const float*)p + off) : load8((const bf16*)p + off);
#pragma unroll
  for (int i = 0; i < 8; i++) o.v[i] = i < n ? (f32 ? ((const float*)p)[off + i] : (float)((const bf16*)p)[off + i]) : 0.f;
  return o;
}
__global__ void __launch_bounds__(256) colsum_k(ColsumBatch q, float* __restrict__ partial_all, int* __restrict__ ticket) {
  __shared__ float red[8][256];
  __shared__ int last;
  int z = 0;
#pragma unroll
  for (int i = 1; i < COLSUM_MAX; i++) if (i < q.n && (int)blockIdx.x >= q.p[i].tile0) z = i;
  Colsum p = q.p[0];
#pragma unroll
  for (int i = 1; i < COLSUM_MAX; i++) if (z == i) p = q.p[i];     // (constant indices: no copy of the arguments)
  const int chunk = colsum_chunk_rows(p.rows), chunks = (p.rows + chunk - 1) / chunk;
  if ((int)blockIdx.y >= chunks) return;
  float* partial = partial_all + (i64)blockIdx.x * (COLSUM_CHUNKS + 1) * 256;
  const int cg = threadIdx.x & 31, qd = threadIdx.x >> 5;
  const int c0 = ((int)blockIdx.x - p.tile0) * 256, c = c0 + cg * 8;
  const int r0 = blockIdx.y * chunk, r1 = min(p.rows, r0 + chunk);
  const int n = min(8, p.cols - c);
  const bool va = n == 8 && (p.lda & 7) == 0 && ((uintptr_t)p.a & 15) == 0, vb = n == 8 && (p.ldb & 7) == 0 && ((uintptr_t)p.b & 15) == 0;
  float acc[8];
#pragma unroll
  for (int i = 0; i < 8; i++) acc[i] = 0.f;
  if (n > 0) {
#pragma unroll 4
    for (int t = r0 + qd; t < r1; t += 8) {
      const f32x8 av = colsum_load(p.a, p.a_f32, (i64)t * p.lda + c, n, va);
      const float w = p.sc ? p.sc[t] : 1.f;
      if (p.b) {
        const f32x8 bv = colsum_load(p.b, p.b_f32, (i64)t * p.ldb + c, n, vb);
#pragma unroll
        for (int i = 0; i < 8; i++) acc[i] += av.v[i] * bv.v[i] * w;
      } else {
#pragma unroll
        for (int i = 0; i < 8; i++) acc[i] += av.v[i] * w;
      }
    }
  }
#pragma unroll
  for (int i = 0; i < 8; i++) red[qd][cg * 8 + i] = acc[i];
  __syncthreads();
  float v = 0.f;
#pragma unroll
  for (int j = 0; j < 8; j++) v += red[j][threadIdx.x];
  if (chunks > 1) {
    // Agent scope: the other chunks' workgroups may run on other XCDs.  What orders the sums before the ticket is not the
    // memory model, which would ask for a release here and an acquire below, but this chip: an agent-scope store is written
    // through to where every XCD reads it, s_waitcnt vmcnt(0) returns when that has happened, the barrier makes it so for
    // all four waves, and agent-scope loads do not read the caches of their own XCD.  (The release writes the whole L2
    // back in every workgroup: 151 us instead of 9 at T = 2048.)
#if defined(__HIP_DEVICE_COMPILE__) && !defined(__gfx950__)
#error "the ticket below rests on how gfx950 carries out agent-scope stores"
#endif
    __hip_atomic_store(partial + (i64)blockIdx.y * 256 + threadIdx.x, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) last = __hip_atomic_fetch_add(ticket + blockIdx.x, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == chunks - 1;
    __syncthreads();
    if (!last) return;
    v = 0.f;
#pragma unroll 8
    for (int i = 0; i < chunks; i++) v += __hip_atomic_load(partial + (i64)i * 256 + threadIdx.x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (threadIdx.x == 0) __hip_atomic_store(ticket + blockIdx.x, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (c0 + (int)threadIdx.x < p.cols) {
    if (p.out_f32) ((float*)p.out)[c0 + threadIdx.x] = v;
    else ((bf16*)p.out)[c0 + threadIdx.x] = (bf16)v;
  }
}
void launch_colsum_batch(ColsumBatch& q, float* partial, int* ticket, hipStream_t s) {
  int tiles = 0, chunks = 1;
  for (int i = 0; i < q.n; i++) {
    q.p[i].tile0 = tiles;
    tiles += cdiv(q.p[i].cols, 256);
    const int ch = cdiv(q.p[i].rows, colsum_chunk_rows(q.p[i].rows));
    if (ch > chunks) chunks = ch;
  }
  if (tiles > 0) hipLaunchKernelGGL(colsum_k, dim3(tiles, chunks), dim3(256), 0, s, q, partial, ticket);
}

// ---------------------------------------------------------------------------------
// Rotary encoding in place on buf[T, H*dh]; half-split pairing (i, i+dh/2); the angle of
// pair i at sequence position s comes from a host-built table cs[s][i] = (cos, sin).
// sign = -1 applies the inverse rotation (the backward of the forward rotation).
// ---------------------------------------------------------------------------------
template <class T>
__global__ void __launch_bounds__(256) rope_k(T* __restrict__ buf, T* __restrict__ buf2, const float2* __restrict__ cs,
                                              i64 total, int S, int H, int half, float sign,
                                              const unsigned char* __restrict__ row_skip) {
  i64 e = (i64)blockIdx.x * 256 + threadIdx.x;
  if (e >= total) return;
  if (blockIdx.y) buf = buf2;                // second tensor of the launch
  int i = (int)(e % half);
  i64 th = e / half;          // token*H + head
  i64 t = th / H;
  if (row_skip && row_skip[t]) return;
  int spos = (int)(t % S);
  float2 c = cs[(i64)spos * half + i];
  float sn = sign * c.y;
  T* p = buf + th * (2 * half);
  float a = to_f(p[i]), b = to_f(p[i + half]);
  p[i] = from_f<T>(a * c.x - b * sn);
  p[i + half] = from_f<T>(b * c.x + a * sn);
}

// bf16, half % 8 == 0: one lane rotates 8 consecutive pairs of one (token, head) with 16-byte accesses
__global__ void __launch_bounds__(256) rope_v8_k(bf16* __restrict__ buf, bf16* __restrict__ buf2,
                                                 const float2* __restrict__ cs, int total8, int S, int H, int half8,
                                                 float sign, const unsigned char* __restrict__ row_skip) {
  const int e = blockIdx.x * 256 + threadIdx.x;
  if (e >= total8) return;
  if (blockIdx.y) buf = buf2;                // second tensor of the launch
  const int i = (e % half8) * 8;
  const int th = e / half8;          // token*H + head
  if (row_skip && row_skip[th / H]) return;
  const int spos = (th / H) % S;
  const int half = half8 * 8;
  bf16* p = buf + (i64)th * (2 * half) + i;
  const bf16x8_v a = *(const bf16x8_v*)p, b = *(const bf16x8_v*)(p + half);
  const float2* c = cs + (i64)spos * half + i;
  bf16x8_v oa, ob;
#pragma unroll
  for (int q = 0; q < 8; q++) {
    const float2 cq = c[q];
    const float sn = sign * cq.y, av = (float)a[q], bv = (float)b[q];
    oa[q] = (__bf16)(av * cq.x - bv * sn);
    ob[q] = (__bf16)(bv * cq.x + av * sn);
  }
  *(bf16x8_v*)p = oa;
  *(bf16x8_v*)(p + half) = ob;
}

void launch_rope(int dt, void* buf, const float* cs_table, int Tn, int S, int H, int dh, float sign,
                 hipStream_t s, void* buf2, const unsigned char* row_skip) {
  i64 total = (i64)Tn * H * (dh / 2);
  if (total <= 0) return;
  const unsigned ny = buf2 ? 2 : 1;
  if (dt == 1 && (dh & 15) == 0 && (((uintptr_t)buf | (uintptr_t)buf2) & 15) == 0 && total / 8 < (i64)1 << 31) {
    hipLaunchKernelGGL(rope_v8_k, dim3(cdiv(total / 8, 256), ny), dim3(256), 0, s, (bf16*)buf, (bf16*)buf2,
                       (const float2*)cs_table, (int)(total / 8), S, H, dh / 16, sign, row_skip);
    return;
  }
  DISPATCH_DT(dt, hipLaunchKernelGGL(rope_k<T>, dim3(cdiv(total, 256), ny), dim3(256), 0, s, (T*)buf, (T*)buf2,
                                     (const float2*)cs_table, total, S, H, dh / 2, sign, row_skip));
}

// ---------------------------------------------------------------------------------
// SwiGLU: hh = silu(G) * U on gu[rows, 2I] = [G | U]; and its backward.
// ---------------------------------------------------------------------------------
template <class T>
__global__ void __launch_bounds__(256) swiglu_fwd_k(const T* __restrict__ gu, T* __restrict__ hh, i64 total, int I) {
  i64 e = (i64)blockIdx.x * 256 + threadIdx.x;
  if (e >= total) return;
  i64 r = e / I;
  int j = (int)(e % I);
  float g = to_f(gu[r * 2 * I + j]), u = to_f(gu[r * 2 * I + I + j]);
  hh[e] = from_f<T>(g * sigmoid_f(g) * u);
}
template <class T>
__global__ void __launch_bounds__(256) swiglu_bwd_k(const T* __restrict__ dhh, const T* __restrict__ gu,
                                                    T* __restrict__ dgu, i64 total, int I) {
  i64 e = (i64)blockIdx.x * 256 + threadIdx.x;
  if (e >= total) return;
  i64 r = e / I;
  int j = (int)(e % I);
  float g = to_f(gu[r * 2 * I + j]), u = to_f(gu[r * 2 * I + I + j]);
  float dg, du;
  swiglu_grad(to_f(dhh[e]), g, u, &dg, &du);
  dgu[r * 2 * I + j] = from_f<T>(dg);
  dgu[r * 2 * I + I + j] = from_f<T>(du);
}
// bf16, I % 8 == 0: one thread handles 8 consecutive columns with 16-byte accesses
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
__global__ void __launch_bounds__(256) swiglu_fwd_v8_k(const bf16* __restrict__ gu, bf16* __restrict__ hh, i64 total8,
                                                       int I8) {
  i64 e = (i64)blockIdx.x * 256 + threadIdx.x;
  if (e >= total8) return;
  i64 r = e / I8;
  int j = (int)(e % I8) * 8;
  const int I = I8 * 8;
  bf16x8_t g = *(const bf16x8_t*)(gu + r * 2 * I + j), u = *(const bf16x8_t*)(gu + r * 2 * I + I + j), o;
#pragma unroll
  for (int q = 0; q < 8; q++) { float gv = (float)g[q]; o[q] = (__bf16)(gv * sigmoid_f(gv) * (float)u[q]); }
  *(bf16x8_t*)(hh + r * I + j) = o;
}
__global__ void __launch_bounds__(256) swiglu_bwd_v8_k(const bf16* __restrict__ dhh, const bf16* __restrict__ gu,
                                                       bf16* __restrict__ dgu, i64 total8, int I8) {
  i64 e = (i64)blockIdx.x * 256 + threadIdx.x;
  if (e >= total8) return;
  i64 r = e / I8;
  int j = (int)(e % I8) * 8;
  const int I = I8 * 8;
  bf16x8_t g = *(const bf16x8_t*)(gu + r * 2 * I + j), u = *(const bf16x8_t*)(gu + r * 2 * I + I + j);
  bf16x8_t dh = *(const bf16x8_t*)(dhh + r * I + j), og, ou;
#pragma unroll
  for (int q = 0; q < 8; q++) {
    float dg, du;
    swiglu_grad((float)dh[q], (float)g[q], (float)u[q], &dg, &du);
    og[q] = (__bf16)dg;
    ou[q] = (__bf16)du;
  }
  *(bf16x8_t*)(dgu + r * 2 * I + j) = og;
  *(bf16x8_t*)(dgu + r * 2 * I + I + j) = ou;
}

void launch_swiglu_fwd(int dt, const void* gu, void* hh, i64 rows, int I, hipStream_t s) {
  i64 total = rows * I;
  if (total <= 0) return;
  if (dt == 1 && (I & 7) == 0 && (((uintptr_t)gu | (uintptr_t)hh) & 15) == 0) {
    hipLaunchKernelGGL(swiglu_fwd_v8_k, dim3(cdiv(total / 8, 256)), dim3(256), 0, s, (const bf16*)gu, (bf16*)hh,
                       total / 8, I / 8);
    return;
  }
  DISPATCH_DT(dt, hipLaunchKernelGGL(swiglu_fwd_k<T>, dim3(cdiv(total, 256)), dim3(256), 0, s, (const T*)gu,
                                     (T*)hh, total, I));
}
void launch_swiglu_bwd(int dt, const void* dhh, const void* gu, void* dgu, i64 rows, int I, hipStream_t s) {
  i64 total = rows * I;
  if (total <= 0) return;
  if (dt == 1 && (I & 7) == 0 && (((uintptr_t)gu | (uintptr_t)dhh | (uintptr_t)dgu) & 15) == 0) {
    hipLaunchKernelGGL(swiglu_bwd_v8_k, dim3(cdiv(total / 8, 256)), dim3(256), 0, s, (const bf16*)dhh,
                       (const bf16*)gu, (bf16*)dgu, total / 8, I / 8);
    return;
  }
  DISPATCH_DT(dt, hipLaunchKernelGGL(swiglu_bwd_k<T>, dim3(cdiv(total, 256)), dim3(256), 0, s, (const T*)dhh,
                                     (const T*)gu, (T*)dgu, total, I));
}

// ---------------------------------------------------------------------------------
// Strided row copy.
// ---------------------------------------------------------------------------------
template <class T>
__global__ void __launch_bounds__(256) copy_rows_k(const T* __restrict__ src, i64 lds_, T* __restrict__ dst, i64 ldd,
                                                   int rows, int cols) {
  i64 e = (i64)blockIdx.x * 256 + threadIdx.x;
  if (e >= (i64)rows * cols) return;
  i64 r = e / cols;
  int c = (int)(e % cols);
  dst[r * ldd + c] = src[r * lds_ + c];
}
void launch_copy_rows(int dt, const void* src, i64 lds_, void* dst, i64 ldd, int rows, int cols, hipStream_t s) {
  i64 total = (i64)rows * cols;
  if (total <= 0) return;
  DISPATCH_DT(dt, hipLaunchKernelGGL(copy_rows_k<T>, dim3(cdiv(total, 256)), dim3(256), 0, s, (const T*)src, lds_,
                                     (T*)dst, ldd, rows, cols));
}

template <class T>
__global__ void zero_k(T* p, int n) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = from_f<T>(0.f);
}
void launch_zero(int dt, void* p, int n, hipStream_t s) {
  if (n <= 0) return;
  DISPATCH_DT(dt, hipLaunchKernelGGL(zero_k<T>, dim3(cdiv(n, 256)), dim3(256), 0, s, (T*)p, n));
}

__global__ void fill_u32_k(uint32_t* p, uint32_t v, int n) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}
void launch_fill_u32(uint32_t* p, uint32_t v, int n, hipStream_t s) {
  if (n <= 0) return;
  hipLaunchKernelGGL(fill_u32_k, dim3(cdiv(n, 256)), dim3(256), 0, s, p, v, n);
}

// res = max |a - b| over all elements (non-negative floats compare like their bit patterns, so
// an integer atomic max is exact and order-independent); then dst = a.
template <class T>
__global__ void __launch_bounds__(256) absdiff_max_copy_k(const T* __restrict__ a, i64 lda, const T* b, i64 ldb,
                                                          T* dst, i64 ldd, float* res, int rows, int cols) {
  __shared__ float red[4];
  i64 e = (i64)blockIdx.x * 256 + threadIdx.x;
  float m = 0.f;
  if (e < (i64)rows * cols) {
    i64 r = e / cols;
    int c = (int)(e % cols);
    T av = a[r * lda + c];
    m = fabsf(to_f(av) - to_f(b[r * ldb + c]));
    dst[r * ldd + c] = av;
  }
  m = wave_max(m);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    m = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
    atomicMax((unsigned int*)res, __float_as_uint(m));
  }
}
void launch_absdiff_max_copy(int dt, const void* a, i64 lda, const void* b, i64 ldb, void* dst, i64 ldd,
                             float* res, int rows, int cols, hipStream_t s) {
  i64 total = (i64)rows * cols;
  if (total <= 0) return;
  DISPATCH_DT(dt, hipLaunchKernelGGL(absdiff_max_copy_k<T>, dim3(cdiv(total, 256)), dim3(256), 0, s, (const T*)a,
                                     lda, (const T*)b, ldb, (T*)dst, ldd, res, rows, cols));
}

// ---------------------------------------------------------------------------------
// Stopping rule of the inverse's fixed-point iteration (x <- Y1 - attention branch(x, X2^)), decided on the device.
// Each query row's iterate depends on that row alone (keys and values come from X2^, which is fixed), so a block of
// rows can stop on its own: once max |x_n - x_(n-1)| over the block is <= tol its rows are marked, and the kernels of
// later iterations leave marked rows alone.  The host enqueues max_iters iterations and never waits.
// ---------------------------------------------------------------------------------
__device__ __forceinline__ int conv_block_of(int row, int S, int bp, int nj) {
  if (bp <= 0) return 0;
  const int b = row / S;
  return b * nj + (row - b * S) / bp;
}
template <class T>
__global__ void __launch_bounds__(256) conv_update_k(const T* __restrict__ xn, i64 ldn, const T* xin, i64 ldi, T* dst,
                                                     i64 ldd, ConvState cs, int rows, int cols) {
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (row >= rows || cs.row_done[row]) return;            // whole wave
  float m = 0.f;
  for (int c = lane; c < cols; c += 64) {
    const T a = xn[(i64)row * ldn + c];
    m = fmaxf(m, fabsf(to_f(a) - to_f(xin[(i64)row * ldi + c])));   // (dst may be xin: read before the write)
    dst[(i64)row * ldd + c] = a;
  }
  // fmaxf drops a NaN operand; a row with a non-finite difference must not look converged
  for (int c = lane; c < cols; c += 64) { const float a = to_f(xn[(i64)row * ldn + c]); if (!(a == a)) m = INFINITY; }
  m = wave_max(m);
  if (lane == 0) atomicMax(cs.blk_bits + conv_block_of(row, cs.S, cs.bp, cs.nj), __float_as_uint(m));
}
__global__ void __launch_bounds__(64) conv_decide_k(ConvState cs, int rows, float tol, int it) {
  const int blk = blockIdx.x;
  if (cs.blk_done[blk]) return;
  const float res = __uint_as_float(cs.blk_bits[blk]);
  const bool done = res <= tol;
  __syncthreads();                                        // every lane has read the running maximum
  if (threadIdx.x == 0) {
    cs.blk_iters[blk] = it;
    cs.blk_res[blk] = res;
    cs.blk_bits[blk] = 0u;
    if (done) cs.blk_done[blk] = 1;
  }
  if (!done) return;
  int r0, r1;
  if (cs.bp <= 0) { r0 = 0; r1 = rows; }
  else {
    const int b = blk / cs.nj, j = blk - b * cs.nj;
    r0 = b * cs.S + j * cs.bp;
    r1 = min(b * cs.S + min(cs.S, (j + 1) * cs.bp), rows);
  }
  for (int r = r0 + (int)threadIdx.x; r < r1; r += 64) cs.row_done[r] = 1;
}
__global__ void __launch_bounds__(256) conv_finalize_k(ConvState cs, float* residual_out) {
  __shared__ unsigned rb[4];
  __shared__ int ri[4];
  unsigned bits = 0;
  int iters = 0;
  for (int b = threadIdx.x; b < cs.nblk; b += 256) {
    bits = max(bits, __float_as_uint(cs.blk_res[b]));     // residuals are non-negative (or +inf / NaN, which rank above)
    iters = max(iters, cs.blk_iters[b]);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) { bits = max(bits, (unsigned)__shfl_xor((int)bits, o, WAVE)); iters = max(iters, __shfl_xor(iters, o, WAVE)); }
  if ((threadIdx.x & 63) == 0) { rb[threadIdx.x >> 6] = bits; ri[threadIdx.x >> 6] = iters; }
  __syncthreads();
  if (threadIdx.x == 0) {
    bits = max(max(rb[0], rb[1]), max(rb[2], rb[3]));
    iters = max(max(ri[0], ri[1]), max(ri[2], ri[3]));
    if (residual_out) *residual_out = __uint_as_float(bits);
    cs.stats[0] += 1;
    cs.stats[1] += iters;
    cs.stats[2] = iters;
    cs.stats[3] = (int)bits;
  }
}
void launch_conv_update(int dt, const void* xn, i64 ldn, const void* xin, i64 ldi, void* dst, i64 ldd,
                        const ConvState& cs, int rows, int cols, hipStream_t s) {
  if (rows <= 0) return;
  DISPATCH_DT(dt, hipLaunchKernelGGL(conv_update_k<T>, dim3(cdiv(rows, 4)), dim3(256), 0, s, (const T*)xn, ldn,
                                     (const T*)xin, ldi, (T*)dst, ldd, cs, rows, cols));
}
void launch_conv_decide(const ConvState& cs, int rows, float tol, int it, hipStream_t s) {
  hipLaunchKernelGGL(conv_decide_k, dim3(cs.nblk), dim3(64), 0, s, cs, rows, tol, it);
}
void launch_conv_finalize(const ConvState& cs, float* residual_out, hipStream_t s) {
  hipLaunchKernelGGL(conv_finalize_k, dim3(1), dim3(256), 0, s, cs, residual_out);
}
