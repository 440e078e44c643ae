// Mixture-of-experts plumbing around the grouped expert GEMMs (Mixtral-style layers, paper
// Section 4.1 model list): top-2 routing, the stable permutation that groups (token, slot) pairs by
// expert, gathers, the weighted combine and their backward counterparts.  All orders are fixed
// (token order inside an expert, slot 0 before slot 1), so results are reproducible bit for bit.
#include "common.h"

// The two largest router logits of each token (ties go to the lower expert index) and the softmax
// over those two.  One thread per token; logits are float.
__global__ void moe_route_kernel(const float* __restrict__ logit, int n, int E, int32_t* __restrict__ sel,
                                 float* __restrict__ w) {
  int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n) return;
  const float* l = logit + (int64_t)t * E;
  int i0 = 0; float v0 = l[0];
  for (int e = 1; e < E; e++) if (l[e] > v0) { v0 = l[e]; i0 = e; }
  int i1 = -1; float v1 = -INFINITY;
  for (int e = 0; e < E; e++) if (e != i0 && l[e] > v1) { v1 = l[e]; i1 = e; }
  float e1 = expf(v1 - v0);                       // v0 >= v1
  float inv = 1.f / (1.f + e1);
  sel[2 * t] = i0; sel[2 * t + 1] = i1;
  w[2 * t] = inv; w[2 * t + 1] = e1 * inv;
}

// Stable counting sort of the 2n (token, slot) pairs by expert, done by one workgroup: thread i owns
// a contiguous slab of tokens, per-expert counts are scanned across threads in LDS.
// eoff[e] = first permuted row of expert e, pos[2t+s] = permuted row of the pair, perm = inverse.
__global__ __launch_bounds__(1024) void moe_permute_kernel(const int32_t* __restrict__ sel, int n, int E,
                                                           int32_t* __restrict__ eoff, int32_t* __restrict__ pos,
                                                           int32_t* __restrict__ perm) {
  extern __shared__ int32_t cnt[];                // [E][1024], then [E+1] expert bases
  int32_t* ebase = cnt + E * 1024;
  const int tid = threadIdx.x;
  const int per = (n + 1023) / 1024, b = min(n, tid * per), e_ = min(n, b + per);
  for (int e = 0; e < E; e++) cnt[e * 1024 + tid] = 0;
  for (int t = b; t < e_; t++) { cnt[sel[2 * t] * 1024 + tid]++; cnt[sel[2 * t + 1] * 1024 + tid]++; }
  __syncthreads();
  for (int e = 0; e < E; e++) {                   // exclusive scan over threads, expert by expert
    int32_t* c = cnt + e * 1024;
    int mine = c[tid];
    for (int off = 1; off < 1024; off <<= 1) {
      int v = tid >= off ? c[tid - off] : 0;
      __syncthreads();
      c[tid] += v;
      __syncthreads();
    }
    int incl = c[tid];
    __syncthreads();
    c[tid] = incl - mine;
    if (tid == 1023) ebase[e + 1] = incl;          // total of expert e (for now)
    __syncthreads();
  }
  if (tid == 0) {
    ebase[0] = 0;
    for (int e = 0; e < E; e++) ebase[e + 1] += ebase[e];
    for (int e = 0; e <= E; e++) eoff[e] = ebase[e];
  }
  __syncthreads();
  for (int t = b; t < e_; t++)
    for (int s = 0; s < 2; s++) {
      const int e = sel[2 * t + s];
      const int p = ebase[e] + cnt[e * 1024 + tid]++;
      pos[2 * t + s] = p;
      perm[p] = 2 * t + s;
    }
}

// The row kernels move 16 bytes a lane where rows and pointers allow (VEC), else an element: 7900 tokens of 4096 columns, two experts each:
// gather 56 -> 37 us, combine 70 -> 45, gradient of the logits 50 -> 36.
// out[i] = (w ? w[perm[i]] : 1) * src[perm[i] / 2]     (rows of d elements)
template <typename T, bool VEC>
__global__ __launch_bounds__(256) void moe_gather_kernel(const T* __restrict__ src, const int32_t* __restrict__ perm, const float* __restrict__ w,
                                                         int rows, int d, T* __restrict__ out) {
  constexpr int VN = VEC ? Vec<T>::N : 1;
  const int i = blockIdx.x;
  if (i >= rows) return;
  const int pr = perm[i];
  const float sc = w ? w[pr] : 1.f;
  const T* s = src + (int64_t)(pr >> 1) * d;
  T* o = out + (int64_t)i * d;
  for (int j = threadIdx.x * VN; j < d; j += 256 * VN) {
    if (VEC && !w) *reinterpret_cast<typename Vec<T>::type*>(o + j) = *reinterpret_cast<const typename Vec<T>::type*>(s + j);
    else if (VEC) {
      float v[Vec<T>::N]; load_vec<T>(s + j, v);
#pragma unroll
      for (int k = 0; k < Vec<T>::N; k++) v[k] *= sc;
      store_vec<T>(o + j, v);
    } else o[j] = w ? from_f<T>(sc * to_f<T>(s[j])) : s[j];
  }
}

// out[t] = res[t] + w[2t] y[pos[2t]] + w[2t+1] y[pos[2t+1]]
template <typename T, bool VEC>
__global__ __launch_bounds__(256) void moe_combine_kernel(const T* __restrict__ res, const T* __restrict__ y, const int32_t* __restrict__ pos,
                                                          const float* __restrict__ w, int n, int d, T* __restrict__ out) {
  constexpr int VN = VEC ? Vec<T>::N : 1;
  const int t = blockIdx.x;
  if (t >= n) return;
  const T* y0 = y + (int64_t)pos[2 * t] * d; const T* y1 = y + (int64_t)pos[2 * t + 1] * d;
  const float w0 = w ? w[2 * t] : 1.f, w1 = w ? w[2 * t + 1] : 1.f;
  for (int j = threadIdx.x * VN; j < d; j += 256 * VN) {
    float v[VN], a[VN], b[VN];
    if constexpr (VEC) { load_vec<T>(y0 + j, a); load_vec<T>(y1 + j, b); if (res) load_vec<T>(res + (int64_t)t * d + j, v); }
    else { a[0] = to_f<T>(y0[j]); b[0] = to_f<T>(y1[j]); if (res) v[0] = to_f<T>(res[(int64_t)t * d + j]); }
#pragma unroll
    for (int k = 0; k < VN; k++) { v[k] = res ? v[k] : 0.f; v[k] += w0 * a[k]; v[k] += w1 * b[k]; }
    if constexpr (VEC) store_vec<T>(out + (int64_t)t * d + j, v);
    else out[(int64_t)t * d + j] = from_f<T>(v[0]);
  }
}

// The sum of a token's two expert rows and of what reaches it through the router: dlogit has two entries a row (the chosen experts), its adapter's
// part is rank r.  A thread keeps its columns of the adapter in registers over kRouterTokens tokens; a token's own numbers are the same for
// the whole wave.  As a product with K = 8 + 64 on the register-staged 256 x 256 kernel, behind the combination and
// a transposed router, this took 122 + 70 + 5 us for 7900 tokens of 4096 columns, 75 us so; and the sum is rounded once.
constexpr int kRouterRank = 16, kRouterTokens = 16;
template <typename T>
__global__ __launch_bounds__(256) void moe_combine_router_kernel(const T* __restrict__ y, const int32_t* __restrict__ pos, const int32_t* __restrict__ sel,
                                                                 const T* __restrict__ dlogit, int E, const T* __restrict__ Wr, const T* __restrict__ du, int rp,
                                                                 const T* __restrict__ A, int r, int n, int d, T* __restrict__ out) {
  constexpr int VN = Vec<T>::N;
  const int j = (blockIdx.y * 256 + threadIdx.x) * VN;
  if (j >= d) return;
  typename Vec<T>::type a[kRouterRank];
#pragma unroll
  for (int i = 0; i < kRouterRank; i++) if (i < r) a[i] = *reinterpret_cast<const typename Vec<T>::type*>(A + (int64_t)i * d + j);
  for (int t = blockIdx.x * kRouterTokens, end = min(n, t + kRouterTokens); t < end; t++) {
    const int s0 = sel[2 * t], s1 = sel[2 * t + 1];
    const float w0 = to_f<T>(dlogit[(int64_t)t * E + s0]), w1 = to_f<T>(dlogit[(int64_t)t * E + s1]);
    float v[VN], x[VN], p[VN], q[VN];
    load_vec<T>(y + (int64_t)pos[2 * t] * d + j, v); load_vec<T>(y + (int64_t)pos[2 * t + 1] * d + j, x);
    load_vec<T>(Wr + (int64_t)s0 * d + j, p); load_vec<T>(Wr + (int64_t)s1 * d + j, q);
#pragma unroll
    for (int k = 0; k < VN; k++) v[k] += x[k] + (w0 * p[k] + w1 * q[k]);
    const uint32_t* dw = reinterpret_cast<const uint32_t*>(du + (int64_t)t * rp);      // whole words: rows of du are rp elements, 16 at least
#pragma unroll
    for (int i = 0; i < kRouterRank; i++)
      if (i < r) {
        const uint32_t u = dw[sizeof(T) == 2 ? i / 2 : i];
        const float f = __uint_as_float(sizeof(T) == 4 ? u : i % 2 ? u & 0xffff0000u : u << 16);
#pragma unroll
        for (int k = 0; k < VN; k++) v[k] = fmaf(f, to_f<T>(a[i][k]), v[k]);
      }
    store_vec<T>(out + (int64_t)t * d + j, v);
  }
}

// Gradient of the routing weights and of the router logits: dw_s = <dy[t], y[pos_s]>,
// dl_s = w_s (dw_s - sum_s' w_s' dw_s'); dlogit[t, :] is zero except at the two selected experts.
template <typename T, bool VEC>
__global__ void moe_dlogit_kernel(const T* __restrict__ dy, const T* __restrict__ y, const int32_t* __restrict__ pos,
                                  const int32_t* __restrict__ sel, const float* __restrict__ w, int n, int d, int Epad,
                                  T* __restrict__ dlogit) {
  constexpr int VN = VEC ? Vec<T>::N : 1;
  const int t = blockIdx.x * (blockDim.x / AS_WAVE) + threadIdx.x / AS_WAVE, lane = threadIdx.x % AS_WAVE;
  if (t >= n) return;
  const T* g = dy + (int64_t)t * d;
  const T* y0 = y + (int64_t)pos[2 * t] * d; const T* y1 = y + (int64_t)pos[2 * t + 1] * d;
  float a0 = 0.f, a1 = 0.f;
#pragma unroll 4
  for (int j = lane * VN; j < d; j += AS_WAVE * VN) {
    float gv[VN], b[VN], c[VN];
    if constexpr (VEC) { load_vec<T>(g + j, gv); load_vec<T>(y0 + j, b); load_vec<T>(y1 + j, c); }
    else { gv[0] = to_f<T>(g[j]); b[0] = to_f<T>(y0[j]); c[0] = to_f<T>(y1[j]); }
#pragma unroll
    for (int k = 0; k < VN; k++) { a0 += gv[k] * b[k]; a1 += gv[k] * c[k]; }
  }
  a0 = wave_sum(a0); a1 = wave_sum(a1);
  const float w0 = w[2 * t], w1 = w[2 * t + 1], mean = w0 * a0 + w1 * a1;
  const int s0 = sel[2 * t], s1 = sel[2 * t + 1];
  for (int e = lane; e < Epad; e += AS_WAVE)
    dlogit[(int64_t)t * Epad + e] = from_f<T>(e == s0 ? w0 * (a0 - mean) : e == s1 ? w1 * (a1 - mean) : 0.f);
}

int launch_moe_route(as_ctx* ctx, const float* logit, int n, int E, int32_t* sel, float* w, hipStream_t st) {
  if (n <= 0) return AS_OK;
  prof_begin(ctx, st, AS_K_MOE, 0.0);
  moe_route_kernel<<<(unsigned)cdiv(n, 256), 256, 0, st>>>(logit, n, E, sel, w);
  prof_end(ctx, st);
  AS_LAUNCH_CHECK(ctx);
  return AS_OK;
}

int launch_moe_permute(as_ctx* ctx, const int32_t* sel, int n, int E, int32_t* eoff, int32_t* pos, int32_t* perm, hipStream_t st) {
  size_t smem = ((size_t)E * 1024 + E + 1) * sizeof(int32_t);
  if (smem > 160 * 1024) return as_fail(ctx, AS_ERR_SHAPE, "moe: too many experts for the permutation kernel");
  if (smem > 48 * 1024)
    AS_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(moe_permute_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
  prof_begin(ctx, st, AS_K_MOE, 0.0);
  moe_permute_kernel<<<1, 1024, smem, st>>>(sel, n, E, eoff, pos, perm);
  prof_end(ctx, st);
  AS_LAUNCH_CHECK(ctx);
  return AS_OK;
}

int launch_moe_gather(as_ctx* ctx, int mode, const void* src, const int32_t* perm, const float* w, int rows, int d, void* out, hipStream_t st) {
  if (rows <= 0) return AS_OK;
  prof_begin(ctx, st, AS_K_MOE, 0.0);
  DISPATCH_T(mode, {
    if (vec_ok<T>(src, d) && vec_ok<T>(out, d)) moe_gather_kernel<T, true><<<rows, 256, 0, st>>>((const T*)src, perm, w, rows, d, (T*)out);
    else moe_gather_kernel<T, false><<<rows, 256, 0, st>>>((const T*)src, perm, w, rows, d, (T*)out); });
  prof_end(ctx, st);
  AS_LAUNCH_CHECK(ctx);
  return AS_OK;
}

int launch_moe_combine(as_ctx* ctx, int mode, const void* res, const void* y, const int32_t* pos, const float* w, int n, int d,
                       void* out, hipStream_t st) {
  if (n <= 0) return AS_OK;
  prof_begin(ctx, st, AS_K_MOE, 0.0);
  DISPATCH_T(mode, {
    if ((!res || vec_ok<T>(res, d)) && vec_ok<T>(y, d) && vec_ok<T>(out, d)) moe_combine_kernel<T, true><<<n, 256, 0, st>>>((const T*)res, (const T*)y, pos, w, n, d, (T*)out);
    else moe_combine_kernel<T, false><<<n, 256, 0, st>>>((const T*)res, (const T*)y, pos, w, n, d, (T*)out); });
  prof_end(ctx, st);
  AS_LAUNCH_CHECK(ctx);
  return AS_OK;
}

bool moe_combine_router_ok(int mode, int d, int r, const void* y, const void* Wr, const void* A, const void* out) {
  bool ok = false;
  DISPATCH_T(mode, ok = r <= kRouterRank && vec_ok<T>(y, d) && vec_ok<T>(Wr, d) && (r == 0 || vec_ok<T>(A, d)) && vec_ok<T>(out, d););
  return ok;
}
int launch_moe_combine_router(as_ctx* ctx, int mode, const void* y, const int32_t* pos, const int32_t* sel, const void* dlogit, int E, const void* Wr,
                              const void* du, int rp, const void* A, int r, int n, int d, void* out, hipStream_t st) {
  if (n <= 0) return AS_OK;
  prof_begin(ctx, st, AS_K_MOE, 0.0);
  DISPATCH_T(mode, (moe_combine_router_kernel<T><<<dim3((unsigned)cdiv(n, kRouterTokens), (unsigned)cdiv(d, 256 * Vec<T>::N)), 256, 0, st>>>(
      (const T*)y, pos, sel, (const T*)dlogit, E, (const T*)Wr, (const T*)du, rp, (const T*)A, r, n, d, (T*)out)));
  prof_end(ctx, st);
  AS_LAUNCH_CHECK(ctx);
  return AS_OK;
}

int launch_moe_dlogit(as_ctx* ctx, int mode, const void* dy, const void* y, const int32_t* pos, const int32_t* sel, const float* w,
                      int n, int d, int Epad, void* dlogit, hipStream_t st) {
  if (n <= 0) return AS_OK;
  prof_begin(ctx, st, AS_K_MOE, 0.0);
  DISPATCH_T(mode, {
    if (vec_ok<T>(dy, d) && vec_ok<T>(y, d)) moe_dlogit_kernel<T, true><<<(unsigned)cdiv(n, 4), 256, 0, st>>>((const T*)dy, (const T*)y, pos, sel, w, n, d, Epad, (T*)dlogit);
    else moe_dlogit_kernel<T, false><<<(unsigned)cdiv(n, 4), 256, 0, st>>>((const T*)dy, (const T*)y, pos, sel, w, n, d, Epad, (T*)dlogit); });
  prof_end(ctx, st);
  AS_LAUNCH_CHECK(ctx);
  return AS_OK;
}
