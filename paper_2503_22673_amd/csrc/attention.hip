// Varlen causal attention with grouped KV heads over packed rows: a query at
// token t sees keys seg_start[t] .. t only, so nothing crosses a trajectory
// boundary.  Query head j reads KV head j / (Hq/Hkv).
//
// Plain kernels (any type; the fp32 tier): one workgroup per (token, head), scores of the whole visible range kept in LDS.
// What bounds them is latency: the scores of a token are 256 rows at a time, one row per thread; the weighted sums over the
// visible rows take 256 / dh row groups side by side (their sums are added in order at the end), so that neither loop is a
// long chain of dependent loads.  469 tokens, 4 heads of 32: forward 24 us, dQ 21, dK and dV 103 with one wave per token;
// 12, 15 and 19 us so.
// The one shape that lost by it is the forward of many segments of 8 to 48 tokens (4096 tokens in segments of 16, 8 heads of 32: 51 us
// against 44 with one wave per token), where three of the four waves have no row; its backward takes 137 us against 243.
// Leaving short ranges to the first wave gave the 44 back and cost long segments 3 to 7 %; 128 threads cost them 7 %.
#include "common.h"

constexpr int kPlainThreads = 256;
__device__ __forceinline__ float block_sum_plain(float v, float* red) {      // sum over the workgroup in wave order; red: 4 floats
  v = wave_sum(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  return red[0] + red[1] + red[2] + red[3];
}
__device__ __forceinline__ float block_max_plain(float v, float* red) {
  v = wave_max(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  return fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
}
// rows of dh values: dot product of a row in memory with one in LDS, four columns at a time (dh is a multiple of 32)
template <typename T> __device__ __forceinline__ float dot_row(const float* a, const T* row, int dh) {
  float d = 0.f;
#pragma unroll 4
  for (int c = 0; c < dh; c += 4) {
    float x[4];
#pragma unroll
    for (int q = 0; q < 4; q++) x[q] = to_f<T>(row[c + q]);
#pragma unroll
    for (int q = 0; q < 4; q++) d = fmaf(a[c + q], x[q], d);
  }
  return d;
}

// --------------------------------------------------------------- plain fwd
template <typename T>
__global__ __launch_bounds__(256) void attn_fwd_plain(AttnParams p, float scale) {
  extern __shared__ float sm[];
  float* qs = sm;                  // [dh]; also the reductions' four values, once the scores are there
  float* sc = sm + p.dh;           // [max(max_seg, 256)]
  const int t = blockIdx.x, j = blockIdx.y, tid = threadIdx.x, dh = p.dh;
  const int g = j / (p.Hq / p.Hkv);
  const int s0 = p.seg_start[t], len = t - s0 + 1;
  const T* q = (const T*)p.q + (int64_t)t * p.ldq + j * dh;
  const T* kb = (const T*)p.k + (int64_t)s0 * p.ldkv + g * dh;
  const T* vb = (const T*)p.v + (int64_t)s0 * p.ldkv + g * dh;
  for (int c = tid; c < dh; c += kPlainThreads) qs[c] = to_f<T>(q[c]);
  __syncthreads();
  float mx = -INFINITY;
  for (int u = tid; u < len; u += kPlainThreads) {
    const float d = dot_row<T>(qs, kb + (int64_t)u * p.ldkv, dh) * scale;
    sc[u] = d;
    mx = fmaxf(mx, d);
  }
  mx = block_max_plain(mx, qs);
  float sum = 0.f;
  for (int u = tid; u < len; u += kPlainThreads) { float e = expf(sc[u] - mx); sc[u] = e; sum += e; }
  sum = block_sum_plain(sum, qs);                        // its barriers also publish the scores
  const int ng = kPlainThreads / dh, grp = tid / dh, c = tid % dh;
  float acc = 0.f;
  if (grp < ng) {
#pragma unroll 4
    for (int u = grp; u < len; u += ng) acc = fmaf(sc[u], to_f<T>(vb[(int64_t)u * p.ldkv + c]), acc);
  }
  __syncthreads();
  sc[tid] = acc;
  __syncthreads();
  if (grp == 0) {
    for (int i = 1; i < ng; i++) acc += sc[i * dh + c];
    ((T*)p.o)[((int64_t)t * p.Hq + j) * dh + c] = from_f<T>(acc / sum);
  }
  if (tid == 0) p.lse[(int64_t)t * p.Hq + j] = mx + logf(sum);
}

// --------------------------------------------------------------- plain bwd
// dq for one (token, head); also writes delta = sum_c dO*O for the dK/dV pass.
template <typename T>
__global__ __launch_bounds__(256) void attn_bwd_dq_plain(AttnParams p, float scale) {
  extern __shared__ float sm[];
  float* qs = sm; float* dos = sm + p.dh; float* sc = sm + 2 * p.dh;
  const int t = blockIdx.x, j = blockIdx.y, tid = threadIdx.x, dh = p.dh;
  const int g = j / (p.Hq / p.Hkv);
  const int s0 = p.seg_start[t], len = t - s0 + 1;
  const T* q = (const T*)p.q + (int64_t)t * p.ldq + j * dh;
  const T* o = (const T*)p.o + ((int64_t)t * p.Hq + j) * dh;
  const T* d_o = (const T*)p.d_o + ((int64_t)t * p.Hq + j) * dh;
  const T* kb = (const T*)p.k + (int64_t)s0 * p.ldkv + g * dh;
  const T* vb = (const T*)p.v + (int64_t)s0 * p.ldkv + g * dh;
  float dl = 0.f;
  for (int c = tid; c < dh; c += kPlainThreads) {
    float a = to_f<T>(d_o[c]);
    qs[c] = to_f<T>(q[c]); dos[c] = a;
    dl += a * to_f<T>(o[c]);
  }
  dl = block_sum_plain(dl, sc);
  __syncthreads();                                       // before the scores go where the sum's four values are
  const float lse = p.lse[(int64_t)t * p.Hq + j];
  if (tid == 0) p.delta[(int64_t)t * p.Hq + j] = dl;
  for (int u = tid; u < len; u += kPlainThreads) {
    const float d = dot_row<T>(qs, kb + (int64_t)u * p.ldkv, dh), dp = dot_row<T>(dos, vb + (int64_t)u * p.ldkv, dh);
    float pr = expf(d * scale - lse);
    sc[u] = pr * (dp - dl);
  }
  __syncthreads();
  const int ng = kPlainThreads / dh, grp = tid / dh, c = tid % dh;
  float acc = 0.f;
  if (grp < ng) {
#pragma unroll 4
    for (int u = grp; u < len; u += ng) acc = fmaf(sc[u], to_f<T>(kb[(int64_t)u * p.ldkv + c]), acc);
  }
  __syncthreads();
  sc[tid] = acc;
  __syncthreads();
  if (grp == 0) {
    for (int i = 1; i < ng; i++) acc += sc[i * dh + c];
    ((T*)p.dq)[(int64_t)t * p.ldq + j * dh + c] = from_f<T>(acc * scale);
  }
}

// dk, dv for one (token u, KV head): sums over the query heads of the group in
// head order and over later tokens of the segment in token order, per row group.
template <typename T>
__global__ __launch_bounds__(256) void attn_bwd_dkv_plain(AttnParams p, float scale) {
  extern __shared__ float sm[];
  float* ks = sm; float* vs = sm + p.dh; float* sp = sm + 2 * p.dh; float* sd = sp + max(p.max_seg, kPlainThreads);
  const int u = blockIdx.x, g = blockIdx.y, tid = threadIdx.x, dh = p.dh;
  const int grp_q = p.Hq / p.Hkv;
  const int e = p.seg_end[u], len = e - u;
  const T* k = (const T*)p.k + (int64_t)u * p.ldkv + g * dh;
  const T* v = (const T*)p.v + (int64_t)u * p.ldkv + g * dh;
  for (int c = tid; c < dh; c += kPlainThreads) { ks[c] = to_f<T>(k[c]); vs[c] = to_f<T>(v[c]); }
  const int ng = kPlainThreads / dh, grp = tid / dh, c = tid % dh;
  float dk = 0.f, dv = 0.f;
  for (int jj = 0; jj < grp_q; jj++) {
    const int j = g * grp_q + jj;
    __syncthreads();
    for (int i = tid; i < len; i += kPlainThreads) {
      const int t = u + i;
      const float d = dot_row<T>(ks, (const T*)p.q + (int64_t)t * p.ldq + j * dh, dh);
      const float dp = dot_row<T>(vs, (const T*)p.d_o + ((int64_t)t * p.Hq + j) * dh, dh);
      float pr = expf(d * scale - p.lse[(int64_t)t * p.Hq + j]);
      sp[i] = pr;
      sd[i] = pr * (dp - p.delta[(int64_t)t * p.Hq + j]);
    }
    __syncthreads();
    if (grp < ng) {
      const T* qr = (const T*)p.q + (int64_t)u * p.ldq + j * dh + c;
      const T* dor = (const T*)p.d_o + ((int64_t)u * p.Hq + j) * dh + c;
#pragma unroll 4
      for (int i = grp; i < len; i += ng) {
        dv = fmaf(sp[i], to_f<T>(dor[(int64_t)i * p.Hq * dh]), dv);
        dk = fmaf(sd[i], to_f<T>(qr[(int64_t)i * p.ldq]), dk);
      }
    }
  }
  __syncthreads();
  sp[tid] = dk; sd[tid] = dv;
  __syncthreads();
  if (grp == 0) {
    for (int i = 1; i < ng; i++) { dk += sp[i * dh + c]; dv += sd[i * dh + c]; }
    ((T*)p.dk)[(int64_t)u * p.ldkv + g * dh + c] = from_f<T>(dk * scale);
    ((T*)p.dv)[(int64_t)u * p.ldkv + g * dh + c] = from_f<T>(dv);
  }
}

static int check_plain(as_ctx* ctx, const AttnParams& p, size_t smem) {
  if (p.dh > 128) return as_fail(ctx, AS_ERR_SHAPE, "attention: head_dim <= 128");
  if (smem > 160 * 1024) return as_fail(ctx, AS_ERR_SHAPE, "attention (plain kernels): segment too long for LDS");
  return AS_OK;
}

template <typename K>
static int set_smem(as_ctx* ctx, K kern, size_t smem) {
  if (smem > 48 * 1024)
    AS_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
  return AS_OK;
}

int launch_attention_fwd_mfma(as_ctx* ctx, const AttnParams& p, int variant, hipStream_t st);
int launch_attention_bwd_mfma(as_ctx* ctx, const AttnParams& p, int variant, hipStream_t st);
bool attention_mfma_ok(const AttnParams& p);

int launch_attention_fwd(as_ctx* ctx, int mode, int variant, const AttnParams& p, hipStream_t st) {
  if (p.n <= 0) return AS_OK;
  bool mf = mode == AS_BF16 && variant != 1 && attention_mfma_ok(p);
  if (variant >= 2 && !mf) return as_fail(ctx, AS_ERR_SHAPE, "attention: MFMA kernel needs bf16, head_dim 64/128, aligned strides");
  if (mf) { prof_begin(ctx, st, AS_K_ATTN_FWD, 0.0); int r = launch_attention_fwd_mfma(ctx, p, variant, st); prof_end(ctx, st); return r; }
  const int seg = std::max(p.max_seg, kPlainThreads);    // the score arrays also take one value per thread at the end
  size_t smem = (size_t)(p.dh + seg) * sizeof(float);
  int rc = check_plain(ctx, p, smem); if (rc) return rc;
  float scale = 1.f / sqrtf((float)p.dh);
  dim3 grid(p.n, p.Hq);
  if (mode == AS_FP32) { rc = set_smem(ctx, attn_fwd_plain<float>, smem); if (rc) return rc;
                         attn_fwd_plain<float><<<grid, kPlainThreads, smem, st>>>(p, scale); }
  else { rc = set_smem(ctx, attn_fwd_plain<bf16_t>, smem); if (rc) return rc;
         attn_fwd_plain<bf16_t><<<grid, kPlainThreads, smem, st>>>(p, scale); }
  AS_LAUNCH_CHECK(ctx);
  return AS_OK;
}

bool attention_bwd_is_mfma(int mode, int variant, const AttnParams& p) { return mode == AS_BF16 && variant != 1 && attention_mfma_ok(p); }

int launch_attention_bwd(as_ctx* ctx, int mode, int variant, const AttnParams& p, hipStream_t st) {
  if (p.n <= 0) return AS_OK;
  bool mf = mode == AS_BF16 && variant != 1 && attention_mfma_ok(p);
  if (!mf && p.rope_cos) return as_fail(ctx, AS_ERR_SHAPE, "attention: only the MFMA kernels rotate their gradients");
  if (variant >= 2 && !mf) return as_fail(ctx, AS_ERR_SHAPE, "attention: MFMA kernel needs bf16, head_dim 64/128, aligned strides");
  if (mf) { prof_begin(ctx, st, AS_K_ATTN_BWD, 0.0); int r = launch_attention_bwd_mfma(ctx, p, variant, st); prof_end(ctx, st); return r; }
  const int seg = std::max(p.max_seg, kPlainThreads);
  size_t smem1 = (size_t)(2 * p.dh + seg) * sizeof(float);
  size_t smem2 = (size_t)(2 * p.dh + 2 * seg) * sizeof(float);
  int rc = check_plain(ctx, p, smem2); if (rc) return rc;
  float scale = 1.f / sqrtf((float)p.dh);
  dim3 g1(p.n, p.Hq), g2(p.n, p.Hkv);
  if (mode == AS_FP32) {
    rc = set_smem(ctx, attn_bwd_dq_plain<float>, smem1); if (rc) return rc;
    rc = set_smem(ctx, attn_bwd_dkv_plain<float>, smem2); if (rc) return rc;
    attn_bwd_dq_plain<float><<<g1, kPlainThreads, smem1, st>>>(p, scale);
    AS_LAUNCH_CHECK(ctx);
    attn_bwd_dkv_plain<float><<<g2, kPlainThreads, smem2, st>>>(p, scale);
  } else {
    rc = set_smem(ctx, attn_bwd_dq_plain<bf16_t>, smem1); if (rc) return rc;
    rc = set_smem(ctx, attn_bwd_dkv_plain<bf16_t>, smem2); if (rc) return rc;
    attn_bwd_dq_plain<bf16_t><<<g1, kPlainThreads, smem1, st>>>(p, scale);
    AS_LAUNCH_CHECK(ctx);
    attn_bwd_dkv_plain<bf16_t><<<g2, kPlainThreads, smem2, st>>>(p, scale);
  }
  AS_LAUNCH_CHECK(ctx);
  return AS_OK;
}
