// HBM-bound kernels of the fine-tuning step: packing, embedding gather,
// RMSNorm, RoPE, SwiGLU, transposes, LoRA operand preparation, target
// selection, the cross-entropy row pass, reductions and AdamW.
// One wavefront (64 lanes) owns one token row wherever a row reduction is
// needed, so reductions are shuffles only; rows are read with 16-byte loads.
#include "common.h"

// ------------------------------------------------------------------ pack
// The packed stream lies in pinned host memory, put together there: one pass over the bus.  Four tokens a thread, so that a wave asks
// for a kilobyte of tokens at a time and the whole stream is under way at once.
template <bool VEC>
__global__ __launch_bounds__(256) void pack_kernel(const int32_t* __restrict__ h_tok, const int32_t* __restrict__ h_cu, const uint8_t* __restrict__ h_mask, int n_out, int n_cu,
                                                   int32_t* __restrict__ tok, int32_t* __restrict__ cu, uint8_t* __restrict__ mask) {
  const int i = blockIdx.x * 256 + threadIdx.x;            // below 2^29: n_out is an int
  for (int k = i; k < n_cu; k += gridDim.x * 256) cu[k] = h_cu[k];
  if (VEC && i < n_out / 4) {
    const int4 t = reinterpret_cast<const int4*>(h_tok)[i];
    const uint32_t m = reinterpret_cast<const uint32_t*>(h_mask)[i];
    reinterpret_cast<int4*>(tok)[i] = t; reinterpret_cast<uint32_t*>(mask)[i] = m;
    return;
  }
  for (int k = 4 * i, end = k + min(4, n_out - k); k < end; k++) { tok[k] = h_tok[k]; mask[k] = h_mask[k]; }      // 4 i + 4 may not be an int
}

int launch_pack(as_ctx* ctx, const int32_t* h_tokens, const int32_t* h_cu, const uint8_t* h_mask, int n_out, int n_cu, int32_t* d_tokens, int32_t* d_cu, uint8_t* d_mask, hipStream_t st) {
  const unsigned grid = (unsigned)std::max<int64_t>(1, cdiv(n_out, 1024));
  if (!((uintptr_t)d_tokens % 16) && !((uintptr_t)d_mask % 4)) pack_kernel<true><<<grid, 256, 0, st>>>(h_tokens, h_cu, h_mask, n_out, n_cu, d_tokens, d_cu, d_mask);
  else pack_kernel<false><<<grid, 256, 0, st>>>(h_tokens, h_cu, h_mask, n_out, n_cu, d_tokens, d_cu, d_mask);
  AS_LAUNCH_CHECK(ctx);
  return AS_OK;
}

__global__ void compact_kernel(const int32_t* __restrict__ tok, const uint8_t* __restrict__ mask,
                               const int32_t* __restrict__ cu_c, const int32_t* __restrict__ src_start, int n_seg, int n,
                               int32_t* __restrict__ tok_c, uint8_t* __restrict__ mask_c) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  int lo = 0, hi = n_seg - 1;               // last s with cu_c[s] <= i
  while (lo < hi) {
    int mid = (lo + hi + 1) >> 1;
    if (cu_c[mid] <= i) lo = mid; else hi = mid - 1;
  }
  int src = src_start[lo] + (i - cu_c[lo]);
  tok_c[i] = tok[src];
  mask_c[i] = mask[src];
}

int launch_compact(as_ctx* ctx, const int32_t* tok, const uint8_t* mask, const int32_t* cu_c, const int32_t* src_start,
                   int n_seg, int n, int32_t* tok_c, uint8_t* mask_c, hipStream_t st) {
  if (n <= 0) return AS_OK;
  compact_kernel<<<cdiv(n, 256), 256, 0, st>>>(tok, mask, cu_c, src_start, n_seg, n, tok_c, mask_c);
  AS_LAUNCH_CHECK(ctx);
  return AS_OK;
}

// token t predicts a target: the next token is of the same segment and bears loss
__device__ __forceinline__ bool predicts_target(int t, int seg_end, const uint8_t* mask) { return t + 1 < seg_end && mask[t + 1]; }

__device__ __forceinline__ void segment_info_block(const StepBegin& b, int block) {      // of kTargetBlock threads
  const int t = block * kTargetBlock + threadIdx.x;
  bool is = false;
  if (t < b.n) {
    int lo = 0, hi = b.n_seg - 1;           // last s with cu[s] <= t
    while (lo < hi) {
      int mid = (lo + hi + 1) >> 1;
      if (b.cu[mid] <= t) lo = mid; else hi = mid - 1;
    }
    const int e = b.cu[lo + 1];
    b.seg_start[t] = b.cu[lo];
    b.seg_end[t] = e;
    is = predicts_target(t, e, b.mask);
  }
  const int c = __syncthreads_count(is);
  if (threadIdx.x == 0) b.block_targets[block] = c;
}

// ------------------------------------------------------------------ RoPE
// cos/sin of p * base^(-2i/dh), evaluated in double and rounded once.
__device__ __forceinline__ void rope_table_block(const StepBegin& b, int block) {
  const int half = b.dh / 2, idx = block * 256 + threadIdx.x;
  if (idx >= b.max_pos * half) return;
  int p = idx / half, i = idx % half;
  double theta = pow(b.rope_base, -2.0 * (double)i / (double)b.dh);
  double s, c;
  sincos((double)p * theta, &s, &c);
  b.cosb[idx] = (float)c;
  b.sinb[idx] = (float)s;
}

// Rotates pairs (i, i + dh/2) of every head in place; the position of token t
// is t - seg_start[t].  One thread per (token, head, 2 adjacent i).
template <typename T>
__global__ void rope_kernel(int n, int n_heads, int dh, T* __restrict__ x, int64_t ldx,
                            const int32_t* __restrict__ seg_start, const float* __restrict__ cosb,
                            const float* __restrict__ sinb) {
  int half = dh >> 1;
  int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t tot = (int64_t)n * n_heads * half;
  if (idx >= tot) return;
  int i = idx % half;
  int64_t r = idx / half;
  int hd = r % n_heads;
  int t = r / n_heads;
  int p = t - seg_start[t];
  float c = cosb[(int64_t)p * half + i], s = sinb[(int64_t)p * half + i];
  T* row = x + (int64_t)t * ldx + (int64_t)hd * dh;
  float x1 = to_f<T>(row[i]), x2 = to_f<T>(row[i + half]);
  row[i] = from_f<T>(x1 * c - x2 * s);
  row[i + half] = from_f<T>(x1 * s + x2 * c);
}

// Same rotation, one thread per (token, head, Vec<T>::N adjacent i): 16-byte loads and stores.
template <typename T>
__global__ void rope_vec_kernel(int n, int n_heads, int dh, T* __restrict__ x, int64_t ldx,
                                const int32_t* __restrict__ seg_start, const float* __restrict__ cosb,
                                const float* __restrict__ sinb) {
  constexpr int VN = Vec<T>::N;
  const int half = dh >> 1, per = half / VN;
  int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (int64_t)n * n_heads * per) return;
  const int i = (int)(idx % per) * VN;
  const int64_t r = idx / per;
  const int hd = (int)(r % n_heads), t = (int)(r / n_heads);
  const int p = t - seg_start[t];
  T* row = x + (int64_t)t * ldx + (int64_t)hd * dh;
  float x1[VN], x2[VN], o1[VN], o2[VN];
  load_vec<T>(row + i, x1); load_vec<T>(row + i + half, x2);
#pragma unroll
  for (int k = 0; k < VN; k += 4) {
    const f32x4 c = *reinterpret_cast<const f32x4*>(cosb + (int64_t)p * half + i + k);
    const f32x4 s = *reinterpret_cast<const f32x4*>(sinb + (int64_t)p * half + i + k);
#pragma unroll
    for (int q = 0; q < 4; q++) {
      o1[k + q] = x1[k + q] * c[q] - x2[k + q] * s[q];
      o2[k + q] = x1[k + q] * s[q] + x2[k + q] * c[q];
    }
  }
  store_vec<T>(row + i, o1); store_vec<T>(row + i + half, o2);
}

int launch_rope(as_ctx* ctx, int mode, int n, int n_heads, int dh, void* x, int64_t ldx,
                const int32_t* seg_start, const float* cosb, const float* sinb, hipStream_t st) {
  int64_t tot = (int64_t)n * n_heads * (dh / 2);
  if (tot <= 0) return AS_OK;
  prof_begin(ctx, st, AS_K_ROPE, 0.0);
  DISPATCH_T(mode, {
    constexpr int VN = Vec<T>::N;
    if ((dh / 2) % VN == 0 && vec_ok<T>(x, ldx) && ((uintptr_t)cosb % 16) == 0 && ((uintptr_t)sinb % 16) == 0)
      rope_vec_kernel<T><<<cdiv(tot / VN, 256), 256, 0, st>>>(n, n_heads, dh, (T*)x, ldx, seg_start, cosb, sinb);
    else
      rope_kernel<T><<<cdiv(tot, 256), 256, 0, st>>>(n, n_heads, dh, (T*)x, ldx, seg_start, cosb, sinb); });
  prof_end(ctx, st);
  AS_LAUNCH_CHECK(ctx);
  return AS_OK;
}

// --------------------------------------------------------------- embedding
template <typename T>
__device__ __forceinline__ void embed_row(const StepBegin& b, int t) {
  const int d = b.d;
  const T* src = (const T*)b.embed + (int64_t)b.tok[t] * d;
  T* dst = (T*)b.h + (int64_t)t * d;
  if (b.vec) {
    constexpr int VN = Vec<T>::N;
    for (int j = threadIdx.x * VN; j < d; j += 256 * VN)
      *reinterpret_cast<typename Vec<T>::type*>(dst + j) = *reinterpret_cast<const typename Vec<T>::type*>(src + j);
  } else {
    for (int j = threadIdx.x; j < d; j += 256) dst[j] = src[j];
  }
}

// ----------------------------------------------------------------- RMSNorm
// One wavefront per row, four rows per block.  The first KEEP 16-byte pieces a lane has of a row, its gains and its addend (bf16: 2048 columns with KEEP = 4,
// 4096 with 8) are asked for before any of them is used: piece by piece, each waited for the one before, and again in the second pass (626 rows of
// 2048: forward 5.8 -> 5.1 us, backward 7.3 -> 5.3; 24,710: 33 -> 30 and 67 -> 60).
template <typename T, int KEEP>
__device__ __forceinline__ void load_pieces(const T* row, int d, int lane, typename Vec<T>::type (&v)[KEEP]) {
#pragma unroll
  for (int q = 0; q < KEEP; q++)                           // a piece past the end: the last one, which nobody uses
    if (q * AS_WAVE * Vec<T>::N < d) v[q] = *reinterpret_cast<const typename Vec<T>::type*>(row + min((q * AS_WAVE + lane) * Vec<T>::N, d - Vec<T>::N));
}
template <typename T, int KEEP>
__global__ __launch_bounds__(256) void rmsnorm_fwd_kernel(int n, int d, const T* __restrict__ x, const int32_t* __restrict__ row_idx,
                                   const int* __restrict__ n_dev, const T* __restrict__ g, float eps,
                                   T* __restrict__ y, float* __restrict__ rstd, int vec) {
  int row = blockIdx.x * (blockDim.x / AS_WAVE) + threadIdx.x / AS_WAVE;
  int lane = threadIdx.x % AS_WAVE;
  int nn = n_dev ? min(n, *n_dev) : n;
  if (row >= nn) return;
  const T* xr = x + (int64_t)(row_idx ? row_idx[row] : row) * d;
  T* yr = y + (int64_t)row * d;
  constexpr int VN = Vec<T>::N, STEP = AS_WAVE * VN;
  typedef typename Vec<T>::type VT;
  VT kept[KEEP], kg[KEEP];
  float ss = 0.f;
  if (vec) {
    load_pieces<T, KEEP>(xr, d, lane, kept); load_pieces<T, KEEP>(g, d, lane, kg);
#pragma unroll
    for (int c = 0; c < KEEP; c++)
      if (c * STEP + lane * VN < d) {
#pragma unroll
        for (int i = 0; i < VN; i++) { const float v = to_f<T>(kept[c][i]); ss += v * v; }
      }
    for (int j = KEEP * STEP + lane * VN; j < d; j += STEP) {
      float v[VN]; load_vec<T>(xr + j, v);
#pragma unroll
      for (int i = 0; i < VN; i++) ss += v[i] * v[i];
    }
  } else {
    for (int j = lane; j < d; j += AS_WAVE) { float v = to_f<T>(xr[j]); ss += v * v; }
  }
  ss = wave_sum(ss);
  float r = rsqrtf(ss / (float)d + eps);
  // one Newton step: rsqrtf is an approximation, the fp32 tier needs ~1e-7
  { float a = ss / (float)d + eps; r = r * (1.5f - 0.5f * a * r * r); }
  if (lane == 0) rstd[row] = r;
  if (vec) {
#pragma unroll
    for (int c = 0; c < KEEP; c++) {
      const int j = c * STEP + lane * VN;
      if (j < d) {
        float v[VN];
#pragma unroll
        for (int i = 0; i < VN; i++) v[i] = to_f<T>(kept[c][i]) * r * to_f<T>(kg[c][i]);
        store_vec<T>(yr + j, v);
      }
    }
    for (int j = KEEP * STEP + lane * VN; j < d; j += STEP) {
      float v[VN], gg[VN]; load_vec<T>(xr + j, v); load_vec<T>(g + j, gg);
#pragma unroll
      for (int i = 0; i < VN; i++) v[i] = v[i] * r * gg[i];
      store_vec<T>(yr + j, v);
    }
  } else {
    for (int j = lane; j < d; j += AS_WAVE) yr[j] = from_f<T>(to_f<T>(xr[j]) * r * to_f<T>(g[j]));
  }
}

int launch_rmsnorm_fwd(as_ctx* ctx, int mode, int n, int d, const void* x, const int32_t* row_idx,
                       const int* n_dev, const void* g, float eps, void* y, float* rstd, hipStream_t st) {
  if (n <= 0) return AS_OK;
  prof_begin(ctx, st, AS_K_NORM, 0.0);
  DISPATCH_T(mode, { int vec = vec_ok<T>(x, d) && vec_ok<T>(y, d) && vec_ok<T>(g, d);
                     auto k = d <= 4 * AS_WAVE * Vec<T>::N ? rmsnorm_fwd_kernel<T, 4> : rmsnorm_fwd_kernel<T, 8>;
                     k<<<cdiv(n, 4), 256, 0, st>>>(n, d, (const T*)x, row_idx, n_dev, (const T*)g, eps, (T*)y, rstd, vec); });
  prof_end(ctx, st);
  AS_LAUNCH_CHECK(ctx);
  return AS_OK;
}

template <typename T, int KEEP>
__global__ __launch_bounds__(256) void rmsnorm_bwd_kernel(int n, int d, const T* __restrict__ dy, const int32_t* __restrict__ src_pos,
                                   const T* __restrict__ x, const T* __restrict__ g,
                                   const float* __restrict__ rstd, const T* __restrict__ add,
                                   T* __restrict__ dx, int vec) {
  int row = blockIdx.x * (blockDim.x / AS_WAVE) + threadIdx.x / AS_WAVE;
  int lane = threadIdx.x % AS_WAVE;
  if (row >= n) return;
  constexpr int VN = Vec<T>::N;
  int64_t src = src_pos ? src_pos[row] : row;
  T* dxr = dx + (int64_t)row * d;
  const T* ar = add ? add + (int64_t)row * d : nullptr;
  if (src < 0) {                         // no upstream gradient for this row
    for (int j = lane; j < d; j += AS_WAVE) dxr[j] = ar ? ar[j] : from_f<T>(0.f);
    return;
  }
  const T* dyr = dy + src * d;
  const T* xr = x + (int64_t)row * d;
  float r = rstd[src_pos ? src : row];
  float dot = 0.f;
  constexpr int STEP = AS_WAVE * VN;
  typedef typename Vec<T>::type VT;
  VT kdy[KEEP], kx[KEEP], kg[KEEP], ka[KEEP];
  if (vec) {
    load_pieces<T, KEEP>(dyr, d, lane, kdy); load_pieces<T, KEEP>(xr, d, lane, kx); load_pieces<T, KEEP>(g, d, lane, kg);
    if (ar) load_pieces<T, KEEP>(ar, d, lane, ka);
#pragma unroll
    for (int q = 0; q < KEEP; q++)
      if (q * STEP + lane * VN < d) {
#pragma unroll
        for (int i = 0; i < VN; i++) dot += to_f<T>(kdy[q][i]) * to_f<T>(kx[q][i]) * to_f<T>(kg[q][i]);
      }
    for (int j = KEEP * STEP + lane * VN; j < d; j += STEP) {
      float a[VN], b[VN], c[VN]; load_vec<T>(dyr + j, a); load_vec<T>(xr + j, b); load_vec<T>(g + j, c);
#pragma unroll
      for (int i = 0; i < VN; i++) dot += a[i] * b[i] * c[i];
    }
  } else {
    for (int j = lane; j < d; j += AS_WAVE) dot += to_f<T>(dyr[j]) * to_f<T>(xr[j]) * to_f<T>(g[j]);
  }
  dot = wave_sum(dot);
  float k = r * r * r * dot / (float)d;
  if (vec) {
#pragma unroll
    for (int q = 0; q < KEEP; q++) {
      const int j = q * STEP + lane * VN;
      if (j < d) {
        float o[VN];
#pragma unroll
        for (int i = 0; i < VN; i++) o[i] = (ar ? to_f<T>(ka[q][i]) : 0.f) + (r * to_f<T>(kg[q][i]) * to_f<T>(kdy[q][i]) - to_f<T>(kx[q][i]) * k);
        store_vec<T>(dxr + j, o);
      }
    }
    for (int j = KEEP * STEP + lane * VN; j < d; j += STEP) {
      float a[VN], b[VN], c[VN], o[VN]; load_vec<T>(dyr + j, a); load_vec<T>(xr + j, b); load_vec<T>(g + j, c);
      if (ar) load_vec<T>(ar + j, o);
#pragma unroll
      for (int i = 0; i < VN; i++) o[i] = (ar ? o[i] : 0.f) + (r * c[i] * a[i] - b[i] * k);
      store_vec<T>(dxr + j, o);
    }
  } else {
    for (int j = lane; j < d; j += AS_WAVE) {
      float v = r * to_f<T>(g[j]) * to_f<T>(dyr[j]) - to_f<T>(xr[j]) * k;
      dxr[j] = from_f<T>((ar ? to_f<T>(ar[j]) : 0.f) + v);
    }
  }
}

int launch_rmsnorm_bwd(as_ctx* ctx, int mode, int n, int d, const void* dy, const int32_t* src_pos,
                       const void* x, const void* g, const float* rstd, const void* add, void* dx,
                       hipStream_t st) {
  if (n <= 0) return AS_OK;
  prof_begin(ctx, st, AS_K_NORM, 0.0);
  DISPATCH_T(mode, { int vec = vec_ok<T>(dy, d) && vec_ok<T>(x, d) && vec_ok<T>(g, d) && vec_ok<T>(dx, d) &&
                               (!add || vec_ok<T>(add, d));
                     auto k = d <= 4 * AS_WAVE * Vec<T>::N ? rmsnorm_bwd_kernel<T, 4> : rmsnorm_bwd_kernel<T, 8>;
                     k<<<cdiv(n, 4), 256, 0, st>>>(n, d, (const T*)dy, src_pos, (const T*)x, (const T*)g, rstd, (const T*)add, (T*)dx, vec); });
  prof_end(ctx, st);
  AS_LAUNCH_CHECK(ctx);
  return AS_OK;
}

// The same with the gain gradient dg_j = sum_t dy[t,j] x[t,j] rstd[t] out of the same pass over dy and x (full fine-tuning):
// up to 256 workgroups walk the rows, a lane adds up the columns it holds of every row it sees, the waves of a workgroup are
// added in order through LDS into partial[workgroup, :], and a second launch adds the workgroups in order.  Bound by memory (dy, x,
// add in, dx out).  8 waves with KEEP = 4 (2048 16-bit columns), 4 with KEEP = 8: the registers for a row's three operands and the column sums.
// Twice as many waves spilled 40 and 92 registers, the column sums among them, to scratch memory for every row: 13,800 rows of 2048, bf16, 71 us
// where this takes 43 (5.2 TB/s).  As three launches (backward, a second pass over dy and x, a sum of 256 slabs by one thread per column) it was
// 130 us against 77 with the spills and the sum.
template <typename T, int KEEP>
__global__ __launch_bounds__(2048 / KEEP) void rmsnorm_bwd_gain_kernel(int n, int d, const T* __restrict__ dy, const int32_t* __restrict__ src_pos,
                                                               const T* __restrict__ x, const T* __restrict__ g, const float* __restrict__ rstd,
                                                               const T* __restrict__ add, T* __restrict__ dx, float* __restrict__ partial) {
  constexpr int VN = Vec<T>::N, STEP = AS_WAVE * VN, NW = 32 / KEEP;
  typedef typename Vec<T>::type VT;
  extern __shared__ __align__(16) float gsum[];          // [d]
  const int lane = threadIdx.x % AS_WAVE, wave = threadIdx.x / AS_WAVE;
  float acc[KEEP][VN];
#pragma unroll
  for (int q = 0; q < KEEP; q++)
#pragma unroll
    for (int i = 0; i < VN; i++) acc[q][i] = 0.f;
  for (int64_t row = (int64_t)blockIdx.x * NW + wave; row < n; row += (int64_t)gridDim.x * NW) {
    const int64_t src = src_pos ? src_pos[row] : row;
    T* dxr = dx + row * d;
    const T* ar = add ? add + row * d : nullptr;
    if (src < 0) {                                       // no upstream gradient for this row
#pragma unroll
      for (int q = 0; q < KEEP; q++) {
        const int j = q * STEP + lane * VN;
        if (j < d) {
          float o[VN];
#pragma unroll
          for (int i = 0; i < VN; i++) o[i] = 0.f;
          if (ar) load_vec<T>(ar + j, o);
          store_vec<T>(dxr + j, o);
        }
      }
      continue;
    }
    const T* dyr = dy + src * d; const T* xr = x + row * d;
    const float r = rstd[src_pos ? src : row];
    VT kdy[KEEP], kx[KEEP], ka[KEEP];
#pragma unroll
    for (int q = 0; q < KEEP; q++) {
      const int j = q * STEP + lane * VN;
      if (j < d) {
        kdy[q] = *reinterpret_cast<const VT*>(dyr + j); kx[q] = *reinterpret_cast<const VT*>(xr + j);
        if (ar) ka[q] = *reinterpret_cast<const VT*>(ar + j);
      }
    }
    float dot = 0.f;
#pragma unroll
    for (int q = 0; q < KEEP; q++) {
      const int j = q * STEP + lane * VN;
      if (j < d) {
        float c[VN]; load_vec<T>(g + j, c);
#pragma unroll
        for (int i = 0; i < VN; i++) {
          const float p = to_f<T>(kdy[q][i]) * to_f<T>(kx[q][i]);
          dot += p * c[i]; acc[q][i] += p * r;
        }
      }
    }
    dot = wave_sum(dot);
    const float k = r * r * r * dot / (float)d;
#pragma unroll
    for (int q = 0; q < KEEP; q++) {
      const int j = q * STEP + lane * VN;
      if (j < d) {
        float c[VN], o[VN]; load_vec<T>(g + j, c);
#pragma unroll
        for (int i = 0; i < VN; i++) o[i] = (ar ? to_f<T>(ka[q][i]) : 0.f) + (r * c[i] * to_f<T>(kdy[q][i]) - to_f<T>(kx[q][i]) * k);
        store_vec<T>(dxr + j, o);
      }
    }
  }
  for (int w = 0; w < NW; w++) {
    if (wave == w) {
#pragma unroll
      for (int q = 0; q < KEEP; q++) {
        const int j = q * STEP + lane * VN;
        if (j < d) {
#pragma unroll
          for (int i = 0; i < VN; i++) gsum[j + i] = (w ? gsum[j + i] : 0.f) + acc[q][i];
        }
      }
    }
    __syncthreads();
  }
  for (int j = threadIdx.x; j < d; j += NW * AS_WAVE) partial[(int64_t)blockIdx.x * d + j] = gsum[j];
}

// Gain gradient alone (rows the kernel above does not take): each block sums a slab of rows into partial[block, :].
template <typename T>
__global__ void rmsnorm_dgain_part(int n, int d, const T* __restrict__ dy, const int32_t* __restrict__ src_pos,
                                   const T* __restrict__ x, const float* __restrict__ rstd,
                                   float* __restrict__ partial, int rows_per) {
  int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= d) return;
  int r0 = blockIdx.y * rows_per, r1 = min(n, r0 + rows_per);
  float acc = 0.f;
  for (int t = r0; t < r1; t++) {
    int64_t src = src_pos ? src_pos[t] : t;
    if (src < 0) continue;
    acc += to_f<T>(dy[src * d + j]) * to_f<T>(x[(int64_t)t * d + j]) * rstd[src_pos ? src : t];
  }
  partial[(int64_t)blockIdx.y * d + j] = acc;
}
// out[j] = sum over the slabs: 32 columns per workgroup, eight threads per column with every eighth slab each, added in order
__global__ __launch_bounds__(256) void sum_partials_kernel(const float* __restrict__ partial, int n_part, int64_t len, float* __restrict__ out) {
  __shared__ float sh[8][32];
  const int c = threadIdx.x & 31, k = threadIdx.x >> 5;
  const int64_t j = (int64_t)blockIdx.x * 32 + c;
  float acc = 0.f;
  if (j < len) {
#pragma unroll 8
    for (int p = k; p < n_part; p += 8) acc += partial[(int64_t)p * len + j];
  }
  sh[k][c] = acc;
  __syncthreads();
  if (k == 0 && j < len) {
    for (int i = 1; i < 8; i++) acc += sh[i][c];
    out[j] = acc;
  }
}

int launch_rmsnorm_bwd_gain(as_ctx* ctx, int mode, int n, int d, const void* dy, const int32_t* src_pos, const void* x, const void* g,
                            const float* rstd, const void* add, void* dx, float* partial, int n_part, float* dg, hipStream_t st) {
  if (n <= 0 || n_part <= 0) return AS_OK;
  bool fused = false;
  DISPATCH_T(mode, fused = d <= 8 * AS_WAVE * Vec<T>::N && vec_ok<T>(dy, d) && vec_ok<T>(x, d) && vec_ok<T>(g, d) && vec_ok<T>(dx, d) && (!add || vec_ok<T>(add, d)););
  prof_begin(ctx, st, AS_K_NORM, 0.0);
  if (fused) {
    DISPATCH_T(mode, {
      const bool small = d <= 4 * AS_WAVE * Vec<T>::N;
      n_part = (int)std::min<int64_t>(n_part, cdiv(n, small ? 8 : 4));
      if (small) rmsnorm_bwd_gain_kernel<T, 4><<<n_part, 512, (size_t)d * 4, st>>>(n, d, (const T*)dy, src_pos, (const T*)x, (const T*)g, rstd, (const T*)add, (T*)dx, partial);
      else rmsnorm_bwd_gain_kernel<T, 8><<<n_part, 256, (size_t)d * 4, st>>>(n, d, (const T*)dy, src_pos, (const T*)x, (const T*)g, rstd, (const T*)add, (T*)dx, partial); });
  } else {
    int rc = launch_rmsnorm_bwd(ctx, mode, n, d, dy, src_pos, x, g, rstd, add, dx, st);
    if (rc) return rc;
    DISPATCH_T(mode, (rmsnorm_dgain_part<T><<<dim3(cdiv(d, 256), n_part), 256, 0, st>>>(n, d, (const T*)dy, src_pos, (const T*)x, rstd, partial, (int)cdiv(n, n_part))));
  }
  AS_LAUNCH_CHECK(ctx);
  sum_partials_kernel<<<(unsigned)cdiv(d, 32), 256, 0, st>>>(partial, n_part, d, dg);
  prof_end(ctx, st);
  AS_LAUNCH_CHECK(ctx);
  return AS_OK;
}

// ------------------------------------------------------------------ SwiGLU
// gu holds [gate | up] side by side, row length 2F.  The divisions are exact ones: the reciprocal instruction is a unit of the last place off and
// loses gates under -87.3, where 1 + exp(-gate) passes 2^126, altogether.
__device__ __forceinline__ float sigmoid(float a) { return 1.f / (1.f + __expf(-a)); }
__device__ __forceinline__ float silu_times(float a, float b) { return a / (1.f + __expf(-a)) * b; }
template <typename T>
__global__ void swiglu_fwd_kernel(int64_t n, int F, const T* __restrict__ gu, T* __restrict__ m, int vec) {
  constexpr int VN = Vec<T>::N;
  int64_t per_row = vec ? F / VN : F;
  int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= n * per_row) return;
  int64_t t = idx / per_row; int j = (idx % per_row) * (vec ? VN : 1);
  const T* gr = gu + t * 2 * F;
  if (vec) {
    float a[VN], b[VN], o[VN]; load_vec<T>(gr + j, a); load_vec<T>(gr + F + j, b);
#pragma unroll
    for (int i = 0; i < VN; i++) o[i] = silu_times(a[i], b[i]);
    store_vec<T>(m + t * F + j, o);
  } else {
    float a = to_f<T>(gr[j]), b = to_f<T>(gr[F + j]);
    m[t * F + j] = from_f<T>(silu_times(a, b));
  }
}

template <typename T>
__global__ void swiglu_bwd_kernel(int64_t n, int F, const T* __restrict__ dm, const T* __restrict__ gu,
                                  T* __restrict__ dgu, T* __restrict__ m_out, int vec) {
  constexpr int VN = Vec<T>::N;
  int64_t per_row = vec ? F / VN : F;
  int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= n * per_row) return;
  int64_t t = idx / per_row; int j = (idx % per_row) * (vec ? VN : 1);
  const T* gr = gu + t * 2 * F;
  T* dr = dgu + t * 2 * F;
  if (vec) {
    float a[VN], b[VN], c[VN], og[VN], ou[VN];
    load_vec<T>(gr + j, a); load_vec<T>(gr + F + j, b); load_vec<T>(dm + t * F + j, c);
#pragma unroll
    for (int i = 0; i < VN; i++) {
      const float sg = sigmoid(a[i]);
      og[i] = c[i] * b[i] * sg * (1.f + a[i] * (1.f - sg));
      ou[i] = c[i] * a[i] * sg;
    }
    store_vec<T>(dr + j, og); store_vec<T>(dr + F + j, ou);
    if (m_out) {                                       // the forward product again, in the forward kernel's arithmetic
      float o[VN];
#pragma unroll
      for (int i = 0; i < VN; i++) o[i] = silu_times(a[i], b[i]);
      store_vec<T>(m_out + t * F + j, o);
    }
  } else {
    float a = to_f<T>(gr[j]), b = to_f<T>(gr[F + j]), c = to_f<T>(dm[t * F + j]);
    const float sg = sigmoid(a);
    dr[j] = from_f<T>(c * b * sg * (1.f + a * (1.f - sg)));
    dr[F + j] = from_f<T>(c * a * sg);
    if (m_out) m_out[t * F + j] = from_f<T>(silu_times(a, b));
  }
}

int launch_swiglu_fwd(as_ctx* ctx, int mode, int64_t n, int F, const void* gu, void* m, hipStream_t st) {
  if (n <= 0) return AS_OK;
  prof_begin(ctx, st, AS_K_SWIGLU, 0.0);
  DISPATCH_T(mode, { int vec = vec_ok<T>(gu, F) && vec_ok<T>(m, F);
                     int64_t tot = n * (vec ? F / Vec<T>::N : F);
                     swiglu_fwd_kernel<T><<<cdiv(tot, 256), 256, 0, st>>>(n, F, (const T*)gu, (T*)m, vec); });
  prof_end(ctx, st);
  AS_LAUNCH_CHECK(ctx);
  return AS_OK;
}
// m_out (may be NULL): also writes silu(gate) * up, bit for bit what launch_swiglu_fwd writes
int launch_swiglu_bwd(as_ctx* ctx, int mode, int64_t n, int F, const void* dm, const void* gu, void* dgu, void* m_out, hipStream_t st) {
  if (n <= 0) return AS_OK;
  prof_begin(ctx, st, AS_K_SWIGLU, 0.0);
  DISPATCH_T(mode, { int vec = vec_ok<T>(gu, F) && vec_ok<T>(dm, F) && vec_ok<T>(dgu, F) && (!m_out || vec_ok<T>(m_out, F));
                     int64_t tot = n * (vec ? F / Vec<T>::N : F);
                     swiglu_bwd_kernel<T><<<cdiv(tot, 256), 256, 0, st>>>(n, F, (const T*)dm, (const T*)gu, (T*)dgu, (T*)m_out, vec); });
  prof_end(ctx, st);
  AS_LAUNCH_CHECK(ctx);
  return AS_OK;
}

// SwiGLU and the adapter products that read its result, in one pass (bf16, rank up to 16): u = m A^T forward (down's adapter), du = dgate Bg
// and dup Bu backward (gate's and up's).  A kernel of their own reads m, or dgate and dup, a second time.  16 tokens per workgroup, its eight
// waves take every eighth 64 columns, the next step's operands on their way.  Loads and stores are eight lanes to 128 bytes of a row
// (neighbouring lanes in different rows, the product's own operand layout, cost a clock a lane: 590 us where this takes 457); the
// rounded result passes through 2 KB of the wave's LDS into that layout, the adapter comes from L2 in it (PrepMatrix::frag), the waves' sums meet at the end.
// 24,710 tokens x 8192: forward 262 us, 307 as two kernels (5.2 TB/s of what has to move), backward 457 and 539 (4.9); the exact divisions are 2 and 7 of them.  Of rank 64, on 14336
// columns, it takes 270 + 524 us where the kernels one after the other take 262 + 515 (the adapter's rows are then four times the traffic from L2).
// Under one workgroup per CU (sixteen waves each: 626 tokens, a step of two layers 1.420 ms, 1.412 with two kernels) the rows stay with two kernels.
struct SwigluAdapter { const bf16_t* frag[2]; int rp; bf16_t* u; };        // frag: A of down forward; B of gate, of up backward
constexpr int kSwigluRank = 16, kSwigluTokens = 16 * 256;
template <bool BWD>
__global__ __launch_bounds__(512) void swiglu_adapter_kernel(int n, int F, const bf16_t* __restrict__ dm, const bf16_t* __restrict__ gu, bf16_t* __restrict__ dgu,
                                                                 bf16_t* __restrict__ m, const SwigluAdapter ad) {
  constexpr int MT = BWD ? 2 : 1, NW = 8;                  // products, waves
  __shared__ __align__(16) unsigned char smem[NW * MT * 2048];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l15 = lane & 15, q = lane >> 4, r8 = lane >> 3, ch = lane & 7;
  const int row0 = blockIdx.x * 16;
  unsigned char* my = smem + wave * (MT * 2048);
  f32x4 acc[MT] = {};
  struct Operands { bf16x8 g[2], x[2], z[2]; };
  auto load = [&](int c, Operands& v) {
#pragma unroll
    for (int h = 0; h < 2; h++) {
      const int64_t row = min(row0 + 8 * h + r8, n - 1);
      const bf16_t* gr = gu + row * 2 * F + c + ch * 8;
      v.g[h] = *reinterpret_cast<const bf16x8*>(gr); v.x[h] = *reinterpret_cast<const bf16x8*>(gr + F);
      if (BWD) v.z[h] = *reinterpret_cast<const bf16x8*>(dm + row * F + c + ch * 8);
    }
  };
  auto step = [&](int c, const Operands& v) {
    bf16x8 w[MT][2];
#pragma unroll
    for (int p = 0; p < MT; p++)
#pragma unroll
      for (int k = 0; k < 2; k++) w[p][k] = *reinterpret_cast<const bf16x8*>(ad.frag[p] + (int64_t)(c / 32 + k) * 512 + lane * 8);
#pragma unroll
    for (int h = 0; h < 2; h++) {
      const int row = row0 + 8 * h + r8;
      const bool mine = row < n;
      bf16x8 y[MT], mo;
#pragma unroll
      for (int i = 0; i < 8; i++) {
        const float a = (float)v.g[h][i], b = (float)v.x[h][i];
        if (BWD) {
          const float d = (float)v.z[h][i], sg = sigmoid(a);
          y[0][i] = (bf16_t)(d * b * sg * (1.f + a * (1.f - sg)));
          y[MT - 1][i] = (bf16_t)(d * a * sg);
          if (m) mo[i] = (bf16_t)silu_times(a, b);         // the forward product again, in the forward kernel's arithmetic
        } else y[0][i] = (bf16_t)silu_times(a, b);
      }
      if (mine) {
        if (BWD) {
          bf16_t* o = dgu + (int64_t)row * 2 * F + c + ch * 8;
          *reinterpret_cast<bf16x8*>(o) = y[0]; *reinterpret_cast<bf16x8*>(o + F) = y[MT - 1];
          if (m) *reinterpret_cast<bf16x8*>(m + (int64_t)row * F + c + ch * 8) = mo;
        } else *reinterpret_cast<bf16x8*>(m + (int64_t)row * F + c + ch * 8) = y[0];
      }
#pragma unroll
      for (int p = 0; p < MT; p++) *reinterpret_cast<bf16x8*>(my + p * 2048 + (h * 8 + r8) * 128 + ((ch ^ r8) * 16)) = y[p];
    }
    asm volatile("" ::: "memory");                         // LDS operations of a wave complete in order
#pragma unroll
    for (int p = 0; p < MT; p++)
#pragma unroll
      for (int k = 0; k < 2; k++) {
        const bf16x8 a = *reinterpret_cast<const bf16x8*>(my + p * 2048 + l15 * 128 + (((k * 4 + q) ^ (l15 & 7)) * 16));
        acc[p] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, w[p][k], acc[p], 0, 0, 0);
      }
    asm volatile("" ::: "memory");
  };
  const int steps = F / 64;
  int s = wave;
  Operands v0, v1;
  if (s < steps) load(s * 64, v0);
  for (; s + NW < steps; s += 2 * NW) {
    load((s + NW) * 64, v1);
    step(s * 64, v0);
    if (s + 2 * NW < steps) load((s + 2 * NW) * 64, v0);
    step((s + NW) * 64, v1);
  }
  if (s < steps) step(s * 64, v0);
  // the waves' sums in wave order to u [rows, MT rp]; columns past 16 are zero
  f32x4 (*red)[MT][64] = reinterpret_cast<f32x4 (*)[MT][64]>(smem);
  __syncthreads();
#pragma unroll
  for (int p = 0; p < MT; p++) red[wave][p][lane] = acc[p];
  __syncthreads();
  for (int o = threadIdx.x; o < 16 * MT * ad.rp; o += 64 * NW) {           // token t is element t % 4 of lane 16 (t / 4) + rank index
    const int t = o / (MT * ad.rp), p = o / ad.rp % MT, j = o % ad.rp;
    float v = 0.f;
    if (j < 16)
      for (int w = 0; w < NW; w++) v += red[w][p][(t >> 2) * 16 + j][t & 3];
    if (row0 + t < n) ad.u[(int64_t)(row0 + t) * (MT * ad.rp) + p * ad.rp + j] = (bf16_t)v;
  }
}
// Products of token rows with adapters of rank up to 16, in the same manner: u = x A^T, du = dY B.  NB adapters on one x (q, k, v; gate, up), or (NB = 1) up
// to three of their own, one per blockIdx.y.  Columns past 16 of an adapter's rp are written as zeros.
// As narrow GEMMs through LDS tiles (64 columns computed for 16, the sum of a split contraction a second launch) the products of two 1B layers took 432 us at
// 24,710 tokens and 206 at 626; 300 and 103 so (24,710 x 2048: 24 us, 4.3 TB/s of the rows).  Steps: 626 tokens 1.292 -> 1.215 ms, 24,710 15.25 -> 15.10.
template <int NB, int NW>
__global__ __launch_bounds__(64 * NW) void adapter_rows_kernel(const AdapterRows p) {
  __shared__ __align__(16) unsigned char smem[NW * (NB > 2 ? NB * 1024 : 2048)];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l15 = lane & 15, q = lane >> 4, r8 = lane >> 3, ch = lane & 7;
  const int item = blockIdx.y, row0 = blockIdx.x * 16;
  const bf16_t* x = (const bf16_t*)(item == 0 ? p.x[0] : item == 1 ? p.x[1] : p.x[2]);
  const bf16_t* f0 = (const bf16_t*)(item == 0 ? p.frag[0] : item == 1 ? p.frag[1] : p.frag[2]);
  const int steps = (item == 0 ? p.K[0] : item == 1 ? p.K[1] : p.K[2]) / 64;
  const bf16_t* xr[2];
#pragma unroll
  for (int h = 0; h < 2; h++) xr[h] = x + (int64_t)min(row0 + 8 * h + r8, p.n - 1) * p.ldx + ch * 8;
  unsigned char* my = smem + wave * 2048;
  f32x4 acc[NB] = {};
  constexpr int AHEAD = 2;                                 // steps whose operands are under way
  struct Operands { bf16x8 x[2], w[NB][2]; };
  auto load = [&](int s, Operands& v) {
#pragma unroll
    for (int h = 0; h < 2; h++) v.x[h] = *reinterpret_cast<const bf16x8*>(xr[h] + s * 64);
#pragma unroll
    for (int b = 0; b < NB; b++)
#pragma unroll
      for (int k = 0; k < 2; k++) v.w[b][k] = *reinterpret_cast<const bf16x8*>((b == 0 ? f0 : (const bf16_t*)p.frag[b]) + (int64_t)(2 * s + k) * 512 + lane * 8);
  };
  auto step = [&](const Operands& v) {
#pragma unroll
    for (int h = 0; h < 2; h++) *reinterpret_cast<bf16x8*>(my + (h * 8 + r8) * 128 + ((ch ^ r8) * 16)) = v.x[h];
    asm volatile("" ::: "memory");                         // LDS operations of a wave complete in order
#pragma unroll
    for (int k = 0; k < 2; k++) {
      const bf16x8 a = *reinterpret_cast<const bf16x8*>(my + l15 * 128 + (((k * 4 + q) ^ (l15 & 7)) * 16));
#pragma unroll
      for (int b = 0; b < NB; b++) acc[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, v.w[b][k], acc[b], 0, 0, 0);
    }
    asm volatile("" ::: "memory");
  };
  Operands v[AHEAD];
  int s = wave;
#pragma unroll
  for (int i = 0; i < AHEAD; i++) if (s + i * NW < steps) load(s + i * NW, v[i]);
  for (; s < steps; s += AHEAD * NW) {
#pragma unroll
    for (int i = 0; i < AHEAD; i++)
      if (s + i * NW < steps) {
        step(v[i]);
        if (s + (i + AHEAD) * NW < steps) load(s + (i + AHEAD) * NW, v[i]);
      }
  }
  // the waves' sums in wave order
  f32x4 (*red)[NB][64] = reinterpret_cast<f32x4 (*)[NB][64]>(smem);
  __syncthreads();
#pragma unroll
  for (int b = 0; b < NB; b++) red[wave][b][lane] = acc[b];
  __syncthreads();
  for (int o = threadIdx.x; o < 16 * NB * p.rp; o += 64 * NW) {             // token t is element t % 4 of lane 16 (t / 4) + rank index
    const int t = o / (NB * p.rp), b = o / p.rp % NB, j = o % p.rp;
    float sum = 0.f;
    if (j < 16)
      for (int w = 0; w < NW; w++) sum += red[w][b][(t >> 2) * 16 + j][t & 3];
    bf16_t* u = (bf16_t*)(NB == 1 ? (item == 0 ? p.u[0] : item == 1 ? p.u[1] : p.u[2]) : b == 0 ? p.u[0] : b == 1 ? p.u[1] : p.u[2]);
    if (row0 + t < p.n) u[(int64_t)(row0 + t) * p.ldu + j] = (bf16_t)sum;
  }
}
bool adapter_rows_ok(int mode, int r, int64_t ldx, std::initializer_list<const void*> ptrs) {
  uintptr_t x = 0;
  for (const void* p : ptrs) x |= (uintptr_t)p;
  return mode == AS_BF16 && r <= kSwigluRank && ldx % 8 == 0 && x % 16 == 0;
}
int launch_adapter_rows(as_ctx* ctx, const AdapterRows& p, int items, bool one_x, hipStream_t st) {
  if (p.n <= 0 || items < 1) return AS_OK;
  const dim3 g((unsigned)cdiv(p.n, 16), one_x ? 1 : items);
  const bool wide = (int64_t)g.x * g.y < 512;              // under two workgroups of eight waves a CU: sixteen
  double flops = 0;
  for (int i = 0; i < items; i++) flops += 2.0 * p.n * 16 * p.K[one_x ? 0 : i];
  auto go = [&](auto nb) { if (wide) adapter_rows_kernel<nb(), 16><<<g, 1024, 0, st>>>(p); else adapter_rows_kernel<nb(), 8><<<g, 512, 0, st>>>(p); };
  prof_begin(ctx, st, AS_K_GEMM_MFMA_SKINNY, flops);
  if (!one_x || items == 1) go(std::integral_constant<int, 1>());
  else if (items == 2) go(std::integral_constant<int, 2>());
  else go(std::integral_constant<int, 3>());
  prof_end(ctx, st);
  AS_LAUNCH_CHECK(ctx);
  return AS_OK;
}

bool swiglu_adapter_ok(int mode, int n, int F, int r, std::initializer_list<const void*> ptrs) {
  uintptr_t x = 0;
  for (const void* p : ptrs) x |= (uintptr_t)p;
  return mode == AS_BF16 && n >= kSwigluTokens && F % 64 == 0 && r <= kSwigluRank && x % 16 == 0;
}
template <bool BWD>
static int launch_swiglu_adapter(as_ctx* ctx, int n, int F, const void* dm, const void* gu, void* dgu, void* m, const SwigluAdapter& ad, hipStream_t st) {
  if (n <= 0) return AS_OK;
  prof_begin(ctx, st, AS_K_SWIGLU, 0.0);
  swiglu_adapter_kernel<BWD><<<(unsigned)cdiv(n, 16), 512, 0, st>>>(n, F, (const bf16_t*)dm, (const bf16_t*)gu, (bf16_t*)dgu, (bf16_t*)m, ad);
  prof_end(ctx, st);
  AS_LAUNCH_CHECK(ctx);
  return AS_OK;
}
int launch_swiglu_fwd_adapter(as_ctx* ctx, int n, int F, const void* gu, void* m, const void* fragA, int rp, void* u, hipStream_t st) {
  return launch_swiglu_adapter<false>(ctx, n, F, nullptr, gu, nullptr, m, SwigluAdapter{{(const bf16_t*)fragA, nullptr}, rp, (bf16_t*)u}, st);
}
int launch_swiglu_bwd_adapter(as_ctx* ctx, int n, int F, const void* dm, const void* gu, void* dgu, void* m_out, const void* fragBg, const void* fragBu, int rp, void* du,
                              hipStream_t st) {
  return launch_swiglu_adapter<true>(ctx, n, F, dm, gu, dgu, m_out, SwigluAdapter{{(const bf16_t*)fragBg, (const bf16_t*)fragBu}, rp, (bf16_t*)du}, st);
}

// --------------------------------------------------------------- transpose
// out[c, r] = in[r, c] through a padded LDS tile; rows past the
// device-side row count (if given) read as zero.
// QS: inside every group of 16 output positions the two middle quads are exchanged (position order
// 0-3, 8-11, 4-7, 12-15 of the source rows), which is the order one lane half of a 32x32x16 MFMA
// holds its 8 contraction indices in: such a fragment is then one 16-byte read.
// 32 x 32 tiles, four elements per thread in flight: what comes here is small (fp32 tier) or oddly shaped.
template <typename T, bool QS>
__global__ __launch_bounds__(256) void transpose_kernel(int rows, int rows_pad, int cols, const T* __restrict__ in, int64_t ldi,
                                                        T* __restrict__ out, int64_t ldo, const int* __restrict__ rows_dev, int row_off) {
  __shared__ T tile[32][33];
  const int live = rows_dev ? min(rows, *rows_dev - row_off) : rows;
  const int r0 = blockIdx.y * 32, c0 = blockIdx.x * 32, tx = threadIdx.x % 32, ty = threadIdx.x / 32;
  T v[4];
#pragma unroll
  for (int i = 0; i < 4; i++) {
    const int r = r0 + ty + 8 * i, c = c0 + tx;
    v[i] = (r < live && c < cols) ? in[(int64_t)r * ldi + c] : from_f<T>(0.f);
  }
#pragma unroll
  for (int i = 0; i < 4; i++) tile[ty + 8 * i][tx] = v[i];
  __syncthreads();
  const int src = QS ? ((tx & ~12) | ((tx & 4) << 1) | ((tx & 8) >> 1)) : tx;
#pragma unroll
  for (int i = 0; i < 4; i++) {
    const int c = c0 + ty + 8 * i, r = r0 + tx;
    if (c < cols && r < rows_pad) out[(int64_t)c * ldo + r] = tile[src][ty + 8 * i];
  }
}

// bf16, 16-byte accesses on both sides, through registers: a lane reads eight rows of eight elements, turns the 8 x 8 block
// with byte permutes (dword k of output row c is the pair of elements c of rows 2 k and 2 k + 1) and writes eight rows of
// eight.  The lanes of a wave lie 8 x 8, so that every access of a wave is eight whole 128-byte lines, in and out; no LDS,
// no barrier, eight loads in flight per lane.  Memory bound: one read and one write of the matrix.  Through an LDS tile
// (eight 2-byte reads per output vector) the expert matrices of a sparse layer took 1693 us, 1407 us so (4.4 TB/s); the copies of a
// 1B layer's weight gradients 1371 and 712 us (4.9 TB/s).
// QS: the lane of an even output chunk takes source rows 0-3 and 8-11 of its 16, that of an odd one the others.
// Needs cols, ldi, ldo and rows_pad multiples of 8 (QS: rows_pad of 16) and 16-byte aligned bases.
// grid.z = 2: a second matrix of the same shape and strides (in2 -> out2).
template <bool QS>
__global__ __launch_bounds__(256) void transpose_vec_kernel(int rows, int rows_pad, int cols, const bf16_t* __restrict__ in, int64_t ldi,
                                                            bf16_t* __restrict__ out, int64_t ldo, const int* __restrict__ rows_dev, int row_off,
                                                            const bf16_t* __restrict__ in2, bf16_t* __restrict__ out2) {
  if (blockIdx.z) { in = in2; out = out2; }
  typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
  const int live = rows_dev ? min(rows, *rows_dev - row_off) : rows;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int c0 = blockIdx.x * 64, r0 = (blockIdx.y * 4 + wave) * 64;
  // reading, neighbouring lanes are neighbouring column blocks; the result is written in the same arrangement: lanes of equal
  // column block write one output row each of eight, 16 bytes apart along it
  const int cb = lane & 7, rbk = lane >> 3;
  const int c = c0 + cb * 8, ro = r0 + rbk * 8;            // output rows c .. c + 7, positions ro .. ro + 7
  if (c >= cols || ro >= rows_pad) return;
  const int rs = QS ? r0 + (rbk >> 1) * 16 + (rbk & 1) * 4 : ro;                        // first source row; QS: rows rs .. + 3 and rs + 8 .. + 11
  const bf16_t* src = in + (int64_t)rs * ldi + c;
  u32x4 v[8];
#pragma unroll
  for (int i = 0; i < 8; i++) {
    const int o = QS ? (i & 3) + (i >> 2) * 8 : i;
    v[i] = (u32x4){0u, 0u, 0u, 0u};
    if (rs + o < live) v[i] = *reinterpret_cast<const u32x4*>(src + (int64_t)o * ldi);
  }
  bf16_t* dst = out + (int64_t)c * ldo + ro;
#pragma unroll
  for (int q = 0; q < 8; q++) {
    u32x4 w;
#pragma unroll
    for (int k = 0; k < 4; k++) w[k] = __builtin_amdgcn_perm(v[2 * k + 1][q >> 1], v[2 * k][q >> 1], (q & 1) ? 0x07060302u : 0x05040100u);
    *reinterpret_cast<u32x4*>(dst + (int64_t)q * ldo) = w;
  }
}

static bool transpose_vec_ok(int mode, int rows_pad, int cols, const void* in, int64_t ldi, const void* out, int64_t ldo) {
  return mode == AS_BF16 && rows_pad % 8 == 0 && cols % 8 == 0 && ldi % 8 == 0 && ldo % 8 == 0 &&
         (uintptr_t)in % 16 == 0 && (uintptr_t)out % 16 == 0;
}

int launch_transpose(as_ctx* ctx, int mode, int rows, int rows_pad, int cols, const void* in, int64_t ldi, void* out,
                     int64_t ldo, const int* rows_dev, int row_off, hipStream_t st) {
  if (rows <= 0 || cols <= 0) return AS_OK;
  dim3 grid(cdiv(cols, 32), cdiv(rows_pad, 32));
  prof_begin(ctx, st, AS_K_TRANSPOSE, 0.0);
  if (transpose_vec_ok(mode, rows_pad, cols, in, ldi, out, ldo))
    transpose_vec_kernel<false><<<dim3((unsigned)cdiv(cols, 64), (unsigned)cdiv(rows_pad, 256)), 256, 0, st>>>(rows, rows_pad, cols, (const bf16_t*)in, ldi, (bf16_t*)out, ldo, rows_dev, row_off, nullptr, nullptr);
  else
  DISPATCH_T(mode, (transpose_kernel<T, false><<<grid, 256, 0, st>>>(rows, rows_pad, cols, (const T*)in, ldi, (T*)out, ldo, rows_dev, row_off)));
  prof_end(ctx, st);
  AS_LAUNCH_CHECK(ctx);
  return AS_OK;
}

int launch_transpose_pair(as_ctx* ctx, int mode, int rows, int rows_pad, int cols, const void* in, const void* in2, int64_t ldi,
                          void* out, void* out2, int64_t ldo, hipStream_t st) {
  if (rows <= 0 || cols <= 0) return AS_OK;
  if (transpose_vec_ok(mode, rows_pad, cols, in, ldi, out, ldo) && transpose_vec_ok(mode, rows_pad, cols, in2, ldi, out2, ldo)) {
    prof_begin(ctx, st, AS_K_TRANSPOSE, 0.0);
    transpose_vec_kernel<false><<<dim3((unsigned)cdiv(cols, 64), (unsigned)cdiv(rows_pad, 256), 2), 256, 0, st>>>(
        rows, rows_pad, cols, (const bf16_t*)in, ldi, (bf16_t*)out, ldo, nullptr, 0, (const bf16_t*)in2, (bf16_t*)out2);
    prof_end(ctx, st);
    AS_LAUNCH_CHECK(ctx);
    return AS_OK;
  }
  const int rc = launch_transpose(ctx, mode, rows, rows_pad, cols, in, ldi, out, ldo, nullptr, 0, st);
  return rc ? rc : launch_transpose(ctx, mode, rows, rows_pad, cols, in2, ldi, out2, ldo, nullptr, 0, st);
}

// the quad-swapped variant (rows_pad must be a multiple of 16)
int launch_transpose_qs(as_ctx* ctx, int mode, int rows, int rows_pad, int cols, const void* in, int64_t ldi, void* out,
                        int64_t ldo, hipStream_t st) {
  if (rows <= 0 || cols <= 0) return AS_OK;
  if (rows_pad % 16) return as_fail(ctx, AS_ERR_SHAPE, "transpose: the quad-swapped layout needs a row count padded to 16");
  dim3 grid(cdiv(cols, 32), cdiv(rows_pad, 32));
  prof_begin(ctx, st, AS_K_TRANSPOSE, 0.0);
  if (transpose_vec_ok(mode, rows_pad, cols, in, ldi, out, ldo))
    transpose_vec_kernel<true><<<dim3((unsigned)cdiv(cols, 64), (unsigned)cdiv(rows_pad, 256)), 256, 0, st>>>(rows, rows_pad, cols, (const bf16_t*)in, ldi, (bf16_t*)out, ldo, nullptr, 0, nullptr, nullptr);
  else
  DISPATCH_T(mode, (transpose_kernel<T, true><<<grid, 256, 0, st>>>(rows, rows_pad, cols, (const T*)in, ldi, (T*)out, ldo, nullptr, 0)));
  prof_end(ctx, st);
  AS_LAUNCH_CHECK(ctx);
  return AS_OK;
}

// ------------------------------------------------------ LoRA operand copies
// out[rp, cp] = scale * in[r, c] inside, 0 in the padding; out_t is its transpose.  Up to kPrepBatch matrices per launch,
// described in the kernel argument; a workgroup takes one 64 x 64 tile of one of them, writes it and, through LDS, its transpose, both in whole row pieces.  One launch per matrix wrote the
// transposes two bytes at a time and took 102 us
// for the 28 matrices of two 1B layers; 17.6 with its loads one after the other, 13.9 so.
struct PrepArgs { PrepMatrix m[kPrepBatch]; int first[kPrepBatch]; };        // first: past the last matrix, past every tile
template <typename T>
__device__ __forceinline__ void lora_prep_tile(const PrepArgs& b, int item, float (&tile)[64][65]) {
  const PrepMatrix& m = b.m[table_item<kPrepBatch>(kPrepBatch, item, [&](int k) { return b.first[k]; })];
  const int tiles_c = (m.cols_pad + 63) / 64, t = item - m.first_tile;
  const int r0 = (t / tiles_c) * 64, c0 = (t % tiles_c) * 64;
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  T* out = (T*)m.out; T* out_t = (T*)m.out_t;
  // every load is made, inside the matrix, before the first value is used: a load under a condition of its own waits for the one before
  float v[16];
#pragma unroll
  for (int i = 0; i < 16; i++) v[i] = m.in[(int64_t)min(r0 + ty + 4 * i, m.rows - 1) * m.cols + min(c0 + tx, m.cols - 1)];
#pragma unroll
  for (int i = 0; i < 16; i++) tile[ty + 4 * i][tx] = r0 + ty + 4 * i < m.rows && c0 + tx < m.cols ? m.scale * v[i] : 0.f;
#pragma unroll
  for (int i = 0; i < 16; i++) {
    const int r = r0 + ty + 4 * i, c = c0 + tx;
    if (r < m.rows_pad && c < m.cols_pad) out[(int64_t)r * m.ldo + c] = from_f<T>(tile[ty + 4 * i][tx]);
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 16; i++) {
    const int c = c0 + ty + 4 * i, r = r0 + tx;
    if (r < m.rows_pad && c < m.cols_pad) out_t[(int64_t)c * m.ldo_t + r] = from_f<T>(tile[tx][ty + 4 * i]);
  }
  const bool by_row = m.frag_rank_rows;
  if (m.frag && (by_row ? r0 : c0) == 0 && threadIdx.x < 128) {            // whole 64 x 64 tiles: two 32-wide chunks of the contraction
    const int lane = threadIdx.x & 63, kc = threadIdx.x >> 6, j = lane & 15, k = kc * 32 + (lane >> 4) * 8;
    T* o = (T*)m.frag + (int64_t)((by_row ? c0 : r0) / 32 + kc) * 512 + lane * 8;
#pragma unroll
    for (int x = 0; x < 8; x++) o[x] = from_f<T>(by_row ? tile[j][k + x] : tile[k + x][j]);
  }
}

template <typename T>
__global__ __launch_bounds__(256) void lora_prep_kernel(const PrepArgs b) {
  __shared__ float tile[64][65];
  lora_prep_tile<T>(b, (int)blockIdx.x, tile);
}
// What a step needs before its first layer, in one launch: nothing in it reads what another part of it writes.  The tiles of the first batch of adapters
// come first (the longest), then segments, rotary table and one workgroup per embedded row.
// What bounds it is the latency of its longest chain: as four launches one after the other 15 us of a 478-token float step and 24 of 626 tokens of two 1B
// layers; steps 267 -> 259 us and 1.169 -> 1.158 ms.
template <typename T>
__global__ __launch_bounds__(256) void step_begin_kernel(const StepBegin s, const PrepArgs b, int tiles, int seg_blocks, int rope_blocks) {
  __shared__ float tile[64][65];
  int block = (int)blockIdx.x;
  if (block < tiles) { lora_prep_tile<T>(b, block, tile); return; }
  block -= tiles;
  if (block < seg_blocks) { segment_info_block(s, block); return; }
  block -= seg_blocks;
  if (block < rope_blocks) { rope_table_block(s, block); return; }
  embed_row<T>(s, block - rope_blocks);
}

static PrepArgs prep_args(const PrepBatch& b) {
  PrepArgs a;
  for (int k = 0; k < kPrepBatch; k++) { a.m[k] = b.m[k < b.n ? k : 0]; a.first[k] = k < b.n ? b.m[k].first_tile : INT32_MAX; }
  return a;
}
int launch_step_begin(as_ctx* ctx, int mode, const StepBegin& s_in, const PrepBatch& b, hipStream_t st) {
  StepBegin s = s_in;
  if (s.n <= 0) return AS_OK;
  const int tiles = b.n > 0 ? b.n_tiles : 0, seg_blocks = (int)cdiv(s.n, kTargetBlock), rope_blocks = (int)cdiv((int64_t)s.max_pos * (s.dh / 2), 256);
  const PrepArgs a = prep_args(b);
  DISPATCH_T(mode, { s.vec = vec_ok<T>(s.embed, s.d) && vec_ok<T>(s.h, s.d);
                     step_begin_kernel<T><<<(unsigned)(tiles + seg_blocks + rope_blocks + s.n), 256, 0, st>>>(s, a, tiles, seg_blocks, rope_blocks); });
  AS_LAUNCH_CHECK(ctx);
  return AS_OK;
}
int launch_lora_prep_batch(as_ctx* ctx, int mode, const PrepBatch& b, hipStream_t st) {
  if (b.n <= 0 || b.n_tiles <= 0) return AS_OK;
  const PrepArgs a = prep_args(b);
  DISPATCH_T(mode, (lora_prep_kernel<T><<<b.n_tiles, 256, 0, st>>>(a)));
  AS_LAUNCH_CHECK(ctx);
  return AS_OK;
}

__global__ void fill_zero_kernel(uint32_t* p, size_t n_words) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  size_t stride = (size_t)gridDim.x * blockDim.x;
  for (; i < n_words; i += stride) p[i] = 0u;
}
int launch_fill_zero(as_ctx* ctx, void* p, size_t bytes, hipStream_t st) {
  size_t w = bytes / 4;                        // callers pass multiples of 4 bytes
  if (!w) return AS_OK;
  int blocks = (int)(cdiv((int64_t)w, 256) < 4096 ? cdiv((int64_t)w, 256) : 4096);
  fill_zero_kernel<<<blocks, 256, 0, st>>>((uint32_t*)p, w);
  AS_LAUNCH_CHECK(ctx);
  return AS_OK;
}

// Rows live .. of two bf16 matrices up to the next multiple of 64 become zero (a contraction over rows runs in steps of 64); live = rows, or
// *n_dev - off within [0, rows].  Column counts are multiples of 8.
__global__ __launch_bounds__(256) void zero_tail_rows_kernel(int rows, const int* n_dev, int off, bf16_t* a, int64_t lda, int ca, bf16_t* b, int64_t ldb, int cb) {
  const int live = n_dev ? min(max(*n_dev - off, 0), rows) : rows, r = live + blockIdx.x;
  if (r >= (live + 63) / 64 * 64) return;
  const uint4 z = make_uint4(0u, 0u, 0u, 0u);
  for (int c = (blockIdx.y * 256 + threadIdx.x) * 8; c < ca; c += gridDim.y * 2048) *reinterpret_cast<uint4*>(a + (int64_t)r * lda + c) = z;
  for (int c = (blockIdx.y * 256 + threadIdx.x) * 8; c < cb; c += gridDim.y * 2048) *reinterpret_cast<uint4*>(b + (int64_t)r * ldb + c) = z;
}
int launch_zero_tail_rows(as_ctx* ctx, int rows, const int* n_dev, int off, void* a, int64_t lda, int ca, void* b, int64_t ldb, int cb, hipStream_t st) {
  if (!n_dev && rows % 64 == 0) return AS_OK;
  zero_tail_rows_kernel<<<dim3(63, (unsigned)std::min<int64_t>(16, cdiv(std::max(ca, cb), 2048))), 256, 0, st>>>(rows, n_dev, off, (bf16_t*)a, lda, ca, (bf16_t*)b, ldb, cb);
  AS_LAUNCH_CHECK(ctx);
  return AS_OK;
}

// ---------------------------------------------------------- target selection
// Stable compaction of the target rows.  A workgroup takes kTargetBlock tokens and adds up the counts of the blocks before it: 24,710 tokens 55 -> 4.7 us
// (one workgroup with a slab of tokens a thread before).
__global__ __launch_bounds__(kTargetBlock) void select_targets_kernel(const int32_t* __restrict__ seg_end, const int32_t* __restrict__ block_targets,
                                                                      const uint8_t* __restrict__ mask, const int32_t* __restrict__ tok, int n,
                                                                      int32_t* __restrict__ tgt_idx, int32_t* __restrict__ tgt_pos, int32_t* __restrict__ labels,
                                                                      int32_t* __restrict__ count) {
  constexpr int WAVES = kTargetBlock / AS_WAVE;
  __shared__ int32_t before[WAVES], mine[WAVES];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, t = blockIdx.x * kTargetBlock + tid;
  int sum = 0;
  for (int b = tid; b < (int)blockIdx.x; b += kTargetBlock) sum += block_targets[b];
  const bool is = t < n && predicts_target(t, seg_end[t], mask);
  const uint64_t set = __ballot(is);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
  if (lane == 0) { before[wave] = sum; mine[wave] = __popcll(set); }
  __syncthreads();
  int base = 0, all = 0;
#pragma unroll
  for (int w = 0; w < WAVES; w++) { base += before[w] + (w < wave ? mine[w] : 0); all += before[w] + mine[w]; }
  if (t < n) {
    const int at = base + __popcll(set & ((1ull << lane) - 1));
    if (is) { tgt_idx[at] = t; labels[at] = tok[t + 1]; }
    tgt_pos[t] = is ? at : -1;
  }
  if (blockIdx.x == gridDim.x - 1 && tid == 0) *count = all;
}

int launch_select_targets(as_ctx* ctx, const int32_t* seg_end, const int32_t* block_targets, const uint8_t* mask, const int32_t* tok,
                          int n, int32_t* tgt_idx, int32_t* tgt_pos, int32_t* labels, int32_t* count,
                          hipStream_t st) {
  if (n <= 0) return AS_OK;
  select_targets_kernel<<<(unsigned)cdiv(n, kTargetBlock), kTargetBlock, 0, st>>>(seg_end, block_targets, mask, tok, n, tgt_idx, tgt_pos, labels, count);
  AS_LAUNCH_CHECK(ctx);
  return AS_OK;
}

// ------------------------------------------------------------ cross-entropy
__device__ __forceinline__ float block_reduce(float v, float* sh, bool is_max) {
  v = is_max ? wave_max(v) : wave_sum(v);
  int w = threadIdx.x / AS_WAVE, nw = blockDim.x / AS_WAVE;
  __syncthreads();
  if (threadIdx.x % AS_WAVE == 0) sh[w] = v;
  __syncthreads();
  float r = sh[0];
  for (int i = 1; i < nw; i++) r = is_max ? fmaxf(r, sh[i]) : r + sh[i];
  return r;
}

// One block per target row of a chunk: logsumexp, the row's loss, and the
// gradient with respect to the logits: (softmax - one-hot) times the row's factor,
// row_w[row] when given, else 1 / target count (the mean loss).  P == nullptr: losses only.
template <typename T>
__global__ void ce_rows_kernel(const float* __restrict__ logits, int V, int row0, const int32_t* __restrict__ labels,
                               const int32_t* __restrict__ count, float* __restrict__ loss_rows,
                               const float* __restrict__ row_w, T* __restrict__ P) {
  __shared__ float sh[16];
  int cnt = *count;
  int row = row0 + blockIdx.x;
  if (row >= cnt) return;
  const float* z = logits + (int64_t)blockIdx.x * V;
  T* p = P + (int64_t)blockIdx.x * V;
  float mx = -INFINITY;
  for (int v = threadIdx.x; v < V; v += blockDim.x) mx = fmaxf(mx, z[v]);
  mx = block_reduce(mx, sh, true);
  float s = 0.f;
  for (int v = threadIdx.x; v < V; v += blockDim.x) s += expf(z[v] - mx);
  s = block_reduce(s, sh, false);
  float lse = mx + logf(s);
  int y = labels[row];
  if (threadIdx.x == 0 && loss_rows) loss_rows[row] = lse - z[y];
  if (!P) return;
  float inv = row_w ? row_w[row] : 1.f / (float)cnt;
  for (int v = threadIdx.x; v < V; v += blockDim.x) {
    float g = expf(z[v] - lse) - (v == y ? 1.f : 0.f);
    p[v] = from_f<T>(g * inv);
  }
}

int launch_ce_rows(as_ctx* ctx, int mode, const float* logits, int rows_cap, int V, int row0,
                   const int32_t* labels, const int32_t* count, float* loss_rows, const float* row_w, void* P, hipStream_t st) {
  if (rows_cap <= 0) return AS_OK;
  prof_begin(ctx, st, AS_K_CE, 0.0);
  DISPATCH_T(mode, (ce_rows_kernel<T><<<rows_cap, 512, 0, st>>>(logits, V, row0, labels, count, loss_rows, row_w, (T*)P)));
  prof_end(ctx, st);
  AS_LAUNCH_CHECK(ctx);
  return AS_OK;
}

// ---- head without stored logits: the two small row kernels around the GEMMs
// z_lab[row] = hf[row] . W[label[row]], one wave per target row (bf16 operands, float sum in a fixed order)
__global__ __launch_bounds__(256) void label_logit_kernel(const bf16_t* __restrict__ hf, const bf16_t* __restrict__ W, int d,
                                                          const int32_t* __restrict__ labels, const int32_t* __restrict__ count,
                                                          float* __restrict__ zlab) {
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (row >= *count) return;
  const bf16_t* a = hf + (int64_t)row * d; const bf16_t* b = W + (int64_t)labels[row] * d;
  float acc = 0.f;
  for (int c = lane * 8; c < d; c += 512) {
    const bf16x8 x = *reinterpret_cast<const bf16x8*>(a + c), y = *reinterpret_cast<const bf16x8*>(b + c);
#pragma unroll
    for (int k = 0; k < 8; k++) acc = fmaf((float)x[k], (float)y[k], acc);
  }
  acc = wave_sum(acc);
  if (lane == 0) zlab[row] = acc;
}
int launch_label_logit(as_ctx* ctx, const void* hf, const void* W, int d, const int32_t* labels, const int32_t* count, int rows_cap,
                       float* zlab, hipStream_t st) {
  if (rows_cap <= 0) return AS_OK;
  if (d % 8) return as_fail(ctx, AS_ERR_SHAPE, "label logits: d_model must be a multiple of 8");
  prof_begin(ctx, st, AS_K_CE, 0.0);
  label_logit_kernel<<<(unsigned)cdiv(rows_cap, 4), 256, 0, st>>>((const bf16_t*)hf, (const bf16_t*)W, d, labels, count, zlab);
  prof_end(ctx, st);
  AS_LAUNCH_CHECK(ctx);
  return AS_OK;
}

// One wave per row of the chunk: combines the (maximum, sum of exponentials) pairs of the row's column blocks.
// Rows are chunk-relative in `part`, absolute (row0 + r) in zlab / lse / loss_rows.
__global__ __launch_bounds__(256) void ce_finish_kernel(const float* __restrict__ part, int nblk, int row0, const int32_t* __restrict__ count,
                                                        const float* __restrict__ zlab, float* __restrict__ lse_out, float* __restrict__ loss_rows) {
  const int r = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int row = row0 + r;
  if (row >= *count) return;
  const float2* pr = reinterpret_cast<const float2*>(part) + (int64_t)r * nblk;
  float m = -INFINITY;
  for (int b = lane; b < nblk; b += 64) m = fmaxf(m, pr[b].x);
  m = wave_max(m);
  float s = 0.f;
  for (int b = lane; b < nblk; b += 64) { const float2 v = pr[b]; s += v.y * expf(v.x - m); }
  s = wave_sum(s);
  if (lane == 0) { const float lse = m + logf(s); lse_out[row] = lse; loss_rows[row] = lse - zlab[row]; }
}
// The same for GEMM_EPI_SOFT, loss and statistics in the same arithmetic (a policy has its reference's log-probabilities to the bit); the product's elements
// E [rows, V] are completed: the label's loses the sum, and 1 / sum goes to inv (which holds the label's element as a float when the kernel
// begins): inv * w_row * E is the gradient of the logits.  Only a row with a logit 2^40 above its label's has blocks of different exponents; those
// are brought to one.
__global__ __launch_bounds__(256) void soft_finish_kernel(const float* __restrict__ part, int V, int row0, const int32_t* __restrict__ count,
                                                          const float* __restrict__ zlab, const int32_t* __restrict__ labels, float* __restrict__ inv,
                                                          float* __restrict__ loss_rows, bf16_t* __restrict__ E) {
  const int r = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63, nblk = V / 128;
  const int row = row0 + r;
  if (row >= *count) return;
  const float2* pr = reinterpret_cast<const float2*>(part) + (int64_t)r * nblk;
  const float zl = zlab[row];
  float m = -INFINITY, hi = -INFINITY, lo = INFINITY;
  for (int b = lane; b < nblk; b += 64) { const float x = pr[b].x, e = soft_exponent(zl, x); m = fmaxf(m, x); hi = fmaxf(hi, e); lo = fminf(lo, e); }
  m = wave_max(m); hi = wave_max(hi); lo = -wave_max(-lo);
  float s = 0.f, es = 0.f;
  for (int b = lane; b < nblk; b += 64) { const float2 v = pr[b]; s += v.y * expf(v.x - m); es += v.y * soft_scale(v.x, hi); }
  s = wave_sum(s); es = wave_sum(es);
  const int lab = labels[row];
  const float rl = soft_exponent(zl, pr[lab / 128].x);
  const bf16_t el = (bf16_t)(inv[row] * exp2f(rl - hi) - es);
  bf16_t* e = E + (int64_t)r * V;
  if (lo < hi)                                             // the same for the whole wave
    for (int b = 0; b < nblk; b++) {
      const float f = exp2f(soft_exponent(zl, pr[b].x) - hi);
      if (f == 1.f) continue;
      const int c = b * 128 + 2 * lane;
      bf16x2 x = *reinterpret_cast<const bf16x2*>(e + c);
      x[0] = c == lab ? el : (bf16_t)((float)x[0] * f);
      x[1] = c + 1 == lab ? el : (bf16_t)((float)x[1] * f);
      *reinterpret_cast<bf16x2*>(e + c) = x;
    }
  if (lane == 0) {
    if (!(rl < hi)) e[lab] = el;
    inv[row] = 1.f / es;
    const float lse = m + logf(s);
    loss_rows[row] = lse - zl;
  }
}
int launch_soft_finish(as_ctx* ctx, const float* part, int V, int row0, int rows_cap, const int32_t* count, const float* zlab, const int32_t* labels,
                       float* inv, float* loss_rows, void* E, hipStream_t st) {
  if (rows_cap <= 0) return AS_OK;
  prof_begin(ctx, st, AS_K_CE, 0.0);
  soft_finish_kernel<<<(unsigned)cdiv(rows_cap, 4), 256, 0, st>>>(part, V, row0, count, zlab, labels, inv, loss_rows, (bf16_t*)E);
  prof_end(ctx, st);
  AS_LAUNCH_CHECK(ctx);
  return AS_OK;
}

int launch_ce_finish(as_ctx* ctx, const float* part, int nblk, int row0, int rows_cap, const int32_t* count, const float* zlab,
                     float* lse, float* loss_rows, hipStream_t st) {
  if (rows_cap <= 0) return AS_OK;
  prof_begin(ctx, st, AS_K_CE, 0.0);
  ce_finish_kernel<<<(unsigned)cdiv(rows_cap, 4), 256, 0, st>>>(part, nblk, row0, count, zlab, lse, loss_rows);
  prof_end(ctx, st);
  AS_LAUNCH_CHECK(ctx);
  return AS_OK;
}

// Sums the per-target losses in a fixed order: thread i takes a contiguous
// slab, slabs are combined by a tree in LDS.
__global__ void loss_finalize_kernel(const float* __restrict__ loss_rows, const int32_t* __restrict__ count,
                                     float* __restrict__ loss, float* __restrict__ loss_sum) {
  __shared__ double sh[1024];
  int n = *count;
  int per = (n + 1023) / 1024;
  int b = threadIdx.x * per, e = min(n, b + per);
  double acc = 0.0;
  for (int i = b; i < e; i++) acc += (double)loss_rows[i];
  sh[threadIdx.x] = acc;
  __syncthreads();
  for (int off = 512; off > 0; off >>= 1) {
    if (threadIdx.x < off) sh[threadIdx.x] += sh[threadIdx.x + off];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    *loss_sum = (float)sh[0];
    *loss = n > 0 ? (float)(sh[0] / (double)n) : 0.f;
  }
}

int launch_loss_finalize(as_ctx* ctx, const float* loss_rows, const int32_t* count, float* loss,
                         float* loss_sum, hipStream_t st) {
  loss_finalize_kernel<<<1, 1024, 0, st>>>(loss_rows, count, loss, loss_sum);
  AS_LAUNCH_CHECK(ctx);
  return AS_OK;
}

// -------------------------------------------------------- split-K reduction
__global__ void splitk_reduce_kernel(const float* __restrict__ partial, int splitk, int64_t mn, int N,
                                     float alpha, float* __restrict__ C, int64_t ldc) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= mn) return;
  float acc = 0.f;
  for (int s = 0; s < splitk; s++) acc += partial[(int64_t)s * mn + i];
  C[(i / N) * ldc + (i % N)] = alpha * acc;
}
int launch_splitk_reduce(as_ctx* ctx, const float* partial, int splitk, int64_t mn, int N, float alpha,
                         float* C, int64_t ldc, hipStream_t st) {
  if (mn <= 0) return AS_OK;
  splitk_reduce_kernel<<<cdiv(mn, 256), 256, 0, st>>>(partial, splitk, mn, N, alpha, C, ldc);
  AS_LAUNCH_CHECK(ctx);
  return AS_OK;
}

// -------------------------------------------------------------------- AdamW
// Up to kAdamBatch tensors per launch, described in the kernel argument itself: workgroup b takes the b-th chunk of
// kAdamChunk consecutive elements of the batch (tensor found by bisection over the batch's first-chunk numbers).
// Bound by memory (28 bytes per element, 30 with a 16-bit copy), so a thread asks for everything it will touch before it
// computes: four groups of four elements of w, g, m, v are 256 bytes in flight per thread, and 4096-element chunks give a
// launch tens of workgroups per CU.  168 M elements in 448 tensors: 1660 us with 65,536-element chunks and scalar loads
// (2.8 TB/s), 907 us so (5.2 TB/s; a large copy runs at 4.9).
__device__ __forceinline__ void adamw_one(float& w, float g, float& m, float& v, float lr, float b1, float b2, float eps, float bc1, float bc2, float wd) {
  m = b1 * m + (1.f - b1) * g;
  v = b2 * v + (1.f - b2) * g * g;
  const float upd = (m / bc1) / (sqrtf(v / bc2) + eps) + wd * w;
  w = w - lr * upd;
}
__global__ __launch_bounds__(256) void adamw_batch_kernel(const AdamBatch b, float lr, float b1, float b2, float eps, float bc1, float bc2) {
  int ti = 0, hi_t = b.n - 1;                            // last tensor whose first chunk is at or before this workgroup's
  while (ti < hi_t) { const int mid = (ti + hi_t + 1) >> 1; if ((int)blockIdx.x >= b.t[mid].first_chunk) ti = mid; else hi_t = mid - 1; }
  const AdamTensor& t = b.t[ti];
  const int64_t lo = (int64_t)((int)blockIdx.x - t.first_chunk) * kAdamChunk, hi = min(t.n, lo + kAdamChunk);
  const float wd = t.wd;
  const uintptr_t al = (uintptr_t)t.w | (uintptr_t)t.g | (uintptr_t)t.m | (uintptr_t)t.v;
  if (hi - lo == kAdamChunk && al % 16 == 0 && (uintptr_t)t.w_lowp % 8 == 0) {   // a whole chunk of aligned tensors
    constexpr int GROUPS = kAdamChunk / 1024;
    f32x4 w[GROUPS], g[GROUPS], m[GROUPS], v[GROUPS];
#pragma unroll
    for (int i = 0; i < GROUPS; i++) {
      const int64_t e = lo + i * 1024 + threadIdx.x * 4;
      g[i] = *reinterpret_cast<const f32x4*>(t.g + e); m[i] = *reinterpret_cast<const f32x4*>(t.m + e);
      v[i] = *reinterpret_cast<const f32x4*>(t.v + e); w[i] = *reinterpret_cast<const f32x4*>(t.w + e);
    }
#pragma unroll
    for (int i = 0; i < GROUPS; i++) {
      const int64_t e = lo + i * 1024 + threadIdx.x * 4;
      bf16x4 low;
#pragma unroll
      for (int k = 0; k < 4; k++) {
        float wk = w[i][k], mk = m[i][k], vk = v[i][k];
        adamw_one(wk, g[i][k], mk, vk, lr, b1, b2, eps, bc1, bc2, wd);
        w[i][k] = wk; m[i][k] = mk; v[i][k] = vk; low[k] = (bf16_t)wk;
      }
      *reinterpret_cast<f32x4*>(t.m + e) = m[i]; *reinterpret_cast<f32x4*>(t.v + e) = v[i]; *reinterpret_cast<f32x4*>(t.w + e) = w[i];
      if (t.w_lowp) *reinterpret_cast<bf16x4*>(t.w_lowp + e) = low;
    }
    return;
  }
  for (int64_t i = lo + threadIdx.x; i < hi; i += 256) {
    float wi = t.w[i], mi = t.m[i], vi = t.v[i];
    adamw_one(wi, t.g[i], mi, vi, lr, b1, b2, eps, bc1, bc2, wd);
    t.m[i] = mi; t.v[i] = vi; t.w[i] = wi;
    if (t.w_lowp) t.w_lowp[i] = (bf16_t)wi;
  }
}
int launch_adamw_batch(as_ctx* ctx, const AdamBatch& b, float lr, float b1, float b2, float eps, float bc1, float bc2, hipStream_t st) {
  if (b.n <= 0 || b.n_chunks <= 0) return AS_OK;
  adamw_batch_kernel<<<b.n_chunks, 256, 0, st>>>(b, lr, b1, b2, eps, bc1, bc2);
  AS_LAUNCH_CHECK(ctx);
  return AS_OK;
}

// ------------------------------------------------- embedding gradient (full)
// dE[v] = sum of dh[t] over the positions t holding token v, in ascending t.  Token frequencies fall off like 1 / rank: one
// token may hold an eighth of all positions, so neither a workgroup per token nor a walk along its positions balances.
// The positions are sorted by token (stable, least significant 9 bits first: a histogram, a scan and a scatter per digit),
// the sorted list is cut into pieces of EMB_PIECE positions, and a workgroup adds up the runs inside its piece.  A run that
// lies inside one piece is written straight to dE; a run that crosses pieces leaves a float partial row per piece, which
// the workgroup of the piece it starts in adds in order.  Bound by reading dh and writing dE once.
// 15,700 positions, d 2048, vocabulary 32,000, Zipf(1.1): 121 us in all (sums 35, zero fill of dE 34, sort 42,
// join 10) against 5950 us for a walk along each token's positions.
constexpr int EMB_BITS = 9, EMB_BINS = 1 << EMB_BITS, EMB_TILE = 2048, EMB_PIECE = 32;

// cnt[bin * n_tiles + tile] = positions of this tile whose token has `bin` as its current digit
__global__ __launch_bounds__(256) void embed_hist_kernel(const int32_t* __restrict__ tok, const int32_t* __restrict__ pos, int n, int shift,
                                                         int n_tiles, int32_t* __restrict__ cnt) {
  __shared__ int32_t h[EMB_BINS];
  for (int i = threadIdx.x; i < EMB_BINS; i += 256) h[i] = 0;
  __syncthreads();
  for (int i = threadIdx.x; i < EMB_TILE; i += 256) {
    const int k = blockIdx.x * EMB_TILE + i;
    if (k < n) atomicAdd(&h[((uint32_t)tok[pos ? pos[k] : k] >> shift) & (EMB_BINS - 1)], 1);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < EMB_BINS; i += 256) cnt[(int64_t)i * n_tiles + blockIdx.x] = h[i];
}
// exclusive scan of m integers in place, one workgroup
__global__ __launch_bounds__(1024) void embed_scan_kernel(int32_t* __restrict__ cnt, int m) {
  __shared__ int32_t wsum[16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int per = (m + 1023) / 1024, b = min(m, tid * per), e = min(m, b + per);
  int s = 0;
  for (int i = b; i < e; i++) s += cnt[i];
  int incl = s;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) { const int v = __shfl_up(incl, o, 64); if (lane >= o) incl += v; }
  if (lane == 63) wsum[wave] = incl;
  __syncthreads();
  int base = incl - s;
  for (int w = 0; w < wave; w++) base += wsum[w];
  for (int i = b; i < e; i++) { const int v = cnt[i]; cnt[i] = base; base += v; }
}
// stable scatter of the tile's positions in order, 256 at a time; the rank of a position among those with its digit is that
// among the lower lanes of its wave (ballots over the digit's bits) plus the counts of the waves and rounds before
__device__ __forceinline__ void embed_scatter_tile(const int32_t* __restrict__ tok, const int32_t* pos, int first, int n, int shift,
                                                   int32_t* base, int32_t (*wcnt)[EMB_BINS], int32_t* out) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  for (int r = 0; r < EMB_TILE / 256 && first + r * 256 < n; r++) {
    for (int i = tid; i < 4 * EMB_BINS; i += 256) (&wcnt[0][0])[i] = 0;
    __syncthreads();
    const int k = first + r * 256 + tid;
    const bool live = k < n;
    const int p = live ? (pos ? pos[k] : k) : 0;
    const int d = live ? (int)(((uint32_t)tok[p] >> shift) & (EMB_BINS - 1)) : 0;
    uint64_t same = __ballot(live);
#pragma unroll
    for (int bit = 0; bit < EMB_BITS; bit++) { const uint64_t m = __ballot((d >> bit) & 1); same &= ((d >> bit) & 1) ? m : ~m; }
    const int rank = __popcll(same & ((1ull << lane) - 1));
    if (live && rank == 0) wcnt[wave][d] = __popcll(same);
    __syncthreads();
    if (live) {
      int at = base[d] + rank;
      for (int w = 0; w < wave; w++) at += wcnt[w][d];
      out[at] = p;
    }
    __syncthreads();
    for (int i = tid; i < EMB_BINS; i += 256) base[i] += wcnt[0][i] + wcnt[1][i] + wcnt[2][i] + wcnt[3][i];
    __syncthreads();
  }
}
__global__ __launch_bounds__(256) void embed_scatter_kernel(const int32_t* __restrict__ tok, const int32_t* __restrict__ pos, int n, int shift,
                                                            int n_tiles, const int32_t* __restrict__ cnt, int32_t* __restrict__ out) {
  __shared__ int32_t base[EMB_BINS], wcnt[4][EMB_BINS];
  for (int i = threadIdx.x; i < EMB_BINS; i += 256) base[i] = cnt[(int64_t)i * n_tiles + blockIdx.x];
  embed_scatter_tile(tok, pos, blockIdx.x * EMB_TILE, n, shift, base, wcnt, out);
}
// at most one tile of positions: every digit in one launch, the positions in LDS
__global__ __launch_bounds__(256) void embed_sort_tile_kernel(const int32_t* __restrict__ tok, int n, int V, int32_t* __restrict__ out) {
  __shared__ int32_t base[EMB_BINS], wcnt[4][EMB_BINS], buf[2][EMB_TILE];
  const int tid = threadIdx.x, lane = tid & 63;
  const int32_t* in = nullptr;
  int b = 0;
  for (int shift = 0; shift == 0 || (shift < 31 && (V - 1) >> shift); shift += EMB_BITS, b ^= 1) {
    for (int i = tid; i < EMB_BINS; i += 256) base[i] = 0;
    __syncthreads();
    for (int k = tid; k < n; k += 256) atomicAdd(&base[((uint32_t)tok[in ? in[k] : k] >> shift) & (EMB_BINS - 1)], 1);
    __syncthreads();
    if (tid < 64) {                                        // exclusive scan of the bins, eight per lane
      int c[EMB_BINS / 64], s = 0;
#pragma unroll
      for (int i = 0; i < EMB_BINS / 64; i++) { c[i] = base[lane * (EMB_BINS / 64) + i]; s += c[i]; }
      int incl = s;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) { const int v = __shfl_up(incl, o, 64); if (lane >= o) incl += v; }
      int at = incl - s;
#pragma unroll
      for (int i = 0; i < EMB_BINS / 64; i++) { base[lane * (EMB_BINS / 64) + i] = at; at += c[i]; }
    }
    __syncthreads();
    embed_scatter_tile(tok, in, 0, n, shift, base, wcnt, buf[b]);
    in = buf[b];
  }
  for (int k = tid; k < n; k += 256) out[k] = in[k];
}
// piece blockIdx.x of the sorted positions, columns of blockIdx.y.  part[2 * piece]: the run that began in an earlier piece,
// part[2 * piece + 1]: the run that begins here and goes on in the next piece (rows of d floats).
template <typename T, int VN>
__global__ __launch_bounds__(256) void embed_sum_kernel(const int32_t* __restrict__ tok, const int32_t* __restrict__ pos, int n, int d, int V,
                                                        const T* __restrict__ dh, float* __restrict__ dE, float* __restrict__ part) {
  __shared__ int32_t sp[EMB_PIECE], sv[EMB_PIECE + 2];     // sv[i + 1] = token of entry i; neighbours at both ends, -1 past the list
  const int k0 = blockIdx.x * EMB_PIECE, cnt = min(EMB_PIECE, n - k0);
  if (threadIdx.x < EMB_PIECE + 2) {
    const int i = (int)threadIdx.x - 1, k = k0 + i;
    const int p = k >= 0 && k < n ? pos[k] : -1;
    if (i >= 0 && i < EMB_PIECE) sp[i] = p;
    sv[threadIdx.x] = p >= 0 ? tok[p] : -1;
  }
  __syncthreads();
  const int j = (blockIdx.y * 256 + threadIdx.x) * VN;
  if (j >= d) return;
  float acc[VN];
#pragma unroll
  for (int c = 0; c < VN; c++) acc[c] = 0.f;
  auto put = [&](float* q) {
    if constexpr (VN % 4 == 0) {
#pragma unroll
      for (int c = 0; c < VN; c += 4) *reinterpret_cast<f32x4*>(q + c) = (f32x4){acc[c], acc[c + 1], acc[c + 2], acc[c + 3]};
    } else {
#pragma unroll
      for (int c = 0; c < VN; c++) q[c] = acc[c];
    }
  };
  bool began_here = sv[0] != sv[1];
  for (int i0 = 0; i0 < cnt; i0 += 8) {
    float x[8][VN];
#pragma unroll
    for (int q = 0; q < 8; q++)                            // eight rows in flight
      if (i0 + q < cnt) {
        const T* row = dh + (int64_t)sp[i0 + q] * d + j;
        if constexpr (VN == Vec<T>::N) load_vec<T>(row, x[q]); else x[q][0] = to_f<T>(row[0]);
      }
#pragma unroll
    for (int q = 0; q < 8; q++) {
      const int i = i0 + q;
      if (i >= cnt) break;
#pragma unroll
      for (int c = 0; c < VN; c++) acc[c] += x[q][c];
      const int v = sv[i + 1];
      const bool run_ends = sv[i + 2] != v;
      if (!run_ends && i + 1 < cnt) continue;
      if (!began_here) put(part + (int64_t)(2 * blockIdx.x) * d + j);
      else if (!run_ends) put(part + (int64_t)(2 * blockIdx.x + 1) * d + j);
      else if ((uint32_t)v < (uint32_t)V) put(dE + (int64_t)v * d + j);
      began_here = true;
#pragma unroll
      for (int c = 0; c < VN; c++) acc[c] = 0.f;
    }
  }
}
// the run that begins in piece blockIdx.x and goes on: its partial rows in order
__global__ __launch_bounds__(256) void embed_join_kernel(const int32_t* __restrict__ tok, const int32_t* __restrict__ pos, int n, int d, int V,
                                                         const float* __restrict__ part, float* __restrict__ dE) {
  const int k0 = blockIdx.x * EMB_PIECE, last = k0 + EMB_PIECE - 1;
  if (last + 1 >= n) return;
  const int v = tok[pos[last]];
  if (tok[pos[last + 1]] != v || (uint32_t)v >= (uint32_t)V) return;
  if (tok[pos[k0]] == v && k0 > 0 && tok[pos[k0 - 1]] == v) return;                   // began in an earlier piece
  int end = blockIdx.x + 1;                                                           // last piece that holds the token: bisection over the sorted list
  { int lo = last + 1, hi = n - 1;                                                    // entry lo holds v; entries holding v are contiguous
    const int t = v;
    while (lo < hi) { const int mid = lo + (hi - lo + 1) / 2; if (tok[pos[mid]] == t) lo = mid; else hi = mid - 1; }
    end = lo / EMB_PIECE; }
  const int j = blockIdx.y * 256 + threadIdx.x;
  if (j >= d) return;
  float acc = part[(int64_t)(2 * blockIdx.x + 1) * d + j];
  int q = blockIdx.x + 1;
  for (; q + 8 <= end + 1; q += 8) {
    float x[8];
#pragma unroll
    for (int i = 0; i < 8; i++) x[i] = part[(int64_t)(2 * (q + i)) * d + j];
#pragma unroll
    for (int i = 0; i < 8; i++) acc += x[i];
  }
  for (; q <= end; q++) acc += part[(int64_t)(2 * q) * d + j];
  dE[(int64_t)v * d + j] = acc;
}

size_t embed_bwd_aux_bytes(int n, int d) {
  const size_t cnt = ((size_t)EMB_BINS * cdiv(n, EMB_TILE) * 4 + 255) & ~(size_t)255;
  return cnt + (size_t)2 * cdiv(n, EMB_PIECE) * d * 4;
}
int launch_embed_bwd(as_ctx* ctx, int mode, const int32_t* tok, int n, int d, int V, const void* dh,
                     int32_t* scratch, void* aux, size_t aux_bytes, float* dE, hipStream_t st) {
  // scratch: 2n int32 (the positions, sorted by one digit after the other); dE is zeroed first (rows of unused tokens stay zero)
  int rc = launch_fill_zero(ctx, dE, (size_t)V * d * sizeof(float), st);
  if (rc) return rc;
  if (n <= 0) return AS_OK;
  if (embed_bwd_aux_bytes(n, d) > aux_bytes) return as_fail(ctx, AS_ERR_WORKSPACE, "embedding gradient: scratch too small");
  const int tiles = (int)cdiv(n, EMB_TILE), pieces = (int)cdiv(n, EMB_PIECE);
  int32_t* cnt = (int32_t*)aux;
  float* part = (float*)((char*)aux + (((size_t)EMB_BINS * tiles * 4 + 255) & ~(size_t)255));
  const int32_t* in = nullptr; int32_t* out = scratch;
  if (tiles == 1) {
    embed_sort_tile_kernel<<<1, 256, 0, st>>>(tok, n, V, out);
    AS_LAUNCH_CHECK(ctx);
    in = out;
  } else
  for (int shift = 0; shift == 0 || (shift < 31 && (V - 1) >> shift); shift += EMB_BITS) {
    embed_hist_kernel<<<tiles, 256, 0, st>>>(tok, in, n, shift, tiles, cnt);
    embed_scan_kernel<<<1, 1024, 0, st>>>(cnt, EMB_BINS * tiles);
    embed_scatter_kernel<<<tiles, 256, 0, st>>>(tok, in, n, shift, tiles, cnt, out);
    AS_LAUNCH_CHECK(ctx);
    in = out; out = out == scratch ? scratch + n : scratch;
  }
  DISPATCH_T(mode, {
    constexpr int VN = Vec<T>::N;
    if (vec_ok<T>(dh, d) && (uintptr_t)dE % 16 == 0 && d % 4 == 0)
      embed_sum_kernel<T, VN><<<dim3(pieces, (unsigned)cdiv(d, 256 * VN)), 256, 0, st>>>(tok, in, n, d, V, (const T*)dh, dE, part);
    else
      embed_sum_kernel<T, 1><<<dim3(pieces, (unsigned)cdiv(d, 256)), 256, 0, st>>>(tok, in, n, d, V, (const T*)dh, dE, part); });
  AS_LAUNCH_CHECK(ctx);
  embed_join_kernel<<<dim3(pieces, (unsigned)cdiv(d, 256)), 256, 0, st>>>(tok, in, n, d, V, part, dE);
  AS_LAUNCH_CHECK(ctx);
  return AS_OK;
}
