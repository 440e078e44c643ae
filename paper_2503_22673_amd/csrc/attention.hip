// Varlen causal attention with grouped KV heads over packed rows: a query at
// token t sees keys seg_start[t] .. t only, so nothing crosses a trajectory
// boundary.  Query head j reads KV head j / (Hq/Hkv).
//
// Plain kernels (any type; the fp32 tier): one workgroup per (token, head).  What bounds them is latency, then the address unit, which takes a
// clock per lane where neighbouring lanes read different rows.  So a row is read by dh / 4 neighbouring lanes, four columns each, dot products
// are sums over those lanes, and the workgroup's 32, 16 or 8 such groups take rows in turn, four (forward) or two of them under way at once; each
// group adds up its own rows, and the groups meet at the end in a fixed order.  The backward needs no scores of other rows (the log-sum-exp is there), so a row is
// read once for both its dot products and its sum; dQ and dK / dV are one launch (dK / dV forms the dO O of its rows itself), which also
// rotates dq and dk back.  A row per thread, then a column per thread, in three launches with scores in LDS, took 12.5 + 15.4 + 18.4 us and 3.7 for the rotation
// (478 tokens, 4 heads of 32); 9.3 and 13.9 so.  Two rows backward leave registers for eight workgroups a CU: with four rows, four workgroups, 15.6.
#include "common.h"

constexpr int kPlainThreads = 256;
template <typename T, bool VEC> __device__ __forceinline__ f32x4 load4(const T* p) {       // four values of a row; VEC: as one piece
  f32x4 v;
  if constexpr (VEC && sizeof(T) == 4) return *reinterpret_cast<const f32x4*>(p);
  if constexpr (VEC) {
    const bf16x4 x = *reinterpret_cast<const bf16x4*>(p);
#pragma unroll
    for (int e = 0; e < 4; e++) v[e] = (float)x[e];
  } else {
#pragma unroll
    for (int e = 0; e < 4; e++) v[e] = to_f<T>(p[e]);
  }
  return v;
}
template <typename T> __device__ __forceinline__ void put4(T* p, const f32x4& v) {
#pragma unroll
  for (int e = 0; e < 4; e++) p[e] = from_f<T>(v[e]);
}
__device__ __forceinline__ float dot4(const f32x4& a, const f32x4& b) { return fmaf(a[3], b[3], fmaf(a[2], b[2], fmaf(a[1], b[1], a[0] * b[0]))); }
template <int CTRL> __device__ __forceinline__ float add_dpp(float x) {
  return x + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, true));
}
// sum over LPR (8, 16, 32) neighbouring lanes, in all of them; every lane of the wave takes part
template <int LPR> __device__ __forceinline__ float row_sum(float x) {
  x = add_dpp<0xB1>(x);                                    // lane ^ 1, lane ^ 2, the other half of eight, of sixteen
  x = add_dpp<0x4E>(x);
  x = add_dpp<0x141>(x);
  if (LPR > 8) x = add_dpp<0x140>(x);
  if (LPR > 16) x += __shfl_xor(x, 16, 64);
  return x;
}
// sums of the groups' four columns: within a wave, then over the waves; the first LPR threads have them
template <int LPR> __device__ __forceinline__ f32x4 group_sum(f32x4 v, f32x4* red) {
#pragma unroll
  for (int e = 0; e < 4; e++) for (int o = LPR; o < 64; o <<= 1) v[e] += __shfl_xor(v[e], o, 64);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  __syncthreads();
  if (lane < LPR) red[wave * LPR + lane] = v;
  __syncthreads();
  if (threadIdx.x < LPR) v = red[lane] + red[LPR + lane] + red[2 * LPR + lane] + red[3 * LPR + lane];
  return v;
}

// --------------------------------------------------------------- plain fwd
// A group's rows against the largest score it has met so far; the groups' sums are brought to the largest of all at the end.
template <typename T, int DH, bool VEC>
__global__ __launch_bounds__(256) void attn_fwd_plain(AttnParams p, float scale) {
  constexpr int LPR = DH / 4, G = 64 / LPR, ROWS = 4 * G, U = 4;                    // U: rows of a group under way together
  __shared__ f32x4 racc[4 * LPR];
  __shared__ float rmx[4], rsum[4];
  const int t = blockIdx.x, j = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lc = lane % LPR, grp = wave * G + lane / LPR;
  const int g = j / (p.Hq / p.Hkv);
  const int s0 = p.seg_start[t], len = t - s0 + 1;
  const f32x4 q = load4<T, VEC>((const T*)p.q + (int64_t)t * p.ldq + j * DH + 4 * lc);
  const T* kb = (const T*)p.k + (int64_t)s0 * p.ldkv + g * DH + 4 * lc;
  const T* vb = (const T*)p.v + (int64_t)s0 * p.ldkv + g * DH + 4 * lc;
  float mx = -INFINITY, sum = 0.f;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  for (int base = 0; base < len; base += ROWS * U) {
    f32x4 k[U], v[U]; float d[U];
#pragma unroll
    for (int i = 0; i < U; i++) {                          // past the end the last row, which nobody uses
      const int64_t r = (int64_t)min(base + grp + i * ROWS, len - 1) * p.ldkv;
      k[i] = load4<T, VEC>(kb + r); v[i] = load4<T, VEC>(vb + r);
    }
    float m = mx;
#pragma unroll
    for (int i = 0; i < U; i++) {
      d[i] = row_sum<LPR>(dot4(q, k[i])) * scale;
      if (base + grp + i * ROWS < len) m = fmaxf(m, d[i]);
    }
    const float f = m > mx ? expf(mx - m) : 1.f;           // the first rows: exp(-inf)
    mx = m; sum *= f;
#pragma unroll
    for (int c = 0; c < 4; c++) acc[c] *= f;
#pragma unroll
    for (int i = 0; i < U; i++)
      if (base + grp + i * ROWS < len) {
        const float e = d[i] == -INFINITY ? 0.f : expf(d[i] - mx);      // no -inf - -inf where a group has met nothing else yet
        sum += e;
#pragma unroll
        for (int c = 0; c < 4; c++) acc[c] = fmaf(e, v[i][c], acc[c]);
      }
  }
  // a group without rows has sum 0 and maximum -inf: its factor is 0; the wave of the first group has a row
  float all = mx;
  for (int o = LPR; o < 64; o <<= 1) all = fmaxf(all, __shfl_xor(all, o, 64));
  const float f = mx > -INFINITY ? expf(mx - all) : 0.f;
  sum *= f;
  for (int o = LPR; o < 64; o <<= 1) sum += __shfl_xor(sum, o, 64);
#pragma unroll
  for (int c = 0; c < 4; c++) {
    acc[c] *= f;
    for (int o = LPR; o < 64; o <<= 1) acc[c] += __shfl_xor(acc[c], o, 64);
  }
  if (lane < LPR) racc[wave * LPR + lane] = acc;
  if (lane == 0) { rmx[wave] = all; rsum[wave] = sum; }
  __syncthreads();
  if (tid >= LPR) return;
  all = fmaxf(fmaxf(rmx[0], rmx[1]), fmaxf(rmx[2], rmx[3]));
  sum = 0.f; acc = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int w = 0; w < 4; w++) {
    const float fw = expf(rmx[w] - all);                   // a wave without rows: 0; no finite score at all: no number, in o and lse
    sum += rsum[w] * fw;
#pragma unroll
    for (int c = 0; c < 4; c++) acc[c] = fmaf(racc[w * LPR + lane][c], fw, acc[c]);
  }
#pragma unroll
  for (int c = 0; c < 4; c++) acc[c] /= sum;
  put4<T>((T*)p.o + ((int64_t)t * p.Hq + j) * DH + 4 * lc, acc);
  if (tid == 0) p.lse[(int64_t)t * p.Hq + j] = all + logf(sum);
}

// --------------------------------------------------------------- plain bwd
// the inverse of the rotary embedding on a gradient row whose columns 4 lc .. lie in lane lc; all lanes of the first wave come here
template <int LPR> __device__ __forceinline__ f32x4 rotate_back(const AttnParams& p, f32x4 x, int t, int lc) {
  const int half = LPR / 2, i = lc % half;
  const int64_t at = (int64_t)(t - p.seg_start[t]) * (2 * LPR) + 4 * i;
  const f32x4 c = *reinterpret_cast<const f32x4*>(p.rope_cos + at), s = *reinterpret_cast<const f32x4*>(p.rope_sin + at);
  f32x4 r;
#pragma unroll
  for (int e = 0; e < 4; e++) {
    const float y = __shfl_xor(x[e], half, 64);            // the row's other half
    r[e] = lc < half ? x[e] * c[e] + y * s[e] : x[e] * c[e] - y * s[e];
  }
  return r;
}
// Workgroups with blockIdx.y < Hkv: dk, dv of one (token, KV head), summed over the query heads of the group in head order and the later tokens
// of the segment; the others: dq of one (token, head).
template <typename T, int DH, bool VEC>
__global__ __launch_bounds__(256, 8) void attn_bwd_plain(AttnParams p, float scale) {
  constexpr int LPR = DH / 4, G = 64 / LPR, ROWS = 4 * G, U = 2;
  __shared__ f32x4 red[4 * LPR];
  const int t = blockIdx.x, tid = threadIdx.x, lane = tid & 63, lc = lane % LPR, grp = (tid >> 6) * G + lane / LPR, grp_q = p.Hq / p.Hkv;
  const int64_t ldo = (int64_t)p.Hq * DH;
  f32x4 a0 = {0.f, 0.f, 0.f, 0.f}, a1 = {0.f, 0.f, 0.f, 0.f};
  if ((int)blockIdx.y < p.Hkv) {
    const int g = blockIdx.y, len = p.seg_end[t] - t;
    const f32x4 k = load4<T, VEC>((const T*)p.k + (int64_t)t * p.ldkv + g * DH + 4 * lc), v = load4<T, VEC>((const T*)p.v + (int64_t)t * p.ldkv + g * DH + 4 * lc);
    for (int jj = 0; jj < grp_q; jj++) {
      const int j = g * grp_q + jj;
      const T* qb = (const T*)p.q + (int64_t)t * p.ldq + j * DH + 4 * lc;
      const T* db = (const T*)p.d_o + t * ldo + j * DH + 4 * lc; const T* ob = (const T*)p.o + t * ldo + j * DH + 4 * lc;
      const float* lb = p.lse + (int64_t)t * p.Hq + j;
      for (int base = 0; base < len; base += ROWS * U) {
        f32x4 q[U], d[U], o[U]; float l[U];
#pragma unroll
        for (int i = 0; i < U; i++) {
          const int64_t r = min(base + grp + i * ROWS, len - 1);
          q[i] = load4<T, VEC>(qb + r * p.ldq); d[i] = load4<T, VEC>(db + r * ldo); o[i] = load4<T, VEC>(ob + r * ldo); l[i] = lb[r * p.Hq];
        }
#pragma unroll
        for (int i = 0; i < U; i++) {
          const float s = row_sum<LPR>(dot4(k, q[i])), dp = row_sum<LPR>(dot4(v, d[i])), dl = row_sum<LPR>(dot4(d[i], o[i]));
          if (base + grp + i * ROWS < len) {
            const float pr = expf(s * scale - l[i]), ds = pr * (dp - dl);
#pragma unroll
            for (int c = 0; c < 4; c++) { a0[c] = fmaf(ds, q[i][c], a0[c]); a1[c] = fmaf(pr, d[i][c], a1[c]); }
          }
        }
      }
    }
    a0 = group_sum<LPR>(a0, red); a1 = group_sum<LPR>(a1, red);
    if (tid >= 64) return;
#pragma unroll
    for (int c = 0; c < 4; c++) a0[c] *= scale;
    if (p.rope_cos) a0 = rotate_back<LPR>(p, a0, t, lc);
    if (tid >= LPR) return;
    put4<T>((T*)p.dk + (int64_t)t * p.ldkv + g * DH + 4 * lc, a0);
    put4<T>((T*)p.dv + (int64_t)t * p.ldkv + g * DH + 4 * lc, a1);
    return;
  }
  const int j = blockIdx.y - p.Hkv, g = j / grp_q, s0 = p.seg_start[t], len = t - s0 + 1;
  const int64_t at = t * ldo + j * DH + 4 * lc;
  const f32x4 q = load4<T, VEC>((const T*)p.q + (int64_t)t * p.ldq + j * DH + 4 * lc), d = load4<T, VEC>((const T*)p.d_o + at), o = load4<T, VEC>((const T*)p.o + at);
  const T* kb = (const T*)p.k + (int64_t)s0 * p.ldkv + g * DH + 4 * lc;
  const T* vb = (const T*)p.v + (int64_t)s0 * p.ldkv + g * DH + 4 * lc;
  const float lse = p.lse[(int64_t)t * p.Hq + j], dl = row_sum<LPR>(dot4(d, o));
  for (int base = 0; base < len; base += ROWS * U) {
    f32x4 k[U], v[U];
#pragma unroll
    for (int i = 0; i < U; i++) {
      const int64_t r = (int64_t)min(base + grp + i * ROWS, len - 1) * p.ldkv;
      k[i] = load4<T, VEC>(kb + r); v[i] = load4<T, VEC>(vb + r);
    }
#pragma unroll
    for (int i = 0; i < U; i++) {
      const float s = row_sum<LPR>(dot4(q, k[i])), dp = row_sum<LPR>(dot4(d, v[i]));
      if (base + grp + i * ROWS < len) {
        const float ds = expf(s * scale - lse) * (dp - dl);
#pragma unroll
        for (int c = 0; c < 4; c++) a0[c] = fmaf(ds, k[i][c], a0[c]);
      }
    }
  }
  a0 = group_sum<LPR>(a0, red);
  if (tid >= 64) return;
#pragma unroll
  for (int c = 0; c < 4; c++) a0[c] *= scale;
  if (p.rope_cos) a0 = rotate_back<LPR>(p, a0, t, lc);
  if (tid < LPR) put4<T>((T*)p.dq + (int64_t)t * p.ldq + j * DH + 4 * lc, a0);
}

// The plain kernels have no limit of their own: they answer for the segments that they have always answered for, up to 40,960 - head_dim
// tokens forward and half as many backward.
constexpr int kPlainTokens = 40960;
static int check_plain(as_ctx* ctx, const AttnParams& p, int limit) {
  if (p.dh != 32 && p.dh != 64 && p.dh != 128) return as_fail(ctx, AS_ERR_SHAPE, "attention: head_dim 32, 64 or 128");
  if (p.max_seg > limit) return as_fail(ctx, AS_ERR_SHAPE, "attention (plain kernels): segments of at most %d tokens", limit);
  return AS_OK;
}

// rows of q, k, v (and o, dO, whose rows are Hq dh values) in pieces of four values
static bool plain_vec(int mode, const AttnParams& p, std::initializer_list<const void*> ptrs) {
  uintptr_t x = 0;
  for (const void* q : ptrs) x |= (uintptr_t)q;
  return x % (mode == AS_FP32 ? 16 : 8) == 0 && p.ldq % 4 == 0 && p.ldkv % 4 == 0;
}
template <typename F> static void plain_kernel(int mode, const AttnParams& p, bool vec, const F& f) {
  auto dims = [&](auto t, auto v) {
    p.dh == 32 ? f(t, std::integral_constant<int, 32>(), v) : p.dh == 64 ? f(t, std::integral_constant<int, 64>(), v) : f(t, std::integral_constant<int, 128>(), v);
  };
  auto types = [&](auto v) { mode == AS_FP32 ? dims(0.f, v) : dims(bf16_t(0.f), v); };
  vec ? types(std::true_type()) : types(std::false_type());
}
int launch_attention_fwd_mfma(as_ctx* ctx, const AttnParams& p, int variant, hipStream_t st);
int launch_attention_bwd_mfma(as_ctx* ctx, const AttnParams& p, int variant, hipStream_t st);
bool attention_mfma_ok(const AttnParams& p);

int launch_attention_fwd(as_ctx* ctx, int mode, int variant, const AttnParams& p, hipStream_t st) {
  if (p.n <= 0) return AS_OK;
  bool mf = mode == AS_BF16 && variant != 1 && attention_mfma_ok(p);
  if (variant >= 2 && !mf) return as_fail(ctx, AS_ERR_SHAPE, "attention: MFMA kernel needs bf16, head_dim 64/128, aligned strides");
  if (mf) { prof_begin(ctx, st, AS_K_ATTN_FWD, 0.0); int r = launch_attention_fwd_mfma(ctx, p, variant, st); prof_end(ctx, st); return r; }
  int rc = check_plain(ctx, p, kPlainTokens - p.dh); if (rc) return rc;
  plain_kernel(mode, p, plain_vec(mode, p, {p.q, p.k, p.v}), [&](auto t, auto dh, auto vec) {
    attn_fwd_plain<decltype(t), dh(), vec()><<<dim3(p.n, p.Hq), kPlainThreads, 0, st>>>(p, 1.f / sqrtf((float)p.dh)); });
  AS_LAUNCH_CHECK(ctx);
  return AS_OK;
}

int launch_attention_bwd(as_ctx* ctx, int mode, int variant, const AttnParams& p, hipStream_t st) {
  if (p.n <= 0) return AS_OK;
  bool mf = mode == AS_BF16 && variant != 1 && attention_mfma_ok(p);
  if (variant >= 2 && !mf) return as_fail(ctx, AS_ERR_SHAPE, "attention: MFMA kernel needs bf16, head_dim 64/128, aligned strides");
  if (mf) { prof_begin(ctx, st, AS_K_ATTN_BWD, 0.0); int r = launch_attention_bwd_mfma(ctx, p, variant, st); prof_end(ctx, st); return r; }
  int rc = check_plain(ctx, p, kPlainTokens / 2 - p.dh); if (rc) return rc;
  plain_kernel(mode, p, plain_vec(mode, p, {p.q, p.k, p.v, p.o, p.d_o}), [&](auto t, auto dh, auto vec) {
    attn_bwd_plain<decltype(t), dh(), vec()><<<dim3(p.n, p.Hkv + p.Hq), kPlainThreads, 0, st>>>(p, 1.f / sqrtf((float)p.dh)); });
  AS_LAUNCH_CHECK(ctx);
  return AS_OK;
}
