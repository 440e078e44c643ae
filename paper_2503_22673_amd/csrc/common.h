// Shared declarations of the gfx950 fine-tuning library: element types,
// error plumbing, the context, and the launchers each .hip file exports to
// the C interface in api.hip.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>
#include <string>
#include <vector>
#include <algorithm>
#include <atomic>
#include <initializer_list>
#include <type_traits>
#include "actionstudio.h"
#include "gemm_items.h"
#include "per_kernel.h"

typedef __bf16 bf16_t;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;

#define AS_WAVE 64

struct as_ctx {
  as_model_config cfg;
  int device;
  std::string err;
  // staging owned by the context (as_pack only)
  void* h_stage = nullptr; size_t h_stage_bytes = 0;
  // optional per-launch timing (as_profile): event pairs around kernels of the tracked classes
  struct ProfRec { hipEvent_t a, b; double flops; int cls; };
  bool prof_on = false; int prof_depth = 0;
  int prof_only = -1; bool prof_skipping = false;   // >= 0: only this class is bracketed
  std::vector<ProfRec> prof; size_t prof_used = 0;
};
// Brackets one kernel launch with events when profiling is on (no-ops otherwise).
void prof_begin(as_ctx* ctx, hipStream_t st, int cls, double flops);
void prof_end(as_ctx* ctx, hipStream_t st);

int as_fail(as_ctx* ctx, int code, const char* fmt, ...);
#define AS_HIP(ctx, call) do { hipError_t e_ = (call); if (e_ != hipSuccess) \
  return as_fail((ctx), AS_ERR_HIP, "%s: %s", #call, hipGetErrorString(e_)); } while (0)
#define AS_LAUNCH_CHECK(ctx) AS_HIP(ctx, hipGetLastError())
// Raises a kernel's dynamic LDS limit once per device (the attribute belongs to the code object loaded on that device); kern: a constant expression,
// and of one kernel always the same number of bytes.
#define AS_SET_SMEM(ctx, kern, bytes) do { std::atomic<uint64_t>& done_ = smem_devices<kern>; const uint64_t bit_ = 1ull << ((ctx)->device & 63); \
  if (!(done_.load(std::memory_order_relaxed) & bit_)) { \
    AS_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)(bytes))); \
    done_.fetch_or(bit_, std::memory_order_relaxed); } } while (0)

// The item of a launch's table that x lies in, first(k) being where item k begins: the begins are read side by side and counted.  A search
// reads them one after the other, and each of those reads is a first touch of memory: 0.2 to 0.4 us of the
// adapter gradients' launches, their sums' and the 4-bit unpacking.
template <int MAX, typename X, typename F> __device__ __forceinline__ int table_item(int n, X x, F first) {
  int it = 0;
#pragma unroll
  for (int k = 1; k < MAX; k++) it += k < n && x >= first(k) ? 1 : 0;
  return it;
}

static inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

template <typename T> __device__ __forceinline__ float to_f(T x);
template <> __device__ __forceinline__ float to_f<float>(float x) { return x; }
template <> __device__ __forceinline__ float to_f<bf16_t>(bf16_t x) { return (float)x; }
template <typename T> __device__ __forceinline__ T from_f(float x);
template <> __device__ __forceinline__ float from_f<float>(float x) { return x; }
template <> __device__ __forceinline__ bf16_t from_f<bf16_t>(float x) { return (bf16_t)x; }

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}

// Softmax without the sum (GEMM_EPI_SOFT): the power of two that a row's block of logits is held against, whole numbers, so that blocks of one row differ
// by exact powers of two, and what the exponentials against the block's maximum are multiplied by for it.  A label logit that is no number or
// out of reach counts for nothing.
constexpr float kLog2e = 1.4426950408889634f;
__device__ __forceinline__ float soft_exponent(float label_logit, float block_max) {
  return fmaxf(fminf(fmaxf(rintf(label_logit * kLog2e), -4e6f), 4e6f), ceilf(block_max * kLog2e) - 40.f);
}
__device__ __forceinline__ float soft_scale(float block_max, float exponent) { return __builtin_amdgcn_exp2f(fmaf(block_max, kLog2e, -exponent)); }

// 16 bytes of a row at a time
template <typename T> struct Vec;
template <> struct Vec<float> { static constexpr int N = 4; typedef f32x4 type; };
template <> struct Vec<bf16_t> { static constexpr int N = 8; typedef bf16x8 type; };

template <typename T> __device__ __forceinline__ void load_vec(const T* p, float* out) {
  typename Vec<T>::type v = *reinterpret_cast<const typename Vec<T>::type*>(p);
#pragma unroll
  for (int i = 0; i < Vec<T>::N; i++) out[i] = to_f<T>(v[i]);
}
template <typename T> __device__ __forceinline__ void store_vec(T* p, const float* in) {
  typename Vec<T>::type v;
#pragma unroll
  for (int i = 0; i < Vec<T>::N; i++) v[i] = from_f<T>(in[i]);
  *reinterpret_cast<typename Vec<T>::type*>(p) = v;
}
template <typename T> static bool vec_ok(const void* p, int64_t ld) {
  return ((uintptr_t)p % 16 == 0) && (ld % Vec<T>::N == 0);
}

#define DISPATCH_T(mode, ...) do { if ((mode) == AS_FP32) { typedef float T; __VA_ARGS__; } \
  else { typedef bf16_t T; __VA_ARGS__; } } while (0)

// ---- GEMM (gemm.hip) ------------------------------------------------------
// GemmParams, what one product is, lies in gemm_items.h
// the hand-scheduled kernel would take this product (whole 256 x 256 tiles, K in 64-wide steps, alignment)
bool gemm_rd_applies(int mode, const GemmParams& p);
// the launch (p.nn set) would go to a kernel that reads B as [K, N]: the hand-scheduled one, or (float operands) gemm_f32_kernel where it pays
bool gemm_nn_applies(int mode, int variant, const GemmParams& p);
bool gemm_tn_applies(int mode, int variant, const GemmParams& p);
// floats of scratch (GemmParams::tail_part given by the caller through `tail_ws`) that let the launcher split the last round
constexpr size_t kGemmTailFloats = (size_t)128 * 2 * 256 * 256;
int launch_gemm(as_ctx* ctx, int mode, int variant, const GemmParams& p, hipStream_t st);
// live rows = *p.m_dev - m_off, clamped to [0, p.M]
int launch_gemm_off(as_ctx* ctx, int mode, int variant, const GemmParams& p, int m_off, hipStream_t st);

int launch_gemm_batch(as_ctx* ctx, int mode, const GemmParams& p, hipStream_t st);   // GemmParams::nbat

int launch_feed_probe(as_ctx* ctx, int k, const void* buf, size_t span, int iters, int blocks, int* sink, hipStream_t st);
int launch_mfma_peak(as_ctx* ctx, int iters, int blocks, float* sink, hipStream_t st);

// ---- adapter gradients (lora_grad.hip) ---------------------------------------
// C[m*sm + j*sj] = alpha * sum_t X[t, m] * UT[j, t]  (bf16 X row-major, float C); UT is U token-major with rows of ldu tokens, or, where
// tn_grads_take_rows(rank), U itself, rows of ldu columns of which 16 are read
bool tn_grads_take_rows(int r);
struct TnGrad { const void* X; int64_t ldx; const void* UT; int M; float alpha; float* C; int64_t sm, sj; int first_block; int64_t first_out; };
struct TnGradBatch { TnGrad m[6]; int n; int64_t ldu, total; };
size_t tn_grad_partial_floats(int n, const int* M, int items, int r);
int launch_tn_grads(as_ctx* ctx, TnGradBatch b, int n, int r, float* partial, size_t partial_floats, hipStream_t st);

// fp32 tier: C[m*sm + j*sj] = alpha * sum_t X[t, m] * U[t, j] for up to eight products of one rank r over the same n tokens; U
// rows hold r rounded up to 16 columns
struct PlainGrad { const float *X, *U; int64_t ldx, ldu; float* C; int64_t sm, sj, first_out; int M, first_block; float alpha; };
struct PlainGradBatch { PlainGrad m[8]; int n; int64_t total; };
size_t plain_grad_partial_floats(int n, int64_t cols, int r);      // cols: sum of M over the batch
int launch_plain_grads(as_ctx* ctx, PlainGradBatch b, int n, int r, float* partial, size_t partial_floats, hipStream_t st);

// ---- attention (attention.hip) -----------------------------------------------
struct AttnParams {
  int n, Hq, Hkv, dh;
  const int32_t* seg_start; const int32_t* seg_end;
  const void *q, *k, *v; int64_t ldq, ldkv;
  void* o; float* lse;
  const void* d_o; void *dq, *dk, *dv; float* delta;
  int max_seg;             // longest segment (host knowledge, sizes LDS of the plain kernels)
  // MFMA kernels: scratch for token-major copies ([column][token], row length ldT = tokens rounded up
  // to 64): forward needs Hkv*dh rows (V^T), backward (2*Hq + Hkv)*dh rows (K^T, Q^T, dO^T)
  void* t_scratch;
  const void *qT, *kT, *vT, *doT; int64_t ldT;   // filled by the launchers
  // optional launch orders (device arrays, longest workgroups first): order_q[i] = query tile of workgroup i
  // (tiles of attention_query_tile() tokens), order_k[i] = key block (256 keys) of workgroup i in the dK / dV launches
  const int32_t* order_q; const int32_t* order_k;
  // backward: when set, dq and dk leave the kernels already rotated back (the inverse of the rotary
  // embedding applied to q and k before attention): tables [position][dh / 2] of cos and sin, position = t - seg_start[t]
  const float* rope_cos; const float* rope_sin;
};
int launch_attention_fwd(as_ctx* ctx, int mode, int variant, const AttnParams& p, hipStream_t st);
int attention_query_tile(int n_q_heads, int n_kv_heads);   // tokens per workgroup of the forward and dQ MFMA kernels
int launch_attention_bwd(as_ctx* ctx, int mode, int variant, const AttnParams& p, hipStream_t st);

// ---- element-wise and friends (elementwise.hip) ---------------------------------
int launch_pack(as_ctx* ctx, const int32_t* h_tokens, const int32_t* h_cu, const uint8_t* h_mask, int n_out, int n_cu, int32_t* d_tokens, int32_t* d_cu, uint8_t* d_mask, hipStream_t st);
// tok_c[i], mask_c[i] = tok[src], mask[src] with src = src_start[s] + (i - cu_c[s]) for the kept segment s holding i
int launch_compact(as_ctx* ctx, const int32_t* tok, const uint8_t* mask, const int32_t* cu_c, const int32_t* src_start,
                   int n_seg, int n, int32_t* tok_c, uint8_t* mask_c, hipStream_t st);
constexpr int kTargetBlock = 256;                          // tokens of a block of StepBegin::block_targets
int launch_rmsnorm_fwd(as_ctx* ctx, int mode, int n, int d, const void* x, const int32_t* row_idx,
                       const int* n_dev, const void* g, float eps, void* y, float* rstd, hipStream_t st);
// dx[t] = vjp(dy[row_of(t)]) + add[t]; src_pos (optional) maps t -> row of dy or -1 (then dx = add or 0)
int launch_rmsnorm_bwd(as_ctx* ctx, int mode, int n, int d, const void* dy, const int32_t* src_pos,
                       const void* x, const void* g, const float* rstd, const void* add, void* dx,
                       hipStream_t st);
// the same, and dg = sum_t dy[t] x[t] rstd[t] (partial: n_part rows of d floats)
int launch_rmsnorm_bwd_gain(as_ctx* ctx, int mode, int n, int d, const void* dy, const int32_t* src_pos, const void* x, const void* g,
                            const float* rstd, const void* add, void* dx, float* partial, int n_part, float* dg, hipStream_t st);
int launch_rope(as_ctx* ctx, int mode, int n, int n_heads, int dh, void* x, int64_t ldx,
                const int32_t* seg_start, const float* cosb, const float* sinb, hipStream_t st);
// NF4 block quantisation (quant.hip)
int launch_nf4_quantize(as_ctx* ctx, int mode, const void* w, int64_t numel, uint8_t* codes, float* absmax, hipStream_t st);
int launch_nf4_dequantize(as_ctx* ctx, int mode, const uint8_t* codes, const float* absmax, int64_t numel, void* out, hipStream_t st);
// out[c, r] = the dequantised element (r, c) of a [rows, cols] matrix (bf16), where nf4_transposed_ok
bool nf4_transposed_ok(int mode, const uint8_t* codes, int rows, int cols, const void* out, int64_t ldo);
// up to three quantised matrices [rows, cols] and where their values go; first: set by the launcher
struct Nf4Piece { const uint8_t* codes; const float* absmax; void* out; int rows, cols, first; };
struct Nf4Batch { Nf4Piece m[3]; int n; };
int launch_nf4_dequantize_batch(as_ctx* ctx, int mode, Nf4Batch b, hipStream_t st);
int launch_nf4_dequantize_transposed(as_ctx* ctx, Nf4Batch b, int64_t ldo, hipStream_t st);   // all with the same cols, each nf4_transposed_ok;
// mixture-of-experts routing and row grouping (moe.hip)
int launch_moe_route(as_ctx* ctx, const float* logit, int n, int E, int32_t* sel, float* w, hipStream_t st);
int launch_moe_permute(as_ctx* ctx, const int32_t* sel, int n, int E, int32_t* eoff, int32_t* pos, int32_t* perm, hipStream_t st);
int launch_moe_gather(as_ctx* ctx, int mode, const void* src, const int32_t* perm, const float* w, int rows, int d, void* out, hipStream_t st);
int launch_moe_combine(as_ctx* ctx, int mode, const void* res, const void* y, const int32_t* pos, const float* w, int n, int d,
                       void* out, hipStream_t st);
// out[t] = y[pos[2t]] + y[pos[2t+1]] + dlogit[t] Wr + du[t] A: the gradient of a sparse layer's input from its experts' and its router's (adapter of
// rank r, rows of du rp apart; r = 0: none), where moe_combine_router_ok
bool moe_combine_router_ok(int mode, int d, int r, const void* y, const void* Wr, const void* A, const void* out);
int launch_moe_combine_router(as_ctx* ctx, int mode, const void* y, const int32_t* pos, const int32_t* sel, const void* dlogit, int E, const void* Wr,
                              const void* du, int rp, const void* A, int r, int n, int d, void* out, hipStream_t st);
int launch_moe_dlogit(as_ctx* ctx, int mode, const void* dy, const void* y, const int32_t* pos, const int32_t* sel, const float* w,
                      int n, int d, int Epad, void* dlogit, hipStream_t st);
int launch_swiglu_fwd(as_ctx* ctx, int mode, int64_t n, int F, const void* gu, void* m, hipStream_t st);
int launch_swiglu_bwd(as_ctx* ctx, int mode, int64_t n, int F, const void* dm, const void* gu, void* dgu, void* m_out, hipStream_t st);
// the same with the adapter products of what they write, rank up to 16, from 4096 tokens on: u [n, rp] = m A^T; du [n, 2 rp] = dgate Bg | dup Bu; the adapters as PrepMatrix::frag
bool swiglu_adapter_ok(int mode, int n, int F, int r, std::initializer_list<const void*> ptrs);
int launch_swiglu_fwd_adapter(as_ctx* ctx, int n, int F, const void* gu, void* m, const void* fragA, int rp, void* u, hipStream_t st);
int launch_swiglu_bwd_adapter(as_ctx* ctx, int n, int F, const void* dm, const void* gu, void* dgu, void* m_out, const void* fragBg, const void* fragBu, int rp, void* du,
                              hipStream_t st);
// products of token rows with adapters of rank up to 16: u[i] [n, rp columns, rows of ldu] = x[i] [n, K[i], rows of ldx] times the adapter frag[i] (PrepMatrix::frag);
// one_x: all on x[0].  K in multiples of 64
struct AdapterRows { const void* x[3]; const void* frag[3]; void* u[3]; int K[3]; int64_t ldx, ldu; int n, rp; };
bool adapter_rows_ok(int mode, int r, int64_t ldx, std::initializer_list<const void*> ptrs);
int launch_adapter_rows(as_ctx* ctx, const AdapterRows& p, int items, bool one_x, hipStream_t st);
// out[c, r] = in[r, c] for r < rows_pad, reading zero for r >= rows (and, with rows_dev, for rows at
// or past *rows_dev - row_off)
int launch_transpose(as_ctx* ctx, int mode, int rows, int rows_pad, int cols, const void* in, int64_t ldi, void* out,
                     int64_t ldo, const int* rows_dev, int row_off, hipStream_t st);
int launch_transpose_qs(as_ctx* ctx, int mode, int rows, int rows_pad, int cols, const void* in, int64_t ldi, void* out,
                        int64_t ldo, hipStream_t st);
// two matrices of one shape and layout in one launch where the 16-bit kernel takes them
int launch_transpose_pair(as_ctx* ctx, int mode, int rows, int rows_pad, int cols, const void* in, const void* in2, int64_t ldi,
                          void* out, void* out2, int64_t ldo, hipStream_t st);
// out[rows_pad, cols_pad] (type T, row stride ldo) = scale * in[rows, cols] (float), zero in the
// padding; out_t (row stride ldo_t) receives the transpose.  frag (may be NULL; bf16, both padded sizes multiples of 64): the
// first 16 of the rank, which is the row of `in` (frag_rank_rows) or its column, as operands of v_mfma_f32_16x16x32_bf16, 512 elements for every
// 32 of the contraction.
struct PrepMatrix { const float* in; void *out, *out_t; int64_t ldo, ldo_t; int rows, cols, rows_pad, cols_pad; float scale; int first_tile; void* frag; int frag_rank_rows; };
constexpr int kPrepBatch = 40;                             // a batch is a kernel argument (3.4 KB)

struct PrepBatch { PrepMatrix m[kPrepBatch]; int n, n_tiles; };
int launch_lora_prep_batch(as_ctx* ctx, int mode, const PrepBatch& b, hipStream_t st);
// What a step needs before its first layer: a token's segment, the number of targets among every kTargetBlock tokens (mask: tokens that bear
// loss; a target is predicted by the token before it), the rotary table, the embedded tokens, and a batch of adapters (b.n may be 0)
struct StepBegin {
  const int32_t* cu; int n_seg; const uint8_t* mask; int n; int32_t *seg_start, *seg_end, *block_targets;
  int max_pos, dh; double rope_base; float *cosb, *sinb;
  const int32_t* tok; int d; const void* embed; void* h; int vec;
};
int launch_step_begin(as_ctx* ctx, int mode, const StepBegin& s, const PrepBatch& b, hipStream_t st);
int launch_fill_zero(as_ctx* ctx, void* p, size_t bytes, hipStream_t st);
int launch_zero_tail_rows(as_ctx* ctx, int rows, const int* n_dev, int off, void* a, int64_t lda, int ca, void* b, int64_t ldb, int cb, hipStream_t st);
int launch_select_targets(as_ctx* ctx, const int32_t* seg_end, const int32_t* block_targets, const uint8_t* mask, const int32_t* tok,
                          int n, int32_t* tgt_idx, int32_t* tgt_pos, int32_t* labels, int32_t* count,
                          hipStream_t st);
// one row of logits per target: loss_t, and P = (softmax - onehot) / count written as T
int launch_ce_rows(as_ctx* ctx, int mode, const float* logits, int rows_cap, int V, int row0,
                   const int32_t* labels, const int32_t* count, float* loss_rows, const float* row_w, void* P, hipStream_t st);
// preference loss (dpo.hip)
int launch_seq_logp(as_ctx* ctx, const float* loss_rows, const int32_t* tgt_idx, const int32_t* count, const int32_t* cu,
                    const int32_t* kept_of, int n_seg, float* logp, hipStream_t st);
int launch_dpo_pairs(as_ctx* ctx, const int32_t* pairs, int n_pairs, const float* logp, const float* ref, float beta, int n_seg,
                     const int32_t* kept_of, int n_kept, float* w_kept, float* stats, hipStream_t st);
// again (may be NULL): the number of rows, or 0 if there are at most `held`
int launch_dpo_row_weights(as_ctx* ctx, const int32_t* tgt_idx, const int32_t* count, const int32_t* cu, int n_kept,
                           const float* w_kept, int n, float* row_w, int held, int32_t* again, hipStream_t st);
int launch_fill_float(as_ctx* ctx, float* p, int n, float v, hipStream_t st);
// head without stored logits: z_lab[row] = hf[row] . W[labels[row]] for rows < *count; then per row the log-sum-exp from the
// per-block statistics of the GEMM and loss = lse - z_lab
int launch_label_logit(as_ctx* ctx, const void* hf, const void* W, int d, const int32_t* labels, const int32_t* count, int rows_cap,
                       float* zlab, hipStream_t st);
int launch_ce_finish(as_ctx* ctx, const float* part, int nblk, int row0, int rows_cap, const int32_t* count, const float* zlab,
                     float* lse, float* loss_rows, hipStream_t st);
int launch_soft_finish(as_ctx* ctx, const float* part, int V, int row0, int rows_cap, const int32_t* count, const float* zlab, const int32_t* labels,
                       float* inv, float* loss_rows, void* E, hipStream_t st);
int launch_loss_finalize(as_ctx* ctx, const float* loss_rows, const int32_t* count, float* loss,
                         float* loss_sum, hipStream_t st);
int launch_splitk_reduce(as_ctx* ctx, const float* partial, int splitk, int64_t mn, int N, float alpha,
                         float* C, int64_t ldc, hipStream_t st);
// one tensor of a multi-tensor update; a workgroup takes kAdamChunk elements of it
struct AdamTensor { float* w; bf16_t* w_lowp; const float* g; float* m; float* v; int64_t n; float wd; int first_chunk; };
// a batch of tensors travels as a kernel argument: no table in device memory, nothing to allocate or to keep alive
constexpr int kAdamBatch = 64, kAdamChunk = 4096;
struct AdamBatch { AdamTensor t[kAdamBatch]; int n; int n_chunks; };
int launch_adamw_batch(as_ctx* ctx, const AdamBatch& b, float lr, float b1, float b2, float eps, float bc1, float bc2, hipStream_t st);
// scratch: 2n int32; aux: embed_bwd_aux_bytes(n, d), 256-byte aligned
size_t embed_bwd_aux_bytes(int n, int d);
int launch_embed_bwd(as_ctx* ctx, int mode, const int32_t* tok, int n, int d, int V, const void* dh,
                     int32_t* scratch, void* aux, size_t aux_bytes, float* dE, hipStream_t st);
