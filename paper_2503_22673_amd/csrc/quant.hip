// 4-bit NormalFloat block quantisation of frozen projection weights (quantised base + LoRA, paper
// Section 4.5 and Table 3; format of the public QLoRA description): blocks of 64 consecutive elements,
// one float absolute maximum per block, per element the index of the nearest of 16 fixed levels.
#include "common.h"

namespace {
// the 16 levels (quantiles of N(0,1) normalised to [-1, 1], with an exact zero)
__device__ __constant__ float kLevel[16] = {
    -1.0f, -0.6961928009986877f, -0.5250730514526367f, -0.39491748809814453f,
    -0.28444138169288635f, -0.18477343022823334f, -0.09105003625154495f, 0.0f,
    0.07958029955625534f, 0.16093020141124725f, 0.24611230194568634f, 0.33791524171829224f,
    0.44070982933044434f, 0.5626170039176941f, 0.7229568362236023f, 1.0f};

// one wave per 64-element block, lane i owns element i
template <typename T>
__global__ void nf4_quantize_kernel(const T* __restrict__ w, int64_t n_blocks, uint8_t* __restrict__ codes, float* __restrict__ absmax) {
  const int lane = threadIdx.x & 63;
  const int64_t blk = (int64_t)blockIdx.x * (blockDim.x / 64) + threadIdx.x / 64;
  if (blk >= n_blocks) return;
  const float v = to_f<T>(w[blk * 64 + lane]);
  float m = fabsf(v);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
  const float x = v / (m > 0.f ? m : 1.f);
  int code = 0;
#pragma unroll
  for (int i = 0; i < 15; i++) code += (x >= (kLevel[i] + kLevel[i + 1]) * 0.5f) ? 1 : 0;   // a midpoint goes to the higher level
  const int hi = __shfl_down(code, 1, 64);
  if ((lane & 1) == 0) codes[blk * 32 + (lane >> 1)] = (uint8_t)(code | (hi << 4));
  if (lane == 0) absmax[blk] = m;
}

// one thread per 8 elements: four code bytes in, 8 values of type T out
template <typename T>
__global__ void nf4_dequantize_kernel(const uint8_t* __restrict__ codes, const float* __restrict__ absmax, int64_t n8, T* __restrict__ out) {
  __shared__ float lut[16];
  if (threadIdx.x < 16) lut[threadIdx.x] = kLevel[threadIdx.x];
  __syncthreads();
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n8) return;
  const uint32_t c = *reinterpret_cast<const uint32_t*>(codes + i * 4);
  const float a = absmax[i >> 3];
  T* o = out + i * 8;
#pragma unroll
  for (int e = 0; e < 8; e++) o[e] = from_f<T>(lut[(c >> (4 * e)) & 15] * a);
}

// the matrix of a batch that a block works on
__device__ __forceinline__ int piece_of(const Nf4Batch& b, int block) { return table_item<3>(b.n, block, [&](int k) { return b.m[k].first; }); }

// bf16, `out` 16-byte and `codes` 4-byte aligned, the matrices of one input group (q, k, v; gate, up) in one launch.
// Memory bound: 0.5 bytes in, 2 out per weight.  A wave takes kVecRuns runs of 512 elements one after the other, so that a load reads 256 and a store
// writes 1024 bytes in a row, and all its loads are under way together: the fourteen matrices of two
// 1B layers in eight launches 95 -> 80 us (two 16-byte stores 32 bytes apart a lane before).
constexpr int kVecRuns = 4;
__global__ __launch_bounds__(256) void nf4_dequantize_vec_kernel(const Nf4Batch b) {
  __shared__ float lut[16];
  if (threadIdx.x < 16) lut[threadIdx.x] = kLevel[threadIdx.x];
  __syncthreads();
  const Nf4Piece& m = b.m[piece_of(b, blockIdx.x)];
  const uint8_t* codes = m.codes; const float* absmax = m.absmax; bf16_t* out = (bf16_t*)m.out;
  const int64_t n8 = (int64_t)m.rows * m.cols / 8;         // groups of eight elements
  const int64_t i0 = ((int64_t)((int)blockIdx.x - m.first) * 4 + (threadIdx.x >> 6)) * (64 * kVecRuns) + (threadIdx.x & 63);
  uint32_t c[kVecRuns]; float a[kVecRuns];
#pragma unroll
  for (int k = 0; k < kVecRuns; k++) {
    const int64_t i = i0 + 64 * k;
    if (i < n8) { c[k] = *reinterpret_cast<const uint32_t*>(codes + i * 4); a[k] = absmax[i >> 3]; }
  }
#pragma unroll
  for (int k = 0; k < kVecRuns; k++) {
    const int64_t i = i0 + 64 * k;
    bf16x8 v;
#pragma unroll
    for (int e = 0; e < 8; e++) v[e] = (bf16_t)(lut[(c[k] >> (4 * e)) & 15] * a[k]);
    if (i < n8) *reinterpret_cast<bf16x8*>(out + i * 8) = v;
  }
}

// Dequantised and transposed in one pass: out[c, r] = level * absmax of element (r, c) of a [rows, cols] matrix, for the
// backward products, which contract over the rows.  A workgroup takes 64 rows x 256 columns (whole 128-byte lines of codes),
// a wave 64 x 64 of them, a lane an 8 x 8 block: eight 4-byte code reads, eight 16-byte output rows; no dense copy in between.
// Needs rows a multiple of 8, cols of 64 (a block of 64 codes lies in one row), ldo of 8, aligned bases.
// The 11 matrices of two 1B layers that the backward needs: 203 us as a dense copy and its transpose, 96 us so, and those of one product
// (gate over up, q over k over v: their outputs side by side) in one launch.
__global__ __launch_bounds__(256) void nf4_dequantize_transposed_kernel(const Nf4Batch b, int64_t ldo) {
  __shared__ float lut[16];
  if (threadIdx.x < 16) lut[threadIdx.x] = kLevel[threadIdx.x];
  __syncthreads();
  const Nf4Piece& m = b.m[piece_of(b, blockIdx.y)];
  const uint8_t* codes = m.codes; const float* absmax = m.absmax; bf16_t* out = (bf16_t*)m.out;
  const int rows = m.rows, cols = m.cols;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int c = blockIdx.x * 256 + wave * 64 + (lane & 7) * 8, r = ((int)blockIdx.y - m.first) * 64 + (lane >> 3) * 8;
  if (c >= cols || r >= rows) return;
  uint32_t code[8]; float a[8];
#pragma unroll
  for (int i = 0; i < 8; i++) {
    const int64_t e = (int64_t)(r + i) * cols + c;
    code[i] = *reinterpret_cast<const uint32_t*>(codes + (e >> 1));
    a[i] = absmax[e >> 6];
  }
#pragma unroll
  for (int q = 0; q < 8; q++) {
    bf16x8 v;
#pragma unroll
    for (int i = 0; i < 8; i++) v[i] = (bf16_t)(lut[(code[i] >> (4 * q)) & 15] * a[i]);
    *reinterpret_cast<bf16x8*>(out + (int64_t)(c + q) * ldo + r) = v;
  }
}
}  // namespace

int launch_nf4_quantize(as_ctx* ctx, int mode, const void* w, int64_t numel, uint8_t* codes, float* absmax, hipStream_t st) {
  if (numel <= 0) return AS_OK;
  if (numel % 64) return as_fail(ctx, AS_ERR_SHAPE, "nf4: the element count must be a multiple of 64");
  const int64_t nb = numel / 64;
  if (mode == AS_FP32) nf4_quantize_kernel<float><<<(unsigned)cdiv(nb, 4), 256, 0, st>>>((const float*)w, nb, codes, absmax);
  else nf4_quantize_kernel<bf16_t><<<(unsigned)cdiv(nb, 4), 256, 0, st>>>((const bf16_t*)w, nb, codes, absmax);
  AS_LAUNCH_CHECK(ctx);
  return AS_OK;
}

int launch_nf4_dequantize(as_ctx* ctx, int mode, const uint8_t* codes, const float* absmax, int64_t numel, void* out, hipStream_t st) {
  if (numel <= 0) return AS_OK;
  if (numel % 64) return as_fail(ctx, AS_ERR_SHAPE, "nf4: the element count must be a multiple of 64");
  if ((uintptr_t)codes % 4) return as_fail(ctx, AS_ERR_SHAPE, "nf4: the code array must be 4-byte aligned");
  const int64_t n8 = numel / 8;
  if (mode == AS_FP32) nf4_dequantize_kernel<float><<<(unsigned)cdiv(n8, 256), 256, 0, st>>>(codes, absmax, n8, (float*)out);
  else if (numel / 64 <= INT32_MAX && (uintptr_t)out % 16 == 0 && (uintptr_t)codes % 8 == 0) {
    Nf4Batch b{}; b.n = 1; b.m[0] = {codes, absmax, out, (int)(numel / 64), 64, 0};
    return launch_nf4_dequantize_batch(ctx, mode, b, st);
  } else nf4_dequantize_kernel<bf16_t><<<(unsigned)cdiv(n8, 256), 256, 0, st>>>(codes, absmax, n8, (bf16_t*)out);
  AS_LAUNCH_CHECK(ctx);
  return AS_OK;
}

int launch_nf4_dequantize_batch(as_ctx* ctx, int mode, Nf4Batch b, hipStream_t st) {
  bool vec = mode == AS_BF16;
  for (int k = 0; k < b.n; k++) vec = vec && b.m[k].cols % 64 == 0 && !((uintptr_t)b.m[k].out % 16) && !((uintptr_t)b.m[k].codes % 8);
  if (!vec) {
    for (int k = 0; k < b.n; k++) {
      const int rc = launch_nf4_dequantize(ctx, mode, b.m[k].codes, b.m[k].absmax, (int64_t)b.m[k].rows * b.m[k].cols, b.m[k].out, st);
      if (rc) return rc;
    }
    return AS_OK;
  }
  int64_t blocks = 0;
  for (int k = 0; k < b.n; k++) { b.m[k].first = (int)blocks; blocks += cdiv((int64_t)b.m[k].rows * b.m[k].cols, 8 * 256 * kVecRuns); }
  if (blocks <= 0) return AS_OK;
  if (blocks > INT32_MAX) return as_fail(ctx, AS_ERR_SHAPE, "nf4: too many elements for one launch");
  nf4_dequantize_vec_kernel<<<(unsigned)blocks, 256, 0, st>>>(b);
  AS_LAUNCH_CHECK(ctx);
  return AS_OK;
}

bool nf4_transposed_ok(int mode, const uint8_t* codes, int rows, int cols, const void* out, int64_t ldo) {
  return mode == AS_BF16 && rows % 8 == 0 && cols % 64 == 0 && ldo % 8 == 0 && (uintptr_t)out % 16 == 0 && (uintptr_t)codes % 4 == 0;
}
int launch_nf4_dequantize_transposed(as_ctx* ctx, Nf4Batch b, int64_t ldo, hipStream_t st) {
  int64_t blocks = 0;
  for (int k = 0; k < b.n; k++) { b.m[k].first = (int)blocks; blocks += cdiv(b.m[k].rows, 64); }
  if (blocks <= 0 || b.m[0].cols <= 0) return AS_OK;
  nf4_dequantize_transposed_kernel<<<dim3((unsigned)cdiv(b.m[0].cols, 256), (unsigned)blocks), 256, 0, st>>>(b, ldo);
  AS_LAUNCH_CHECK(ctx);
  return AS_OK;
}
