// Adapter gradients: C[m, j] = alpha * sum_t X[t, m] * U[t, j], a product contracted over TOKENS,
// i.e. over the row index of both operands (dB = s dy^T u with X = dy, U = u; dA^T = x^T du with
// X = x, U = du).  X is a big row-major activation ([tokens, M] bf16, up to 14336 columns), U is
// 64 columns wide at most, so the kernel is a single streaming pass over X at HBM speed.
//
// Matrix cores want the contraction index contiguous per lane.  Instead of transposing X through
// memory, each lane loads an 8-token x 8-column block (eight 16-byte loads, 256 B contiguous per
// 16 lanes and token) and transposes it in registers (v_perm), which yields the A operands of eight
// v_mfma_f32_16x16x32_bf16 -- one per column of the block; MFMA row m then stands for column
// c0 + 8 m + q of X.  U comes from its small token-major copy ([j][token]), one 16-byte load per
// lane and 16-column block; of rank 16 and less, as it is: 32 tokens of 16 columns are one 16-byte load a lane, pass through a kilobyte of the wave's LDS and
// come back through the transposing reads
// (copies of both for every input group, a launch of 4.5 us each at 626 tokens: a step of two 1B layers 1.334 -> 1.305 ms).  Token ranges (splits) go to a partial buffer reduced in split order.
// The products of an input group (dB and dA of q, k, v) are one launch and one sum: each of them alone is a ramp of a few
// microseconds around little work when tokens are few: steps of two 1B layers with seven adapters at 1003 tokens 1708 -> 1555 us,
// at 32768 tokens 18.19 -> 17.68 ms.
#include "common.h"
#include <cmath>

namespace {
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;

struct TnParams {
  TnGradBatch b;
  int n, r;
  float* partial;                    // [splits][every product's M x r behind one another]
  int steps_per_split, total_steps;  // 32-token steps
};

#include "lora_grad_loop.inc"
template <int NB>
__global__ __launch_bounds__(256) void lora_grad_tn_kernel(TnParams batch) {
  const int it = table_item<6>(batch.b.n, (int)blockIdx.x, [&](int k) { return batch.b.m[k].first_block; });
  struct { const bf16_t* X; int64_t ldx; const bf16_t* UT; int64_t ldu; int n, M, r, steps_per_split, total_steps; float* partial; int64_t split_stride; } p;
  {
    const TnGrad& m = batch.b.m[it];
    p.X = (const bf16_t*)m.X; p.ldx = m.ldx; p.UT = (const bf16_t*)m.UT; p.ldu = batch.b.ldu; p.n = batch.n; p.M = m.M; p.r = batch.r;
    p.steps_per_split = batch.steps_per_split; p.total_steps = batch.total_steps; p.partial = batch.partial + m.first_out; p.split_stride = batch.b.total;
  }
  const int tid = threadIdx.x, lane = tid & 63, lm = lane & 15, lg = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // the four waves of a workgroup take four neighbouring 128-column slabs and the same tokens, so that
  // the workgroup reads 1 KB of every token row at a time
  const int slab = ((int)blockIdx.x - batch.b.m[it].first_block) * 4 + wave, split = blockIdx.y;
  if (slab * 128 >= p.M) return;
  const int col = slab * 128 + 8 * lm;
  const bool col_ok = col < p.M;
  // NB = 1: U [token][16 of its columns] as rows
  constexpr bool ROWS = NB == 1;
  __shared__ __align__(16) bf16_t turn[ROWS ? 4 * 512 : 8];
  bf16_t* mine = turn + (ROWS ? wave * 512 : 0);
  f32x4 acc[8][NB];
#pragma unroll
  for (int q = 0; q < 8; q++)
#pragma unroll
    for (int nb = 0; nb < NB; nb++) acc[q][nb] = (f32x4){0.f, 0.f, 0.f, 0.f};
  const int s_end = min((split + 1) * p.steps_per_split, p.total_steps);
  auto load = [&](int step, u32x4 (&x)[8], bf16x8 (&b)[NB]) {
    const int t0 = step * 32 + 8 * lg;
#pragma unroll
    for (int r = 0; r < 8; r++) {
      const int t = t0 + r;
      const bool ok = col_ok && t < p.n;
      const u32x4 v = *reinterpret_cast<const u32x4*>(p.X + (int64_t)(ok ? t : 0) * p.ldx + (ok ? col : 0));
      x[r] = ok ? v : (u32x4){0u, 0u, 0u, 0u};
    }
    if constexpr (ROWS) {
      const int t = step * 32 + (lane >> 1);
      b[0] = *reinterpret_cast<const bf16x8*>(p.UT + (int64_t)min(t, p.n - 1) * p.ldu + (lane & 1) * 8);
      if (t >= p.n) b[0] = __builtin_bit_cast(bf16x8, (u32x4){0u, 0u, 0u, 0u});
    } else {
#pragma unroll
      for (int nb = 0; nb < NB; nb++) b[nb] = *reinterpret_cast<const bf16x8*>(p.UT + (int64_t)(nb * 16 + lm) * p.ldu + t0);
    }
  };
  // rows as they were loaded -> the operand: column lm of tokens 8 lg .. + 7 (LDS operations of a wave complete in order)
  auto operand = [&](bf16x8& b) {
    if constexpr (ROWS) {
      *reinterpret_cast<bf16x8*>(mine + lane * 8) = b;
      asm volatile("" ::: "memory");
      const bf16_t* at = mine + (8 * lg + (lm >> 2)) * 16 + (lm & 3) * 4;
      const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((__attribute__((address_space(3))) bf16x4*)at);
      const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((__attribute__((address_space(3))) bf16x4*)(at + 64));
      b = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
      asm volatile("" ::: "memory");
    }
  };
  auto compute = [&](const u32x4 (&x)[8], const bf16x8 (&b)[NB]) {
#pragma unroll
    for (int q = 0; q < 8; q++) {
      // column q of the 8x8 block: dword d of the operand = (x[2d][q], x[2d+1][q])
      u32x4 a;
#pragma unroll
      for (int d = 0; d < 4; d++)
        a[d] = __builtin_amdgcn_perm(x[2 * d + 1][q >> 1], x[2 * d][q >> 1], (q & 1) ? 0x07060302u : 0x05040100u);
      const bf16x8 av = __builtin_bit_cast(bf16x8, a);
#pragma unroll
      for (int nb = 0; nb < NB; nb++) acc[q][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, b[nb], acc[q][nb], 0, 0, 0);
    }
  };
  int step = split * p.steps_per_split;
  // Whole steps of a full-width slab with all four column blocks of the narrow operand run in the generated loop
  // (gen_lora_grad_loop.py: four register sets, three steps in flight); what is left -- a last step that runs past the
  // tokens, narrower operands, a ragged slab -- takes the loop below.
  if constexpr (NB == 4) {
    const int s_full = min(s_end, p.n / 32);
    if (p.M % 128 == 0 && s_full > step) {
      uint32_t vx[8], vu[4];
#pragma unroll
      for (int r = 0; r < 8; r++) vx[r] = (uint32_t)((((int64_t)(8 * lg + r)) * p.ldx + col) * 2);
#pragma unroll
      for (int nb = 0; nb < 4; nb++) vu[nb] = (uint32_t)((((int64_t)(nb * 16 + lm)) * p.ldu + 8 * lg) * 2);
      const uint64_t gx = (uint64_t)(p.X + (int64_t)step * 32 * p.ldx), gu = (uint64_t)(p.UT + (int64_t)step * 32);
      const uint32_t stride = (uint32_t)(32 * p.ldx * 2), nsteps = (uint32_t)(s_full - step);
      asm volatile(LORA_GRAD_LOOP_ASM
                   : "+a"(acc[0][0]), "+a"(acc[0][1]), "+a"(acc[0][2]), "+a"(acc[0][3]), "+a"(acc[1][0]), "+a"(acc[1][1]), "+a"(acc[1][2]), "+a"(acc[1][3]),
                     "+a"(acc[2][0]), "+a"(acc[2][1]), "+a"(acc[2][2]), "+a"(acc[2][3]), "+a"(acc[3][0]), "+a"(acc[3][1]), "+a"(acc[3][2]), "+a"(acc[3][3]),
                     "+a"(acc[4][0]), "+a"(acc[4][1]), "+a"(acc[4][2]), "+a"(acc[4][3]), "+a"(acc[5][0]), "+a"(acc[5][1]), "+a"(acc[5][2]), "+a"(acc[5][3]),
                     "+a"(acc[6][0]), "+a"(acc[6][1]), "+a"(acc[6][2]), "+a"(acc[6][3]), "+a"(acc[7][0]), "+a"(acc[7][1]), "+a"(acc[7][2]), "+a"(acc[7][3])
                   : "v"(vx[0]), "v"(vx[1]), "v"(vx[2]), "v"(vx[3]), "v"(vx[4]), "v"(vx[5]), "v"(vx[6]), "v"(vx[7]),
                     "v"(vu[0]), "v"(vu[1]), "v"(vu[2]), "v"(vu[3]), "s"(gx), "s"(gu), "s"(stride), "s"(nsteps)
                   : LORA_GRAD_LOOP_CLOBBERS);
      step = s_full;
    }
  }
  // two register sets: the block of the next step is in flight while this one is multiplied
  u32x4 xa[8], xb[8];
  bf16x8 ba[NB], bb[NB];
  if (step < s_end) load(step, xa, ba);
  for (; step < s_end; step += 2) {
    if (step + 1 < s_end) load(step + 1, xb, bb);
    operand(ba[0]);
    compute(xa, ba);
    if (step + 1 >= s_end) break;
    if (step + 2 < s_end) load(step + 2, xa, ba);
    operand(bb[0]);
    compute(xb, bb);
  }
  // accumulator row 4*lg + i of MFMA q is column c0 + 8*(4*lg + i) + q; its column is j = nb*16 + lm
  float* out = p.partial + (int64_t)split * p.split_stride;
#pragma unroll
  for (int q = 0; q < 8; q++)
#pragma unroll
    for (int nb = 0; nb < NB; nb++) {
      const int j = nb * 16 + lm;
#pragma unroll
      for (int i = 0; i < 4; i++) {
        const int m = slab * 128 + 8 * (4 * lg + i) + q;
        if (m < p.M && j < p.r) out[(int64_t)m * p.r + j] = acc[q][nb][i];
      }
    }
}

__global__ void tn_reduce_kernel(const TnGradBatch b, const float* __restrict__ partial, int splits, int r) {
  // a thread owns four consecutive elements (M is a multiple of 8) and adds the splits in order; eight loads in flight
  const int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * 4, total = b.total;
  if (i >= total) return;
  const TnGrad& m = b.m[table_item<6>(b.n, i, [&](int k) { return b.m[k].first_out; })];
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  int s = 0;
  for (; s + 8 <= splits; s += 8) {
    f32x4 v[8];
#pragma unroll
    for (int k = 0; k < 8; k++) v[k] = *reinterpret_cast<const f32x4*>(partial + (int64_t)(s + k) * total + i);
#pragma unroll
    for (int k = 0; k < 8; k++) acc += v[k];
  }
  for (; s < splits; s++) acc += *reinterpret_cast<const f32x4*>(partial + (int64_t)s * total + i);
#pragma unroll
  for (int k = 0; k < 4; k++) { const int64_t e = i - m.first_out + k; m.C[(e / r) * m.sm + (e % r) * m.sj] = m.alpha * acc[k]; }
}
}  // namespace

// One workgroup of four column blocks fits a CU (the accumulators fill the register file): the token range is split so that the
// launch is whole rounds of 256 workgroups, one per product (14336 columns alone: 28 x 9 = 252 workgroups; with 28 x 10 the last
// 24 ran alone and the launch took half as long again).  Short token ranges: a split of `s` steps costs their latency, its
// partial sums are written and read again, so the best split grows with the root of the range; with r 16, kernel and sum of the
// splits, at 16 steps per split and so: 1003 tokens x 2048: 16.4 and 8.2 us; 4000 x 2048: 17.6 and 12.1; 7500 x 512: 19.2 and
// 11.7; 15,500 x 2048: 24.3 and 21.3.  (Not trimmed to the steps that are used: the bound on partial sums must grow with n.)
static int tn_blocks(int M) { return (int)cdiv(cdiv(M, 128), 4); }
static int tn_splits(int n, int blocks, int items) {
  const int steps = (int)cdiv(n, 32);
  return (int)std::max<int64_t>(1, std::min<int64_t>(256 * items / blocks, (int64_t)std::sqrt(8.0 * steps)));
}

size_t tn_grad_partial_floats(int n, const int* M, int items, int r) {
  int blocks = 0; int64_t cols = 0;
  for (int i = 0; i < items; i++) { blocks += tn_blocks(M[i]); cols += M[i]; }
  return items ? (size_t)tn_splits(n, blocks, items) * cols * r : 0;
}

bool tn_grads_take_rows(int r) { return r <= 16; }
// C[m * sm + j * sj] = alpha * sum_t X[t, m] * U[t, j] for every product of the batch, U as rows or token-major (tn_grads_take_rows);  r <= 64, M a multiple of 8, ldx a multiple of 8.
int launch_tn_grads(as_ctx* ctx, TnGradBatch b, int n, int r, float* partial, size_t partial_floats, hipStream_t st) {
  if (n <= 0 || b.n <= 0 || r <= 0) return AS_OK;
  if (r > 64 || (b.ldu % 8) || ((uintptr_t)partial % 16)) return as_fail(ctx, AS_ERR_SHAPE, "lora_grad_tn: rank <= 64 and 8-element alignment needed");
  int blocks = 0; b.total = 0;
  for (int i = 0; i < b.n; i++) {
    TnGrad& m = b.m[i];
    if ((m.M % 8) || (m.ldx % 8) || ((uintptr_t)m.X % 16) || ((uintptr_t)m.UT % 16)) return as_fail(ctx, AS_ERR_SHAPE, "lora_grad_tn: rank <= 64 and 8-element alignment needed");
    m.first_block = blocks; m.first_out = b.total;
    blocks += tn_blocks(m.M); b.total += (int64_t)m.M * r;
  }
  const int steps = (int)cdiv(n, 32);
  const int per = (int)cdiv(steps, tn_splits(n, blocks, b.n)), splits = (int)cdiv(steps, per);
  if ((size_t)splits * b.total > partial_floats) return as_fail(ctx, AS_ERR_WORKSPACE, "lora_grad_tn: partial buffer too small");
  TnParams p{b, n, r, partial, per, steps};
  const int nb = (int)cdiv(r, 16);
  dim3 grid(blocks, splits);
  prof_begin(ctx, st, AS_K_LORA_GRAD, 2.0 * n * (double)b.total);
#define TN_LAUNCH(NB) { lora_grad_tn_kernel<NB><<<grid, 256, 0, st>>>(p); }
  switch (nb) { case 1: TN_LAUNCH(1) break; case 2: TN_LAUNCH(2) break; case 3: TN_LAUNCH(3) break; default: TN_LAUNCH(4) break; }
#undef TN_LAUNCH
  AS_LAUNCH_CHECK(ctx);
  tn_reduce_kernel<<<(unsigned)cdiv(b.total, 1024), 256, 0, st>>>(b, partial, splits, r);
  prof_end(ctx, st);
  AS_LAUNCH_CHECK(ctx);
  return AS_OK;
}

// ---- fp32 tier -------------------------------------------------------------------------------------------------------
// The same products with float operands, all those of one input group in one launch (a projection's dB and dA; the six of
// q, k, v), X and U read as they are.  A workgroup owns 16 columns of one X and 16 of its U; its 16 waves take every 16th group of
// four tokens each (v_mfma_f32_16x16x4f32: float products and sums; a lane loads its column of one token, 64 bytes a row), the loads of
// eight groups in flight, and are added in order through LDS.  More than 1024 tokens are split over grid.y, partial sums added in order by
// a second launch.  Bound by latency at the tier's sizes: two layers of four adapters at 478 tokens, four launches: 44 us with
// 64 columns per workgroup, FMAs and a chain of 30 tokens per wave (4 to 12 workgroups a launch), 21 us so.
constexpr int PG_WAVES = 16, PG_B = 16, PG_U = 8;
__global__ __launch_bounds__(PG_WAVES * 64) void plain_grad_kernel(const PlainGradBatch b, int n, int r, int splits, float* __restrict__ partial) {
  __shared__ __align__(16) f32x4 sh[PG_WAVES][64];
  const PlainGrad& m = b.m[table_item<8>(b.n, (int)blockIdx.x, [&](int k) { return b.m[k].first_block; })];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l15 = lane & 15, q = lane >> 4;
  const int nj = (r + PG_B - 1) / PG_B, blk = (int)blockIdx.x - m.first_block, col0 = (blk / nj) * PG_B, j0 = (blk % nj) * PG_B;
  const int per = (n + splits - 1) / splits, t_lo = blockIdx.y * per, t_hi = min(n, t_lo + per);
  const bool in_x = col0 + l15 < m.M, in_u = j0 + l15 < r;
  const float* X = m.X + (in_x ? col0 + l15 : 0); const float* U = m.U + (in_u ? j0 + l15 : 0);
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  for (int t = t_lo + 4 * wave; t < t_hi; t += 4 * PG_WAVES * PG_U) {
    float x[PG_U], u[PG_U];
#pragma unroll
    for (int k = 0; k < PG_U; k++) {
      const int tt = t + 4 * PG_WAVES * k + q;             // past the end: zeros in both operands
      x[k] = in_x && tt < t_hi ? X[(int64_t)tt * m.ldx] : 0.f;
      u[k] = in_u && tt < t_hi ? U[(int64_t)tt * m.ldu] : 0.f;
    }
#pragma unroll
    for (int k = 0; k < PG_U; k++) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(u[k], x[k], acc, 0, 0, 0);   // lane: column l15 of X, columns 4 q .. + 3 of U
  }
  sh[wave][lane] = acc;
  __syncthreads();
  if (threadIdx.x >= 256) return;
  const int src = threadIdx.x >> 2, e = threadIdx.x & 3;   // one element each
  float s = 0.f;
#pragma unroll
  for (int w = 0; w < PG_WAVES; w++) s += reinterpret_cast<const float*>(&sh[w][src])[e];
  const int col = col0 + (src & 15), j = j0 + 4 * (src >> 4) + e;
  if (col < m.M && j < r) {
    if (splits > 1) partial[(int64_t)blockIdx.y * b.total + m.first_out + (int64_t)col * r + j] = s;
    else m.C[(int64_t)col * m.sm + (int64_t)j * m.sj] = m.alpha * s;
  }
}
__global__ __launch_bounds__(256) void plain_grad_sum_kernel(const PlainGradBatch b, int r, int splits, const float* __restrict__ partial) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= b.total) return;
  const PlainGrad& m = b.m[table_item<8>(b.n, i, [&](int k) { return b.m[k].first_out; })];
  float s = 0.f;
#pragma unroll 8
  for (int k = 0; k < splits; k++) s += partial[(int64_t)k * b.total + i];
  const int64_t e = i - m.first_out;
  m.C[(e / r) * m.sm + (e % r) * m.sj] = m.alpha * s;
}

static int plain_grad_splits(int n) { return (int)std::min<int64_t>(32, cdiv(std::max(n, 1), 1024)); }
size_t plain_grad_partial_floats(int n, int64_t cols, int r) { return n > 1024 ? (size_t)plain_grad_splits(n) * cols * r : 0; }

int launch_plain_grads(as_ctx* ctx, PlainGradBatch b, int n, int r, float* partial, size_t partial_floats, hipStream_t st) {
  if (n <= 0 || b.n <= 0 || r <= 0) return AS_OK;
  const int nj = (int)cdiv(r, PG_B);
  int64_t blocks = 0; b.total = 0;
  for (int i = 0; i < b.n; i++) {
    b.m[i].first_block = (int)blocks; b.m[i].first_out = b.total;
    blocks += cdiv(b.m[i].M, PG_B) * nj; b.total += (int64_t)b.m[i].M * r;
  }
  const int splits = plain_grad_splits(n);
  if (splits > 1 && (size_t)splits * b.total > partial_floats) return as_fail(ctx, AS_ERR_WORKSPACE, "adapter gradients: partial buffer too small");
  prof_begin(ctx, st, AS_K_LORA_GRAD, 2.0 * n * (double)b.total);
  plain_grad_kernel<<<dim3((unsigned)blocks, splits), PG_WAVES * 64, 0, st>>>(b, n, r, splits, partial);
  AS_LAUNCH_CHECK(ctx);
  if (splits > 1) plain_grad_sum_kernel<<<(unsigned)cdiv(b.total, 256), 256, 0, st>>>(b, r, splits, partial);
  prof_end(ctx, st);
  AS_LAUNCH_CHECK(ctx);
  return AS_OK;
}
