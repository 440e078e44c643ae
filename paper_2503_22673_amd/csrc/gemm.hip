// C[M,N] = alpha * sum_s A_s[M,K_s] * B_s[N,K_s]^T (+ R): the projection GEMMs
// of the fine-tuning step.  The second K segment carries the low-rank LoRA
// product (x A^T)(s B)^T, so the adapter costs one extra pass over r columns
// inside the same accumulators instead of a second GEMM and an add.
//
// Kernels:
//  * gemm_f32_kernel        -- float operands on the matrix cores, 16x16 and 32x32 results per workgroup: the fp32 tier's small products (f32_pick).
//  * gemm_fma_kernel        -- any type, any shape; fp32 FMAs: the fp32 tier's large products, bf16 rows that are not 16-byte aligned, variant 1.
//  * gemm_mfma_rd_kernel    -- bf16, hand-scheduled 256x256 tiles, persistent: the large products; also with B, or A and B, given by rows of K.
//  * gemm_mfma_ring_kernel  -- bf16, 128x128 and 64x64 tiles in a ring of LDS stages: few rows or narrow outputs.
//  * gemm_mfma_dlds_kernel, gemm_mfma_kernel -- bf16: K that is no multiple of 64, rows counted on the device that the
//    hand-scheduled kernel does not take, rows that are not 16-byte aligned.
// In all of them workgroup ids are first de-interleaved over the 8 XCDs (ids are dealt round-robin to XCDs, each with a
// private L2) and then walked in groups of row tiles, so that the tiles resident on one XCD share A and B panels.
#include "common.h"
#include <cmath>
#include <type_traits>

// ------------------------------------------------------------------ helpers
struct KRange { int beg, end; };   // k-tile range of one segment for this split
__device__ __forceinline__ KRange split_range(int K, int BK, int splitk, int z) {
  int tiles = (K + BK - 1) / BK;
  int per = (tiles + splitk - 1) / splitk;
  KRange r; r.beg = min(tiles, z * per); r.end = min(tiles, r.beg + per);
  return r;
}

// operands and result of product b of a launch of several (selects: indexing the argument would copy it to scratch memory)
__device__ __forceinline__ GemmSeg batch_seg(const GemmParams& p, int b) {
  GemmSeg s = p.seg[0];
  if (p.nbat > 0) {
    s.A = b == 0 ? p.bt_A[0] : b == 1 ? p.bt_A[1] : p.bt_A[2]; s.B = b == 0 ? p.bt_B[0] : b == 1 ? p.bt_B[1] : p.bt_B[2];
    s.K = b == 0 ? p.bt_K[0] : b == 1 ? p.bt_K[1] : p.bt_K[2]; s.ldb = s.K;
  }
  return s;
}
__device__ __forceinline__ void* batch_c(const GemmParams& p, int b) { return p.nbat <= 0 ? p.C : b == 0 ? p.bt_C[0] : b == 1 ? p.bt_C[1] : p.bt_C[2]; }

template <typename T>
__device__ __forceinline__ void store_out(const GemmParams& p, int z, int row, int col, float v, int rb, void* C) {
  if (p.splitk > 1) { p.partial[((int64_t)z * p.M + row) * p.N + col] = v; return; }
  v *= p.alpha;
  row += rb;
  if (p.R) v += to_f<T>(((const T*)p.R)[(int64_t)row * p.ldr + col]);
  if (p.c_f32) {
    float* c = (float*)C + (int64_t)row * p.ldc + col;
    *c = p.accumulate ? *c + v : v;
  } else {
    ((T*)C)[(int64_t)row * p.ldc + col] = from_f<T>(v);
  }
}

// ------------------------------------------------------------- plain kernel
// float FMAs, every product of an output in ascending order of k.  Tiles of BT x BT with 16 x 16 threads, rows in LDS with k
// contiguous, so that a thread reads four k of a row at a time; the next K step's elements are on their way from memory
// while this one is multiplied.  64-wide steps and 32 x 32 tiles while those do not fill the chip, 64 x 64 tiles beyond.
template <typename T, int BT, int BK>
__global__ __launch_bounds__(256) void gemm_fma_kernel(GemmParams p, int m_off) {
  constexpr int TT = BT / 16, LS = BK + 4, PER = BT * BK / 4 / 256;      // outputs per thread and side; groups of four elements a thread loads
  static_assert(BT * BK / 4 % 256 == 0 && BK % 4 == 0, "whole groups per thread");
  __shared__ __align__(16) float As[BT][LS];
  __shared__ __align__(16) float Bs[BT][LS];
  int rb, mmax;
  const int M = gemm_rows(p, m_off, rb, mmax);
  const int row0 = blockIdx.y * BT, col0 = blockIdx.x * BT, z = blockIdx.z;
  if (row0 >= M) return;
  const int tid = threadIdx.x, tx = tid % 16, ty = tid / 16;
  float acc[TT][TT] = {};
  f32x4 ra[PER], rbv[PER];
  for (int s = 0; s < p.nseg; s++) {
    const T* A = (const T*)p.seg[s].A; const T* B = (const T*)p.seg[s].B;
    const int64_t lda = p.seg[s].lda, ldb = p.seg[s].ldb; const int K = p.seg[s].K;
    if (p.ncg > 0) {                                     // which weight matrix this column tile belongs to (column groups are whole tiles wide)
      int g = 0;
      while (g + 1 < p.ncg && col0 >= p.cg_end[g]) g++;
      B = (const T*)(s ? p.cg_B2[g] : p.cg_B1[g]) - (g ? (int64_t)p.cg_end[g - 1] * ldb : 0);
      if (s) A += p.cg_a2[g];
    }
    const bool va = sizeof(T) == 4 && lda % 4 == 0 && (uintptr_t)A % 16 == 0, vb = sizeof(T) == 4 && ldb % 4 == 0 && (uintptr_t)B % 16 == 0;
    const KRange kr = split_range(K, BK, p.splitk, z);
    auto four = [&](const T* row, bool row_in, int k, bool vec) {
      f32x4 v = {0.f, 0.f, 0.f, 0.f};
      if (!row_in || k >= K) return v;
      if (vec && k + 4 <= K) return *reinterpret_cast<const f32x4*>((const float*)row + k);
#pragma unroll
      for (int q = 0; q < 4; q++) if (k + q < K) v[q] = to_f<T>(row[k + q]);
      return v;
    };
    auto fetch = [&](int kt) {
#pragma unroll
      for (int i = 0; i < PER; i++) {
        const int g = tid + i * 256, r = g / (BK / 4), k = kt * BK + (g % (BK / 4)) * 4;
        ra[i] = four(A + (int64_t)(rb + row0 + r) * lda, row0 + r < M, k, va);
        rbv[i] = four(B + (int64_t)(col0 + r) * ldb, col0 + r < p.N, k, vb);
      }
    };
    if (kr.beg < kr.end) fetch(kr.beg);
    for (int kt = kr.beg; kt < kr.end; kt++) {
      __syncthreads();                                   // the step before has been read
#pragma unroll
      for (int i = 0; i < PER; i++) {
        const int g = tid + i * 256, r = g / (BK / 4), k = (g % (BK / 4)) * 4;
        *reinterpret_cast<f32x4*>(&As[r][k]) = ra[i]; *reinterpret_cast<f32x4*>(&Bs[r][k]) = rbv[i];
      }
      __syncthreads();
      if (kt + 1 < kr.end) fetch(kt + 1);
#pragma unroll 4
      for (int k = 0; k < BK; k += 4) {
        f32x4 a[TT], b[TT];
#pragma unroll
        for (int i = 0; i < TT; i++) { a[i] = *reinterpret_cast<const f32x4*>(&As[ty + 16 * i][k]); b[i] = *reinterpret_cast<const f32x4*>(&Bs[tx + 16 * i][k]); }
#pragma unroll
        for (int q = 0; q < 4; q++)
#pragma unroll
          for (int i = 0; i < TT; i++)
#pragma unroll
            for (int j = 0; j < TT; j++) acc[i][j] = fmaf(a[i][q], b[j][q], acc[i][j]);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < TT; i++)
#pragma unroll
    for (int j = 0; j < TT; j++) {
      const int r = row0 + ty + 16 * i, c = col0 + tx + 16 * j;
      if (r < M && c < p.N) store_out<T>(p, z, r, c, acc[i][j], rb, p.C);
    }
}

// ------------------------------------------------------------- small float products
// The fp32 tier's products on the matrix cores (v_mfma_f32_16x16x4f32: float products and sums, as FMAs), for models small enough
// that a product is one chain load -> multiply -> store and little else.  So: a workgroup owns 16 T x 16 T results, its NW waves take
// every NW-th 16-wide chunk of the contraction each, operands come from memory into the fragments without LDS (a lane loads four
// consecutive k of its row, 16 bytes; the four k of one matrix instruction are then 4 apart, in both operands alike), the next four
// chunks' loads are in flight behind the products of these, and one sum over the waves ends it.  Four waves up to 16
// chunks, eight up to 32, else sixteen (T = 1): up to 64 chunks every load of the product is then under way at once.  T = 2, beyond two to four
// 16 x 16 tiles per CU, reads half the operands per product; from two 64 x 64 tiles per CU on gemm_fma_kernel is ahead, which reads each once per tile (f32_pick).
// NN: B is [K, N], rows of up to three matrices below one another (p.nn): the layout of a weight matrix in the product with its output
// gradient, so that no matrix is transposed first.  A lane then loads its column of four rows, 4 bytes each.
// 2-layer model of width 128, 478 tokens, a product: 9.4 us with 32x32 tiles through LDS and FMAs, 5.6 so (K 688 and 1024: 20 and 28, now 8).
template <int T, bool NN, int NW>
__global__ __launch_bounds__(64 * NW) void gemm_f32_kernel(GemmParams p, int m_off) {
  constexpr int U = 4;                                     // chunks in flight
  __shared__ __align__(16) f32x4 red[NW][T * T][64];
  int rb, mmax;
  const int M = gemm_rows(p, m_off, rb, mmax);
  const int row0 = blockIdx.y * (16 * T), col0 = blockIdx.x * (16 * T), z = p.nbat > 0 ? 0 : blockIdx.z;
  if (row0 >= M) return;
  const GemmSeg s0 = batch_seg(p, blockIdx.z);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l15 = lane & 15, q = lane >> 4;
  // which weight matrix this lane's columns belong to (groups that end inside a tile: one segment only, so that A is the same for all)
  const float* bp[2][T]; int64_t a2 = 0;
#pragma unroll
  for (int t = 0; t < T; t++) {
    const int n = min(col0 + 16 * t + l15, p.N - 1);
    int g = 0;
    if (!NN && p.ncg > 0) while (g + 1 < p.ncg && n >= p.cg_end[g]) g++;
    const int nb = n - (g ? p.cg_end[g - 1] : 0);
#pragma unroll
    for (int s = 0; s < 2; s++) {
      const float* B = (const float*)(p.ncg > 0 ? (s ? p.cg_B2[g] : p.cg_B1[g]) : (s ? p.seg[1].B : s0.B));
      bp[s][t] = NN ? B + n : B + (int64_t)nb * (s ? p.seg[1].ldb : s0.ldb);
    }
    if (p.ncg > 0 && p.nseg > 1) a2 = p.cg_a2[g];
  }
  const float* ap[2][T];
#pragma unroll
  for (int t = 0; t < T; t++) {
    const int64_t r = rb + min(row0 + 16 * t + l15, max(M, 1) - 1);
    ap[0][t] = (const float*)s0.A + r * s0.lda; ap[1][t] = (const float*)p.seg[1].A + r * p.seg[1].lda + a2;
  }
  const int K0 = s0.K, K1 = p.nseg > 1 ? p.seg[1].K : 0;
  bool va[2], vb[2];                                       // rows in whole 16-byte pieces
#pragma unroll
  for (int s = 0; s < 2; s++) {
    const int K = s ? K1 : K0;
    va[s] = K % 4 == 0 && (s ? p.seg[1].lda : s0.lda) % 4 == 0 && (uintptr_t)ap[s][0] % 16 == 0;
    vb[s] = K % 4 == 0 && (s ? p.seg[1].ldb : s0.ldb) % 4 == 0 && (uintptr_t)bp[s][0] % 16 == 0 && (p.ncg == 0 || (((uintptr_t)(s ? p.cg_B2[0] : p.cg_B1[0]) | (uintptr_t)(s ? p.cg_B2[p.ncg - 1] : p.cg_B1[p.ncg - 1]) | (uintptr_t)(s ? p.cg_B2[p.ncg / 2] : p.cg_B1[p.ncg / 2])) % 16 == 0));
  }
  const int n0 = (K0 + 15) / 16, nall = n0 + (K1 + 15) / 16;
  const int c_lo = (int)((int64_t)nall * z / p.splitk), c_hi = (int)((int64_t)nall * (z + 1) / p.splitk);
  auto four = [&](const float* row, int k, int K, bool vec) {
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    if (k >= K) return v;
    if (vec) return *reinterpret_cast<const f32x4*>(row + k);
#pragma unroll
    for (int e = 0; e < 4; e++) if (k + e < K) v[e] = row[k + e];
    return v;
  };
  auto fetch = [&](int c, f32x4 (&a)[T], f32x4 (&b)[T]) {
    const int s = c < n0 ? 0 : 1, k = (s ? c - n0 : c) * 16 + 4 * q, K = c >= c_hi ? 0 : s ? K1 : K0;       // past the end: zeros
#pragma unroll
    for (int t = 0; t < T; t++) {
      a[t] = four(s ? ap[1][t] : ap[0][t], k, K, s ? va[1] : va[0]);
      if (!NN) { b[t] = four(s ? bp[1][t] : bp[0][t], k, K, s ? vb[1] : vb[0]); continue; }
#pragma unroll
      for (int e = 0; e < 4; e++) {
        const float* col = s ? bp[1][t] : bp[0][t];
        int64_t kk = k + e;
        if (!s && p.nn > 1) {
          const int n = min(col0 + 16 * t + l15, p.N - 1);
          if (p.nn > 2 && kk >= p.nb_row[1]) { col = (const float*)p.nb[1] + n; kk -= p.nb_row[1]; }
          else if (kk >= p.nb_row[0]) { col = (const float*)p.nb[0] + n; kk -= p.nb_row[0]; }
        }
        b[t][e] = k + e < K ? col[kk * s0.ldb] : 0.f;
      }
    }
  };
  f32x4 acc[T][T];
#pragma unroll
  for (int i = 0; i < T; i++)
#pragma unroll
    for (int j = 0; j < T; j++) acc[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
  f32x4 a[U][T], b[U][T];
  int c = c_lo + wave;
#pragma unroll
  for (int u = 0; u < U; u++) fetch(c + NW * u, a[u], b[u]);
  while (c < c_hi) {
    f32x4 na[U][T], nb[U][T];
    const bool more = c + NW * U < c_hi;
    if (more) {
#pragma unroll
      for (int u = 0; u < U; u++) fetch(c + NW * (U + u), na[u], nb[u]);
    }
#pragma unroll
    for (int u = 0; u < U; u++)
      if (c + NW * u < c_hi) {
#pragma unroll
        for (int e = 0; e < 4; e++)
#pragma unroll
          for (int i = 0; i < T; i++)
#pragma unroll
            for (int j = 0; j < T; j++) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(b[u][j][e], a[u][i][e], acc[i][j], 0, 0, 0);   // transposed: a lane owns a row
      }
    if (more) {
#pragma unroll
      for (int u = 0; u < U; u++)
#pragma unroll
        for (int t = 0; t < T; t++) { a[u][t] = na[u][t]; b[u][t] = nb[u][t]; }
    }
    c += NW * U;
  }
#pragma unroll
  for (int i = 0; i < T; i++)
#pragma unroll
    for (int j = 0; j < T; j++) red[wave][i * T + j][lane] = acc[i][j];
  __syncthreads();
  if (wave >= T * T) return;
  const int i = wave / T, j = wave % T, r = row0 + 16 * i + l15, n = col0 + 16 * j + 4 * q;
  f32x4 v = red[0][wave][lane];
#pragma unroll
  for (int w = 1; w < NW; w++) v += red[w][wave][lane];
  if (r >= M) return;
#pragma unroll
  for (int e = 0; e < 4; e++) if (n + e < p.N) store_out<float>(p, z, r, n + e, v[e], rb, batch_c(p, blockIdx.z));
}

// -------------------------------------------------------------- MFMA kernel
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;

// Epilogue shared by the MFMA kernels.  Lane l holds column l%32 and rows 8*(e/4) + 4*(l/32) + e%4 of
// each 32x32 block.  The output kind is uniform for the launch, so it is tested once, outside the
// element loops; `full` tiles skip the bounds tests.
template <int TM, int TN>
__device__ __forceinline__ void gemm_epilogue(const GemmParams& p, f32x16 (&acc)[TM][TN], int M, int z, int row0, int col0,
                                              int rb0, int cb0, bool full, int rb) {
  auto each = [&](auto f) {
#pragma unroll
    for (int i = 0; i < TM; i++)
#pragma unroll
      for (int j = 0; j < TN; j++) {
        const int c = cb0 + j * 32;
#pragma unroll
        for (int e = 0; e < 16; e++) {
          const int r = rb0 + i * 32 + 8 * (e >> 2) + (e & 3);
          if (full || (r < M && c < p.N)) f(r + rb, c, acc[i][j][e]);
        }
      }
  };
  if (p.splitk > 1) {
    float* part = p.partial + (int64_t)z * p.M * p.N;
    each([&](int r, int c, float v) { part[(int64_t)(r - rb) * p.N + c] = v; });
  } else if (p.c_f32) {
    float* C = (float*)p.C; const float alpha = p.alpha; const bf16_t* R = (const bf16_t*)p.R;
    if (p.accumulate || R)
      each([&](int r, int c, float v) {
        float* q = C + (int64_t)r * p.ldc + c;
        float x = alpha * v + (R ? (float)R[(int64_t)r * p.ldr + c] : 0.f);
        *q = p.accumulate ? *q + x : x;
      });
    else each([&](int r, int c, float v) { C[(int64_t)r * p.ldc + c] = alpha * v; });
  } else if (p.R) {
    bf16_t* C = (bf16_t*)p.C; const bf16_t* R = (const bf16_t*)p.R; const float alpha = p.alpha;
    each([&](int r, int c, float v) { C[(int64_t)r * p.ldc + c] = (bf16_t)(alpha * v + (float)R[(int64_t)r * p.ldr + c]); });
  } else {
    bf16_t* C = (bf16_t*)p.C; const float alpha = p.alpha;
    each([&](int r, int c, float v) { C[(int64_t)r * p.ldc + c] = (bf16_t)(alpha * v); });
  }
}

// EDGE = false: every K segment is a multiple of 64, so tile loads need no k guard.
template <int BM, int BN, int WM, int WN, bool EDGE>
__global__ __launch_bounds__(WM * WN * 64) void gemm_mfma_kernel(GemmParams p, int m_off, int tiles_m, int tiles_n) {
  constexpr int BK = 64, LS = BK + 8, NT = WM * WN * 64;
  constexpr int TM = BM / WM / 32, TN = BN / WN / 32;
  constexpr int CA = BM * 8 / NT, CB = BN * 8 / NT;      // 16-byte chunks per thread and tile
  static_assert(CA >= 1 && CB >= 1, "tile too small for the thread count");
  extern __shared__ __align__(16) unsigned char smem[];
  bf16_t* sA = (bf16_t*)smem;                            // [2][BM][LS]
  bf16_t* sB = sA + 2 * BM * LS;                         // [2][BN][LS]

  int rb, mmax;
  const int M = gemm_rows(p, m_off, rb, mmax);
  // XCD de-interleave, then grouped walk over the tile grid (over the live row tiles only when
  // the row count is a device-side value)
  if (p.m_dev || p.grp_off) tiles_m = min(tiles_m, (max(M, 0) + BM - 1) / BM);
  int nblk = tiles_m * tiles_n, pid = blockIdx.x, z = blockIdx.y;
  if (pid >= nblk) return;
  int q8 = nblk / 8, rem = nblk % 8, xcd = pid % 8, loc = pid / 8;
  int logical = xcd * q8 + min(xcd, rem) + loc;
  constexpr int GROUP = 8;
  int in_group = GROUP * tiles_n, grp = logical / in_group, first_m = grp * GROUP;
  int gsize = min(tiles_m - first_m, GROUP);
  int tile_m = first_m + (logical % in_group) % gsize, tile_n = (logical % in_group) / gsize;
  const int row0 = tile_m * BM, col0 = tile_n * BN;
  if (row0 >= M) return;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WN, wn = wave % WN;

  KRange kr0 = split_range(p.seg[0].K, BK, p.splitk, z);
  KRange kr1 = {0, 0};
  if (p.nseg > 1) kr1 = split_range(p.seg[1].K, BK, p.splitk, z);
  const int nt0 = kr0.end - kr0.beg, nt = nt0 + (kr1.end - kr1.beg);

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; i++)
#pragma unroll
    for (int j = 0; j < TN; j++)
#pragma unroll
      for (int e = 0; e < 16; e++) acc[i][j][e] = 0.f;

  u32x4 ra[CA], rbv[CB];
  // per-thread row offsets inside the tile are fixed; only the k offset moves
  int64_t offA[CA], offB[CB];
  {
    const int mclamp = mmax, nclamp = p.N - 1;
#pragma unroll
    for (int i = 0; i < CA; i++) { int c = tid + i * NT; offA[i] = (int64_t)(rb + min(row0 + (c >> 3), mclamp)); }
#pragma unroll
    for (int i = 0; i < CB; i++) { int c = tid + i * NT; offB[i] = (int64_t)min(col0 + (c >> 3), nclamp); }
  }
  const int kc = (tid & 7) * 8;                          // NT is a multiple of 8: same k chunk for every i

  auto fetch = [&](int it) {
    const bool first = it < nt0;
    const bf16_t* A = (const bf16_t*)(first ? p.seg[0].A : p.seg[1].A);
    const bf16_t* B = (const bf16_t*)(first ? p.seg[0].B : p.seg[1].B);
    const int64_t lda = first ? p.seg[0].lda : p.seg[1].lda, ldb = first ? p.seg[0].ldb : p.seg[1].ldb;
    const int K = first ? p.seg[0].K : p.seg[1].K;
    const int k = (first ? kr0.beg + it : kr1.beg + it - nt0) * BK + kc;
    const bool in = !EDGE || k < K;
    const int ks = in ? k : 0;                           // a valid address either way
#pragma unroll
    for (int i = 0; i < CA; i++) {
      u32x4 v = *reinterpret_cast<const u32x4*>(A + offA[i] * lda + ks);
      ra[i] = in ? v : (u32x4){0u, 0u, 0u, 0u};
    }
#pragma unroll
    for (int i = 0; i < CB; i++) {
      u32x4 v = *reinterpret_cast<const u32x4*>(B + offB[i] * ldb + ks);
      rbv[i] = in ? v : (u32x4){0u, 0u, 0u, 0u};
    }
  };
  auto stash = [&](int buf) {
    bf16_t* a = sA + buf * BM * LS; bf16_t* b = sB + buf * BN * LS;
#pragma unroll
    for (int i = 0; i < CA; i++) { int c = tid + i * NT; *reinterpret_cast<u32x4*>(a + (c >> 3) * LS + kc) = ra[i]; }
#pragma unroll
    for (int i = 0; i < CB; i++) { int c = tid + i * NT; *reinterpret_cast<u32x4*>(b + (c >> 3) * LS + kc) = rbv[i]; }
  };

  if (nt > 0) { fetch(0); stash(0); }
  __syncthreads();
  for (int it = 0; it < nt; it++) {
    const int buf = it & 1;
    if (it + 1 < nt) fetch(it + 1);
    const bf16_t* a = sA + buf * BM * LS + (wm * TM * 32 + (lane & 31)) * LS + (lane >> 5) * 8;
    const bf16_t* b = sB + buf * BN * LS + (wn * TN * 32 + (lane & 31)) * LS + (lane >> 5) * 8;
#pragma unroll
    for (int ks = 0; ks < BK / 16; ks++) {
      bf16x8 af[TM], bfr[TN];
#pragma unroll
      for (int i = 0; i < TM; i++) af[i] = *reinterpret_cast<const bf16x8*>(a + i * 32 * LS + ks * 16);
#pragma unroll
      for (int j = 0; j < TN; j++) bfr[j] = *reinterpret_cast<const bf16x8*>(b + j * 32 * LS + ks * 16);
#pragma unroll
      for (int i = 0; i < TM; i++)
#pragma unroll
        for (int j = 0; j < TN; j++)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[i], bfr[j], acc[i][j], 0, 0, 0);
    }
    if (it + 1 < nt) stash(buf ^ 1);
    __syncthreads();
  }

  gemm_epilogue<TM, TN>(p, acc, M, z, row0, col0, row0 + wm * TM * 32 + 4 * (lane >> 5), col0 + wn * TN * 32 + (lane & 31),
                        (row0 + BM <= M) && (col0 + BN <= p.N), rb);
}

// Same tiling, but tiles travel global -> LDS directly (global_load_lds_dwordx4: a wavefront
// deposits 64 x 16 bytes contiguously, i.e. 8 rows of 8 chunks), so no VGPR staging and no LDS
// stores.  The destination cannot be padded, so chunks are XOR-swizzled instead: LDS slot
// (row, c) holds the row's chunk c ^ ((row >> 1) & 7); each lane picks the matching global chunk.  Fragment
// reads of 8 consecutive rows then touch 8 different 16-byte columns: no bank conflicts.
// Fragments are double-buffered in registers.  The barrier of a K step sits before the last of its four
// 16-wide slices: by then every fragment of the current tile is in registers, so the next tile's loads can
// be issued into the buffer just released and the first fragments of the next tile are read while the last
// slice's MFMAs run, instead of right after a barrier with nothing to overlap them.
// Needs every K segment to be a multiple of 64.
__device__ __forceinline__ int swz(int r) { return (r >> 1) & 7; }

template <int BM, int BN, int WM, int WN>
__global__ __launch_bounds__(WM * WN * 64) void gemm_mfma_dlds_kernel(GemmParams p, int m_off, int tiles_m, int tiles_n) {
  constexpr int BK = 64, NW = WM * WN;
  constexpr int TM = BM / WM / 32, TN = BN / WN / 32;
  constexpr int LA = BM / 8 / NW, LB = BN / 8 / NW;      // 1 KB wave-loads per wave and tile
  static_assert(LA >= 1 && LB >= 1, "tile too small for the wave count");
  static_assert(BK / 16 == 4, "the loop is written for four K slices");
  extern __shared__ __align__(16) unsigned char smem[];
  bf16_t* sA = (bf16_t*)smem;                            // [2][BM][64]
  bf16_t* sB = sA + 2 * BM * BK;                         // [2][BN][64]

  int rb, mmax;
  const int M = gemm_rows(p, m_off, rb, mmax);
  // the row count may live on the device (target rows, rows of one expert): map the workgroups
  // over the live row tiles only, so that they still spread over all XCDs
  if (p.m_dev || p.grp_off) tiles_m = min(tiles_m, (max(M, 0) + BM - 1) / BM);
  int nblk = tiles_m * tiles_n, pid = blockIdx.x, z = blockIdx.y;
  if (pid >= nblk) return;
  int q8 = nblk / 8, rem = nblk % 8, xcd = pid % 8, loc = pid / 8;
  int logical = xcd * q8 + min(xcd, rem) + loc;
  constexpr int GROUP = 8;
  int in_group = GROUP * tiles_n, grp = logical / in_group, first_m = grp * GROUP;
  int gsize = min(tiles_m - first_m, GROUP);
  int tile_m = first_m + (logical % in_group) % gsize, tile_n = (logical % in_group) / gsize;
  const int row0 = tile_m * BM, col0 = tile_n * BN;
  if (row0 >= M) return;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WN, wn = wave % WN;
  KRange kr0 = split_range(p.seg[0].K, BK, p.splitk, z);
  KRange kr1 = {0, 0};
  if (p.nseg > 1) kr1 = split_range(p.seg[1].K, BK, p.splitk, z);
  const int nt0 = kr0.end - kr0.beg, nt = nt0 + (kr1.end - kr1.beg);

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; i++)
#pragma unroll
    for (int j = 0; j < TN; j++)
#pragma unroll
      for (int e = 0; e < 16; e++) acc[i][j][e] = 0.f;

  // loader: wave-load i of this wave covers tile rows (wave*L + i)*8 .. +7; lane l sits at row l/8,
  // LDS chunk l%8, and fetches global chunk (l%8) ^ swz(row)
  const int lrow = lane >> 3;
  int rowA[LA], rowB[LB];
  {
    const int mclamp = mmax, nclamp = p.N - 1;
#pragma unroll
    for (int i = 0; i < LA; i++) rowA[i] = rb + min(row0 + (wave * LA + i) * 8 + lrow, mclamp);
#pragma unroll
    for (int i = 0; i < LB; i++) rowB[i] = min(col0 + (wave * LB + i) * 8 + lrow, nclamp);
  }
  // per-lane row pointers of the first K segment are kept in registers (no 64-bit multiplies per step)
  const bf16_t* pA[LA]; const bf16_t* pB[LB];
#pragma unroll
  for (int i = 0; i < LA; i++) pA[i] = (const bf16_t*)p.seg[0].A + (int64_t)rowA[i] * p.seg[0].lda + (((lane & 7) ^ swz((wave * LA + i) * 8 + lrow)) * 8);
#pragma unroll
  for (int i = 0; i < LB; i++) pB[i] = (const bf16_t*)p.seg[0].B + (int64_t)rowB[i] * p.seg[0].ldb + (((lane & 7) ^ swz((wave * LB + i) * 8 + lrow)) * 8);
  auto fetch = [&](int it, int buf) {
    const bool first = it < nt0;
    bf16_t* a = sA + buf * BM * BK + wave * LA * 8 * BK;
    bf16_t* b = sB + buf * BN * BK + wave * LB * 8 * BK;
    if (first) {
      const int k1 = (kr0.beg + it) * BK;
#pragma unroll
      for (int i = 0; i < LA; i++)
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(pA[i] + k1),
                                         (__attribute__((address_space(3))) void*)(a + i * 8 * BK), 16, 0, 0);
#pragma unroll
      for (int i = 0; i < LB; i++)
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(pB[i] + k1),
                                         (__attribute__((address_space(3))) void*)(b + i * 8 * BK), 16, 0, 0);
      return;
    }
    const bf16_t* A = (const bf16_t*)p.seg[1].A; const bf16_t* B = (const bf16_t*)p.seg[1].B;
    const int64_t lda = p.seg[1].lda, ldb = p.seg[1].ldb;
    const int k = (kr1.beg + it - nt0) * BK;
#pragma unroll
    for (int i = 0; i < LA; i++)
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(A + (int64_t)rowA[i] * lda + k + (((lane & 7) ^ swz((wave * LA + i) * 8 + lrow)) * 8)),
                                       (__attribute__((address_space(3))) void*)(a + i * 8 * BK), 16, 0, 0);
#pragma unroll
    for (int i = 0; i < LB; i++)
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(B + (int64_t)rowB[i] * ldb + k + (((lane & 7) ^ swz((wave * LB + i) * 8 + lrow)) * 8)),
                                       (__attribute__((address_space(3))) void*)(b + i * 8 * BK), 16, 0, 0);
  };

  // reader: row = base + l%32, logical chunk 2*ks + l/32 lives at chunk (2*ks + l/32) ^ swz(row)
  const int x7 = swz(lane & 31), hh = lane >> 5;
  int coff[BK / 16];
#pragma unroll
  for (int ks = 0; ks < BK / 16; ks++) coff[ks] = ((2 * ks + hh) ^ x7) * 8;

  if (nt > 0) fetch(0, 0);
  __builtin_amdgcn_s_waitcnt(0x0f70);                    // vmcnt(0): the first tile has landed
  __syncthreads();
  bf16x8 af[2][TM], bfr[2][TN];
  auto rd = [&](int buf, int ks, int slot) {
    const bf16_t* a = sA + buf * BM * BK + (wm * TM * 32 + (lane & 31)) * BK;
    const bf16_t* b = sB + buf * BN * BK + (wn * TN * 32 + (lane & 31)) * BK;
#pragma unroll
    for (int i = 0; i < TM; i++) af[slot][i] = *reinterpret_cast<const bf16x8*>(a + i * 32 * BK + coff[ks]);
#pragma unroll
    for (int j = 0; j < TN; j++) bfr[slot][j] = *reinterpret_cast<const bf16x8*>(b + j * 32 * BK + coff[ks]);
  };
  auto mm = [&](int slot) {
#pragma unroll
    for (int i = 0; i < TM; i++)
#pragma unroll
      for (int j = 0; j < TN; j++)
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[slot][i], bfr[slot][j], acc[i][j], 0, 0, 0);
  };
  auto weave = [&]() {                                   // one LDS read between MFMAs, then the rest of the MFMAs
#pragma unroll
    for (int r = 0; r < TM + TN; r++) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, TM * TN - (TM + TN), 0);
  };
  if (nt > 1) fetch(1, 1);
  if (nt > 0) rd(0, 0, 0);
  for (int it = 0; it < nt; it++) {
    const int buf = it & 1;
    rd(buf, 1, 1); mm(0); weave();
    rd(buf, 2, 0); mm(1); weave();
    rd(buf, 3, 1); mm(0); weave();
    __builtin_amdgcn_s_waitcnt(0x0070);                  // vmcnt(0) lgkmcnt(0)
    __syncthreads();                                     // tile it is in registers everywhere, tile it+1 has landed
    // straight-line tail (the last two steps re-request the final tile into a buffer nobody reads
    // again, and read fragments nobody uses), so that loads, LDS reads and MFMAs can interleave
    fetch(min(it + 2, nt - 1), buf);
    rd(buf ^ 1, 0, 0);
    mm(1);
#pragma unroll
    for (int r = 0; r < TM + TN; r++) {
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x020, LA + LB, 0);
    __builtin_amdgcn_sched_group_barrier(0x008, TM * TN - (TM + TN), 0);
  }
  __builtin_amdgcn_s_waitcnt(0x0f70);                    // the re-requested tile must land before the workgroup's LDS is released
  gemm_epilogue<TM, TN>(p, acc, M, z, row0, col0, row0 + wm * TM * 32 + 4 * (lane >> 5), col0 + wn * TN * 32 + (lane & 31),
                        (row0 + BM <= M) && (col0 + BN <= p.N), rb);
}

// Ring of LDS stages, for products with too few 256 x 256 tiles for the chip and for narrow outputs.  Tiles of BM x BN, four
// waves of (BM / 2) x (BN / 2), NST stages of one 64-wide K step each, filled straight from global memory (swizzled chunks, as
// above); a step waits for its own stage only (`vmcnt` of the younger ones), passes one barrier and asks for the stage
// NST - 1 ahead.  What bounds it: a CU's path into LDS carries about 40 bytes per clock, 800 clocks (0.33 us) for the 32 KB of a
// 128 x 128 step against 512 of matrix work, so a CU runs two workgroups (64 KB of LDS each) whose waits and barriers fall
// at different times: 0.51 us per step and tile with two on a CU, 0.74 with one.  Three and four stages are level: 32 KB a step of every
// CU at once is 25 bytes per clock and CU, what the 256x256 kernel draws from the L2s too (64 KB in 2200 clocks).  64 x 64 tiles read twice the operand
// bytes per flop but give four times the workgroups: the adapters' 64-wide products, bound by reading A once, run
// at 4.6 TB/s (15,500 rows, K 14336: 97 us; 128 x 64 register-staged tiles: 240; at 59,000 rows, where those fill the chip
// too, the two are level).
// The contraction may be split over `splitk` workgroups (grid.y): float partials, added in order by a second launch.
// Results leave through LDS, 32 rows of a wave's block at a time, as whole 16-byte pieces; blocks are computed transposed, so
// that a lane owns four consecutive columns of a row.
// Needs: plain rows, K segments in 64-wide steps, 16-byte aligned rows of every operand (ring_ok).
template <int N> __device__ __forceinline__ void wait_vm() {
  // vmcnt(N) and lgkmcnt(0): bits 3:0 and 15:14 vmcnt, 6:4 expcnt (untouched), 11:8 lgkmcnt.  The barrier behind it lets other waves
  // overwrite the stage this wave has read, so its reads must have returned (their MFMAs have waited for them already)
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0070);
}
template <int L, int D> __device__ __forceinline__ void wait_stages(int younger) {   // all but the loads of the `younger` newest stages have landed
  if constexpr (D <= 0) wait_vm<0>();
  else { if (younger >= D) wait_vm<L * D>(); else wait_stages<L, D - 1>(younger); }
}

template <int BM, int BN, int NST>
__global__ __launch_bounds__(256) void gemm_mfma_ring_kernel(GemmParams p, int tiles_m, int tiles_n) {
  constexpr int BK = 64, WM = 2, WN = 2, NW = WM * WN, TM = BM / WM / 32, TN = BN / WN / 32;
  constexpr int LA = BM / 8 / NW, LB = BN / 8 / NW, L = LA + LB, ST_E = (BM + BN) * BK;
  extern __shared__ __align__(16) unsigned char smem[];
  bf16_t* sm = (bf16_t*)smem;
  const int nblk = tiles_m * tiles_n, pid = blockIdx.x, z = blockIdx.y;
  const int q8 = nblk / 8, rem = nblk % 8, xcd = pid % 8, loc = pid / 8;
  const int logical = xcd * q8 + min(xcd, rem) + loc;
  constexpr int GROUP = 8;
  const int in_group = GROUP * tiles_n, grp = logical / in_group, first_m = grp * GROUP;
  const int gsize = min(tiles_m - first_m, GROUP);
  const int row0 = (first_m + (logical % in_group) % gsize) * BM, col0 = ((logical % in_group) / gsize) * BN;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave / WN, wn = wave % WN;
  const int bt = blockIdx.z;
  const GemmSeg s0 = batch_seg(p, bt), s1 = p.seg[1];
  void* const Cp = batch_c(p, bt);
  float* part = p.partial + (int64_t)bt * p.splitk * p.M * p.N;
  // K steps of this split, over both segments one after the other
  const int n0 = s0.K / BK, ntot = n0 + (p.nseg > 1 ? s1.K / BK : 0);
  const int k_lo = (int)((int64_t)ntot * z / p.splitk), nt = (int)((int64_t)ntot * (z + 1) / p.splitk) - k_lo;
  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; i++)
#pragma unroll
    for (int j = 0; j < TN; j++)
#pragma unroll
      for (int e = 0; e < 16; e++) acc[i][j][e] = 0.f;
  const int lrow = lane >> 3;
  uint32_t offA[2][LA], offB[2][LB];                     // byte offsets of this lane's rows and chunk inside the panels
#pragma unroll
  for (int i = 0; i < LA; i++) {
    const int rt = (wave * LA + i) * 8 + lrow, r = min(row0 + rt, p.M - 1) - row0, ch = ((lane & 7) ^ swz(rt)) * 8;
    offA[0][i] = (uint32_t)((r * s0.lda + ch) * 2); offA[1][i] = (uint32_t)((r * s1.lda + ch) * 2);
  }
#pragma unroll
  for (int i = 0; i < LB; i++) {
    const int rt = (wave * LB + i) * 8 + lrow, r = min(col0 + rt, p.N - 1) - col0, ch = ((lane & 7) ^ swz(rt)) * 8;
    offB[0][i] = (uint32_t)((r * s0.ldb + ch) * 2); offB[1][i] = (uint32_t)((r * s1.ldb + ch) * 2);
  }
  // which weight matrix this column tile belongs to (column groups are whole tiles wide)
  const bf16_t* b0 = (const bf16_t*)s0.B; const bf16_t* b1 = (const bf16_t*)s1.B;
  int colg = col0, a2 = 0;
  if (p.ncg > 0) {
    int g = 0;
    while (g + 1 < p.ncg && col0 >= p.cg_end[g]) g++;
    colg = col0 - (g ? p.cg_end[g - 1] : 0);
    b0 = (const bf16_t*)p.cg_B1[g];
    if (p.nseg > 1) { b1 = (const bf16_t*)p.cg_B2[g]; a2 = p.cg_a2[g]; }
  }
  const char* A0 = (const char*)s0.A + (int64_t)row0 * s0.lda * 2; const char* B0 = (const char*)(b0 + (int64_t)colg * s0.ldb);
  const char* A1 = (const char*)((const bf16_t*)s1.A + a2 + (int64_t)row0 * s1.lda); const char* B1 = (const char*)(b1 + (int64_t)colg * s1.ldb);
  auto fetch = [&](int it, int slot) {
    const int ks = k_lo + it;
    const bool first = ks < n0;
    const char* a = first ? A0 + (int64_t)ks * (BK * 2) : A1 + (int64_t)(ks - n0) * (BK * 2);
    const char* b = first ? B0 + (int64_t)ks * (BK * 2) : B1 + (int64_t)(ks - n0) * (BK * 2);
    bf16_t* da = sm + slot * ST_E + wave * LA * 8 * BK; bf16_t* db = sm + slot * ST_E + BM * BK + wave * LB * 8 * BK;
#pragma unroll
    for (int i = 0; i < LA; i++)
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(a + (first ? offA[0][i] : offA[1][i])),
                                       (__attribute__((address_space(3))) void*)(da + i * 8 * BK), 16, 0, 0);
#pragma unroll
    for (int i = 0; i < LB; i++)
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(b + (first ? offB[0][i] : offB[1][i])),
                                       (__attribute__((address_space(3))) void*)(db + i * 8 * BK), 16, 0, 0);
  };
  const int x7 = swz(lane & 31), hh = lane >> 5, l31 = lane & 31;
  int coff[4];
#pragma unroll
  for (int ks = 0; ks < 4; ks++) coff[ks] = ((2 * ks + hh) ^ x7) * 8;
#pragma unroll
  for (int s = 0; s < NST - 1; s++) if (s < nt) fetch(s, s);
  int slot = 0;
  for (int it = 0; it < nt; it++) {
    wait_stages<L, NST - 2>(nt - 1 - it);
    __builtin_amdgcn_s_barrier();                        // stage `it` is in LDS for every wave, and every wave has read stage it - 1
    asm volatile("" ::: "memory");
    const int nslot = slot == 0 ? NST - 1 : slot - 1;
    if (it + NST - 1 < nt) fetch(it + NST - 1, nslot);
    const bf16_t* a = sm + slot * ST_E + (wm * TM * 32 + l31) * BK; const bf16_t* b = sm + slot * ST_E + BM * BK + (wn * TN * 32 + l31) * BK;
    // 128 x 128: all of the step's fragments are asked for before the first product, so that LDS latency is paid once and not once per
    // slice (with two workgroups on a CU 1 % on average, up to 16; 64 x 64 tiles lose 1.5 % by it)
    constexpr int AHEAD = TM * TN > 1 ? 4 : 1;             // slices read together
#pragma unroll
    for (int k0 = 0; k0 < 4; k0 += AHEAD) {
      bf16x8 af[AHEAD][TM], bf[AHEAD][TN];
#pragma unroll
      for (int ks = 0; ks < AHEAD; ks++) {
#pragma unroll
        for (int i = 0; i < TM; i++) af[ks][i] = *reinterpret_cast<const bf16x8*>(a + i * 32 * BK + coff[k0 + ks]);
#pragma unroll
        for (int j = 0; j < TN; j++) bf[ks][j] = *reinterpret_cast<const bf16x8*>(b + j * 32 * BK + coff[k0 + ks]);
      }
#pragma unroll
      for (int ks = 0; ks < AHEAD; ks++)
#pragma unroll
        for (int i = 0; i < TM; i++)
#pragma unroll
          for (int j = 0; j < TN; j++) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bf[ks][j], af[ks][i], acc[i][j], 0, 0, 0);   // transposed blocks
    }
    if constexpr (AHEAD > 1) {
      __builtin_amdgcn_sched_group_barrier(0x100, 4 * (TM + TN), 0);
      __builtin_amdgcn_sched_group_barrier(0x008, 4 * TM * TN, 0);
    }
    asm volatile("" ::: "memory");
    slot = slot == NST - 1 ? 0 : slot + 1;
  }
  // epilogue through LDS, 32 rows of the wave's block at a time; a lane owns row l31 and columns 32 j + 8 b4 + 4 hh ..+3
  wait_vm<0>();
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  constexpr int WC = TN * 32;                            // columns of the wave's block
  const int rw = row0 + wm * TM * 32, cw = col0 + wn * WC;
  if (p.splitk > 1 || p.c_f32) {
    constexpr int PITCH = WC + 4;                        // floats
    float* my = (float*)smem + wave * 32 * PITCH;
    static_assert(NW * 32 * PITCH * 4 <= NST * ST_E * 2, "epilogue fits the stages");
    constexpr int LPR = WC / 4, RPI = 64 / LPR;
    float* C = p.splitk > 1 ? part + (int64_t)z * p.M * p.N : (float*)Cp;
    const int64_t ldc = p.splitk > 1 ? p.N : p.ldc;
    const float alpha = p.splitk > 1 ? 1.f : p.alpha;
#pragma unroll
    for (int i = 0; i < TM; i++) {
#pragma unroll
      for (int j = 0; j < TN; j++)
#pragma unroll
        for (int b4 = 0; b4 < 4; b4++)
          *reinterpret_cast<f32x4*>(my + l31 * PITCH + 32 * j + 8 * b4 + 4 * hh) =
              (f32x4){alpha * acc[i][j][4 * b4], alpha * acc[i][j][4 * b4 + 1], alpha * acc[i][j][4 * b4 + 2], alpha * acc[i][j][4 * b4 + 3]};
      __builtin_amdgcn_s_waitcnt(0xc07f);
      asm volatile("" ::: "memory");
#pragma unroll
      for (int r = 0; r < 32; r += RPI) {
        const int rr = r + lane / LPR, cc = (lane % LPR) * 4, row = rw + i * 32 + rr, col = cw + cc;
        if (row < p.M && col < p.N) {
          f32x4 v = *reinterpret_cast<const f32x4*>(my + rr * PITCH + cc);
          float* q = C + (int64_t)row * ldc + col;
          if (p.splitk <= 1) {
            if (p.R) { const bf16x4 x = *reinterpret_cast<const bf16x4*>((const bf16_t*)p.R + (int64_t)row * p.ldr + col);
#pragma unroll
              for (int k = 0; k < 4; k++) v[k] += (float)x[k]; }
            if (p.accumulate) v += *reinterpret_cast<const f32x4*>(q);
          }
          *reinterpret_cast<f32x4*>(q) = v;
        }
      }
      asm volatile("" ::: "memory");
    }
  } else {
    constexpr int PITCH = WC + 8;                        // bf16
    float alpha = p.alpha;
    bf16_t* my = (bf16_t*)smem + wave * 32 * PITCH;
    constexpr int LPR = WC / 8, RPI = 64 / LPR;
#pragma unroll
    for (int i = 0; i < TM; i++) {
      if (p.R) {
#pragma unroll
        for (int r = 0; r < 32; r += RPI) {
          const int rr = r + lane / LPR, cc = (lane % LPR) * 8, row = rw + i * 32 + rr, col = cw + cc;
          if (row < p.M && col < p.N) *reinterpret_cast<u32x4*>(my + rr * PITCH + cc) = *reinterpret_cast<const u32x4*>((const bf16_t*)p.R + (int64_t)row * p.ldr + col);
        }
        __builtin_amdgcn_s_waitcnt(0xc07f);
        asm volatile("" ::: "memory");
      }
#pragma unroll
      for (int j = 0; j < TN; j++)
#pragma unroll
        for (int b4 = 0; b4 < 4; b4++) {
          bf16x4* q = reinterpret_cast<bf16x4*>(my + l31 * PITCH + 32 * j + 8 * b4 + 4 * hh);
          f32x4 v;
#pragma unroll
          for (int k = 0; k < 4; k++) v[k] = alpha * acc[i][j][4 * b4 + k];
          if (p.R) { const bf16x4 x = *q;
#pragma unroll
            for (int k = 0; k < 4; k++) v[k] += (float)x[k]; }
          bf16x4 w;
#pragma unroll
          for (int k = 0; k < 4; k++) w[k] = (bf16_t)v[k];
          *q = w;
        }
      __builtin_amdgcn_s_waitcnt(0xc07f);
      asm volatile("" ::: "memory");
#pragma unroll
      for (int r = 0; r < 32; r += RPI) {
        const int rr = r + lane / LPR, cc = (lane % LPR) * 8, row = rw + i * 32 + rr, col = cw + cc;
        if (row < p.M && col < p.N) *reinterpret_cast<u32x4*>((bf16_t*)Cp + (int64_t)row * p.ldc + col) = *reinterpret_cast<const u32x4*>(my + rr * PITCH + cc);
      }
      asm volatile("" ::: "memory");
    }
  }
}

// sum of the splits in order, then the epilogue
__global__ __launch_bounds__(256) void gemm_splitk_finish_kernel(GemmParams p) {
  const int64_t idx = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4, mn = (int64_t)p.M * p.N;
  if (idx >= mn) return;
  const int bt = blockIdx.y;
  const float* part = p.partial + (int64_t)bt * p.splitk * mn + idx;
  const int64_t row = idx / p.N; const int col = (int)(idx % p.N);
  f32x4 v = *reinterpret_cast<const f32x4*>(part);
  for (int s = 1; s < p.splitk; s++) v += *reinterpret_cast<const f32x4*>(part + (int64_t)s * mn);
#pragma unroll
  for (int k = 0; k < 4; k++) v[k] *= p.alpha;
  if (p.R) { const bf16x4 x = *reinterpret_cast<const bf16x4*>((const bf16_t*)p.R + row * p.ldr + col);
#pragma unroll
    for (int k = 0; k < 4; k++) v[k] += (float)x[k]; }
  if (p.c_f32) {
    f32x4* q = reinterpret_cast<f32x4*>((float*)p.C + row * p.ldc + col);
    if (p.accumulate) v += *q;
    *q = v;
  } else {
    bf16x4 w;
#pragma unroll
    for (int k = 0; k < 4; k++) w[k] = (bf16_t)v[k];
    *reinterpret_cast<bf16x4*>((bf16_t*)batch_c(p, bt) + row * p.ldc + col) = w;
  }
}

typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4_t;
// the matrix that a result row lies in, minus the rows above it (float results, whole tiles per group)
__device__ __forceinline__ void* row_group_base(const GemmParams& p, int row) {
  int g = 0;
  while (g < p.nrg && row >= p.rg_row[g]) g++;
  return g ? (float*)p.rg_C[g - 1] - (int64_t)p.rg_row[g - 1] * p.ldc : (float*)p.C;
}
// ------------------------------------------------------------- persistent 256 x 256 tiles
// The large products: N in whole 256-column tiles, at least 256 rows, K segments that are multiples of 64 (rd_ok); the launcher sends
// everything else to the other kernels.  Four waves of 128 x 128, one per SIMD, whose 256 accumulators live in the accumulation half of
// the register file.  With one wave per SIMD every wait in the instruction stream idles the matrix pipe, so the loop over a tile's
// contraction is written out instruction by instruction (gen_gemm_rd_loop.py).  What it is built on, each against a kernel with 32x32x16
// products, tiles staged through registers and one workgroup per tile:
// * Under the chip's power limit the clock follows the energy of an operation, and a 16x16x32 product costs less of it than a 32x32x16
//   one (register-resident loops on random operands: 2025 against 1788 TFLOP/s).  A slot of 16 clocks has no room for LDS stores
//   (staged through registers with 16x16x32 products: 2510 clocks a step instead of 2170 and 2 % in all), so tiles go straight to LDS,
//   through a ring of five 32 KB half stages that keeps the loads one to 1.7 steps ahead: 2190 clocks a step of 2048 of matrix work, at
//   1.65 to 1.75 GHz where the staged kernel held 1.5 to 1.57.
// * The workgroups are persistent, one per CU: the first two steps of the next tile are on their way while the last ones of a tile are
//   multiplied and while its result is written.  A tile costs its steps, an epilogue of 7,400 clocks and 2,100 between tiles; the staged
//   kernel lost 21,000 (epilogue 10,500, first loads, launch).  The epilogue takes 64 accumulators at a time: with all 256 in the
//   compiler's hands it spilled a hundred registers.
// * LAYOUT NN: B as [K, N] rows, the layout of a weight matrix in the product with its output gradient: no transposed copy first (16384
//   tokens on a dense 8B model spent 700 us of 33.1 ms in those copies, 8192 tokens on a sparse 8x7B one 1150 us of 15.0 ms; the
//   products take as long either way).  TN: A as [K, M] too, the gradient of a weight matrix, tokens contracted, from the output gradient
//   and the input as they are: a full step of one 1B layer at 16384 tokens, 4350 of them targets, 8.00 ms with token-major copies, 6.28 so.
// * The contraction of a tile may be shared by several workgroups, as parts with float sums (gemm_items.h: which tiles, where parts begin).
// TFLOP/s before and now, random operands, launches back to back: 16384 x 14336 x 4096 1333 and 1525, 16384 x 4096 x 14336 1365 and 1558,
// 32768 x 8192 x 2048 1234 and 1407, 32768 x 2048 x 8192 1346 and 1535.
#include "gemm_rd_loop.inc"
#include "gemm_rd_nn_loop.inc"
#include "gemm_rd_tn_loop.inc"
constexpr size_t kRdSmem = 5 * 32768;

// A wave's block leaves in four pieces of 32 rows, whose 64 accumulators are taken to vector registers first: t[j] is the 32 x 32 block of
// column j, its 16 x 16 block (a, b) elements 4 (2 a + b) .. + 3; a lane owns row 16 a + lane % 16 and the four columns from 16 b + 4 (lane / 16).
struct RdOut { int row0, col0, row_lo, row_hi; };          // the wave's block; with MASK only rows row_lo .. row_hi - 1 are read and written
__device__ __forceinline__ f32x4 quad(const f32x16& v, int a, int b, float alpha) {
  f32x4 r;
#pragma unroll
  for (int k = 0; k < 4; k++) r[k] = alpha * v[4 * (2 * a + b) + k];
  return r;
}

// float results, or bf16 ones whose rows are no whole 16-byte pieces: straight from the registers.  EXTRA: a residual, or a sum with what is there.
template <bool MASK, bool F32, bool EXTRA>
__device__ __forceinline__ void rd_rows(const GemmParams& p, const f32x16 (&t)[4], const RdOut& o, int i, int lane) {
#pragma unroll
  for (int a = 0; a < 2; a++) {
    const int64_t r = o.row0 + 32 * i + 16 * a + (lane & 15);
    const int c0 = o.col0 + 4 * (lane >> 4);
    if (MASK && (r < o.row_lo || r >= o.row_hi)) continue;
    const bf16_t* rr = (const bf16_t*)p.R + r * p.ldr + c0;
    float* cf = (float*)p.C + r * p.ldc + c0;
    bf16_t* cb = (bf16_t*)p.C + r * p.ldc + c0;
#pragma unroll
    for (int j = 0; j < 4; j++)
#pragma unroll
      for (int b = 0; b < 2; b++) {
        f32x4 v = quad(t[j], a, b, p.alpha);
        if (EXTRA && p.R) { const bf16x4_t x = *reinterpret_cast<const bf16x4_t*>(rr + 32 * j + 16 * b);
#pragma unroll
          for (int k = 0; k < 4; k++) v[k] += (float)x[k]; }
        if (F32) {
          f32x4* q = reinterpret_cast<f32x4*>(cf + 32 * j + 16 * b);
          if (EXTRA && p.accumulate) { const f32x4 x = *q;
#pragma unroll
            for (int k = 0; k < 4; k++) v[k] += x[k]; }
          *q = v;
        } else {
          bf16x4_t w;
#pragma unroll
          for (int k = 0; k < 4; k++) w[k] = (bf16_t)v[k];
          *reinterpret_cast<bf16x4_t*>(cb + 32 * j + 16 * b) = w;
        }
      }
  }
}

// Softmax statistics of the rows 16 a + lane % 16 of a 128-column block: the maximum of alpha * value and the sum of exp(alpha * value - maximum), whose terms
// take the values' place (a lane owns 32 of a row's columns, the others sit in lane ^ 16, lane ^ 32).  What a loss is made of, whichever epilogue wants it.
__device__ __forceinline__ float2 row_stats(f32x16 (&t)[4], int a, float alpha) {
  float m = -INFINITY;
#pragma unroll
  for (int j = 0; j < 4; j++)
#pragma unroll
    for (int e = 0; e < 8; e++) m = fmaxf(m, alpha * t[j][8 * a + e]);
  m = fmaxf(m, __shfl_xor(m, 32, 64));
  m = fmaxf(m, __shfl_xor(m, 16, 64));
  const float nm2 = -kLog2e * m;
  float s = 0.f;
#pragma unroll
  for (int j = 0; j < 4; j++)
#pragma unroll
    for (int e = 0; e < 8; e++) { t[j][8 * a + e] = __builtin_amdgcn_exp2f(fmaf(alpha * t[j][8 * a + e], kLog2e, nm2)); s += t[j][8 * a + e]; }
  s += __shfl_xor(s, 32, 64);
  s += __shfl_xor(s, 16, 64);
  return make_float2(m, s);
}

// bf16 results through the wave's 8 KB of the free half stage, so that a store instruction writes four whole 256-byte row pieces; 16-byte
// chunk c of row r lies at c ^ (r % 16).  A residual takes the same way in: loaded 16 bytes per lane, parked at the place of the result,
// picked up by the lane that owns the element and rounded once with the sum.
// EPI PROB: the values are turned into w_row * (exp(value - lse_row) - [column is the row's label]) before they are rounded.
// EPI ROWS: a row is multiplied by its row_scale * w_row.
// EPI SOFT: exp(value) over a whole power of two, see GemmParams: the statistics' exponentials times one factor per row and block.
template <bool MASK>
__device__ __forceinline__ void rd_load_residual(const GemmParams& p, u32x4 (&res)[8], const RdOut& o, int i, int lane) {
  const int r4 = lane >> 4, c16 = lane & 15;
  if (MASK) {
#pragma unroll
    for (int it = 0; it < 8; it++)
      res[it] = *reinterpret_cast<const u32x4*>((const bf16_t*)p.R + (int64_t)min(max(o.row0 + 32 * i + 4 * it + r4, o.row_lo), o.row_hi - 1) * p.ldr + o.col0 + c16 * 8);
    return;
  }
  const uint32_t at = (uint32_t)((r4 * p.ldr + c16 * 8) * 2);
  const int64_t step = 8 * p.ldr;                          // bytes of four rows
  const char* src = (const char*)((const bf16_t*)p.R + (int64_t)(o.row0 + 32 * i) * p.ldr + o.col0);
#pragma unroll
  for (int it = 0; it < 8; it++, src += step) res[it] = *reinterpret_cast<const u32x4*>(src + at);
}
template <bool MASK, int EPI, bool RES>
__device__ __forceinline__ void rd_staged(const GemmParams& p, f32x16 (&t)[4], u32x4 (&res)[8], unsigned char* my, const RdOut& o, int i, int lane) {
  const int l15 = lane & 15, q = lane >> 4, r4 = lane >> 4, c16 = lane & 15;
  unsigned char* mine = my + l15 * 256 + (q & 1) * 8;      // this lane's row of 16 and its half of a chunk
  const int ch = ((q >> 1) ^ l15) * 16;
  // whole rows: row 4 it + r4, chunk c16 ^ (row % 16), that is (c16 ^ r4) ^ 4 (it % 4)
  unsigned char* rows = my + r4 * 256;
  const int cr = (c16 ^ r4) * 16;
  if (RES) {
#pragma unroll
    for (int it = 0; it < 8; it++) *reinterpret_cast<u32x4*>(rows + it * 1024 + (cr ^ ((it & 3) * 64))) = res[it];
    asm volatile("" ::: "memory");
    if (i < 3) rd_load_residual<MASK>(p, res, o, i + 1, lane);
  }
  if (p.alpha != 1.f) {
#pragma unroll
    for (int j = 0; j < 4; j++)
#pragma unroll
      for (int e = 0; e < 16; e++) t[j][e] *= p.alpha;
  }
#pragma unroll
  for (int a = 0; a < 2; a++) {
    float neg_lse2 = 0.f, wrow = 0.f, soft = 0.f; int clab = -1;
    // rows outside the live range compute with the last live row's values and are not written
    const int rr = o.row0 + 32 * i + 16 * a + l15, r = MASK ? min(max(rr, o.row_lo), o.row_hi - 1) : rr;
    if (EPI == GEMM_EPI_PROB) neg_lse2 = -kLog2e * p.epi_lse[r];
    if (EPI == GEMM_EPI_PROB || EPI == GEMM_EPI_ROWS) wrow = p.epi_w ? p.epi_w[r] : 1.f / (float)*p.epi_cnt;
    if (EPI == GEMM_EPI_ROWS) wrow *= p.row_scale[r];
    if (EPI == GEMM_EPI_PROB || EPI == GEMM_EPI_SOFT) clab = p.epi_lab[r] - o.col0 - 4 * q;   // position of the label among this lane's columns of the block, if any
    if (EPI == GEMM_EPI_SOFT) {
      const float2 st = row_stats(t, a, 1.f);              // t: the exponentials of the statistics from here on
      soft = soft_scale(st.x, soft_exponent(p.epi_zlab[r], st.x));
      if (lane < 16 && (!MASK || r == rr)) *(reinterpret_cast<float2*>(p.epi_part) + (int64_t)r * (p.N / 128) + o.col0 / 128) = st;
    }
#pragma unroll
    for (int j = 0; j < 4; j++)
#pragma unroll
      for (int b = 0; b < 2; b++) {
        bf16x4_t* at = reinterpret_cast<bf16x4_t*>(mine + a * 4096 + (ch ^ ((4 * j + 2 * b) * 16)));
        f32x4 v = quad(t[j], a, b, 1.f);
        if (EPI == GEMM_EPI_ROWS) {
#pragma unroll
          for (int k = 0; k < 4; k++) v[k] *= wrow;
        }
        if (EPI == GEMM_EPI_SOFT) {
#pragma unroll
          for (int k = 0; k < 4; k++) v[k] *= soft;
          const int at_k = clab - (32 * j + 16 * b);       // one block in V / 128 holds a row's label
          if (at_k >= 0 && at_k < 4 && (!MASK || r == rr)) p.epi_elab[r] = at_k == 0 ? v[0] : at_k == 1 ? v[1] : at_k == 2 ? v[2] : v[3];
        }
        if (EPI == GEMM_EPI_PROB) {
#pragma unroll
          for (int k = 0; k < 4; k++)
            v[k] = wrow * (__builtin_amdgcn_exp2f(fmaf(v[k], kLog2e, neg_lse2)) - (clab == 32 * j + 16 * b + k ? 1.f : 0.f));
        }
        if (RES) { const bf16x4_t x = *at;
#pragma unroll
          for (int k = 0; k < 4; k++) v[k] += (float)x[k]; }
        bf16x4_t w;
#pragma unroll
        for (int k = 0; k < 4; k++) w[k] = (bf16_t)v[k];
        *at = w;
      }
  }
  asm volatile("" ::: "memory");                           // LDS operations of a wave complete in order
  u32x4 out[8];
#pragma unroll
  for (int it = 0; it < 8; it++) out[it] = *reinterpret_cast<const u32x4*>(rows + it * 1024 + (cr ^ ((it & 3) * 64)));
  const uint32_t at = (uint32_t)((r4 * p.ldc + c16 * 8) * 2);
  const int64_t step = 8 * p.ldc;                          // bytes of four rows
  char* c = (char*)((bf16_t*)p.C + (int64_t)(o.row0 + 32 * i) * p.ldc + o.col0);
#pragma unroll
  for (int it = 0; it < 8; it++, c += step) {
    const int r = o.row0 + 32 * i + 4 * it + r4;
    if (!MASK || (r >= o.row_lo && r < o.row_hi)) *reinterpret_cast<u32x4*>(c + at) = out[it];
  }
  asm volatile("" ::: "memory");
}

// Softmax statistics of the logits, nothing of which is written.
template <bool MASK>
__device__ __forceinline__ void rd_stats(const GemmParams& p, f32x16 (&t)[4], const RdOut& o, int i, int lane) {
#pragma unroll
  for (int a = 0; a < 2; a++) {
    const float2 st = row_stats(t, a, p.alpha);
    const int r = o.row0 + 32 * i + 16 * a + (lane & 15);
    if (lane < 16 && (!MASK || (r >= o.row_lo && r < o.row_hi))) *(reinterpret_cast<float2*>(p.epi_part) + (int64_t)r * (p.N / 128) + o.col0 / 128) = st;
  }
}

// wave-uniform values the compiler does not know to be so, into scalar registers
__device__ __forceinline__ int uni(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ uint64_t uni(uint64_t x) { return (uint64_t)(uint32_t)uni((int)(x >> 32)) << 32 | (uint32_t)uni((int)x); }

template <int LIVE, int EPI = GEMM_EPI_NONE, int LAYOUT = RD_NT>
__global__ __launch_bounds__(256) void gemm_mfma_rd_kernel(GemmParams p, int m_off, int tiles_m, int tiles_n) {
  constexpr int BM = 256, BN = 256;
  constexpr bool NN = LAYOUT == RD_NN, AK = LAYOUT == RD_TN;      // B is [K, N]; A is [K, M] and B [K, N]
  extern __shared__ __align__(16) unsigned char smem[];
  const RdLaunch g = rd_launch<LIVE, LAYOUT, EPI == GEMM_EPI_NONE || EPI == GEMM_EPI_ROWS>(p, m_off, tiles_m, tiles_n);
  const int items = g.items, first_split = g.first_split, parts = g.parts;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave >> 1, wn = wave & 1;
  const GemmSeg s0 = p.seg[0], s1 = p.nseg > 1 ? p.seg[1] : p.seg[0];

  if ((int)blockIdx.x >= items) return;
  // per-lane LDS read addresses, by slice or (transposing reads) by pair of column blocks, and global offsets of even and odd loads
  unsigned ar[4], br[4], oa0[2], ob0[2], oa1[2], ob1[2];
  {
    const int l15 = lane & 15, q = lane >> 4, r = (lane >> 2) & 3, lrow = lane >> 3, lch = lane & 7, l31 = lane & 31, hh = lane >> 5;
#pragma unroll
    for (int k = 0; k < 4; k++) {
      const unsigned c = (unsigned)(l15 * 128 + (((4 * (k & 1) + q) ^ (l15 >> 1)) * 16)), t = (unsigned)((8 * q + r) * 512 + ((k ^ r) * 64) + (lane & 3) * 8);
      ar[k] = AK ? t + (unsigned)(wm * 256) : c + (unsigned)(wm * 128 * 128);
      br[k] = LAYOUT != RD_NT ? t + (unsigned)(wn * 256) : c + (unsigned)(wn * 128 * 128);
    }
#pragma unroll
    for (int o = 0; o < 2; o++) {
      const int ch = (lch ^ ((lrow >> 1) | (o * 4))) * 8, cu = ((l31 >> 2) ^ (2 * o + hh)) * 32 + (l31 & 3) * 8;
      oa0[o] = (unsigned)((AK ? hh * s0.lda + cu : lrow * s0.lda + ch) * 2); oa1[o] = (unsigned)((lrow * s1.lda + ch) * 2);
      ob0[o] = (unsigned)((LAYOUT != RD_NT ? hh * s0.ldb + cu : lrow * s0.ldb + ch) * 2); ob1[o] = (unsigned)((lrow * s1.ldb + ch) * 2);
    }
  }
  // bytes between two loads: eight rows, or two rows of the contraction; bytes of a step of the contraction
  const int sa0 = (int)((AK ? 4 : 16) * s0.lda), sa1 = (int)(16 * s1.lda), sb0 = (int)((LAYOUT != RD_NT ? 4 : 16) * s0.ldb), sb1 = (int)(16 * s1.ldb);
  const int ka = (int)(128 * s0.lda), kb = (int)(128 * s0.ldb);
  int half = 0, fresh = 1;                                 // LDS half stage of the next item's first step; nothing of it under way
  for (int item = blockIdx.x; item < items; item += (int)gridDim.x) {
    const RdItem w = rd_item<LIVE, LAYOUT>(p, g, item, wave);
    const RdNext nx = rd_next<LIVE, LAYOUT>(p, g, w, item, (int)gridDim.x, wave);
    if (AK && w.nt == 0) {                                 // no live rows to contract (in any item, or in this part): the sum is zero
      if (!p.accumulate || w.kpart >= 0) {
        float* c = w.kpart >= 0 ? p.tail_part + ((int64_t)(w.pid - first_split) * parts + w.kpart) * (BM * BN) : (float*)row_group_base(p, w.row0) + (int64_t)w.row0 * p.ldc + w.col0;
        const int64_t ld = w.kpart >= 0 ? BN : p.ldc;
        for (int r = tid >> 6; r < BM; r += 4) *reinterpret_cast<f32x4*>(c + r * ld + lane * 4) = (f32x4){0.f, 0.f, 0.f, 0.f};
      }
    } else {
      f32x16 acc[4][4];
      const int off = half * 32768, lw = wave * 8192;
#define RD_LOOP(name) \
      asm volatile(GEMM_##name##_LOOP_ASM \
                   : "={a[0:15]}"(acc[0][0]), "={a[16:31]}"(acc[0][1]), "={a[32:47]}"(acc[0][2]), "={a[48:63]}"(acc[0][3]), \
                     "={a[64:79]}"(acc[1][0]), "={a[80:95]}"(acc[1][1]), "={a[96:111]}"(acc[1][2]), "={a[112:127]}"(acc[1][3]), \
                     "={a[128:143]}"(acc[2][0]), "={a[144:159]}"(acc[2][1]), "={a[160:175]}"(acc[2][2]), "={a[176:191]}"(acc[2][3]), \
                     "={a[192:207]}"(acc[3][0]), "={a[208:223]}"(acc[3][1]), "={a[224:239]}"(acc[3][2]), "={a[240:255]}"(acc[3][3]) \
                   : "v"(ar[0]), "v"(ar[1]), "v"(ar[2]), "v"(ar[3]), "v"(br[0]), "v"(br[1]), "v"(br[2]), "v"(br[3]), \
                     "v"(oa0[0]), "v"(oa0[1]), "v"(ob0[0]), "v"(ob0[1]), "v"(oa1[0]), "v"(oa1[1]), "v"(ob1[0]), "v"(ob1[1]), \
                     "s"(uni(w.a0)), "s"(uni(w.b0)), "s"(uni(w.a1)), "s"(uni(w.b1)), "s"(uni(nx.an)), "s"(uni(nx.bn)), "s"(sa0), "s"(sb0), "s"(sa1), "s"(sb1), \
                     "s"(uni(w.nt0)), "s"(uni(w.nt)), "s"(uni(nx.lim)), "s"(uni(off)), "s"(lw), "s"(uni(fresh)), "s"(uni(w.b2)), "s"(uni(w.b3)), "s"(uni(w.n1)), "s"(uni(w.n2)), "s"(kb), "s"(ka) \
                   : GEMM_##name##_LOOP_CLOBBERS)
      if constexpr (AK) RD_LOOP(RD_TN);
      else if constexpr (NN) RD_LOOP(RD_NN);
      else RD_LOOP(RD);
#undef RD_LOOP
      half = (half + 2 * (w.nt % 5)) % 5; fresh = !nx.chain;
      unsigned char* my = smem + ((half + 4) % 5) * 32768 + wave * 8192;
      GemmParams q = p;
      RdOut o = {w.row0 + wm * 128, w.col0 + wn * 128, w.row_lo, w.row_hi};
      const bool part = (EPI == GEMM_EPI_NONE || EPI == GEMM_EPI_ROWS) && w.kpart >= 0;
      if (part) {                                          // raw float sums of this part into the tile's scratch
        q.C = p.tail_part + ((int64_t)(w.pid - first_split) * parts + w.kpart) * (BM * BN); q.ldc = BN; q.c_f32 = 1; q.alpha = 1.f; q.R = nullptr; q.accumulate = 0;
        o = {wm * 128, wn * 128, 0, BM};
      } else if (AK) q.C = row_group_base(p, w.row0);
      const bool staged = EPI == GEMM_EPI_PROB || EPI == GEMM_EPI_SOFT || (!AK && EPI == GEMM_EPI_NONE && !q.c_f32 && !(q.ldc % 8) && (!q.R || (!(q.ldr % 8) && !((uintptr_t)q.R % 16))));
      constexpr bool MASK = LIVE != 0;
      u32x4 res[8];
      if (EPI == GEMM_EPI_NONE && staged && q.R) rd_load_residual<MASK>(q, res, o, 0, lane);
#pragma unroll
      for (int i = 0; i < 4; i++) {
        f32x16 t[4] = {acc[i][0], acc[i][1], acc[i][2], acc[i][3]};
        int el = lane;                                     // the piece's per-lane addresses are formed here, not kept across the loop
        asm volatile("" : "+v"(t[0]), "+v"(t[1]), "+v"(t[2]), "+v"(t[3]), "+v"(el));
        if constexpr (EPI == GEMM_EPI_STATS) rd_stats<MASK>(q, t, o, i, el);
        else if constexpr (EPI == GEMM_EPI_PROB) rd_staged<MASK, GEMM_EPI_PROB, false>(q, t, res, my, o, i, el);
        else if constexpr (EPI == GEMM_EPI_SOFT) rd_staged<MASK, GEMM_EPI_SOFT, false>(q, t, res, my, o, i, el);
        else if constexpr (EPI == GEMM_EPI_ROWS) {
          if (part) rd_rows<MASK, true, false>(q, t, o, i, el); else rd_staged<MASK, GEMM_EPI_ROWS, false>(q, t, res, my, o, i, el);
        }
        else if constexpr (AK) {
          if (q.accumulate) rd_rows<false, true, true>(q, t, o, i, el); else rd_rows<false, true, false>(q, t, o, i, el);
        } else if (staged && q.R) rd_staged<MASK, GEMM_EPI_NONE, true>(q, t, res, my, o, i, el);
        else if (staged) rd_staged<MASK, GEMM_EPI_NONE, false>(q, t, res, my, o, i, el);
        else if (q.c_f32 && !q.R && !q.accumulate) rd_rows<MASK, true, false>(q, t, o, i, el);
        else if (q.c_f32) rd_rows<MASK, true, true>(q, t, o, i, el);
        else rd_rows<MASK, false, true>(q, t, o, i, el);
      }
    }
  }
  __builtin_amdgcn_s_waitcnt(0x0f70);                    // loads that nobody reads must land before the workgroup's LDS is released
}

template <int BM, int BN, int WM, int WN>
static int launch_dlds_cfg(as_ctx* ctx, const GemmParams& p, int m_off, hipStream_t st) {
  size_t smem = (size_t)2 * (BM + BN) * 64 * sizeof(bf16_t);
  constexpr auto k0 = gemm_mfma_dlds_kernel<BM, BN, WM, WN>;
  AS_SET_SMEM(ctx, k0, smem);
  int tm = (int)cdiv(p.M, BM), tn = (int)cdiv(p.N, BN);
  dim3 grid(tm * tn, p.splitk > 1 ? p.splitk : 1);
  k0<<<grid, WM * WN * 64, smem, st>>>(p, m_off, tm, tn);
  AS_LAUNCH_CHECK(ctx);
  return AS_OK;
}

// Second launch for split tiles: sum of the parts in order, then the usual epilogue.
// Sixteen workgroups per tile (16 rows each), the same workgroup -> tile mapping as the main kernel; a thread owns 4
// consecutive columns.
__global__ __launch_bounds__(256) void gemm_tail_fixup_kernel(GemmParams p, int m_off, int tiles_m, int tiles_n) {
  constexpr int BM = 256, BN = 256, GROUP = 4, WPT = 16;
  const int tile = blockIdx.x / WPT, r_first = (blockIdx.x % WPT) * (BM / WPT);
  int live = p.M, parts = p.tail_parts, first = p.tail_first, rb = 0;
  const bool counted = p.m_dev || p.grp_n > 0;
  if (counted) {
    int mmax;
    if (p.grp_n > 0) tiles_m = min(tiles_m, group_row_tiles(p));
    else { live = gemm_rows(p, m_off, rb, mmax); tiles_m = min(tiles_m, (max(live, 0) + BM - 1) / BM); }
    const LiveSplit v = live_split(p, tiles_m * tiles_n);
    if (v.parts <= 1) return;
    first = v.first; parts = v.parts;
  }
  const int nblk = tiles_m * tiles_n, pid = first + tile;
  if (pid >= nblk) return;
  const int q8 = nblk / 8, rem = nblk % 8, xcd = pid % 8, loc = pid / 8;
  const int logical = xcd * q8 + min(xcd, rem) + loc;
  const int in_group = GROUP * tiles_n, grp = logical / in_group, first_m = grp * GROUP;
  const int gsize = min(tiles_m - first_m, GROUP);
  int tile_m = first_m + (logical % in_group) % gsize;
  const int tile_n = (logical % in_group) / gsize;
  if (p.grp_n > 0) {                                     // the tile's group and which of its tiles it is
    int e = 0;
    live = p.grp_off[1] - p.grp_off[0];
    while (tile_m >= (live + BM - 1) / BM && e + 1 < p.grp_n) {
      tile_m -= (live + BM - 1) / BM; e++;
      live = p.grp_off[e + 1] - p.grp_off[e];
    }
    rb = p.grp_off[e];
  }
  const float* h0 = p.tail_part + (int64_t)tile * parts * (BM * BN);
  const int c = (threadIdx.x & 63) * 4;
  // as the main kernel: a ragged last tile was moved up; it writes its own rows (and rows past M where the operands have them)
  const bool spare = !counted && p.rows_cap >= tiles_m * BM;
  const int row_lo = rb + tile_m * BM, row0 = spare ? row_lo : min(row_lo, (p.grp_off ? p.rows_cap : p.M) - BM), row_hi = spare ? tiles_m * BM : rb + live;
  constexpr int RPT = BM / WPT / 4;                      // rows of a thread, four apart
  f32x4 sum[RPT];
  const float* h = h0 + (r_first + (threadIdx.x >> 6)) * BN + c;
#pragma unroll
  for (int i = 0; i < RPT; i++) sum[i] = *reinterpret_cast<const f32x4*>(h + i * 4 * BN);
  for (int s = 1; s < parts; s++) {
    h += BM * BN;
#pragma unroll
    for (int i = 0; i < RPT; i++) sum[i] += *reinterpret_cast<const f32x4*>(h + i * 4 * BN);
  }
#pragma unroll
  for (int i = 0; i < RPT; i++) {
    const int64_t row = (int64_t)row0 + r_first + (threadIdx.x >> 6) + 4 * i; const int col = tile_n * BN + c;
    if (row >= row_lo && row < row_hi) {
      f32x4 v = sum[i];
      float f = p.alpha;
      if (p.row_scale) f = p.row_scale[row] * (p.epi_w ? p.epi_w[row] : 1.f / (float)*p.epi_cnt);
#pragma unroll
      for (int k = 0; k < 4; k++) v[k] *= f;
      if (p.R) { const bf16x4_t x = *reinterpret_cast<const bf16x4_t*>((const bf16_t*)p.R + row * p.ldr + col);
#pragma unroll
        for (int k = 0; k < 4; k++) v[k] += (float)x[k]; }
      if (p.c_f32) {
        f32x4* q = reinterpret_cast<f32x4*>((float*)(p.nrg ? row_group_base(p, row0) : p.C) + row * p.ldc + col);
        if (p.accumulate) v += *q;
        *q = v;
      } else {
        bf16x4_t w;
#pragma unroll
        for (int k = 0; k < 4; k++) w[k] = (bf16_t)v[k];
        *reinterpret_cast<bf16x4_t*>((bf16_t*)p.C + row * p.ldc + col) = w;
      }
    }
  }
}

// whole 256 x 256 tiles of a plain launch (host-side row count, no split-K, K segments in 64-wide steps, 16-byte rows)
static bool rd_ok(const GemmParams& p) {
  if (p.splitk > 1 || p.M < 256 || (p.N % 256)) return false;
  if (p.grp_off && p.rows_cap < 256) return false;       // grouped rows: the caller states how many rows the operands have
  if (p.grp_n > 0 && (p.nseg != 1 || p.m_dev)) return false;
  // the epilogue stores four consecutive columns of a row at a time
  if ((p.ldc % 4) || ((uintptr_t)p.C % 16) || (p.R && ((p.ldr % 4) || ((uintptr_t)p.R % 8)))) return false;
  for (int s = 0; s < p.nseg; s++)
    if ((p.seg[s].K % 64) || p.seg[s].K < 64 || p.seg[s].lda * 16 > INT32_MAX || p.seg[s].ldb * 16 > INT32_MAX) return false;
  int nt = 0; for (int s = 0; s < p.nseg; s++) nt += (int)(p.seg[s].K / 64);
  return nt >= 1;
}

static bool rd_live(const GemmParams& p) { return p.m_dev || p.grp_off; }
static int fma_tile(const GemmParams& p) { return cdiv(p.N, 64) * cdiv(p.M, 64) * p.splitk >= kCus ? 64 : 32; }

// Float products: gemm_f32_kernel with 16 x 16 or 32 x 32 results per workgroup, gemm_fma_kernel with 32 x 32 or 64 x 64; B by rows of K: the first
// two only.  Which one: the time that a fit to measured ones expects (us): a launch, the chain of one tile's contraction, and the work of
// n tiles per CU, the last two joined as max (16 x 16) or as hypotenuse; rows that are not whole 16-byte pieces, which gemm_f32_kernel loads
// value by value, have a fit of their own.  Fitted to all four kernels, operands new to the L2s, on 41 pairs of N and K (8 x 16 to 32000 x
// 2048, a fifth of them odd) and row counts from 16 to 200,000, 532 shapes, and held against 678 shapes on operands just used.  gemm_fma_kernel's
// own choice of tile, which had these products alone, is given 8 % ahead (20 where rows are not whole pieces: the fit is worse there): the pick is 1.5 times as fast as that one on average, 8 % slower at
// worst and more than 2 % at four shapes; 1.3 % over the best of the four on average.  Of the small tiles the 16 x 16 ones are 5 % ahead: four
// times the workgroups where operands come from further away than measured.  (us, kernels in the order below: 478 x 384 x 128 5.7, 5.8, 6.6,
// 11.6; 1003 x 1024 x 128 15, 12, 10.5, 12.6; 478 x 1024 x 1024 40, 25, 33, 60; 8192 x 3072 x 1024 -, 901, 970, 717; 2048 x 452 x 654 111, 70, 52, 49.)
enum { F32_16, F32_32, FMA_32, FMA_64 };
static constexpr int kF32Shift[4] = {4, 5, 5, 6}, kF32Tile[4] = {16, 32, 32, 64};
static bool f32_whole_rows(const GemmParams& p, bool nn) {
  for (int s = 0; s < p.nseg; s++) {
    const GemmSeg& g = p.seg[s];
    if (g.K % 4 || g.lda % 4 || (uintptr_t)g.A % 16 || (!nn && (g.ldb % 4 || (uintptr_t)g.B % 16))) return false;
  }
  return true;
}
struct F32Shape { int64_t rows; bool whole; int K1, K2; double parts; };
static double f32_time(int kernel, int nn, const F32Shape& x, int N) {
  struct Fit { double launch, step, base, tile_step, tile_base; };
  static constexpr Fit nt_fit[2][4] = {{{3.11, 0.0101, 0.253, 0.01, 0.343}, {1.75, 0.0295, 1.61, 0.0222, 1.41}, {3.8, 0.0297, 0.073, 0.0147, 0.747}, {5.16, 0.0626, 0., 0.0339, 1.59}},
                                       {{3.61, 0.00397, 0., 0.00425, 0.265}, {3.44, 0.0105, 0.174, 0.00835, 1.32}, {3.32, 0.023, 0., 0.0101, 0.474}, {3.99, 0.0533, 0., 0.029, 1.02}}};
  static constexpr Fit nn_fit[2][2] = {{{3.02, 0.00667, 0.723, 0.00732, 0.522}, {1.1, 0.0208, 3.17, 0.0153, 1.8}}, {{3.65, 0.00382, 0., 0.0045, 0.271}, {2.04, 0.0117, 2.12, 0.00869, 1.46}}};
  const Fit& f = nn ? nn_fit[x.whole][kernel] : nt_fit[x.whole][kernel];
  const int s = kF32Shift[kernel], b1 = kF32Tile[kernel] - 1;
  static constexpr int step[4] = {16, 16, 64, 32};         // of the contraction: what a short second segment costs
  const double K = (double)(x.K1 + (x.K2 + step[kernel] - 1) / step[kernel] * step[kernel]) / x.parts;
  const double n = (double)((((int64_t)N + b1) >> s) * ((x.rows + b1) >> s)) * x.parts * (1. / kCus);     // (a step of a small model asks some hundred times: shifts, no hypot)
  if (kernel == F32_16 && n > 16.) return 1e30;            // beyond what was measured
  const double chain = f.base + f.step * K, work = (f.tile_base + f.tile_step * K) * n;
  const double several = nn < 2 ? 1. : kernel == F32_16 ? 1.22 : 1.45;       // more than one matrix: a choice per element (1.06-1.34 and 1.13-1.63 measured)
  return (f.launch + (kernel == F32_16 ? std::max(chain, work) : std::sqrt(chain * chain + work * work))) * several * (kernel == F32_32 ? 1.05 : 1.);
}
// column groups side by side in one launch: groups of whole tiles, or (gemm_f32_kernel) any if A is the same for all
static bool f32_groups_fit(const GemmParams& p, int kernel) {
  if (kernel <= F32_32 && p.nseg == 1) return true;
  for (int g = 0; g < p.ncg; g++) if (p.cg_end[g] % kF32Tile[kernel]) return false;
  return true;
}
struct F32Pick { int kernel; double time; };
static F32Pick f32_pick(const GemmParams& p, int variant, bool nn) {
  const int usual = fma_tile(p) == 64 ? FMA_64 : FMA_32;
  if (variant == 1) return {usual, 0.};
  // rows: those a group may expect; of rows counted on the device (targets) a quarter
  const int64_t rows = p.grp_off && p.grp_rows > 0 ? std::max<int64_t>(1, (int64_t)p.grp_rows / std::max(1, p.grp_n)) : p.m_dev ? (p.M + 3) / 4 : p.M;
  const F32Shape x = {rows, f32_whole_rows(p, nn), p.seg[0].K, p.nseg > 1 ? p.seg[1].K : 0, (double)p.splitk};
  F32Pick best{nn ? F32_32 : usual, 1e30};
  for (int k = 0; k < (nn ? 2 : 4); k++) {
    if (k != FMA_64 && (p.M - 1) >> kF32Shift[k] >= 65535) continue;  // rows of a grid
    double t = 0.;
    if (f32_groups_fit(p, k)) t = f32_time(k, nn ? p.nn : 0, x, p.N);
    else for (int g = 0; g < p.ncg; g++) t += f32_time(k, 0, x, p.cg_end[g] - (g ? p.cg_end[g - 1] : 0));      // one launch each
    if (!nn && k != usual) t *= x.whole ? 1.08 : 1.2;
    if (t < best.time) best = {k, t};
  }
  return best;
}
static bool f32_nn_ok(int variant, const GemmParams& p) {
  return variant == 0 && p.nn >= 1 && p.nn <= 3 && !p.ncg && (p.nseg < 2 || p.seg[1].ldb == p.seg[0].ldb) && (p.M - 1) >> 5 < 65535;
}
// B by rows of K, against a transposed copy of its matrices (at least 2.4 us each, 1.4 us per million elements) and the product with that one;
// 10 % ahead for the copy, which was the only way: 1.7 times as fast on average over the shapes above, 7 % slower at worst
static bool f32_nn_pays(const GemmParams& p) {
  const double launches = 2.4 * p.nn, bytes = 1.4e-6 * p.seg[0].K * p.N, copy = std::sqrt(launches * launches + bytes * bytes);
  return f32_pick(p, 0, true).time * 1.1 < copy + f32_pick(p, 0, false).time;
}
// rows counted on the device whose contraction is long enough (sixteen parts of eight steps) to be split by the live count
static bool live_split_ok(const GemmParams& p) {
  return (p.grp_off ? p.grp_n > 0 : p.m_dev != nullptr) && p.tail_part && p.nseg == 1 && p.epi == GEMM_EPI_NONE && k_steps(p) >= 8 * kLiveParts;
}
// what the ring kernels need: plain rows, whole K steps, rows of C and R in 16-byte pieces, 32-bit offsets inside a tile
static bool ring_ok(const GemmParams& p) {
  if (rd_live(p) || p.splitk > 1 || p.epi != GEMM_EPI_NONE || p.N % 8 || p.ldc % 8 || ((uintptr_t)p.C % 16)) return false;
  if (p.R && (p.ldr % 8 || ((uintptr_t)p.R % 16))) return false;
  for (int s = 0; s < p.nseg; s++)
    if (p.seg[s].K % 64 || p.seg[s].K < 64 || p.seg[s].lda > (1 << 22) || p.seg[s].ldb > (1 << 22)) return false;
  return true;
}
static bool mfma_ok(const GemmParams& p);
bool gemm_rd_applies(int mode, const GemmParams& p) { return mode == AS_BF16 && mfma_ok(p) && rd_ok(p); }

template <int LIVE, int LAYOUT, int EPI = GEMM_EPI_NONE>
static int launch_tiles(as_ctx* ctx, const GemmParams& p, int m_off, int wgs, int tm, int tn, hipStream_t st) {
  AS_SET_SMEM(ctx, (gemm_mfma_rd_kernel<LIVE, EPI, LAYOUT>), kRdSmem);
  gemm_mfma_rd_kernel<LIVE, EPI, LAYOUT><<<dim3(std::min(wgs, kCus)), 256, kRdSmem, st>>>(p, m_off, tm, tn);
  AS_LAUNCH_CHECK(ctx);
  return AS_OK;
}

// parts > 1: the contraction of every tile is split over that many workgroups.
static int launch_256(as_ctx* ctx, const GemmParams& p_in, int m_off, int parts, hipStream_t st) {
  GemmParams p = p_in;
  const int tn = p.N / 256;
  int rc;
  p.tail_first = -1; p.tail_parts = 2;
  if (p.epi != GEMM_EPI_NONE && !p.m_dev) return as_fail(ctx, AS_ERR_SHAPE, "gemm: the head epilogues run over a device-side row count");
  if (rd_live(p)) {                                      // every row tile the live rows can reach; the kernel drops the rest
    const int tm = p.grp_n > 0 ? (int)cdiv(p.rows_cap, 256) + p.grp_n : (int)cdiv(p.M, 256);
    if (p.epi == GEMM_EPI_STATS) return launch_tiles<1, RD_NT, GEMM_EPI_STATS>(ctx, p, m_off, tm * tn, tm, tn, st);
    if (p.epi == GEMM_EPI_PROB) return launch_tiles<1, RD_NT, GEMM_EPI_PROB>(ctx, p, m_off, tm * tn, tm, tn, st);
    if (p.epi == GEMM_EPI_SOFT) return launch_tiles<1, RD_NT, GEMM_EPI_SOFT>(ctx, p, m_off, tm * tn, tm, tn, st);
    if (!live_split_ok(p)) p.tail_part = nullptr;
    const int wgs = p.tail_part ? std::max(tm * tn, kCus) : tm * tn;
    rc = p.row_scale ? launch_tiles<1, RD_NN, GEMM_EPI_ROWS>(ctx, p, m_off, wgs, tm, tn, st) : p.nn ? launch_tiles<1, RD_NN>(ctx, p, m_off, wgs, tm, tn, st) : launch_tiles<1, RD_NT>(ctx, p, m_off, wgs, tm, tn, st);
    if (!rc && p.tail_part) { gemm_tail_fixup_kernel<<<dim3(16 * std::min(tm * tn, 128)), 256, 0, st>>>(p, m_off, tm, tn); AS_LAUNCH_CHECK(ctx); }
    return rc;
  }
  // a ragged last row tile runs over rows past M when the operands have them, else it is moved up (instance 2)
  const int tm = (int)cdiv(p.M, 256), T = tm * tn;
  const bool whole = p.rows_cap >= tm * 256 || p.M % 256 == 0;
  if (p.M % 256 == 0) p.rows_cap = p.M;
  if (parts > 1) { p.tail_first = 0; p.tail_parts = parts; }
  else if (tail_splits(p, T)) { p.tail_first = T / kCus * kCus; p.tail_parts = tail_parts(p, T % kCus); }
  const int split = p.tail_first >= 0 ? T - p.tail_first : 0;
  const int wgs = T - split + split * p.tail_parts;
  if (p.tn) rc = launch_tiles<0, RD_TN>(ctx, p, 0, wgs, tm, tn, st);
  else if (p.nn && whole) rc = launch_tiles<0, RD_NN>(ctx, p, 0, wgs, tm, tn, st);
  else if (p.nn) rc = launch_tiles<2, RD_NN>(ctx, p, 0, wgs, tm, tn, st);
  else if (whole) rc = launch_tiles<0, RD_NT>(ctx, p, 0, wgs, tm, tn, st);
  else rc = launch_tiles<2, RD_NT>(ctx, p, 0, wgs, tm, tn, st);
  if (!rc && split) { gemm_tail_fixup_kernel<<<dim3(16 * split), 256, 0, st>>>(p, 0, tm, tn); AS_LAUNCH_CHECK(ctx); }
  return rc;
}

template <int BM, int BN, int NST>
static int launch_ring_cfg(as_ctx* ctx, const GemmParams& p_in, int splits, hipStream_t st) {
  GemmParams p = p_in;
  if (p.nseg < 2) p.seg[1] = p.seg[0];                   // the kernel forms the second segment's addresses in any case
  p.splitk = splits; p.partial = p.tail_part;
  constexpr size_t smem = (size_t)NST * (BM + BN) * 64 * sizeof(bf16_t);
  AS_SET_SMEM(ctx, (gemm_mfma_ring_kernel<BM, BN, NST>), smem);
  const int tm = (int)cdiv(p.M, BM), tn = (int)cdiv(p.N, BN), nb = std::max(p.nbat, 1);
  gemm_mfma_ring_kernel<BM, BN, NST><<<dim3((unsigned)((int64_t)tm * tn), splits, nb), 256, smem, st>>>(p, tm, tn);
  AS_LAUNCH_CHECK(ctx);
  if (splits > 1) {
    gemm_splitk_finish_kernel<<<dim3((unsigned)cdiv((int64_t)p.M * p.N, 1024), nb), 256, 0, st>>>(p);
    AS_LAUNCH_CHECK(ctx);
  }
  return AS_OK;
}

template <int BM, int BN, int WM, int WN>
static int launch_mfma_cfg(as_ctx* ctx, const GemmParams& p, int m_off, hipStream_t st) {
  constexpr int LS = 72;
  size_t smem = (size_t)2 * (BM + BN) * LS * sizeof(bf16_t);
  bool edge = false;
  for (int s = 0; s < p.nseg; s++) edge = edge || (p.seg[s].K % 64 != 0);
  constexpr auto k0 = gemm_mfma_kernel<BM, BN, WM, WN, false>;
  constexpr auto k1 = gemm_mfma_kernel<BM, BN, WM, WN, true>;
  AS_SET_SMEM(ctx, k0, smem);
  AS_SET_SMEM(ctx, k1, smem);
  int tm = (int)cdiv(p.M, BM), tn = (int)cdiv(p.N, BN);
  dim3 grid(tm * tn, p.splitk > 1 ? p.splitk : 1);
  if (edge) k1<<<grid, WM * WN * 64, smem, st>>>(p, m_off, tm, tn);
  else k0<<<grid, WM * WN * 64, smem, st>>>(p, m_off, tm, tn);
  AS_LAUNCH_CHECK(ctx);
  return AS_OK;
}

static bool mfma_ok(const GemmParams& p) {
  if (p.R && (p.ldr % 1)) return false;
  for (int s = 0; s < p.nseg; s++) {
    const GemmSeg& g = p.seg[s];
    if (g.K % 8 || g.lda % 8 || g.ldb % 8) return false;
    if (((uintptr_t)g.A | (uintptr_t)g.B) % 16) return false;
  }
  return true;
}

// Tile configuration of the MFMA kernels.  Register-staged (any K that is a multiple of 8): 0 = 256x256 (8 waves,
// 128x64 each), 1 = 256x64, 2 = 64x256, 3 = 128x128, 4 = 128x64.  20 = direct-to-LDS 256x256 with 8 waves (K in 64-wide steps);
// 24 = the hand-scheduled persistent 256x256 kernel with 4 waves; 25, 26 = ring of stages, 128x128 and 64x64 tiles.
struct GemmPick { int cfg, parts; };                     // parts: workgroups that share a tile's contraction

// Plain rows in whole K steps: the kernel and the split that a time model (us) says is fastest:
//   256x256 hand-scheduled  0.815 per K step and 14.4 per round of 256 workgroups (start-up and epilogue of a tile)
//   128x128 ring            0.684 per step and 2.32 per round with two workgroups on every CU, 0.644 with one, 2.28 per launch
//   64x64 ring              0.387 and 0.275, 4.36 per launch
// and for a split the second launch, its partials written and read at about 4 TB/s, and its serial sum over the parts.
// More than half a round of 256x256 tiles goes to the hand-scheduled kernel unsplit without looking further: from there on it
// is mostly 15-40 % ahead; behind only where few steps meet a second round of few tiles (822 x 18432 x 832, 288 tiles: 43 against 33).  Fitted to the choice itself, over every candidate (1 to 12 parts) of 19 pairs of N and K, those of
// the 1B and 8B projections and adapters and narrow ones of 256 to 1280 columns, at ten row counts from 100 to 18,787, operands new to the
// L2s: the pick is 0.4 % over the best on average, more than 10 % at two of 182 shapes, 19 % at worst (100 x 14336 x 4160); with 129 more,
// from 2 rows and one step on, 0.7 %.  Constants fitted to the projections' widths alone were 3.7 % over it on average and 35 % at worst (588 x
// 1024 x 4160: 23.7 where three parts take 18.3).
// Examples (us): 1531 x 4096 x 14400: 64x64 ring 330, 128x128 218, 256x256 in two parts 158; 1003 x 2048 x 8256: 72, 49 (four parts), 51 (six);
// 1003 x 2048 x 16512: 128x128 in four parts 86, 256x256 in eight 73.
static GemmPick pick_plain(const GemmParams& p) {
  const int steps = k_steps(p);
  const double mb = (double)p.M * p.N * 4e-6;
  const bool can_split = p.tail_part != nullptr;
  GemmPick best{24, 1}; double best_t = 1e30;
  auto offer = [&](int cfg, int parts, double t) { if (t < best_t) { best_t = t; best = {cfg, parts}; } };
  const int try_parts[] = {1, 2, 3, 4, 6, 8, 12};
  const bool rs = rd_ok(p);
  if (rs && cdiv(p.M, 256) * (p.N / 256) > kCus / 2) return best;
  for (int parts : try_parts) {
    if (parts > 1 && (!can_split || parts > steps / 2)) break;
    const double per = (double)cdiv(steps, parts);
    if (rs) {
      const int64_t T = cdiv(p.M, 256) * (p.N / 256);      // at most half a round
      if (parts == 1) offer(24, 1, per * 0.815 + 14.4);
      else if (T * parts <= kCus && steps / parts >= 3 && (steps - cdiv(steps, parts)) < (int64_t)(p.seg[0].K / 64))
        offer(24, parts, per * 0.815 + 14.4 + 5.47 + 0.237 * parts + 0.206 * (parts + 0.5) * mb);
    }
    if (p.tn || ((double)parts * p.M * p.N > (double)kGemmTailFloats && parts > 1)) continue;   // tn: the hand-scheduled kernel only
    auto ring = [&](int cfg, int b, double launch, double one, double two, double round, double f0, double f_part, double f_mb) {
      const int64_t T = cdiv(p.M, b) * cdiv(p.N, b) * parts, full = T / (2 * kCus), rest = T % (2 * kCus);
      double t = launch + full * (per * two + round) + (rest ? per * (rest > kCus ? two : one) + round : 0.);
      if (parts > 1) t += f0 + f_part * parts + f_mb * (parts + 0.5) * mb;
      offer(cfg, parts, t);
    };
    ring(25, 128, 2.28, 0.644, 0.684, 2.32, 3.16, 0.316, 0.25);
    ring(26, 64, 4.36, 0.275, 0.387, 0., 1.43, 0.352, 0.281);
  }
  return best;
}

static GemmPick pick_cfg(const GemmParams& p) {
  if (ring_ok(p)) return pick_plain(p);
  // the head's gradient: few target rows against a contraction over the vocabulary (about 1900 rows x 2048 x 32000: 64 tiles,
  // 565 us unsplit, 231 in four parts; 250 rows: 497 us on 128x128 tiles, 75 in sixteen parts)
  if (rd_ok(p) && live_split_ok(p) && !p.grp_off) return {24, 1};
  // narrow outputs stream A once: 128 x 128 tiles measured 2-33 % ahead of 256 x 64 here (58,880 rows; N = 128: 121 against
  // 181 us, where two 64-wide column tiles read A twice); up to 64 columns a 128 x 64 tile loads half the B rows per step
  if (p.N <= 64 && p.M > 128) return {4, 1};
  if (p.N <= 128 && p.M > 128) return {3, 1};
  if (p.M <= 128) return {2, 1};
  if ((int64_t)cdiv(p.M, 256) * cdiv(p.N, 256) * p.splitk < 128) return {3, 1};
  // The hand-scheduled kernel is ahead on every large shape it covers (4096 and 16384 rows of an 8B model: 27 to 30 %)
  if (rd_ok(p)) return {24, 1};
  return {20, 1};                                        // direct-to-LDS tiles when K allows, else staged (0)
}

bool gemm_nn_applies(int mode, int variant, const GemmParams& p) {
  if (mode == AS_FP32) return f32_nn_ok(variant, p) && f32_nn_pays(p);
  if (mode != AS_BF16 || (variant != 0 && variant != 2 && variant != 34) || !mfma_ok(p) || !rd_ok(p)) return false;
  if (p.nn < 1 || p.nn > 3 || p.ncg || p.epi != GEMM_EPI_NONE || p.seg[0].ldb > (1 << 22) || (p.nseg > 1 && p.seg[1].ldb != p.seg[0].ldb)) return false;
  int row = 0;
  for (int i = 0; i + 1 < p.nn; i++) {
    if (((uintptr_t)p.nb[i] % 16) || p.nb_row[i] % 64 || p.nb_row[i] <= row || p.nb_row[i] >= p.seg[0].K) return false;
    row = p.nb_row[i];
  }
  return variant == 34 || pick_cfg(p).cfg == 24;
}

// Splits as pick_plain says.  Under half a chip of workgroups even then (small weight matrices), copies and a kernel of smaller tiles are as fast.
bool gemm_tn_applies(int mode, int variant, const GemmParams& p) {
  if (mode != AS_BF16 || (variant != 0 && variant != 2 && variant != 34) || !p.tn || p.nseg != 1 || !p.c_f32 || p.R) return false;
  if (!mfma_ok(p) || !rd_ok(p) || rd_live(p) || p.ncg || p.nn || p.M % 256 || p.seg[0].lda > (1 << 22) || p.seg[0].ldb > (1 << 22)) return false;
  for (int i = 0; i < p.nrg; i++) if (p.rg_row[i] % 256 || ((uintptr_t)p.rg_C[i] % 16)) return false;
  return p.M / 256 * (p.N / 256) * pick_plain(p).parts >= kCus / 2;
}

// m_dev semantics: the live row count is *m_dev - m_off (clamped to [0, M]).
// variant: 0 pick, 1 plain FMA kernel, 2 MFMA kernel with the default tile choice, 10 + c forces tile configuration c.
int launch_gemm_off(as_ctx* ctx, int mode, int variant, const GemmParams& p_in, int m_off, hipStream_t st) {
  GemmParams p = p_in;
  if (p.M <= 0 || p.N <= 0) return AS_OK;
  if (p.nseg < 1 || p.nseg > 2) return as_fail(ctx, AS_ERR_SHAPE, "gemm: 1 or 2 K segments");
  if (p.splitk < 1) p.splitk = 1;
  if (p.splitk > 1 && !p.partial) return as_fail(ctx, AS_ERR_WORKSPACE, "gemm: split-K needs a partial buffer");
  if (p.accumulate && !p.c_f32) return as_fail(ctx, AS_ERR_SHAPE, "gemm: accumulate needs float output");
  if (p.grp_off && p.splitk > 1) return as_fail(ctx, AS_ERR_SHAPE, "gemm: grouped rows and split-K do not combine");
  if (p.nn && (!(mode == AS_FP32 ? f32_nn_ok(variant, p) : gemm_nn_applies(mode, variant, p)) || (m_off && !p.m_dev))) return as_fail(ctx, AS_ERR_SHAPE, "gemm: B as [K, N] needs the hand-scheduled kernel or the float one");
  if (p.tn) {
    if (!gemm_tn_applies(mode, variant, p) || m_off) return as_fail(ctx, AS_ERR_SHAPE, "gemm: only the hand-scheduled kernel reads A as [K, M]");
    prof_begin(ctx, st, p.k_dev ? AS_K_GEMM_DEVROWS : AS_K_GEMM_RS, p.k_dev ? 0.0 : 2.0 * p.M * p.N * p.seg[0].K);
    const int rc = launch_256(ctx, p, 0, pick_plain(p).parts, st);
    prof_end(ctx, st);
    return rc;
  }
  if (p.grp_n > 0) {
    if (!p.grp_off || p.nseg != 1 || p.m_dev || m_off) return as_fail(ctx, AS_ERR_SHAPE, "gemm: all groups in one launch need a group table and one K segment");
    const int c0 = variant >= 10 ? variant - 10 : pick_cfg(p).cfg;
    if (!(mode == AS_BF16 && variant != 1 && mfma_ok(p) && c0 == 24 && rd_ok(p))) {       // one launch per group
      const size_t esz = mode == AS_BF16 ? 2 : 4;
      for (int e = 0; e < p.grp_n; e++) {
        GemmParams q = p; q.grp_n = 0; q.grp = e; q.grp_rows = p.grp_rows / p.grp_n;
        q.seg[0].B = (const char*)p.seg[0].B + (size_t)e * p.grp_b_stride * esz;
        for (int i = 0; i + 1 < p.nn; i++) q.nb[i] = (const char*)p.nb[i] + (size_t)e * p.grp_b_stride * esz;
        const int rc1 = launch_gemm_off(ctx, mode, variant, q, 0, st);
        if (rc1) return rc1;
      }
      return AS_OK;
    }
  }
  if (p.epi != GEMM_EPI_NONE) {
    if (!gemm_rd_applies(mode, p) || variant == 1 || (variant >= 10 && variant != 34)) return as_fail(ctx, AS_ERR_SHAPE, "gemm: the head epilogues need the hand-scheduled kernel (bf16, N a multiple of 256, K in 64-wide steps)");
    if (p.epi == GEMM_EPI_STATS && !p.epi_part) return as_fail(ctx, AS_ERR_NULL, "gemm: statistics epilogue without a buffer");
    if (p.epi == GEMM_EPI_PROB && (!p.epi_lse || !p.epi_lab || (!p.epi_w && !p.epi_cnt) || p.c_f32 || p.R || (p.ldc % 8))) return as_fail(ctx, AS_ERR_SHAPE, "gemm: probability epilogue needs lse, labels, a row factor and bf16 output");
  }
  if (p.epi == GEMM_EPI_SOFT && (!p.epi_part || !p.epi_zlab || !p.epi_elab || !p.epi_lab || p.c_f32 || p.R || (p.ldc % 8) || p.alpha != 1.f))
    return as_fail(ctx, AS_ERR_SHAPE, "gemm: softmax epilogue needs buffers, label logits and bf16 output");
  if (p.row_scale && (!p.nn || !p.m_dev || p.grp_off || p.epi != GEMM_EPI_NONE || p.c_f32 || p.R || (p.ldc % 8) || p.alpha != 1.f || (!p.epi_w && !p.epi_cnt)))
    return as_fail(ctx, AS_ERR_SHAPE, "gemm: row factors need the product of device-counted rows with a [K, N] matrix and bf16 output");
  if (p.ncg > 0) {
    if (p.ncg > 3 || p.grp_off || p.m_dev || p.splitk > 1 || p.cg_end[p.ncg - 1] != p.N) return as_fail(ctx, AS_ERR_SHAPE, "gemm: column groups need plain rows and ends that add up to N");
    // the hand-scheduled kernel and the ring kernels take all groups at once when every group is whole tiles wide
    const int c = variant >= 10 ? variant - 10 : mode == AS_BF16 && variant != 1 ? pick_cfg(p).cfg : -1;
    const int width = c == 24 ? 256 : c == 25 ? 128 : 64;
    bool fused = mode == AS_BF16 && variant != 1 && mfma_ok(p) && ((c == 24 && rd_ok(p)) || c == 25 || c == 26);
    for (int g = 0; g < p.ncg && fused; g++) fused = p.cg_end[g] % width == 0 && !((uintptr_t)p.cg_B1[g] % 16) && (p.nseg < 2 || !((uintptr_t)p.cg_B2[g] % 16));
    if (mode == AS_FP32) {
      fused = f32_groups_fit(p, f32_pick(p, variant, false).kernel);
    }
    if (!fused) {                                        // one launch per group
      const size_t esz = mode == AS_BF16 ? 2 : 4;
      for (int g = 0, c0 = 0; g < p.ncg; c0 = p.cg_end[g], g++) {
        GemmParams q = p; q.ncg = 0; q.N = p.cg_end[g] - c0;
        q.seg[0].B = p.cg_B1[g];
        if (p.nseg > 1) { q.seg[1].B = p.cg_B2[g]; q.seg[1].A = (const char*)p.seg[1].A + (size_t)p.cg_a2[g] * esz; }
        q.C = (char*)p.C + (size_t)c0 * (p.c_f32 ? 4 : esz);
        if (p.R) q.R = (const char*)p.R + (size_t)c0 * esz;
        const int rc1 = launch_gemm_off(ctx, mode, variant, q, m_off, st);
        if (rc1) return rc1;
      }
      return AS_OK;
    }
  }
  if (variant < 0 || (variant > 2 && variant != 10 && variant != 11 && variant != 12 && variant != 13 && variant != 14 && variant != 30 && variant != 34)) return as_fail(ctx, AS_ERR_SHAPE, "gemm: unknown variant");
  bool use_mfma = (mode == AS_BF16) && variant != 1 && mfma_ok(p);
  if (variant >= 2 && !use_mfma) return as_fail(ctx, AS_ERR_SHAPE, "gemm: MFMA kernel needs bf16 and 8-element alignment");
  int rc = AS_OK;
  double ksum = 0; for (int s = 0; s < p.nseg; s++) ksum += p.seg[s].K;
  const GemmPick pick = variant >= 10 ? GemmPick{variant - 10, 1} : use_mfma ? pick_cfg(p) : GemmPick{0, 1};
  int cfg = pick.cfg;
  if (p.epi != GEMM_EPI_NONE) cfg = 24;                    // only the hand-scheduled kernel has those epilogues (checked above)
  if (cfg >= 20) for (int s = 0; s < p.nseg; s++) if (p.seg[s].K % 64) cfg = 0;     // direct-to-LDS tiles need whole 64-wide K steps
  const bool big = use_mfma && (cfg == 0 || cfg == 20 || cfg == 24);
  const bool rs = use_mfma && cfg == 24 && rd_ok(p) && !rd_live(p) && !m_off;     // live-row launches keep their own timing classes
  prof_begin(ctx, st, rs ? AS_K_GEMM_RS : p.grp_off ? AS_K_GEMM_GROUPED : p.m_dev ? AS_K_GEMM_DEVROWS : !use_mfma ? AS_K_GEMM_FMA : big ? AS_K_GEMM_MFMA_256 : AS_K_GEMM_MFMA_SKINNY,
             p.grp_off ? 2.0 * p.grp_rows * p.N * ksum : p.m_dev ? 0.0 : 2.0 * p.M * p.N * ksum);
  if (use_mfma) {
    switch (cfg) {
      case 1: rc = launch_mfma_cfg<256, 64, 4, 1>(ctx, p, m_off, st); break;
      case 2: rc = launch_mfma_cfg<64, 256, 1, 4>(ctx, p, m_off, st); break;
      case 3: rc = launch_mfma_cfg<128, 128, 2, 2>(ctx, p, m_off, st); break;
      case 4: rc = launch_mfma_cfg<128, 64, 2, 2>(ctx, p, m_off, st); break;
      case 20: rc = launch_dlds_cfg<256, 256, 2, 4>(ctx, p, m_off, st); break;
      case 24: {
        if (!rd_ok(p) || (m_off && !p.m_dev)) { rc = launch_dlds_cfg<256, 256, 2, 4>(ctx, p, m_off, st); break; }
        rc = launch_256(ctx, p, m_off, pick.parts, st);
        break; }
      case 25: rc = launch_ring_cfg<128, 128, 2>(ctx, p, pick.parts, st); break;
      case 26: rc = launch_ring_cfg<64, 64, 4>(ctx, p, pick.parts, st); break;
      default: rc = launch_mfma_cfg<256, 256, 2, 4>(ctx, p, m_off, st); break;
    }
  } else {
    const int bt = fma_tile(p);
    const bool big = bt == 64;
    dim3 grid((unsigned)cdiv(p.N, bt), (unsigned)cdiv(p.M, bt), (unsigned)p.splitk);
    if (mode == AS_FP32) {
      const int k = f32_pick(p, variant, p.nn > 0).kernel, b = kF32Tile[k];
      const dim3 g((unsigned)cdiv(p.N, b), (unsigned)cdiv(p.M, b), (unsigned)p.splitk);
      auto run = [&](auto nn) {
        constexpr bool NN = decltype(nn)::value;
        const int chunks = (int)(cdiv(p.seg[0].K, 16) + (p.nseg > 1 ? cdiv(p.seg[1].K, 16) : 0)) / p.splitk;
        if (k == F32_32) gemm_f32_kernel<2, NN, 4><<<g, 256, 0, st>>>(p, m_off);
        else if (chunks <= 16) gemm_f32_kernel<1, NN, 4><<<g, 256, 0, st>>>(p, m_off);
        else if (chunks <= 32) gemm_f32_kernel<1, NN, 8><<<g, 512, 0, st>>>(p, m_off);
        else gemm_f32_kernel<1, NN, 16><<<g, 1024, 0, st>>>(p, m_off);
      };
      if (p.nn) run(std::true_type{});
      else if (k <= F32_32) run(std::false_type{});
      else if (k == FMA_32) gemm_fma_kernel<float, 32, 64><<<g, 256, 0, st>>>(p, m_off);
      else gemm_fma_kernel<float, 64, 32><<<g, 256, 0, st>>>(p, m_off);
    } else if (big) gemm_fma_kernel<bf16_t, 64, 32><<<grid, 256, 0, st>>>(p, m_off);
    else gemm_fma_kernel<bf16_t, 32, 64><<<grid, 256, 0, st>>>(p, m_off);
    AS_LAUNCH_CHECK(ctx);
  }
  prof_end(ctx, st);
  if (rc) return rc;
  if (p.splitk > 1) {
    if (!p.c_f32) return as_fail(ctx, AS_ERR_SHAPE, "gemm: split-K writes float output");
    rc = launch_splitk_reduce(ctx, p.partial, p.splitk, (int64_t)p.M * p.N, p.N, p.alpha, (float*)p.C, p.ldc, st);
  }
  return rc;
}

// Up to three products of one shape (p.nbat; one segment each, plain rows, no residual).  Side by side where the kernel that would take them one
// by one has that: few tokens' launches are mostly latency, many tokens' end on partial rounds.  626 tokens on two 1B layers: 1.434 -> 1.394 ms,
// 478 on two layers of width 128 in float 289 -> 276 us; level on 13,000 tokens of the 8B model.
int launch_gemm_batch(as_ctx* ctx, int mode, const GemmParams& p, hipStream_t st) {
  if (p.M <= 0 || p.N <= 0 || p.nbat < 1) return AS_OK;
  auto one = [&](int i) {
    GemmParams q = p;
    q.nbat = 0; q.seg[0].A = p.bt_A[i]; q.seg[0].B = p.bt_B[i]; q.seg[0].K = p.bt_K[i]; q.seg[0].ldb = p.bt_K[i]; q.C = p.bt_C[i];
    return q;
  };
  int kernel = -1, parts = 1, kmax = 0;
  double flops = 0, ksum = 0;
  for (int i = 0; i < p.nbat; i++) ksum += p.bt_K[i];
  bool same = p.nbat > 1;
  for (int i = 0; i < p.nbat && same; i++) {
    const GemmParams q = one(i);
    kmax = std::max(kmax, q.seg[0].K); flops += 2.0 * q.M * q.N * q.seg[0].K;
    int k;
    if (mode == AS_FP32) { k = f32_pick(q, 0, false).kernel; same = k <= F32_32; }
    else {
      GemmParams all = q;                                  // the tiles of all products
      all.M = (int)std::min<double>(q.M * (ksum / q.seg[0].K), 1 << 30);
      const GemmPick c = mfma_ok(q) && ring_ok(q) ? pick_plain(i == 0 ? all : q) : GemmPick{0, 1}; k = c.cfg; same = k == 25 || k == 26; if (i == 0) parts = c.parts;
    }
    if (i == 0) kernel = k;                              // the first product is the one of the longest contraction: its kernel and parts
  }
  if (!same) {
    for (int i = 0; i < p.nbat; i++) { const int rc = launch_gemm_off(ctx, mode, 0, one(i), 0, st); if (rc) return rc; }
    return AS_OK;
  }
  while (parts > 1 && (size_t)parts * p.nbat * p.M * p.N > kGemmTailFloats) parts--;
  int rc = AS_OK;
  prof_begin(ctx, st, mode == AS_FP32 ? AS_K_GEMM_FMA : AS_K_GEMM_MFMA_SKINNY, flops);
  if (mode == AS_FP32) {
    const int b = kF32Tile[kernel], chunks = (int)cdiv(kmax, 16);
    const dim3 g((unsigned)cdiv(p.N, b), (unsigned)cdiv(p.M, b), (unsigned)p.nbat);
    if (kernel == F32_32) gemm_f32_kernel<2, false, 4><<<g, 256, 0, st>>>(p, 0);
    else if (chunks <= 16) gemm_f32_kernel<1, false, 4><<<g, 256, 0, st>>>(p, 0);
    else if (chunks <= 32) gemm_f32_kernel<1, false, 8><<<g, 512, 0, st>>>(p, 0);
    else gemm_f32_kernel<1, false, 16><<<g, 1024, 0, st>>>(p, 0);
    AS_LAUNCH_CHECK(ctx);
  } else rc = kernel == 25 ? launch_ring_cfg<128, 128, 2>(ctx, p, parts, st) : launch_ring_cfg<64, 64, 4>(ctx, p, parts, st);
  prof_end(ctx, st);
  return rc;
}

int launch_gemm(as_ctx* ctx, int mode, int variant, const GemmParams& p, hipStream_t st) {
  return launch_gemm_off(ctx, mode, variant, p, 0, st);
}

// ------------------------------------------------- matrix-core peak probe
// Register-resident MFMA loop: no memory traffic at all, eight independent accumulators per
// wavefront, two wavefronts per SIMD.  What this sustains is the ceiling any GEMM on the chip can
// reach at the clocks the part holds under matrix load.
__global__ __launch_bounds__(512) void mfma_peak_kernel(int iters, float* sink) {
  bf16x8 a, b;
#pragma unroll
  for (int j = 0; j < 8; j++) { a[j] = (bf16_t)(0.001f * (threadIdx.x + j)); b[j] = (bf16_t)(0.002f * (threadIdx.x - j)); }
  f32x16 acc[8];
#pragma unroll
  for (int i = 0; i < 8; i++)
#pragma unroll
    for (int e = 0; e < 16; e++) acc[i][e] = 0.f;
  for (int it = 0; it < iters; it++) {
#pragma unroll
    for (int i = 0; i < 8; i++) acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc[i], 0, 0, 0);
  }
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < 8; i++) s += acc[i][0] + acc[i][15];
  if (s == 123.456f) sink[0] = s;          // never true; keeps the loop alive
}

int launch_mfma_peak(as_ctx* ctx, int iters, int blocks, float* sink, hipStream_t st) {
  mfma_peak_kernel<<<blocks, 512, 0, st>>>(iters, sink);
  AS_LAUNCH_CHECK(ctx);
  return AS_OK;
}

// ------------------------------------------------ global -> LDS feed probe
// Every wavefront keeps K 1-KB direct-to-LDS loads in flight, waits for them, and repeats, walking a
// region of `span` bytes (power of two).  With a span that fits L2 this measures the L2 -> LDS path,
// with a larger one the MALL / HBM mix.  A 256x256x64 bf16 GEMM tile step needs 64 KB per CU.
template <int K>
__global__ __launch_bounds__(512) void feed_probe_kernel(const char* src, size_t span_mask, int iters, int* sink) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const size_t base = (size_t)blockIdx.x * 7919u * 65536u;
  for (int it = 0; it < iters; it++) {
#pragma unroll
    for (int i = 0; i < K; i++) {
      const size_t off = (base + ((size_t)it * 8 * K + wave * K + i) * 1024 + lane * 16) & span_mask;
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src + off),
                                       (__attribute__((address_space(3))) void*)(smem + (wave * K + i) * 1024), 16, 0, 0);
    }
    __builtin_amdgcn_s_waitcnt(0x0f70);
    __builtin_amdgcn_s_barrier();
  }
  if (iters < 0 && smem[threadIdx.x] == 123) sink[0] = 1;
}

int launch_feed_probe(as_ctx* ctx, int k, const void* buf, size_t span, int iters, int blocks, int* sink, hipStream_t st) {
  const size_t mask = (span - 1) & ~(size_t)15;
#define FEED(K) { AS_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(feed_probe_kernel<K>), hipFuncAttributeMaxDynamicSharedMemorySize, 8 * K * 1024)); \
                  feed_probe_kernel<K><<<blocks, 512, 8 * K * 1024, st>>>((const char*)buf, mask, iters, sink); }
  switch (k) { case 1: FEED(1) break; case 2: FEED(2) break; case 4: FEED(4) break; case 8: FEED(8) break;
               default: return as_fail(ctx, AS_ERR_SHAPE, "feed probe: loads in flight per wave must be 1, 2, 4 or 8"); }
#undef FEED
  AS_LAUNCH_CHECK(ctx);
  return AS_OK;
}
