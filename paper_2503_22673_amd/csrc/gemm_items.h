// What a product is (GemmParams), and how the persistent 256 x 256 kernel deals one out: which tile, or which part of a tile's
// contraction, a workgroup takes in which order, and from where its loads read.  Plain integer code without a device header: gemm.hip
// compiles it for the device and for its launcher, the tests compile it for the host and run the generated loops over the items of a launch.
#pragma once
#include <cstdint>

#ifdef __HIPCC__
#define AS_HD __host__ __device__ __forceinline__
#else
#define AS_HD inline
#endif

// C[M,N] = alpha * sum_s A_s[M,K_s] B_s[N,K_s]^T (+ R), optional split over K.
struct GemmSeg { const void* A; const void* B; int64_t lda, ldb; int K; };
struct GemmParams {
  GemmSeg seg[2]; int nseg;
  int M, N;
  const int* m_dev;        // if set, the row count is read from the device (<= M)
  void* C; int64_t ldc; int c_f32;
  float alpha;
  const void* R; int64_t ldr;
  int accumulate;          // C += result (float output only)
  int splitk; float* partial;   // splitk > 1: partial [splitk, M, N] float, reduced afterwards
  // grouped rows (mixture of experts): with grp_off set, the product covers rows
  // [grp_off[grp], grp_off[grp+1]) of A, R and C (device-side table), at most M of them
  const int* grp_off; int grp;
  double grp_rows;            // expected live rows of the launch (timing records only)
  // grp_n > 0: ALL groups 0 .. grp_n - 1 in one launch (grp is ignored); group e multiplies with the matrix that
  // starts grp_b_stride elements after that of group e - 1 (B of segment 0; one segment only)
  int grp_n; int64_t grp_b_stride;
  // rows that every row operand (A of each segment, R, C) really has allocated, or 0: lets a kernel that works in
  // whole 256-row tiles run over the ragged last tile too (rows past M are computed from whatever is there and
  // written to rows past M of C; no row of the result depends on another row)
  int rows_cap;
  // Column groups: several weight matrices whose outputs sit side by side in C (q | k | v, gate | up) as ONE launch: fewer,
  // larger grids (every launch ends on a partial round of tiles) and the shared row panel of A is read once per tile row.
  // Group g covers columns [cg_end[g-1], cg_end[g]) (multiples of 256); its rows of B come from cg_B1[g] (segment 0) and
  // cg_B2[g] (segment 1), both indexed from the group's first column, and segment 1 reads A at column offset cg_a2[g]
  // (each projection has its own adapter activations).  ncg == 0: seg[].B as usual.
  int ncg; int cg_end[3]; const void* cg_B1[3]; const void* cg_B2[3]; int cg_a2[3];
  // Vocabulary head without stored logits (hand-scheduled kernel only; rows and row arrays are those of A):
  //  epi == GEMM_EPI_STATS: nothing is written to C; for every row and every 128-column block of the result the maximum and
  //    the sum of exp(value - maximum) go to epi_part[(row * (N / 128) + block) * 2 + {0, 1}];
  //  epi == GEMM_EPI_PROB:  C = w_row * (exp(value - epi_lse[row]) - [column == epi_lab[row]]), w_row = epi_w[row] when
  //    given, else 1 / *epi_cnt: the gradient of the masked loss with respect to the logits, straight from the accumulators.
  //  epi == GEMM_EPI_SOFT:  C = exp(value) / 2^R, R a whole number per row and 128-column block: the row's label logit epi_zlab in powers of
  //    two, more only where a value lies 2^40 above it; the statistics go to epi_part as above, the label's own element to
  //    epi_elab[row] as a float.  Up to whole powers of two and the factor w_row / (sum over the row) this is the gradient, before the sum is known.
  // row_scale (with epi_w or epi_cnt; the product of device-counted rows with a [K, N] matrix only): row r of the result times
  //    row_scale[r] * w_row.
  // Split tiles (hand-scheduled kernel, plain rows): with tail_first >= 0 the tiles tail_first .. of the launch are each
  // computed by tail_parts workgroups, one per part of the contraction, as float partials in tail_part
  // [tile - tail_first][part][256 x 256]; a second small launch adds the parts in order and applies the epilogue.
  // Set by the launcher, which finds room for kGemmTailFloats floats at tail_part.
  int tail_first, tail_parts; float* tail_part;
  // nn > 0: B of both segments is [K, N], rows of N elements with ONE row stride (seg[0].ldb == seg[1].ldb); segment 0's rows are those of
  // nn <= 3 matrices below one another: seg[0].B, and from row nb_row[i] (bf16: a multiple of 64) on nb[i].  Not all kernels: ask
  // gemm_nn_applies first.
  int nn; const void* nb[2]; int nb_row[2];
  // tn: A of the one segment is [K, M] and B [K, N] (hand-scheduled kernel only: gemm_tn_applies), float result.  Its rows may be those of
  // several matrices: from row rg_row[i] (a multiple of 256) on they go to rg_C[i], all with row stride ldc.  k_dev: the
  // contraction ends with row *k_dev - k_off (rows up to the next multiple of 64 must be zero in both operands).
  int tn; const int* k_dev; int k_off; int nrg; void* rg_C[2]; int rg_row[2];
  // nbat > 0: up to three products of one shape M x N side by side in a launch (the adapters' du of q, k and v): product i has A bt_A[i] (row stride
  // seg[0].lda), B bt_B[i] [N, bt_K[i]] (row stride bt_K[i]), result bt_C[i] (row stride ldc).  launch_gemm_batch only.
  int nbat; const void* bt_A[3]; const void* bt_B[3]; void* bt_C[3]; int bt_K[3];
  int epi; const float* epi_lse; const int32_t* epi_lab; const float* epi_w; const int32_t* epi_cnt; float* epi_part;
  const float* epi_zlab; float* epi_elab; const float* row_scale;
};
enum { GEMM_EPI_NONE = 0, GEMM_EPI_STATS = 1, GEMM_EPI_PROB = 2, GEMM_EPI_SOFT = 3, GEMM_EPI_ROWS = 4 };   // ROWS: what row_scale selects inside the kernel

// ------------------------------------------------------------------ shape rules of the 256 x 256 kernel
constexpr int kTile = 256, kStep = 64;                   // rows and columns of a tile; contraction of a step
constexpr int kCus = 256;                                // workgroups of a round: one per CU
constexpr int kLiveParts = 16;                           // parts of a tile's contraction at most
enum { RD_NT = 0, RD_NN = 1, RD_TN = 2 };                // A [M, K], B [N, K]; B [K, N]; A [K, M] and B [K, N]

AS_HD int as_min(int a, int b) { return a < b ? a : b; }
AS_HD int as_max(int a, int b) { return a > b ? a : b; }

AS_HD int k_steps(const GemmParams& p) { return p.seg[0].K / kStep + (p.nseg > 1 ? p.seg[1].K / kStep : 0); }

// The tiles of a last partial round are split when that round would leave at least half of the CUs idle, the launch
// has full rounds before it and the contraction is long enough to be worth a second small launch: a launch of 3696 tiles
// on 256 CUs then ends after 14.5 rounds instead of 15.  Two parts begin where segment 1 does at the latest.
AS_HD bool tail_splits(const GemmParams& p, int T) {
  const int rest = T % kCus, nt = k_steps(p);
  return p.tail_part && p.epi == GEMM_EPI_NONE && T > kCus && rest > 0 && rest <= kCus / 2 && nt >= 32 && nt / 2 <= p.seg[0].K / kStep;
}
// As many parts as fill the round, of at least eight steps each; more than two only if the last one starts inside segment 0.  24,710
// tokens on matrices of 2048 x 8192 leave eight tiles behind three rounds: in two parts they took half a tile's time, in sixteen a
// sixteenth (step of two 1B layers 16.64 -> 16.46 ms; 13,429 tokens on an 8B model, 80 tiles in three parts: 29.8 -> 29.6).
AS_HD int tail_parts(const GemmParams& p, int rest) {
  const int nt = k_steps(p), nt0 = p.seg[0].K / kStep;
  int parts = as_min(as_min(kLiveParts, kCus / rest), nt / 8);
  while (parts > 2 && nt - (nt + parts - 1) / parts >= nt0) parts--;
  return as_max(parts, 2);
}

// Rows counted on the device, with scratch for partial sums: when the last round of tiles is at most half full, the contraction of each
// of its tiles is split over as many workgroups as fit the round, up to kLiveParts.  Host code cannot know the count, so both launches
// work the split out from it.  Experts of 8x7B widths over 8192 tokens in their two slots each, 4.1 rounds of tiles: down 1652 -> 1410 us,
// input gradients of gate and up 2736 -> 2377, and 15 each for the sum of the parts (they had unsplit last rounds).
struct LiveSplit { int first, parts; };                  // tiles from `first` on, in that many parts
AS_HD LiveSplit live_split(const GemmParams& p, int tiles) {
  const int rest = tiles % kCus;
  if (!p.tail_part || rest == 0 || rest > kCus / 2) return {tiles, 1};
  return {tiles - rest, as_min(kLiveParts, kCus / rest)};
}
// row tiles that the groups' rows fill, one group after the other
AS_HD int group_row_tiles(const GemmParams& p) {
  int total = 0;
  for (int e = 0; e < p.grp_n; e++) total += (p.grp_off[e + 1] - p.grp_off[e] + kTile - 1) / kTile;
  return total;
}
// Live row count of a launch and, for grouped rows, the first row of the group (rb): rows of A, R
// and C are then rb + (0 .. M-1).  mmax is the largest row index a clamped load may touch.
AS_HD int gemm_rows(const GemmParams& p, int m_off, int& rb, int& mmax) {
  int M = p.m_dev ? as_min(p.M, *p.m_dev - m_off) : p.M;
  rb = 0; mmax = p.M - 1;
  if (p.grp_off) {
    rb = p.grp_off[p.grp];
    M = as_min(M, p.grp_off[p.grp + 1] - rb);
    mmax = as_max(M, 1) - 1;
  }
  return M;
}

// ------------------------------------------------------------------ items
// A launch as its workgroups see it: the tiles there are, which of them are split, and how many items of work that makes.
// LIVE = 0: plain rows in whole row tiles, or a ragged last one whose spare rows the operands have.
// LIVE = 2: plain rows whose number is no multiple of 256; the last row tile is moved up to end with the last row and writes
// only the rows that are its own.
// LIVE = 1: the row count is a device-side value and / or the rows are those of groups (experts).  Tiles past the live
// rows do not exist; a tile still computes 256 rows, moved up if need be so that they lie inside the rows the operands
// are known to have (M for a plain row count, rows_cap for grouped rows), and writes the rows that are its own and live.
// SPLIT = false: no tile is split (the head's epilogues).
struct RdLaunch { int tiles_m, tiles_n, tiles, first_split, parts, items, rb, mlive, nt0, nt; };
template <int LIVE, int LAYOUT, bool SPLIT = true>
AS_HD RdLaunch rd_launch(const GemmParams& p, int m_off, int tiles_m, int tiles_n) {
  RdLaunch g;
  g.rb = 0; g.mlive = p.M;
  if (LIVE == 1) {
    if (p.grp_n > 0) tiles_m = as_min(tiles_m, group_row_tiles(p));
    else {
      int mmax;
      g.mlive = gemm_rows(p, m_off, g.rb, mmax);
      tiles_m = as_min(tiles_m, (as_max(g.mlive, 0) + kTile - 1) / kTile);
    }
  }
  g.tiles_m = tiles_m; g.tiles_n = tiles_n; g.tiles = tiles_m * tiles_n;
  g.parts = p.tail_parts; g.first_split = g.tiles;         // tiles from first_split on are split into parts
  if (SPLIT && LIVE == 1) { const LiveSplit v = live_split(p, g.tiles); g.first_split = v.first; g.parts = v.parts; }
  if (SPLIT && LIVE != 1 && p.tail_first >= 0) g.first_split = p.tail_first;
  g.items = g.first_split + (g.tiles - g.first_split) * g.parts;
  g.nt0 = p.seg[0].K / kStep; g.nt = k_steps(p);
  if (LAYOUT == RD_TN && p.k_dev) g.nt0 = g.nt = as_min(g.nt, (as_max(*p.k_dev - p.k_off, 0) + kStep - 1) / kStep);
  return g;
}

// One tile, or one part of a split tile's contraction.  Pointers are those of the asking wave.
struct RdItem {
  int row0, col0, row_lo, row_hi, pid, kpart, nt0, nt, n1, n2;
  uint64_t a0, a1, b0, b1, b2, b3;                         // bases of both segments (NN: of the matrices below one another), for a step counted from this item's first
  uint64_t bf; bool two;                                   // base of B in the first step; whether the second step has the same bases
};
template <int LIVE, int LAYOUT>
AS_HD RdItem rd_item(const GemmParams& p, const RdLaunch& g, int item, int wave) {
  const GemmSeg s0 = p.seg[0], s1 = p.nseg > 1 ? p.seg[1] : p.seg[0];
  RdItem w;
  w.kpart = -1; w.pid = item;
  if (item >= g.first_split) { const int i = item - g.first_split; w.kpart = i % g.parts; w.pid = g.first_split + i / g.parts; }
  const int q8 = g.tiles / 8, rem = g.tiles % 8, xcd = w.pid % 8, loc = w.pid / 8;
  const int logical = xcd * q8 + as_min(xcd, rem) + loc;
  constexpr int GROUP = 4;                                 // the 32 workgroups of an XCD cover 4 row tiles x 8 column tiles at a time
  const int in_group = GROUP * g.tiles_n, grp = logical / in_group, first_m = grp * GROUP;
  const int gsize = as_min(g.tiles_m - first_m, GROUP);
  int tile_m = first_m + (logical % in_group) % gsize;
  const int tile_n = (logical % in_group) / gsize;
  int b_group = 0, rb = g.rb, mlive = g.mlive;
  if (LIVE == 1 && p.grp_n > 0) {                          // which group this row tile belongs to, and which of its tiles it is
    int e = 0, rows_e = p.grp_off[1] - p.grp_off[0], nt_e = (rows_e + kTile - 1) / kTile;
    while (tile_m >= nt_e && e + 1 < p.grp_n) {
      tile_m -= nt_e; e++;
      rows_e = p.grp_off[e + 1] - p.grp_off[e]; nt_e = (rows_e + kTile - 1) / kTile;
    }
    rb = p.grp_off[e]; mlive = rows_e; b_group = e;
  }
  w.row_lo = rb + tile_m * kTile; w.row_hi = rb + mlive;
  w.row0 = LIVE ? as_min(w.row_lo, (LIVE == 1 && p.grp_off ? p.rows_cap : p.M) - kTile) : tile_m * kTile;
  w.col0 = tile_n * kTile;
  w.nt0 = g.nt0; w.nt = g.nt;
  int64_t lo = 0;
  if (w.kpart >= 0) {                                      // steps [lo, hi) of the contraction; nt0 <= 0: all of them are segment 1's
    lo = (int64_t)g.nt * w.kpart / g.parts;
    const int hi = (int)((int64_t)g.nt * (w.kpart + 1) / g.parts);
    w.nt0 = as_min(g.nt0, hi) - (int)lo; w.nt = hi - (int)lo;
  }
  // Segment 0's bases begin with this part's first step.  A part without steps of segment 0 keeps those of its first one: no product
  // uses them, but loads past the item's end that nobody reads do (rd_next), and those have to stay inside the operands too.
  const int64_t k_skip = lo < g.nt0 || LAYOUT == RD_TN ? lo * kStep : 0;
  const uint64_t b_at = (uint64_t)s0.B + (uint64_t)(2 * ((int64_t)b_group * p.grp_b_stride));
  w.n1 = w.n2 = w.nt0; w.b2 = w.b3 = 0; w.two = w.nt0 >= 2;
  if (LAYOUT == RD_TN) {
    w.a0 = w.a1 = (uint64_t)s0.A + (uint64_t)(2 * ((k_skip + wave * 16) * s0.lda + w.row0));
    w.b0 = w.b1 = b_at + (uint64_t)(2 * ((k_skip + wave * 16) * s0.ldb + w.col0));
    w.bf = w.b0;
    return w;
  }
  int colg = w.col0, a2off = 0;
  uint64_t b0p = b_at, b1p = (uint64_t)s1.B;
  if (p.ncg > 0) {                                         // which weight matrix this column tile belongs to
    int c = 0;
    while (c + 1 < p.ncg && w.col0 >= p.cg_end[c]) c++;
    colg = w.col0 - (c ? p.cg_end[c - 1] : 0);
    b0p = (uint64_t)p.cg_B1[c]; b1p = (uint64_t)(p.nseg > 1 ? p.cg_B2[c] : p.cg_B1[c]); a2off = p.nseg > 1 ? p.cg_a2[c] : 0;
  }
  w.a0 = (uint64_t)s0.A + (uint64_t)(2 * ((int64_t)(w.row0 + wave * 64) * s0.lda + k_skip));
  w.a1 = (uint64_t)s1.A + (uint64_t)(2 * (a2off + (int64_t)(w.row0 + wave * 64) * s1.lda - (int64_t)w.nt0 * kStep));
  if (LAYOUT == RD_NN) {
    const int64_t ldb = s0.ldb, row_w = (int64_t)(wave * 16) * ldb + w.col0, grp_b = (int64_t)b_group * p.grp_b_stride;
    // bases of the matrices, each minus its first row: step t of this item reads rows 64 t .. of it
    w.b0 = (uint64_t)s0.B + (uint64_t)(2 * (grp_b + row_w + k_skip * ldb));
    w.b2 = (uint64_t)p.nb[0] + (uint64_t)(2 * (grp_b + row_w + (k_skip - p.nb_row[0]) * ldb));
    w.b3 = (uint64_t)p.nb[1] + (uint64_t)(2 * (grp_b + row_w + (k_skip - p.nb_row[1]) * ldb));
    w.b1 = (uint64_t)s1.B + (uint64_t)(2 * (row_w - (int64_t)w.nt0 * kStep * ldb));
    if (w.nt0 > 0) {
      if (p.nn > 1) w.n1 = (int)(p.nb_row[0] / kStep - lo);
      if (p.nn > 2) w.n2 = (int)(p.nb_row[1] / kStep - lo);
    }
  } else {
    w.b0 = b0p + (uint64_t)(2 * ((int64_t)(colg + wave * 64) * s0.ldb + k_skip));
    w.b1 = b1p + (uint64_t)(2 * ((int64_t)(colg + wave * 64) * s1.ldb - (int64_t)w.nt0 * kStep));
  }
  const int end = w.n1 > 0 ? w.n1 : w.n2 > 0 ? w.n2 : w.nt0;
  w.bf = w.n1 > 0 || w.nt0 <= 0 ? w.b0 : w.n2 > 0 ? w.b2 : w.b3; w.two = w.two && end >= 2;
  return w;
}

// Where the loads behind an item's last step go: the first two steps of the workgroup's next item, if both have the same bases; else this
// item's own first steps (segment 0's) again, which nobody reads.  an, bn: bases for a step counted on from this item's first; lim: the
// step at which they stop moving.
struct RdNext { bool chain; uint64_t an, bn; int lim; };
template <int LIVE, int LAYOUT>
AS_HD RdNext rd_next(const GemmParams& p, const RdLaunch& g, const RdItem& w, int item, int grid, int wave) {
  RdNext n;
  n.chain = false; n.an = w.a0; n.bn = w.bf;
  if (item + grid < g.items) {
    const RdItem nx = rd_item<LIVE, LAYOUT>(p, g, item + grid, wave);
    if (nx.two) { n.chain = true; n.an = nx.a0; n.bn = nx.bf; }
  }
  const int64_t step_a = LAYOUT == RD_TN ? 128 * p.seg[0].lda : 2 * kStep, step_b = LAYOUT != RD_NT ? 128 * p.seg[0].ldb : 2 * kStep;
  n.an -= (uint64_t)(w.nt * step_a); n.bn -= (uint64_t)(w.nt * step_b);
  n.lim = w.nt + (n.chain || w.two ? 1 : 0);
  return n;
}
