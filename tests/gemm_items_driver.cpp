// Items of the persistent 256x256 GEMM as csrc/gemm_items.h deals them out, for tests/test_gemm_items.py.  Reads launches, one per line, as
// key=value pairs; prints the launch and, per workgroup, every item with its bases for each of the four waves.
#include "gemm_items.h"
#include <cstdio>
#include <cstring>
#include <iostream>
#include <map>
#include <sstream>
#include <string>

typedef std::map<std::string, long long> Args;

template <int LIVE, int LAYOUT>
static void launch(const GemmParams& p, Args& a) {
  const RdLaunch g = rd_launch<LIVE, LAYOUT>(p, (int)a["m_off"], (int)a["tiles_m"], (int)a["tiles_n"]);
  printf("launch %d %d %d %d %d %d %d %d %d\n", g.tiles_m, g.tiles_n, g.tiles, g.first_split, g.parts, g.items, g.nt0, g.nt, p.tail_first);
  const int grid = (int)a["grid"];
  for (int wg = 0; wg < grid && wg < g.items; wg++)
    for (int item = wg; item < g.items; item += grid) {
      const RdItem w = rd_item<LIVE, LAYOUT>(p, g, item, 0);
      const RdNext n = rd_next<LIVE, LAYOUT>(p, g, w, item, grid, 0);
      printf("item %d %d %d %d %d %d %d %d %d %d %d %d %d %d %d", wg, item, w.row0, w.col0, w.row_lo, w.row_hi, w.pid, w.kpart, w.nt0, w.nt, w.n1, w.n2, (int)w.two, (int)n.chain, n.lim);
      for (int wave = 0; wave < 4; wave++) {
        const RdItem v = rd_item<LIVE, LAYOUT>(p, g, item, wave);
        const RdNext m = rd_next<LIVE, LAYOUT>(p, g, v, item, grid, wave);
        const uint64_t at[9] = {v.a0, v.a1, v.b0, v.b1, v.b2, v.b3, v.bf, m.an, m.bn};
        for (uint64_t x : at) printf(" %lld", (long long)x);
      }
      printf("\n");
    }
}

// the split of a last round for every pair of segments up to `most` steps and every rest of up to half a round
static void rules(int most) {
  long long split = 0, at_segment_1 = 0, bad = 0;
  for (int n0 = 1; n0 <= most; n0++)
    for (int n1 = 0; n1 <= most; n1++)
      for (int rest = 1; rest < kCus; rest++) {
        GemmParams p; memset(&p, 0, sizeof p);
        float scratch;
        p.tail_part = &scratch; p.nseg = n1 ? 2 : 1; p.seg[0].K = n0 * kStep; p.seg[1].K = n1 * kStep;
        const int nt = n0 + n1, T = kCus + rest;
        const bool want = nt >= 32 && rest <= kCus / 2 && nt / 2 <= n0;
        if (tail_splits(p, T) != want) { bad++; continue; }
        if (!want) continue;
        const int parts = tail_parts(p, rest);
        split++;
        // room in the scratch and in the round; whole steps; the start of the last part
        if (parts < 2 || parts > kLiveParts || parts * rest > kCus || nt / parts < 8) bad++;
        const int last = (int)((long long)nt * (parts - 1) / parts);
        if (parts > 2 ? last >= n0 : last > n0) bad++;
        at_segment_1 += last == n0;
      }
  printf("rules %lld %lld %lld\n", split, at_segment_1, bad);
}

int main() {
  std::string line;
  while (std::getline(std::cin, line)) {
    Args a;
    std::istringstream is(line);
    std::string tok;
    while (is >> tok) { const size_t e = tok.find('='); a[tok.substr(0, e)] = std::stoll(tok.substr(e + 1)); }
    if (a.count("rules")) { rules((int)a["rules"]); continue; }
    GemmParams p; memset(&p, 0, sizeof p);
    float scratch;
    int off[16], m_dev, k_dev;
    p.M = (int)a["M"]; p.N = (int)a["N"]; p.nseg = a["K2"] ? 2 : 1;
    p.seg[0] = {(const void*)a["A"], (const void*)a["B0"], a["lda"], a["ldb"], (int)a["K1"]};
    p.seg[1] = {(const void*)a["A2"], (const void*)a["B2"], a["lda2"], a["ldb2"], (int)a["K2"]};
    p.nn = (int)a["nn"]; p.nb[0] = (const void*)a["B1"]; p.nb[1] = (const void*)a["B3"]; p.nb_row[0] = (int)a["nb0"]; p.nb_row[1] = (int)a["nb1"];
    p.ncg = (int)a["ncg"];
    for (int i = 0; i < p.ncg; i++) {
      const std::string n = std::to_string(i);
      p.cg_end[i] = (int)a["cg_end" + n]; p.cg_B1[i] = (const void*)a["cg_B" + n]; p.cg_B2[i] = (const void*)a["cg_C" + n]; p.cg_a2[i] = (int)a["cg_a" + n];
    }
    p.rows_cap = (int)a["rows_cap"]; p.grp_b_stride = a["grp_b_stride"]; p.grp_n = (int)a["grp_n"]; p.grp = (int)a["grp"];
    if (a.count("off0")) { for (int i = 0; i < 16; i++) off[i] = (int)a["off" + std::to_string(i)]; p.grp_off = off; }
    if (a.count("m_dev")) { m_dev = (int)a["m_dev"]; p.m_dev = &m_dev; }
    if (a.count("k_dev")) { k_dev = (int)a["k_dev"]; p.k_dev = &k_dev; }
    p.k_off = (int)a["k_off"]; p.tn = a["layout"] == RD_TN;
    if (a["scratch"]) p.tail_part = &scratch;
    p.tail_first = a.count("tail_first") ? (int)a["tail_first"] : -1; p.tail_parts = a.count("tail_parts") ? (int)a["tail_parts"] : 2;
    const int live = (int)a["live"], layout = (int)a["layout"];
    // as the launcher: the rule of the split last round
    if (a["tail"] && tail_splits(p, (int)(a["tiles_m"] * a["tiles_n"]))) { const int T = (int)(a["tiles_m"] * a["tiles_n"]); p.tail_first = T / kCus * kCus; p.tail_parts = tail_parts(p, T % kCus); }
    if (layout == RD_TN) launch<0, RD_TN>(p, a);
    else if (layout == RD_NN) { if (live == 0) launch<0, RD_NN>(p, a); else if (live == 1) launch<1, RD_NN>(p, a); else launch<2, RD_NN>(p, a); }
    else if (live == 0) launch<0, RD_NT>(p, a);
    else if (live == 1) launch<1, RD_NT>(p, a);
    else launch<2, RD_NT>(p, a);
    printf("end\n");
  }
  return 0;
}
