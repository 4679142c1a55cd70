// Host replay of the many-row GEMM's index arithmetic (gemm.h, plan_tiles): run by test_abi.py, no device access.
//
// For a matrix of N x K and M rows: every (column tile, row block, k-step) of the product is computed by exactly one
// workgroup; every weight tile is read where the streaming plan stores it; every workgroup's K segments are the
// matrix's own; places of running and partial sums are distinct and inside part_bytes; counters stay inside max_split.
#include <cstdio>
#include <cstdlib>
#include <set>
#include <vector>

#include "../paper_2608_14787_amd/csrc/gemm.h"

using namespace sdd;

#define CHECK(c)                                                                                             \
  do {                                                                                                       \
    if (!(c)) {                                                                                              \
      std::printf("FAILED %s: N %d K %d ng %d pairs %d M %d part %zu (wc %d rtw %d split %d per %d)\n", #c, N, K, ng, \
                  (int)pairs, M, part, p.wc, p.rtw, p.ksplit, p.per);                                        \
      std::exit(1);                                                                                          \
    }                                                                                                        \
  } while (0)

static int modes[4];  // whole, chain, compact chain, split

static void replay(int N, int K, int ng, bool pairs, int M, size_t part, int64_t max_split) {
  const int n_cu = 256;
  const MatPlan mp = plan_matrix(N, K, 32, ng, n_cu);
  const TilePlan p = plan_tiles(mp, pairs, M, n_cu, part, max_split);
  CHECK(p.wc >= 1 && p.per >= 1 && p.ksplit >= 1);
  const int KT = mp.KT, CT = mp.G * ng, CG = 8 * p.wc, RT = 8 / p.wc * p.rtw, S = p.ksplit;
  CHECK(p.ncb * CG >= CT && p.nrb * RT * 16 >= M);
  ++modes[S > 1 ? 3 : p.sums.nseg == 1 ? 0 : p.compact ? 2 : 1];
  // the matrix's segment ends by its definition: owners of a group's units
  const SumPlan& s = p.sums;
  std::vector<std::vector<int>> ends(s.G);
  for (int g = 0; g < s.G; ++g) {
    for (int k = 0; k + 1 < KT; ++k)
      if (unit_owner((uint32_t)g * KT + k, KT, s.G, s.c, s.n) != unit_owner((uint32_t)g * KT + k + 1, KT, s.G, s.c, s.n))
        ends[g].push_back(k + 1);
    CHECK((int)ends[g].size() < s.nseg);
  }
  GemmArgs a{};
  a.KT = KT;
  a.G = mp.G;
  a.N = N;
  a.n_wg = mp.n_wg;
  a.segc = mp.c;
  a.share = mp.S;
  a.ng = ng;
  a.M = M;
  std::vector<int> seen((size_t)p.ncb * p.nrb * KT);
  for (int cb0 = 0; cb0 < p.ncb; cb0 += p.per) {
    tile_launch(a, p, cb0);
    std::set<int64_t> places;
    for (int b = 0; b < tile_grid(a); ++b) {
      const TileItem it = tile_item(a, b, S);
      if (it.cbl < 0) continue;
      CHECK(it.cb < p.ncb && it.rb < p.nrb && it.sp < S);
      TileRange r{0, KT, 0, 1, 0, 1, 1};
      const int ct0 = it.cb * CG, g0 = std::min(ct0 / s.tiles, s.G - 1);
      if (S > 1) {
        r = tile_range(a, ct0, it.sp);
        CHECK(r.nseg == (int)ends[g0].size() + 1 && r.nseg - r.n0 + 1 <= a.nslot && r.E <= 31);
        if (it.sp >= r.E) continue;
        CHECK((int64_t)it.rb * a.ncb + it.cbl < max_split);
      }
      CHECK(r.kb >= 0 && r.kb < r.ke && r.ke <= KT);
      for (int k = r.kb; k < r.ke; ++k) ++seen[((size_t)it.cb * p.nrb + it.rb) * KT + k];
      // segments, as the kernel walks them, for every 64 columns
      for (int ct = ct0; ct < ct0 + CG && 16 * ct < N; ct += 4) {
        const uint32_t base = sum_base(a, S > 1 ? ct0 : ct);
        const int g = std::min(ct / s.tiles, s.G - 1);
        if (S > 1) CHECK(ends[g] == ends[g0]);
        std::vector<int> walked;
        int own = S > 1 ? r.own0 + r.seg0 : sum_owner(a, base);
        if (S == 1 && s.nseg > 1) {
          const int at = chain_place(a, it.rb, ct, own, CG, RT);
          CHECK(at >= 0 && (size_t)at + (size_t)RT * 4096 <= part && at % (RT * 4096) == 0);
          if (!ends[g].empty()) CHECK(places.insert(at).second);
        }
        for (int e; (e = sum_start(a, base, own + 1)) < r.ke; ++own) walked.push_back(e);
        std::vector<int> want;
        for (int e : ends[g])
          if (e > r.kb && e < r.ke) want.push_back(e);
        CHECK(walked == want);
        if (S > 1) {
          CHECK(r.kb == 0 || ends[g][r.seg0 - 1] == r.kb);
          CHECK(own - r.own0 < r.nseg);
        }
      }
      if (S > 1) {
        std::set<int> slots;
        for (int seg = r.seg0; seg < r.nseg && (seg == 0 || ends[g0][seg - 1] < r.ke); ++seg) slots.insert(part_slot(r, seg));
        for (int slot : slots)
          for (int rt = 0; rt < RT; ++rt)
            for (int w = 0; w < p.wc; ++w) {
              const int at = part_place(a, it.rb * a.ncb + it.cbl, slot, rt, w, RT, p.wc);
              CHECK(at >= 0 && (size_t)at + 8192 <= part && slot < a.nslot);
              CHECK(places.insert(at).second);
            }
      }
      // weight tiles (one row block is enough)
      if (it.rb == 0)
        for (int ct = ct0; ct < ct0 + CG && ct < CT; ++ct) {
          TileTrk t{ct / ng, 0, 0, 0};
          trk_set(a, t, unit_owner((uint32_t)t.g * KT + r.kb, KT, mp.G, mp.c, mp.n_wg));
          for (int k = r.kb; k < r.ke; ++k) {
            while (k >= t.kend) trk_set(a, t, t.o + 1);
            const int64_t slot = t.base + (int64_t)k * mp.n_wg;
            CHECK(slot == plan_slot(mp, t.g, k) && slot < plan_slots(mp));
          }
        }
    }
  }
  for (int n : seen) CHECK(n == 1);
}

int main() {
  struct Shape {
    int d, hq, hkv, hd, ff, V;
  };
  // the named shapes' widths, and narrow or odd ones: groups of 4 and 8 tiles, uneven shares, one k-step per segment
  const Shape shapes[] = {{5120, 64, 8, 128, 25600, 151936}, {3584, 28, 4, 128, 18944, 152064}, {320, 5, 5, 64, 672, 1056},
                          {384, 6, 2, 128, 1088, 2176},      {512, 8, 2, 64, 1024, 4224},       {256, 64, 8, 128, 512, 1056},
                          {6400, 25, 5, 128, 3200, 33280},   {1024, 8, 4, 128, 40960, 2048},    {9216, 100, 4, 64, 3200, 4096}};
  for (const Shape& h : shapes) {
    auto pick = [](int tiles, int most) {
      for (int g : {8, 4, 2})
        if (g <= most && tiles % g == 0) return g;
      return 1;
    };
    const int q = (h.hq + 2 * h.hkv) * h.hd, o = h.hq * h.hd;
    const int64_t max_split = h.V / 16 + 2 * h.ff / 16 + h.d / 16 + 64;
    const struct {
      int N, K, ng;
      bool pairs;
    } mats[] = {{q, h.d, h.hd / 16, false},
                {h.d, o, pick(h.d / 16, 4), false},
                {2 * h.ff, h.d, pick(2 * h.ff / 16, 8), true},
                {h.d, h.ff, pick(h.d / 16, 8), false},
                {h.V, h.d, pick(h.V / 16, 8), true}};
    for (const auto& m : mats) {
      if (m.ng < 4) continue;  // other kernels
      for (int M : {65, 99, 128, 129, 264, 513, 1136, 4096})
        for (size_t part : {(size_t)256 * 65536, (size_t)256 * 655360})
          if (h.V < 100000 || m.N < 100000 || M < 600) replay(m.N, m.K, m.ng, m.pairs, M, part, max_split);
    }
  }
  std::printf("whole %d chain %d compact %d split %d\n", modes[0], modes[1], modes[2], modes[3]);
  return modes[0] && modes[1] && modes[2] && modes[3] ? 0 : 1;
}
