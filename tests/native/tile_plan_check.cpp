// The GEMMs' tile order and tile height (tile_plan.hpp): xcd_tile visits every
// tile once, each XCD a contiguous run, for every count up to 4096; split_tile
// does for every grid, and an XCD's tiles touch no more rows of the longer operand
// than its run needs; the chosen height is one of the three and takes least under
// the stated model.
#include <stdint.h>
#include <stdio.h>

#include <vector>

#include "tile_plan.hpp"

int main() {
  long long checked = 0, bad = 0;
  for (int total = 1; total <= 4096; ++total) {
    std::vector<int> seen(total, 0);
    for (int id = 0; id < total; ++id) {
      const int t = qg::xcd_tile(id, total);
      ++checked;
      if (t < 0 || t >= total || seen[t]++) { ++bad; printf("total %d id %d -> %d\n", total, id, t); continue; }
      if (id >= 8 && t != qg::xcd_tile(id - 8, total) + 1) { ++bad; printf("total %d id %d not contiguous\n", total, id); }
    }
  }
  for (int tm = 1; tm <= 130; tm += (tm < 12 ? 1 : 7))
    for (int tn = 1; tn <= 130; tn += (tn < 12 ? 1 : 7))
      for (int tall = 0; tall < 2; ++tall) {
        std::vector<int> seen(tm * tn, 0);
        std::vector<std::vector<char>> band(8, std::vector<char>(tall ? tm : tn, 0));
        for (int id = 0; id < tm * tn; ++id) {
          const qg::TileAt at = qg::split_tile(id, tm, tn, tall != 0);
          ++checked;
          if (at.bm < 0 || at.bm >= tm || at.bn < 0 || at.bn >= tn || seen[at.bm * tn + at.bn]++) {
            ++bad;
            printf("split_tile %d x %d id %d -> %d %d\n", tm, tn, id, at.bm, at.bn);
            continue;
          }
          band[id & 7][tall ? at.bm : at.bn] = 1;
        }
        const int len = tall ? tn : tm, run = (tm * tn + 7) / 8;  // tiles across a band, tiles of an XCD
        for (int x = 0; x < 8; ++x) {
          int used = 0;
          for (char b : band[x]) used += b;
          if (used > (run + len - 1) / len + 1) { ++bad; printf("split_tile %d x %d tall %d: XCD %d takes %d bands\n", tm, tn, tall, x, used); }
        }
      }
  const qg::RoundCost costs[] = {{83, 56}, {92, 70}, {86, 62}, {80, 62}, {86, 71}};
  for (int64_t cus : {256, 304, 64})
    for (const qg::RoundCost& c : costs)
      for (int64_t m = 1; m <= 6000; m += 7)
        for (int64_t tn = 1; tn <= 48; ++tn) {
          ++checked;
          const int tm = qg::plan_tile_rows(m, tn, cus, c).tm;
          if (tm < 2 || tm > 4) { ++bad; printf("m %lld tn %lld tm %d\n", (long long)m, (long long)tn, tm); continue; }
          const auto time = [&](int h) {  // the stated model, in rounds of 256-row tiles
            const int64_t tiles = (m + 64 * h - 1) / (64 * h) * tn;
            const double part = double(tiles % cus) / cus;
            return (double(tiles / cus) + (part > 0 ? 0.72 + 0.28 * part : 0.0)) * (h == 4 ? 1.0 : (h == 3 ? c.rows192 : c.rows128) / 100.0);
          };
          for (int h = 2; h <= 4; ++h)
            if (time(tm) > time(h) + 1e-9) { ++bad; printf("m %lld tn %lld: %d, %d is cheaper\n", (long long)m, (long long)tn, tm, h); }
        }
  printf("checked %lld violations %lld\n", checked, bad);
  return bad != 0;
}
