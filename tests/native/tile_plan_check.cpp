// The GEMMs' tile order and tile height (tile_plan.hpp): xcd_tile visits every
// tile once, each XCD a contiguous run, for every count up to 4096; the chosen
// height is one of the three and takes least under the stated model.
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
