// Row of a 16-byte unit by multiplication (UnitRows in quant_plan.hpp) against
// the division, for every row width up to 4096 units, wider ones, and widths
// around powers of two: the units at both ends of rows near 0, 2^16 and 2^31.
#include <stdint.h>
#include <stdio.h>

#include <vector>

#include "quant_plan.hpp"

int main() {
  long long checked = 0, bad = 0;
  std::vector<int64_t> widths;
  for (int64_t w = 1; w <= 4096; ++w) widths.push_back(w);
  for (int b = 12; b <= 27; ++b)
    for (int d = -2; d <= 2; ++d) widths.push_back((int64_t(1) << b) + d);
  for (int64_t w : {999983, 1000003, 16777259, 99999989, 268435455}) widths.push_back(w);
  for (int64_t w : widths) {
    const qg::UnitRows r = qg::unit_rows(8 * w, 8 * w + 8);
    const int64_t last = (int64_t(1) << 31) - 1;
    for (int64_t near : {int64_t(0), int64_t(65536), last / 2, last})
      for (int64_t row = near / w - 2; row <= near / w + 2; ++row)
        for (int64_t u : {row * w - 1, row * w, row * w + 1, row * w + w / 2, row * w + w - 1}) {
          if (u < 0 || u > last) continue;
          ++checked;
          if ((int64_t)r.row_of((uint32_t)u) != u / w) { ++bad; printf("width %lld unit %lld\n", (long long)w, (long long)u); }
        }
  }
  printf("checked %lld violations %lld\n", checked, bad);
  return bad != 0;
}
