// The pieces of very large tensors (for_pieces in quant_plan.hpp): in order,
// without gap or overlap, whole rows of a slice, whole blocks of every format;
// no launch of 8 or more elements a thread reaches HIP's 2^32 threads, and a
// slice's units stay below 2^31 (UnitRows::row_of).
#include <stdint.h>
#include <stdio.h>

#include "quant_plan.hpp"

int main() {
  long long checked = 0, bad = 0;
  const int64_t top = (int64_t(1) << 31) - 32;
  for (int64_t cols : {int64_t(8), int64_t(24), int64_t(3072), int64_t(9216), int64_t(16777216), int64_t(1) << 30, top})
    for (int64_t rows : {int64_t(0), int64_t(1), int64_t(7), int64_t(4608), int64_t(1999993), int64_t(16777217), int64_t(715827883), top}) {
      if (cols > 0 && rows > (int64_t(1) << 38) / cols) continue;  // 512 GB of bf16
      for (int64_t ldx : {cols, cols + 8, 3 * cols}) {
        int64_t next = 0, pieces = 0;
        qg::for_pieces(rows, cols, ldx, [&](int64_t src, int64_t e, int64_t cnt) {
          ++checked;
          ++pieces;
          const int64_t block = cols % 32 == 0 ? 32 : 8;
          bool ok = e == next && cnt > 0 && cnt <= int64_t(1) << 34 && e % block == 0;
          ok = ok && (cnt + 8 * 256 - 1) / 8 < int64_t(1) << 32;
          if (ldx == cols) ok = ok && src == e;
          else ok = ok && e % cols == 0 && cnt % cols == 0 && src == e / cols * ldx && cnt / 8 <= int64_t(1) << 31;
          if (!ok) { ++bad; printf("rows %lld cols %lld ldx %lld: piece at %lld of %lld\n", (long long)rows, (long long)cols,
                                   (long long)ldx, (long long)e, (long long)cnt); }
          next = e + cnt;
        });
        if (next != rows * cols || (rows * cols <= int64_t(1) << 33 && pieces > 1)) { ++bad; printf("rows %lld cols %lld ldx %lld: %lld pieces end at %lld\n",
            (long long)rows, (long long)cols, (long long)ldx, (long long)pieces, (long long)next); }
      }
    }
  printf("checked %lld violations %lld\n", checked, bad);
  return bad != 0;
}
