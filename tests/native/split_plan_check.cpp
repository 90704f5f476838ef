// Which kernel a GEMM takes (plan_* in tile_plan.hpp) at 256 CUs, for the shapes
// that the rules were measured at and that decide them: format, M, N, K and the
// tiling that took least (mt np nw d; 0 0 0 0: no split-K tiling).
#include <stdint.h>
#include <stdio.h>
#include <string.h>

#include "tile_plan.hpp"

int main() {
  struct Row { const char* kind; int64_t m, n, k; qg::SplitK want; };
  static const Row rows[] = {
#include "split_plan_rows.inc"
  };
  int bad = 0;
  for (const Row& r : rows) {
    qg::SplitK p{-1, 0, 0, 0};
    if (!strcmp(r.kind, "w4a16")) p = qg::plan_w4a16(r.m, r.n, r.k, 256);
    if (!strcmp(r.kind, "nvfp4")) p = qg::plan_nvfp4(r.m, r.n, r.k, 256);
    if (!strcmp(r.kind, "mxfp4")) p = qg::plan_mx(r.m, r.n, r.k, 256, false);
    if (!strcmp(r.kind, "mxfp8")) p = qg::plan_mx(r.m, r.n, r.k, 256, true);
    if (!strcmp(r.kind, "fp8")) p = qg::plan_fp8(r.m, r.n, r.k, 256);
    if (!(p == r.want)) {
      ++bad;
      printf("%s %lld x %lld x %lld: %d %d %d %d, wanted %d %d %d %d\n", r.kind, (long long)r.m, (long long)r.n, (long long)r.k,
             p.mt, p.np, p.nw, p.d, r.want.mt, r.want.np, r.want.nw, r.want.d);
    }
  }
  printf("checked %d violations %d\n", (int)(sizeof rows / sizeof rows[0]), bad);
  return bad != 0;
}
