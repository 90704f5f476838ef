// tile_plan.hpp -- how the GEMMs (gemm.hip) cut the rows of the output into
// tiles and in which order they take them, checked over many sizes without a GPU.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace qg {

// Tile of workgroup `id` of `total`: workgroups are dealt round-robin to the 8
// XCDs, and every XCD takes one contiguous run of tiles (the first total % 8 of
// them one more). Totals that 8 does not divide used to keep the launch order,
// which spreads every operand panel over all eight L2s: MXFP8 2800 x 9216 x
// 3072 (396 tiles) 76.2 -> 70.1 us, calls back to back.
__host__ __device__ inline int xcd_tile(int id, int total) {
  const int x = id & 7, extra = total & 7;
  return x * (total >> 3) + (x < extra ? x : extra) + (id >> 3);
}

// Time of a full round (one tile a CU) of tiles of 64 tm rows x 256 columns, in
// percent of one of 256 rows: more than 75 and 50, since every tile still reads
// (and for NVFP4 expands) the whole weight panel group.
struct RoundCost {
  int rows192, rows128;
};

// Time of `tiles` equal tiles, one a CU at a time, in percent of a full round
// times the CUs. A tile walks K serially, so a round that is partly empty costs
// nearly what a full one does (72 % of it and up: fewer busy CUs run at a higher
// clock and share less bandwidth).
inline int64_t rounds_cost(int64_t tiles, int64_t cus) {
  const int64_t rest = tiles % cus;
  return 100 * (tiles / cus) * cus + (rest > 0 ? 72 * cus + 28 * rest : 0);
}

// Height of the tiles of a persistent large-tile GEMM, 64 tm rows (tm = 4, 3, 2),
// for m rows and tiles_n tile columns: the one whose rounds of tiles take least
// (shorter tiles are cheaper where they don't start another round).
struct TileRows {
  int tm;
  int64_t cost;  // rounds_cost x percent of a 256-row round
};
inline TileRows plan_tile_rows(int64_t m, int64_t tiles_n, int64_t cus, RoundCost cost) {
  TileRows best = {0, 0};
  for (int tm = 4; tm >= 2; --tm) {
    const int64_t c = rounds_cost((m + 64 * tm - 1) / (64 * tm) * tiles_n, cus) *
                      (tm == 4 ? 100 : tm == 3 ? cost.rows192 : cost.rows128);
    if (best.tm == 0 || c < best.cost) best = {tm, c};
  }
  return best;
}

}  // namespace qg
