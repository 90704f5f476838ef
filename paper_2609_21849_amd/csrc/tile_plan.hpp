// tile_plan.hpp -- how the GEMMs (gemm.hip) cut the output into tiles, in which
// order they take them and where they share K instead, checked without a GPU.
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

// Tile of workgroup `id` of a split-K kernel. An XCD's run of tiles goes along the
// side with fewer rows of operands (tall: more activation than weight rows), so
// that its L2 holds a band of the longer operand and the shorter one: FP8 872 x 272
// x 7424 13.3 us with the runs down the rows, 11.5 across; 3867 x 320 x 2560 14.2, 12.3;
// NVFP4 5285 x 1024 x 12032 151, 143; 512 x 3072 x 3072 the other way round 13.2, 16.8.
// (A single row of tiles: the launch order is within 1% of the runs on average, 7%
// better at FP8 2 x 12704 x 3456 and 8% worse at NVFP4 2 x 3456 x 13312.)
struct TileAt {
  int bm, bn;
};
__host__ __device__ inline TileAt split_tile(int id, int tiles_m, int tiles_n, bool tall) {
  const int t = xcd_tile(id, tiles_m * tiles_n), len = tall ? tiles_n : tiles_m;
  const int band = t / len, in = t - band * len;
  return tall ? TileAt{band, in} : TileAt{in, band};
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

// A tiling of a split-K kernel: tiles of 32 mt x 32 np outputs, nw waves sharing
// the reduction, each with d 128-wide chunks in flight. {}: not a split-K kernel.
struct SplitK {
  int mt = 0, np = 0, nw = 0, d = 0;
  constexpr bool operator==(const SplitK& o) const { return mt == o.mt && np == o.np && nw == o.nw && d == o.d; }
};

// W4A16 beside the two weight-pool kernels. {}: the persistent kernel, past the
// ridge point with enough large tiles: from 21/32 of a round of 128 x 256 tiles
// (split-K against 128-row tiles, back to back: 500 x 9216 x 3072, 144 tiles, 50.5 / 53.6
// us; 1280 x 4096 x 4096, 160, 66.1 / 69.2; 3500 x 1536 x 3072, 168, 57.6 / 53.0), or 3/8 of
// one of 256 x 256; up to K = 512, where the split's reduction is most of its
// time, from 5/16 of a round of the former (7674 x 432 x 256, 120 tiles, 14.6 / 9.9; 1117
// x 2112 x 384, 81, 12.4 / 11.3; 1643 x 1392 x 512, 78, 13.2 / 13.0; 1523 x 976 x 384, 48, 9.2 /
// 11.2). Not for 129 to 192 rows at long K, a third of whose 128-row tiles is padding
// (150 x 21568 x 8192 97 us split, 129; 141 x 23488 x 3200 53.5, 55.0; 147 x 24080 x 1408
// 31.5, 27.3). Heights (256 rows -> chosen): 1024 x 6144 x 3072 68.4 -> 54.0 us (128),
// 2304 x 9216 x 3072 146.7 -> 128.8 (192), 1900 x 3072 x 1024 28.3 -> 21.3 (128).
// Split-K tilings. Up to 32 rows: one-panel workgroups, at K > 3072 with three
// chunks of a wave in one batch of loads, else one at a time where the workgroups
// all run at once or read few activations: 1 x 3072 x 1024 4.4 -> 3.9 us, 24 x 9216 x
// 3072 13.2 -> 12.9, 24 x 90880 x 1024 30.9 -> 29.1; where more follow each other the
// batch keeps more in flight (17 x 363520 x 3072 224 us against 308, 30 x 52944 x 2304
// 37.7 against 46.0, 16 x 18432 x 3072 16.0 against 16.9, 32 x 9216 x 3072 15.3 against
// 16.1; 32 x 2048 x 6144 15.6 against 17.3). Above 32 rows the narrowest 32-row tile
// that gives every workgroup a CU of its own; past that 64-row tiles, which expand
// each weight once for two row blocks (the expansion is the bound there): 64 x 96
// where those make one round that 64 x 64 tiles would overflow. 32 x 64 tiles of
// four waves, several workgroups per CU, stay for short reductions (256 x 3072 x
// 1024 8.5 us against 8.9) and where 64-row tiles would pad the rows by more than
// an eighth (200 x 9216 x 3072 30.3 against 34.0). Measured (GPU time from graph
// replays, 24 shapes, 21 tilings) against a rule by M and N: 64 x 3072 x 3072 10.9 ->
// 7.4 us, 512 x 3072 x 3072 25.6 -> 21.2, 1024 x 3072 x 3072 47 -> 36, 2048 x 1024 x 3072
// 73 -> 27, 1148 x 352 x 2304 57 -> 11, 1446 x 1984 x 6016 140 -> 63.
inline SplitK plan_w4a16(int64_t m, int64_t n, int64_t k, int64_t cus) {
  const int64_t rows32 = (m + 31) / 32, rows64 = (m + 63) / 64, npan = (n + 31) / 32;
  const int64_t tiles256 = (m + 255) / 256 * ((n + 255) / 256), tiles128 = (m + 127) / 128 * ((n + 255) / 256);
  if (m > 128 && (8 * tiles256 >= 3 * cus || (k <= 512 && 16 * tiles128 >= 5 * cus))) return {};
  if (m > 128 && 32 * tiles128 >= 21 * cus) return m <= 192 && k >= 3072 ? SplitK{2, 2, 4, 1} : SplitK{};
  const int64_t t12 = rows32 * ((npan + 1) / 2), t22 = rows64 * ((npan + 1) / 2), t23 = rows64 * ((npan + 2) / 3);
  if (m <= 32) return {1, 1, 8, k <= 3072 && (npan <= cus || m * k <= (npan <= 2 * cus ? 72 : 24) * 1024) ? 1 : 3};
  if (rows32 * npan <= cus) return {1, 1, 8, 3};
  if (k <= 1024 && t12 <= 2 * cus) return {1, 2, 4, 3};
  if (t12 <= cus) return {1, 2, 8, 3};
  if (16 * rows64 > 9 * rows32) return {1, 2, 4, 3};
  if (t22 > cus && t23 <= cus) return {2, 3, 4, 1};
  return {2, 2, 4, 1};
}

// NVFP4. {}: the persistent kernel. Below half a round of 256 x 256 tiles and 11/16
// of a round of 128 x 256 ones the split-K kernel is faster (back to back, split-K
// against 128-row tiles: 500 x 9216 x 3072, 144 tiles, 35.7 / 37.2 us; 1280 x 4096 x
// 4096, 160, 46.9 / 48.3; 640 x 9216 x 3072, 180, 42.6 / 38.4; 1900 x 3072 x 1024, 180,
// 21.3 / 16.8; 1024 x 6144 x 3072, 192, 44.3 / 40.1; 2300 x 3072 x 9216, 216, 164 / 113),
// and for 129 to 192 rows at long K, a third of whose 128-row tiles is padding (151 x
// 27472 x 5376 66.5 / 72.9; 141 x 23488 x 3200 35.7 / 41.8; 168 x 25664 x 1152 22.4 / 20.6).
// The narrowest tile that gives every workgroup a CU of its own (64 x 64 before 64
// x 96: 1520 x 624 x 768 6.4 us against 8.0, 315 x 3056 x 11136 25.9 against 30.7);
// past that 64 x 64 tiles of four waves, two workgroups per CU, so that one's
// reduction runs beside the other's loop, except at long K, where that hides
// little, 64 x 96 if they make no more rounds (4743 x 480 x 5120 35.3 us against 40.2,
// 1173 x 3808 x 11392 104 against 115, 666 x 6128 x 4096 41.7 against 45.8; at K = 2944 1896 x
// 1248 23.9 against 22.8).
// Measured (GPU time from graph replays,
// 24 shapes, 12 tilings) against a 32 x 64 / 64 x 64 / 64 x 96 rule: 1 x 3072 x 1024
// 5.1 -> 3.8 us, 64 x 3072 x 3072 8.0 -> 5.8, 300 x 1024 x 3072 8.1 -> 6.9, 151 x 3520 x
// 5504 21.6 -> 14.8, 2048 x 1024 x 3072 25.0 -> 20.3, 1555 x 4512 x 3968 80 -> 69.
inline SplitK plan_nvfp4(int64_t m, int64_t n, int64_t k, int64_t cus) {
  const int64_t rows32 = (m + 31) / 32, rows64 = (m + 63) / 64, chunks = k / 128;
  const int64_t tiles256 = (m + 255) / 256 * ((n + 255) / 256), tiles128 = (m + 127) / 128 * ((n + 255) / 256);
  if (m > 128 && (2 * tiles256 >= cus || (16 * tiles128 >= 11 * cus && (m > 192 || k < 3072)))) return {};
  if (rows32 * ((n + 31) / 32) <= cus) return chunks >= 32 ? SplitK{1, 1, 8, 1} : SplitK{1, 1, 4, 2};  // 44 x 352 x 7296 8.8 -> 8.2 us
  if (rows32 * ((n + 63) / 64) <= cus) return chunks >= 32 ? SplitK{1, 2, 8, 3} : SplitK{1, 2, 8, 1};  // 16 x 9216 x 9216 14.5 -> 13.5 us
  if (rows32 * ((n + 95) / 96) <= cus) return {1, 3, 8, 1};
  const int64_t t22 = rows64 * ((n + 63) / 64), t23 = rows64 * ((n + 95) / 96);
  if (t22 <= cus) return {2, 2, 8, 1};
  if (t23 <= cus) return {2, 3, 8, 1};
  const int64_t rounds22 = (t22 + 2 * cus - 1) / (2 * cus), rounds23 = (t23 + cus - 1) / cus;
  if (k >= (rounds23 > 2 ? 4096 : 5120) && rows64 > 1 && rounds23 <= rounds22) return {2, 3, 8, 1};
  return {2, 2, 4, 2};
}

// MXFP4 / MXFP8. Up to a round of 64 x 96 tiles on the CUs the split-K kernel,
// above that the large tiles ({}): those walk K serially, while a split-K tile's
// waves share K (and are bound by their L1 requests). Inside the
// split-K range the narrowest tile that still gives every workgroup a CU of its own.
// Measured (GPU time from graph replays, 256 x 256 -> split-K; best of 16 tilings
// within 8% everywhere): MXFP4 1 x 3072 x 1024 12.7 -> 2.8 us, 256 x 3072 x 3072 25.0 ->
// 6.8, 500 x 3072 x 3072 38 -> 10.8; MXFP8 14.3 -> 3.1, 32.0 -> 10.3, 37.5 -> 15.0.
// Two rounds of split-K tiles against 128-row large ones: MXFP4 355 x 7664 x 256 10.5 /
// 6.1 us, 166 x 16176 x 1536 14.1 / 10.1, 1024 x 3072 x 3072 18.8 / 14.2, 700 x 4096 x 9216
// 41.1 / 37.9; MXFP8 1024 x 3072 x 512 14.4 / 8.1, 310 x 7008 x 1792 19.5 / 15.3, 1180 x 2224 x
// 6144 48.3 / 48.1, but with long K MXFP8's split is level or better (12 shapes: 518 x
// 4816 x 7680 56.2 / 57.3, 5262 x 496 x 8448 65.7 / 64.0, 406 x 6016 x 9472 64.0 / 67.5, 699 x 4016
// x 11520 79.2 / 84.9, 968 x 2528 x 14848 102 / 107).
inline SplitK plan_mx(int64_t m, int64_t n, int64_t k, int64_t cus, bool fp8) {
  const int64_t rows32 = (m + 31) / 32, rows64 = (m + 63) / 64;
  if (rows32 * ((n + 31) / 32) <= cus) return {1, 1, 4, 2};
  if (rows32 * ((n + 63) / 64) <= cus) return {1, 2, 4, 2};
  if (rows32 * ((n + 95) / 96) <= cus) return {1, 3, 8, 1};
  const int64_t t23 = rows64 * ((n + 95) / 96);
  if (t23 > cus && rows64 * ((n + 127) / 128) <= cus) return {2, 4, 8, 1};
  if (t23 <= cus || (t23 <= 2 * cus && fp8 && k > 6144)) return {2, 3, 4, 2};
  return {};
}

// FP8. {}: the persistent kernels of large tiles; kFp8Tiles64: the 64 x 128 tiles
// of four waves (k_gemm_fp8), which share no K.
// Few tokens: the split-K kernel. FP8 operands need no expansion, so
// narrow tiles cost nothing extra: the narrowest 32-row tile (32 x 32 NP,
// NP = 1 .. 4) that still gives every workgroup a CU of its own, with
// eight waves and one chunk in flight each (NP = 2: four waves, two
// chunks); else 32 x 64 tiles while those number at most two per CU.
// Measured at M = 16 .. 1024, N, K in {256, 1024, 3072, 9216} (GPU time
// from graph replays): the best of five tilings within 2% at every shape
// (128 x 256 x 256 3.8 -> 3.2 us, 256 x 3072 x 1024 6.6 -> 5.7 us,
// 1024 x 1024 x 3072 11.9 -> 10.0 us; the 32 x 64 rule alone was 1.2-1.9x
// faster than the 64 x 128 kernel where K >= 3072).
constexpr SplitK kFp8Tiles64 = {2, 4, 4, 0};

inline SplitK plan_fp8(int64_t m, int64_t n, int64_t k, int64_t cus) {
  const int64_t rows32 = (m + 31) / 32, rows64 = (m + 63) / 64, t12 = rows32 * ((n + 63) / 64);
  if (m <= 1024) {
    // (at most four chunks, K <= 512: four waves, 128 x 256 x 256 3.2 -> 2.8 us)
    if (rows32 * ((n + 31) / 32) <= cus) return k <= 512 ? SplitK{1, 1, 4, 1} : SplitK{1, 1, 8, 1};
    if (t12 <= cus) return {1, 2, 4, 2};
    if (rows32 * ((n + 95) / 96) <= cus) return {1, 3, 8, 1};
    if (rows32 * ((n + 127) / 128) <= cus) return {1, 4, 8, 1};
  }
  if (t12 <= 2 * cus) return {1, 2, 4, 2};
  // one round of 64 x 96 split-K tiles at long K, where the 64 x 128 kernel
  // below walks K in too few workgroups: 512 x 3072 x 3072 15.1 -> 14.0 us, 512 x
  // 3072 x 9216 34.2 -> 29.4 (at 889 x 1584 x 1152 it loses, 8.8 -> 9.2)
  if (k >= 2048 && rows64 * ((n + 95) / 96) <= cus) return {2, 3, 4, 2};
  // Too few large tiles to fill the chip: the 64 x 128 kernel's many more
  // workgroups win. Measured crossover: 3/8 of a 128 x 256 tile per CU (1024 x
  // 3072 x 3072, 96 tiles, 20.7 us against 20.4; 700 x 4096 x 9216, 96, 49.2 against
  // 50.6; 1500 x 3072 x 3072, 144, 28.4 against 21.2), and below K = 4608 as long as
  // its workgroups are at most two per CU, which run at once (6351 x 528 x 1152,
  // 500 workgroups, 11.2 us against 12.2; 4278 x 528 x 2432, 335, 17.5 against 19.0;
  // 620 x 5360 x 4224, 420, 27.8 against 28.6; but 5668 x 704 x 2048, 534, 21.5 against
  // 17.3, and 473 x 7808 x 6528, 488, 41.1 against 39.7); below K = 1024 3/8 of a
  // 256 x 256 tile.
  const int64_t tiles256 = (m + 255) / 256 * ((n + 255) / 256), tiles128 = (m + 127) / 128 * ((n + 255) / 256);
  if (m <= 128 || (k < 1024 ? 8 * tiles256 < 3 * cus : 8 * tiles128 <= 3 * cus)) return kFp8Tiles64;
  if (k >= 1024 && k < 4608 && rows64 * ((n + 127) / 128) <= 2 * cus) return kFp8Tiles64;
  return {};
}

}  // namespace qg
