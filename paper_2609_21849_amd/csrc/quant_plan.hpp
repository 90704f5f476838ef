// quant_plan.hpp -- what host and device share of the quantizers' (quantize.hip)
// addressing, checked by host-only tests over many sizes: the launch plan of
// the two-launch dynamic quantizer (how many amax workgroups P leave their
// maxima, into how many code regions G, and where region j begins), the rows
// of a column slice read in 16-byte units, and the pieces of very large tensors.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

namespace qg {

constexpr int kSlotsAmaxLoads = 4;          // 16-byte loads per lane in flight
constexpr int64_t kSlotsAmaxGroups = 1024;  // P, a multiple of 8
constexpr int64_t kSlotsQuantGroups = 2048;
// The P x G scattered 4-byte slot stores grow with the tensor: at 4608 x
// 3072 (P = 1024 or 512, G = 1728 or 1024) the two launches took 17-22 us
// against the chain's 12.4 (GPU time from graph replays); at 256 x 3072 5.7
// against 6.7 us (FP8) and 6.4 against 7.7 (NVFP4), at 512 x 3072 6.2 against
// 7.0 and 6.8 against 7.9, level from 3 Mi elements on (1024 x 4096: 8.2
// against 7.8). Larger tensors take the chain.
constexpr int64_t kSlotsMaxElements = int64_t(3) << 20;

// First 16-byte unit (8 elements) of region j of g over `pairs` unit pairs:
// regions start on even units, so an NVFP4 16-block never straddles two.
__host__ __device__ inline int64_t slot_region_lo(int64_t pairs, int64_t j, int64_t g) { return 2 * (pairs * j / g); }

struct SlotsPlan {
  int64_t P;  // amax workgroups (a multiple of 8), one 4-byte slot each per region
  int64_t G;  // code regions = quantize workgroups; 0: the plan does not apply
};

// Plan for a tensor of n elements in whole units (n % 8 == 0), code bytes per unit
// cb = 8 (FP8) or 4 (NVFP4): every region's codes must hold the P slots.
inline SlotsPlan slots_plan(int64_t n, int cb) {
  if (n <= 0 || n % 8 != 0 || n > kSlotsMaxElements) return {0, 0};
  const int64_t units = n / 8, pairs = units / 2;
  const int64_t P =
      std::min<int64_t>(kSlotsAmaxGroups, ((units + 256 * kSlotsAmaxLoads - 1) / (256 * kSlotsAmaxLoads) + 7) / 8 * 8);
  const int64_t need = (4 * P + 2 * cb - 1) / (2 * cb);  // unit pairs per region that hold the slots
  const int64_t G = std::min<int64_t>(std::min<int64_t>(kSlotsQuantGroups, (units + 1023) / 1024), pairs / need);
  return {P, G >= 1 ? G : 0};
}

// A tensor read as 16-byte units (8 elements): unit u of the tensor in row
// order is unit c of row r, u = r upr + c. The row comes from a multiplication
// by mul = ceil(2^shift / upr): exact for u < 2^31, since the excess e = mul upr -
// 2^shift is below upr <= 2^(shift - 32), so u e < 2^shift, and mul < 2^33 keeps
// the product in 64 bits. A column slice of a wider tensor is then read in the
// same wave-contiguous runs as a dense one.
struct UnitRows {
  uint64_t mul = 0;
  uint32_t upr = 0;   // units per row
  int shift = 0;      // 32 + ceil(log2 upr)
  int64_t pitch = 0;  // units between rows

  __host__ __device__ uint32_t row_of(uint32_t u) const { return (uint32_t)((mul * u) >> shift); }
};

inline UnitRows unit_rows(int64_t cols, int64_t ldx) {  // cols % 8 == 0, ldx % 8 == 0, cols > 0
  UnitRows r;
  r.upr = (uint32_t)(cols / 8);
  r.pitch = ldx / 8;
  r.shift = 32;
  while ((int64_t(1) << (r.shift - 32)) < (int64_t)r.upr) ++r.shift;
  r.mul = ((uint64_t(1) << r.shift) + r.upr - 1) / r.upr;
  return r;
}

// A launch takes at most this many elements, eight or more a thread: from 2^32
// threads on HIP launches only what is left of their number modulo 2^32 and
// reports success (static FP8 of 2^36 elements and more left its codes unwritten),
// and the units of a slice must number 2^31 at most. A multiple of every format's
// block.
constexpr int64_t kLaunchElements = int64_t(1) << 34;

// fn(offset in x, offset in the dense codes, elements) for the pieces of a tensor
// of rows `ldx` apart: runs of a dense tensor, whole rows of a slice.
template <class F>
inline void for_pieces(int64_t rows, int64_t cols, int64_t ldx, F fn) {
  if (ldx == cols) {
    for (int64_t e = 0, n = rows * cols; e < n; e += kLaunchElements) fn(e, e, std::min(kLaunchElements, n - e));
    return;
  }
  const int64_t step = kLaunchElements / cols;
  for (int64_t r = 0; r < rows; r += step) fn(r * ldx, r * cols, std::min(step, rows - r) * cols);
}

}  // namespace qg
