// pack.hip -- offline weight re-layout into matrix-core operand order.
//
// PTQ weights are quantized once (Sec. 4, quantization paragraph) and then
// laid out so that the GEMM streams them with no index arithmetic. The
// weight [n, k] is cut into panels of 32 rows (n rounded up to 32 with zero
// rows) and each panel into chunks of 128 reduction elements. Inside a chunk
// the 64 lanes of a wavefront each own one row r = l % 32 and one contiguous
// half of the chunk's reduction range, g = l / 32 -- the operand order of the
// 32x32 MFMAs once the reduction index is permuted the same way for both
// operands. A lane's bytes are split into 16-byte pieces h, stored as
// [h][lane][16 B], so that each piece is one contiguous 1 KiB wave access:
//   FP8  : 4096-byte chunk made of two 2048-byte steps of 64 reduction
//          elements; in step t, piece h of lane l = row r, bytes
//          64 t + 32 g + 16 h (each step is one self-contained MFMA operand);
//   NVFP4: 2048-byte code chunk, piece h of lane l = row r, bytes 32 g + 16 h;
//          block scales in their own region, 256 bytes per chunk = [row][8].
//   MXFP4: per 64-wide step t one 1024-byte image [lane][16 B], lane l = row
//          r, elements 64 t + 32 g .. + 31 (bytes 32 t + 16 g): exactly one
//          32-element scale block per lane, the operand of a scaled fp4 MFMA;
//          E8M0 scales in their own region, per 256-wide chunk c one run of
//          4 bytes per lane = the scales of the lane's blocks in steps
//          4c .. 4c + 3 (blocks 8c + 2s + g), read as one dword per lane.
//   MXFP8: 2048-byte step images like FP8, but lane half g and register
//          half h hold elements 64 t + 32 h + 16 g .. + 15: the block-scaled
//          fp8 instruction reads scale block h of a row from register half h
//          of both lane halves (its fp8 reduction order), so each of the
//          row's two 32-element scale blocks of the step must sit there; the
//          MXFP4 scale region (lane half g carries the scale of block 2 t + g).
// Chunks of one panel follow each other along k, so a panel is one
// contiguous stream. The header keeps format, n, k and the tensor scale
// (1.0 for the MX formats, which have none).
#include <algorithm>

#include "common.hpp"
#include "kernels.hpp"

namespace qg {

// One launch packs (or unpacks) codes, block scales and header. Memory-bound:
// 2 x the weight's bytes. A workgroup's 256 threads are 8 neighbouring pieces of
// each of the panel's 32 rows, so a wave reads whole 128-byte runs of 8 rows and
// writes 128-byte runs of the packed images (8 rows of one piece), and the panel
// and column come from the grid, with no division. Against a thread per packed
// piece (a wave reading 16 bytes of each of 64 places, two 64-bit divisions) in
// three launches, NVFP4 9216 x 3072: 11.5 us of kernels -> 7.6, unpack
// 12.1 -> 7.8 us.

// Byte offset inside a panel's packed codes of the 16-byte piece at byte o of
// its row r (see the layout above).
template <int FMT>
__device__ inline int64_t packed_piece(int64_t o, int r) {
  const int h16 = (int)(o >> 4) & 1, h32 = (int)(o >> 5) & 1, h64 = (int)(o >> 6) & 1;
  if (FMT == 1) return (o >> 7) * 4096 + h64 * 2048 + h16 * 1024 + (32 * h32 + r) * 16;
  if (FMT == 4) return (o >> 7) * 4096 + h64 * 2048 + h32 * 1024 + (32 * h16 + r) * 16;
  if (FMT == 2) return (o >> 6) * 2048 + h16 * 1024 + (32 * h32 + r) * 16;
  return (o >> 5) * 1024 + (32 * h16 + r) * 16;
}

constexpr int kPackSegs = 2;  // 128-byte column segments per workgroup, loaded together

template <int FMT, bool PACK>
__global__ void __launch_bounds__(256) k_pack(uint8_t* canon, uint8_t* bscale, float* tscale, int64_t n, int64_t k,
                                              int64_t panels, int64_t code_blocks, uint8_t* packed) {
  constexpr bool MX = FMT == 3 || FMT == 4;
  if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) {
    float* scale = reinterpret_cast<float*>(packed + kPackScaleOffset);
    if (PACK) {
      uint32_t* h = reinterpret_cast<uint32_t*>(packed);
      h[0] = kPackMagic;
      h[1] = kPackVersion;
      h[2] = (uint32_t)FMT;
      h[3] = 0u;
      reinterpret_cast<int64_t*>(packed)[2] = n;
      reinterpret_cast<int64_t*>(packed)[3] = k;
      *scale = tscale ? *tscale : 1.0f;
    } else if (tscale) {
      *tscale = *scale;
    }
  }
  const int64_t rb = (FMT == 1 || FMT == 4) ? k : k / 2;  // code bytes of a row, a multiple of 64
  uint8_t* codes = packed + kPackHeader;
  const int r = threadIdx.x >> 3, j = threadIdx.x & 7;
  for (int64_t panel = blockIdx.y; panel < panels; panel += gridDim.y) {
    const int64_t row = panel * 32 + r;
    const bool live = row < n;
    if ((int64_t)blockIdx.x < code_blocks) {
      uint8_t* c = canon + row * rb;
      uint8_t* p = codes + panel * 32 * rb;
      uint4 v[kPackSegs];
#pragma unroll
      for (int s = 0; s < kPackSegs; ++s) {
        const int64_t o = ((int64_t)blockIdx.x * kPackSegs + s) * 128 + 16 * j;
        v[s] = make_uint4(0u, 0u, 0u, 0u);
        if (o < rb && (live || !PACK))
          v[s] = *reinterpret_cast<const uint4*>(PACK ? c + o : p + packed_piece<FMT>(o, r));
      }
#pragma unroll
      for (int s = 0; s < kPackSegs; ++s) {
        const int64_t o = ((int64_t)blockIdx.x * kPackSegs + s) * 128 + 16 * j;
        if (o < rb && (live || PACK)) *reinterpret_cast<uint4*>(PACK ? p + packed_piece<FMT>(o, r) : c + o) = v[s];
      }
    } else if (FMT == 2) {  // 8-byte scale run of row r in 128-wide chunk kc
      const int64_t kc = ((int64_t)blockIdx.x - code_blocks) * 8 + j, kcn = k / 128;
      if (kc >= kcn) continue;
      uint2* c = reinterpret_cast<uint2*>(bscale + row * (k / 16)) + kc;
      uint2* p = reinterpret_cast<uint2*>(codes + panels * 32 * rb) + (panel * kcn + kc) * 32 + r;
      if (PACK) *p = live ? *c : make_uint2(0u, 0u);
      else if (live) *c = *p;
    } else if (MX) {  // the 8 scale bytes of row r in 256-wide chunk kc: blocks 2 s + g to byte s of lane 32 g + r
      const int64_t kc = ((int64_t)blockIdx.x - code_blocks) * 8 + j, kcn = k / 256;
      if (kc >= kcn) continue;
      uint8_t* c = bscale + row * (k / 32) + 8 * kc;
      uint32_t* p = reinterpret_cast<uint32_t*>(codes + panels * 32 * rb) + (panel * kcn + kc) * 64 + r;
      if (PACK) {
        uint32_t w[2] = {0u, 0u};
        if (live)
          for (int s = 0; s < 4; ++s) {
            w[0] |= (uint32_t)c[2 * s] << (8 * s);
            w[1] |= (uint32_t)c[2 * s + 1] << (8 * s);
          }
        p[0] = w[0];
        p[32] = w[1];
      } else if (live) {
        const uint32_t w[2] = {p[0], p[32]};
        for (int s = 0; s < 4; ++s) {
          c[2 * s] = (uint8_t)(w[0] >> (8 * s));
          c[2 * s + 1] = (uint8_t)(w[1] >> (8 * s));
        }
      }
    }
  }
}

template <bool PACK>
static hipError_t launch(int fmt, uint8_t* codes, uint8_t* bscale, float* tscale, int64_t n, int64_t k,
                         uint8_t* packed, hipStream_t st) {
  const bool empty = packed_codes_bytes(fmt, n, k) == 0;  // the header alone
  const int64_t panels = empty ? 0 : padded_rows(n) / 32;
  const int64_t rb = (fmt == 1 || fmt == 4) ? k : k / 2;
  const int64_t code_blocks = empty ? 0 : (rb + 128 * kPackSegs - 1) / (128 * kPackSegs);
  const int64_t chunks = (fmt == 2) ? k / 128 : (fmt == 1 || empty) ? 0 : k / 256;  // 8 a workgroup
  const dim3 grid((unsigned)std::max<int64_t>(1, code_blocks + (chunks + 7) / 8),
                  (unsigned)std::max<int64_t>(1, std::min<int64_t>(panels, 65535)));
  switch (fmt) {
    case 1: hipLaunchKernelGGL((k_pack<1, PACK>), grid, dim3(256), 0, st, codes, bscale, tscale, n, k, panels, code_blocks, packed); break;
    case 2: hipLaunchKernelGGL((k_pack<2, PACK>), grid, dim3(256), 0, st, codes, bscale, tscale, n, k, panels, code_blocks, packed); break;
    case 3: hipLaunchKernelGGL((k_pack<3, PACK>), grid, dim3(256), 0, st, codes, bscale, tscale, n, k, panels, code_blocks, packed); break;
    default: hipLaunchKernelGGL((k_pack<4, PACK>), grid, dim3(256), 0, st, codes, bscale, tscale, n, k, panels, code_blocks, packed); break;
  }
  return hipGetLastError();
}

hipError_t launch_pack(int fmt, const uint8_t* codes, const uint8_t* bscale, const float* tscale,
                       int64_t n, int64_t k, uint8_t* packed, hipStream_t st) {
  return launch<true>(fmt, const_cast<uint8_t*>(codes), const_cast<uint8_t*>(bscale), const_cast<float*>(tscale), n, k,
                      packed, st);
}

hipError_t launch_unpack(int fmt, const uint8_t* packed, int64_t n, int64_t k, uint8_t* codes,
                         uint8_t* bscale, float* tscale, hipStream_t st) {
  return launch<false>(fmt, codes, bscale, tscale, n, k, const_cast<uint8_t*>(packed), st);
}

}  // namespace qg
