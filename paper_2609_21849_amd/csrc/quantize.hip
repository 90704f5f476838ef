// quantize.hip -- activation/weight quantizers and dequantizers (gfx950).
//
// Dynamic per-tensor quantization of bf16 tensors to FP8 E4M3 and to NVFP4
// (E2M1 elements, E4M3 scale per 16 consecutive elements, fp32 tensor
// scale), the run-time activation quantization that the paper's recipe
// relies on for its speed-up on compute-bound stages (Sec. 4, quantization
// paragraph; Table 2). The same kernels quantize weights offline (PTQ).
//
// A tensor-wide scale needs the tensor-wide max before any element can be
// coded. A small tensor (at most 3072 units of 16 elements) is quantized in
// one launch (k_quant_small); one of at most 3 Mi elements whose rows are 16-byte
// aligned and whole 8-element units (dense, or a column slice) in two
// (k_amax_slots, k_quant_slots: the maxima handed over inside the code
// buffer); any other is a short chain on the caller's stream:
//   k_amax_units / : max |x| as an integer max of bf16 magnitude bits (the
//   k_amax_partial   bit pattern of a non-negative value orders like the
//                    value); one partial per workgroup, parked in the code
//                    buffer that the last kernel overwrites anyway
//   k_finalize     : max of the partials -> decode scale s or s_t
//   k_quant_*      : code the elements with the finished scale
// Stream order separates the kernels; nothing waits on the host.
#include "common.hpp"
#include "kernels.hpp"
#include "quant_plan.hpp"

namespace qg {

__global__ void k_fill_u32(uint32_t* p, uint32_t v) { *p = v; }

// ---------------------------------------------------------------- units of 8
// 16-byte unit u of a tensor (UnitRows in quant_plan.hpp); DENSE: ldx == cols.
template <bool DENSE>
__device__ inline uint4 load_unit(const uint4* __restrict__ x, int64_t u, const UnitRows& r) {
  if (DENSE) return x[u];
  const uint32_t row = r.row_of((uint32_t)u);
  return x[(int64_t)row * r.pitch + ((uint32_t)u - row * r.upr)];
}

// ---------------------------------------------------------------- amax
// Rows of `cols` bf16 elements, `ldx` apart, of any alignment. Each workgroup
// writes the bf16 magnitude bits of its max to partial[id]; there are no
// atomics, so thousands of workgroups do not serialise on one address.
// k_finalize reduces the partials.
__global__ void __launch_bounds__(256) k_amax_partial(const uint16_t* __restrict__ x, int64_t rows,
                                                      int64_t cols, int64_t ldx,
                                                      uint32_t* __restrict__ partial) {
  uint32_t m = 0;
  const int64_t stride = (int64_t)gridDim.x * 256;
  for (int64_t r = blockIdx.y; r < rows; r += gridDim.y) {
    const uint16_t* xr = x + r * ldx;
    for (int64_t c = (int64_t)blockIdx.x * 256 + threadIdx.x; c < cols; c += stride)
      m = max(m, (uint32_t)(xr[c] & 0x7FFFu));
  }
  for (int off = 32; off > 0; off >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, off));
  __shared__ uint32_t part[4];
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0)
    partial[blockIdx.y * gridDim.x + blockIdx.x] = max(max(part[0], part[1]), max(part[2], part[3]));
}

// 16-byte aligned rows of whole 8-element units: a grid of at most
// kAmaxGroups workgroups strides over blocks of 1024 units, each block read
// as four wave-contiguous runs with all four 16-byte loads of a thread issued
// before the first max. Measured against one-shot grids (every workgroup one
// block of 1024, 2048 or 4096 units): 3.5 us faster on a dense 4608 x 3072
// activation, 1.3 us on 4608 x 9216. The same columns as a slice of 9216-wide
// rows: 6.7 -> 4.4 us against a workgroup per row (kernel trace).
constexpr int64_t kAmaxGroups = 1024;  // four workgroups per CU on 256 CUs

template <bool DENSE>
__global__ void __launch_bounds__(256) k_amax_units(const uint16_t* __restrict__ x, int64_t units, UnitRows rows,
                                                    uint32_t* __restrict__ partial) {
  constexpr int U = 4;
  const uint4* xv = reinterpret_cast<const uint4*>(x);
  uint32_t m = 0;
  for (int64_t base = (int64_t)blockIdx.x * 256 * U + threadIdx.x; base < units; base += (int64_t)gridDim.x * 256 * U) {
    uint4 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u)
      v[u] = (base + u * 256 < units) ? load_unit<DENSE>(xv, base + u * 256, rows) : make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t w[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const uint32_t t = w[i] & 0x7FFF7FFFu;
        m = max(m, max(t & 0xFFFFu, t >> 16));
      }
    }
  }
  for (int off = 32; off > 0; off >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, off));
  __shared__ uint32_t part[4];
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) partial[blockIdx.x] = max(max(part[0], part[1]), max(part[2], part[3]));
}

// Max of `count` partials (bf16 magnitude bits) -> decode scale, written to
// `slot`. divisor = 448 (FP8) or 2688 = 448 * 6 (NVFP4). Inf/NaN anywhere in
// the tensor leaves a NaN scale as the sentinel. `partial` may be `slot`
// itself (count 1): every read happens before the barrier, the write after.
__global__ void __launch_bounds__(256) k_finalize(const uint32_t* partial, int count, float* slot,
                                                  float divisor) {
  // eight loads per thread in flight at once: the partials were just written
  // by workgroups on every XCD, so each round trip is a far-cache latency
  constexpr int U = 8;
  uint32_t m = 0;
  for (int base = 0; base < count; base += 256 * U) {
    uint32_t v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = base + u * 256 + (int)threadIdx.x;
      v[u] = (i < count) ? partial[i] : 0u;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) m = max(m, v[u]);
  }
  for (int off = 32; off > 0; off >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, off));
  __shared__ uint32_t part[4];
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    const uint32_t a = max(max(part[0], part[1]), max(part[2], part[3])) << 16;
    *slot = (a >= 0x7F800000u) ? __builtin_nanf("") : __fdiv_rn(u2f(a), divisor);
  }
}

// ---------------------------------------------------------------- units of 16
// A unit: cnt (<= 16) consecutive bf16 of a row, held as 8 words (element
// 2 i in the low half of word i, missing elements zero). VEC: the unit is
// whole and 16-byte aligned (two 16-byte loads).
template <bool VEC>
__device__ inline void unit_load(const uint16_t* __restrict__ p, int64_t cnt, uint32_t (&w)[8]) {
  if (VEC && cnt == 16) {
    const uint4 a = reinterpret_cast<const uint4*>(p)[0], b = reinterpret_cast<const uint4*>(p)[1];
    w[0] = a.x; w[1] = a.y; w[2] = a.z; w[3] = a.w; w[4] = b.x; w[5] = b.y; w[6] = b.z; w[7] = b.w;
  } else {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const uint32_t lo = (2 * i < cnt) ? (uint32_t)p[2 * i] : 0u;
      const uint32_t hi = (2 * i + 1 < cnt) ? (uint32_t)p[2 * i + 1] : 0u;
      w[i] = lo | (hi << 16);
    }
  }
}

// FP8 codes of a unit: q = E4M3(x * r) by the hardware conversion (hw_e4m3x4,
// equal to enc_e4m3 on every finite input); one 16-byte store when vec_store
// (whole unit, 16-byte aligned destination), else byte stores.
__device__ inline void fp8_words(const uint32_t (&w)[8], uint32_t (&c)[4], float r) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float y[4] = {__fmul_rn(bf16_lo(w[2 * i]), r), __fmul_rn(bf16_hi(w[2 * i]), r),
                        __fmul_rn(bf16_lo(w[2 * i + 1]), r), __fmul_rn(bf16_hi(w[2 * i + 1]), r)};
    c[i] = hw_e4m3x4(y);
  }
}

__device__ inline void quant_fp8_words(const uint32_t (&w)[8], int64_t cnt, uint8_t* __restrict__ dst, float r,
                                       bool vec_store) {
  uint32_t c[4];
  fp8_words(w, c, r);
  if (vec_store && cnt == 16) {
    *reinterpret_cast<uint4*>(dst) = make_uint4(c[0], c[1], c[2], c[3]);
  } else {
    for (int64_t i = 0; i < cnt; ++i) dst[i] = (uint8_t)((c[i >> 2] >> (8 * (i & 3))) & 0xFFu);
  }
}

// NVFP4 block of a whole unit: block max, E4M3 block scale (returned), then
// the 16 E2M1 codes packed into 8 bytes at q8 (element 2i in the low nibble;
// hardware conversion hw_e2m1x8, equal to enc_e2m1 on every input).
__device__ inline uint32_t quant_nvfp4_words(const uint32_t (&w)[8], uint8_t* __restrict__ q8, float s_t) {
  float v[16];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    v[2 * i] = bf16_lo(w[i]);
    v[2 * i + 1] = bf16_hi(w[i]);
  }
  uint32_t amax_bits = 0;
#pragma unroll
  for (int i = 0; i < 16; ++i) amax_bits = max(amax_bits, f2u(v[i]) & 0x7FFFFFFFu);
  const float d_t = __fmul_rn(6.0f, s_t);
  const float vb = (d_t > 0.0f) ? __fdiv_rn(u2f(amax_bits), d_t) : 0.0f;
  const uint32_t sb = enc_e4m3(vb);
  const float S = __fmul_rn(dec_e4m3(sb), s_t);
  const float r = (S > 0.0f) ? __fdiv_rn(1.0f, S) : 0.0f;
  float y[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) y[i] = __fmul_rn(v[i], r);
  *reinterpret_cast<uint2*>(q8) = make_uint2(hw_e2m1x8(y), hw_e2m1x8(y + 8));
  return sb;
}

// ---------------------------------------------------------------- FP8

// One thread codes 16 consecutive elements of a row: q = E4M3(x * r), r = 1/s.
// CONTIG: the tensor is one dense run of n elements (ldx == cols); a thread
// owns elements [16 t, 16 t + 16) and the last thread may be partial.
// Otherwise rows are handled as units of 16. Rows of any alignment.
template <bool CONTIG>
__global__ void __launch_bounds__(256) k_quant_fp8(const uint16_t* __restrict__ x, int64_t rows,
                                                   int64_t cols, int64_t ldx,
                                                   uint8_t* __restrict__ q,
                                                   const float* __restrict__ scale) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const float s = *scale;
  const float r = (s > 0.0f) ? __fdiv_rn(1.0f, s) : 0.0f;
  int64_t src, dst, cnt;
  if (CONTIG) {
    const int64_t n = rows * cols;
    src = dst = t * 16;
    if (src >= n) return;
    cnt = min((int64_t)16, n - src);
  } else {
    const int64_t upr = (cols + 15) >> 4;
    const int64_t row = t / upr, u = t - row * upr;
    if (row >= rows) return;
    src = row * ldx + u * 16;
    dst = row * cols + u * 16;
    cnt = min((int64_t)16, cols - u * 16);
  }
  uint32_t w[8];
  unit_load<false>(x + src, cnt, w);
  quant_fp8_words(w, cnt, q + dst, r, false);
}

// ---------------------------------------------------------------- NVFP4
// One thread per 16-element block; rows of any alignment.
template <bool CONTIG>
__global__ void __launch_bounds__(256) k_quant_nvfp4(const uint16_t* __restrict__ x, int64_t rows,
                                                     int64_t cols, int64_t ldx,
                                                     uint8_t* __restrict__ q,
                                                     uint8_t* __restrict__ bscale,
                                                     const float* __restrict__ tscale) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t bpr = cols >> 4;
  int64_t src;
  if (CONTIG) {
    if (t >= rows * bpr) return;
    src = t * 16;
  } else {
    const int64_t row = t / bpr, b = t - row * bpr;
    if (row >= rows) return;
    src = row * ldx + b * 16;
  }
  uint32_t w[8];
  unit_load<false>(x + src, 16, w);
  bscale[t] = (uint8_t)quant_nvfp4_words(w, q + t * 8, *tscale);
}

// ---------------------------------------------------------------- small tensors
// The whole dynamic quantization of a small tensor (at most 3072 units of 16
// elements) in one launch: every workgroup loads the whole tensor into
// registers (up to three units per thread) and reduces its max; workgroup b
// of G codes its G-th of the units from the same registers -- one launch
// instead of the three-kernel chain, whose launch latencies dominate at these
// sizes, with the coding and the stores spread over G CUs. The same arithmetic
// as the chain, so the same bits: the max of the bf16 magnitude bits,
// s = fl(amax / 448) or fl(amax / 2688) (NaN if the tensor holds inf or NaN),
// then the unit helpers above. FP8 rows may end in a shorter unit; NVFP4
// rows are whole blocks. VEC: 16-byte aligned rows of a multiple of 8
// elements; vec_store (FP8): 16-byte aligned codes and cols % 16 == 0.
constexpr int kSmallPerThread = 3;
constexpr int64_t kSmallUnits = 1024 * kSmallPerThread;
constexpr int64_t kSmallGroups = 8;  // workgroups that share the coding

template <int FMT, bool VEC>
__global__ void __launch_bounds__(1024) k_quant_small(const uint16_t* __restrict__ x, int64_t rows, int64_t cols,
                                                      int64_t ldx, uint8_t* __restrict__ q,
                                                      uint8_t* __restrict__ bscale, float* __restrict__ tscale,
                                                      bool vec_store) {
  // at most kSmallUnits units: 32-bit unit arithmetic
  const int upr = (int)((cols + 15) >> 4);
  const int units = (int)rows * upr;
  uint32_t w[kSmallPerThread][8];
#pragma unroll
  for (int i = 0; i < kSmallPerThread; ++i) {
    const int u = (int)threadIdx.x + 1024 * i;
    if (u < units) {
      const int row = u / upr, c = (u - row * upr) * 16;
      unit_load<VEC>(x + (int64_t)row * ldx + c, min((int64_t)16, cols - c), w[i]);
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j) w[i][j] = 0u;
    }
  }
  uint32_t m = 0;
#pragma unroll
  for (int i = 0; i < kSmallPerThread; ++i)
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const uint32_t t = w[i][j] & 0x7FFF7FFFu;
      m = max(m, max(t & 0xFFFFu, t >> 16));
    }
  for (int off = 32; off > 0; off >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, off));
  __shared__ uint32_t part[16];
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = m;
  __syncthreads();
  uint32_t a = 0;
#pragma unroll
  for (int i = 0; i < 16; ++i) a = max(a, part[i]);
  a <<= 16;
  const float s = (a >= 0x7F800000u) ? __builtin_nanf("") : __fdiv_rn(u2f(a), FMT == 1 ? 448.0f : 2688.0f);
  if (blockIdx.x == 0 && threadIdx.x == 0) *tscale = s;
  // every workgroup reduces the whole tensor; workgroup b codes the units
  // [b U / G, (b + 1) U / G) of the U units (G workgroups)
  const int lo = gridDim.x == 1 ? 0 : units * (int)blockIdx.x / (int)gridDim.x;
  const int hi = gridDim.x == 1 ? units : units * ((int)blockIdx.x + 1) / (int)gridDim.x;
  const float r = (FMT == 1 && s > 0.0f) ? __fdiv_rn(1.0f, s) : 0.0f;
#pragma unroll
  for (int i = 0; i < kSmallPerThread; ++i) {
    const int u = (int)threadIdx.x + 1024 * i;
    if (u < lo || u >= hi) continue;
    const int row = u / upr, c = (u - row * upr) * 16;
    if (FMT == 1) quant_fp8_words(w[i], min((int64_t)16, cols - c), q + (int64_t)row * cols + c, r, vec_store);
    else bscale[u] = (uint8_t)quant_nvfp4_words(w[i], q + (int64_t)u * 8, s);
  }
}

// ---------------------------------------------------------------- whole units, aligned rows
// FP8 codes of one whole 16-byte unit (8 consecutive elements, index u)
// held in `raw`: one 8-byte store, gated by `in`.
__device__ inline void code_unit8_fp8(const uint4 raw, int64_t u, bool in, uint8_t* __restrict__ q, float r) {
  const uint32_t ww[4] = {raw.x, raw.y, raw.z, raw.w};
  float y[8];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    y[2 * j] = __fmul_rn(bf16_lo(ww[j]), r);
    y[2 * j + 1] = __fmul_rn(bf16_hi(ww[j]), r);
  }
  const uint32_t lo = hw_e4m3x4(y), hi = hw_e4m3x4(y + 4);
  if (in) *reinterpret_cast<uint2*>(q + u * 8) = make_uint2(lo, hi);
}

// NVFP4 codes of two whole units per lane from two load steps: lanes 2j and
// 2j+1 hold the halves of block A (units u[0]) and of block B (units u[1]);
// the even lane derives A's scale, the odd lane B's, so each lane does one
// block's two divisions for two blocks' worth of elements, and the two
// reciprocals are swapped across the pair. Every lane of the wave calls it
// together; in[] only gates the stores. The arithmetic of quant_nvfp4_words.
__device__ inline void code_units8_nv_pair(const uint4 (&raw)[2], const int64_t (&u)[2], const bool (&in)[2],
                                           uint8_t* __restrict__ q, uint8_t* __restrict__ bscale, float s,
                                           float d_t, int lane) {
  float v[2][8];
  uint32_t am[2];
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    const uint32_t ww[4] = {raw[p].x, raw[p].y, raw[p].z, raw[p].w};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      v[p][2 * j] = bf16_lo(ww[j]);
      v[p][2 * j + 1] = bf16_hi(ww[j]);
    }
    uint32_t a = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) a = max(a, f2u(v[p][j]) & 0x7FFFFFFFu);
    am[p] = max(a, (uint32_t)__shfl_xor((int)a, 1));
  }
  const bool odd = lane & 1;
  const float vb = (d_t > 0.0f) ? __fdiv_rn(u2f(odd ? am[1] : am[0]), d_t) : 0.0f;
  const uint32_t sb = enc_e4m3(vb);
  const float S = __fmul_rn(dec_e4m3(sb), s);
  const float rb = (S > 0.0f) ? __fdiv_rn(1.0f, S) : 0.0f;
  const float rp = __shfl_xor(rb, 1);
  const float rr[2] = {odd ? rp : rb, odd ? rb : rp};
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    float y[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) y[j] = __fmul_rn(v[p][j], rr[p]);
    const uint32_t w = hw_e2m1x8(y);
    if (in[p]) {
      *reinterpret_cast<uint32_t*>(q + u[p] * 4) = w;
      if (odd == (p == 1)) bscale[u[p] >> 1] = (uint8_t)sb;
    }
  }
}

// 16-byte aligned rows of whole 8-element units (dense FP8 tensors may end in a
// shorter one): each lane codes H blocks of 16 consecutive elements, 64 blocks
// apart (two adjacent 16-byte loads each, all issued before the first is used),
// and writes FP8 codes with one 16-byte store, NVFP4 with an 8-byte store and
// its scale byte. HBM-bound. H: one where the scale is the caller's, two in the
// dynamic chain, where every wave waits for the scale the kernel before just
// wrote (4608 x 3072 FP8, static: H = 1 7.4 us, H = 2 7.8; chain 15.9 and 14.0).
// Against lanes of 8 elements (8-byte stores, a block's two divisions shared
// over a lane pair), four loads apart: static FP8 4608 x 3072 8.4 -> 7.4 us,
// 512 x 3072 2.7 -> 2.4, NVFP4 8.1 -> 7.3; chain 14.3 -> 14.0, 14.6 -> 14.2.
// PLAIN: whole blocks and 16-byte aligned codes (NVFP4 always); behind run-time
// branches in one kernel the FP8 case lost half of that (7.4 -> 8.2 us).
// Otherwise whole 8-element units in 8-byte stores and the last 1 to 7 elements of
// a dense tensor one by one (the whole last block element by element, in a loop,
// held its wave up: static 1 x 1032 3.4 us, now 2.8; 63 x 1000 3.7, now 3.0).
template <int FMT, int H, bool DENSE, bool PLAIN>
__global__ void __launch_bounds__(256) k_quant_units(const uint16_t* __restrict__ x, int64_t n, UnitRows rows,
                                                     uint8_t* __restrict__ q, uint8_t* __restrict__ bscale,
                                                     const float* __restrict__ tscale) {
  const int64_t b0 = (((int64_t)blockIdx.x * 256 + threadIdx.x) >> 6) * (64 * H) + (threadIdx.x & 63);
  const uint4* xv = reinterpret_cast<const uint4*>(x);
  uint32_t w[H][8];
#pragma unroll
  for (int h = 0; h < H; ++h) {
    const int64_t e = 16 * (b0 + 64 * h);
    const uint4 lo = (e + (PLAIN ? 16 : 8) <= n) ? load_unit<DENSE>(xv, e >> 3, rows) : make_uint4(0u, 0u, 0u, 0u);
    const uint4 hi = (e + 16 <= n) ? load_unit<DENSE>(xv, (e >> 3) + 1, rows) : make_uint4(0u, 0u, 0u, 0u);
    w[h][0] = lo.x; w[h][1] = lo.y; w[h][2] = lo.z; w[h][3] = lo.w;
    w[h][4] = hi.x; w[h][5] = hi.y; w[h][6] = hi.z; w[h][7] = hi.w;
  }
  const float s = *tscale;
  const float r = (FMT == 1 && s > 0.0f) ? __fdiv_rn(1.0f, s) : 0.0f;
#pragma unroll
  for (int h = 0; h < H; ++h) {
    const int64_t b = b0 + 64 * h, left = n - 16 * b;
    if (left <= 0) continue;
    if (FMT == 2) {
      bscale[b] = (uint8_t)quant_nvfp4_words(w[h], q + 8 * b, s);
      continue;
    }
    uint32_t c[4];
    fp8_words(w[h], c, r);
    if (PLAIN) {
      *reinterpret_cast<uint4*>(q + 16 * b) = make_uint4(c[0], c[1], c[2], c[3]);
      continue;
    }
    if (left >= 8) reinterpret_cast<uint2*>(q + 16 * b)[0] = make_uint2(c[0], c[1]);
    if (left >= 16) reinterpret_cast<uint2*>(q + 16 * b)[1] = make_uint2(c[2], c[3]);
    if (DENSE && left < 16 && (left & 7) != 0) {  // the tensor ends in part of a unit
      const int64_t e = 16 * b + (left & 8);
      const int cnt = (int)(left & 7);
      float y[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) y[j] = (j < cnt) ? __fmul_rn(u2f((uint32_t)x[e + j] << 16), r) : 0.0f;
      const uint32_t t[2] = {hw_e4m3x4(y), hw_e4m3x4(y + 4)};
#pragma unroll
      for (int j = 0; j < 7; ++j)
        if (j < cnt) q[e + j] = (uint8_t)(t[j >> 2] >> (8 * (j & 3)));
    }
  }
}

// ---------------------------------------------------------------- two launches
// Dynamic quantization without the one-workgroup finalize kernel, of a dense
// tensor or of aligned rows of whole units (DENSE false). k_amax_slots leaves each of its P workgroup maxima not in one
// place but in every code region of the quantize launch (slot i among the
// first 4 P bytes of each region); each workgroup of k_quant_slots
// reduces the P maxima found at the start of its own region to the tensor
// scale before any of its codes overwrite them. No workgroup reads what
// another writes within a launch, so stream order between the two launches
// is the only synchronisation, and the caller's code buffer the only memory.
// Region j of G: the 16-byte units [slot_region_lo(j), slot_region_lo(j + 1))
// of the n / 8 (the last region ends at n / 8), whose codes start at byte CB
// times their first unit (CB = 8 for FP8, 4 for NVFP4). The host picks G so
// that every region's codes hold the 4 P bytes of slots.
// (the plan: slot_region_lo, slots_plan and their limits in quant_plan.hpp)

template <int U, bool DENSE>
__global__ void __launch_bounds__(256) k_amax_slots(const uint16_t* __restrict__ x, int64_t units, UnitRows rows,
                                                    uint8_t* __restrict__ q, int cb, int gq) {
  const uint4* xv = reinterpret_cast<const uint4*>(x);
  uint32_t m = 0;
  for (int64_t base = (int64_t)blockIdx.x * 256 * U + threadIdx.x; base < units; base += (int64_t)gridDim.x * 256 * U) {
    uint4 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u)
      v[u] = (base + u * 256 < units) ? load_unit<DENSE>(xv, base + u * 256, rows) : make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t w[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const uint32_t t = w[i] & 0x7FFF7FFFu;
        m = max(m, max(t & 0xFFFFu, t >> 16));
      }
    }
  }
  for (int off = 32; off > 0; off >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, off));
  __shared__ uint32_t part[4];
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = m;
  __syncthreads();
  const uint32_t mw = max(max(part[0], part[1]), max(part[2], part[3]));
  // workgroup b runs on XCD b mod 8: with the slots ordered XCD-major, the
  // maxima of one XCD's workgroups fill whole cache lines of each region
  const int P = (int)gridDim.x, b = (int)blockIdx.x;
  const int slot = (P % 8 == 0) ? (b % 8) * (P / 8) + b / 8 : b;
  const int64_t pairs = units >> 1;
  for (int j = (int)threadIdx.x; j < gq; j += 256)
    reinterpret_cast<uint32_t*>(q + slot_region_lo(pairs, j, gq) * cb)[slot] = mw;
}

// Each wave codes runs of 64 consecutive units (one 16-byte load per lane,
// four per lane in flight); rounds of 1024 units until the region ends.
template <int FMT, bool DENSE>
__global__ void __launch_bounds__(256) k_quant_slots(const uint16_t* __restrict__ x, int64_t units, UnitRows rows,
                                                           uint8_t* __restrict__ q, uint8_t* __restrict__ bscale,
                                                           float* __restrict__ tscale, int P) {
  constexpr int H = 4;
  constexpr int CB = FMT == 1 ? 8 : 4;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int64_t pairs = units >> 1;
  const int64_t lo = slot_region_lo(pairs, blockIdx.x, gridDim.x);
  const int64_t hi = (blockIdx.x + 1 == gridDim.x) ? units : slot_region_lo(pairs, blockIdx.x + 1, gridDim.x);
  const uint4* xv = reinterpret_cast<const uint4*>(x);
  uint4 raw[H];
#pragma unroll
  for (int h = 0; h < H; ++h) {
    const int64_t u = lo + 256 * wv + 64 * h + lane;
    raw[h] = (u < hi) ? load_unit<DENSE>(xv, u, rows) : make_uint4(0u, 0u, 0u, 0u);
  }
  // the tensor max from this region's slots, all read before the barrier
  const uint32_t* slots = reinterpret_cast<const uint32_t*>(q + lo * CB);
  uint32_t m = 0;
  for (int i = (int)threadIdx.x; i < P; i += 256) m = max(m, slots[i]);
  for (int off = 32; off > 0; off >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, off));
  __shared__ uint32_t part[4];
  if (lane == 0) part[wv] = m;
  __syncthreads();
  const uint32_t a = max(max(part[0], part[1]), max(part[2], part[3])) << 16;
  const float s = (a >= 0x7F800000u) ? __builtin_nanf("") : __fdiv_rn(u2f(a), FMT == 1 ? 448.0f : 2688.0f);
  if (blockIdx.x == 0 && threadIdx.x == 0) *tscale = s;
  const float r = (FMT == 1 && s > 0.0f) ? __fdiv_rn(1.0f, s) : 0.0f;
  const float d_t = __fmul_rn(6.0f, s);
  for (int64_t base = lo;;) {
    if constexpr (FMT == 2) {
#pragma unroll
      for (int h = 0; h < H; h += 2) {
        const int64_t u0 = base + 256 * wv + 64 * h + lane;
        const uint4 rw[2] = {raw[h], raw[h + 1]};
        const int64_t u[2] = {u0, u0 + 64};
        const bool in[2] = {u0 < hi, u0 + 64 < hi};
        code_units8_nv_pair(rw, u, in, q, bscale, s, d_t, lane);
      }
    } else {
#pragma unroll
      for (int h = 0; h < H; ++h) {
        const int64_t u = base + 256 * wv + 64 * h + lane;
        code_unit8_fp8(raw[h], u, u < hi, q, r);
      }
    }
    base += 1024;
    if (base >= hi) break;
#pragma unroll
    for (int h = 0; h < H; ++h) {
      const int64_t u = base + 256 * wv + 64 * h + lane;
      raw[h] = (u < hi) ? load_unit<DENSE>(xv, u, rows) : make_uint4(0u, 0u, 0u, 0u);
    }
  }
}

// ---------------------------------------------------------------- MX formats
// OCP MX (MXFP4: E2M1 elements, MXFP8: E4M3 elements), one E8M0 scale per 32
// consecutive elements of a row, no tensor scale: the block scaling gfx950's
// matrix cores consume natively. Shared exponent = floor(log2 max|x|) - emax
// (emax 2 for E2M1, 8 for E4M3), E8M0 code = that + 127 clamped to [0, 254],
// 0 for an all-zero block; elements = RNE_sat(x * 2^(127 - code)), the
// multiply exact (a power of two, inside the normal range for bf16 inputs).
// Rows hold whole blocks (cols % 32 == 0), so the four 8-element units of a
// block are units 4 j .. 4 j + 3 of the tensor and lanes 4 j .. 4 j + 3 of one
// wave, which share its max with two lane swaps.

// E8M0 code of a block from the fp32 bits of its largest magnitude and the
// factor its elements are multiplied by.
template <bool FP4>
__device__ inline uint32_t mx_block(uint32_t am, float& r) {
  // floor(log2(max)) from the fp32 bits (normal or denormal), then the code.
  // A block holding inf or NaN gets the E8M0 NaN code 255 (its element codes
  // are then unspecified: r = 0 makes them signed zeros).
  int e = 0;
  if (am >= 0x7F800000u) {
    e = 255;
  } else if (am != 0u) {
    const int ef = (int)(am >> 23);
    const int fl = (ef > 0) ? ef - 127 : (31 - __builtin_clz(am)) - 149;
    e = min(max(fl - (FP4 ? 2 : 8) + 127, 0), 254);
  }
  // 2^(127 - e); finite bf16 inputs give e <= 252, so this is a normal number
  r = (e == 255) ? 0.0f : u2f((uint32_t)(254 - e) << 23);
  return (uint32_t)e;
}

// 16-byte aligned rows. Each lane codes H half blocks of 16 elements, 64 apart
// (two adjacent 16-byte loads each, all issued before the first is used); a lane
// pair shares a block's max. Codes and scales are contiguous in unit order, so
// every store instruction of a wave covers one run. HBM-bound; against one unit
// of 8 per thread with a 64-bit division: MXFP4 4608 x 3072 8.5 -> 7.0 us, MXFP8
// 2800 x 3072 6.8 -> 5.7, 4608 x 9216 26.5 -> 23.9 (two half blocks per lane were
// 3-10% slower). PLAIN: codes aligned to a half block's (MXFP8 16 bytes, MXFP4 8;
// MXFP4 codes are always 4-byte aligned).
template <bool FP4, int H, bool DENSE, bool PLAIN>
__global__ void __launch_bounds__(256) k_quant_mx_units(const uint16_t* __restrict__ x, int64_t halves, UnitRows rows,
                                                        uint8_t* __restrict__ q, uint8_t* __restrict__ scales) {
  const int64_t b0 = (((int64_t)blockIdx.x * 256 + threadIdx.x) >> 6) * (64 * H) + (threadIdx.x & 63);
  const uint4* xv = reinterpret_cast<const uint4*>(x);
  uint32_t w[H][8];
#pragma unroll
  for (int h = 0; h < H; ++h) {
    uint4 lo = make_uint4(0u, 0u, 0u, 0u), hi = lo;
    if (b0 + 64 * h < halves) {
      lo = load_unit<DENSE>(xv, 2 * (b0 + 64 * h), rows);
      hi = load_unit<DENSE>(xv, 2 * (b0 + 64 * h) + 1, rows);
    }
    w[h][0] = lo.x; w[h][1] = lo.y; w[h][2] = lo.z; w[h][3] = lo.w;
    w[h][4] = hi.x; w[h][5] = hi.y; w[h][6] = hi.z; w[h][7] = hi.w;
  }
#pragma unroll
  for (int h = 0; h < H; ++h) {
    const int64_t b = b0 + 64 * h;
    uint32_t am = 0;  // bf16 magnitude bits
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const uint32_t t = w[h][j] & 0x7FFF7FFFu;
      am = max(am, max(t & 0xFFFFu, t >> 16));
    }
    am = max(am, (uint32_t)__shfl_xor((int)am, 1));
    float r;
    const uint32_t e = mx_block<FP4>(am << 16, r);
    if (b >= halves) continue;
    if (FP4) {
      float y[16];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        y[2 * j] = __fmul_rn(bf16_lo(w[h][j]), r);
        y[2 * j + 1] = __fmul_rn(bf16_hi(w[h][j]), r);
      }
      const uint32_t c0 = hw_e2m1x8(y), c1 = hw_e2m1x8(y + 8);
      if (PLAIN) {
        reinterpret_cast<uint2*>(q)[b] = make_uint2(c0, c1);
      } else {
        reinterpret_cast<uint32_t*>(q)[2 * b] = c0;
        reinterpret_cast<uint32_t*>(q)[2 * b + 1] = c1;
      }
    } else {
      quant_fp8_words(w[h], 16, q + 16 * b, r, PLAIN);
    }
    if ((b & 1) == 0) scales[b >> 1] = (uint8_t)e;
  }
}

// Rows of any alignment: one unit per thread. Its eight elements are loaded
// under one branch: with the condition on each of them the compiler made eight
// dependent 2-byte loads instead of one wide one (MXFP4 7029 x 3616 from an odd
// address 32.6 us, MXFP8 12705 x 1088 of 1152 20.4; 15.1 and 10.2 so).
template <bool FP4>
__global__ void __launch_bounds__(256) k_quant_mx(const uint16_t* __restrict__ x, int64_t rows, int64_t cols,
                                                  int64_t ldx, uint8_t* __restrict__ q,
                                                  uint8_t* __restrict__ scales) {
  const int64_t upr = cols >> 3;  // 8-element units per row
  const int64_t u = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const bool live = u < rows * upr;
  const int64_t row = live ? u / upr : 0, c8 = live ? u - row * upr : 0;
  float v[8];
  if (live) {
    const uint16_t* p = x + row * ldx + 8 * c8;
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = u2f((uint32_t)p[j] << 16);
  } else {
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = 0.0f;
  }
  uint32_t am = 0;
#pragma unroll
  for (int j = 0; j < 8; ++j) am = max(am, f2u(v[j]) & 0x7FFFFFFFu);
  am = max(am, (uint32_t)__shfl_xor((int)am, 1));
  am = max(am, (uint32_t)__shfl_xor((int)am, 2));
  float r;
  const uint32_t e = mx_block<FP4>(am, r);
  float y[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) y[j] = __fmul_rn(v[j], r);
  if (!live) return;
  if (FP4) {
    *reinterpret_cast<uint32_t*>(q + row * (cols >> 1) + 4 * c8) = hw_e2m1x8(y);
  } else {
    const uint32_t lo = hw_e4m3x4(y), hi = hw_e4m3x4(y + 4);
    uint8_t* d = q + row * cols + 8 * c8;
    if ((reinterpret_cast<uintptr_t>(d) & 7) == 0) *reinterpret_cast<uint2*>(d) = make_uint2(lo, hi);
    else for (int j = 0; j < 8; ++j) d[j] = (uint8_t)(((j < 4 ? lo : hi) >> (8 * (j & 3))) & 0xFFu);
  }
  if ((c8 & 3) == 0) scales[row * (cols >> 5) + (c8 >> 2)] = (uint8_t)e;
}

// ---------------------------------------------------------------- dequant
// out = fl(e4m3(q) * s), fl(fl(e2m1(q) * e4m3(s_b)) * s_t) or (MX) e * 2^(E - 127),
// as fp32 or RNE bf16; HBM-bound. One thread per 8 consecutive elements of the
// dense tensor, so that the 16-byte stores of a wave lie next to each other (bf16)
// or leave gaps that its next store fills (fp32). With 16 elements a thread they
// were 32 and 64 bytes apart: 9216 x 3072 to fp32 36.7 us (MXFP4), 37.8 (MXFP8),
// 36.8 (NVFP4), 45.3 (FP8), now 22.8, 24.1, 22.7 and 23.1 (5.5-6.1 TB/s); to bf16
// 16.4, 19.5, 15.3 and 19.3, now 13.4, 15.4, 13.0 and 14.4.
// Codes are decoded by the hardware conversions at unit scale (exact) and bf16
// results rounded by v_cvt_pk_bf16_f32; a thread that could produce a NaN (a NaN
// code or scale, an infinite scale) gives it the fixed bits of dec_e4m3 and
// f32_to_bf16. VEC: 16-byte aligned output (a template argument: behind a run-time
// one the compiler merged both forms into 4-byte stores, 71 us for NVFP4 to fp32).
template <bool F32OUT, bool VEC, bool NANS>
__device__ inline void store8(void* out, int64_t e, const float (&v)[8]) {
  if (F32OUT) {
    float* o = reinterpret_cast<float*>(out) + e;
    if (VEC) {
      reinterpret_cast<float4*>(o)[0] = make_float4(v[0], v[1], v[2], v[3]);
      reinterpret_cast<float4*>(o)[1] = make_float4(v[4], v[5], v[6], v[7]);
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i) o[i] = v[i];
    }
  } else {
    uint16_t* o = reinterpret_cast<uint16_t*>(out) + e;
    uint32_t w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
      w[i] = NANS ? f32_to_bf16(v[2 * i]) | (f32_to_bf16(v[2 * i + 1]) << 16) : pk_bf16(v[2 * i], v[2 * i + 1]);
    if (VEC) {
      *reinterpret_cast<uint4*>(o) = make_uint4(w[0], w[1], w[2], w[3]);
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i) o[i] = (uint16_t)(w[i >> 1] >> (16 * (i & 1)));
    }
  }
}

__device__ inline bool finite(float f) { return (f2u(f) & 0x7F800000u) != 0x7F800000u; }

// 8 E4M3 codes times s. A finite s and no NaN code (0x7F, 0xFF) leave no NaN;
// the NaN codes become the fp32 NaN of their sign.
template <bool F32OUT>
__device__ inline void dequant_e4m3x8(const uint2 c, float s, void* out, int64_t e) {
  const uint32_t w[2] = {c.x, c.y};
  const uint32_t nan = ((w[0] & 0x7F7F7F7Fu) + 0x01010101u) | ((w[1] & 0x7F7F7F7Fu) + 0x01010101u);
  float v[8];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const v2f a = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(w[i], 1.0f, false);
    const v2f b = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(w[i], 1.0f, true);
    v[4 * i] = a.x;
    v[4 * i + 1] = a.y;
    v[4 * i + 2] = b.x;
    v[4 * i + 3] = b.y;
  }
  if (finite(s) && (nan & 0x80808080u) == 0u) {
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = __fmul_rn(v[i], s);
    store8<F32OUT, true, false>(out, e, v);
  } else {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const uint32_t code = (w[i >> 2] >> (8 * (i & 3))) & 0xFFu;
      v[i] = __fmul_rn((code & 0x7Fu) == 0x7Fu ? dec_e4m3(code) : v[i], s);
    }
    store8<F32OUT, true, true>(out, e, v);
  }
}

// 8 E2M1 codes times sb (the product exact), then times s_t.
template <bool F32OUT, bool VEC>
__device__ inline void dequant_e2m1x8(uint32_t w, float sb, float s_t, void* out, int64_t e) {
  const v2f d[4] = {__builtin_amdgcn_cvt_scalef32_pk_f32_fp4(w, 1.0f, 0),
                    __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(w, 1.0f, 1),
                    __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(w, 1.0f, 2),
                    __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(w, 1.0f, 3)};
  float v[8];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    v[2 * j] = __fmul_rn(__fmul_rn(d[j].x, sb), s_t);
    v[2 * j + 1] = __fmul_rn(__fmul_rn(d[j].y, sb), s_t);
  }
  if (F32OUT || (finite(sb) && finite(s_t))) store8<F32OUT, VEC, false>(out, e, v);
  else store8<F32OUT, VEC, true>(out, e, v);
}

// VEC: 8-byte aligned codes and a 16-byte aligned output.
template <bool F32OUT, bool VEC>
__global__ void __launch_bounds__(256) k_dequant_fp8(const uint8_t* __restrict__ q, int64_t n,
                                                     const float* __restrict__ scale, void* out) {
  const int64_t e = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 8;
  if (VEC && e + 8 <= n) {
    dequant_e4m3x8<F32OUT>(*reinterpret_cast<const uint2*>(q + e), *scale, out, e);
    return;
  }
  const int cnt = (int)min((int64_t)8, n - e);  // the last of a tensor, or unaligned
  const float s = *scale;
  for (int i = 0; i < cnt; ++i) {
    const float v = __fmul_rn(dec_e4m3(q[e + i]), s);
    if (F32OUT) reinterpret_cast<float*>(out)[e + i] = v;
    else reinterpret_cast<uint16_t*>(out)[e + i] = (uint16_t)f32_to_bf16(v);
  }
}

// Two threads per 16-element block (8-byte aligned codes). VEC: a 16-byte
// aligned output.
template <bool F32OUT, bool VEC>
__global__ void __launch_bounds__(256) k_dequant_nvfp4(const uint8_t* __restrict__ q,
                                                       const uint8_t* __restrict__ bscale, int64_t n,
                                                       const float* __restrict__ tscale, void* out) {
  const int64_t u = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (u * 8 >= n) return;
  dequant_e2m1x8<F32OUT, VEC>(reinterpret_cast<const uint32_t*>(q)[u], dec_e4m3(bscale[u >> 1]), *tscale, out, u * 8);
}

// MX: four threads per 32-element block (codes aligned to a thread's: 4 bytes
// for MXFP4, 8 for MXFP8).
template <bool FP4, bool F32OUT>
__global__ void __launch_bounds__(256) k_dequant_mx(const uint8_t* __restrict__ q, const uint8_t* __restrict__ sc,
                                                    int64_t n, void* __restrict__ out) {
  const int64_t u = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (u * 8 >= n) return;
  const uint32_t e = sc[u >> 2];
  // 2^(e - 127); code 255 is the E8M0 NaN (a block that held inf or NaN)
  const float scale = (e == 0u) ? u2f(0x00400000u) : (e == 255u) ? __builtin_nanf("") : u2f(e << 23);
  if (FP4) dequant_e2m1x8<F32OUT, true>(reinterpret_cast<const uint32_t*>(q)[u], scale, 1.0f, out, u * 8);
  else dequant_e4m3x8<F32OUT>(reinterpret_cast<const uint2*>(q)[u], scale, out, u * 8);
}

// ---------------------------------------------------------------- launchers
static inline unsigned grid_for(int64_t threads) { return (unsigned)((threads + 255) / 256); }

// Whether the unit kernels take rows of this tensor: 16-byte aligned units,
// whole ones in every row of a slice.
static inline bool unit_tensor(const uint16_t* x, int64_t cols, int64_t ldx) {
  if (reinterpret_cast<uintptr_t>(x) % 16 != 0) return false;
  return ldx == cols || (ldx % 8 == 0 && cols % 8 == 0);
}

template <int H, bool DENSE>
static void launch_units(int fmt, const uint16_t* x, int64_t n, const UnitRows& ur, uint8_t* codes, uint8_t* bscale,
                         const float* tscale, hipStream_t st) {
  const dim3 g((unsigned)((n + 4096 * H - 1) / (4096 * H)));  // 4 waves x 64 H blocks of 16 per workgroup
  const bool plain = reinterpret_cast<uintptr_t>(codes) % 16 == 0 && n % 16 == 0;
  if (fmt == 2)
    hipLaunchKernelGGL((k_quant_units<2, H, DENSE, true>), g, dim3(256), 0, st, x, n, ur, codes, bscale, tscale);
  else if (plain)
    hipLaunchKernelGGL((k_quant_units<1, H, DENSE, true>), g, dim3(256), 0, st, x, n, ur, codes, bscale, tscale);
  else
    hipLaunchKernelGGL((k_quant_units<1, H, DENSE, false>), g, dim3(256), 0, st, x, n, ur, codes, bscale, tscale);
}

// The element kernels alone, reading a finished decode scale from `tscale`:
// the last kernel of the dynamic chain (chained), and the whole of a
// quantization with a static (calibrated) scale.
static hipError_t launch_elements(int fmt, const uint16_t* x, int64_t rows, int64_t cols, int64_t ldx, uint8_t* codes,
                                  uint8_t* bscale, const float* tscale, bool chained, hipStream_t st) {
  if (rows == 0 || cols == 0) return hipSuccess;
  const bool contig = (ldx == cols);
  if (unit_tensor(x, cols, ldx) && reinterpret_cast<uintptr_t>(codes) % 8 == 0) {
    const UnitRows ur = contig ? UnitRows() : unit_rows(cols, ldx);
    for_pieces(rows, cols, ldx, [&](int64_t src, int64_t e, int64_t cnt) {
      uint8_t* q = codes + (fmt == 1 ? e : e / 2);
      uint8_t* sc = fmt == 1 ? nullptr : bscale + e / 16;
      if (contig && chained) launch_units<2, true>(fmt, x + src, cnt, ur, q, sc, tscale, st);
      else if (contig) launch_units<1, true>(fmt, x + src, cnt, ur, q, sc, tscale, st);
      else if (chained) launch_units<2, false>(fmt, x + src, cnt, ur, q, sc, tscale, st);
      else launch_units<1, false>(fmt, x + src, cnt, ur, q, sc, tscale, st);
    });
  } else {
    for_pieces(rows, cols, ldx, [&](int64_t src, int64_t e, int64_t cnt) {
      const int64_t r = contig ? 1 : cnt / cols, c = contig ? cnt : cols;
      const dim3 g(grid_for(r * ((c + 15) / 16))), t(256);
      const uint16_t* p = x + src;
      uint8_t* q = codes + (fmt == 1 ? e : e / 2);
      uint8_t* sc = fmt == 1 ? nullptr : bscale + e / 16;
      if (fmt == 1 && contig) hipLaunchKernelGGL((k_quant_fp8<true>), g, t, 0, st, p, r, c, c, q, tscale);
      else if (fmt == 1) hipLaunchKernelGGL((k_quant_fp8<false>), g, t, 0, st, p, r, c, ldx, q, tscale);
      else if (contig) hipLaunchKernelGGL((k_quant_nvfp4<true>), g, t, 0, st, p, r, c, c, q, sc, tscale);
      else hipLaunchKernelGGL((k_quant_nvfp4<false>), g, t, 0, st, p, r, c, ldx, q, sc, tscale);
    });
  }
  return hipGetLastError();
}

hipError_t launch_quantize_static(int fmt, const uint16_t* x, int64_t rows, int64_t cols, int64_t ldx,
                                  uint8_t* codes, uint8_t* bscale, const float* tscale, hipStream_t st) {
  return launch_elements(fmt, x, rows, cols, ldx, codes, bscale, tscale, false, st);
}

// MX formats: block scales only, one kernel.
template <bool FP4>
static hipError_t launch_quantize_mx(const uint16_t* x, int64_t rows, int64_t cols, int64_t ldx,
                                     uint8_t* codes, uint8_t* scales, hipStream_t st) {
  if (rows == 0 || cols == 0) return hipSuccess;
  if (!unit_tensor(x, cols, ldx)) {
    for_pieces(rows, cols, ldx, [&](int64_t src, int64_t e, int64_t cnt) {
      const int64_t c = ldx == cols ? cnt : cols;
      hipLaunchKernelGGL((k_quant_mx<FP4>), dim3(grid_for(cnt / 8)), dim3(256), 0, st, x + src, cnt / c, c,
                         ldx == cols ? c : ldx, codes + (FP4 ? e / 2 : e), scales + e / 32);
    });
    return hipGetLastError();
  }
  constexpr int H = 1;
  const bool plain = reinterpret_cast<uintptr_t>(codes) % (FP4 ? 8 : 16) == 0;
  const UnitRows ur = ldx == cols ? UnitRows() : unit_rows(cols, ldx);
  for_pieces(rows, cols, ldx, [&](int64_t src, int64_t e, int64_t cnt) {
    const int64_t halves = cnt / 16;
    const dim3 g((unsigned)((halves + 256 * H - 1) / (256 * H))), t(256);
    const uint16_t* p = x + src;
    uint8_t* q = codes + (FP4 ? e / 2 : e);
    uint8_t* sc = scales + e / 32;
    if (ldx == cols) {
      if (plain) hipLaunchKernelGGL((k_quant_mx_units<FP4, H, true, true>), g, t, 0, st, p, halves, ur, q, sc);
      else hipLaunchKernelGGL((k_quant_mx_units<FP4, H, true, false>), g, t, 0, st, p, halves, ur, q, sc);
    } else {
      if (plain) hipLaunchKernelGGL((k_quant_mx_units<FP4, H, false, true>), g, t, 0, st, p, halves, ur, q, sc);
      else hipLaunchKernelGGL((k_quant_mx_units<FP4, H, false, false>), g, t, 0, st, p, halves, ur, q, sc);
    }
  });
  return hipGetLastError();
}

template <int FMT, bool DENSE>
static void launch_slots(const uint16_t* x, int64_t units, const UnitRows& ur, uint8_t* codes, uint8_t* bscale,
                         float* tscale, const SlotsPlan& plan, hipStream_t st) {
  hipLaunchKernelGGL((k_amax_slots<kSlotsAmaxLoads, DENSE>), dim3((unsigned)plan.P), dim3(256), 0, st, x, units, ur,
                     codes, FMT == 1 ? 8 : 4, (int)plan.G);
  hipLaunchKernelGGL((k_quant_slots<FMT, DENSE>), dim3((unsigned)plan.G), dim3(256), 0, st, x, units, ur, codes,
                     bscale, tscale, (int)plan.P);
}

hipError_t launch_quantize(int fmt, const uint16_t* x, int64_t rows, int64_t cols, int64_t ldx,
                           uint8_t* codes, uint8_t* bscale, float* tscale, hipStream_t st) {
  if (fmt == 3) return launch_quantize_mx<true>(x, rows, cols, ldx, codes, bscale, st);
  if (fmt == 4) return launch_quantize_mx<false>(x, rows, cols, ldx, codes, bscale, st);
  if (rows == 0 || cols == 0) {
    hipLaunchKernelGGL(k_fill_u32, dim3(1), dim3(1), 0, st, reinterpret_cast<uint32_t*>(tscale), 0u);
    return hipGetLastError();
  }
  const bool contig = (ldx == cols);
  const bool aligned = (reinterpret_cast<uintptr_t>(x) % 16 == 0);
  if (rows * ((cols + 15) / 16) <= kSmallUnits) {
    // one launch does it all (NVFP4 codes are 8-byte aligned: checked by
    // the caller); one workgroup per 256 units, at most eight. Measured
    // against the chain (GPU time from graph replays): 1 x 1024 3.1 us,
    // 128 x 256 4.3 us, 16 x 3072 4.6 us, where the chain takes 6.5 us
    // (FP8) to 7.4 us (NVFP4); one workgroup took 5.0 and 5.9 us on the last
    // two. Raising the limit to 8192 units (eight per thread) lost to the
    // chain from 6144 units on.
    const bool rvec = aligned && (cols % 8 == 0) && (contig || ldx % 8 == 0);
    const bool qvec = (reinterpret_cast<uintptr_t>(codes) % 16 == 0) && (cols % 16 == 0);
    const int64_t units = rows * ((cols + 15) / 16);
    const unsigned G = (unsigned)std::min<int64_t>(kSmallGroups, (units + 255) / 256);
    if (fmt == 1) {
      if (rvec) hipLaunchKernelGGL((k_quant_small<1, true>), dim3(G), dim3(1024), 0, st, x, rows, cols, ldx, codes, bscale, tscale, qvec);
      else hipLaunchKernelGGL((k_quant_small<1, false>), dim3(G), dim3(1024), 0, st, x, rows, cols, ldx, codes, bscale, tscale, qvec);
    } else {
      if (rvec) hipLaunchKernelGGL((k_quant_small<2, true>), dim3(G), dim3(1024), 0, st, x, rows, cols, ldx, codes, bscale, tscale, false);
      else hipLaunchKernelGGL((k_quant_small<2, false>), dim3(G), dim3(1024), 0, st, x, rows, cols, ldx, codes, bscale, tscale, false);
    }
    return hipGetLastError();
  }
  const int64_t n = rows * cols;
  const bool unit = unit_tensor(x, cols, ldx);
  const UnitRows ur = (unit && !contig) ? unit_rows(cols, ldx) : UnitRows();
  if (unit && reinterpret_cast<uintptr_t>(codes) % 8 == 0) {
    // two launches, the maxima handed over in every code region
    const SlotsPlan plan = slots_plan(n, fmt == 1 ? 8 : 4);
    if (plan.G >= 1) {
      if (contig) {
        if (fmt == 1) launch_slots<1, true>(x, n / 8, ur, codes, bscale, tscale, plan, st);
        else launch_slots<2, true>(x, n / 8, ur, codes, bscale, tscale, plan, st);
      } else {
        if (fmt == 1) launch_slots<1, false>(x, n / 8, ur, codes, bscale, tscale, plan, st);
        else launch_slots<2, false>(x, n / 8, ur, codes, bscale, tscale, plan, st);
      }
      return hipGetLastError();
    }
  }
  // amax: per-workgroup partial maxima are parked in the code buffer, which
  // the quantize kernel overwrites afterwards (stream order separates them).
  // More than kSmallUnits units: the codes hold a partial per 1024 16-byte units.
  {
    const uintptr_t base = (reinterpret_cast<uintptr_t>(codes) + 3) & ~uintptr_t(3);
    uint32_t* partial = reinterpret_cast<uint32_t*>(base);
    int64_t gx = 0, gy = 1;
    if (unit && n % 8 == 0) {
      for_pieces(rows, cols, ldx, [&](int64_t src, int64_t, int64_t cnt) {
        const int64_t groups = std::min<int64_t>((cnt / 8 + 1023) / 1024, kAmaxGroups);
        const dim3 g((unsigned)groups), t(256);
        if (contig) hipLaunchKernelGGL(k_amax_units<true>, g, t, 0, st, x + src, cnt / 8, ur, partial + gx);
        else hipLaunchKernelGGL(k_amax_units<false>, g, t, 0, st, x + src, cnt / 8, ur, partial + gx);
        gx += groups;
      });
    } else {
      const int64_t r_eff = contig ? 1 : rows, c_eff = contig ? n : cols;
      gy = std::min<int64_t>(r_eff, 1024);
      gx = std::min<int64_t>(std::max<int64_t>(1, (c_eff + 1023) / 1024), std::max<int64_t>(1, 1024 / gy));
      const int64_t cap = ((fmt == 1 ? n : n / 2) - (int64_t)(base - reinterpret_cast<uintptr_t>(codes))) / 4;
      if (gx * gy > cap) {  // short rows in many units: one workgroup, its max goes straight to the scale slot
        gx = gy = 1;
        partial = reinterpret_cast<uint32_t*>(tscale);
      }
      hipLaunchKernelGGL(k_amax_partial, dim3((unsigned)gx, (unsigned)gy), dim3(256), 0, st, x, r_eff, c_eff,
                         contig ? c_eff : ldx, partial);
    }
    hipLaunchKernelGGL(k_finalize, dim3(1), dim3(256), 0, st, partial, (int)(gx * gy), tscale,
                       fmt == 1 ? 448.0f : 2688.0f);
  }
  return launch_elements(fmt, x, rows, cols, ldx, codes, bscale, tscale, true, st);
}

hipError_t launch_dequant(int fmt, const uint8_t* codes, const uint8_t* bscale, const float* tscale,
                          int64_t rows, int64_t cols, void* out, bool f32out, hipStream_t st) {
  if (rows == 0 || cols == 0) return hipSuccess;
  for_pieces(rows, cols, cols, [&](int64_t, int64_t e0, int64_t n) {
    const uint8_t* q = codes + (fmt == 1 || fmt == 4 ? e0 : e0 / 2);
    void* o = reinterpret_cast<uint8_t*>(out) + e0 * (f32out ? 4 : 2);
    const dim3 g(grid_for((n + 7) / 8)), t(256);
    if (fmt == 3 || fmt == 4) {  // whole blocks, 16-byte aligned output (checked by the caller)
      const uint8_t* sc = bscale + e0 / 32;
      if (fmt == 3 && f32out) hipLaunchKernelGGL((k_dequant_mx<true, true>), g, t, 0, st, q, sc, n, o);
      else if (fmt == 3) hipLaunchKernelGGL((k_dequant_mx<true, false>), g, t, 0, st, q, sc, n, o);
      else if (f32out) hipLaunchKernelGGL((k_dequant_mx<false, true>), g, t, 0, st, q, sc, n, o);
      else hipLaunchKernelGGL((k_dequant_mx<false, false>), g, t, 0, st, q, sc, n, o);
      return;
    }
    const bool vec = reinterpret_cast<uintptr_t>(out) % 16 == 0 && reinterpret_cast<uintptr_t>(codes) % 8 == 0;
    const uint8_t* sc = bscale + e0 / 16;  // NVFP4
#define QG_DEQUANT(F32, VEC)                                                                                      \
  do {                                                                                                            \
    if (fmt == 1) hipLaunchKernelGGL((k_dequant_fp8<F32, VEC>), g, t, 0, st, q, n, tscale, o);                    \
    else hipLaunchKernelGGL((k_dequant_nvfp4<F32, VEC>), g, t, 0, st, q, sc, n, tscale, o);                       \
  } while (0)
    if (f32out && vec) QG_DEQUANT(true, true);
    else if (f32out) QG_DEQUANT(true, false);
    else if (vec) QG_DEQUANT(false, true);
    else QG_DEQUANT(false, false);
#undef QG_DEQUANT
  });
  return hipGetLastError();
}

}  // namespace qg
