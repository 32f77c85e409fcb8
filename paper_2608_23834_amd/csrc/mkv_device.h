// Device-side helpers shared by the Minima-KV gfx950 kernels: physical page
// layouts, FP8 E4M3 / binary16 conversions, the TQ3 code layout and MFMA
// operand types.  Layout definitions follow the pool description in
// include/minima_kv.h.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mkv {

constexpr int PAGE = 16;
constexpr int TAG_R = 0, TAG_A = 1, TAG_S = 2, TAG_NONE = 0xFF;

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef float float16v __attribute__((ext_vector_type(16)));

// ---------------------------------------------------------------------------
// ctrl buffer (int32 words): counters, free stacks, work list, rotation signs.
// ---------------------------------------------------------------------------
enum CtrlSlot {
  CTRL_FP8_TOP = 0,
  CTRL_TQ3_TOP = 1,
  CTRL_ERR = 2,
  CTRL_NLIST = 3,
  CTRL_ABORT = 4,
  CTRL_APPEND_ARRIVE = 5,  // waves of a decode-step append that have finished (reset by the last)
  CTRL_HEADER = 64
};
constexpr int MIG_BLOCKS = 256;  // most workgroups of a migration plan
struct CtrlLayout {
  int64_t fp8_stack, tq3_stack, list, sigma_bytes, mig, rc8, rc3, occ8, occ3, last8, last3,
      total_words;
};
// mig: migration-plan scratch, per-workgroup counts [MIG_BLOCKS], per-workgroup
// error bits [MIG_BLOCKS], the TQ3 free-list top the plan started from.
// rc8 / rc3: references per FP8 / TQ3 page (0: free).  occ* / last*: release
// scratch per page (occurrences in the call, last list index), 0 / -1 at rest.
__host__ __device__ inline CtrlLayout ctrl_layout(int n_fp8, int n_tq3, int d) {
  CtrlLayout c;
  c.fp8_stack = CTRL_HEADER;
  c.tq3_stack = c.fp8_stack + n_fp8;
  c.list = c.tq3_stack + n_tq3;
  c.sigma_bytes = (c.list + 4LL * n_fp8) * 4;  // byte offset of int8 sigma[d]
  c.mig = c.list + 4LL * n_fp8 + (d + 3) / 4;
  c.rc8 = c.mig + 2LL * MIG_BLOCKS + 1;
  c.rc3 = c.rc8 + n_fp8;
  c.occ8 = c.rc3 + n_tq3;
  c.occ3 = c.occ8 + n_fp8;
  c.last8 = c.occ3 + n_tq3;
  c.last3 = c.last8 + n_fp8;
  c.total_words = c.last3 + n_tq3;
  return c;
}

// ---------------------------------------------------------------------------
// Page layouts (per layer, physical page, KV head).
//  FP8 region: 2*16*d bytes.  K at [t*d + c] (token-major).  V in lane-chunk
//  order: with CL = d/16, r = c/CL, m = c%CL, g = t/4, u = t%4 the V byte of
//  (t, c) is at 16*d + ((r*4 + g)*CL + m)*4 + u.
//  TQ3 region: 16*d + 32 bytes: K codes [0, 6d), V codes [6d, 12d), gamma
//  fp16[16] at 12d, V scale fp16[d] at 12d+32, V zero fp16[d] at 14d+32.
//  Codes live in "chunks" of 3d/32 bytes holding d/16 quads of 4 codes:
//   K chunk (t, g) at (g*16+t)*3d/32: quad q, position b = channel d/4*g+4q+b
//   V chunk (r, g) at (g*16+r)*3d/32: quad q = channel CL*r+q, position b =
//   token 4g+b.  Chunks are ordered g-major: the 16 lanes of an MFMA row
//   group read chunks 16g .. 16g+15, contiguous in LDS, without bank conflicts.
//  Within a chunk of n_dw = 3d/128 dwords, quad q < 2*n_dw occupies bits
//  [8b + 3(q%2), +3) of dword q/2; the remaining quads use bits 6-7 of every
//  byte (see quad_sel below).
// ---------------------------------------------------------------------------
__host__ __device__ constexpr int64_t fp8_region_bytes(int d) { return 2LL * PAGE * d; }
__host__ __device__ constexpr int64_t tq3_region_bytes(int d) { return 16LL * d + 32; }
__host__ __device__ constexpr int chunk_bytes(int d) { return 3 * d / 32; }

// Byte selector of the 4 codes of quad q (one code in the low 3 bits of each
// byte) from the chunk's dwords D[].  (The encode's pack_quads is its inverse.)
template <int NDW>
__device__ __forceinline__ uint32_t quad_sel(const uint32_t* D, int q) {
  if (q < 2 * NDW) {
    return (D[q >> 1] >> (3 * (q & 1))) & 0x07070707u;
  }
  int e = q - 2 * NDW, p = e >> 1;
  if ((e & 1) == 0)
    return ((D[3 * p] >> 6) & 0x03030303u) | ((D[3 * p + 1] >> 4) & 0x04040404u);
  return ((D[3 * p + 1] >> 7) & 0x01010101u) | ((D[3 * p + 2] >> 5) & 0x06060606u);
}

// TQ3 codebook levels as E4M3 bytes, code 0..7 ascending:
// -2.25, -1.375, -0.75, -0.25, 0.25, 0.75, 1.375, 2.25
constexpr uint32_t KLUT_LO = 0xA8B4BBC1u, KLUT_HI = 0x413B3428u;

// ---------------------------------------------------------------------------
// Scalar conversions
// ---------------------------------------------------------------------------
__device__ __forceinline__ float bf16_to_f32(uint16_t b) {
  return __uint_as_float(((uint32_t)b) << 16);
}
// E4M3 value of a byte (exact).
__device__ __forceinline__ float e4m3_to_f32(uint32_t byte) {
  return __builtin_amdgcn_cvt_f32_fp8((int)byte, 0);
}
// fp32 -> E4M3, nearest-even, saturating at +-448 (the hardware conversion
// does not saturate, so clamp first).
__device__ __forceinline__ uint32_t f32_to_e4m3(float x) {
  x = fminf(fmaxf(x, -448.0f), 448.0f);
  return (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(x, 0.0f, 0, false) & 0xFFu;
}

// fp64 -> binary16, round to nearest even, saturating at +-65504 (stored
// metadata stays finite).  Method: round to fp32 to odd -- truncate, and set the
// last bit when anything was cut off -- then to binary16 with the hardware's
// conversion: an odd last bit keeps the value off every binary16 tie, and fp32
// carries more than two bits beyond binary16's, so the second rounding sees on
// which side of a boundary x lies (one rounding in effect).  The truncation
// comes from the fp64 -> fp32 conversion by stepping back where it rounded away
// from zero.  Ten instructions, against about thirty through frexp and ldexp.
__device__ __forceinline__ uint16_t f64_to_f16_rne_sat(double x) {
  const float f = (float)x;
  const double d = (double)f;
  uint32_t u = __float_as_uint(f);
  u -= fabs(d) > fabs(x) ? 1u : 0u;
  u |= d != x ? 1u : 0u;
  const float c = fminf(fmaxf(__uint_as_float(u), -65504.0f), 65504.0f);  // largest finite binary16
  const uint16_t h = __builtin_bit_cast(uint16_t, (_Float16)c);
  return x != x ? (uint16_t)((signbit(x) ? 0x8000u : 0u) | 0x7E00u) : h;
}
__device__ __forceinline__ double f16_bits_to_f64(uint16_t h) {
  _Float16 v = __builtin_bit_cast(_Float16, h);
  return (double)v;
}

// ---------------------------------------------------------------------------
// Block-wide helpers (blockDim.x threads, wave64)
// ---------------------------------------------------------------------------
// Exclusive prefix sum of one int per thread; returns the prefix, writes the
// total to *total.  Uses scratch[blockDim.x/64 + 1] ints of LDS.
__device__ inline int block_excl_scan(int v, int* scratch, int* total) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = blockDim.x >> 6;
  int x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    int y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) scratch[wid] = x;
  __syncthreads();
  if (threadIdx.x == 0) {
    int acc = 0;
    for (int w = 0; w < nw; ++w) {
      int t = scratch[w];
      scratch[w] = acc;
      acc += t;
    }
    scratch[nw] = acc;
  }
  __syncthreads();
  int res = scratch[wid] + x - v;
  *total = scratch[nw];
  __syncthreads();
  return res;
}

}  // namespace mkv
