// Device helpers shared by the matrix-core kernels of libkvprm (projections in kvprm_mfma.hip,
// attention in kvprm_attn.hip): vector types, the streaming load, the MFMA wrapper, bf16 hi/lo
// splitting of fp32 operands, the operand-buffer store and wave/block reductions.
#pragma once

#include <type_traits>

#include "kvprm_internal.h"

namespace kvprm {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// four floats of a caller's array, which may be aligned to 4 bytes only (16-byte global loads take
// that)
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));

// 16-byte load of data that a call reads exactly once (cache pages of the private ranges, weight
// tiles): non-temporal, so the stream does not allocate in the caches and displace lines that
// are reused. Measured on the paged K/V read pattern: 6.5 TB/s instead of 5.6 with plain loads.
__device__ __forceinline__ uint4 ld_stream(const uint4 *p) {
  const u32x4 v = __builtin_nontemporal_load((const u32x4 *)p);
  return make_uint4(v.x, v.y, v.z, v.w);
}

__device__ __forceinline__ floatx4 mfma16(const uint4 &a, const uint4 &b, const floatx4 &c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                 __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

__device__ __forceinline__ floatx4 mfma4(float a, float b, const floatx4 &c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Two fp32 values -> packed bf16 pairs hi (RNE) and lo = RNE(x - hi) (the hardware pack-convert,
// one instruction per pair): hi + lo carries 16 significant bits of each value.
__device__ __forceinline__ void split2(float x0, float x1, uint32_t &hi, uint32_t &lo) {
  typedef __bf16 bf16x2v __attribute__((ext_vector_type(2)));
  typedef float f32x2v __attribute__((ext_vector_type(2)));
  const f32x2v xv = {x0, x1};
  hi = __builtin_bit_cast(uint32_t, __builtin_convertvector(xv, bf16x2v));
  const f32x2v rv = {x0 - __uint_as_float(hi << 16), x1 - __uint_as_float(hi & 0xFFFF0000u)};
  lo = __builtin_bit_cast(uint32_t, __builtin_convertvector(rv, bf16x2v));
}

// Two fp32 values -> packed bf16 pairs hi, mid, lo (nearest-even each, mid of the rest after hi,
// lo of the rest after mid; the differences are exact): hi + mid + lo carries 24 significant bits.
__device__ __forceinline__ void split3(float x0, float x1, uint32_t &hi, uint32_t &mid,
                                       uint32_t &lo) {
  typedef __bf16 bf16x2v __attribute__((ext_vector_type(2)));
  typedef float f32x2v __attribute__((ext_vector_type(2)));
  const f32x2v xv = {x0, x1};
  hi = __builtin_bit_cast(uint32_t, __builtin_convertvector(xv, bf16x2v));
  split2(x0 - __uint_as_float(hi << 16), x1 - __uint_as_float(hi & 0xFFFF0000u), mid, lo);
}

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

__device__ __forceinline__ float ld_w(const void *p, size_t i, int wdt) {
  return wdt ? __uint_as_float((uint32_t)((const uint16_t *)p)[i] << 16) : ((const float *)p)[i];
}

// Store v for input k of candidate cand into an operand buffer: columns cand and cand + Bp hold
// its hi and lo halves. Bp = 4 (one column tile, at most 4 candidates) leaves room for a third
// term at cand + 2 Bp, so that a few candidates' activations keep 24 bits at no cost.
__device__ __forceinline__ void store_operand(uint16_t *op, int NT, int Bp, int k, int cand,
                                              float v) {
  const int kb = k >> 5, c = (k >> 3) & 3, i = k & 7;
  auto put = [&](int col, uint32_t w) {
    op[((size_t)((kb * NT + (col >> 4)) * 64 + c * 16 + (col & 15))) * 8 + i] = (uint16_t)w;
  };
  uint32_t hi, mid, lo;
  split3(v, 0.f, hi, mid, lo);
  put(cand, hi);
  put(cand + Bp, mid);
  if (Bp == 4) put(cand + 8, lo);
}

// The same for inputs k .. k + 3 (k a multiple of 4): 8-byte stores.
__device__ __forceinline__ void store_operand4(uint16_t *op, int NT, int Bp, int k, int cand,
                                               const float (&v)[4]) {
  const int kb = k >> 5, c = (k >> 3) & 3, i = k & 7;
  auto put = [&](int col, const uint2 &w) {
    *(uint2 *)(op + (size_t)((kb * NT + (col >> 4)) * 64 + c * 16 + (col & 15)) * 8 + i) = w;
  };
  uint2 hi, mid, lo;
  split3(v[0], v[1], hi.x, mid.x, lo.x);
  split3(v[2], v[3], hi.y, mid.y, lo.y);
  put(cand, hi);
  put(cand + Bp, mid);
  if (Bp == 4) put(cand + 8, lo);
}

// The sum of a candidate's terms over the columns of one column tile (lane l, column l % 16),
// valid in columns below Bp: columns n, n + 8 and, with three terms, n + 4, by row rotations (lane i
// of 16 receives lane i - r; one vector instruction, where an LDS permute costs a round trip).
__device__ __forceinline__ float sum_terms(float v, int Bp) {
  auto ror = [](float x, auto r) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x120 + decltype(r)::value, 0xF,
                                                   0xF, false));
  };
  float s = v + ror(v, std::integral_constant<int, 8>{});
  if (Bp == 4) s += ror(v, std::integral_constant<int, 12>{});
  return s;
}

__device__ __forceinline__ float wsum(float v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

__device__ __forceinline__ float wmax(float v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = fmaxf(v, __shfl_xor(v, off, 64));
  return v;
}

// v combined over the four lanes l % 16, l % 16 + 16, + 32, + 48 (the lanes of one column of a
// matrix-core accumulator), in every lane: gfx950's row swaps instead of two LDS permutes. Each
// swap of a register with itself leaves a row pair's lower rows in one result and its upper rows
// in the other.
template <typename F>
__device__ __forceinline__ float column_reduce(float v, F f) {
  const uint32_t a = __float_as_uint(v);
  const auto r = __builtin_amdgcn_permlane16_swap(a, a, false, false);
  const uint32_t b = __float_as_uint(f(__uint_as_float(r[0]), __uint_as_float(r[1])));
  const auto t = __builtin_amdgcn_permlane32_swap(b, b, false, false);
  return f(__uint_as_float(t[0]), __uint_as_float(t[1]));
}
__device__ __forceinline__ float column_max(float v) {
  return column_reduce(v, [](float x, float y) { return fmaxf(x, y); });
}
__device__ __forceinline__ float column_sum(float v) {
  return column_reduce(v, [](float x, float y) { return x + y; });
}

// Deterministic 256-thread block reductions; every thread receives the result.
__device__ __forceinline__ float bsum(float v, float *red) {
  v = wsum(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  return (red[0] + red[1]) + (red[2] + red[3]);
}

__device__ __forceinline__ float ld_bf16(const void *p, size_t i) {
  return __uint_as_float((uint32_t)((const uint16_t *)p)[i] << 16);
}

}  // namespace kvprm
