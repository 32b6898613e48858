// fp32 operands on the bf16 matrix cores: a float is the exact sum of three bf16 values (8 + 8 + 8 significant bits),
// so a product of two floats is the sum of nine bf16 products, of which the six largest are taken; the three left out
// are below 2^-23 of the product.  A bf16 16x16x32 instruction does 32 channels in 16 clk where the fp32 16x16x4
// needs eight instructions of 32 clk, and, unlike the fp32 one, runs beside the vector ALU: six of them take 53 ns per
// SIMD against 124 ns (measured, two waves per SIMD), and the sums round once per 32 terms instead of after each, so
// that a dot product of 64 comes out at 0.9e-7 of its 64-bit value in norm against 1.05e-7 to 1.45e-7.
//
// An infinite or NaN operand makes every sum it enters NaN (its parts do not exist).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "rotconv_bf16.h"
#include "rotconv_internal.h"

namespace rotconv {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float s3_f4 __attribute__((ext_vector_type(4)));
typedef __bf16 s3_bf8 __attribute__((ext_vector_type(8)));

// The upper halves of two floats side by side: `lo` in the low half.
__device__ __forceinline__ uint32_t s3_pack_hi(float lo, float hi) {
  return __builtin_amdgcn_perm(__builtin_bit_cast(uint32_t, hi), __builtin_bit_cast(uint32_t, lo), 0x07060302u);
}

__device__ __forceinline__ float s3_trunc(float v) {
  return __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, v) & 0xffff0000u);
}

// Two values -> their three parts, each a packed pair (truncating split: eleven vector instructions, no overflow).
struct S3Pair { uint32_t p[3]; };
__device__ __forceinline__ S3Pair s3_split2(float a, float b) {
  S3Pair s;
  s.p[0] = s3_pack_hi(a, b);
  const float ra = a - s3_trunc(a), rb = b - s3_trunc(b);
  s.p[1] = s3_pack_hi(ra, rb);
  s.p[2] = s3_pack_hi(ra - s3_trunc(ra), rb - s3_trunc(rb));
  return s;
}

// One stored operand value (a weight, split once per call): parts to nearest, so that what the six products leave out
// is half as large and has no sign of its own.
__device__ __forceinline__ uint32_t s3_round_part(float v) {      // bits of a bf16 value in the upper half
  const uint32_t u = __builtin_bit_cast(uint32_t, v);
  const uint32_t r = u + 0x7fffu + ((u >> 16) & 1u);
  const bool keep = (r & 0x7f800000u) == 0x7f800000u;            // would overflow (or is no finite value): truncate
  return (keep ? u : r) & 0xffff0000u;
}
__device__ __forceinline__ void s3_split_weight(float v, uint16_t& p0, uint16_t& p1, uint16_t& p2) {
  const uint32_t a = s3_round_part(v);
  const float r1 = v - __builtin_bit_cast(float, a);
  const uint32_t b = s3_round_part(r1);
  const float r2 = r1 - __builtin_bit_cast(float, b);
  p0 = (uint16_t)(a >> 16);
  p1 = (uint16_t)(b >> 16);
  p2 = (uint16_t)(s3_round_part(r2) >> 16);
}

__device__ __forceinline__ s3_f4 s3_mfma(u32x4 a, u32x4 b, s3_f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(s3_bf8, a), __builtin_bit_cast(s3_bf8, b), c, 0, 0, 0);
}

// One element (bank q, tap u) of the expansion of a base slice; src: the nine taps of (filter, channel).  round16: bf16
// plans, the combination in fp64, rounded to fp32 and to bf16 once each.
__device__ __forceinline__ float s3_expand_tap(const float* __restrict__ src, size_t bank_stride, int row, bool in,
                                               const int32_t* __restrict__ fq_src, const float* __restrict__ fq_coef,
                                               const double* __restrict__ fq_coef64, int round16) {
  if (round16) {
    double a64 = 0.0;
    for (int z = 0; z < kMaxNnz; ++z) {
      const int s = fq_src[row * kMaxNnz + z];
      if (in && s >= 0) a64 += fq_coef64[row * kMaxNnz + z] * (double)src[(size_t)(s / 9) * bank_stride + s % 9];
    }
    return bf16_to_f32(f32_to_bf16((float)a64));
  }
  float acc = 0.f;
#pragma unroll
  for (int z = 0; z < kMaxNnz; ++z) {
    const int s = fq_src[row * kMaxNnz + z];
    if (in && s >= 0) acc += fq_coef[row * kMaxNnz + z] * src[(size_t)(s / 9) * bank_stride + s % 9];
  }
  return acc;
}

}  // namespace rotconv
