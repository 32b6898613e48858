// fp32 operands on the bf16 matrix cores: a float is the sum of three bf16 values (8 + 8 + 8 significant bits, each to
// nearest), so a product of two floats is the sum of nine bf16 products, of which the six largest are taken.  A bf16
// 16x16x32 instruction does 32 channels in 16 clk where the fp32 16x16x4 needs eight instructions of 32 clk, and, unlike
// the fp32 one, runs beside the vector ALU: six of them take 53 ns per SIMD against 124 ns (measured, two waves per SIMD).
//
// Precision.  For v in [1, 2) the second part is at most 2^-8 and the third at most 2^-17, so the three products left out
// come to at most 2^-24 of the product, with no sign of their own.  (Parts cut instead of rounded leave out up to 2^-21,
// always of the product's sign.)  The matrix instruction adds its 32 terms and cuts the sum to fp32 towards minus infinity:
// at most 2^-23, on average 2^-24, of a lone product.  Measured against 64 bits, normal operands, in norm: one product
// 3.1e-8 (fp32 instruction 2.5e-8, parts cut 6.3e-8), two 2.8e-8 (2.9e-8, 5.4e-8), 32 of any sign 3.8e-8 (1.03e-7, 7.1e-8), 32
// positive ones 3.4e-8 (8.6e-8, 5.6e-8).
//
// The parts hold a value whole while its last bit is a bf16 number: from 2^-110 up.  Below, the third part is subnormal and
// the value is held to 2^-134.
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
typedef float s3_f16 __attribute__((ext_vector_type(16)));
typedef __bf16 s3_bf8 __attribute__((ext_vector_type(8)));

typedef float s3_f2 __attribute__((ext_vector_type(2)));
typedef __bf16 s3_bf2 __attribute__((ext_vector_type(2)));

// Two floats as bf16, to nearest, side by side: `lo` in the low half (one instruction).
__device__ __forceinline__ uint32_t s3_round2(float lo, float hi) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((s3_f2{lo, hi}), s3_bf2));
}
// The upper halves of two floats side by side.
__device__ __forceinline__ uint32_t s3_pack_hi(float lo, float hi) {
  return __builtin_amdgcn_perm(__builtin_bit_cast(uint32_t, hi), __builtin_bit_cast(uint32_t, lo), 0x07060302u);
}
__device__ __forceinline__ float s3_low(uint32_t p) { return __builtin_bit_cast(float, p << 16); }
__device__ __forceinline__ float s3_high(uint32_t p) { return __builtin_bit_cast(float, p & 0xffff0000u); }

// Two values -> their three parts, each a packed pair (eleven vector instructions).  What is left after two parts has at
// most seven bits, so cutting it (CUT) gives the same part; which of the two instructions is the faster one depends on
// its neighbours (rounded / cut: weight gradient of 8x64 -> 64, 256x256 321 / 311 us, input gradient of 4x512 -> 512, 32x32
// 163 / 170 us).
struct S3Pair { uint32_t p[3]; };
template <bool CUT = false>
__device__ __forceinline__ S3Pair s3_split2(float a, float b) {
  S3Pair s;
  s.p[0] = s3_round2(a, b);
  const float ra = a - s3_low(s.p[0]), rb = b - s3_high(s.p[0]);
  s.p[1] = s3_round2(ra, rb);
  const float qa = ra - s3_low(s.p[1]), qb = rb - s3_high(s.p[1]);
  s.p[2] = CUT ? s3_pack_hi(qa, qb) : s3_round2(qa, qb);
  return s;
}

// The same with the parts rounded by integer additions (ties away from zero) instead of conversions: fifteen instructions.
// Measured the faster form for the waves that only split (the weight gradient's X: 126 against 130.5 us at 4x128 -> 128,
// 128x128) and the slower one where D is split (133) and in the other two kernels (input gradient 178 against 171, forward
// 136 against 134 us, same layer).
__device__ __forceinline__ S3Pair s3_split2_add(float a, float b) {
  auto up = [](float v) { return __builtin_bit_cast(uint32_t, v) + 0x8000u; };      // rounded where its low half is dropped
  auto pack = [](uint32_t lo, uint32_t hi) { return __builtin_amdgcn_perm(hi, lo, 0x07060302u); };
  S3Pair s;
  const uint32_t ua = up(a), ub = up(b);
  s.p[0] = pack(ua, ub);
  const float ra = a - s3_high(ua), rb = b - s3_high(ub);
  const uint32_t va = up(ra), vb = up(rb);
  s.p[1] = pack(va, vb);
  s.p[2] = s3_pack_hi(ra - s3_high(va), rb - s3_high(vb));
  return s;
}

// One stored operand value (a weight, split once per call).
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

__device__ __forceinline__ s3_f16 s3_mfma32(u32x4 a, u32x4 b, s3_f16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(s3_bf8, a), __builtin_bit_cast(s3_bf8, b), c, 0, 0, 0);
}

// In the forward the matrix instruction's cut towards minus infinity is an offset of one sign in every product P_u that grows
// with the channels while their sum grows with the root of their number (1024 -> 32 channels: 1.1e-7 of the norm, more than
// all else together).  So the parts of every other tap's weights are stored with their signs turned, and those taps'
// products are subtracted where they are placed: the offsets cancel (five taps against four).
__device__ __host__ constexpr bool s3_tap_turned(int u) { return u & 1; }

// A sum that the parts do not hold: not finite, or below 2^-100 and not zero.
__device__ __forceinline__ bool beyond_parts(float v) {
  const float m = __builtin_fabsf(v);
  return !(m < __builtin_inff()) || (m < 0x1p-100f && m != 0.f);
}

// Four indices (a byte each) at any alignment.
__device__ __forceinline__ uint32_t load4(const uint8_t* p) {
  uint32_t v;
  __builtin_memcpy(&v, p, 4);
  return v;
}

// Byte offset of positions outside an image in loads through its buffer descriptor: beyond the descriptor's size (the
// kernels' limits on an image see to that), so that they read as zero.
constexpr uint32_t kOutside = 0xfffffff0u;

}  // namespace rotconv
