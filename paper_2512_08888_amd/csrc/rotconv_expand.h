// Expansion of the base bank(s) into first-quadrant banks (Sec. III-D / Eq. 17) inside the kernels that pack a layer's
// weights.  These kernels are small and run ahead of a large one that waits for them, so their time is the length of their
// chain of dependent loads: every load of a tap is issued whether its coefficient is used or not (under a branch each would be
// waited for before the next: 12-17 us a launch, 5-9 so), the plans whose bank is the base bank itself look nothing up, and
// a thread forms three taps of nine.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "rotconv_bf16.h"
#include "rotconv_internal.h"

namespace rotconv {

struct ExpandTables {
  const int32_t* src;       // [(bank q, tap u)][kMaxNnz]: base bank * k^2 + base tap, or -1
  const float* coef;
  const double* coef64;     // bf16 plans
  int identity;             // one bank, which is the base bank
};

inline ExpandTables expand_tables(const rotconv_plan* p) {
  return ExpandTables{p->dev.fq_src, p->dev.fq_coef, p->dev.fq_coef64, p->base_bank};
}

__device__ __forceinline__ float weight_value(float v) { return v; }
__device__ __forceinline__ float weight_value(uint16_t v) { return bf16_to_f32(v); }

// Tap u of bank q from the k^2 taps of a (filter, channel) at src (a valid address; !in: the result is zero).  round16: bf16
// plans, the combination in fp64, rounded to fp32 and to bf16 once each.
template <typename T>
__device__ __forceinline__ float expand_tap(const T* __restrict__ src, size_t bank_stride, int kk, int q, int u, bool in,
                                            const ExpandTables& t, bool round16) {
  if (t.identity) {
    const float v = weight_value(src[u]);
    return in ? v : 0.f;
  }
  const int row = (q * kk + u) * kMaxNnz;
  int s[kMaxNnz];
  float v[kMaxNnz];
#pragma unroll
  for (int z = 0; z < kMaxNnz; ++z) s[z] = t.src[row + z];
#pragma unroll
  for (int z = 0; z < kMaxNnz; ++z) {
    const int a = s[z] < 0 ? 0 : s[z];
    v[z] = weight_value(src[(size_t)(a / kk) * bank_stride + a % kk]);
  }
  if (round16) {
    double a64 = 0.0;
#pragma unroll
    for (int z = 0; z < kMaxNnz; ++z) {
      const double next = a64 + t.coef64[row + z] * (double)v[z];
      a64 = in && s[z] >= 0 ? next : a64;
    }
    return bf16_to_f32(f32_to_bf16((float)a64));
  }
  float acc = 0.f;
#pragma unroll
  for (int z = 0; z < kMaxNnz; ++z) {
    const float next = acc + t.coef[row + z] * v[z];
    acc = in && s[z] >= 0 ? next : acc;
  }
  return acc;
}

}  // namespace rotconv
