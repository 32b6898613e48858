// Forward (and weight gradient) of layers with at most four input channels on the vector ALU.
#pragma once

#include <hip/hip_runtime.h>

#include "rotconv_internal.h"

namespace rotconv {

bool direct_fwd_supported(const rotconv_plan* p);
size_t direct_fwd_pack_floats(const rotconv_plan* p);
// x, ypool: float for fp32 plans, bfloat16 for bf16 plans
void launch_direct_fwd(const rotconv_plan* p, const void* x, const void* w, void* ypool, uint8_t* idx, float* wb,
                       hipStream_t st);

// the same on bf16 parts: fp32 plans of at most three channels, a single bank of four quarter turns
bool first_fwd_layer(const rotconv_plan* p);      // ... for tensors on their alignment
bool first_fwd_supported(const rotconv_plan* p, const void* x, const void* ypool, const void* idx);
void launch_first_fwd(const rotconv_plan* p, const float* x, const float* w, float* ypool, uint8_t* idx, hipStream_t st);

// the weight gradient on bf16 parts: fp32 plans, single bank of four quarter turns
bool first_bwd_weight_layer(const rotconv_plan* p);
size_t first_bwd_weight_ws_floats(const rotconv_plan* p);
void launch_first_bwd_weight(const rotconv_plan* p, const float* x, const float* gpool, const uint8_t* idx, float* part,
                             float* dw, hipStream_t st);

// weight gradient (single-bank layers): `part` holds direct_bwd_weight_ws_floats(p) floats of partial sums
bool direct_bwd_weight_supported(const rotconv_plan* p);
size_t direct_bwd_weight_ws_floats(const rotconv_plan* p);
void launch_direct_bwd_weight(const rotconv_plan* p, const void* x, const void* gpool, const uint8_t* idx, float* part,
                              float* dw, hipStream_t st);

}  // namespace rotconv
