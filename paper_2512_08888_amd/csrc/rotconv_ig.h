// Passes of fp32 layers as one contraction with the four quarter turns apart (rotconv_ig_fwd.hip, rotconv_ig_bwd_data.hip,
// rotconv_ig_bwd_weight.hip).
#pragma once

#include <hip/hip_runtime.h>

#include "rotconv_internal.h"

namespace rotconv {

bool ig_fwd_supported(const rotconv_plan* p);                  // the layer is one that the kernels take
IgShape ig_fwd_shape(const rotconv_plan* p, size_t budget);     // budget: bytes for a block's weights and shares (0: no shares)
size_t ig_fwd_block_bytes(const rotconv_plan* p, const IgShape& s);     // packed weights of a filter block
size_t ig_fwd_pack_bytes(const rotconv_plan* p, const IgShape& s);      // ... of all
// y: pooled values with idx (pooled, one share), else the responses of every orientation, the shares one after the other.  The packed
// weights of as many filter blocks at a time as ws_bytes hold.
void launch_ig_fwd(const rotconv_plan* p, const IgShape& s, bool pooled, const float* x, const float* w, float* y, uint8_t* idx,
                   void* ws, size_t ws_bytes, hipStream_t st);


// Input gradient of the same layers with four turns, pooled over them.  Shapes as above, `blocks` of input channels; the budget is that
// of shares, beside the weights.
bool ig_bwd_data_supported(const rotconv_plan* p);
IgShape ig_bwd_data_shape(const rotconv_plan* p, size_t budget);
size_t ig_bwd_data_ws_bytes(const rotconv_plan* p, const IgShape& s);       // packed weights and shares
void launch_ig_bwd_data(const rotconv_plan* p, const IgShape& s, const float* gpool, const uint8_t* idx, const float* w, float* dx,
                        void* ws, hipStream_t st);


// Weight gradient of the same layers (k from 2, strides 1 and 2, rows of at least eight outputs).
bool ig_bwd_weight_supported(const rotconv_plan* p);
size_t ig_bwd_weight_ws_bytes(const rotconv_plan* p);
void launch_ig_bwd_weight(const rotconv_plan* p, const float* x, const float* gpool, const uint8_t* idx, float* dw, void* ws,
                          hipStream_t st);

}  // namespace rotconv
