// Instances of the fused forward on products of the base bank (rotconv_p4_fwd_base_kernel.h) that multiply the operands' bf16
// parts.
#include <hip/hip_runtime.h>

#include "rotconv_kernels.h"
#include "rotconv_p4_fwd_base_kernel.h"

namespace rotconv {
namespace {

struct Args {
  const float *x, *wt, *w, *coef;
  const int32_t* rot_of;
  float* ov;
  uint8_t* oi;
};

template <int NWX, int NWY, bool FASTW, bool STREAM, int NQ, int CLS, int PARK>
void go(const P4Geom& g, const Args& a, hipStream_t st) {
  const size_t lds = (size_t)(STREAM ? 2 : g.cper) * kS3FwdChunk * 4 + base_lds_extra(PARK);
  auto kern = k_p4_fwd_base<NWX, NWY, FASTW, STREAM, 8, NQ, CLS, PARK, true>;
  (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  hipLaunchKernelGGL(kern, dim3((g.units + 7) / 8 * 8), dim3(64 * NWX * NWY), lds, st, a.x, a.wt, a.w, a.coef, a.rot_of, a.ov,
                     a.oi, g);
}

template <int NWX, int NWY, int NQ, int CLS>
void go_rows(const P4Geom& g, bool whole, bool stream, const Args& a, hipStream_t st) {
  constexpr int deep = parts_park(NQ, 4), flat = parts_park(NQ, 2), one = parts_park(NQ, 1);
  if (stream) {
    if (whole) go<NWX, NWY, true, true, NQ, CLS, parts_park(NQ, 0)>(g, a, st);
    else go<NWX, NWY, false, true, NQ, CLS, parts_park(NQ, 0)>(g, a, st);
  } else if (parts_park(NQ, g.cper) == deep) {
    if (whole) go<NWX, NWY, true, false, NQ, CLS, deep>(g, a, st);
    else go<NWX, NWY, false, false, NQ, CLS, deep>(g, a, st);
  } else if (parts_park(NQ, g.cper) == one) {
    if (whole) go<NWX, NWY, true, false, NQ, CLS, one>(g, a, st);
    else go<NWX, NWY, false, false, NQ, CLS, one>(g, a, st);
  } else {
    if (whole) go<NWX, NWY, true, false, NQ, CLS, flat>(g, a, st);
    else go<NWX, NWY, false, false, NQ, CLS, flat>(g, a, st);
  }
}

template <int NQ, int CLS>
void go_chain(const P4Geom& g, bool whole, bool stream, const Args& a, hipStream_t st) {
  switch (g.nwx) {
    case 1: go_rows<1, 8, NQ, CLS>(g, whole, stream, a, st); break;
    case 2: go_rows<2, 4, NQ, CLS>(g, whole, stream, a, st); break;
    case 4: go_rows<4, 2, NQ, CLS>(g, whole, stream, a, st); break;
    default: go_rows<8, 1, NQ, CLS>(g, whole, stream, a, st); break;
  }
}

}  // namespace

void launch_p4_fwd_base_parts(const rotconv_plan* p, const P4Geom& g, bool stream, const float* x, const float* wt, const float* w,
                              float* ypool, uint8_t* idx, hipStream_t st) {
  const Args a{x, wt, w, p->dev.fwd_base_coef, p->dev.rot_of, ypool, idx};
  const bool whole = (p->d.W & 3) == 0 && g.inside;
  if (p->fwd_base_cls == kCls16) go_chain<4, kCls16>(g, whole, stream, a, st);
  else if (p->fwd_base_cls == kCls8) go_chain<2, kCls8>(g, whole, stream, a, st);
  else go_chain<2, kClsP4m>(g, whole, stream, a, st);
}

}  // namespace rotconv
