// extern "C" entry points of the rotation-convolution library (see include/rotconv.h).
// This layer checks arguments, uploads the plan's tables on first use, picks the
// kernel family and enqueues; it never synchronises with the host.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cstring>

#include "rotconv_kernels.h"
#include "rotconv_bf16.h"
#include "rotconv_p4.h"
#include "rotconv_gs.h"
#include "rotconv_ig.h"
#include "rotconv_direct.h"
#include "rotconv_px_fwd_bf16.h"

namespace rotconv {

namespace {

template <typename T>
bool upload(const std::vector<T>& h, T** d) {
  const size_t bytes = std::max<size_t>(h.size(), 1) * sizeof(T);
  if (hipMalloc(reinterpret_cast<void**>(d), bytes) != hipSuccess) return false;
  if (!h.empty() && hipMemcpy(*d, h.data(), h.size() * sizeof(T), hipMemcpyHostToDevice) != hipSuccess) return false;
  return true;
}

}  // namespace

int ensure_device_tables(rotconv_plan* p) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess) return ROTCONV_ERR_LAUNCH;
  if (p->dev.device == dev) return ROTCONV_OK;
  if (p->dev.device >= 0) return ROTCONV_ERR_UNSUPPORTED;  // a plan is bound to the first device it ran on
  const HostTables& t = p->host;
  DeviceTables& d = p->dev;
  std::vector<int32_t> rq(p->d.R);
  for (int r = 0; r < p->d.R; ++r) rq[r] = t.bank_of_r[r] * 4 + t.quarter_of_r[r];
  const bool bf = p->d.dtype == ROTCONV_BF16;      // only bf16 plans read the fp64 coefficients
  const std::vector<double> none64;
  const bool ok = upload(t.exp_src, &d.exp_src) && upload(t.exp_coef, &d.exp_coef) && upload(t.tr_ptr, &d.tr_ptr) &&
                  upload(t.tr_col, &d.tr_col) && upload(t.tr_coef, &d.tr_coef) && upload(t.fq_src, &d.fq_src) &&
                  upload(t.fq_coef, &d.fq_coef) && upload(t.fqt_ptr, &d.fqt_ptr) && upload(t.fqt_col, &d.fqt_col) &&
                  upload(t.fqt_coef, &d.fqt_coef) && upload(p->rot_of, &d.rot_of) && upload(rq, &d.rq_of_r) &&
                  upload(t.turn_tap, &d.turn_tap) && upload(t.lut_bwd, &d.lut_bwd) &&
                  upload(bf ? t.exp_coef64 : none64, &d.exp_coef64) && upload(bf ? t.fq_coef64 : none64, &d.fq_coef64) &&
                  upload(t.fwd_base_coef, &d.fwd_base_coef) && upload(bf ? t.fq_dense64 : none64, &d.fq_dense64);
  if (!ok) {
    (void)hipGetLastError();
    free_device_tables(p);
    return ROTCONV_ERR_LAUNCH;
  }
  d.device = dev;
  // the plans this one runs some passes through: their tables go up with the parent's, so that no pass of the
  // parent allocates after the parent's first call
  for (rotconv_plan* ch : {p->avg_child, p->pad_child})
    if (ch) {
      const int rc = ensure_device_tables(ch);
      if (rc != ROTCONV_OK) return rc;
    }
  return ROTCONV_OK;
}

void free_device_tables(rotconv_plan* p) {
  DeviceTables& d = p->dev;
  void* ptrs[] = {d.exp_src, d.exp_coef, d.tr_ptr, d.tr_col, d.tr_coef, d.fq_src,
                  d.fq_coef, d.fqt_ptr, d.fqt_col, d.fqt_coef, d.rot_of, d.rq_of_r, d.turn_tap, d.lut_bwd,
                  d.exp_coef64, d.fq_coef64, d.fwd_base_coef, d.fq_dense64};
  for (void* q : ptrs)
    if (q) (void)hipFree(q);
  d = DeviceTables();
}

// Are the plan's tables (and those of the plans it runs passes through) on the current device already?
bool tables_on_current_device(const rotconv_plan* p) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || p->dev.device != dev) return false;
  for (const rotconv_plan* ch : {p->avg_child, p->pad_child})
    if (ch && !tables_on_current_device(ch)) return false;
  return true;
}

namespace {

int finish() { return hipGetLastError() == hipSuccess ? ROTCONV_OK : ROTCONV_ERR_LAUNCH; }

size_t align256(size_t v) { return (v + 255) / 256 * 256; }

bool aligned(const void* p, size_t a) { return reinterpret_cast<uintptr_t>(p) % a == 0; }

// Bytes reserved for the packed banks of the fast forward: the larger of the fp32 kernels' image and, for bf16 plans, the
// bf16 kernel's.
size_t fwd_pack_region(const rotconv_plan* p) {
  size_t b = p4_fwd_pack_floats(p) * sizeof(float);
  if (p->d.dtype == ROTCONV_BF16) b = std::max(b, p4_fwd_bf16_pack_bytes(p));
  return align256(b);
}

// Scratch of the fast forward beside the packed banks: per-bank candidates or the unpooled map.
size_t fwd_extra_bytes(const rotconv_plan* p) {
  const size_t hw = (size_t)p->d.H * p->d.W;
  const int mode = p4_fwd_pool_mode(p);
  if (mode == kOutPartial) return align256((size_t)p->host.Q * p->d.N * p->d.Cout * hw * 4) +
                                  align256((size_t)p->host.Q * p->d.N * p->d.Cout * hw);
  if (mode == kOutUnpooled) return align256((size_t)p->d.N * p->d.Cout * p->d.R * hw * 4);
  return 0;
}

// One unpooled part per channel split (of all filters, or of some).
size_t fwd_part_bytes(const rotconv_plan* p, int cs, int filters = 0) {
  return cs > 1 ? align256((size_t)cs * p->d.N * (filters ? filters : p->d.Cout) * p->d.R * p->d.H * p->d.W * 4) : 0;
}

size_t fwd_fast_ws_bytes(const rotconv_plan* p) {
  const int cs = std::max(p->fwd_csplit[0], p->fwd_csplit[1]);
  return fwd_pack_region(p) + std::max(fwd_extra_bytes(p), fwd_part_bytes(p, cs));
}

// What the pooled forward can make do with: banks of four bytes a weight beside its candidates, or one filter block's
// image beside its channel parts (a larger image is packed and multiplied in slices of filter blocks, bit for bit the
// same result).
size_t fwd_fast_least_bytes(const rotconv_plan* p) {
  const int cs = p->fwd_csplit[1], nq = cs == 1 && p4_fwd_pool_mode(p) == kOutPartial ? p4_fwd_fold(p) : 1;
  const size_t block = p->fwd_base ? 0 : p4_fwd_least_pack_bytes(p, nq, cs);
  const size_t bf = p->d.dtype == ROTCONV_BF16 ? p4_fwd_bf16_pack_bytes(p) : 0;
  if (cs > 1) return align256(std::max(block, bf)) + fwd_part_bytes(p, cs, p->fwd_sliced ? std::min(16, p->d.Cout) : 0);
  return align256(std::max({p4_fwd_weights(p) * sizeof(float), block, bf})) + fwd_extra_bytes(p);
}

// The fp32 forward's form and channel splits.  The waves on their own split more layers than the chained ones (4x994 -> 69, 19x70,
// eight turns: eight parts of 12 MB, modelled 206 us instead of 291), which must not cost the call without a workspace a
// layer that it took: where chained waves would not split and the whole contraction is one that rotconv_pool_fwd_static
// holds, it takes the parts in slices of filter blocks, bit for bit the same, or, where one block's do not fit, the contraction
// stays whole for every call.  A layer of one filter block, whose parts cannot be packed in slices, keeps
// the fp32 instructions where rotconv_pool_fwd_static holds its banks at four bytes a weight but not at six.
void choose_fwd(rotconv_plan* p) {
  // fp32 copies in front of a call's scratch: widened ones of bf16 tensors; padded ones of odd rows, on chained waves
  const rotconv_desc& d = p->d;
  const double hw4 = 4.0 * d.N * d.H * d.W, nx = hw4 * d.Cin, ny = hw4 * d.Cout * d.R;
  const double widened = d.dtype == ROTCONV_BF16 ? nx + ny + 36.0 * p->B * d.Cout * d.Cin : 0.;
  const double padded = d.dtype == ROTCONV_F32 && (d.W & 1) ? nx + ny : 0.;
  auto choose = [&](int s3) {
    p->fwd_s3 = s3;
    p->fwd_csplit[0] = p4_fwd_csplit(p, false);
    p->fwd_csplit[1] = p4_fwd_csplit(p, true);
    const auto fits = [&](double front) { return front + fwd_fast_least_bytes(p) <= (double)ROTCONV_STATIC_SCRATCH_BYTES; };
    const int split = p->fwd_csplit[1];
    p->fwd_sliced = 0;
    if (split > 1 && s3 && p->opt.fwd_csplit == 0 && !fits(widened) && p4_fwd_chain_whole(p)) {
      p->fwd_csplit[1] = 1;
      const bool whole = fits(widened + padded);
      p->fwd_csplit[1] = split;
      p->fwd_sliced = whole;
      if (whole && !fits(widened)) {
        p->fwd_csplit[1] = 1;
        p->fwd_sliced = 0;
      }
    }
    return fits(0.);
  };

  const int s3 = p4_fwd_parts_wanted(p);
  if (!choose(s3) && s3 && p->d.Cout <= 16 && p->opt.bf16_parts == 0 && p4_fwd_f32_rows(p) && !choose(0)) choose(1);
  p4_fwd_choose_launches(p);
}

// One contraction over channels and taps instead of products that are placed, or of gradients routed through memory.
// Filters of other sizes and strides with the four quarter turns, pooled, whose products it forms four times as often: 60 layers
// of 12 to 64 channels and filters, k = 2, 5, 7, stride 1 and 2: forward 0.45, weight gradient 0.49, input gradient 0.31 of the
// time in the mean, at most 0.78, 0.97 and 0.81.  With a stride of up to 8 wherever a tile fits LDS (4x128 -> 128, 128x128, stride 2
// 429 -> 102, 379 -> 160, 303 -> 144 us; 120 layers, k = 1 to 7, strides 3 to 8: input gradient 0.42 in the mean, 0.09 to 0.83;
// forward 0.61, 0.20 to 1.06, but 1 x 1 with a stride from 5 on, which uses few of the pixels it stages, 0.41 to 1.25; the weight
// gradient has strides 1 and 2 only).  k = 8 to 15, 40 layers: forward 0.03 to 0.58, input gradient 0.03 to 0.97, weight gradient
// 0.09 to 1.02.
// Without a stride, 70 layers of 48 to 400 channels: the forward up to 96 (0.51 to 0.98; 161 and more 0.6 to 1.7), the weight
// gradient up to 64 with up to 128 filters (0.43 to 0.97; beyond up to 2.0), the input gradient up to 64, and where the other's
// matrix multiply has fewer tiles (64 x 64) than the chip has CUs (0.10 to 0.91; beyond up to 1.6).
// Single orientations: with other filters and strides always (120 layers of 5 to 400 channels and filters, k = 1 to 8, strides 1
// to 8: 0.38 in the mean, 0.02 to 0.93); 3 x 3 at stride 1 where modelled at less than 0.85 of the time of the kernels that place
// (200 layers of 5 to 600 channels and filters: 0.93 in the mean of all with that rule, 0.23 to 1.05; taken everywhere up to 1.3 on
// large maps).
// Not for few filters, of which a tile has 16: stride 1 and at most eight from 5e9 products of one turn on (padded, times the
// padding: 7x66 -> 1, 238x240, 5 x 5 125 us and 417 so; 148 layers above the line 0.45 to 3.34, 1.21 in the mean), single
// orientations from 20e9; nor for 1 x 1 to 2 x 2 filters with longer strides, more than 64 channels and 3 MB of images, of whose staged
// pixels few are used (3x114 -> 50, 212x33, 1 x 1, stride 3 19 / 37; 0.6 to 2.0).
// The input gradient from nine filters on, eight from 5 x 5 taps on: with fewer a sum of 32 is mostly padding (4x59 -> 3, 198x105,
// 5 x 5 49 us and 150 so) and its cuts show (error up to 1.23 of the routed form's, from there on 0.71 in the mean); and not for
// filters smaller than their stride with up to 24 filters from 30 MB of images on (8x235 -> 14, 180x81, 1 x 1, stride 4 53 / 112).
// The weight gradient not for at most eight filters from 4e9 such products on, strided 12e9 (4x112 -> 1, 292x170, 7 x 7, stride 2 70 us
// and 268 so; above the line 1.15 in the mean), nor 2 x 2 taps where three of four products are padding and there are
// more than 20000 outputs (8x3 -> 1, 50x146 24 / 43; 0.9 to 1.8).
// averaged: the plan of an averaged bank (or its padded one), whose forward is the one that the call without a workspace runs: on
// the kernels that place, whose scratch is small.
size_t ig_part_bytes(const rotconv_plan* p, const IgShape& s) {
  return s.parts() > 1 ? align256((size_t)s.parts() * p->d.N * p->d.Cout * p->d.R * p->Ho * p->Wo * 4) : 0;
}
// ... and the least that either forward makes do with: the shares and one block's weights
size_t ig_least_bytes(const rotconv_plan* p, const IgShape& s) { return ig_part_bytes(p, s) + ig_fwd_block_bytes(p, s); }
// rows or columns of whole tiles for each one there is
double padding(int n, int tile) { return (double)((n + tile - 1) / tile * tile) / n; }
void choose_ig(rotconv_plan* p, bool averaged) {
  if (!ig_fwd_supported(p) || p->d.stride > 8) return;
  if (p->gs && p->opt.gs == 0) {
    // what rotconv_pool_fwd_static holds wherever it holds the products (behind widened copies that may be less than its array); no
    // more than these where the caller bounds them (option gs_chunk_mb)
    const bool bounded = p->opt.gs_chunk_mb != 0;
    size_t holds = gs_ws_bytes(p);
    if (p->d.dtype == ROTCONV_F32 && !bounded) holds = std::max<size_t>(holds, ROTCONV_STATIC_SCRATCH_BYTES);
    const rotconv_desc& d = p->d;
    const bool strided = d.stride > 1;
    const double image_bytes = 4.0 * d.N * d.Cin * d.H * d.W;      // of all images
    // products of one turn, filters padded to a tile, times what the padding adds to each that is needed
    const double outputs = (double)d.N * p->Ho * p->Wo, padded = padding(d.Cout, 16);
    const double products = outputs * p->kk * d.Cin * d.Cout * padded * padded;
    bool fwd = strided ? d.stride <= 4 * d.k && (d.k >= d.stride || d.stride < 3 || d.Cin <= 64 || image_bytes < 3e6) : d.Cin <= 96;
    fwd = fwd || d.R == 1;
    if (!strided && d.Cout <= 8 && products * padding(d.Cin, 32) > (d.R == 1 ? 20e9 : 5e9)) fwd = false;
    const IgShape s = !averaged && fwd ? ig_fwd_shape(p, holds) : IgShape();
    if (s.mt && ig_fwd_block_bytes(p, s) <= holds) p->ig[1] = s;
    if (d.R == 1) p->ig[0] = p->ig[1];
    const double narrow = padding(d.Cin, 16);
    const bool few = (d.Cout <= 8 && products * narrow > (strided ? 12e9 : 4e9)) ||
                     (!strided && d.k == 2 && padded * narrow >= 4 && outputs > 2e4);
    if ((strided || (d.Cin <= 64 && d.Cout <= 128)) && !few && ig_bwd_weight_supported(p)) {
      p->ig_dw = 1;
      p->ws_bytes = std::max(p->ws_bytes, ig_bwd_weight_ws_bytes(p));
    }
    const long tiles = (long)((d.Cin + 63) / 64) * ((d.H * d.W + 63) / 64) * d.N;
    const bool sparse = d.k < d.stride && d.Cout <= 24 && image_bytes > 3e7;
    if ((strided || d.Cin <= 64 || tiles < 256) && d.Cout >= (d.k < 5 ? 9 : 8) && !sparse && ig_bwd_data_supported(p))
      p->ig_dx = ig_bwd_data_shape(p, bounded ? std::min(gs_chunk_budget(p), (size_t)256 << 20) : (size_t)256 << 20);
    if (p->ig_dx.mt) p->ws_bytes = std::max(p->ws_bytes, ig_bwd_data_ws_bytes(p, p->ig_dx));
  } else if (!averaged && p->d.dtype == ROTCONV_F32 && p->d.R == 1 && p->fast[0] && p->opt.fwd_csplit == 0) {
    const IgShape s = ig_fwd_shape(p, (size_t)64 << 20);
    const double other = p4_fwd_us(p);
    if (s.mt && s.us < 0.85 * other) p->ig[0] = s;      // (other: negative where there is no such kernel)
  }
  for (const IgShape& s : p->ig)
    if (s.mt) p->ws_bytes = std::max(p->ws_bytes, ig_part_bytes(p, s) + align256(ig_fwd_pack_bytes(p, s)));
}
// Either forward of such a plan.
int run_ig(const rotconv_plan* p, bool pooled, const float* x, const float* w, float* y, uint8_t* idx, void* ws, size_t ws_bytes,
           hipStream_t st) {
  const IgShape& s = p->ig[pooled];
  if (ws_bytes < ig_least_bytes(p, s)) return ROTCONV_ERR_WORKSPACE;
  const size_t parts = ig_part_bytes(p, s);
  char* pack = static_cast<char*>(ws) + parts;
  if (!parts) {
    launch_ig_fwd(p, s, pooled, x, w, y, idx, pack, ws_bytes, st);
    return finish();
  }
  float* part = static_cast<float*>(ws);
  launch_ig_fwd(p, s, false, x, w, part, nullptr, pack, ws_bytes - parts, st);
  if (pooled) launch_p4_sum_pool(p, part, s.parts(), y, idx, 0, p->d.Cout, st);
  else launch_p4_sum_parts(p, part, s.parts(), y, st, true);
  return finish();
}

// the fp32 path's own need (a bf16 plan adds its staging areas in front, see carve())
int check_ws_inner(const rotconv_plan* p, const void* ws, size_t ws_bytes) {
  if (p->ws_inner == 0) return ROTCONV_OK;
  if (!ws || ws_bytes < p->ws_inner) return ROTCONV_ERR_WORKSPACE;
  return ROTCONV_OK;
}

// Scratch of an average-pooling plan: rotated banks, the group-averaged bank (or its gradient), an all-zero idx
// map for the R = 1 plan's fused gradient calls, then that plan's own scratch.
struct AvgLayout { size_t wexp, wavg, idx0, child, total; };
AvgLayout avg_layout(const rotconv_plan* p) {
  AvgLayout L;
  const size_t bank = (size_t)p->d.Cout * p->d.Cin * p->kk * sizeof(float);
  L.wexp = 0;
  L.wavg = align256((size_t)p->d.R * bank);
  L.idx0 = L.wavg + align256((size_t)p->ng * bank);
  L.child = L.idx0 + align256(p->n_yp);
  L.total = L.child + align256(p->avg_child ? p->avg_child->ws_bytes : 0);
  return L;
}

// Staging areas of a plan whose calls run on zero-padded rows (pad_child): an input-sized area, an output-sized area
// (pooled; unpooled if rotconv_fwd goes that way too), the idx map, then the child's own scratch.
struct PadLayout { size_t in, out, idx, child, total; };
PadLayout pad_layout(const rotconv_plan* p) {
  const rotconv_plan* ch = p->pad_child;
  const size_t es = p->d.dtype == ROTCONV_BF16 ? 2 : 4;
  PadLayout L;
  L.in = 0;
  L.out = align256(ch->n_x * es);
  L.idx = L.out + align256((p->pad_use[0] ? ch->n_yu : ch->n_yp) * es);
  L.child = L.idx + align256(ch->n_yp);
  L.total = L.child + align256(ch->ws_bytes);
  return L;
}

// Scratch with which the unfused gradient calls (dense dy) of an fp32 plan leave the generic kernels for the matrix
// multiply + scatter family; equals the plan's own need where that family is used anyway or does not apply.
size_t unfused_ws_inner(const rotconv_plan* p) {
  if (p->gs || p->d.pool_op == ROTCONV_POOL_AVG || !gs_wanted(p)) return p->ws_inner;
  return std::max(p->ws_inner, align256(gs_ws_bytes(p)));
}

// Do the unfused gradient calls (dense dy) run matrix multiply + scatter with this much scratch?  Plans whose fused
// calls run that family anyway: always; plans on the register-resident kernels: when the family is wanted for the
// layer and the caller brought rotconv_workspace_bytes_unfused.
bool unfused_on_gs(const rotconv_plan* p, const void* ws, size_t ws_bytes) {
  if (p->gs) return true;
  if (p->d.pool_op == ROTCONV_POOL_AVG || !gs_wanted(p)) return false;
  return ws && ws_bytes >= unfused_ws_inner(p);
}

// how a pass runs: 2 bf16 matrix-core kernel, 1 fp32 matrix-core kernel, 0 generic
int pass_level(const rotconv_plan* p, int pass) {
  if (p->direct[pass] || (pass == 0 && p->px16)) return 2;
  if (p->d.dtype == ROTCONV_BF16 && p->native16[pass]) return 2;
  return p->fast[pass] ? 1 : 0;
}

}  // namespace
}  // namespace rotconv

using namespace rotconv;

extern "C" {

int rotconv_plan_create(const rotconv_desc* desc, rotconv_plan** out) {
  return rotconv_plan_create_opt(desc, nullptr, out);
}

namespace {

// averaged: the plan is the one that an average-pooling plan runs its fused calls through, or that one's padded plan.
int create_plan(const rotconv_desc* desc, const rotconv_plan_options* opts, bool averaged, rotconv_plan** out) {
  if (!desc || !out) return ROTCONV_ERR_NULL;
  if (opts && (opts->reserved[0] || opts->reserved[1] || opts->reserved[2])) return ROTCONV_ERR_UNSUPPORTED;
  rotconv_plan* p = nullptr;
  const int rc = validate_and_build(desc, &p);
  if (rc != ROTCONV_OK) return rc;
  if (opts) p->opt = *opts;
  p->bwdw_splits = generic_bwdw_splits(p);
  p->ws_bytes = generic_ws_bytes(p);
  p->fast[0] = p4_fwd_supported(p) ? 1 : 0;
  if (p->fast[0]) choose_fwd(p);
  if (p->fast[0]) p->ws_bytes = std::max(p->ws_bytes, fwd_fast_ws_bytes(p));
  // one pool group over several banks: products of the base bank only.  Maps below 32 x 32 pixels with deep inputs
  // keep the channel split of the per-bank kernel where its cost model chose one (few workgroups either way).
  if (p->fast[0] && p4_fwd_base_supported(p) && (p->fwd_csplit[1] == 1 || (long)p->d.H * p->d.W >= 1024)) {
    p->fwd_base = 1;
    p->fwd_csplit[1] = 1;
    p->fwd_base_cls = p4_fwd_base_classify(p, &p->host.fwd_base_coef);
  }
  if (direct_fwd_supported(p)) {     // first layers: kernels of their own for the pooled forward
    p->direct[0] = 1;
    p->ws_bytes = std::max(p->ws_bytes, direct_fwd_pack_floats(p) * sizeof(float));
  }
  if (!p->direct[0] && px_fwd_bf16_supported(p)) {     // bf16, shallow layers: a lane per pixel column
    p->px16 = 1;
    p->ws_bytes = std::max(p->ws_bytes, px_fwd_bf16_pack_bytes(p));
  }
  if (direct_bwd_weight_supported(p)) {     // ... and, with a single bank, the weight gradient
    p->direct[2] = 1;
    p->ws_bytes = std::max(p->ws_bytes, direct_bwd_weight_ws_floats(p) * sizeof(float));
  }
  p->bwd_lut = p4_bwd_lut_choice(p) ? 1 : 0;
  p->fast[1] = p4_bwd_data_supported(p) ? 1 : 0;
  if (p->fast[1])
    p->ws_bytes = std::max(p->ws_bytes, align256(p4_bwd_data_pack_floats(p) * sizeof(float)) +
                                            p4_bwd_data_part_floats(p) * sizeof(float));
  if (s3_bwd_data_supported(p))
    p->ws_bytes = std::max(p->ws_bytes, align256(s3_bwd_data_pack_bytes(p)) + s3_bwd_data_part_floats(p) * sizeof(float));
  p->fast[2] = p4_bwd_weight_supported(p) ? 1 : 0;
  if (p->fast[2]) p->ws_bytes = std::max(p->ws_bytes, p4_bwd_weight_ws_floats(p) * sizeof(float));
  if (p->d.dtype == ROTCONV_BF16) {     // scratch of the kernels that take bf16 tensors directly
    if (p->fast[0] && p4_fwd_bf16_supported(p)) p->ws_bytes = std::max(p->ws_bytes, p4_fwd_bf16_pack_bytes(p));
    if (p->fast[1] && p4_bwd_data_bf16_supported(p))
      p->ws_bytes = std::max(p->ws_bytes, align256(p4_bwd_data_bf16_pack_bytes(p)) + p4_bwd_data_bf16_part_bytes(p));
    if (p->fast[1] && p4_bwd_data_bf16_lut_supported(p))
      p->ws_bytes = std::max(p->ws_bytes, align256(p4_bwd_data_bf16_lut_pack_bytes(p)) + p4_bwd_data_bf16_lut_part_bytes(p));
  }
  // other layers (k, stride, pad, or a pool group that cuts through a bank): matrix multiply + scatter
  const bool is3x3 = p->d.k == 3 && p->d.stride == 1 && p->d.pad == 1;
  if (!(p->fast[0] && p->fast[1] && p->fast[2]) && !(is3x3 && p4_fwd_pool_mode(p) != kOutUnpooled) && gs_wanted(p)) {
    p->gs = 1;
    p->gs_chunk_bytes = gs_chunk_budget(p);
    p->ws_bytes = std::max(p->ws_bytes, gs_ws_bytes(p));
  }
  choose_ig(p, averaged);
  p->ws_inner = p->ws_bytes = align256(p->ws_bytes);
  const size_t hw_in = (size_t)p->d.H * p->d.W, hw_out = (size_t)p->Ho * p->Wo;
  p->n_x = (size_t)p->d.N * p->d.Cin * hw_in;
  p->n_w = (size_t)p->B * p->d.Cout * p->d.Cin * p->kk;
  p->n_yp = (size_t)p->d.N * p->d.Cout * p->ng * hw_out;
  p->n_yu = (size_t)p->d.N * p->d.Cout * p->d.R * hw_out;
  if (p->d.dtype == ROTCONV_BF16) {
    p->ws_bytes = align256(p->n_x * 4) + align256(p->n_w * 4) + align256(p->n_yu * 4) + p->ws_inner;
    p->native16[0] = p->fast[0] && p4_fwd_bf16_supported(p) ? 1 : 0;
    p->native16[1] = p->fast[1] && p4_bwd_data_bf16_supported(p) ? 1 : 0;
    if (p->fast[1] && p4_bwd_data_bf16_lut_supported(p)) p->native16[1] = p->bwd_lut16[1] = 1;
    p->native16[2] = p->fast[2] && p4_bwd_weight_bf16_supported(p) ? 1 : 0;
    if (p->native16[2] && p4_bwd_lut16_choice(p)) p->bwd_lut16[2] = 1;
  }
  if (p->d.pool_op == ROTCONV_POOL_AVG) {
    // the fused calls of an average-pooling plan run an ordinary convolution (R = 1) with Cout * R/G filters
    rotconv_desc cd = p->d;
    cd.Cout = p->d.Cout * p->ng; cd.R = 1; cd.angles_deg = nullptr; cd.mode = ROTCONV_EXACT90; cd.pool_group = 0;
    cd.pool_op = ROTCONV_POOL_MAX;
    cd.dtype = ROTCONV_F32;       // a bf16 plan runs it on widened copies
    const int crc = create_plan(&cd, &p->opt, true, &p->avg_child);
    if (crc != ROTCONV_OK) {
      delete p;
      return crc;
    }
    const AvgLayout L = avg_layout(p);
    const size_t staging = p->ws_bytes - p->ws_inner;       // a bf16 plan's fp32 copies in front (0 for fp32 plans)
    p->ws_inner = std::max(p->ws_inner, L.total);
    p->ws_bytes = staging + p->ws_inner;
    p->native16[0] = p->native16[1] = p->native16[2] = 0;   // the fused calls go through the averaged bank in fp32
  }
  // 3x3 / stride 1 / pad 1 layers whose row width keeps a pass off the matrix-core kernels: the same layer on rows
  // padded to a multiple of 8 (32 beyond 256 pixels)
  if (p->d.pool_op != ROTCONV_POOL_AVG && p->d.k == 3 && p->d.stride == 1 && p->d.pad == 1) {
    const int top = p->d.dtype == ROTCONV_BF16 ? 2 : 1;
    const int Wp = p->d.W > 256 ? (p->d.W + 31) / 32 * 32 : (p->d.W + 7) / 8 * 8;
    const bool lacking = pass_level(p, 0) < top || pass_level(p, 1) < top || pass_level(p, 2) < top;
    if (lacking && Wp != p->d.W) {
      rotconv_desc cd = p->d;       // angles_deg points at the plan's own list (the defaults where none were given)
      cd.W = Wp;
      if (cd.mode == ROTCONV_P4M) cd.angles_deg = nullptr;   // that mode takes no explicit angles
      rotconv_plan* ch = nullptr;
      const int crc = create_plan(&cd, &p->opt, averaged, &ch);
      if (crc != ROTCONV_OK) {
        delete p;
        return crc;
      }
      int any = 0;
      for (int i = 0; i < 3; ++i) any |= p->pad_use[i] = pass_level(ch, i) > pass_level(p, i) ? 1 : 0;
      if (any) {
        p->pad_child = ch;
        p->ws_bytes = std::max(p->ws_bytes, pad_layout(p).total);
      } else {
        rotconv_plan_destroy(ch);
      }
    }
  }
  *out = p;
  return ROTCONV_OK;
}

}  // namespace

int rotconv_plan_create_opt(const rotconv_desc* desc, const rotconv_plan_options* opts, rotconv_plan** out) {
  return create_plan(desc, opts, false, out);
}

int rotconv_plan_destroy(rotconv_plan* plan) {
  if (!plan) return ROTCONV_OK;
  if (plan->avg_child) rotconv_plan_destroy(plan->avg_child);
  if (plan->pad_child) rotconv_plan_destroy(plan->pad_child);
  free_device_tables(plan);
  delete plan;
  return ROTCONV_OK;
}

size_t rotconv_workspace_bytes(const rotconv_plan* plan) { return plan ? plan->ws_bytes : 0; }

size_t rotconv_workspace_bytes_unfused(const rotconv_plan* plan) {
  if (!plan) return 0;
  if (plan->d.dtype == ROTCONV_BF16) return plan->ws_bytes - plan->ws_inner + unfused_ws_inner(plan);   // staging areas in front
  return std::max(plan->ws_bytes, unfused_ws_inner(plan));
}

int rotconv_out_shape(const rotconv_plan* plan, int32_t* Ho, int32_t* Wo, int32_t* Cunpooled, int32_t* Cpooled) {
  if (!plan) return ROTCONV_ERR_NULL;
  if (Ho) *Ho = plan->Ho;
  if (Wo) *Wo = plan->Wo;
  if (Cunpooled) *Cunpooled = plan->d.Cout * plan->d.R;
  if (Cpooled) *Cpooled = plan->d.Cout * plan->ng;
  return ROTCONV_OK;
}

int rotconv_plan_orientations(const rotconv_plan* plan, int32_t* Q, int32_t* bank_of_r, int32_t* quarter_of_r) {
  if (!plan) return ROTCONV_ERR_NULL;
  if (Q) *Q = plan->host.Q;
  for (int r = 0; r < plan->d.R; ++r) {
    if (bank_of_r) bank_of_r[r] = plan->host.bank_of_r[r];
    if (quarter_of_r) quarter_of_r[r] = plan->host.quarter_of_r[r];
  }
  return ROTCONV_OK;
}

int rotconv_plan_expansion(const rotconv_plan* plan, float* E) {
  if (!plan || !E) return ROTCONV_ERR_NULL;
  const int kk = plan->kk, B = plan->B, R = plan->d.R;
  std::memset(E, 0, sizeof(float) * R * kk * B * kk);
  for (int row = 0; row < R * kk; ++row)
    for (int e = 0; e < kMaxNnz; ++e) {
      const int s = plan->host.exp_src[row * kMaxNnz + e];
      if (s >= 0) E[(size_t)row * B * kk + s] += plan->host.exp_coef[row * kMaxNnz + e];
    }
  return ROTCONV_OK;
}

int rotconv_plan_routed_table(const rotconv_plan* plan, float* T) {
  if (!plan || !T) return ROTCONV_ERR_NULL;
  if (plan->host.lut_bwd.empty() || plan->B != 1) return ROTCONV_ERR_UNSUPPORTED;
  const int R1 = plan->d.R + 1;
  for (int rel = 0; rel < 9; ++rel)
    for (int r = 0; r < R1; ++r)
      for (int u = 0; u < 9; ++u) T[((size_t)rel * R1 + r) * 9 + u] = plan->host.lut_bwd[((size_t)rel * R1 + r) * 12 + u];
  return ROTCONV_OK;
}

}  // extern "C" (the fp32 implementations below have internal linkage)

// Alignment that the register-resident forward needs: that of a float (and a byte) where the waves are on their own, eight
// bytes of x for the pixel pairs of the others, vectors of the results where those kernels write them themselves (not the
// sums, maxima and combinations of what they leave in the scratch, which go element by element).
struct FwdAlign { size_t x, y, idx; };
static FwdAlign fwd_align(const rotconv_plan* p, bool pooled) {
  if (pooled && p->fwd_base) return {8, 16, 8};
  const rotconv_plan::FwdLaunch& l = p->fwd_launch[pooled];
  if (!l.chain) return {4, 4, 1};
  const bool direct = l.csplit == 1 && l.out_mode == (pooled ? kOutPooled : kOutUnpooled);
  return {8, (size_t)(direct ? 16 : 4), (size_t)(direct ? 8 : 1)};
}

// Does the unpooled forward of an fp32 plan run the register-resident kernel for these pointers?
static bool f32_fwd_is_fast(const rotconv_plan* p, const void* x, const void* y, const void* ws) {
  const FwdAlign a = fwd_align(p, false);
  return p->fast[0] && aligned(x, a.x) && aligned(ws, p->fwd_csplit[0] > 1 ? 256 : 16) && aligned(y, a.y);
}

// Scratch of either forward off the register-resident kernels: the products of a few images, or the rotated banks.
static size_t f32_other_fwd_need(const rotconv_plan* p) {
  return p->gs ? gs_ws_bytes(p) : align256((size_t)p->d.R * p->d.Cout * p->d.Cin * p->kk * sizeof(float));
}

// Does a forward of an fp32 plan run as one contraction over channels and taps for these pointers?
static bool f32_fwd_is_ig(const rotconv_plan* p, bool pooled, const void* x, const void* y, const void* ws) {
  return p->ig[pooled].mt && aligned(x, 4) && aligned(y, 4) && aligned(ws, 256);
}

// Scratch the unpooled forward of an fp32 plan needs for these pointers, whatever the plan's other calls need.
static size_t f32_fwd_need(const rotconv_plan* p, const void* x, const void* y, const char* ws) {
  if (p->pad_child && p->pad_use[0]) {
    const PadLayout L = pad_layout(p);
    return L.child + f32_fwd_need(p->pad_child, ws + L.in, ws + L.out, ws + L.child);
  }
  if (f32_fwd_is_ig(p, false, x, y, ws)) return ig_least_bytes(p, p->ig[0]);
  const int cs = p->fwd_csplit[0];
  return f32_fwd_is_fast(p, x, y, ws) ? fwd_part_bytes(p, cs) + p4_fwd_least_pack_bytes(p, 1, cs) : f32_other_fwd_need(p);
}

static int fwd_impl(const rotconv_plan* plan, const void* x, const void* w, void* y, void* ws, size_t ws_bytes,
                    void* stream, bool own_need);

// own_need: `ws` has to hold what this call touches (f32_fwd_need), not the plan's largest call
static int f32_rotconv_fwd(const rotconv_plan* plan, const void* x, const void* w, void* y, void* ws, size_t ws_bytes,
                void* stream, bool own_need = false) {
  if (!plan || !x || !w || !y) return ROTCONV_ERR_NULL;
  const size_t need = own_need ? f32_fwd_need(plan, x, y, static_cast<const char*>(ws)) : plan->ws_inner;
  if (need && (!ws || ws_bytes < need)) return ROTCONV_ERR_WORKSPACE;
  int rc;
  rotconv_plan* p = const_cast<rotconv_plan*>(plan);
  if ((rc = ensure_device_tables(p))) return rc;
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (f32_fwd_is_ig(p, false, x, y, ws))
    return run_ig(p, false, static_cast<const float*>(x), static_cast<const float*>(w), static_cast<float*>(y), nullptr, ws, ws_bytes, st);
  const int cs = p->fwd_csplit[0];
  if (f32_fwd_is_fast(p, x, y, ws)) {
    const size_t parts = fwd_part_bytes(p, cs);       // small map, deep input: the channels are split over workgroups
    float* out = cs > 1 ? static_cast<float*>(ws) : static_cast<float*>(y);
    launch_p4_fwd(p, kOutUnpooled, static_cast<const float*>(x), static_cast<const float*>(w),
                  reinterpret_cast<float*>(static_cast<char*>(ws) + parts), ws_bytes - parts, out, nullptr, st, 1, cs);
    if (cs > 1) launch_p4_sum_parts(p, out, cs, static_cast<float*>(y), st);
    return finish();
  }
  if (p->gs) {
    launch_gs_fwd(p, static_cast<const float*>(x), static_cast<const float*>(w), static_cast<float*>(y), ws, st);
    return finish();
  }
  float* wexp = static_cast<float*>(ws);
  launch_expand_bank(p, static_cast<const float*>(w), wexp, st);
  launch_fwd_generic(p, static_cast<const float*>(x), wexp, static_cast<float*>(y), st);
  return finish();
}

static int f32_rotconv_bwd_data(const rotconv_plan* plan, const void* dy, const void* w, void* dx, void* ws, size_t ws_bytes,
                     void* stream) {
  if (!plan || !dy || !w || !dx) return ROTCONV_ERR_NULL;
  int rc = check_ws_inner(plan, ws, ws_bytes);
  if (rc) return rc;
  rotconv_plan* p = const_cast<rotconv_plan*>(plan);
  if ((rc = ensure_device_tables(p))) return rc;
  hipStream_t st = static_cast<hipStream_t>(stream);
  // the unfused gradients of a plan whose fused calls run the register-resident kernels: matrix multiply + scatter
  // if the caller brought the larger workspace that family needs (rotconv_workspace_bytes_unfused), else generic
  if (unfused_on_gs(p, ws, ws_bytes)) {
    launch_gs_bwd_data(p, static_cast<const float*>(dy), static_cast<const float*>(w), static_cast<float*>(dx), ws, st);
    return finish();
  }
  float* wexp = static_cast<float*>(ws);
  launch_expand_bank(p, static_cast<const float*>(w), wexp, st);
  launch_bwd_data_generic(p, static_cast<const float*>(dy), wexp, static_cast<float*>(dx), st);
  return finish();
}

static int f32_rotconv_bwd_weight(const rotconv_plan* plan, const void* x, const void* dy, float* dw, void* ws, size_t ws_bytes,
                       void* stream) {
  if (!plan || !x || !dy || !dw) return ROTCONV_ERR_NULL;
  int rc = check_ws_inner(plan, ws, ws_bytes);
  if (rc) return rc;
  rotconv_plan* p = const_cast<rotconv_plan*>(plan);
  if ((rc = ensure_device_tables(p))) return rc;
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (unfused_on_gs(p, ws, ws_bytes)) {
    launch_gs_bwd_weight(p, static_cast<const float*>(x), static_cast<const float*>(dy), dw, ws, st);
    return finish();
  }
  launch_bwd_weight_generic(p, static_cast<const float*>(x), static_cast<const float*>(dy), nullptr, nullptr,
                            static_cast<float*>(ws), dw, st);
  return finish();
}

static int f32_orient_maxpool_fwd(const rotconv_plan* plan, const void* y, void* ypool, uint8_t* idx, void* stream) {
  if (plan && plan->avg_child) {
    if (!y || !ypool) return ROTCONV_ERR_NULL;
    launch_avgpool_fwd(plan, static_cast<const float*>(y), static_cast<float*>(ypool), static_cast<hipStream_t>(stream));
    return finish();
  }
  if (!plan || !y || !ypool || !idx) return ROTCONV_ERR_NULL;
  launch_maxpool_fwd(plan, static_cast<const float*>(y), static_cast<float*>(ypool), idx,
                     static_cast<hipStream_t>(stream));
  return finish();
}

static int f32_orient_maxpool_bwd(const rotconv_plan* plan, const void* gpool, const uint8_t* idx, void* dy, void* stream) {
  if (plan && plan->avg_child) {
    if (!gpool || !dy) return ROTCONV_ERR_NULL;
    launch_avgpool_bwd(plan, static_cast<const float*>(gpool), static_cast<float*>(dy), static_cast<hipStream_t>(stream));
    return finish();
  }
  if (!plan || !gpool || !idx || !dy) return ROTCONV_ERR_NULL;
  launch_maxpool_bwd(plan, static_cast<const float*>(gpool), idx, static_cast<float*>(dy),
                     static_cast<hipStream_t>(stream));
  return finish();
}

// Does the pooled forward of an fp32 plan run the register-resident kernel for these pointers?
static bool f32_pool_fwd_is_fast(const rotconv_plan* p, const void* x, const void* ypool, const uint8_t* idx,
                                 const void* ws) {
  const FwdAlign a = fwd_align(p, true);
  return !p->avg_child && p->fast[0] && aligned(x, a.x) && aligned(ws, 256) && aligned(ypool, a.y) && aligned(idx, a.idx);
}

// Scratch the pooled forward of an fp32 plan needs for these pointers, whatever the plan's other calls need: the packed
// banks (+ candidates) of the register-resident kernel, the averaged bank and its convolution, or the other families'.
static size_t f32_pool_fwd_need(const rotconv_plan* p, const void* x, const void* ypool, const uint8_t* idx,
                                const void* ws) {
  if (f32_pool_fwd_is_fast(p, x, ypool, idx, ws)) return std::min(p->ws_inner, fwd_fast_least_bytes(p));
  // (one contraction has to fit where the products, whose place it takes, would)
  if (!p->avg_child) return std::max(f32_other_fwd_need(p), f32_fwd_is_ig(p, true, x, ypool, ws) ? ig_least_bytes(p, p->ig[1]) : (size_t)0);
  const AvgLayout L = avg_layout(p);
  return L.child + f32_fwd_need(p->avg_child, x, ypool, static_cast<const char*>(ws) + L.child);
}

// no_upload: the caller may not allocate, so a plan whose tables are not on this device yet is refused
static int f32_rotconv_pool_fwd(const rotconv_plan* plan, const void* x, const void* w, void* ypool, uint8_t* idx, void* ws,
                     size_t ws_bytes, void* stream, bool own_need = false, bool no_upload = false) {
  if (!plan || !x || !w || !ypool || (!idx && !plan->avg_child)) return ROTCONV_ERR_NULL;
  // own_need: the buffer only has to hold what THIS call touches, not the plan's largest call
  const size_t need = own_need ? f32_pool_fwd_need(plan, x, ypool, idx, ws) : plan->ws_inner;
  if (need && (!ws || ws_bytes < need)) return ROTCONV_ERR_WORKSPACE;
  int rc;
  rotconv_plan* p = const_cast<rotconv_plan*>(plan);
  if (no_upload && !tables_on_current_device(p)) return ROTCONV_ERR_UNSUPPORTED;
  if ((rc = ensure_device_tables(p))) return rc;
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (p->avg_child) {     // Eq. 9: the mean over a group = one convolution with the group-averaged bank
    const AvgLayout L = avg_layout(p);
    char* c = static_cast<char*>(ws);
    float* wexp = reinterpret_cast<float*>(c + L.wexp);
    float* wavg = reinterpret_cast<float*>(c + L.wavg);
    launch_expand_bank(p, static_cast<const float*>(w), wexp, st);
    launch_avg_bank(p, wexp, wavg, st);
    return fwd_impl(p->avg_child, x, wavg, ypool, c + L.child, ws_bytes - L.child, stream, own_need);
  }
  if (f32_pool_fwd_is_fast(p, x, ypool, idx, ws)) {
    const int mode = p4_fwd_pool_mode(p);
    const size_t hw = (size_t)p->d.H * p->d.W;
    const float *xf = static_cast<const float*>(x), *wf = static_cast<const float*>(w);
    float* yf = static_cast<float*>(ypool);
    char* front = static_cast<char*>(ws);      // candidates / parts; the packed banks behind them
    auto run = [&](int m, size_t used, float* out, uint8_t* oi, int nq, int cs) {
      launch_p4_fwd(p, m, xf, wf, reinterpret_cast<float*>(front + used), ws_bytes - used, out, oi, st, nq, cs);
    };
    // small map, deep input: the channels are split over workgroups, summed and pooled afterwards
    const int cs = p->fwd_csplit[1];
    if (cs > 1) {
      float* part = reinterpret_cast<float*>(front);
      const size_t block = p4_fwd_least_pack_bytes(p, 1, cs);
      const int blocks = (p->d.Cout + 15) / 16;
      int per = blocks;                        // filter blocks at a time
      if (p->fwd_sliced)
        while (per > 1 && fwd_part_bytes(p, cs, std::min(p->d.Cout, 16 * per)) + block > ws_bytes) --per;
      for (int b = 0; b < blocks; b += per) {
        const int end = std::min(blocks, b + per), nc = std::min(p->d.Cout, 16 * end) - 16 * b;
        const size_t used = fwd_part_bytes(p, cs, nc);
        launch_p4_fwd_parts(p, b, end, xf, wf, reinterpret_cast<float*>(front + used), ws_bytes - used, part, st, cs);
        launch_p4_sum_pool(p, part, cs, yf, idx, 16 * b, nc, st);
      }
      return finish();
    }
    if (p->fwd_base) {     // the pool group spans all banks: products of the base bank, banks combined in the kernel
      launch_p4_fwd_base(p, xf, wf, static_cast<float*>(ws), yf, idx, st);
      return finish();
    }
    const int nq = mode == kOutPartial ? p4_fwd_fold(p) : 1;
    if (mode == kOutPooled) {
      run(mode, 0, yf, idx, 1, 1);
    } else if (nq > 1) {     // the pool group spans all banks: pooled across them inside the kernel
      run(kOutPooled, 0, yf, idx, nq, 1);
    } else if (mode == kOutPartial) {
      float* pv = reinterpret_cast<float*>(front);
      uint8_t* pi = reinterpret_cast<uint8_t*>(front + align256((size_t)p->host.Q * p->d.N * p->d.Cout * hw * 4));
      run(mode, fwd_extra_bytes(p), pv, pi, 1, 1);
      launch_p4_combine(p, pv, pi, yf, idx, st);
    } else {
      float* yu = reinterpret_cast<float*>(front);
      run(mode, fwd_extra_bytes(p), yu, nullptr, 1, 1);
      launch_maxpool_fwd(p, yu, yf, idx, st, true);
    }
    return finish();
  }
  if (f32_fwd_is_ig(p, true, x, ypool, ws))
    return run_ig(p, true, static_cast<const float*>(x), static_cast<const float*>(w), static_cast<float*>(ypool), idx, ws, ws_bytes, st);
  if (p->gs) {
    launch_gs_pool_fwd(p, static_cast<const float*>(x), static_cast<const float*>(w), static_cast<float*>(ypool), idx,
                       ws, st);
    return finish();
  }
  float* wexp = static_cast<float*>(ws);
  launch_expand_bank(p, static_cast<const float*>(w), wexp, st);
  launch_pool_fwd_generic(p, static_cast<const float*>(x), wexp, static_cast<float*>(ypool), idx, st);
  return finish();
}

static int f32_rotconv_pool_bwd_data(const rotconv_plan* plan, const void* gpool, const uint8_t* idx, const void* w, void* dx,
                          void* ws, size_t ws_bytes, void* stream) {
  if (!plan || !gpool || (!idx && !plan->avg_child) || !w || !dx) return ROTCONV_ERR_NULL;
  int rc = check_ws_inner(plan, ws, ws_bytes);
  if (rc) return rc;
  rotconv_plan* p = const_cast<rotconv_plan*>(plan);
  if ((rc = ensure_device_tables(p))) return rc;
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (p->avg_child) {     // Eq. 11 + 13 + 15: the input gradient of that one convolution (its only orientation is 0)
    const AvgLayout L = avg_layout(p);
    char* c = static_cast<char*>(ws);
    float* wexp = reinterpret_cast<float*>(c + L.wexp);
    float* wavg = reinterpret_cast<float*>(c + L.wavg);
    uint8_t* idx0 = reinterpret_cast<uint8_t*>(c + L.idx0);
    launch_expand_bank(p, static_cast<const float*>(w), wexp, st);
    launch_avg_bank(p, wexp, wavg, st);
    launch_fill_u8(idx0, p->n_yp, 0, st);
    return rotconv_pool_bwd_data(p->avg_child, gpool, idx0, wavg, dx, c + L.child, p->avg_child->ws_bytes, stream);
  }
  const bool odd = p->d.W & 1;       // (such rows are loaded and stored pixel by pixel)
  if (p->fast[1] && aligned(gpool, odd ? 4 : 8) && aligned(idx, odd ? 1 : 2) && aligned(dx, odd ? 4 : 16) && aligned(ws, 16)) {
    if (s3_bwd_data_supported(p)) {
      float* part = reinterpret_cast<float*>(static_cast<char*>(ws) + align256(s3_bwd_data_pack_bytes(p)));
      launch_s3_bwd_data(p, static_cast<const float*>(gpool), idx, static_cast<const float*>(w), ws, static_cast<float*>(dx), part, st);
      return finish();
    }
    const bool raw = p4_bwd_data_raw_weights(p) && aligned(w, 16);   // the kernel takes w itself, 16 bytes at a time
    const float* wd = static_cast<const float*>(w);
    if (!raw) {                                                       // ... or the banks packed into ws
      launch_p4_pack_bwd(p, static_cast<const float*>(w), static_cast<float*>(ws), st);
      wd = static_cast<const float*>(ws);
    }
    float* part = reinterpret_cast<float*>(static_cast<char*>(ws) + align256(p4_bwd_data_pack_floats(p) * sizeof(float)));
    launch_p4_bwd_data(p, static_cast<const float*>(gpool), idx, wd, static_cast<float*>(dx), part, st, raw);
    return finish();
  }
  if (p->ig_dx.mt && aligned(gpool, 4) && aligned(dx, 4) && aligned(ws, 256)) {
    launch_ig_bwd_data(p, p->ig_dx, static_cast<const float*>(gpool), idx, static_cast<const float*>(w), static_cast<float*>(dx), ws, st);
    return finish();
  }
  if (p->gs) {
    launch_gs_pool_bwd_data(p, static_cast<const float*>(gpool), idx, static_cast<const float*>(w),
                            static_cast<float*>(dx), ws, st);
    return finish();
  }
  float* wexp = static_cast<float*>(ws);
  launch_expand_bank(p, static_cast<const float*>(w), wexp, st);
  launch_pool_bwd_data_generic(p, static_cast<const float*>(gpool), idx, wexp, static_cast<float*>(dx), st);
  return finish();
}

static int f32_rotconv_pool_bwd_weight(const rotconv_plan* plan, const void* x, const void* gpool, const uint8_t* idx, float* dw,
                            void* ws, size_t ws_bytes, void* stream) {
  if (!plan || !x || !gpool || (!idx && !plan->avg_child) || !dw) return ROTCONV_ERR_NULL;
  int rc = check_ws_inner(plan, ws, ws_bytes);
  if (rc) return rc;
  rotconv_plan* p = const_cast<rotconv_plan*>(plan);
  if ((rc = ensure_device_tables(p))) return rc;
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (p->avg_child) {     // Eq. 11 + 14 + 16: that convolution's weight gradient, shared out to the R banks, reduced
    const AvgLayout L = avg_layout(p);
    char* c = static_cast<char*>(ws);
    float* rep = reinterpret_cast<float*>(c + L.wexp);
    float* dwavg = reinterpret_cast<float*>(c + L.wavg);
    uint8_t* idx0 = reinterpret_cast<uint8_t*>(c + L.idx0);
    launch_fill_u8(idx0, p->n_yp, 0, st);
    rc = rotconv_pool_bwd_weight(p->avg_child, x, gpool, idx0, dwavg, c + L.child, p->avg_child->ws_bytes, stream);
    if (rc) return rc;
    launch_avg_bank_bwd(p, dwavg, rep, dw, st);
    return finish();
  }
  const bool pixels = p->d.W & 3;       // (such rows are loaded pixel by pixel)
  if (p->fast[2] && aligned(x, pixels ? 4 : 16) && aligned(gpool, pixels ? 4 : 16) && aligned(idx, pixels ? 1 : 4) && aligned(ws, 16)) {
    launch_p4_bwd_weight(p, static_cast<const float*>(x), static_cast<const float*>(gpool), idx,
                         static_cast<float*>(ws), dw, st);
    return finish();
  }
  if (p->ig_dw && aligned(x, 4) && aligned(gpool, 4) && aligned(ws, 16)) {
    launch_ig_bwd_weight(p, static_cast<const float*>(x), static_cast<const float*>(gpool), idx, dw, ws, st);
    return finish();
  }
  if (p->gs) {
    launch_gs_pool_bwd_weight(p, static_cast<const float*>(x), static_cast<const float*>(gpool), idx, dw, ws, st);
    return finish();
  }
  launch_bwd_weight_generic(p, static_cast<const float*>(x), nullptr, static_cast<const float*>(gpool), idx,
                            static_cast<float*>(ws), dw, st);
  return finish();
}

extern "C" {

// ---- public entry points: fp32 plans go straight to the kernels; bf16 plans widen the bf16 tensors into
// fp32 staging areas at the head of the workspace, run the same kernels behind them, and round the results to
// bf16 once (the arg-max is taken on the fp32 values).  dW is fp32 in both cases. ----

namespace {

struct Stage {               // fp32 staging areas of a bf16 plan inside the caller's workspace
  float *x, *w, *y;          // input-sized, weight-sized, (unpooled-)output-sized
  void* inner;               // workspace handed on to the fp32 path
  size_t inner_bytes;
};

Stage carve(const rotconv_plan* p, void* ws, size_t ws_bytes) {
  Stage s;
  char* c = static_cast<char*>(ws);
  s.x = reinterpret_cast<float*>(c); c += align256(p->n_x * 4);
  s.w = reinterpret_cast<float*>(c); c += align256(p->n_w * 4);
  s.y = reinterpret_cast<float*>(c); c += align256(p->n_yu * 4);
  s.inner = c;
  s.inner_bytes = ws_bytes - (size_t)(c - static_cast<char*>(ws));
  return s;
}

bool is_bf16(const rotconv_plan* p) { return p->d.dtype == ROTCONV_BF16; }
const uint16_t* h16(const void* p) { return static_cast<const uint16_t*>(p); }

// The calls of a plan with padded rows: stage the tensors at the child's row width, run the child, crop.
struct PadCtx {
  const rotconv_plan* ch;
  char *in, *out, *idx, *cws;
  size_t cws_bytes;
  int es, W, Wp;
  size_t rows_x, rows_p, rows_u;    // rows of the input, the pooled and the unpooled maps
  hipStream_t st;
};
// need: the least the scratch has to hold (the child's share is what lies behind the staging areas)
int pad_ctx(const rotconv_plan* p, void* ws, size_t ws_bytes, void* stream, PadCtx* c, size_t need) {
  if (!ws || ws_bytes < need) return ROTCONV_ERR_WORKSPACE;
  const PadLayout L = pad_layout(p);
  char* b = static_cast<char*>(ws);
  c->cws_bytes = ws_bytes - L.child;
  c->ch = p->pad_child;
  c->in = b + L.in; c->out = b + L.out; c->idx = b + L.idx; c->cws = b + L.child;
  c->es = is_bf16(p) ? 2 : 4;
  c->W = p->d.W; c->Wp = p->pad_child->d.W;
  c->rows_x = (size_t)p->d.N * p->d.Cin * p->d.H;
  c->rows_p = (size_t)p->d.N * p->d.Cout * p->ng * p->d.H;
  c->rows_u = (size_t)p->d.N * p->d.Cout * p->d.R * p->d.H;
  c->st = static_cast<hipStream_t>(stream);
  return ROTCONV_OK;
}

}  // namespace

static int fwd_impl(const rotconv_plan* plan, const void* x, const void* w, void* y, void* ws, size_t ws_bytes,
                    void* stream, bool own_need) {
  if (!plan || !x || !w || !y) return ROTCONV_ERR_NULL;
  if (plan->pad_child && plan->pad_use[0]) {
    PadCtx c;
    int rc = pad_ctx(plan, ws, ws_bytes, stream, &c,
                     own_need ? f32_fwd_need(plan, x, y, static_cast<const char*>(ws)) : plan->ws_bytes);
    if (rc) return rc;
    launch_repitch(x, c.in, c.rows_x, c.W, c.Wp, c.es, 0, c.st);
    if ((rc = fwd_impl(c.ch, c.in, w, c.out, c.cws, c.cws_bytes, stream, own_need))) return rc;
    launch_repitch(c.out, y, c.rows_u, c.Wp, c.W, c.es, 0, c.st);
    return finish();
  }
  if (!is_bf16(plan)) return f32_rotconv_fwd(plan, x, w, y, ws, ws_bytes, stream, own_need);
  if (!ws || ws_bytes < plan->ws_bytes) return ROTCONV_ERR_WORKSPACE;
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (plan->native16[0] && aligned(x, 4) && aligned(w, 2) && aligned(ws, 256) && aligned(y, 16)) {
    rotconv_plan* p = const_cast<rotconv_plan*>(plan);
    const int rc = ensure_device_tables(p);
    if (rc) return rc;
    uint16_t* wt = static_cast<uint16_t*>(ws);
    launch_p4_pack_fwd_bf16(p, 1, h16(w), wt, st);
    launch_p4_fwd_bf16(p, kOutUnpooled, 1, h16(x), wt, y, nullptr, st);
    return finish();
  }
  const Stage s = carve(plan, ws, ws_bytes);
  launch_widen(h16(x), s.x, plan->n_x, st);
  launch_widen(h16(w), s.w, plan->n_w, st);
  const int rc = f32_rotconv_fwd(plan, s.x, s.w, s.y, s.inner, s.inner_bytes, stream);
  if (rc) return rc;
  launch_narrow(s.y, static_cast<uint16_t*>(y), plan->n_yu, st);
  return finish();
}

int rotconv_fwd(const rotconv_plan* plan, const void* x, const void* w, void* y, void* ws, size_t ws_bytes,
                void* stream) {
  return fwd_impl(plan, x, w, y, ws, ws_bytes, stream, false);
}

int rotconv_bwd_data(const rotconv_plan* plan, const void* dy, const void* w, void* dx, void* ws, size_t ws_bytes,
                     void* stream) {
  if (!plan || !dy || !w || !dx) return ROTCONV_ERR_NULL;
  if (!is_bf16(plan)) return f32_rotconv_bwd_data(plan, dy, w, dx, ws, ws_bytes, stream);
  if (!ws || ws_bytes < plan->ws_bytes) return ROTCONV_ERR_WORKSPACE;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const Stage s = carve(plan, ws, ws_bytes);
  launch_widen(h16(dy), s.y, plan->n_yu, st);
  launch_widen(h16(w), s.w, plan->n_w, st);
  const int rc = f32_rotconv_bwd_data(plan, s.y, s.w, s.x, s.inner, s.inner_bytes, stream);
  if (rc) return rc;
  launch_narrow(s.x, static_cast<uint16_t*>(dx), plan->n_x, st);
  return finish();
}

int rotconv_bwd_weight(const rotconv_plan* plan, const void* x, const void* dy, float* dw, void* ws, size_t ws_bytes,
                       void* stream) {
  if (!plan || !x || !dy || !dw) return ROTCONV_ERR_NULL;
  if (!is_bf16(plan)) return f32_rotconv_bwd_weight(plan, x, dy, dw, ws, ws_bytes, stream);
  if (!ws || ws_bytes < plan->ws_bytes) return ROTCONV_ERR_WORKSPACE;
  hipStream_t st = static_cast<hipStream_t>(stream);
  const Stage s = carve(plan, ws, ws_bytes);
  launch_widen(h16(x), s.x, plan->n_x, st);
  launch_widen(h16(dy), s.y, plan->n_yu, st);
  return f32_rotconv_bwd_weight(plan, s.x, s.y, dw, s.inner, s.inner_bytes, stream);
}

int orient_maxpool_fwd(const rotconv_plan* plan, const void* y, void* ypool, uint8_t* idx, void* stream) {
  if (!plan || !y || !ypool || (!idx && !plan->avg_child)) return ROTCONV_ERR_NULL;
  if (!is_bf16(plan)) return f32_orient_maxpool_fwd(plan, y, ypool, idx, stream);
  if (plan->avg_child) {
    launch_avgpool_fwd_bf16(plan, h16(y), static_cast<uint16_t*>(ypool), static_cast<hipStream_t>(stream));
    return finish();
  }
  launch_maxpool_fwd_bf16(plan, h16(y), static_cast<uint16_t*>(ypool), idx, static_cast<hipStream_t>(stream));
  return finish();
}

int orient_maxpool_bwd(const rotconv_plan* plan, const void* gpool, const uint8_t* idx, void* dy, void* stream) {
  if (!plan || !gpool || (!idx && !plan->avg_child) || !dy) return ROTCONV_ERR_NULL;
  if (!is_bf16(plan)) return f32_orient_maxpool_bwd(plan, gpool, idx, dy, stream);
  if (plan->avg_child) {
    launch_avgpool_bwd_bf16(plan, h16(gpool), static_cast<uint16_t*>(dy), static_cast<hipStream_t>(stream));
    return finish();
  }
  launch_maxpool_bwd_bf16(plan, h16(gpool), idx, static_cast<uint16_t*>(dy), static_cast<hipStream_t>(stream));
  return finish();
}

namespace {

// Does the pooled forward of a bf16 plan run the bf16 matrix-core kernel for these pointers?
bool bf16_pool_fwd_is_native(const rotconv_plan* plan, const void* x, const void* w, const void* ypool,
                             const uint8_t* idx, const void* ws) {
  const int pmode = plan->native16[0] ? p4_fwd_pool_mode(plan) : kOutUnpooled;
  return pmode != kOutUnpooled && aligned(x, 4) && aligned(w, 2) && aligned(ws, 256) && aligned(ypool, 16) &&
         aligned(idx, 8);
}

// Does the pooled forward run the kernels of layers with at most four input channels for these pointers?
bool pool_fwd_is_direct(const rotconv_plan* p, const void* x, const void* ypool, const void* ws) {
  const size_t es = is_bf16(p) ? 2 : 4;
  return p->direct[0] && aligned(x, es) && aligned(ypool, es) && aligned(ws, 16);
}

bool pool_fwd_is_px16(const rotconv_plan* p, const void* x, const void* ypool, const void* ws) {
  return p->px16 && aligned(x, 2) && aligned(ypool, 2) && aligned(ws, 16);
}

// Bytes of `ws` one call of the pooled forward touches, by the route it takes for these pointers (never more than
// rotconv_workspace_bytes, which is the largest need of any call on the plan).
size_t pool_fwd_need(const rotconv_plan* plan, const void* x, const void* w, const void* ypool, const uint8_t* idx,
                     const void* ws) {
  const char* c = static_cast<const char*>(ws);
  if (plan->pad_child && plan->pad_use[0]) {                                  // staging copies + the padded plan's call
    const PadLayout L = pad_layout(plan);
    return L.child + pool_fwd_need(plan->pad_child, c + L.in, w, c + L.out, reinterpret_cast<const uint8_t*>(c + L.idx), c + L.child);
  }
  if (pool_fwd_is_px16(plan, x, ypool, ws)) return align256(px_fwd_bf16_pack_bytes(plan));
  if (pool_fwd_is_direct(plan, x, ypool, ws)) return align256(direct_fwd_pack_floats(plan) * sizeof(float));
  if (!is_bf16(plan)) return f32_pool_fwd_need(plan, x, ypool, idx, ws);
  if (bf16_pool_fwd_is_native(plan, x, w, ypool, idx, ws)) return align256(p4_fwd_bf16_pack_bytes(plan)) + fwd_extra_bytes(plan);
  const Stage s = carve(plan, const_cast<void*>(ws), 0);                      // fp32 staging areas in front
  return (size_t)(static_cast<const char*>(s.inner) - c) + f32_pool_fwd_need(plan, s.x, s.y, idx, s.inner);
}

// own_need: `ws` has to hold what this call touches (pool_fwd_need), not the plan's largest call.
// no_upload: no allocation allowed: a plan whose tables are not on the current device yet is refused.
int pool_fwd_impl(const rotconv_plan* plan, const void* x, const void* w, void* ypool, uint8_t* idx, void* ws,
                  size_t ws_bytes, void* stream, bool own_need, bool no_upload) {
  if (!plan || !x || !w || !ypool || (!idx && !plan->avg_child)) return ROTCONV_ERR_NULL;
  if (plan->pad_child && plan->pad_use[0]) {
    if (no_upload && !tables_on_current_device(plan->pad_child)) return ROTCONV_ERR_UNSUPPORTED;
    PadCtx c;
    int rc = pad_ctx(plan, ws, ws_bytes, stream, &c, own_need ? pool_fwd_need(plan, x, w, ypool, idx, ws) : plan->ws_bytes);
    if (rc) return rc;
    launch_repitch(x, c.in, c.rows_x, c.W, c.Wp, c.es, 0, c.st);
    if ((rc = pool_fwd_impl(c.ch, c.in, w, c.out, reinterpret_cast<uint8_t*>(c.idx), c.cws, c.cws_bytes, stream, own_need,
                            no_upload)))
      return rc;
    launch_repitch(c.out, ypool, c.rows_p, c.Wp, c.W, c.es, 0, c.st);
    launch_repitch(c.idx, idx, c.rows_p, c.Wp, c.W, 1, 0, c.st);
    return finish();
  }
  if (pool_fwd_is_direct(plan, x, ypool, ws)) {     // at most four input channels
    const size_t dneed = own_need ? pool_fwd_need(plan, x, w, ypool, idx, ws) : plan->ws_bytes;
    if (!ws || ws_bytes < dneed) return ROTCONV_ERR_WORKSPACE;
    if (no_upload && !tables_on_current_device(plan)) return ROTCONV_ERR_UNSUPPORTED;
    rotconv_plan* p = const_cast<rotconv_plan*>(plan);
    const int rc = ensure_device_tables(p);
    if (rc) return rc;
    launch_direct_fwd(p, x, w, ypool, idx, static_cast<float*>(ws), static_cast<hipStream_t>(stream));
    return finish();
  }
  if (pool_fwd_is_px16(plan, x, ypool, ws)) {
    const size_t pneed = own_need ? pool_fwd_need(plan, x, w, ypool, idx, ws) : plan->ws_bytes;
    if (!ws || ws_bytes < pneed) return ROTCONV_ERR_WORKSPACE;
    if (no_upload && !tables_on_current_device(plan)) return ROTCONV_ERR_UNSUPPORTED;
    rotconv_plan* p = const_cast<rotconv_plan*>(plan);
    const int rc = ensure_device_tables(p);
    if (rc) return rc;
    launch_px_fwd_bf16(p, h16(x), h16(w), static_cast<uint16_t*>(ypool), idx, static_cast<uint16_t*>(ws),
                       static_cast<hipStream_t>(stream));
    return finish();
  }
  if (!is_bf16(plan)) return f32_rotconv_pool_fwd(plan, x, w, ypool, idx, ws, ws_bytes, stream, own_need, no_upload);
  const size_t need = own_need ? pool_fwd_need(plan, x, w, ypool, idx, ws) : plan->ws_bytes;
  if (!ws || ws_bytes < need) return ROTCONV_ERR_WORKSPACE;
  if (no_upload && !tables_on_current_device(plan)) return ROTCONV_ERR_UNSUPPORTED;
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (bf16_pool_fwd_is_native(plan, x, w, ypool, idx, ws)) {
    // bf16 tensors straight into the bf16 matrix-core kernel; scratch laid out as in the fp32 path
    const int pmode = p4_fwd_pool_mode(plan);
    rotconv_plan* p = const_cast<rotconv_plan*>(plan);
    const int rc = ensure_device_tables(p);
    if (rc) return rc;
    uint16_t* wt = static_cast<uint16_t*>(ws);
    char* extra = static_cast<char*>(ws) + align256(p4_fwd_bf16_pack_bytes(p));
    const size_t hw = (size_t)p->d.H * p->d.W;
    const int nq = pmode == kOutPartial ? p4_fwd_bf16_fold(p) : 1;
    launch_p4_pack_fwd_bf16(p, nq, h16(w), wt, st);
    if (pmode == kOutPooled) {
      launch_p4_fwd_bf16(p, pmode, 1, h16(x), wt, ypool, idx, st);
    } else if (nq > 1) {     // the pool group spans all banks: pooled across them inside the kernel
      launch_p4_fwd_bf16(p, kOutPooled, nq, h16(x), wt, ypool, idx, st);
    } else {
      float* pv = reinterpret_cast<float*>(extra);
      uint8_t* pi = reinterpret_cast<uint8_t*>(extra + align256((size_t)p->host.Q * p->d.N * p->d.Cout * hw * 4));
      launch_p4_fwd_bf16(p, pmode, 1, h16(x), wt, pv, pi, st);
      launch_p4_combine_bf16(p, pv, pi, static_cast<uint16_t*>(ypool), idx, st);
    }
    return finish();
  }
  const Stage s = carve(plan, ws, ws_bytes);
  launch_widen(h16(x), s.x, plan->n_x, st);
  launch_widen(h16(w), s.w, plan->n_w, st);
  const int rc = f32_rotconv_pool_fwd(plan, s.x, s.w, s.y, idx, s.inner, s.inner_bytes, stream, own_need, no_upload);
  if (rc) return rc;
  launch_narrow(s.y, static_cast<uint16_t*>(ypool), plan->n_yp, st);
  return finish();
}

// ---- scratch of the entry point that allocates nothing ------------------------------------------------------
// One array per GPU (each device that loads this code object holds its own copy at its own address, until the
// process ends).  Host code never uses the array's name as an address: static_scratch() resolves the device
// address once per device with hipGetSymbolAddress and hands that pointer to the kernels.
constexpr size_t kStaticScratchBytes = ROTCONV_STATIC_SCRATCH_BYTES;
constexpr int kMaxDevices = 64;

}  // namespace

static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {

static std::atomic<void*> g_scratch_ptr[kMaxDevices];

// Device address of `scratch` on the current device (nullptr on failure).
static void* static_scratch() {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
  void* ptr = g_scratch_ptr[dev].load(std::memory_order_acquire);
  if (ptr) return ptr;
  if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) {
    (void)hipGetLastError();
    return nullptr;
  }
  g_scratch_ptr[dev].store(ptr, std::memory_order_release);     // every thread resolves the same address
  return ptr;
}

}  // namespace

int rotconv_pool_fwd(const rotconv_plan* plan, const void* x, const void* w, void* ypool, uint8_t* idx, void* ws,
                     size_t ws_bytes, void* stream) {
  return pool_fwd_impl(plan, x, w, ypool, idx, ws, ws_bytes, stream, false, false);
}

int rotconv_pool_fwd_static(const rotconv_plan* plan, const void* x, const void* w, void* ypool, uint8_t* idx,
                            void* stream) {
  if (!plan || !x || !w || !ypool || (!idx && !plan->avg_child)) return ROTCONV_ERR_NULL;
  void* ws = static_scratch();
  if (!ws) return ROTCONV_ERR_LAUNCH;
  if (pool_fwd_need(plan, x, w, ypool, idx, ws) > kStaticScratchBytes) return ROTCONV_ERR_WORKSPACE;
  return pool_fwd_impl(plan, x, w, ypool, idx, ws, kStaticScratchBytes, stream, true, true);
}

int rotconv_pool_bwd_data(const rotconv_plan* plan, const void* gpool, const uint8_t* idx, const void* w, void* dx,
                          void* ws, size_t ws_bytes, void* stream) {
  if (!plan || !gpool || (!idx && !plan->avg_child) || !w || !dx) return ROTCONV_ERR_NULL;
  if (plan->pad_child && plan->pad_use[1]) {     // padded columns: zero gradient, idx 255 (matches no orientation)
    PadCtx c;
    int rc = pad_ctx(plan, ws, ws_bytes, stream, &c, plan->ws_bytes);
    if (rc) return rc;
    launch_repitch(gpool, c.out, c.rows_p, c.W, c.Wp, c.es, 0, c.st);
    launch_repitch(idx, c.idx, c.rows_p, c.W, c.Wp, 1, 0xff, c.st);
    if ((rc = rotconv_pool_bwd_data(c.ch, c.out, reinterpret_cast<const uint8_t*>(c.idx), w, c.in, c.cws,
                                    c.ch->ws_bytes, stream)))
      return rc;
    launch_repitch(c.in, dx, c.rows_x, c.Wp, c.W, c.es, 0, c.st);
    return finish();
  }
  if (!is_bf16(plan)) return f32_rotconv_pool_bwd_data(plan, gpool, idx, w, dx, ws, ws_bytes, stream);
  if (!ws || ws_bytes < plan->ws_bytes) return ROTCONV_ERR_WORKSPACE;
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (plan->native16[1] && aligned(gpool, 4) && aligned(idx, 2) && aligned(dx, 16) && aligned(ws, 16)) {
    rotconv_plan* p = const_cast<rotconv_plan*>(plan);
    const int rc = ensure_device_tables(p);
    if (rc) return rc;
    uint16_t* wt = static_cast<uint16_t*>(ws);
    if (p->bwd_lut16[1]) {     // routed-gradient table: one contraction with the base bank
      launch_p4_pack_bwd_bf16_lut(p, h16(w), wt, st);
      float* lpart = reinterpret_cast<float*>(static_cast<char*>(ws) + align256(p4_bwd_data_bf16_lut_pack_bytes(p)));
      launch_p4_bwd_data_bf16_lut(p, h16(gpool), idx, wt, static_cast<uint16_t*>(dx), lpart, st);
      return finish();
    }
    launch_p4_pack_bwd_bf16(p, h16(w), wt, st);
    float* part = reinterpret_cast<float*>(static_cast<char*>(ws) + align256(p4_bwd_data_bf16_pack_bytes(p)));
    launch_p4_bwd_data_bf16(p, h16(gpool), idx, wt, static_cast<uint16_t*>(dx), part, st);
    return finish();
  }
  const Stage s = carve(plan, ws, ws_bytes);
  launch_widen(h16(gpool), s.y, plan->n_yp, st);
  launch_widen(h16(w), s.w, plan->n_w, st);
  const int rc = f32_rotconv_pool_bwd_data(plan, s.y, idx, s.w, s.x, s.inner, s.inner_bytes, stream);
  if (rc) return rc;
  launch_narrow(s.x, static_cast<uint16_t*>(dx), plan->n_x, st);
  return finish();
}

int rotconv_pool_bwd_weight(const rotconv_plan* plan, const void* x, const void* gpool, const uint8_t* idx, float* dw,
                            void* ws, size_t ws_bytes, void* stream) {
  if (!plan || !x || !gpool || (!idx && !plan->avg_child) || !dw) return ROTCONV_ERR_NULL;
  if (plan->pad_child && plan->pad_use[2]) {
    PadCtx c;
    const int rc = pad_ctx(plan, ws, ws_bytes, stream, &c, plan->ws_bytes);
    if (rc) return rc;
    launch_repitch(x, c.in, c.rows_x, c.W, c.Wp, c.es, 0, c.st);
    launch_repitch(gpool, c.out, c.rows_p, c.W, c.Wp, c.es, 0, c.st);
    launch_repitch(idx, c.idx, c.rows_p, c.W, c.Wp, 1, 0xff, c.st);
    return rotconv_pool_bwd_weight(c.ch, c.in, c.out, reinterpret_cast<const uint8_t*>(c.idx), dw, c.cws,
                                   c.ch->ws_bytes, stream);
  }
  if (plan->direct[2] && aligned(x, is_bf16(plan) ? 2 : 4) && aligned(gpool, is_bf16(plan) ? 2 : 4) && aligned(ws, 16)) {
    if (!ws || ws_bytes < plan->ws_bytes) return ROTCONV_ERR_WORKSPACE;
    rotconv_plan* p = const_cast<rotconv_plan*>(plan);
    const int rc = ensure_device_tables(p);
    if (rc) return rc;
    launch_direct_bwd_weight(p, x, gpool, idx, static_cast<float*>(ws), dw, static_cast<hipStream_t>(stream));
    return finish();
  }
  if (!is_bf16(plan)) return f32_rotconv_pool_bwd_weight(plan, x, gpool, idx, dw, ws, ws_bytes, stream);
  if (!ws || ws_bytes < plan->ws_bytes) return ROTCONV_ERR_WORKSPACE;
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (plan->native16[2] && aligned(x, 16) && aligned(gpool, 16) && aligned(idx, 8) && aligned(ws, 16)) {
    rotconv_plan* p = const_cast<rotconv_plan*>(plan);
    const int rc = ensure_device_tables(p);
    if (rc) return rc;
    launch_p4_bwd_weight_bf16(p, h16(x), h16(gpool), idx, static_cast<float*>(ws), dw, st);
    return finish();
  }
  const Stage s = carve(plan, ws, ws_bytes);
  launch_widen(h16(x), s.x, plan->n_x, st);
  launch_widen(h16(gpool), s.y, plan->n_yp, st);
  return f32_rotconv_pool_bwd_weight(plan, s.x, s.y, idx, dw, s.inner, s.inner_bytes, stream);
}

const char* rotconv_status_string(int status) {
  switch (status) {
    case ROTCONV_OK: return "ok";
    case ROTCONV_ERR_NULL: return "null pointer argument";
    case ROTCONV_ERR_SHAPE: return "invalid shape, stride, padding or pool group";
    case ROTCONV_ERR_ANGLES: return "invalid angle set for this mode";
    case ROTCONV_ERR_UNSUPPORTED: return "request not supported by this build";
    case ROTCONV_ERR_WORKSPACE: return "workspace missing or too small";
    case ROTCONV_ERR_LAUNCH: return "HIP runtime error";
    default: return "unknown status";
  }
}

// Does the pass of a plan of the matrix multiply + scatter family run as one contraction?
static bool on_ig(const rotconv_plan* p, int pass) { return pass == 0 ? p->ig[1].mt : pass == 1 ? p->ig_dx.mt : p->ig_dw; }

double rotconv_plan_conv_equivalents(const rotconv_plan* plan, int pass) {
  if (!plan || pass < 0 || pass > 2) return 0.0;
  if (plan->pad_child && plan->pad_use[pass]) return rotconv_plan_conv_equivalents(plan->pad_child, pass);
  const int Q = plan->host.Q, B = plan->B;
  if (plan->avg_child) return (double)plan->ng * rotconv_plan_conv_equivalents(plan->avg_child, pass);
  // the turns are rows of one contraction
  if (plan->direct[pass] && (pass == 0 ? first_fwd_layer(plan) : first_bwd_weight_layer(plan))) return plan->d.R;
  if (plan->direct[pass]) return Q;     // one product set per first-quadrant bank, on the vector ALU
  if (plan->d.dtype == ROTCONV_BF16 && plan->native16[pass]) {
    int present = 0;      // orientations in the set: the bf16 gradient kernels multiply every quarter turn on its own
    for (int i = 0; i < Q * 4; ++i) present += plan->rot_of[i] >= 0 ? 1 : 0;
    if (pass == 0) return Q;
    if (plan->bwd_lut16[pass]) return B;       // routed gradients folded into the base taps
    if (pass == 1) return p4_bwd_data_bf16_sparse(plan) ? 0.5 * present : present;   // 2-of-4 sparse operand: half the instructions
    return present;
  }
  if (plan->fast[pass]) {
    if (pass == 0) return plan->fwd_base ? B : Q;
    return plan->bwd_lut ? B : Q;
  }
  if (plan->gs) return on_ig(plan, pass) ? plan->d.R : Q;
  return plan->d.R;
}

const char* rotconv_plan_kernel_name(const rotconv_plan* plan, int pass) {
  if (!plan || pass < 0 || pass > 4) return "none";
  if (pass >= 3)      // the unfused gradient calls, given rotconv_workspace_bytes_unfused of scratch
    return plan->gs || (plan->d.pool_op != ROTCONV_POOL_AVG && gs_wanted(plan)) ? "mfma_gemm_scatter" : "generic";
  if (plan->pad_child && plan->pad_use[pass]) return rotconv_plan_kernel_name(plan->pad_child, pass);
  if (plan->direct[pass]) return "valu_direct";
  if (pass == 0 && plan->px16) return "mfma_px_bf16";
  if (plan->d.dtype == ROTCONV_BF16 && plan->native16[pass]) return plan->bwd_lut16[pass] ? "mfma_p4_bf16_lut" : "mfma_p4_bf16";
  if (pass == 0 && plan->fast[0] && plan->fwd_base) return "mfma_p4_base";   // the pooled forward; rotconv_fwd: mfma_p4
  return plan->fast[pass] ? "mfma_p4" : plan->gs ? "mfma_gemm_scatter" : "generic";
}

int rotconv_plan_bf16_parts(const rotconv_plan* plan, int pass) {
  if (!plan || pass < 0 || pass > 2) return 0;
  if (plan->avg_child) return rotconv_plan_bf16_parts(plan->avg_child, pass);
  if (plan->pad_child && plan->pad_use[pass]) return rotconv_plan_bf16_parts(plan->pad_child, pass);
  if (plan->direct[pass]) return pass == 0 ? first_fwd_layer(plan) : first_bwd_weight_layer(plan);
  if (!plan->fast[pass] && plan->gs) return on_ig(plan, pass) || gs_on_parts(plan, pass);
  if ((pass == 0 && plan->px16) || !plan->fast[pass]) return 0;
  if (is_bf16(plan) && plan->native16[pass]) return 0;
  if (pass == 0 && plan->fwd_base) return p4_fwd_base_on_parts(plan);
  return pass == 0 ? plan->fwd_s3 : pass == 1 ? s3_bwd_data_supported(plan) : s3_bwd_weight_supported(plan);
}

}  // extern "C"
