// Pooled forward of fp32 layers with at most three input channels and the four quarter turns (a network's first layer) on
// the bf16 matrix cores, operands split into three bf16 parts (rotconv_split3.h).
//
// Nine taps of three channels are 27 of the 32 terms of one matrix instruction, so the whole filter is contracted at once
// and the four turns of a filter are four rows of the weights' tile: row 4 f + s of a tile of four filters holds filter f
// turned s times.  The instruction leaves a lane with the four turns of one filter at one pixel: max, arg-max, ReLU and the
// stores need nothing of another lane.  (The vector-ALU kernel, k_direct_fwd, forms a tap's product once for the four
// turns, but its 36 placement additions per filter and pixel remain; here they are part of the contraction.)
//
// A wave takes 64 pixels, four consecutive ones (W is a multiple of four) per lane column, in four tiles: pixel b of the
// quads is tile b, so that a lane stores four pooled values (16 bytes) and four idx bytes at once.  Its eight terms of the
// 32 are eight 16-byte loads, each at its tap's offset; the weights' parts (three KB per four filters) are split once per
// workgroup into LDS and read once per tile of four filters for all four pixel tiles.
//
// What bounds it: per 64 pixels and 64 filters 384 matrix instructions (3.4 us of a SIMD) beside 900 vector instructions
// that pool and 300 that load and split the pixels; the stores of the 2x3 -> 64, 512x512 layer, 168 MB, take 37 us.
// Measured, the vector-ALU kernel and its pack / this: 2x3 -> 64, 512x512 110 / 68 us; 2x3 -> 64, 128x128 21 / 12; 1x3 -> 8, 64x64
// 10 / 5; 150 layers of 1 to 3 channels, 1 to 128 filters and up to 500 x 512 pixels, as called: 0.73 of the time in the mean,
// 0.62 to 0.89.  Its error against 64 bits is no larger (1.1e-7 both with uniform pixels, 9.8e-8 against 1.0e-7).
//
// Values of 2^60 and more and infinities do not survive the split (or their sums might not): 64 pixels with such a value in
// reach, and all pixels where a weight is one (or NaN), are summed in fp32 on the vector ALU, positions outside the image
// left out.  A NaN pixel makes NaN what it reaches either way.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "rotconv_direct.h"
#include "rotconv_kernels.h"
#include "rotconv_p4_taps.h"
#include "rotconv_split3.h"

namespace rotconv {
namespace {

constexpr int FT = 16;                 // tiles of four filters per workgroup at the most
constexpr float kSplitLimit = 0x1p60f;

struct FirstGeom {
  int H, W, Cout, ft;                  // ft: tiles of four filters per workgroup
  int nquad, qpr, qpi;                 // quads of pixels in all, per row, per image
  uint32_t xbytes, obytes;
};

template <int CIN, bool RELU>
__global__ __launch_bounds__(256, 2) void k_first_fwd(const float* __restrict__ x, const float* __restrict__ w,
                                                      float* __restrict__ ypool, uint8_t* __restrict__ idx, FirstGeom g) {
  extern __shared__ u32x4 Al[];        // [tile][part][lane]
  __shared__ int odd_weight;
  const int tid = threadIdx.x, lane = tid % 64, lg = lane / 16, lc = lane % 16;
  const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
  const int f0 = blockIdx.y * (4 * g.ft), nt = min(g.ft, (g.Cout - f0 + 3) / 4);
  const int HW = g.H * g.W;
  const auto rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(x), 0, (int)g.xbytes, 0x27000);
  const auto ro = __builtin_amdgcn_make_buffer_rsrc(ypool, 0, (int)g.obytes, 0x27000);
  const auto ri = __builtin_amdgcn_make_buffer_rsrc(idx, 0, (int)(g.obytes / 4), 0x27000);

  // ---- the lane's eight terms: k = 8 lg + i is tap k % 9 of channel k / 9
  uint32_t koff[8];                    // from the quad's first pixel, bytes
  uint32_t up = 0, down = 0, left = 0, right = 0, none = 0;      // a bit per term
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int k = 8 * lg + i, ci = k / 9, dy = k % 9 / 3, dx = k % 3;
    koff[i] = (uint32_t)((ci * HW + (dy - 1) * g.W + dx - 1) * 4);
    up |= (uint32_t)(dy == 0) << i;
    down |= (uint32_t)(dy == 2) << i;
    left |= (uint32_t)(dx == 0) << i;
    right |= (uint32_t)(dx == 2) << i;
    none |= (uint32_t)(k >= 9 * CIN) << i;
  }
  struct Quad { int n, y, xq; bool live; };
  auto quad_of = [&](int strip) {
    const int v = strip * 16 + lc;
    const bool live = v < g.nquad;
    const int u = live ? v : 0, n = u / g.qpi, r = u - n * g.qpi, y = r / g.qpr;
    return Quad{n, y, r - y * g.qpr, live};
  };
  s3_f4 raw[8];
  // At a row's ends the load is moved a pixel inwards (no load leaves the tensor) and put right by `shift`.
  auto load = [&](const Quad& p) {
    const uint32_t bad = none | (p.y == 0 ? up : 0u) | (p.y == g.H - 1 ? down : 0u) | (p.live ? 0u : 255u);
    const uint32_t l = p.xq == 0 ? left : 0u, r = p.xq == g.qpr - 1 ? right : 0u;
    const uint32_t at = (uint32_t)(p.n * CIN * HW + p.y * g.W + 4 * p.xq) * 4u;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const uint32_t o = at + koff[i] + (l >> i & 1u) * 4u - (r >> i & 1u) * 4u;
      raw[i] = __builtin_bit_cast(s3_f4, __builtin_amdgcn_raw_buffer_load_b128(rx, bad >> i & 1u ? kOutside : o, 0, 0));
    }
  };
  auto shift = [&](const Quad& p) {
    if (!__any(p.xq == 0 || p.xq == g.qpr - 1)) return;
    const uint32_t l = p.xq == 0 ? left : 0u, r = p.xq == g.qpr - 1 ? right : 0u;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const bool tl = l >> i & 1u, tr = r >> i & 1u;
      const float a = raw[i][0], b = raw[i][1], c = raw[i][2], d = raw[i][3];
      raw[i][0] = tl ? 0.f : tr ? b : a;
      raw[i][1] = tl ? a : tr ? c : b;
      raw[i][2] = tl ? b : tr ? d : c;
      raw[i][3] = tl ? c : tr ? 0.f : d;
    }
  };

  const int nstrip = (g.nquad + 15) / 16, step = gridDim.x * 4;
  int strip = blockIdx.x * 4 + wave;
  Quad q = quad_of(strip);
  load(q);

  // ---- the weights' parts
  if (tid == 0) odd_weight = 0;
  __syncthreads();
  for (int i = tid; i < nt * 256; i += 256) {
    const int j = i % 4, l = i / 4 % 64, t = i / 256, f = f0 + 4 * t + l % 16 / 4, s = l % 4, k = 8 * (l / 16) + 2 * j;
    uint16_t p[2][3];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int pos = (k + e) % 9, back = (4 - s) % 4;             // the tap that s turns bring to this position
      const bool in = k + e < 9 * CIN && f < g.Cout;
      const float v = in ? w[((size_t)f * CIN + (k + e) / 9) * 9 + tap_i(back, pos) * 3 + tap_j(back, pos)] : 0.f;
      if (!(__builtin_fabsf(v) < kSplitLimit)) odd_weight = 1;
      s3_split_weight(v, p[e][0], p[e][1], p[e][2]);
    }
    uint32_t* dst = reinterpret_cast<uint32_t*>(Al) + (t * 3 * 64 + l) * 4 + j;
#pragma unroll
    for (int e = 0; e < 3; ++e) dst[e * 256] = (uint32_t)p[0][e] | (uint32_t)p[1][e] << 16;
  }
  __syncthreads();
  const bool odd_w = odd_weight != 0;

  for (; strip < nstrip; strip += step) {
    shift(q);
    float m = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const float v = raw[i][b];
        m = __builtin_fmaxf(m, __builtin_fabsf(v));                // (a NaN may pass: it makes NaN what it reaches either way)
      }
    const bool odd = odd_w || __any(!(m < kSplitLimit));
    u32x4 ap[4][3];                                                // [pixel of the quad][part]
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const S3Pair s = s3_split2(raw[2 * j][b], raw[2 * j + 1][b]);
#pragma unroll
        for (int e = 0; e < 3; ++e) ap[b][e][j] = s.p[e];
      }
    const Quad here = q;
    q = quad_of(strip + step);
    load(q);
    const uint32_t at = ((uint32_t)(here.n * g.Cout + f0 + lg) * (uint32_t)HW + (uint32_t)(here.y * g.W + 4 * here.xq)) * 4u;

    // y: the filter's four turns at the quad's pixels
    auto pool = [&](int t, const s3_f4 (&y)[4]) {
      s3_f4 out;
      uint32_t bytes = 0;
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        float v = y[b][0];
        uint32_t at_turn = 0;
#pragma unroll
        for (int s = 1; s < 4; ++s) {
          const float c = y[b][s];
          const bool gt = c > v;
          v = gt ? c : v;
          at_turn = gt ? (uint32_t)s << (8 * b) : at_turn;
        }
        if (RELU) {
          const bool dead = v <= 0.f;
          v = dead ? 0.f : v;
          at_turn = dead ? 255u << (8 * b) : at_turn;
        }
        out[b] = v;
        bytes |= at_turn;
      }
      const bool ok = here.live && f0 + 4 * t + lg < g.Cout;
      // The tile's offset is added to the lane's and not left to the instruction's scalar offset: with one, nothing keeps the
      // next vector instruction from overwriting the third register of a 16-byte store before it is read (the compiler
      // waits only where there is none; a few pixels in a thousand held idx bytes so).
      const uint32_t o = at + (uint32_t)(4 * t) * (uint32_t)HW * 4u;
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, out), ro, ok ? o : kOutside, 0, 0);
      __builtin_amdgcn_raw_buffer_store_b32(bytes, ri, ok ? o >> 2 : kOutside, 0, 0);
    };

    if (!odd) {
      const u32x4* al = Al + lane;
      u32x4 a[3] = {al[0], al[64], al[128]};
#pragma unroll 1
      for (int t = 0; t < nt; ++t) {
        const u32x4* an = al + min(t + 1, nt - 1) * 192;           // read a tile ahead
        const u32x4 next[3] = {an[0], an[64], an[128]};
        s3_f4 s[4];
        auto product = [&](int we, int ae) {
#pragma unroll
          for (int b = 0; b < 4; ++b) s[b] = s3_mfma(a[we], ap[b][ae], s[b]);
        };
        // the smallest products first
        s[0] = s[1] = s[2] = s[3] = s3_f4{0.f, 0.f, 0.f, 0.f};
        product(2, 0);
        product(0, 2);
        product(1, 1);
        product(1, 0);
        product(0, 1);
        product(0, 0);
        pool(t, s);
#pragma unroll
        for (int e = 0; e < 3; ++e) a[e] = next[e];
      }
    } else {
#pragma unroll 1
      for (int t = 0; t < nt; ++t) {
        const int f = f0 + 4 * t + lg;
        s3_f4 y[4];
        y[0] = y[1] = y[2] = y[3] = s3_f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
        for (int k = 0; k < 9 * CIN && f < g.Cout; ++k) {
          const int ci = k / 9, pos = k % 9, row = here.y + pos / 3 - 1;
          if (row < 0 || row >= g.H) continue;
#pragma unroll
          for (int s = 0; s < 4; ++s) {
            const int back = (4 - s) % 4;
            const float wv = w[((size_t)f * CIN + ci) * 9 + tap_i(back, pos) * 3 + tap_j(back, pos)];
#pragma unroll
            for (int b = 0; b < 4; ++b) {
              const int col = 4 * here.xq + b + pos % 3 - 1;
              if (col >= 0 && col < g.W) y[b][s] += wv * x[((size_t)here.n * CIN + ci) * HW + (size_t)row * g.W + col];
            }
          }
        }
        pool(t, y);
      }
    }
  }
}

}  // namespace

// The four quarter turns of unchanged filters in their order, rows of whole quads, tensors within a 32-bit offset, aligned
// outputs; four channels are 36 terms, more than an instruction has.
bool first_fwd_layer(const rotconv_plan* p) {
  const rotconv_desc& d = p->d;
  if (d.dtype != ROTCONV_F32 || d.Cin > 3 || d.W % 4 || p->ng != 1 || d.R != 4 || p->host.Q != 1 || !p->base_bank) return false;
  if (p->opt.bf16_parts < 0 || p->opt.direct_ty > 0) return false;          // the vector-ALU kernel asked for
  for (int s = 0; s < 4; ++s)
    if (p->rot_of[s] != s) return false;
  const double hw4 = 4.0 * d.N * d.H * d.W;
  return hw4 * d.Cin < 4e9 && hw4 * d.Cout < 4e9;
}
bool first_fwd_supported(const rotconv_plan* p, const void* x, const void* ypool, const void* idx) {
  return first_fwd_layer(p) && reinterpret_cast<uintptr_t>(x) % 4 == 0 && reinterpret_cast<uintptr_t>(ypool) % 16 == 0 &&
         reinterpret_cast<uintptr_t>(idx) % 4 == 0;
}

void launch_first_fwd(const rotconv_plan* p, const float* x, const float* w, float* ypool, uint8_t* idx, hipStream_t st) {
  const rotconv_desc& d = p->d;
  FirstGeom g{};
  g.H = d.H; g.W = d.W; g.Cout = d.Cout;
  g.qpr = d.W / 4; g.qpi = g.qpr * d.H; g.nquad = g.qpi * d.N;
  g.xbytes = (uint32_t)(4.0 * d.N * d.Cin * d.H * d.W);
  g.obytes = (uint32_t)(4.0 * d.N * d.Cout * d.H * d.W);
  // Two workgroups (of 48 KB at the most) per CU, each keeping its weights for as many strips of 64 pixels as it gets; where
  // there are fewer strips, workgroups of fewer filters, which also have fewer weights to split (2x3 -> 64, 128x128:
  // 12 us, with all 64 filters in a workgroup about 36).
  const int tiles = (d.Cout + 3) / 4, strips = (g.nquad + 15) / 16, groups = (strips + 3) / 4;
  g.ft = std::min(FT, tiles);
  while (g.ft > 1 && (long)groups * ((tiles + g.ft - 1) / g.ft) < 512) g.ft = (g.ft + 1) / 2;
  const int nfb = (tiles + g.ft - 1) / g.ft, wg = std::min(groups, std::max(1, 512 / nfb));
  const size_t lds = (size_t)g.ft * 3 * 64 * 16;
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3(wg, nfb), dim3(256), lds, st, x, w, ypool, idx, g);
  };
  const bool relu = d.activation == ROTCONV_ACT_RELU;
  if (d.Cin == 1) { if (relu) go(k_first_fwd<1, true>); else go(k_first_fwd<1, false>); }
  else if (d.Cin == 2) { if (relu) go(k_first_fwd<2, true>); else go(k_first_fwd<2, false>); }
  else { if (relu) go(k_first_fwd<3, true>); else go(k_first_fwd<3, false>); }
}

}  // namespace rotconv
