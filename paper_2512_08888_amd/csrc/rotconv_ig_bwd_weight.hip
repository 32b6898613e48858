// Weight gradient of fp32 layers with filters of other sizes and strides, pooled over the four quarter turns, as one contraction over
// the output pixels on the bf16 matrix cores, operands split into three bf16 parts (rotconv_split3.h): nothing is routed through
// memory.
//
//   E[co, s][ci, T] = sum_o (G * 1[idx == s])[co, o] X[ci, o stride + T - pad],     dW[co, ci, u] = sum_s E[co, s][ci, rot^s u]
//
// As in the first layers' kernel (rotconv_first_bwd_weight.hip) the result is turned and not the gradients: G is split once and its
// parts are masked for the four turns; the products are formed four times as often as where the turns' gradients are added up
// first (rotconv_gs.hip), but neither these (k^2 values per output) nor their sums leave the registers.
//
// A wave owns 16 filters, 16 channels and a row of the k taps (up to five at a time), and contracts 32 outputs a step: a lane eight consecutive ones of a
// filter, and the pixels that a row of taps meets there, of a channel.  These are split once, in pairs, and a tap's operand is the
// pairs from its own offset on, an odd one joined out of two words; with stride 2 the even and the odd columns are lists of their
// own.  The last eight outputs of a row start at Wo - 8, and those that they repeat are masked.  The eight waves of a workgroup
// take shares of the outputs (every other one contracts -X, as the instruction cuts towards minus infinity) and meet in LDS.
//
// A workgroup's sums that are not finite, or below 2^-100 and not zero, are formed again in fp32 on the vector ALU.
//
// What bounds it: matrix instructions (24 a tap and step) and, beside them, about 330 vector instructions a step of five taps
// (masks and splits, the same for every tap); small maps the start of a wave, which has a step or two.  2x32 -> 32, 96x96, 5 x 5: 54 us
// with routed gradients through memory, 36 so (30 the kernel); stride 2, 2x54 -> 64, 60x90 106 / 26.  The pixels as one load per
// four columns (36 us) and not one each (44): then the address units were as busy as the matrix cores.  Error against 64 bits 0.6
// of the other form's.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "rotconv_ig.h"
#include "rotconv_ig_orbits.h"
#include "rotconv_split3.h"

namespace rotconv {
namespace {

constexpr int kWaves = 8;

struct IgDwGeom {
  int N, Cin, H, W, Cout, k, pad, Ho, Wo;
  int nco, nci, ngrp;                  // blocks of 16 filters, of 16 channels; groups of taps of a row
  int opr, nq, steps, per;             // eights of outputs per row, in all; steps of four, steps per wave
  int dn, dy, dx;                      // four eights on: images, rows, eights
  uint32_t xbytes, gbytes;
};

// TJ: taps of a row per wave (k in groups of TJ)
template <int TJ, int ST>
__global__ __launch_bounds__(64 * kWaves, 2) void k_ig_bwd_weight(const float* __restrict__ x, const float* __restrict__ gpool,
                                                                  const uint8_t* __restrict__ idx, float* __restrict__ part,
                                                                  IgDwGeom g) {
  constexpr int LEN = 7 * ST + TJ;                                 // columns that the taps meet
  constexpr int NX = (LEN + 3) / 4;
  constexpr int NW = (8 + (TJ - 1) / ST + 1) / 2;                  // pairs of a list
  extern __shared__ float red[];       // [wave][tap][filter][17]
  const int tid = threadIdx.x, lane = tid % 64, lg = lane / 16, lc = lane % 16;
  const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
  const int per_xcd = gridDim.x / 8;   // blocks of the same outputs behind each other on one XCD
  const int v0 = gridDim.x % 8 == 0 ? (blockIdx.x % 8) * per_xcd + blockIdx.x / 8 : blockIdx.x;
  const int per_pair = g.k * g.ngrp, nblk = g.nco * g.nci * per_pair, blk = v0 % nblk, split = v0 / nblk;
  const int row = blk % per_pair / g.ngrp, j0 = blk % g.ngrp * TJ;
  const int c0 = blk / per_pair % g.nci * 16, f0 = blk / per_pair / g.nci * 16;
  const int HW = g.H * g.W, HWo = g.Ho * g.Wo;
  const uint32_t turned = wave & 1 ? 0x80000000u : 0u;
  const auto rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(x), 0, (int)g.xbytes, 0x27000);
  const auto rg = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(gpool), 0, (int)g.gbytes, 0x27000);
  const int co = min(f0 + lc, g.Cout - 1);                         // (rows and columns beyond the last are read by nobody)
  const int ci = min(c0 + lc, g.Cin - 1);

  const int first = (split * kWaves + wave) * g.per, stop = min(first + g.per, g.steps);
  int step = first;
  int v = step * 4 + lg, n, y, q;
  n = v / (g.Ho * g.opr);
  y = v / g.opr - n * g.Ho;
  q = v % g.opr;
  auto advance = [&]() {
    v += 4;
    q += g.dx;
    const bool cq = q >= g.opr;
    q -= cq ? g.opr : 0;
    y += g.dy + (cq ? 1 : 0);
    const bool cy = y >= g.Ho;
    y -= cy ? g.Ho : 0;
    n += g.dn + (cy ? 1 : 0);
  };

  s3_f4 xr[NX], gr[2];
  uint32_t ir[2], again[2];
  int ix = 0;                          // the first of the loaded columns
  const int total = g.N * g.Cin * HW;
  auto load = [&]() {
    const bool live = v < g.nq;
    const int ox = min(8 * q, g.Wo - 8), rep = 8 * q - ox;
    const uint32_t o = (uint32_t)(n * g.Cout + co) * (uint32_t)HWo + (uint32_t)(y * g.Wo + ox);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      gr[h] = __builtin_bit_cast(s3_f4, __builtin_amdgcn_raw_buffer_load_b128(rg, live ? (o + 4 * h) * 4u : kOutside, 0, 0));
      ir[h] = load4(idx + (live ? o + 4 * h : 0u));
      const int r = min(max(rep - 4 * h, 0), 4);                   // outputs that the eight before has: a byte each
      again[h] = r == 4 ? 0xffffffffu : (1u << 8 * r) - 1u;
    }
    const int iy = y * ST + row - g.pad;
    ix = ox * ST - g.pad + j0;
    const bool in = live && (unsigned)iy < (unsigned)g.H;
    const int at = (n * g.Cin + ci) * HW + iy * g.W + ix;
    // columns outside the row are another row's, zeroed by `edges`; near the tensor's ends they are loaded one by one
    if (__all(!in || (at >= 0 && at + 4 * NX <= total))) {
#pragma unroll
      for (int e = 0; e < NX; ++e)
        xr[e] = __builtin_bit_cast(s3_f4, __builtin_amdgcn_raw_buffer_load_b128(rx, in ? (uint32_t)(at + 4 * e) * 4u : kOutside, 0, 0));
    } else {
#pragma unroll
      for (int e = 0; e < 4 * NX; ++e)
        xr[e / 4][e % 4] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rx, in && (unsigned)(ix + e) < (unsigned)g.W ? (uint32_t)(at + e) * 4u : kOutside, 0, 0));
    }
  };
  auto edges = [&]() {
    if (__all(ix >= 0 && ix + LEN <= g.W)) return;
#pragma unroll
    for (int e = 0; e < LEN; ++e) xr[e / 4][e % 4] = (unsigned)(ix + e) < (unsigned)g.W ? xr[e / 4][e % 4] : 0.f;
  };

  s3_f4 acc[4][TJ];
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int j = 0; j < TJ; ++j) acc[s][j] = s3_f4{0.f, 0.f, 0.f, 0.f};
  if (step < stop) load();
#pragma unroll 1
  for (; step < stop; ++step) {
    edges();
    u32x4 gp[3];
    uint32_t sel[4];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const float lo = gr[h][2 * e], hi = gr[h][2 * e + 1];
        const S3Pair s = s3_split2(lo, hi);
#pragma unroll
        for (int i = 0; i < 3; ++i) gp[i][2 * h + e] = s.p[i];
      }
      const uint32_t u = ir[h] | again[h];
      const uint32_t no = ((((u & 0x7c7c7c7cu) + 0x7c7c7c7cu) | u) & 0x80808080u) >> 5;      // any idx beyond 3
      const uint32_t at = (u & 0x03030303u) | no;
      sel[2 * h] = __builtin_amdgcn_perm(0u, at, 0x01010000u);
      sel[2 * h + 1] = __builtin_amdgcn_perm(0u, at, 0x03030202u);
    }
    uint32_t w[ST][NW][3];             // [list][pair][part]
#pragma unroll
    for (int l = 0; l < ST; ++l)
#pragma unroll
      for (int t = 0; t < NW; ++t) {
        auto value = [&](int m) {
          const int e = l + ST * m;
          const float f = xr[e < LEN ? e / 4 : 0][e % 4];
          return e < LEN ? __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, f) ^ turned) : 0.f;
        };
        const S3Pair s = s3_split2(value(2 * t), value(2 * t + 1));
#pragma unroll
        for (int e = 0; e < 3; ++e) w[l][t][e] = s.p[e];
      }
    advance();
    load();
    u32x4 a[4][3];
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const uint32_t m = __builtin_amdgcn_perm(0u, 0xffu << 8 * s, sel[i]);
#pragma unroll
        for (int e = 0; e < 3; ++e) a[s][e][i] = gp[e][i] & m;
      }
#pragma unroll
    for (int j = 0; j < TJ; ++j) {
      const int l = j % ST, sh = j / ST;
      u32x4 b[3];
#pragma unroll
      for (int e = 0; e < 3; ++e)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          b[e][i] = sh & 1 ? __builtin_amdgcn_alignbyte(w[l][(sh + 1) / 2 + i < NW ? (sh + 1) / 2 + i : NW - 1][e], w[l][sh / 2 + i][e], 2) : w[l][sh / 2 + i][e];
      s3_f4 c[4];
#pragma unroll
      for (int s = 0; s < 4; ++s) c[s] = s3_f4{0.f, 0.f, 0.f, 0.f};
      auto product = [&](int ge, int xe) {
#pragma unroll
        for (int s = 0; s < 4; ++s) c[s] = s3_mfma(a[s][ge], b[xe], c[s]);
      };
      // the smallest products first
      product(2, 0);
      product(0, 2);
      product(1, 1);
      product(1, 0);
      product(0, 1);
      product(0, 0);
#pragma unroll
      for (int s = 0; s < 4; ++s) acc[s][j] += c[s];
    }
  }

  // the waves' sums, ascending
  __shared__ int beyond;               // is one that the parts do not hold among them?
  if (tid == 0) beyond = 0;
  float* out = part + ((size_t)split * nblk + blk) * 4 * TJ * 256;
  // twice a magnitude as an integer: the largest, and the smallest but for zero (with masks of comparisons the kernel takes 28.4
  // instead of 27.4 us)
  uint32_t most = 0u, least = 0xffffffffu;
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    if (s) __syncthreads();
#pragma unroll
    for (int j = 0; j < TJ; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float sum = acc[s][j][r];
        red[((wave * TJ + j) * 16 + 4 * lg + r) * 17 + lc] = __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, sum) ^ turned);
      }
    __syncthreads();
    for (int o = tid; o < TJ * 256; o += 64 * kWaves) {
      double sum = 0.;
#pragma unroll
      for (int t = 0; t < kWaves; ++t) sum += red[((t * TJ + o / 256) * 16 + o / 16 % 16) * 17 + o % 16];
      out[s * TJ * 256 + o] = (float)sum;
      const uint32_t twice = __builtin_bit_cast(uint32_t, (float)sum) << 1;
      most = max(most, twice);
      least = min(least, twice - 1u);
    }
  }
  if (most >= 0x7f800000u << 1 || least < (0x0d800000u << 1) - 1u) beyond = 1;      // not finite, or below 2^-100
  __syncthreads();
  if (__builtin_expect(__builtin_amdgcn_readfirstlane(beyond) == 0, 1)) return;

  // Such sums in fp32 on the vector ALU, a turn at a time.  A wave takes its share of the outputs, four at a time; a lane's filters are
  // 4 lg + r, its channel c0 + lc.  Gradients of NaN throughout: 0.5 ms instead of 44 us (an element at a time, a wave each: 11.7).
  // (Before the sums meet in LDS the contraction would keep registers for this: the kernel 29.5 -> 31.2 us.)
#pragma unroll 1
  for (int s = 0; s < 4; ++s) {
    s3_f4 fresh[TJ];
#pragma unroll
    for (int j = 0; j < TJ; ++j) fresh[j] = s3_f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int w = first * 4; w < min(stop * 4, g.nq); ++w) {        // eights of outputs
      const int wn = w / (g.Ho * g.opr), wy = w / g.opr - wn * g.Ho, wq = w % g.opr;
      const int ox = min(8 * wq, g.Wo - 8), rep = 8 * wq - ox, iy = wy * ST + row - g.pad;
      if ((unsigned)iy >= (unsigned)g.H) continue;
      const float* xr1 = x + ((size_t)wn * g.Cin + ci) * HW + (size_t)iy * g.W;
      s3_f4 part8[TJ];
#pragma unroll
      for (int j = 0; j < TJ; ++j) part8[j] = s3_f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
      for (int h = rep / 4; h < 2; ++h) {
        constexpr int NCOL = 3 * ST + TJ;
        const int left = (ox + 4 * h) * ST - g.pad + j0;
        float xv[NCOL], gv[4][4];
        uint32_t iv[4];
#pragma unroll
        for (int e = 0; e < NCOL; ++e) xv[e] = xr1[min(max(left + e, 0), g.W - 1)];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const size_t o = ((size_t)wn * g.Cout + min(f0 + 4 * lg + r, g.Cout - 1)) * HWo + (size_t)wy * g.Wo + ox + 4 * h;
          __builtin_memcpy(gv[r], gpool + o, 16);
          iv[r] = load4(idx + o);
        }
#pragma unroll
        for (int b = 0; b < 4; ++b) {
          if (4 * h + b < rep) continue;                           // the eight before has it
          uint32_t mask[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) mask[r] = (iv[r] >> 8 * b & 0xffu) == (uint32_t)s ? 0xffffffffu : 0u;
#pragma unroll
          for (int j = 0; j < TJ; ++j) {
            if ((unsigned)(left + b * ST + j) >= (unsigned)g.W) continue;
#pragma unroll
            for (int r = 0; r < 4; ++r) {                          // (masked products, so that 0 times infinity adds nothing)
              const float p = gv[r][b] * xv[b * ST + j];
              part8[j][r] += __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, p) & mask[r]);
            }
          }
        }
      }
#pragma unroll
      for (int j = 0; j < TJ; ++j) fresh[j] += part8[j];
    }
    if (s) __syncthreads();
#pragma unroll
    for (int j = 0; j < TJ; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) red[((wave * TJ + j) * 16 + 4 * lg + r) * 17 + lc] = fresh[j][r];
    __syncthreads();
    for (int o = tid; o < TJ * 256; o += 64 * kWaves) {
      double sum = 0.;
#pragma unroll
      for (int t = 0; t < kWaves; ++t) sum += red[((t * TJ + o / 256) * 16 + o / 16 % 16) * 17 + o % 16];
      float& old = out[s * TJ * 256 + o];
      if (beyond_parts(old)) old = (float)sum;
    }
  }
}

// dW of a tap, four filters and 16 channels: a wave per turn adds up the shares, ascending, then the turns.
__global__ __launch_bounds__(256) void k_ig_dw_finish(const float* __restrict__ part, float* __restrict__ dw, IgDwGeom g, int tj,
                                                      int nsplit) {
  __shared__ double tot[4][64];
  const int k = g.k, lane = threadIdx.x % 64, s0 = threadIdx.x / 64;
  int v = blockIdx.x;
  const int quarter = v % 4; v /= 4;
  const int u = v % (k * k), blk = v / (k * k), ci = blk % g.nci * 16 + lane % 16;
  const int co = blk / g.nci * 16 + quarter * 4 + lane / 16;
  const size_t share = (size_t)g.nco * g.nci * k * g.ngrp * 4 * tj * 256;
  Orbit at{u / k, u % k};
  for (int s = 0; s < s0; ++s) at = turn(at, k);
  const float* src = part + (((((size_t)blk * k + at.i) * g.ngrp + at.j / tj) * 4 + s0) * tj + at.j % tj) * 256 + quarter * 64 + lane;
  double sum = 0.;
  for (int z = 0; z < nsplit; z += 8) {                            // eight loads on their way
    float v8[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) v8[i] = z + i < nsplit ? src[(z + i) * share] : 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) sum += v8[i];
  }
  tot[s0][lane] = sum;
  __syncthreads();
  if (s0) return;
  sum = (tot[0][lane] + tot[1][lane]) + (tot[2][lane] + tot[3][lane]);
  if (co < g.Cout && ci < g.Cin) dw[((size_t)co * g.Cin + ci) * (k * k) + u] = (float)sum;
}

struct Launch { IgDwGeom g; int tj, splits; };
Launch dw_launch(const rotconv_plan* p) {
  const rotconv_desc& d = p->d;
  Launch l{};
  IgDwGeom& g = l.g;
  g.N = d.N; g.Cin = d.Cin; g.H = d.H; g.W = d.W; g.Cout = d.Cout; g.k = d.k; g.pad = d.pad; g.Ho = p->Ho; g.Wo = p->Wo;
  g.nco = (d.Cout + 15) / 16; g.nci = (d.Cin + 15) / 16;
  g.opr = (p->Wo + 7) / 8; g.nq = g.opr * p->Ho * d.N; g.steps = (g.nq + 3) / 4;
  const int qpi = g.opr * p->Ho;
  g.dn = 4 / qpi; g.dy = 4 % qpi / g.opr; g.dx = 4 % qpi % g.opr;
  g.xbytes = (uint32_t)(4.0 * d.N * d.Cin * d.H * d.W);
  g.gbytes = (uint32_t)(4.0 * d.N * d.Cout * p->Ho * p->Wo);
  // rows of up to five taps at once, longer ones in groups of the size that wastes the least
  l.tj = d.k;
  if (d.k > 5) {
    l.tj = 5;
    for (int t = 4; t >= 3; --t)
      if ((d.k + t - 1) / t * t < (d.k + l.tj - 1) / l.tj * l.tj) l.tj = t;
  }
  g.ngrp = (d.k + l.tj - 1) / l.tj;
  const int blocks = g.nco * g.nci * d.k * g.ngrp;
  // a workgroup per CU; none more, which would be a second round (6x22 -> 2, 211x237, 5 x 5, 260 workgroups: 288 us, 250: 166)
  const int want = std::max(1, 256 / blocks);
  g.per = std::max(1, (g.steps + want * kWaves - 1) / (want * kWaves));
  l.splits = (g.steps + g.per * kWaves - 1) / (g.per * kWaves);
  return l;
}

}  // namespace

bool ig_bwd_weight_supported(const rotconv_plan* p) {
  const rotconv_desc& d = p->d;
  if (!ig_fwd_supported(p) || d.R != 4 || p->Wo < 8) return false;
  if (d.k < 2 || d.stride > 2) return false;
  return 1.0 * d.N * d.Cin * d.H * d.W < 1e9 && 4.0 * d.N * d.Cout * p->Ho * p->Wo < 4.2e9;
}

size_t ig_bwd_weight_ws_bytes(const rotconv_plan* p) {
  const Launch l = dw_launch(p);
  return (size_t)l.splits * l.g.nco * l.g.nci * p->d.k * l.g.ngrp * l.tj * 4 * 256 * sizeof(float);
}

void launch_ig_bwd_weight(const rotconv_plan* p, const float* x, const float* gpool, const uint8_t* idx, float* dw, void* ws,
                          hipStream_t st) {
  const rotconv_desc& d = p->d;
  const Launch l = dw_launch(p);
  float* part = static_cast<float*>(ws);
  const size_t lds = (size_t)kWaves * l.tj * 16 * 17 * sizeof(float);
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3((unsigned)(l.splits * l.g.nco * l.g.nci * d.k * l.g.ngrp)), dim3(64 * kWaves), lds, st, x, gpool, idx, part, l.g);
  };
  const bool two = d.stride == 2;
  switch (l.tj) {
    case 2: if (two) go(k_ig_bwd_weight<2, 2>); else go(k_ig_bwd_weight<2, 1>); break;
    case 3: if (two) go(k_ig_bwd_weight<3, 2>); else go(k_ig_bwd_weight<3, 1>); break;
    case 4: if (two) go(k_ig_bwd_weight<4, 2>); else go(k_ig_bwd_weight<4, 1>); break;
    default: if (two) go(k_ig_bwd_weight<5, 2>); else go(k_ig_bwd_weight<5, 1>); break;
  }
  hipLaunchKernelGGL(k_ig_dw_finish, dim3((unsigned)(l.g.nco * l.g.nci * p->kk * 4)), dim3(256), 0, st, part, dw, l.g, l.tj, l.splits);
}

}  // namespace rotconv
