// Weight gradient of fp32 layers with at most four input channels and the four quarter turns (a network's first layer) on the
// bf16 matrix cores, operands split into three bf16 parts (rotconv_split3.h).
//
// With few channels it is cheaper to turn the result than the routed gradients: instead of D_u (four masked terms per tap),
//   E[co, s][ci, t] = sum_p (G * 1[idx == s])[co, p] * X[ci, p + off(t)],     dF[co, ci, u] = sum_s E[co, s][ci, tap(s, u)]
// is one contraction over the pixels with the four turns of a filter as four rows and the 9 Cin shifted images as columns.
// G is split once and the parts are masked four times (two instructions per pair of pixels, part and turn), nothing is
// added before the products.  k_direct_bwd_weight, which builds D on the vector ALU, spends 36 additions and 27 multiply-adds
// per filter and pixel instead.
//
// A wave contracts 16 FB filters over its share of the pixels, 32 (eight quads of four consecutive ones) a step: rows are 16
// filters of one turn, columns 16 of the 9 Cin images.  A lane's eight pixels are two quads; the last quad of a row that is
// not a whole number of them starts at W - 4, and the pixels it repeats are masked.  The products of a step start from zero,
// smallest first, and their total meets the running sum; the matrix instruction cuts towards minus infinity, so every other
// wave contracts -X.  The eight waves of a workgroup meet in LDS, where the turns are added too, in a fixed order.
//
// What bounds it: 96 matrix instructions a step of 32 filters beside about 480 vector instructions (split 130, masks 130, sums
// 64, loads and their addresses), which the two waves of a SIMD hardly overlap: 2x3 -> 64, 512x512 59 us (floor: 37 us for its
// 174 MB), as called 68 us against 112 on the vector ALU; 1x1 -> 97, 206x112 12.6 / 23.1, 6x1 -> 49, 453x41 18.9 / 34.3; 150 layers of 1 to 4
// channels, 1 to 130 filters and up to 520 x 520 pixels 0.93 in the mean (most are two launches of 5 us whichever the
// kernel).  Its error against 64 bits is smaller (first layer and its forward 9.4e-8 / 1.4e-7) since partial sums are added in
// 64 bits.
//
// A sum that is not finite, or below 2^-100 and not zero, is formed again in fp32 on the vector ALU, as the parts do not hold
// infinities and the smallest values.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>

#include "rotconv_direct.h"
#include "rotconv_kernels.h"
#include "rotconv_p4_taps.h"
#include "rotconv_split3.h"

namespace rotconv {
namespace {

constexpr int kWaves = 8;

struct FirstWGeom {
  int H, W, Cout, CoutPad;
  int qpr, qpi;                        // quads of pixels per row (the last may be partial), per image
  int nquad, steps, per;               // quads in all, steps of eight, steps per wave
  int dn, dy, dx;                      // eight quads on: images, rows, quads
  uint32_t xbytes, gbytes;
};

template <int CIN, int FB>
__global__ __launch_bounds__(64 * kWaves, 2) void k_first_bwd_weight(const float* __restrict__ x, const float* __restrict__ gpool,
                                                                     const uint8_t* __restrict__ idx, float* __restrict__ part,
                                                                     FirstWGeom g) {
  constexpr int NC = 9 * CIN, NT = (NC + 15) / 16, NP = 16 * NT + 1;
  extern __shared__ float red[];       // [wave][turn][filter][NP]
  const int tid = threadIdx.x, lane = tid % 64, lg = lane / 16, lc = lane % 16;
  const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
  const int f0 = blockIdx.y * (16 * FB);
  const int HW = g.H * g.W;
  const uint32_t turned = wave & 1 ? 0x80000000u : 0u;             // every other wave contracts -X
  const auto rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(x), 0, (int)g.xbytes, 0x27000);
  const auto rg = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(gpool), 0, (int)g.gbytes, 0x27000);

  // ---- the lane's columns: image k % 9 of channel k / 9
  uint32_t koff[NT];
  bool up[NT], down[NT], left[NT], right[NT], none[NT];
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    const int k = 16 * j + lc, ci = k / 9, dy = k % 9 / 3, dx = k % 3;
    koff[j] = (uint32_t)((ci * HW + (dy - 1) * g.W + dx - 1) * 4);
    up[j] = dy == 0; down[j] = dy == 2; left[j] = dx == 0; right[j] = dx == 2;
    none[j] = k >= NC;
  }
  uint32_t foff[FB];                   // the lane's filters (those beyond the last repeat it: rows nobody reads)
#pragma unroll
  for (int b = 0; b < FB; ++b) foff[b] = (uint32_t)min(f0 + 16 * b + lc, g.Cout - 1) * (uint32_t)HW;

  struct Quad { int v, n, y, q; };
  Quad qd[2];
  int step = (int)(blockIdx.x * kWaves + wave) * g.per;
  const int stop = min(step + g.per, g.steps);
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int v = step * 8 + 2 * lg + h, n = v / g.qpi, r = v - n * g.qpi, y = r / g.qpr;
    qd[h] = Quad{v, n, y, r - y * g.qpr};
  }
  auto advance = [&]() {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      Quad& p = qd[h];
      p.v += 8;
      p.q += g.dx;
      const bool cq = p.q >= g.qpr;
      p.q -= cq ? g.qpr : 0;
      p.y += g.dy + (cq ? 1 : 0);
      const bool cy = p.y >= g.H;
      p.y -= cy ? g.H : 0;
      p.n += g.dn + (cy ? 1 : 0);
    }
  };
  auto first_col = [&](const Quad& p) { return min(4 * p.q, g.W - 4); };

  s3_f4 xr[NT][2], gr[FB][2];
  uint32_t ir[FB][2];
  auto load_x = [&]() {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const Quad& p = qd[h];
      const int x0 = first_col(p);
      const uint32_t at = (uint32_t)(p.n * (CIN * HW) + p.y * g.W + x0) * 4u;
      const bool live = p.v < g.nquad;
#pragma unroll
      for (int j = 0; j < NT; ++j) {
        const bool in = live && !none[j] && !(up[j] && p.y == 0) && !(down[j] && p.y == g.H - 1);
        // at a row's ends the load is moved a pixel inwards (no load leaves the tensor) and put right by `edges`
        const uint32_t o = at + koff[j] + (left[j] && x0 == 0 ? 4u : 0u) - (right[j] && x0 == g.W - 4 ? 4u : 0u);
        xr[j][h] = __builtin_bit_cast(s3_f4, __builtin_amdgcn_raw_buffer_load_b128(rx, in ? o : kOutside, 0, 0));
      }
    }
  };
  auto edges = [&]() {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int x0 = first_col(qd[h]);
      if (!__any(x0 == 0 || x0 == g.W - 4)) continue;
#pragma unroll
      for (int j = 0; j < NT; ++j) {
        const bool tl = left[j] && x0 == 0, tr = right[j] && x0 == g.W - 4;
        const float a = xr[j][h][0], b = xr[j][h][1], c = xr[j][h][2], d = xr[j][h][3];
        xr[j][h][0] = tl ? 0.f : tr ? b : a;
        xr[j][h][1] = tl ? a : tr ? c : b;
        xr[j][h][2] = tl ? b : tr ? d : c;
        xr[j][h][3] = tl ? c : tr ? 0.f : d;
      }
    }
  };
  auto load_g = [&](int b) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const Quad& p = qd[h];
      const bool live = p.v < g.nquad;
      const uint32_t o = (uint32_t)(p.n * g.Cout * HW + p.y * g.W + first_col(p)) + foff[b];
      gr[b][h] = __builtin_bit_cast(s3_f4, __builtin_amdgcn_raw_buffer_load_b128(rg, live ? o * 4u : kOutside, 0, 0));
      ir[b][h] = load4(idx + (live ? o : 0u));
    }
  };

  s3_f4 acc[FB][4][NT];
#pragma unroll
  for (int b = 0; b < FB; ++b)
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int j = 0; j < NT; ++j) acc[b][s][j] = s3_f4{0.f, 0.f, 0.f, 0.f};

  if (step < stop) {
    load_x();
#pragma unroll
    for (int b = 0; b < FB; ++b) load_g(b);
  }
#pragma unroll 1
  for (; step < stop; ++step) {
    edges();
    u32x4 xp[NT][3];
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          auto flip = [&](float v) { return __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, v) ^ turned); };
          const float lo = xr[j][h][2 * e], hi = xr[j][h][2 * e + 1];
          const S3Pair s = s3_split2(flip(lo), flip(hi));
#pragma unroll
          for (int i = 0; i < 3; ++i) xp[j][i][2 * h + e] = s.p[i];
        }
    uint32_t again[2];                 // pixels of a row's last quad that the one before it has: a byte each
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int rep = 4 * qd[h].q - first_col(qd[h]);
      again[h] = (1u << 8 * rep) - 1u;                             // (0 to 3)
    }
    advance();
    load_x();
#pragma unroll
    for (int b = 0; b < FB; ++b) {
      u32x4 gp[3];
      uint32_t sel[4];                 // a byte per half of a pair's parts: the turn, or 4 for none
#pragma unroll
      for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const float lo = gr[b][h][2 * e], hi = gr[b][h][2 * e + 1];
          const S3Pair s = s3_split2(lo, hi);
#pragma unroll
          for (int i = 0; i < 3; ++i) gp[i][2 * h + e] = s.p[i];
        }
        const uint32_t v = ir[b][h] | again[h];
        const uint32_t no = ((((v & 0x7c7c7c7cu) + 0x7c7c7c7cu) | v) & 0x80808080u) >> 5;      // any idx beyond 3
        const uint32_t turn = (v & 0x03030303u) | no;
        sel[2 * h] = __builtin_amdgcn_perm(0u, turn, 0x01010000u);
        sel[2 * h + 1] = __builtin_amdgcn_perm(0u, turn, 0x03030202u);
      }
      load_g(b);
#pragma unroll
      for (int s2 = 0; s2 < 4; s2 += 2) {
        u32x4 a[2][3];
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const uint32_t m = __builtin_amdgcn_perm(0u, 0xffu << 8 * (s2 + s), sel[i]);
#pragma unroll
            for (int e = 0; e < 3; ++e) a[s][e][i] = gp[e][i] & m;
          }
        s3_f4 c[2][NT];
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
          for (int j = 0; j < NT; ++j) c[s][j] = s3_f4{0.f, 0.f, 0.f, 0.f};
        auto product = [&](int ge, int xe) {
#pragma unroll
          for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int j = 0; j < NT; ++j) c[s][j] = s3_mfma(a[s][ge], xp[j][xe], c[s][j]);
        };
        // the smallest products first
        product(2, 0);
        product(0, 2);
        product(1, 1);
        product(1, 0);
        product(0, 1);
        product(0, 0);
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
          for (int j = 0; j < NT; ++j) acc[b][s2 + s][j] += c[s][j];
      }
    }
  }

  // ---- the workgroup's sums: waves ascending, turns ascending
#pragma unroll
  for (int b = 0; b < FB; ++b) {
    if (b) __syncthreads();
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float v = acc[b][s][j][r];
          red[((wave * 4 + s) * 16 + 4 * lg + r) * NP + 16 * j + lc] =
              __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, v) ^ turned);
        }
    __syncthreads();
    for (int o = tid; o < 16 * NC; o += 64 * kWaves) {
      const int f = o / NC, k = o % NC, ci = k / 9, u = k % 9;
      double sum = 0.;
#pragma unroll
      for (int w = 0; w < kWaves; ++w)
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const int t = s == 0 ? u : s == 1 ? 3 * (2 - u % 3) + u / 3 : s == 2 ? 8 - u : 3 * (u % 3) + 2 - u / 3;
          sum += red[((w * 4 + s) * 16 + f) * NP + 9 * ci + t];
        }
      part[((size_t)blockIdx.x * g.CoutPad + f0 + 16 * b) * NC + o] = (float)sum;
    }
  }
}

// dw[b][co][ci][ub] = sum_z coef_z * (sum over the workgroups, in 16 interleaved groups and a fixed tree, of dF[co][ci][t_z]):
// the transposed first-quadrant table (Eq. 16 / the adjoint of Eq. 17).  A workgroup per (filter, channel).
__global__ __launch_bounds__(256) void k_first_dw_finish(const float* __restrict__ part, float* __restrict__ dw,
                                                         const float* __restrict__ x, const float* __restrict__ gpool,
                                                         const uint8_t* __restrict__ idx, const int32_t* __restrict__ fqt_ptr,
                                                         const int32_t* __restrict__ fqt_col, const float* __restrict__ fqt_coef,
                                                         int B, int N, int H, int W, int Cout, int Cin, int CoutPad, int nchunk) {
  __shared__ double red[256][9];
  __shared__ float tot[9];
  __shared__ int odd;
  const int co = blockIdx.x / Cin, ci = blockIdx.x % Cin;
  const int t = threadIdx.x % 16, grp = threadIdx.x / 16, NA = Cin * 9;
  if (threadIdx.x == 0) odd = 0;
  if (t < 9) {
    const float* src = part + (size_t)co * NA + ci * 9 + t;
    const size_t pitch = (size_t)CoutPad * NA;
    double s = 0.;
    for (int c0 = grp; c0 < nchunk; c0 += 64) {                    // four loads on their way together
      float v[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = c0 + 16 * i < nchunk ? src[(c0 + 16 * i) * pitch] : 0.f;
#pragma unroll
      for (int i = 0; i < 4; ++i) s += v[i];
    }
    red[grp][t] = s;
  }
  __syncthreads();
  if (threadIdx.x < 9) {
    const int u = threadIdx.x;
    double a[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) a[i] = red[i][u];
#pragma unroll
    for (int n = 8; n >= 1; n /= 2)
#pragma unroll
      for (int i = 0; i < n; ++i) a[i] = a[i] + a[i + n];
    tot[u] = (float)a[0];
    if (beyond_parts(tot[u])) odd = 1;
  }
  __syncthreads();
  if (odd) {                           // sums that the parts do not hold, in fp32: a thread four pixels of a row at a time
    // (gradients of NaN throughout, 2x3 -> 64, 512x512: 1.5 ms instead of 68 us; with 36 loads per pixel 13)
    float a[9];
#pragma unroll
    for (int u = 0; u < 9; ++u) a[u] = 0.f;
    const int HW = H * W, qpr = (W + 3) / 4;
#pragma unroll 1
    for (int e = threadIdx.x; e < N * H * qpr; e += 256) {
      const int n = e / (H * qpr), y = e / qpr - n * H, c = 4 * (e % qpr);
      const size_t plane = ((size_t)n * Cout + co) * HW;
      const float* xr = x + ((size_t)n * Cin + ci) * HW + (size_t)y * W;
      float g[3][6];                   // the gradients around them, and their turns
      int t[3][6];
#pragma unroll
      for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 6; ++j) {
          const int yy = y + i - 1, xx = c + j - 1;
          const bool in = (unsigned)yy < (unsigned)H && (unsigned)xx < (unsigned)W;
          const size_t o = plane + (in ? yy * W + xx : 0);
          g[i][j] = gpool[o];
          t[i][j] = in ? idx[o] : 255;
        }
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        if (c + b >= W) continue;
        const float xv = xr[c + b];
#pragma unroll
        for (int u = 0; u < 9; ++u) {
          float d = 0.f;
#pragma unroll
          for (int s = 0; s < 4; ++s) d += t[2 - tap_i(s, u)][b + 2 - tap_j(s, u)] == s ? g[2 - tap_i(s, u)][b + 2 - tap_j(s, u)] : 0.f;
          a[u] += d * xv;
        }
      }
    }
#pragma unroll
    for (int u = 0; u < 9; ++u) red[threadIdx.x][u] = a[u];
    __syncthreads();
    if (threadIdx.x < 9) {
      double s = 0.;
      for (int i = 0; i < 256; ++i) s += red[i][threadIdx.x];
      if (beyond_parts(tot[threadIdx.x])) tot[threadIdx.x] = (float)s;
    }
    __syncthreads();
  }
  if (threadIdx.x < B * 9) {
    const int b = threadIdx.x / 9, ub = threadIdx.x % 9;
    float v = 0.f;
    for (int z = fqt_ptr[b * 9 + ub]; z < fqt_ptr[b * 9 + ub + 1]; ++z) v += fqt_coef[z] * tot[fqt_col[z]];     // col = tap (one bank)
    dw[((size_t)(b * Cout + co) * Cin + ci) * 9 + ub] = v;
  }
}

struct Launch { FirstWGeom g; int fb, nfg, wg; };
Launch first_w_launch(const rotconv_plan* p) {
  const rotconv_desc& d = p->d;
  Launch l{};
  FirstWGeom& g = l.g;
  g.H = d.H; g.W = d.W; g.Cout = d.Cout;
  g.qpr = (d.W + 3) / 4; g.qpi = g.qpr * d.H; g.nquad = g.qpi * d.N;
  g.steps = (g.nquad + 7) / 8;
  // Two blocks of filters share a step's split pixels; one where every wave has a step only (6x2 -> 20, 186x23: 12.7 us with two,
  // 11.6 with one) and for four channels, whose 48 columns would spill.
  l.fb = d.Cout <= 16 || d.Cin > 3 || (long)g.steps * ((d.Cout + 15) / 16) <= 2048 ? 1 : 2;
  l.nfg = (d.Cout + 16 * l.fb - 1) / (16 * l.fb);
  g.CoutPad = l.nfg * 16 * l.fb;
  g.dn = 8 / g.qpi; g.dy = 8 % g.qpi / g.qpr; g.dx = 8 % g.qpi % g.qpr;
  g.xbytes = (uint32_t)(4.0 * d.N * d.Cin * d.H * d.W);
  g.gbytes = (uint32_t)(4.0 * d.N * d.Cout * d.H * d.W);
  // two waves per SIMD, all resident at once
  const int waves = std::max(kWaves, 2048 / l.nfg);
  g.per = std::max(1, (g.steps + waves - 1) / waves);
  l.wg = (g.steps + g.per * kWaves - 1) / (g.per * kWaves);
  return l;
}

template <int CIN>
void launch_cin(const Launch& l, const float* x, const float* gpool, const uint8_t* idx, float* part, hipStream_t st) {
  constexpr int NP = 16 * ((9 * CIN + 15) / 16) + 1;
  const size_t lds = (size_t)kWaves * 4 * 16 * NP * sizeof(float);
  auto go = [&](auto kern) {
    if (lds > 64 << 10) (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL(kern, dim3(l.wg, l.nfg), dim3(64 * kWaves), lds, st, x, gpool, idx, part, l.g);
  };
  if constexpr (CIN <= 3) {
    if (l.fb == 2) return go(k_first_bwd_weight<CIN, 2>);
  }
  go(k_first_bwd_weight<CIN, 1>);
}

}  // namespace

// The four quarter turns of one bank in their order (direct_bwd_weight_supported), rows of at least a quad, tensors within a
// 32-bit offset.  Large images with few of a tile's sixteen rows in use stay on the vector ALU, which takes filters in twos:
// 3x4 -> 1, 518x360 30.4 us there and 34.6 here, 8x2 -> 3, 512x128 23.6 / 26.8, 4 -> 22 channels 65.3 / 67.7; but 3x1 -> 3,
// 518x390 29.7 / 22.2, 6x3 -> 10, 464x292 43.8 / 37.6, and up to 2^17 pixels both are a few steps per wave (20 / 13).
bool first_bwd_weight_layer(const rotconv_plan* p) {
  const rotconv_desc& d = p->d;
  if (d.W < 4 || p->opt.bf16_parts < 0 || p->opt.direct_ty > 0) return false;             // the vector-ALU kernel asked for
  const int used = d.Cin < 2 ? 0 : d.Cin < 4 ? 4 : 11;
  if (p->opt.bf16_parts == 0 && (long)d.N * d.H * d.W > 1 << 17 && d.Cout <= used * ((d.Cout + 15) / 16)) return false;
  const double hw4 = 4.0 * d.N * d.H * d.W;
  return direct_bwd_weight_supported(p) && hw4 * d.Cin < 4e9 && hw4 * d.Cout < 4e9;
}

size_t first_bwd_weight_ws_floats(const rotconv_plan* p) {
  const Launch l = first_w_launch(p);
  return (size_t)l.wg * l.g.CoutPad * p->d.Cin * 9;
}

void launch_first_bwd_weight(const rotconv_plan* p, const float* x, const float* gpool, const uint8_t* idx, float* part,
                             float* dw, hipStream_t st) {
  const rotconv_desc& d = p->d;
  const Launch l = first_w_launch(p);
  switch (d.Cin) {
    case 1: launch_cin<1>(l, x, gpool, idx, part, st); break;
    case 2: launch_cin<2>(l, x, gpool, idx, part, st); break;
    case 3: launch_cin<3>(l, x, gpool, idx, part, st); break;
    default: launch_cin<4>(l, x, gpool, idx, part, st); break;
  }
  hipLaunchKernelGGL(k_first_dw_finish, dim3(d.Cout * d.Cin), dim3(256), 0, st, part, dw, x, gpool, idx, p->dev.fqt_ptr,
                     p->dev.fqt_col, p->dev.fqt_coef, p->B, d.N, d.H, d.W, d.Cout, d.Cin, l.g.CoutPad, l.wg);
}

}  // namespace rotconv
