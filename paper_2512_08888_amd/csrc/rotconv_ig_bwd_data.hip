// Input gradient of fp32 layers with filters of other sizes and strides, pooled over the four quarter turns, as one contraction on
// the bf16 matrix cores, operands split into three bf16 parts (rotconv_split3.h): nothing is routed through memory.
//
//   dX[ci, p] = sum_(co, s, T) w[co, ci, rot^-s T] (G * 1[idx == s])[co, (p + pad - T) / stride]
//
// The forward's contraction (rotconv_ig_fwd.hip) turned round: an orbit of four taps, whose weights are held in registers, meets
// the pooled gradients at the orbit's four positions.  The four turns' gradients at a position are the same numbers masked by
// idx, so G is split once and its parts are masked (two instructions per pair of filters, part and turn); the turns exclude
// each other, so one position's products of all four turns form one sum.
//
// A workgroup owns WC blocks of 16 MT input channels and 64 NT input pixels of an image, four waves a block.  32 filters at a
// time, the outputs that the tile's taps reach are staged in LDS, [pixel][part][filter] and the turns, a byte per half of a pair of
// filters.  With a stride, pixels whose positions leave the same remainder are a tile (stride^2 kinds): every tap that reaches one of
// them reaches all.
//
// Precision: as in the forward; every other position's gradients have their signs turned and the sum is subtracted.
//
// What bounds it: a lone wave's chain of products where the map has few tiles (shares of the filters and orbits then), else matrix
// and mask instructions (16 for 24 MT products) together.  2x32 -> 32, 96x96, 5 x 5: 65 us with routed gradients through memory, 34
// so; 2x13 -> 64, 39x42, 7 x 7 172 / 21; 60 layers of 12 to 64 channels and filters, k = 2, 5, 7, stride 1 and 2: 0.30 of the time
// in the mean, 0.10 to 0.79.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "glue_internal.h"
#include "rotconv_ig.h"
#include "rotconv_ig_orbits.h"
#include "rotconv_split3.h"

namespace rotconv {
namespace {

constexpr int kPixel = 17;             // 16-byte units of an output pixel in LDS: three parts and the turns of 32 filters

struct IgDxGeom {
  int Cin, H, W, Cout, k, kk, stride, pad, Ho, Wo;
  int th, tw, nty, ntx, rw, npix;      // tile of input pixels (of one remainder), tiles per image, its region of outputs
  uint32_t mrw;                        // ceil(2^22 / rw)
  int nch, per, ncb;                   // 32-filter chunks, chunks per share, blocks of channels
  int osplit, oper;                    // shares of the orbits, orbits per share (the last share has the centre)
  uint32_t gbytes;                     // pooled gradients of an image
  size_t part;                         // elements of a share
};

__device__ __host__ __forceinline__ int ceil_div(int a, int b) { return a >= 0 ? (a + b - 1) / b : -(-a / b); }

// MANY: a workgroup has more than 32 filters
template <int MT, int NT, int WC, bool MANY>
__global__ __launch_bounds__(256 * WC, 2) void k_ig_bwd_data(const float* __restrict__ gpool, const uint8_t* __restrict__ idx,
                                                             const u32x4* __restrict__ wp, const float* __restrict__ w,
                                                             float* __restrict__ dx, IgDxGeom g) {
  constexpr int NTH = 256 * WC;
  extern __shared__ u32x4 Gl[];        // [pixel][part or turns][quarter]
  const int tid = threadIdx.x, lane = tid % 64, lg = lane / 16, lc = lane % 16;
  const int wave = __builtin_amdgcn_readfirstlane(tid / 64) % 4, wc = __builtin_amdgcn_readfirstlane(tid / 256);
  const int per_xcd = gridDim.x / 8;   // blocks of one tile behind each other on one XCD
  int v = gridDim.x % 8 == 0 ? (blockIdx.x % 8) * per_xcd + blockIdx.x / 8 : blockIdx.x;
  const int ncw = (g.ncb + WC - 1) / WC;
  const int cb = v % ncw * WC + wc; v /= ncw;
  const int tx = v % g.ntx; v /= g.ntx;
  const int ty = v % g.nty, n = v / g.nty;
  const int c0 = blockIdx.y / g.osplit * g.per, c1 = min(g.nch, c0 + g.per);
  const int os = blockIdx.y % g.osplit, o0 = os * g.oper, o1 = min(g.kk / 4, o0 + g.oper);
  const bool centre = (g.k & 1) && os == g.osplit - 1;
  const int py = blockIdx.z / g.stride, px = blockIdx.z % g.stride;          // the pixels' remainder
  const int first_y = ceil_div(py + g.pad - (g.k - 1), g.stride), first_x = ceil_div(px + g.pad - (g.k - 1), g.stride);
  const int oy0 = ty * g.th + first_y, ox0 = tx * g.tw + first_x;            // the region's first output
  const int HWo = g.Ho * g.Wo;
  const float* gi = gpool + (size_t)n * g.Cout * HWo;
  const uint8_t* ii = idx + (size_t)n * g.Cout * HWo;
  const auto rg = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(gi), 0, (int)g.gbytes, 0x27000);
  const auto ri = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(ii), 0, (int)(g.gbytes / 4), 0x27000);
  const int items = g.npix * 4;        // eight filters of an output each

  int y[NT], x[NT], base[NT];
  bool live[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int p = (wave * NT + t) * 16 + lc, ly = p / g.tw, lx = p - ly * g.tw;
    y[t] = (ty * g.th + ly) * g.stride + py; x[t] = (tx * g.tw + lx) * g.stride + px;
    live[t] = ly < g.th && y[t] < g.H && x[t] < g.W;
    base[t] = (live[t] ? ly * g.rw + lx : 0) * kPixel + lg;
  }

  s3_f4 acc[MT][NT], sum[MANY ? MT : 1][MANY ? NT : 1];
  auto clear = [&](auto& a) {
    for (auto& row : a)
      for (auto& e : row) e = s3_f4{0.f, 0.f, 0.f, 0.f};
  };
  clear(acc);
  if constexpr (MANY) clear(sum);

  auto stage = [&](int c) {
    for (int e = tid; e < items; e += NTH) {
      const int pix = e >> 2, ry = (int)((uint32_t)pix * g.mrw >> 22), rx = pix - ry * g.rw, oy = oy0 + ry, ox = ox0 + rx;
      const bool ok = (unsigned)oy < (unsigned)g.Ho && (unsigned)ox < (unsigned)g.Wo;
      const uint32_t o = (uint32_t)((c * 32 + 8 * (e & 3)) * HWo + oy * g.Wo + ox);
      float r[8];
      uint32_t b[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        r[i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rg, ok ? (o + (uint32_t)(i * HWo)) * 4u : kOutside, 0, 0));
        b[i] = __builtin_amdgcn_raw_buffer_load_b8(ri, ok ? o + (uint32_t)(i * HWo) : kOutside, 0, 0);
      }
      u32x4 q[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const S3Pair s = s3_split2(r[2 * i], r[2 * i + 1]);
#pragma unroll
        for (int d = 0; d < 3; ++d) q[d][i] = s.p[d];
      }
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const uint32_t u = b[4 * h] | b[4 * h + 1] << 8 | b[4 * h + 2] << 16 | b[4 * h + 3] << 24;
        const uint32_t no = ((((u & 0x7c7c7c7cu) + 0x7c7c7c7cu) | u) & 0x80808080u) >> 5;      // any idx beyond 3
        const uint32_t at = (u & 0x03030303u) | no;
        q[3][2 * h] = __builtin_amdgcn_perm(0u, at, 0x01010000u);
        q[3][2 * h + 1] = __builtin_amdgcn_perm(0u, at, 0x03030202u);
      }
#pragma unroll
      for (int d = 0; d < 4; ++d) Gl[pix * kPixel + d * 4 + (e & 3)] = q[d];
    }
  };

  // does tap position (i, j) reach the tile's pixels, and how far into the region?
  auto reach = [&](Orbit t, int& off) {
    const int dy = py + g.pad - t.i, dxx = px + g.pad - t.j;
    if (g.stride == 1) {
      off = ((dy - first_y) * g.rw + dxx - first_x) * kPixel;
      return true;
    }
    const int qy = ceil_div(dy, g.stride), qx = ceil_div(dxx, g.stride);
    off = ((qy - first_y) * g.rw + qx - first_x) * kPixel;
    return qy * g.stride == dy && qx * g.stride == dxx;
  };
  constexpr int kPa[5] = {2, 0, 1, 1, 0}, kPb[5] = {0, 2, 1, 0, 1};          // the small products; then the parts' first ones
  const u32x4* wl = wp + (size_t)min(cb, g.ncb - 1) * g.nch * g.kk * MT * 192 + lane;
  // with strides beyond k no tap reaches most kinds of pixels: their gradients are zero
  const bool reached = (py + g.pad) % g.stride < g.k && (px + g.pad) % g.stride < g.k;
#pragma unroll 1
  for (int c = c0; c < (reached ? c1 : c0); ++c) {
    const u32x4* wq = wl + (size_t)c * g.kk * MT * 192;
    if (c > c0) __syncthreads();
    stage(c);
    __syncthreads();

    auto weights = [&](int tile, u32x4 (&a)[MT][3]) {
#pragma unroll
      for (int r = 0; r < MT; ++r)
#pragma unroll
        for (int d = 0; d < 3; ++d) a[r][d] = wq[((tile * MT + r) * 3 + d) * 64];
    };
#pragma unroll 1
    for (int o = o0; o < o1; ++o) {
      u32x4 a[4][MT][3];
      Orbit pos[4];
      int off[4];
      bool in[4];
      pos[0] = orbit_rep(o, g.k);
#pragma unroll
      for (int m = 1; m < 4; ++m) pos[m] = turn(pos[m - 1], g.k);
      bool any = false;
#pragma unroll
      for (int m = 0; m < 4; ++m) any |= in[m] = reach(pos[m], off[m]);
      if (!any) continue;
#pragma unroll
      for (int d = 0; d < 4; ++d) weights(4 * o + d, a[d]);
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        s3_f4 all[2][MT];              // of positions 0 and 1, of positions 2 and 3
        clear(all);
#pragma unroll
        for (int m = 0; m < 4; ++m) {
          if (!in[m]) continue;
          const u32x4* at = Gl + base[t] + off[m];
          u32x4 b[3], sel = at[12], main[4];
#pragma unroll
          for (int d = 0; d < 3; ++d) b[d] = at[d * 4];
          if (m & 1)
#pragma unroll
            for (int d = 0; d < 3; ++d) b[d] ^= 0x80008000u;
          s3_f4 p[MT];
#pragma unroll
          for (int r = 0; r < MT; ++r) p[r] = s3_f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int s = 0; s < 4; ++s) {
            u32x4 q[3];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const uint32_t mask = __builtin_amdgcn_perm(0u, 0xffu << 8 * s, sel[i]);
#pragma unroll
              for (int d = 0; d < 3; ++d) q[d][i] = b[d][i] & mask;
            }
            main[s] = q[0];
#pragma unroll
            for (int e = 0; e < 5; ++e)
#pragma unroll
              for (int r = 0; r < MT; ++r) p[r] = s3_mfma(a[(m - s) & 3][r][kPa[e]], q[kPb[e]], p[r]);
          }
#pragma unroll
          for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int r = 0; r < MT; ++r) p[r] = s3_mfma(a[(m - s) & 3][r][0], main[s], p[r]);
#pragma unroll
          for (int r = 0; r < MT; ++r) {
            if (m & 1) all[m / 2][r] -= p[r];
            else all[m / 2][r] += p[r];
          }
        }
#pragma unroll
        for (int r = 0; r < MT; ++r) acc[r][t] += all[0][r] + all[1][r];
      }
    }
    int off;
    if (centre && reach(Orbit{g.k / 2, g.k / 2}, off)) {          // every turn's
      u32x4 a[MT][3];
      weights(g.kk - 1, a);
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const u32x4* at = Gl + base[t] + off;
        u32x4 q[3], sel = at[12];
#pragma unroll
        for (int d = 0; d < 3; ++d) q[d] = at[d * 4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const uint32_t mask = __builtin_amdgcn_perm(0u, 0xffffffffu, sel[i]);
#pragma unroll
          for (int d = 0; d < 3; ++d) q[d][i] &= mask;
        }
#pragma unroll
        for (int r = 0; r < MT; ++r) {
          s3_f4 p{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int e = 0; e < 5; ++e) p = s3_mfma(a[r][kPa[e]], q[kPb[e]], p);
          acc[r][t] += s3_mfma(a[r][0], q[0], p);
        }
      }
    }
    if constexpr (MANY) {
#pragma unroll
      for (int r = 0; r < MT; ++r)
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          sum[r][t] += acc[r][t];
          acc[r][t] = s3_f4{0.f, 0.f, 0.f, 0.f};
        }
    }
  }
  if constexpr (MANY) {
#pragma unroll
    for (int r = 0; r < MT; ++r)
#pragma unroll
      for (int t = 0; t < NT; ++t) acc[r][t] = sum[r][t];
  }

  const int f0 = cb * 16 * MT + 4 * lg, fend = cb < g.ncb ? g.Cin : 0;
  bool odd = false;
#pragma unroll
  for (int r = 0; r < MT; ++r)
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i) odd |= beyond_parts(acc[r][t][i]);
  if (__builtin_expect(__any(odd), 0)) {      // the wave's sums in fp32; those that the parts do not hold are replaced
    s3_f4 fresh[MT][NT];
    clear(fresh);
#pragma unroll 1
    for (int co = c0 * 32; co < min(g.Cout, c1 * 32); ++co) {
      const float* wr[MT][4];
#pragma unroll
      for (int r = 0; r < MT; ++r)
#pragma unroll
        for (int i = 0; i < 4; ++i) wr[r][i] = w + ((size_t)co * g.Cin + min(f0 + 16 * r + i, g.Cin - 1)) * g.kk;
      // adds what the output at a position that the tile's pixels reach gives to tile t, by its turn's weights (0 to 3)
      // (gradients of NaN throughout, 2x32 -> 32, 96x96, 5 x 5: 0.32 ms instead of 45 us; an element at a time 6.7)
      auto output = [&](int t, Orbit at, auto weight) {
        const int dy = y[t] + g.pad - at.i, dxx = x[t] + g.pad - at.j, oy = dy / g.stride, ox = dxx / g.stride;
        const bool in = live[t] && dy >= 0 && dxx >= 0 && oy < g.Ho && ox < g.Wo;
        const size_t o = in ? (size_t)co * HWo + (size_t)oy * g.Wo + ox : 0;
        const float gv = gi[o];
        const int s = in ? ii[o] : 255;
        if (s < 4)
#pragma unroll
          for (int r = 0; r < MT; ++r)
#pragma unroll
            for (int i = 0; i < 4; ++i) fresh[r][t][i] += weight(s, r, i) * gv;
      };
#pragma unroll 1
      for (int o = o0; o < o1; ++o) {
        Orbit pos[4];
        int off;
        pos[0] = orbit_rep(o, g.k);
#pragma unroll
        for (int m = 1; m < 4; ++m) pos[m] = turn(pos[m - 1], g.k);
        float wv[4][MT][4];
#pragma unroll
        for (int d = 0; d < 4; ++d)
#pragma unroll
          for (int r = 0; r < MT; ++r)
#pragma unroll
            for (int i = 0; i < 4; ++i) wv[d][r][i] = wr[r][i][pos[d].i * g.k + pos[d].j];
#pragma unroll
        for (int m = 0; m < 4; ++m) {
          if (!reach(pos[m], off)) continue;
#pragma unroll
          for (int t = 0; t < NT; ++t)
            output(t, pos[m], [&](int s, int r, int i) {
              const float lo = s & 1 ? wv[(m - 1) & 3][r][i] : wv[m][r][i], hi = s & 1 ? wv[(m - 3) & 3][r][i] : wv[(m - 2) & 3][r][i];
              return s & 2 ? hi : lo;
            });
        }
      }
      int off;
      if (centre && reach(Orbit{g.k / 2, g.k / 2}, off))
#pragma unroll
        for (int t = 0; t < NT; ++t) output(t, Orbit{g.k / 2, g.k / 2}, [&](int, int r, int i) { return wr[r][i][g.kk / 2]; });
    }
#pragma unroll
    for (int r = 0; r < MT; ++r)
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[r][t][i] = beyond_parts(acc[r][t][i]) ? fresh[r][t][i] : acc[r][t][i];
  }

  float* out = dx + (size_t)blockIdx.y * g.part;
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int r = 0; r < MT; ++r)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int ci = f0 + 16 * r + i;
        if (live[t] && ci < fend) out[(((size_t)n * g.Cin + ci) * g.H + y[t]) * g.W + x[t]] = acc[r][t][i];
      }
}

// The weights' parts in the order of their use: [block of channels][chunk of 32 filters][tap][16 channels of the block][part][lane]
// [8 filters].
__global__ __launch_bounds__(256) void k_ig_pack_t(const float* __restrict__ w, uint32_t* __restrict__ out, int mt, int Cout, int Cin,
                                                   int k, int nch) {
  const int kk = k * k;
  const int j = threadIdx.x % 4, lane = threadIdx.x / 4;
  int v = blockIdx.x;
  const int r = v % mt; v /= mt;
  const int c = v % nch, cb = v / nch;
  const int ci = (cb * mt + r) * 16 + lane % 16, co = c * 32 + 8 * (lane / 16) + 2 * j;
  const float* src = w + ((size_t)min(co, Cout - 1) * Cin + min(ci, Cin - 1)) * kk;
  const size_t second = co + 1 < Cout ? (size_t)Cin * kk : 0;
  uint32_t* dst = out + ((size_t)(cb * nch + c) * kk * mt * 3 * 64 + lane) * 4 + j;
  for (int t = blockIdx.y; t < kk; t += gridDim.y) {
    const int u = packed_tap(t, k);
    float a = src[u], b = src[second + u];
    a = co < Cout && ci < Cin ? a : 0.f;
    b = co + 1 < Cout && ci < Cin ? b : 0.f;
    uint16_t p[2][3];
    s3_split_weight(a, p[0][0], p[0][1], p[0][2]);
    s3_split_weight(b, p[1][0], p[1][1], p[1][2]);
#pragma unroll
    for (int e = 0; e < 3; ++e) dst[((size_t)(t * mt + r) * 3 + e) * 256] = (uint32_t)p[0][e] | (uint32_t)p[1][e] << 16;
  }
}

int chunks(const rotconv_plan* p) { return (p->d.Cout + 31) / 32; }
int channel_blocks(const rotconv_plan* p, int mt) { return (p->d.Cin + 16 * mt - 1) / (16 * mt); }
size_t pack_bytes(const rotconv_plan* p, int mt) { return (size_t)channel_blocks(p, mt) * chunks(p) * p->kk * mt * 3 * 1024; }
size_t lds_bytes(int pix) { return (size_t)pix * kPixel * 16; }
int reach_of(const rotconv_desc& d) { return (d.k + d.stride - 1) / d.stride; }
int region(const rotconv_desc& d, int th, int tw) { return (th - 1 + reach_of(d)) * (tw - 1 + reach_of(d)); }

}  // namespace

bool ig_bwd_data_supported(const rotconv_plan* p) {
  const rotconv_desc& d = p->d;
  return ig_fwd_supported(p) && d.R == 4 && 4.0 * (d.Cout + 32) * p->Ho * p->Wo < 4.2e9;
}

// As for the forward: the shape with the smallest modelled time (24 shapes of 60 layers: 1.4 % off the best in the mean).
IgShape ig_bwd_data_shape(const rotconv_plan* p, size_t budget) {
  const rotconv_desc& d = p->d;
  IgShape best{};
  best.us = 1e30;
  const int nch = chunks(p), st2 = d.stride * d.stride;
  const int Hq = (d.H + d.stride - 1) / d.stride, Wq = (d.W + d.stride - 1) / d.stride;
  const size_t part = 4 * (size_t)d.N * d.Cin * d.H * d.W;
  for (int nt = 2; nt >= 1; --nt)
    for (int mt = d.Cin <= 16 ? 1 : 2; mt <= (d.Cin <= 16 ? 1 : 2); ++mt) {
      int th = 0, tw = 0, pix = 0;
      long tiles = 0;
      for (int w = 1; w <= std::min(Wq, 64 * nt); ++w) {
        const int h = std::min(Hq, 64 * nt / w), px = region(d, h, w);
        if (lds_bytes(px) > 160 << 10) continue;
        const long n = (long)((Hq + h - 1) / h) * ((Wq + w - 1) / w);
        const double cost = n * (256. * nt + px), old = tiles * (256. * nt + pix);
        if (!tiles || cost < old) { th = h; tw = w; pix = px; tiles = n; }
      }
      if (!tiles) continue;
      if (pack_bytes(p, mt) > (size_t)256 << 20) continue;
      const int blocks = channel_blocks(p, mt);
      for (int wc = 1; wc <= (blocks > 1 ? 2 : 1); ++wc)
        for (int ns = 1; ns <= (budget ? nch : 1); ++ns) {
          const int per = (nch + ns - 1) / ns;
          if ((nch + per - 1) / per != ns) continue;
          for (int os = 1; os <= (budget ? std::max(1, p->kk / 4) : 1); ++os) {
            const int oper = (p->kk / 4 + os - 1) / os;
            if (os > 1 && (p->kk / 4 + oper - 1) / oper != os) continue;
            IgShape s{mt, nt, wc, th, tw, ns, os, 0.};
            if (s.parts() > 1 && pack_bytes(p, mt) + s.parts() * part + 512 > budget) continue;
            const double wgs = (double)tiles * d.N * ((blocks + wc - 1) / wc) * ns * os * st2;
            const double mfma = (os > 1 ? 16 * oper + 1 : 4 * p->kk) / (double)st2 * nt * mt * 6e-3;
            const double stage = per * (1.6 + 0.28 * pix * 4 / (256. * wc));
            const int occ = std::max(1, std::min(2 / wc, (int)((160 << 10) / lds_bytes(pix))));
            auto time = [&](int n) {
              const int waves = n * wc;
              return stage + per * mfma * (waves <= 1 ? 20. : 17.6 * waves);
            };
            const double full = 256. * occ, rest = std::fmod(wgs, full);
            s.us = std::floor(wgs / full) * time(occ) + (rest > 0 ? time((int)std::ceil(rest / 256)) : 0.) + 8. + part / 3e6;
            if (s.parts() > 1) s.us += 2.8 + s.parts() * part / 2e6;
            if (s.us < best.us) best = s;
          }
        }
    }
  return best;
}

size_t ig_bwd_data_ws_bytes(const rotconv_plan* p, const IgShape& s) {
  const size_t pack = (pack_bytes(p, s.mt) + 255) / 256 * 256;
  return pack + (s.parts() > 1 ? s.parts() * 4 * (size_t)p->d.N * p->d.Cin * p->d.H * p->d.W : 0);
}

void launch_ig_bwd_data(const rotconv_plan* p, const IgShape& s, const float* gpool, const uint8_t* idx, const float* w, float* dx,
                        void* ws, hipStream_t st) {
  const rotconv_desc& d = p->d;
  IgDxGeom g{};
  g.Cin = d.Cin; g.H = d.H; g.W = d.W; g.Cout = d.Cout; g.k = d.k; g.kk = p->kk; g.stride = d.stride; g.pad = d.pad;
  g.Ho = p->Ho; g.Wo = p->Wo;
  g.th = s.th; g.tw = s.tw;
  g.nty = ((d.H + d.stride - 1) / d.stride + s.th - 1) / s.th; g.ntx = ((d.W + d.stride - 1) / d.stride + s.tw - 1) / s.tw;
  g.rw = s.tw - 1 + reach_of(d); g.npix = region(d, s.th, s.tw);
  g.mrw = ((1u << 22) + g.rw - 1) / g.rw;
  g.nch = chunks(p); g.per = (g.nch + s.nsplit - 1) / s.nsplit; g.ncb = channel_blocks(p, s.mt);
  g.osplit = s.osplit; g.oper = (g.kk / 4 + s.osplit - 1) / s.osplit;
  g.gbytes = (uint32_t)(4.0 * d.Cout * p->Ho * p->Wo);
  g.part = p->n_x;
  const unsigned pb = (unsigned)(g.ncb * g.nch * s.mt);
  hipLaunchKernelGGL(k_ig_pack_t, dim3(pb, std::max(1u, std::min((unsigned)g.kk, 1024u / pb))), dim3(256), 0, st, w,
                     static_cast<uint32_t*>(ws), s.mt, d.Cout, d.Cin, d.k, g.nch);
  float* part = reinterpret_cast<float*>(static_cast<char*>(ws) + (pack_bytes(p, s.mt) + 255) / 256 * 256);
  float* out = s.parts() > 1 ? part : dx;
  const size_t lds = lds_bytes(g.npix);
  auto go = [&](auto kern) {
    if (lds > 64 << 10) (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL(kern, dim3((unsigned)((g.ncb + s.wc - 1) / s.wc * g.nty * g.ntx * d.N), (unsigned)((g.nch + g.per - 1) / g.per * g.osplit),
                                  (unsigned)(d.stride * d.stride)),
                       dim3(256 * s.wc), lds, st, gpool, idx, static_cast<const u32x4*>(ws), w, out, g);
  };
  auto by_many = [&](auto mt, auto nt, auto wc) {
    if (g.per > 1) go(k_ig_bwd_data<decltype(mt)::value, decltype(nt)::value, decltype(wc)::value, true>);
    else go(k_ig_bwd_data<decltype(mt)::value, decltype(nt)::value, decltype(wc)::value, false>);
  };
  const auto i1 = std::integral_constant<int, 1>{};
  const auto i2 = std::integral_constant<int, 2>{};
  auto by_wc = [&](auto mt, auto nt) {
    if (s.wc == 2) by_many(mt, nt, i2); else by_many(mt, nt, i1);
  };
  if (s.mt == 1) { if (s.nt == 2) by_many(i1, i2, i1); else by_many(i1, i1, i1); }      // (up to 16 channels: one block)
  else if (s.nt == 2) by_wc(i2, i2);
  else by_wc(i2, i1);
  if (s.parts() > 1) launch_sum_parts(part, dx, p->n_x, s.parts(), p->n_x, st);
}

}  // namespace rotconv
