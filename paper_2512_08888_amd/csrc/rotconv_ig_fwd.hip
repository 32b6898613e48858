// Forward of fp32 layers as ONE contraction over channels and taps on the bf16 matrix cores, operands split into three bf16
// parts (rotconv_split3.h): filters of any size and stride with the four quarter turns, and single orientations.
//
//   y_s[co, p] = sum_(ci, T) w[co, ci, rot^-s T] X[ci, p stride + T - pad]       (T: a position in the k x k window)
//
// The turns of a filter meet the same pixels with its taps in another order.  The k^2 positions fall into orbits of four
// that a quarter turn permutes (and the centre): the weights of an orbit's four taps, held in registers, and the pixels at its
// four positions give sixteen products, four for each turn.  The products are formed four times as often as where a tap's product
// is shared by the turns (rotconv_gs.hip), but nothing is placed: no product leaves the registers, a lane ends up with
// the four turns of a filter at its pixel and pools them there.
//
// A workgroup of four waves owns 16 filters (four turns) or 16 MT (one) and 64 NT output pixels of an image, a tile of th x tw, 16 NT
// of them a wave.  32 channels at a time, the input region of the tile is split once into LDS, [pixel][part][channel], where a
// position is an offset: a lane reads its pixel's eight channels (16 bytes) of a part.  A pixel takes 13 times 16 bytes, so that
// sixteen neighbours meet all banks.  The weights, packed in the
// order of their use, come from L1 / L2, a step ahead.
//
// Precision: the six products of a tap and 32 channels start from zero, smallest first, and only their total meets the running
// sum; every other tap's weights are packed with their signs turned and subtracted (the instruction cuts towards minus
// infinity); an orbit's four products, a row of taps and 32 channels are added up apart (all in one chain: 7.3e-8 of the norm for 64
// channels, 6.5e-8 so, as where products are placed).  A sum that is not finite, or below 2^-100 and not zero, is formed again
// in fp32 on the vector ALU: infinities, large and small values come out as there.
//
// What bounds it: with four turns the matrix cores where the map fills the chip (2x32 -> 32, 96x96, 5 x 5: 27 us with its pack,
// products through memory 65; 1x96 -> 96, 143x144, 5 x 5, stride 2 64 / 392; 2x50 -> 96, 144x69, 7 x 7, stride 2 70 / 1020: there
// the products of every input pixel are formed, here those of the output's), else a workgroup's own chain: 17 ns an instruction
// for a wave alone on its SIMD, 9.3 for two; maps of few tiles share out the orbits and channels.  With one turn 13 to 16 ns an
// instruction over all (1x512 -> 128, 16x16 17.7 us with placed products, 14.8 so; 0.75 to 1.3 of their time on
// large maps, see the choice in rotconv_api.hip): the weights' reads keep L1 at half its rate, the pixels' LDS too, and the vector
// work (0.75 per matrix instruction, and the splitting, which wc = 2 halves) hardly overlaps.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "rotconv_ig.h"
#include "rotconv_ig_orbits.h"
#include "rotconv_split3.h"

namespace rotconv {
namespace {

struct IgGeom {
  int Cin, H, W, Cout, k, kk, stride, pad, Ho, Wo, relu;
  int th, tw, nty, ntx, rw, npix;      // tile of output pixels, tiles per image, its input region
  uint32_t mrw;                        // ceil(2^22 / rw)
  int nch, per, cb0, ncb;              // 32-channel chunks, chunks per share, first filter block, filter blocks of the launch
  int osplit, oper;                    // shares of the orbits, orbits per share (the last share has the centre)
  uint32_t xbytes;                     // of an image
  size_t part;                         // elements of a share's responses
};

constexpr int kPixel = 13;             // 16-byte units of a pixel in LDS

// What a wave's registers allow.
__device__ __host__ constexpr int waves_per_simd(int S, int MT, int NT, bool MANY) {
  return S == 4 || MT * NT == 8 ? 2 : MANY && MT * NT == 4 ? 3 : 4;
}

// MANY: a workgroup has more than 32 channels; WC: groups of four waves, each with filters of its own
template <int S, int MT, int NT, int WC, bool POOL, bool MANY>
__global__ __launch_bounds__(256 * WC, waves_per_simd(S, MT, NT, MANY)) void k_ig_fwd(const float* __restrict__ x, const u32x4* __restrict__ wp,
                                                   const float* __restrict__ w, float* __restrict__ y, uint8_t* __restrict__ idx,
                                                   IgGeom g) {
  constexpr bool kAhead = S == 4 || NT < 4 || MT == 2;      // weights a step ahead (else no registers for them)
  constexpr int NTH = 256 * WC, NR = S == 4 ? 4 : MT;      // rows of tiles: a filter block's turns, or filter blocks
  extern __shared__ u32x4 Xl[];        // [pixel][part][quarter]
  const int tid = threadIdx.x, lane = tid % 64, lg = lane / 16, lc = lane % 16;
  const int per_xcd = gridDim.x / 8;   // blocks of one tile behind each other on one XCD
  int v = gridDim.x % 8 == 0 ? (blockIdx.x % 8) * per_xcd + blockIdx.x / 8 : blockIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid / 64) % 4, wc = __builtin_amdgcn_readfirstlane(tid / 256);
  const int ncw = (g.ncb + WC - 1) / WC;
  const int cb = v % ncw * WC + wc; v /= ncw;
  const int tx = v % g.ntx; v /= g.ntx;
  const int ty = v % g.nty, n = v / g.nty;
  const int c0 = blockIdx.y / g.osplit * g.per, c1 = min(g.nch, c0 + g.per);
  const int os = blockIdx.y % g.osplit, o0 = os * g.oper, o1 = min(g.kk / 4, o0 + g.oper);      // (four turns)
  const bool centre = S == 4 && (g.k & 1) && os == g.osplit - 1;
  const int oy0 = ty * g.th, ox0 = tx * g.tw, iy0 = oy0 * g.stride - g.pad, ix0 = ox0 * g.stride - g.pad;
  const int HW = g.H * g.W;
  const float* xi = x + (size_t)n * g.Cin * HW;
  const auto rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(xi), 0, (int)g.xbytes, 0x27000);
  const int items = g.npix * 4;        // eight channels of a pixel each

  // the lane's pixels
  int oy[NT], ox[NT], base[NT];
  bool live[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int p = (wave * NT + t) * 16 + lc, ly = p / g.tw, lx = p - ly * g.tw;
    live[t] = ly < g.th && oy0 + ly < g.Ho && ox0 + lx < g.Wo;
    oy[t] = oy0 + ly; ox[t] = ox0 + lx;
    base[t] = (live[t] ? (ly * g.rw + lx) * g.stride : 0) * kPixel + lg;
  }

  s3_f4 acc[NR][NT], sum[MANY ? NR : 1][MANY ? NT : 1];
  auto clear = [&](auto& a) {
    for (auto& row : a)
      for (auto& e : row) e = s3_f4{0.f, 0.f, 0.f, 0.f};
  };
  clear(acc);
  if constexpr (MANY) clear(sum);

  auto stage = [&](int c) {
    auto item = [&](int e, float (&r)[8]) {
      const int pix = e >> 2, ry = (int)((uint32_t)pix * g.mrw >> 22), rx_ = pix - ry * g.rw, iy = iy0 + ry, ix = ix0 + rx_;
      const bool ok = e < items && (unsigned)iy < (unsigned)g.H && (unsigned)ix < (unsigned)g.W;
      const uint32_t o = (uint32_t)((c * 32 + 8 * (e & 3)) * HW + iy * g.W + ix) * 4u;
#pragma unroll
      for (int i = 0; i < 8; ++i)
        r[i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rx, ok ? o + (uint32_t)(i * HW) * 4u : kOutside, 0, 0));
    };
    auto put = [&](int e, const float (&r)[8]) {
      u32x4 q[3];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const S3Pair s = s3_split2(r[2 * i], r[2 * i + 1]);
#pragma unroll
        for (int d = 0; d < 3; ++d) q[d][i] = s.p[d];
      }
      if (e < items)
#pragma unroll
        for (int d = 0; d < 3; ++d) Xl[(e >> 2) * kPixel + d * 4 + (e & 3)] = q[d];
    };
    for (int e = tid; e < items; e += 2 * NTH) {      // two on their way
      float a[8], b[8];
      item(e, a);
      item(e + NTH, b);
      put(e, a);
      put(e + NTH, b);
    }
  };
  auto pixels = [&](int t, int shift, u32x4 (&b)[3]) {
    const u32x4* at = Xl + base[t] + shift * kPixel;
#pragma unroll
    for (int d = 0; d < 3; ++d) b[d] = at[d * 4];
  };
  // the six products of one tile, smallest first
  auto weights = [&](const u32x4* src, u32x4 (&a)[3]) {
#pragma unroll
    for (int d = 0; d < 3; ++d) a[d] = src[d * 64];
  };
  constexpr int kPa[6] = {2, 0, 1, 1, 0, 0}, kPb[6] = {0, 2, 1, 0, 1, 0};

  const int tiles = S == 4 ? g.kk : g.kk * MT;
  const u32x4* wl = wp + (size_t)min(cb, g.ncb - 1) * g.nch * tiles * 192 + lane;
#pragma unroll 1
  for (int c = c0; c < c1; ++c) {
    const u32x4* wq = wl + (size_t)c * tiles * 192;
    u32x4 a[kAhead ? 2 : 1][NR][3];
    if constexpr (kAhead)
#pragma unroll
      for (int r = 0; r < NR; ++r)
        weights(wq + min((S == 4 ? 4 * o0 : 0) + r, tiles - 1) * 192, a[0][r]);
    if (c > c0) __syncthreads();
    stage(c);
    __syncthreads();

    if constexpr (S == 4) {
      // an orbit: the weights of tap d meet position m for turn (m - d) & 3; each turn's four products are added up apart
      auto orbit = [&](int o, const u32x4 (&now)[NR][3], u32x4 (&next)[NR][3]) {
#pragma unroll
        for (int r = 0; r < 4; ++r) weights(wq + min(4 * o + 4 + r, g.kk - 1) * 192, next[r]);
        Orbit pos[4];
        pos[0] = orbit_rep(o, g.k);
#pragma unroll
        for (int m = 1; m < 4; ++m) pos[m] = turn(pos[m - 1], g.k);
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          s3_f4 all[2][4];             // of positions 0 and 1, of positions 2 and 3
#pragma unroll
          for (int m = 0; m < 4; ++m) {
            u32x4 b[3];
            pixels(t, pos[m].i * g.rw + pos[m].j, b);
            s3_f4 p[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) p[r] = s3_f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int e = 0; e < 6; ++e)
#pragma unroll
              for (int r = 0; r < 4; ++r) p[r] = s3_mfma(now[(m - r) & 3][kPa[e]], b[kPb[e]], p[r]);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              if (m % 2 == 0) all[m / 2][r] = (m - r) & 1 ? -p[r] : p[r];
              else if ((m - r) & 1) all[m / 2][r] -= p[r];
              else all[m / 2][r] += p[r];
            }
          }
#pragma unroll
          for (int r = 0; r < 4; ++r) acc[r][t] += all[0][r] + all[1][r];
        }
      };
      int o = o0;
      for (; o + 2 <= o1; o += 2) {
        orbit(o, a[0], a[1]);
        orbit(o + 1, a[1], a[0]);
      }
      const bool left = o < o1;
      if (left) orbit(o, a[0], a[1]);
      if (centre) {                    // every turn's
        u32x4 ac[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) ac[d] = left ? a[1][0][d] : a[0][0][d];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          u32x4 b[3];
          pixels(t, g.k / 2 * (g.rw + 1), b);
          s3_f4 p{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int e = 0; e < 6; ++e) p = s3_mfma(ac[kPa[e]], b[kPb[e]], p);
#pragma unroll
          for (int r = 0; r < 4; ++r) acc[r][t] += p;
        }
      }
    } else {
      // a row of taps is added up apart
      s3_f4 row[NR][NT];
      int i = 0, j = 0;
      auto tap = [&](int u, bool turned, auto& now, auto& next) {
        const int at = kAhead ? min(u + 1, g.kk - 1) : u;
#pragma unroll
        for (int r = 0; r < NR; ++r) weights(wq + (at * MT + r) * 192, next[r]);
        if (j == 0) clear(row);
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          u32x4 b[3];
          pixels(t, i * g.rw + j, b);
          s3_f4 p[NR];
#pragma unroll
          for (int r = 0; r < NR; ++r) p[r] = s3_f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int e = 0; e < 6; ++e)
#pragma unroll
            for (int r = 0; r < NR; ++r) p[r] = s3_mfma(now[r][kPa[e]], b[kPb[e]], p[r]);
#pragma unroll
          for (int r = 0; r < NR; ++r) {
            if (turned) row[r][t] -= p[r];
            else row[r][t] += p[r];
          }
        }
        if (++j == g.k) {
          j = 0;
          ++i;
#pragma unroll
          for (int r = 0; r < NR; ++r)
#pragma unroll
            for (int t = 0; t < NT; ++t) acc[r][t] += row[r][t];
        }
      };
      constexpr int B1 = kAhead ? 1 : 0;
      int u = 0;
      for (; u + 2 <= g.kk; u += 2) {
        tap(u, false, a[0], a[B1]);
        tap(u + 1, true, a[B1], a[0]);
      }
      if (u < g.kk) tap(u, false, a[0], a[B1]);
    }
    if constexpr (MANY) {
#pragma unroll
      for (int r = 0; r < NR; ++r)
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          sum[r][t] += acc[r][t];
          acc[r][t] = s3_f4{0.f, 0.f, 0.f, 0.f};
        }
    }
  }
  if constexpr (MANY) {
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
      for (int t = 0; t < NT; ++t) acc[r][t] = sum[r][t];
  }

  const int f0 = (g.cb0 + cb) * 16 * MT + 4 * lg, fend = cb < g.ncb ? g.Cout : 0;
  bool odd = false;
#pragma unroll
  for (int r = 0; r < NR; ++r)
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i) odd |= beyond_parts(acc[r][t][i]);
  if (__builtin_expect(__any(odd), 0)) {      // the wave's sums in fp32; those that the parts do not hold are replaced
    s3_f4 fresh[NR][NT];
    clear(fresh);
    int ly[NT], lx[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) { ly[t] = oy[t] * g.stride - g.pad; lx[t] = ox[t] * g.stride - g.pad; }
#pragma unroll 1
    for (int ci = c0 * 32; ci < min(g.Cin, c1 * 32); ++ci) {
      const float* xc = xi + (size_t)ci * HW;
      const float* wr[S == 4 ? 1 : NR][4];
#pragma unroll
      for (int r = 0; r < (S == 4 ? 1 : NR); ++r)
#pragma unroll
        for (int i = 0; i < 4; ++i) wr[r][i] = w + ((size_t)min(f0 + 16 * r + i, g.Cout - 1) * g.Cin + ci) * g.kk;
      // (pixels of NaN throughout, 2x32 -> 32, 96x96, 5 x 5: 0.35 ms instead of 35 us; an element at a time 7.5)
      // the pixel of tile t at a position: nothing is added for those outside the image
      auto pixel = [&](int t, Orbit at, bool& in) {
        const int yy = ly[t] + at.i, xx = lx[t] + at.j;
        in = live[t] && (unsigned)yy < (unsigned)g.H && (unsigned)xx < (unsigned)g.W;
        return xc[in ? yy * g.W + xx : 0];
      };
      if constexpr (S == 4) {
#pragma unroll 1
        for (int o = o0; o < o1; ++o) {
          Orbit pos[4];
          pos[0] = orbit_rep(o, g.k);
#pragma unroll
          for (int m = 1; m < 4; ++m) pos[m] = turn(pos[m - 1], g.k);
          float wv[4][4];
#pragma unroll
          for (int d = 0; d < 4; ++d)
#pragma unroll
            for (int i = 0; i < 4; ++i) wv[d][i] = wr[0][i][pos[d].i * g.k + pos[d].j];
#pragma unroll
          for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int m = 0; m < 4; ++m) {
              bool in;
              const float xv = pixel(t, pos[m], in);
              if (in)
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                  for (int i = 0; i < 4; ++i) fresh[r][t][i] += wv[(m - r) & 3][i] * xv;
            }
        }
        if (centre)
#pragma unroll
          for (int t = 0; t < NT; ++t) {
            bool in;
            const float xv = pixel(t, Orbit{g.k / 2, g.k / 2}, in);
            if (in)
#pragma unroll
              for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int i = 0; i < 4; ++i) fresh[r][t][i] += wr[0][i][g.kk / 2] * xv;
          }
      } else {
#pragma unroll 1
        for (int u = 0; u < g.kk; ++u) {
          float wv[NR][4];
#pragma unroll
          for (int r = 0; r < NR; ++r)
#pragma unroll
            for (int i = 0; i < 4; ++i) wv[r][i] = wr[r][i][u];
#pragma unroll
          for (int t = 0; t < NT; ++t) {
            bool in;
            const float xv = pixel(t, Orbit{u / g.k, u % g.k}, in);
            if (in)
#pragma unroll
              for (int r = 0; r < NR; ++r)
#pragma unroll
                for (int i = 0; i < 4; ++i) fresh[r][t][i] += wv[r][i] * xv;
          }
        }
      }
    }
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[r][t][i] = beyond_parts(acc[r][t][i]) ? fresh[r][t][i] : acc[r][t][i];
  }

  float* yo = y + (size_t)blockIdx.y * g.part;
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int r = 0; r < (S == 4 && POOL ? 1 : NR); ++r)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int co = f0 + (S == 4 ? 0 : 16 * r) + i;
        if (!live[t] || co >= fend) continue;
        const size_t plane = S == 4 && !POOL ? ((size_t)n * g.Cout + co) * 4 + r : (size_t)n * g.Cout + co;
        const size_t o = (plane * g.Ho + oy[t]) * g.Wo + ox[t];
        float best = acc[r][t][i];
        if constexpr (!POOL) {
          yo[o] = best;
          continue;
        }
        int at = 0;
        if constexpr (S == 4) {
#pragma unroll
          for (int s = 1; s < 4; ++s) {
            const float c = acc[s][t][i];
            const bool gt = c > best;
            best = gt ? c : best;
            at = gt ? s : at;
          }
        }
        const bool dead = g.relu && best <= 0.f;
        yo[o] = dead ? 0.f : best;
        idx[o] = dead ? (uint8_t)255 : (uint8_t)at;
      }
}

// The weights' parts in the order of their use: [filter block][chunk][tile][part][lane][8 channels], a tile being a tap of 16
// filters; orbits of four taps and the centre (turns), or taps of MT blocks.
__global__ __launch_bounds__(256) void k_ig_pack(const float* __restrict__ w, uint32_t* __restrict__ out, int turns, int mt,
                                                 int cb0, int Cout, int Cin, int k, int nch) {
  const int kk = k * k, tiles = turns ? kk : kk * mt;
  const int j = threadIdx.x % 4, lane = threadIdx.x / 4;
  int v = blockIdx.x;
  const int r = v % mt; v /= mt;
  const int c = v % nch, cb = v / nch;
  const int co = ((cb0 + cb) * mt + r) * 16 + lane % 16, ci = c * 32 + 8 * (lane / 16) + 2 * j;
  const float* src = w + ((size_t)min(co, Cout - 1) * Cin + min(ci, Cin - 1)) * kk;
  const size_t second = ci + 1 < Cin ? kk : 0;
  uint32_t* dst = out + ((size_t)(cb * nch + c) * tiles * 3 * 64 + lane) * 4 + j;
  for (int t = blockIdx.y; t < kk; t += gridDim.y) {
    const int u = turns ? packed_tap(t, k) : t;
    const bool turned = turns ? (t & 1) && t < kk / 4 * 4 : t & 1;
    float a = src[u], b = src[second + u];
    a = co < Cout && ci < Cin ? a : 0.f;
    b = co < Cout && ci + 1 < Cin ? b : 0.f;
    uint16_t p[2][3];
    s3_split_weight(turned ? -a : a, p[0][0], p[0][1], p[0][2]);
    s3_split_weight(turned ? -b : b, p[1][0], p[1][1], p[1][2]);
    const int tile = turns ? t : t * mt + r;
#pragma unroll
    for (int e = 0; e < 3; ++e) dst[((size_t)tile * 3 + e) * 256] = (uint32_t)p[0][e] | (uint32_t)p[1][e] << 16;
  }
}

bool four_turns(const rotconv_plan* p) { return p->d.R == 4; }
int chunks(const rotconv_plan* p) { return (p->d.Cin + 31) / 32; }
size_t lds_bytes(int pix) { return (size_t)pix * kPixel * 16; }
int filter_blocks(const rotconv_plan* p, const IgShape& s) { return (p->d.Cout + 16 * s.mt - 1) / (16 * s.mt); }
size_t block_bytes(const rotconv_plan* p, const IgShape& s) { return (size_t)chunks(p) * p->kk * s.mt * 3 * 1024; }
int region(const rotconv_desc& d, int th, int tw) { return ((th - 1) * d.stride + d.k) * ((tw - 1) * d.stride + d.k); }

}  // namespace

bool ig_fwd_supported(const rotconv_plan* p) {
  const rotconv_desc& d = p->d;
  if (d.pool_op != ROTCONV_POOL_MAX || p->opt.bf16_parts != 0 || p->ng != 1 || p->host.Q != 1 || !p->base_bank) return false;
  if (d.R != 4 && d.R != 1) return false;
  for (int s = 0; s < d.R; ++s)
    if (p->rot_of[s] != s) return false;
  return 4.0 * (d.Cin + 32) * d.H * d.W < 4.2e9;
}

// The shape with the smallest modelled time (us): a workgroup stages and splits `chunk` + `item` per 32 channels and multiplies at
// `one`, `two` and `four` ns an instruction with that many waves on a SIMD; `start` for the launches, `bytes` (per us) for the
// results, `sum` and their bytes for adding up shares.  Fitted to 2300 launches of 130 layers with one turn (rms 10 %), and to the
// choice among 24 shapes of 60 layers with four (1.6 % off the best in the mean).
// budget: bytes that a block's weights and the shares may take.
IgShape ig_fwd_shape(const rotconv_plan* p, size_t budget) {
  const rotconv_desc& d = p->d;
  const bool turns = four_turns(p), may_split = budget > 0;
  struct { double chunk, item, one, two, four, start, bytes, sum; } k;
  if (turns) k = {1.75, 0.39, 13., 15., 15., 7.6, 1e6, 6.};
  else k = {1.4, 0.48, 16., 11.2, 10.6, 8.1, 5e6, 2.8};
  const size_t part = 4 * (size_t)d.N * d.Cout * d.R * p->Ho * p->Wo;
  const double out = 4.0 * d.N * d.Cout * p->Ho * p->Wo;
  IgShape best{};
  best.us = 1e30;
  const int nch = chunks(p);
  for (int nt = turns ? 2 : 4; nt >= 1; nt /= 2)
    for (int mt = 1; mt <= (turns ? 1 : 2); ++mt) {
      if (mt == 2 && d.Cout <= 16) continue;
      // the tile with the fewest workgroups, then the smallest region
      int th = 0, tw = 0, pix = 0;
      long tiles = 0;
      for (int w = 1; w <= std::min(p->Wo, 64 * nt); ++w) {
        const int h = std::min(p->Ho, 64 * nt / w), px = region(d, h, w);
        if (lds_bytes(px) > 160 << 10) continue;
        const long n = (long)((p->Ho + h - 1) / h) * ((p->Wo + w - 1) / w);
        const double cost = n * (256. * nt + px), old = tiles * (256. * nt + pix);
        if (!tiles || cost < old) { th = h; tw = w; pix = px; tiles = n; }
      }
      if (!tiles) continue;
      const int blocks = (d.Cout + 16 * mt - 1) / (16 * mt);
      for (int wc = 1; wc <= (blocks > 1 ? 2 : 1); ++wc)
        for (int ns = 1; ns <= (may_split ? nch : 1); ++ns) {
          const int per = (nch + ns - 1) / ns;
          if ((nch + per - 1) / per != ns) continue;
          for (int os = 1; os <= (turns && may_split ? std::max(1, p->kk / 4) : 1); ++os) {
            const int oper = (p->kk / 4 + os - 1) / os;
            if (os > 1 && (p->kk / 4 + oper - 1) / oper != os) continue;
            IgShape s{mt, nt, wc, th, tw, ns, os, 0.};
            if (s.parts() > 1 && s.parts() * part + block_bytes(p, s) + 256 > budget) continue;
            const double wgs = (double)tiles * d.N * ((blocks + wc - 1) / wc) * ns * os;
            const double mfma = (turns ? (os > 1 ? 16 * oper + 2 : 4 * p->kk) : p->kk * mt) * nt * 6e-3;
            const double stage = per * (k.chunk + k.item * pix * 4 / (256. * wc));
            const int occ = std::max(1, std::min(waves_per_simd(turns ? 4 : 1, mt, nt, per > 1) / wc, (int)((160 << 10) / lds_bytes(pix))));
            auto time = [&](int n) {
              const int waves = n * wc;
              return stage + per * mfma * (waves <= 1 ? k.one : waves <= 2 ? k.two * waves : k.four * waves);
            };
            const double full = 256. * occ, rest = std::fmod(wgs, full);
            double us = std::floor(wgs / full) * time(occ) + (rest > 0 ? time((int)std::ceil(rest / 256)) : 0.) + k.start + out / k.bytes;
            if (s.parts() > 1) us += k.sum + s.parts() * (turns ? 4 : 1) * out / (turns ? 1.65e6 : 2.5e6);
            s.us = us;
            if (us < best.us) best = s;
          }
        }
    }
  return best;
}

size_t ig_fwd_block_bytes(const rotconv_plan* p, const IgShape& s) { return block_bytes(p, s); }
size_t ig_fwd_pack_bytes(const rotconv_plan* p, const IgShape& s) { return filter_blocks(p, s) * block_bytes(p, s); }

void launch_ig_fwd(const rotconv_plan* p, const IgShape& s, bool pooled, const float* x, const float* w, float* y, uint8_t* idx,
                   void* ws, size_t ws_bytes, hipStream_t st) {
  const rotconv_desc& d = p->d;
  const bool turns = four_turns(p);
  IgGeom g{};
  g.Cin = d.Cin; g.H = d.H; g.W = d.W; g.Cout = d.Cout; g.k = d.k; g.kk = p->kk; g.stride = d.stride; g.pad = d.pad;
  g.Ho = p->Ho; g.Wo = p->Wo; g.relu = pooled && d.activation == ROTCONV_ACT_RELU;
  g.th = s.th; g.tw = s.tw; g.nty = (p->Ho + s.th - 1) / s.th; g.ntx = (p->Wo + s.tw - 1) / s.tw;
  g.rw = (s.tw - 1) * d.stride + d.k; g.npix = region(d, s.th, s.tw);
  g.mrw = ((1u << 22) + g.rw - 1) / g.rw;
  g.nch = chunks(p); g.per = (g.nch + s.nsplit - 1) / s.nsplit;
  g.osplit = s.osplit; g.oper = (g.kk / 4 + s.osplit - 1) / s.osplit;
  g.xbytes = (uint32_t)(4.0 * d.Cin * d.H * d.W);
  g.part = (size_t)d.N * d.Cout * d.R * p->Ho * p->Wo;
  const size_t lds = lds_bytes(g.npix);
  const int blocks = filter_blocks(p, s);
  int most = (int)std::min<size_t>(blocks, ws_bytes / block_bytes(p, s));      // (the caller sees to one)
  if (most < 1) return;
  if (most < blocks && most > 1) most -= most % s.wc;
  for (int b = 0; b < blocks; b += most) {
    g.cb0 = b; g.ncb = std::min(most, blocks - b);
    const unsigned pb = (unsigned)(g.ncb * g.nch * s.mt);
    hipLaunchKernelGGL(k_ig_pack, dim3(pb, std::max(1u, std::min((unsigned)g.kk, 1024u / pb))), dim3(256), 0, st, w,
                       static_cast<uint32_t*>(ws), turns ? 1 : 0, s.mt, b, d.Cout, d.Cin, d.k, g.nch);
    auto go = [&](auto kern) {
      if (lds > 64 << 10) (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
      hipLaunchKernelGGL(kern, dim3((unsigned)((g.ncb + s.wc - 1) / s.wc * g.nty * g.ntx * d.N), (unsigned)((g.nch + g.per - 1) / g.per * g.osplit)),
                         dim3(256 * s.wc), lds, st, x,
                         static_cast<const u32x4*>(ws), w, y, idx, g);
    };
    using std::integral_constant;
    const auto i1 = integral_constant<int, 1>{};
    const auto i2 = integral_constant<int, 2>{};
    const auto i4 = integral_constant<int, 4>{};
    auto with = [&](auto S, auto mt, auto nt, auto wc, auto pool) {
      if (g.per > 1) go(k_ig_fwd<decltype(S)::value, decltype(mt)::value, decltype(nt)::value, decltype(wc)::value, decltype(pool)::value, true>);
      else go(k_ig_fwd<decltype(S)::value, decltype(mt)::value, decltype(nt)::value, decltype(wc)::value, decltype(pool)::value, false>);
    };
    auto by_wc = [&](auto S, auto mt, auto nt, auto pool) {
      if (s.wc == 2) with(S, mt, nt, i2, pool); else with(S, mt, nt, i1, pool);
    };
    auto by_nt = [&](auto mt, auto pool) {
      if (s.nt == 4) by_wc(i1, mt, i4, pool);
      else if (s.nt == 2) by_wc(i1, mt, i2, pool);
      else by_wc(i1, mt, i1, pool);
    };
    auto by_mt = [&](auto pool) {
      if (s.mt == 2) by_nt(i2, pool); else by_nt(i1, pool);
    };
    if (turns) {
      auto by_pool = [&](auto nt) {
        if (pooled) by_wc(i4, i1, nt, std::true_type{}); else by_wc(i4, i1, nt, std::false_type{});
      };
      if (s.nt == 2) by_pool(i2); else by_pool(i1);
    } else if (pooled) {
      by_mt(std::true_type{});
    } else {
      by_mt(std::false_type{});
    }
  }
}

}  // namespace rotconv
