// Fast forward kernel for 3x3, stride 1, pad 1 (fp32 tensors) on the bf16 matrix cores, operands split into three bf16
// parts (rotconv_split3.h): shared-product rotation convolution (paper Eq. 8), fused with the orientation max-pool (Eq. 10).
//
// For one first-quadrant bank the nine per-tap channel contractions
//     P_u[co, h, x] = sum_ci F[co,ci,u] * X[ci,h,x]           (u = base tap)
// are formed ONCE and placed at the four quarter-turn positions
//     Y_s[co, y, x] = sum_u P_u[co, y + i_s(u) - 1, x + j_s(u) - 1],  (i_s,j_s) = R_s(u)
// in registers; the maximum over the rotations and its arg-max are stored once.
//
// M = 16 filters, N = 16 pixels, K = 32 channels, two tiles of pixels: a lane owns the pixel pair (2 lc, 2 lc + 1) of 32
// consecutive columns and four filters.  The neighbour columns are the lane's own other pixel or the next lane's, which the
// placement's additions read through lane shifts, so a wave needs nothing of another wave: no exchange, no barrier, and the
// two waves of a SIMD drift apart until one places its products while the other multiplies.  (With the columns of a row
// chained over the waves of a workgroup, edges exchanged through LDS and a barrier per row, matrix and vector work added
// up.)  The inner 30 of a wave's 32 columns are outputs.
//
// The rows of a band (TY output rows) of all bands and images are laid end to end, each followed by one or two empty
// columns (Wv in all, even, so that a pixel pair never spans two rows): a wave takes 32 consecutive columns of that line,
// whatever W is, and walks down its TY + 2 rows.  Loads go through a buffer descriptor; positions outside the image get an
// offset beyond it and read as zero, stores to such positions are dropped.
//
// What bounds it: 108 matrix instructions (16 clk) per 32-channel chunk, row and wave, beside 88 vector instructions that
// split the pixels, 72 that add up the chunks and 420 per row that place and pool; about 16 ns per matrix instruction and
// SIMD in all, whichever loads and LDS reads come earlier (operands read a tap or two chunks ahead, fewer vector instructions:
// no change), 20 % less where the pixels are all zero: the clock under matrix and vector work together is what is left.
// Measured against rows chained over the waves of a workgroup, 256 pixels at the most, masked where W is no multiple of eight:
// 2x55 -> 213, 294x204 400 -> 181 us; 8x54 -> 92, 55x236 148 -> 77; 8x16 -> 144, 225x116 262 -> 120; 8x512 -> 512, 16x16 195 -> 109;
// 4x48 -> 384, 184x112, one orientation 330 -> 200 (a turn that the orientation set lacks is not placed); odd rows 65 -> 33 without
// the copies to padded rows (1x54 -> 117, 193x75).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "rotconv_kernels.h"
#include "rotconv_p4.h"
#include "rotconv_p4_taps.h"
#include "rotconv_split3.h"

namespace rotconv {
namespace {

typedef float f2 __attribute__((ext_vector_type(2)));
typedef float f4 __attribute__((ext_vector_type(4)));

constexpr int CHF = kS3FwdChunk;          // 4-byte words of a 32-channel chunk of a 16-filter block: [tap][part][lane][8 bf16]
constexpr int NWMAX = 8;                  // waves per workgroup at the most
constexpr int COLS = 30;                  // output columns per wave

// the value of the lane to the left / right in the row of sixteen lanes (zero beyond its ends)
__device__ __forceinline__ float from_left16(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x111, 0xf, 0xf, true));
}
__device__ __forceinline__ float from_right16(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x101, 0xf, 0xf, true));
}

// OUT:      every orientation written (rotconv_fwd, channel splits), or max + arg-max over the bank's rotations, all four of
//           which are in the orientation set or not.
// STREAM:   the filter block does not fit LDS: two 32-channel buffers, one barrier per chunk.
// NQ:       banks folded into the sixteen filters of a wave (1, 2 or 4): row m of the tile holds bank m % NQ of filter
//           m / NQ, so a lane holds all banks of its filters and pools them in registers.
// ODD:      W is odd: a pixel pair may be half outside its row and its address is not that of a pair; loads go pixel by pixel.
enum { kEvery, kMaxOfFour, kMaxOfSome };
template <int OUT, bool STREAM, int NQ, bool ODD>
__global__ __launch_bounds__(64 * NWMAX, 2) void k_s3_fwd(const float* __restrict__ x, const float* __restrict__ wt,
                                                          const int32_t* __restrict__ rot_of, float* __restrict__ out_val,
                                                          uint8_t* __restrict__ out_idx, S3FwdGeom g) {
  constexpr bool UNPOOLED = OUT == kEvery;
  extern __shared__ float smem[];
  float* Wl = smem;                      // [chunks of the part, or 2 if streamed][CHF]

  // consecutive units (same columns, different filter blocks / banks) go to the same XCD and share its L2 copy of the input
  const int per_xcd = (g.units + 7) / 8;
  int v = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
  if (v >= g.units) return;
  // Channel split (small maps with deep inputs): the workgroup contracts the chunks [c_lo, c_hi) only and writes its
  // unpooled sums into part `sp`; the parts are added in order afterwards.
  const int sp = v % g.csplit; v /= g.csplit;
  const int nchunk = g.CinPad / 32;
  const int c_lo = sp * g.cper, c_hi = min(nchunk, c_lo + g.cper);
  const int cb = v % g.CB; v /= g.CB;
  const int cbo = g.cb0 + cb;            // the block among the layer's
  const int q = v % g.Q; v /= g.Q;
  const int sg = v % g.nsg;
  const int img = v / g.nsg;             // first image of the line

  const int tid = threadIdx.x, nt = STREAM ? 64 * NWMAX : blockDim.x;
  const float* wsrc = wt + (size_t)(q * g.CB + cb) * nchunk * CHF;
  // A streamed chunk goes through registers in two halves (at most two 16-byte pieces per thread in flight): one is
  // loaded at the chunk's first tap and written at its fifth, the other from there to the chunk's end.
  constexpr int WPT = ((CHF / 4 + 64 * NWMAX - 1) / (64 * NWMAX) + 1) / 2;
  f4 wreg[STREAM ? WPT : 1];
  auto wload = [&](int c, int half) {
#pragma unroll
    for (int k = 0; k < WPT; ++k) {
      const unsigned e = threadIdx.x + (half * WPT + k) * (64 * NWMAX);
      if (e < CHF / 4) wreg[k] = reinterpret_cast<const f4*>(wsrc + (size_t)c * CHF)[e];
    }
  };
  auto wstore = [&](int buf, int half) {
#pragma unroll
    for (int k = 0; k < WPT; ++k) {
      const unsigned e = threadIdx.x + (half * WPT + k) * (64 * NWMAX);
      if (e < CHF / 4) reinterpret_cast<f4*>(Wl + buf * CHF)[e] = wreg[k];
    }
  };
  auto wstage = [&](int c, int buf) {
    for (int half = 0; half < 2; ++half) {
      wload(c, half);
      wstore(buf, half);
    }
  };

  // ---- the wave's columns --------------------------------------------------------------------------------------------
  const int wave = __builtin_amdgcn_readfirstlane(tid / 64), lane = tid % 64;
  const int lg = lane / 16, lc = lane % 16;
  const int HW = g.H * g.W;
  const int strip = sg * g.nw + wave;
  const bool live = strip < g.nstrip;
  const int v0 = strip * COLS - 2 + 2 * lc;            // the lane's first column of the line
  const int vr = v0 < 0 ? 0 : v0 / g.Wv;               // its band, counted over the images of the line
  const int px = v0 - vr * g.Wv;
  const int nl = vr / g.nband;
  const int y0 = (vr - nl * g.nband) * g.TY;
  const bool vok = v0 >= 0 && vr < g.nvr;
  const bool ok0 = vok && px < g.W, ok1 = vok && px + 1 < g.W;
  const uint32_t row4 = (uint32_t)g.W * 4u;
  const size_t ximg = (size_t)g.Cin * HW;
  const auto rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(x + (size_t)img * ximg), 0,
                                                    (int)(uint32_t)(ximg * 4 * g.line_imgs), 0x27000);
  const uint32_t xo = (((uint32_t)nl * (uint32_t)g.Cin + 8u * (uint32_t)lg) * (uint32_t)HW + (uint32_t)((y0 - 1) * g.W + px)) * 4u;

  // The load cursor runs a chunk ahead of the multiplication: chunk cl of row tl.
  int tl = 0, cl = c_lo;
  uint32_t vx0 = kOutside, vx1 = kOutside;             // the lane's pixels in row tl of channel 8 lg
  auto set_row = [&]() {
    const bool rok = (unsigned)(y0 - 1 + tl) < (unsigned)g.H;
    const uint32_t o = xo + (uint32_t)tl * row4;
    vx0 = rok && ok0 ? o : kOutside;
    if (ODD) vx1 = rok && ok1 ? o + 4u : kOutside;
  };
  auto advance = [&]() {
    if (++cl == c_hi) {
      cl = c_lo;
      ++tl;
      set_row();
    }
  };
  f2 raw[8];                                           // eight channels of the pixel pair
  auto load_at = [&](int k, uint32_t o0, uint32_t o1) {
    const uint32_t so = (uint32_t)(cl * 32 + k) * (uint32_t)HW * 4u;
    if (ODD) {
      raw[k].x = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rx, o0, so, 0));
      raw[k].y = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rx, o1, so, 0));
    } else {
      raw[k] = __builtin_bit_cast(f2, __builtin_amdgcn_raw_buffer_load_b64(rx, o0, so, 0));
    }
  };
  auto load = [&]() {
    if (cl * 32 + 32 <= g.Cin) {
#pragma unroll
      for (int k = 0; k < 8; ++k) load_at(k, vx0, vx1);
    } else {                                           // channels beyond Cin read as zero
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const bool in = cl * 32 + 8 * lg + k < g.Cin;
        load_at(k, in ? vx0 : kOutside, in ? vx1 : kOutside);
      }
    }
    advance();
  };
  set_row();
  if (live) {
    load();
  }

  // ---- the filter block -----------------------------------------------------------------------------------------------
  if (STREAM) {
    wstage(c_lo, 0);
  } else if (g.raw_w) {
    // wt is the caller's w[Cout][Cin][9]; zeros beyond Cout / Cin.  A thread splits three taps of two channels of a filter.
    const int n = (c_hi - c_lo) * 768;
    uint32_t* Wu = reinterpret_cast<uint32_t*>(Wl);
    for (int i = tid; i < n; i += nt) {
      const int u0 = i / 256 % 3 * 3, e = i % 256, c = i / 768;
      const int f = (e / 4) % 16, ci = (c_lo + c) * 32 + (e / 64) * 8 + (e % 4) * 2;
      const bool okf = cbo * 16 + f < g.Cout, in0 = okf && ci < g.Cin, in1 = okf && ci + 1 < g.Cin;
      const float* w0 = wt + ((size_t)(in0 ? cbo * 16 + f : 0) * g.Cin + (in0 ? ci : 0)) * 9 + u0;
      float a0[3], a1[3];
#pragma unroll
      for (int u = 0; u < 3; ++u) { a0[u] = in0 ? w0[u] : 0.f; a1[u] = in1 ? w0[9 + u] : 0.f; }
      uint32_t* dst = Wu + c * CHF + u0 * 768 + e;
#pragma unroll
      for (int u = 0; u < 3; ++u) {
        uint16_t a[3], b[3];
        s3_split_weight(a0[u], a[0], a[1], a[2]);
        s3_split_weight(a1[u], b[0], b[1], b[2]);
        const uint32_t sgn = s3_tap_turned(u0 + u) ? 0x80008000u : 0u;
#pragma unroll
        for (int k = 0; k < 3; ++k) dst[(u * 3 + k) * 256] = ((uint32_t)a[k] | (uint32_t)b[k] << 16) ^ sgn;
      }
    }
  } else {
    const f4* src = reinterpret_cast<const f4*>(wsrc + (size_t)c_lo * CHF);
    f4* dst = reinterpret_cast<f4*>(Wl);
    const int n4 = (c_hi - c_lo) * (CHF / 4);
    for (int i = tid; i < n4; i += nt) dst[i] = src[i];
  }
  __syncthreads();
  if (!STREAM && !live) return;                        // no barrier from here on
  const int nsteps = g.TY + 2;
  if (STREAM && !live) {                               // beyond the line: only the workgroup's stages and barriers
    int seq = 0;
    for (int t = 0; t < nsteps; ++t)
      for (int c = c_lo; c < c_hi; ++c) {
        wstage(c + 1 == c_hi ? c_lo : c + 1, (seq + 1) & 1);
        __syncthreads();
        ++seq;
      }
    return;
  }

  // ---- outputs --------------------------------------------------------------------------------------------------------
  constexpr int FPB = 16 / NQ;                         // filters per wave
  constexpr int FPL = 4 / NQ;                          // filters per lane
  int rot[NQ][4];
#pragma unroll
  for (int b = 0; b < NQ; ++b)
#pragma unroll
    for (int s = 0; s < 4; ++s) rot[b][s] = rot_of[(NQ > 1 ? b : q) * 4 + s];
  uint32_t rots[NQ];                                   // the bank's orientations, a byte each
#pragma unroll
  for (int b = 0; b < NQ; ++b)
    rots[b] = (uint32_t)(rot[b][0] & 255) | (uint32_t)(rot[b][1] & 255) << 8 | (uint32_t)(rot[b][2] & 255) << 16 | (uint32_t)(rot[b][3] & 255) << 24;
  const float floor_at = g.relu ? 0.f : __builtin_nanf("");      // no value is at or below a NaN
  int grp = 0;                                         // the bank's pool group
  if (!UNPOOLED && NQ == 1 && g.out_mode == kOutPooled) {
#pragma unroll
    for (int s = 3; s >= 0; --s) grp = rot[0][s] >= 0 ? rot[0][s] : grp;
    grp %= g.ng;
  }
  const int co0 = cbo * FPB + lg * FPL;                // the lane's first filter
  // planes between filters, and what lies in front of the line's first image
  const uint32_t fplanes = UNPOOLED ? g.R : g.out_mode == kOutPooled ? g.ng : 1;
  const size_t oimg = (size_t)g.Cout * fplanes * HW;
  const size_t obase = ((UNPOOLED ? (size_t)sp : g.out_mode == kOutPartial ? (size_t)q : 0) * g.N + img) * oimg;
  const uint32_t osize = (uint32_t)(oimg * g.line_imgs);
  const auto ro = __builtin_amdgcn_make_buffer_rsrc(out_val + obase, 0, (int)(osize * 4u), 0x27000);
  const auto ri = __builtin_amdgcn_make_buffer_rsrc(out_idx + (UNPOOLED ? 0 : obase), 0, (int)(UNPOOLED ? 0 : osize), 0x27000);
  const uint32_t fstep = fplanes * (uint32_t)HW;       // elements from a filter to the next
  const uint32_t oo = ((uint32_t)nl * (uint32_t)g.Cout + (uint32_t)co0) * fstep + (uint32_t)(grp * HW) + (uint32_t)((y0 - 2) * g.W + px);
  const int nf = max(0, min(FPL, g.Cout - co0));       // filters of the lane that exist
  const bool st0 = ok0 && lc > 0, st1 = ok1 && lc < 15;

  float accA[4][4][2], accB[4][4][2];                  // [turn][row of the tile][pixel]: rolling sums of two output rows
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int b = 0; b < 2; ++b) { accA[s][r][b] = 0.f; accB[s][r][b] = 0.f; }

  // ---- operands -------------------------------------------------------------------------------------------------------
  f4 P[9][2];
  int seq = 0;
  const u32x4* wl = reinterpret_cast<const u32x4*>(Wl) + lane;
  auto step = [&](auto first_c, int c) {
    constexpr bool first = decltype(first_c)::value;
    if (STREAM) asm volatile("" : "+s"(c));      // opaque: addresses are formed where they are used, not kept per chunk
    const int cn = c + 1 == c_hi ? c_lo : c + 1;
    if (STREAM) wload(cn, 0);
    const u32x4* wc = wl + (STREAM ? (seq & 1) : c - c_lo) * (CHF / 4);
    u32x4 wv[2][3];                                          // the weights' parts, read a tap ahead
#pragma unroll
    for (int e = 0; e < 3; ++e) wv[0][e] = wc[e * 64];
    u32x4 ap[2][3];                                          // [pixel of the pair][part]
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        const S3Pair s = s3_split2(raw[2 * i][b], raw[2 * i + 1][b]);
#pragma unroll
        for (int e = 0; e < 3; ++e) ap[b][e][i] = s.p[e];
      }
    load();
#pragma unroll
    for (int u = 0; u < 9; ++u) {
      const u32x4 (&w)[3] = wv[u & 1];
      if (u + 1 < 9) {
#pragma unroll
        for (int e = 0; e < 3; ++e) wv[(u + 1) & 1][e] = wc[((u + 1) * 3 + e) * 64];
      }
      __builtin_amdgcn_sched_barrier(0);
      // the smallest products first, their sum from zero: only the chunk's total meets the running sum
      f4 s[2];
      auto product = [&](int we, int ae) {
#pragma unroll
        for (int b = 0; b < 2; ++b) s[b] = s3_mfma(w[we], ap[b][ae], s[b]);
      };
      s[0] = s[1] = f4{0.f, 0.f, 0.f, 0.f};
      product(2, 0);
      product(0, 2);
      product(1, 1);
      product(1, 0);
      product(0, 1);
      product(0, 0);
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        if (first) P[u][b] = s[b];
        else P[u][b] += s[b];
        asm volatile("" : "+v"(P[u][b]));        // here and not later: eighteen such sums at once do not fit the registers
      }
      if (STREAM && u == 4) {
        wstore((seq + 1) & 1, 0);
        wload(cn, 1);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    if (STREAM) {
      wstore((seq + 1) & 1, 1);
      __syncthreads();
    }
    ++seq;
  };

  const bool bad_column = __any(!ok0 || !ok1);
  bool dirty = false;                                  // do empty columns have products (weights that are not finite)?

  for (int t = 0; t < nsteps; ++t) {
    // the matrix work of one wave of a SIMD ahead of the placement of the other
    if (!UNPOOLED) __builtin_amdgcn_s_setprio(2);
    step(std::true_type{}, c_lo);
    for (int c = c_lo + 1; c < c_hi; ++c) step(std::false_type{}, c);
    if (!UNPOOLED) __builtin_amdgcn_s_setprio(0);
    // Positions outside the image were multiplied as zeros.  Their products are zeros too, but for weights that are not
    // finite: those reach no output through the padding, as everywhere in this library.
    const int h = y0 - 1 + t;
    const bool row_bad = (unsigned)h >= (unsigned)g.H;
    if ((t == 0 && bad_column) || dirty || __any(row_bad)) {
      const bool z0 = row_bad || !ok0, z1 = row_bad || !ok1;
      uint32_t left = 0;
#pragma unroll
      for (int u = 0; u < 9; ++u)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float p0 = P[u][0][r], p1 = P[u][1][r];      // copies: a bit cast of a vector's element takes the first one
          left |= (z0 ? __builtin_bit_cast(uint32_t, p0) : 0u) | (z1 ? __builtin_bit_cast(uint32_t, p1) : 0u);
          P[u][0][r] = z0 ? 0.f : p0;
          P[u][1][r] = z1 ? 0.f : p1;
        }
      dirty = dirty || __any((left & 0x7fffffffu) != 0);
    }

    // ---- place the row of products at the rotated positions (Eq. 8) --------------------------------------------------
    auto place = [&](int s, int r, int b) -> float {
      // three taps per filter row; a sum starts from its own columns' products (the shifted one folds into its addition)
      // and from one that is not turned
      float tr[3] = {0.f, 0.f, 0.f};
      bool begun[3] = {false, false, false};
#pragma unroll
      for (int pass = 0; pass < 3; ++pass)
#pragma unroll
        for (int u = 0; u < 9; ++u) {
          const int j = b + tap_j(s, u) - 1, ti = tap_i(s, u);
          const bool shifted = j < 0 || j > 1;
          if (pass != (shifted ? 2 : s3_tap_turned(u) ? 1 : 0)) continue;
          const float val = j < 0 ? from_left16(P[u][1][r]) : j > 1 ? from_right16(P[u][0][r]) : P[u][j][r];
          tr[ti] = !begun[ti] ? val : s3_tap_turned(u) ? tr[ti] - val : tr[ti] + val;
          begun[ti] = true;
        }
      float y = accA[s][r][b] + tr[2];                 // rows h-2, h-1, h are in: output row h-1 done
      accA[s][r][b] = accB[s][r][b] + tr[1];           // output row h has rows h-1, h
      asm("" : "+v"(y), "+v"(accA[s][r][b]), "+v"(tr[0]));      // in this order: accB's register is free for tr[0]
      accB[s][r][b] = tr[0];                           // output row h+1 has row h
      return y;
    };
    const bool fin = t >= 2 && h - 1 < g.H;
    const uint32_t oe = oo + (uint32_t)(t * g.W);
    const uint32_t e0 = fin && st0 ? oe * 4u : kOutside, e1 = fin && st1 ? oe * 4u + 4u : kOutside;
    if constexpr (UNPOOLED) {
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        if (rot[0][s] < 0) continue;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const uint32_t so = ((uint32_t)r * fstep + (uint32_t)rot[0][s] * (uint32_t)HW) * 4u;
          const float ya = place(s, r, 0), yb = place(s, r, 1);
          __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, ya), ro, r < nf ? e0 : kOutside, so, 0);
          __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, yb), ro, r < nf ? e1 : kOutside, so, 0);
        }
      }
    } else {
#pragma unroll
      for (int r = 0; r < 4; r += NQ) {
        const int f = r / NQ;
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          float bv = 0.f;
          uint32_t bi = 0;
#pragma unroll
          for (int bank = 0; bank < NQ; ++bank) {
            float cv = 0.f;
            uint32_t ci = 0;                           // eight times the turn: where its orientation sits in rots
            if constexpr (OUT == kMaxOfFour) {
#pragma unroll
              for (int s = 0; s < 4; ++s) {
                const float y = place(s, r + bank, b);
                const bool gt = s == 0 || y > cv;
                cv = gt ? y : cv;
                ci = gt ? 8u * s : ci;
              }
            } else {
              bool have = false;
#pragma unroll
              for (int s = 0; s < 4; ++s) {
                const float y = place(s, r + bank, b);
                const bool gt = rot[bank][s] >= 0 && (!have || y > cv);
                cv = gt ? y : cv;
                ci = gt ? 8u * s : ci;
                have = have || rot[bank][s] >= 0;
              }
            }
            ci = rots[bank] >> ci;
            if (NQ > 1) {                              // across the banks: ties go to the smallest orientation index
              ci &= 255u;
              const bool take = bank == 0 || cv > bv || (cv == bv && ci < bi);
              bv = take ? cv : bv;
              bi = take ? ci : bi;
            } else {
              bv = cv;
              bi = ci;
            }
          }
          const bool dead = bv <= floor_at;            // fused ReLU: dead elements get idx 255; a NaN stays one
          bv = dead ? 0.f : bv;
          bi = dead ? 255u : bi;
          const uint32_t e = f < nf ? (b ? e1 : e0) : kOutside;
          __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, bv), ro, e, (uint32_t)f * fstep * 4u, 0);
          __builtin_amdgcn_raw_buffer_store_b8((uint8_t)bi, ri, e >> 2, (uint32_t)f * fstep, 0);
        }
      }
    }
  }
}

template <int OUT, int NQ>
void launch_u(const S3FwdGeom& g, const float* x, const float* wt, const int32_t* rot_of, float* ov, uint8_t* oi, hipStream_t st) {
  const size_t lds = (size_t)(g.stream ? 2 : g.cper) * CHF * sizeof(float);
  auto go = [&](auto kern) {
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL(kern, dim3((g.units + 7) / 8 * 8), dim3(64 * g.nw), lds, st, x, wt, rot_of, ov, oi, g);
  };
  if constexpr (NQ == 1) {      // banks are folded on even rows only (p4_fwd_fold)
    if (g.W & 1) {
      if (g.stream) go(k_s3_fwd<OUT, true, 1, true>); else go(k_s3_fwd<OUT, false, 1, true>);
      return;
    }
  }
  if (g.stream) go(k_s3_fwd<OUT, true, NQ, false>); else go(k_s3_fwd<OUT, false, NQ, false>);
}

// A tensor that a buffer descriptor reaches, with kOutside beyond it.
constexpr double kReach = 4294967264.0;

}  // namespace

// An image of the input and of the output each within a 32-bit byte offset.
bool s3_fwd_supported(const rotconv_plan* p) {
  const double hw4 = 4.0 * p->d.H * p->d.W;
  return hw4 * p->d.Cin <= kReach && hw4 * p->d.Cout * p->d.R <= kReach;
}

// The launch of an output mode, a channel split and a number of folded banks.
S3FwdGeom s3_fwd_geom(const rotconv_plan* p, int out_mode, int csplit, int nq, int given_ty, int given_nw) {
  const rotconv_desc& d = p->d;
  S3FwdGeom g{};
  g.N = d.N; g.Cin = d.Cin; g.CinPad = (d.Cin + 31) / 32 * 32; g.H = d.H; g.W = d.W; g.Cout = d.Cout; g.R = d.R;
  g.ng = p->ng; g.out_mode = out_mode; g.nq = nq;
  const int nchunk = g.CinPad / 32;
  g.cper = (nchunk + csplit - 1) / csplit;
  g.csplit = (nchunk + g.cper - 1) / g.cper;
  g.stream = g.cper > kS3FwdResident;
  g.Q = nq > 1 ? 1 : p->host.Q;
  g.CB = nq > 1 ? (d.Cout * nq + 15) / 16 : (d.Cout + 15) / 16;
  g.relu = out_mode == kOutPooled && d.activation == ROTCONV_ACT_RELU;
  g.all_turns = 1;
  for (int i = 0; i < p->host.Q * 4; ++i) g.all_turns &= p->rot_of[i] >= 0;
  const int sep = d.W & 1 ? 1 : 2;
  g.Wv = d.W + sep;
  // all images on one line where descriptors of the whole tensors reach
  const double hw4 = 4.0 * d.H * d.W * d.N;
  const double planes = out_mode == kOutUnpooled ? d.R : out_mode == kOutPooled ? p->ng : 1;
  g.line_imgs = hw4 * d.Cin <= kReach && hw4 * d.Cout * planes <= kReach ? d.N : 1;
  // Rows per band and waves per workgroup.  Short bands cost halo rows (a band of TY rows multiplies TY + 2) but give more
  // workgroups.  In units of 0.1 us, as measured on 130 layers (within a fifth on all but a few): a row of two waves that share
  // a SIMD 26.8 per 32-channel chunk and 13 for the placement and pooling of four turns (3 a turn unpooled), of a wave alone
  // 0.68 of that; the filter block and the launch's start 45 and 8 per chunk.
  int turns = 0;
  for (int i = 0; i < p->host.Q * 4; ++i) turns += p->rot_of[i] >= 0;
  const double placing = out_mode == kOutUnpooled ? 1. + 3. * turns / p->host.Q : 13.;
  double best = -1.;
  for (int nw : {8, 4}) {
    if (given_nw ? nw != given_nw : g.stream && nw != 8) continue;
    const int share = nw == 4 && g.cper <= 2 ? 2 : 1;            // workgroups per CU
    for (int nband = given_ty ? (d.H + given_ty - 1) / given_ty : (d.H + 127) / 128; nband <= d.H;) {
      const int ty = (d.H + nband - 1) / nband;
      const long nvr = (long)g.line_imgs * nband;
      const long nstrip = (nvr * g.Wv - sep) / COLS + 1;
      const long nsg = (nstrip + nw - 1) / nw;
      const long units = nsg * (d.N / g.line_imgs) * g.Q * g.CB * g.csplit;
      const double row = (ty + 2) * (26.8 * g.cper + placing), start = 45. + 8. * g.cper, one = 0.68 * row + start, two = row + start;
      double cost;
      if (share == 2) cost = units / 512 * two + (units % 512 == 0 ? 0. : units % 512 <= 256 ? one : two);
      else cost = (units + 255) / 256 * (nw == 8 && nstrip > 4 ? two : one);
      if (nvr * g.Wv <= (1L << 30) && units <= (1L << 30) && (best < 0. || cost < best)) {
        best = cost;
        g.nw = nw; g.TY = ty; g.nband = nband; g.nvr = (int)nvr; g.nstrip = (int)nstrip; g.nsg = (int)nsg; g.units = (int)units;
      }
      if (ty == 1 || given_ty) break;
      nband = (d.H + ty - 2) / (ty - 1);                         // the fewest bands of fewer rows
    }
  }
  g.cost = best;
  return g;
}

void launch_s3_fwd(const S3FwdGeom& g, const float* x, const float* wt, const int32_t* rot_of, float* out_val, uint8_t* out_idx,
                   hipStream_t st) {
  if (g.out_mode == kOutUnpooled) launch_u<kEvery, 1>(g, x, wt, rot_of, out_val, out_idx, st);
  else if (g.nq == 4) launch_u<kMaxOfFour, 4>(g, x, wt, rot_of, out_val, out_idx, st);      // folded: all four, see p4_fwd_fold
  else if (g.nq == 2) launch_u<kMaxOfFour, 2>(g, x, wt, rot_of, out_val, out_idx, st);
  else if (g.all_turns) launch_u<kMaxOfFour, 1>(g, x, wt, rot_of, out_val, out_idx, st);
  else launch_u<kMaxOfSome, 1>(g, x, wt, rot_of, out_val, out_idx, st);
}

}  // namespace rotconv
