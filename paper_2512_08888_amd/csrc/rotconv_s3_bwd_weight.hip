// Fast weight-gradient kernel for 3x3, stride 1, pad 1 (fp32 tensors), fused with the orientation max-pool backward
// (paper Eq. 12, 14, 16 in shared-product form), on the bf16 matrix cores with operands split into three bf16 parts
// (rotconv_split3.h); layers with more than 16 input channels.
//
//   dF_q[co,ci,u] = sum_{n,h,x} D^q_u[co,h,x] * X[ci,h,x]
//   D^q_u[co,h,x] = sum_s Delta_(q,s)[co, h+1-i_s(u), x+1-j_s(u)],   Delta_r = G * 1[idx == r]
//
// A workgroup owns 32 filters of a bank x 32 CB input channels x nine taps and walks down the rows of its strips of
// sixteen pixels, two rows (32 pixels) a step.  D and its parts cost several times the vector work of anything else here
// and do not depend on the channel, so they are built once per workgroup and step and handed round through LDS: eight
// waves build (a wave four filters, a lane one pixel column of one filter: column neighbours by lane shifts; what a pair of rows
// gives to the next step's D is summed with it, so that a row is routed once), four waves split X, and all twelve multiply,
// a wave three taps of 32 channels (48 accumulator registers, so that three waves fit a SIMD and one's vector
// instructions run beside another's matrix instructions).  LDS is double-buffered, one barrier per step; half of the
// builders multiply first and build afterwards.
//
// What bounds it: with 128 channels per workgroup the matrix cores (six products: 89 us of the 118 at 4x128 -> 128,
// 128x128; fp32 matrix cores, which need 145 us for one product each, took 182), with 64 the vector work of building
// (about 740 instructions per SIMD and step beside 54 matrix instructions; 8x64 -> 64, 256x256: 309 us with the pair before
// routed again, 288 so; with 128 channels the same time either way).
// 4x512 -> 512, 32x32: 126 us, was 188; 2x256 -> 256, 32x32: 39, was 47; 8x512 -> 512, 16x16: 79, was 196.
// Precision: the parts' sum of each 16 pixels starts from zero and only its total meets the running sum.  The matrix
// instruction cuts the low bits of what it adds up towards minus infinity; over the pixels of a batch that offset grows
// with their number while the sum itself grows with its root (8x64 -> 64, 256x256: 1.7e-6 of the norm).  So every
// other split multiplies -X and turns its sums over at the end: the offsets cancel (2.3e-7, where fp32 matrix cores left
// 3.9e-7).  (What the six products leave out has no sign of its own: both operands' parts are rounded.)
//
// M = 32 filters, N = 32 channels, K = 16 pixels: k = 8 (l / 32) + 2 p + r is row h + r, pixel 8 ph + 4 (l / 32) + p.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "rotconv_kernels.h"
#include "rotconv_p4.h"
#include "rotconv_p4_taps.h"
#include "rotconv_split3.h"

namespace rotconv {
namespace {

constexpr int NWV = 12, NTW = 64 * NWV;

// the value of the pixel to the left / right of the lane's; the first / last lane of a 16-lane row keeps `edge`
__device__ __forceinline__ float row_left(float edge, float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, edge), __builtin_bit_cast(int, v), 0x111, 0xf, 0xf, false));
}
__device__ __forceinline__ float row_right(float edge, float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, edge), __builtin_bit_cast(int, v), 0x101, 0xf, 0xf, false));
}

// RAGGED: W % 4 != 0, X is loaded pixel by pixel (a branch instead made the other rows 15 us slower: 8x64 -> 64, 256x256).
template <int CB, bool RAGGED>
__global__ __launch_bounds__(NTW, 3) void k_s3_bwd_weight(const float* __restrict__ x, const float* __restrict__ gpool,
                                                          const uint8_t* __restrict__ idx, const int32_t* __restrict__ rot_of,
                                                          float* __restrict__ partial, P4BwdWGeom g) {
  constexpr int PH = CB == 4 ? 1 : 2;         // waves that share a (taps, channels) tile, one per half of the pixels
  constexpr int NPH = 2 / PH;                 // pixel halves of a wave
  constexpr int DW = 2 * 27 * 256;            // words of one D buffer: [half of the pixels][tap][part][lane][4]
  constexpr int XW = CB * 2 * 3 * 256;
  constexpr int NR = 12;                      // the routed gradient per quarter turn: the lane's pixel and its two neighbours
  extern __shared__ uint32_t sm[];
  uint32_t* Dl = sm;                          // [2][DW]
  uint32_t* Xl = sm + 2 * DW;                 // [2][XW]: [channel block][half][part][lane][4]
  const int per_xcd = gridDim.x / 8;
  int v = gridDim.x % 8 == 0 ? (blockIdx.x % 8) * per_xcd + blockIdx.x / 8 : blockIdx.x;
  const int cg = v % g.ncig; v /= g.ncig;
  const int fb = v % g.ncog;                  // (bank, 32-filter block)
  const int split = v / g.ncog, nsplit = g.splits;

  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid / 64), lane = tid % 64;
  const int half = lane / 32, l31 = lane % 32;
  const int HW = g.H * g.W;
  const int nfb = g.CoutPad / 32;
  const int q = fb / nfb, f0 = (fb % nfb) * 32;
  const int tg = wave % 3, rest = wave / 3;
  const int cb = CB == 4 ? rest : rest % 2, ph0 = CB == 4 ? 0 : rest / 2;

  // Slots: a unit is (image, row range [h0, h1), strip of sixteen pixels); its slot j brings the pair of rows h0 + 2j - 1,
  // h0 + 2j, and from j = 1 on the output rows h0 + 2j - 2, h0 + 2j - 1 are built from its pair and the one before.  What a
  // unit stands for is worked out once, when it begins.
  struct Slot { int unit, j, h0, h1, px0, n; };
  auto begin = [&](int u) {
    const int rng = u / g.nstrip, n = rng / g.nrange, h0 = (rng - n * g.nrange) * g.rows_per;
    return Slot{u, 0, h0, min(g.H, h0 + g.rows_per), (u - rng * g.nstrip) * 16, n};
  };
  auto advance = [&](Slot& s) {
    if (s.h0 + 2 * s.j < s.h1) ++s.j;
    else s = begin(s.unit + nsplit);
  };
  auto live = [&](const Slot& s) { return s.unit < g.units; };

  const float sign = split % 2 ? -1.f : 1.f;  // of X: see above

  // ---- builders (waves 0 .. 7): filter f0 + bf, pixel column bc of the strip
  const int bf = wave * 4 + lane / 16, bc = lane % 16;
  int rot[4];
  int grp = 0;
#pragma unroll
  for (int s = 3; s >= 0; --s) {
    rot[s] = rot_of[q * 4 + s];                // -1 (absent) matches no byte
    if (rot[s] >= 0) grp = rot[s] % g.ng;
  }
  const size_t gimg = (size_t)g.Cout * g.ng * HW, ximg = (size_t)g.Cin * HW;
  const bool fok = f0 + bf < g.Cout;
  const int edge_row = bc == 1 || bc == 14 ? 1 : 0, edge_col = bc < 8 ? -1 : 16;
  const bool edge_lane = bc < 2 || bc > 13;
  const uint32_t gplane = (uint32_t)((fok ? f0 + bf : 0) * g.ng + grp) * (uint32_t)HW;
  // A pair of rows of the lane's filter: its pixel on both, and one pixel beyond the strip: lanes 0 / 15 of a 16-lane row
  // the left / right one of the first row, lanes 1 / 14 those of the second.
  struct Raw { float g, ge; uint32_t i, ie; };
  struct Pair { float g[2], ge; uint32_t i[2], ie; };
  auto load_pair = [&](const Slot& s, Pair& k) {
    const int n = live(s) ? s.n : 0, h = s.h0 + 2 * s.j - 1;
    const auto rg = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(gpool + (size_t)n * gimg), 0, (int)(uint32_t)(gimg * 4), 0x27000);
    const auto ri = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(idx + (size_t)n * gimg), 0, (int)(uint32_t)gimg, 0x27000);
    const int px = s.px0 + bc;
    const bool ok = fok & (px < g.W) & live(s);
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const bool in = ok & (h + r >= 0) & (h + r < g.H);
      const uint32_t o = gplane + (uint32_t)((h + r) * g.W + px);
      k.g[r] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rg, in ? o * 4u : kOutside, 0, 0));
      k.i[r] = __builtin_amdgcn_raw_buffer_load_b8(ri, in ? o : kOutside, 0, 0);
    }
    const int he = h + edge_row, pe = s.px0 + edge_col;
    const bool eok = fok & live(s) & edge_lane & (he >= 0) & (he < g.H) & (pe >= 0) & (pe < g.W);
    const uint32_t oe = gplane + (uint32_t)(he * g.W + pe);
    k.ge = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rg, eok ? oe * 4u : kOutside, 0, 0));
    k.ie = __builtin_amdgcn_raw_buffer_load_b8(ri, eok ? oe : kOutside, 0, 0);
  };
  auto edge_of = [&](int r, float v) { return r == 0 ? v : row_right(row_left(v, v), v); };
  auto raw_of = [&](const Pair& k, int r) {
    const float ie = edge_of(r, __builtin_bit_cast(float, k.ie));
    return Raw{k.g[r], edge_of(r, k.ge), k.i[r], __builtin_bit_cast(uint32_t, ie)};
  };
  auto route = [&](const Raw& r, float (&m)[NR]) {      // [.][0] own, [.][1] left, [.][2] right
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const float a = r.i == (uint32_t)rot[s] ? r.g : 0.f, e = r.ie == (uint32_t)rot[s] ? r.ge : 0.f;
      m[s * 3] = a; m[s * 3 + 1] = row_left(e, a); m[s * 3 + 2] = row_right(e, a);
    }
  };
  // What one row adds to the D of an output row; d: it is the row above (0), the row itself (1) or the row below (2)
  auto add_row = [&](const float (&m)[NR], int d, float (&D)[9]) {
#pragma unroll
    for (int u = 0; u < 9; ++u)
#pragma unroll
      for (int s = 0; s < 4; ++s)
        if (2 - tap_i(s, u) == d) {              // row h + 1 - i, column + 1 - j
          const int w = tap_j(s, u) == 1 ? 0 : tap_j(s, u) == 2 ? 1 : 2;
          bool begun = false;                    // an earlier row or quarter turn has started this sum
#pragma unroll
          for (int s2 = 0; s2 < 4; ++s2) begun |= 2 - tap_i(s2, u) < d || (2 - tap_i(s2, u) == d && s2 < s);
          D[u] = begun ? D[u] + m[s * 3 + w] : m[s * 3 + w];
        }
#pragma unroll
    for (int u = 0; u < 9; ++u) asm volatile("" : "+v"(D[u]));
  };
  // A wave keeps a ring of slots as loaded (a builder the pairs of rows, a wave that splits X its pixels) and loads one
  // slot before the use: a slot is 1 to 2 us of matrix work, enough to cover memory.  A longer ring does not fit the
  // registers with 128 channels and unrolls the loops towards what two CUs share of instruction cache (with 56 KB of code
  // both gradients of 8x64 -> 64, 256x256 took 690 us where 34 KB took 628).
  constexpr int NXP = CB == 4 ? 2 : 1, RING = 2, AHEAD = RING - 1;
  struct XRaw { s3_f4 v[NXP][2]; };
  // the second lane half's filters are stored in another order, so that a wave's four filters x sixteen pixels meet each
  // of the 32 banks twice and not four times
  const int bh = bc % 8 / 4;
  uint32_t* dst0 = Dl + (bc / 8) * (27 * 256) + (bh * 32 + (bf ^ (bh * 4))) * 4 + bc % 4;
  // What the pair of rows gives to the D of its slot's two output rows, which C0 and C1 begin, and then, in their place, to
  // those of the next slot: every row is routed once.
  auto build = [&](float (&C0)[9], float (&C1)[9], const Pair& now, int buf, bool store) {
    float N0[9], N1[9], m[NR];
#pragma unroll
    for (int u = 0; u < 9; ++u) N0[u] = N1[u] = 0.f;
    route(raw_of(now, 0), m);
    add_row(m, 2, C0);
    add_row(m, 1, C1);
    add_row(m, 0, N0);
    __builtin_amdgcn_sched_barrier(0);
    route(raw_of(now, 1), m);
    add_row(m, 2, C1);
    add_row(m, 1, N0);
    add_row(m, 0, N1);
    __builtin_amdgcn_sched_barrier(0);
    uint32_t* dst = dst0 + buf * DW;
    if (store) {
#pragma unroll
      for (int u = 0; u < 9; ++u) {
        const S3Pair p = s3_split2<true>(C0[u], C1[u]);
#pragma unroll
        for (int e = 0; e < 3; ++e) dst[(u * 3 + e) * 256] = p.p[e];
      }
    }
#pragma unroll
    for (int u = 0; u < 9; ++u) {
      C0[u] = N0[u];
      C1[u] = N1[u];
    }
  };

  // ---- X: channel block xcb, pixel halves xph .. ; waves 8 .. 11 split it into LDS
  const int xcb = CB == 4 ? wave - 8 : (wave - 8) % 2, xph = CB == 4 ? 0 : (wave - 8) / 2;
  const int ci = (cg * CB + max(xcb, 0)) * 32 + l31;
  const uint32_t xplane = (uint32_t)(ci < g.Cin ? ci : 0) * (uint32_t)HW;
  auto load_x = [&](const Slot& s, XRaw& k) {
    const int n = live(s) ? s.n : 0;
    const auto rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(x + (size_t)n * ximg), 0, (int)(uint32_t)(ximg * 4), 0x27000);
#pragma unroll
    for (int p = 0; p < NXP; ++p) {
      const int px = s.px0 + (xph + p) * 8 + half * 4;
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        const int h = s.h0 + 2 * s.j - 2 + r;
        const bool ok = (ci < g.Cin) & (px < g.W) & (h < s.h1) & (s.j > 0) & live(s);
        const uint32_t o = (xplane + (uint32_t)(h * g.W + px)) * 4u;
        if constexpr (RAGGED) {
#pragma unroll
          for (int i = 0; i < 4; ++i)
            k.v[p][r][i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rx, (ok & (px + i < g.W)) ? o + 4u * i : kOutside, 0, 0));
        } else {
          k.v[p][r] = __builtin_bit_cast(s3_f4, __builtin_amdgcn_raw_buffer_load_b128(rx, ok ? o : kOutside, 0, 0));
        }
      }
    }
  };
  auto split_x = [&](const XRaw& k, int p, u32x4 (&o)[3]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const S3Pair s = s3_split2_add(sign * k.v[p][0][i], sign * k.v[p][1][i]);
#pragma unroll
      for (int e = 0; e < 3; ++e) o[e][i] = s.p[e];
    }
  };
  auto stage_x = [&](const XRaw& k, int buf) {
#pragma unroll
    for (int p = 0; p < NXP; ++p) {
      u32x4 o[3];
      split_x(k, p, o);
      u32x4* dst = reinterpret_cast<u32x4*>(Xl + buf * XW) + (xcb * 2 + xph + p) * 192 + lane;
#pragma unroll
      for (int e = 0; e < 3; ++e) dst[e * 64] = o[e];
    }
  };

  s3_f16 acc[3];
#pragma unroll
  for (int j = 0; j < 3; ++j)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[j][r] = 0.f;
  auto multiply = [&](int buf) {
    const u32x4* db = reinterpret_cast<const u32x4*>(Dl + buf * DW) + ph0 * (27 * 64) + (lane ^ (half * 4));
    const u32x4* xb = reinterpret_cast<const u32x4*>(Xl + buf * XW) + (cb * 2 + ph0) * 192 + lane;
    u32x4 dv[2][3];
#pragma unroll
    for (int e = 0; e < 3; ++e) dv[0][e] = db[(tg * 9 + e) * 64];
#pragma unroll
    for (int p = 0; p < NPH; ++p) {
      u32x4 xv[3];
#pragma unroll
      for (int e = 0; e < 3; ++e) xv[e] = xb[(p * 3 + e) * 64];
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        const int k = p * 3 + j;
        if (k + 1 < 3 * NPH) {
          const int jn = (k + 1) % 3, pn = (k + 1) / 3;
#pragma unroll
          for (int e = 0; e < 3; ++e) dv[(k + 1) & 1][e] = db[pn * (27 * 64) + ((tg * 3 + jn) * 3 + e) * 64];
        }
        __builtin_amdgcn_sched_barrier(0);
        const u32x4* d = dv[k & 1];
        // the smallest products first; their sum starts from zero and is added to the running one
        s3_f16 t = s3_mfma32(d[2], xv[0], s3_f16{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f});
        t = s3_mfma32(d[0], xv[2], t);
        t = s3_mfma32(d[1], xv[1], t);
        t = s3_mfma32(d[0], xv[1], t);
        t = s3_mfma32(d[1], xv[0], t);
        t = s3_mfma32(d[0], xv[0], t);
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[j][r] += t[r];
      }
    }
  };

  // sb: the slot being built, sl: the one being loaded; what the slot before sb built is multiplied at the same time.  Each
  // kind of wave has a loop of its own (the same barriers in each).
  auto walk = [&](auto builds_c, auto late_c) {
    constexpr bool BUILDS = decltype(builds_c)::value, LATE = decltype(late_c)::value, XS = !BUILDS;
    Slot sb = begin(split), sl = sb;
    Pair kp[BUILDS ? RING : 1];
    float C0[9], C1[9];
#pragma unroll
    for (int u = 0; u < 9; ++u) C0[u] = C1[u] = 0.f;
    XRaw kx[XS ? RING : 1];
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) {
      if constexpr (BUILDS) load_pair(sl, kp[i]);
      if constexpr (XS) load_x(sl, kx[i]);
      advance(sl);
    }
    bool have = false, done = !live(sb);                  // is there something to multiply?
    int buf = 0;
    while (!done) {
#pragma unroll
      for (int at = 0; at < RING; ++at) {
        const bool now = live(sb) && sb.j > 0;
        done = !live(sb);
        if constexpr (BUILDS) load_pair(sl, kp[(at + AHEAD) % RING]);
        if constexpr (XS) load_x(sl, kx[(at + AHEAD) % RING]);
        advance(sb);
        advance(sl);
        __builtin_amdgcn_sched_barrier(0);
        if (LATE && have) multiply(buf);
        if constexpr (BUILDS) build(C0, C1, kp[at], buf ^ 1, now);      // (a unit's first slot only begins its sums)
        else if (now) stage_x(kx[at], buf ^ 1);
        if (!LATE && have) multiply(buf);
        have = now;
        if (done) break;
        __syncthreads();
        buf ^= 1;
      }
    }
  };
  if (wave < 4) walk(std::true_type{}, std::false_type{});
  else if (wave < 8) walk(std::true_type{}, std::true_type{});      // these multiply first and build afterwards
  else walk(std::false_type{}, std::false_type{});

#pragma unroll
  for (int j = 0; j < 3; ++j)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[j][r] *= sign;
  // the two waves of a tile add up their halves of the pixels
  if constexpr (PH == 2) {
    s3_f4* both = reinterpret_cast<s3_f4*>(sm) + (wave % 6) * (12 * 64) + lane;
    __syncthreads();
    if (ph0) {
#pragma unroll
      for (int i = 0; i < 12; ++i) {
        const s3_f16 a = acc[i / 4];
        const int r = i % 4 * 4;
        both[i * 64] = s3_f4{a[r], a[r + 1], a[r + 2], a[r + 3]};
      }
    }
    __syncthreads();
    if (ph0) return;
#pragma unroll
    for (int i = 0; i < 12; ++i) {
      const s3_f4 o = both[i * 64];
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[i / 4][i % 4 * 4 + r] += o[r];
    }
  }
  // partial[split][q][u][CoutPad][CinPad]; element r: filter 8 (r / 4) + 4 half + r % 4, column (channel) l31
  float* out = partial + ((size_t)split * g.Q + q) * 9 * g.CoutPad * g.CinPad;
#pragma unroll
  for (int j = 0; j < 3; ++j)
#pragma unroll
    for (int r = 0; r < 16; ++r)
      out[((size_t)(tg * 3 + j) * g.CoutPad + f0 + 8 * (r / 4) + 4 * half + r % 4) * g.CinPad + (cg * CB + cb) * 32 + l31] = acc[j][r];
}

}  // namespace

// Quarter turns only, more than sixteen channels, and an image of either operand within a 32-bit byte offset.  With sixteen
// channels or fewer three quarters of the workgroup's tiles would be padding, where k_p4_bwd_weight has blocks of sixteen:
// 1.4 times its time in the mean of 45 layers; with 17 to 32, which it pads to 64, 0.77 (2x26 -> 380, 212x100 390 -> 207 us).
// For other turns D is a sum over table entries, three times the vector work, which the matrix cores' gain does not pay for: at 4x128 -> 128, 128x128, 16 turns this split took 248 us with the table in LDS, k_p4_bwd_weight's
// table variant takes 219.
// Nor where a workgroup has a single step and the partial sums of all take longer than it: with up to 16 filters half of
// what is summed is padding, with one image row half of what is multiplied.  Graph replays of 600 layers of up to 64 rows,
// fp32 instructions / these: such layers with partial sums of more than 12 MB 0.90 of the time in the mean (5x393 -> 3, 12x20:
// 21.8 / 31.2 us; 5x415 -> 43, 1x96: 21.4 / 32.2), those of more filters and rows 1.20 (never below 0.94), with smaller partial
// sums up to 16 filters 1.08, two steps and more 1.2 to 2.7.
bool s3_bwd_weight_supported(const rotconv_plan* p) {
  const rotconv_desc& d = p->d;
  const size_t lim = (size_t)1 << 30;
  if (p4_bwd_lut(p) || p->opt.bf16_parts < 0) return false;
  const P4BwdWGeom g = s3_bwd_weight_geom(p);
  const bool one_step = g.units <= g.splits && g.rows_per <= 2;
  const bool short_sums = one_step && (d.Cout <= 16 || d.H == 1) && 36.0 * g.splits * g.Q * g.CoutPad * g.CinPad > 12e6;
  return ((d.Cin > 16 && !short_sums) || p->opt.bf16_parts > 0) && (size_t)d.Cin * d.H * d.W < lim && (size_t)d.Cout * p->ng * d.H * d.W < lim;
}

P4BwdWGeom s3_bwd_weight_geom(const rotconv_plan* p) {
  const rotconv_desc& d = p->d;
  P4BwdWGeom g{};
  g.N = d.N; g.Cin = d.Cin; g.H = d.H; g.W = d.W; g.Cout = d.Cout; g.Q = p->host.Q; g.ng = p->ng;
  g.lut = 0; g.R = d.R;
  // 32-channel blocks per workgroup.  A block of a 128-channel workgroup costs 0.24 ns a pixel (32 filters), one of a
  // 64-channel workgroup, which shares the D of half as many, 0.29: only 129 to 192 channels are cheaper as three of these
  // than as two of those.
  g.ncb = d.Cin <= 64 || (d.Cin > 128 && d.Cin <= 192) ? 2 : 4;
  g.CinPad = (d.Cin + 32 * g.ncb - 1) / (32 * g.ncb) * (32 * g.ncb);
  g.CoutPad = (d.Cout + 31) / 32 * 32;
  g.ncig = g.CinPad / (32 * g.ncb);
  g.ncog = g.Q * (g.CoutPad / 32);
  g.nstrip = (d.W + 15) / 16;
  // one workgroup per CU; a unit's rows come in pairs
  const int combos = g.ncig * g.ncog, want = std::max(1, (256 + combos / 2) / combos);
  const int strips = d.N * g.nstrip;
  // a unit has a slot for its first rows' upper neighbours: four rows a unit rather than two where that still leaves a
  // workgroup for every second CU
  const int most = strips * ((d.H + 3) / 4) * combos >= 128 ? (d.H + 3) / 4 : (d.H + 1) / 2;
  const int per_image = std::max(1, std::min(most, (want + strips - 1) / strips));
  g.rows_per = ((d.H + per_image - 1) / per_image + 1) / 2 * 2;
  g.nrange = (d.H + g.rows_per - 1) / g.rows_per;
  g.units = strips * g.nrange;
  const double per = 4.0 * g.Q * 9.0 * g.CoutPad * g.CinPad;
  g.splits = std::max(1, std::min(std::min(g.units, want), (int)(268435456.0 / per)));
  if (g.splits < 5 && g.splits % 2 && g.units > 1) ++g.splits;     // as many that multiply X as -X
  return g;
}

void launch_s3_bwd_weight(const rotconv_plan* p, const P4BwdWGeom& g, const float* x, const float* gpool, const uint8_t* idx,
                          float* partial, hipStream_t st) {
  const int grid = g.splits * g.ncig * g.ncog;
  const size_t lds = (size_t)2 * 2 * 27 * 1024 + (size_t)2 * g.ncb * 2 * 3 * 1024;
  auto go = [&](auto kern) {
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL(kern, dim3(grid), dim3(NTW), lds, st, x, gpool, idx, p->dev.rot_of, partial, g);
  };
  if (g.W & 3) {
    if (g.ncb == 4) go(k_s3_bwd_weight<4, true>); else go(k_s3_bwd_weight<2, true>);
  } else {
    if (g.ncb == 4) go(k_s3_bwd_weight<4, false>); else go(k_s3_bwd_weight<2, false>);
  }
}

}  // namespace rotconv
