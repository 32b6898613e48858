// Fast forward kernel for 3x3, stride 1, pad 1 (fp32): shared-product rotation
// convolution on the matrix cores (paper Eq. 8, re-designed for CDNA4).
//
// For one first-quadrant bank the nine per-tap channel contractions
//     P_u[co, h, x] = sum_ci F[co,ci,u] * X[ci,h,x]           (u = base tap)
// are formed ONCE (M = 16 pixels, N = 16 filters, K = 32 input channels: six
// v_mfma_f32_16x16x32_bf16 on the operands' bf16 parts, rotconv_split3.h; layers
// with at most four channels: one v_mfma_f32_16x16x4_f32) and then placed at the
// four quarter-turn positions
//     Y_s[co, y, x] = sum_u P_u[co, y + i_s(u) - 1, x + j_s(u) - 1],  (i_s,j_s) = R_s(u)
// entirely in registers: a wave owns 16 filters x 32 consecutive pixels of one
// image row and walks down the rows of its band, so a row of P feeds the output
// rows above, at and below it through two rolling partial sums per rotation;
// column shifts are register renames (each lane holds 8 consecutive pixels),
// with the one neighbouring value per side fetched from the adjacent lane group
// (ds_bpermute) or the adjacent wave (a few words of LDS per row).  The max over
// the bank's rotations and its arg-max are taken in registers and stored once.
// Nothing R-fold ever reaches memory, and the input row is read once per bank.
//
// What bounds it: 108 matrix instructions (16 clk) per 32-channel chunk, row and
// wave, and some 160 vector instructions for splitting the pixel operands and adding
// up the chunks beside about 500 per row for the placement; eight waves of a
// workgroup share a row and meet at its barrier, so the two add up.  8 x 64 -> 64
// channels at 256 x 256, four quarter turns: 0.369 ms with fp32 instructions (32 clk
// each, 288 per chunk pair and row), 0.218 ms so; 512 -> 512 at 32 x 32, batch 4:
// 0.246 -> 0.189 ms; 128 -> 128 at 128 x 128, batch 4: 0.201 -> 0.118 ms.
//
// The filter block (16 filters x all input channels x 9 taps x 3 parts) stays
// resident in LDS for the life of the workgroup when it fits (Cin <= 160; 224 with
// fp32 instructions); deeper inputs stream it through two 32-channel LDS buffers, one
// barrier per chunk.  Input rows go straight from global memory into the A-operand
// registers (8-byte loads, 128 B contiguous per 16 lanes), refilled one chunk ahead;
// scheduling fences keep those loads and the LDS reads of the B operand where
// they are issued (the compiler would otherwise sink them to their first use).
//
// Rows wider than the 256 pixels a workgroup's eight waves can chain are cut
// into segments that overlap by 8 pixels (the products of the overlap are
// recomputed, about 6 % at W = 512); a segment writes only the pixels whose
// both neighbours it holds.
//
// With bf16 parts this kernel takes rows that the chained waves cover exactly (W % 8 == 0 and a whole number of waves); other
// rows run k_s3_fwd (rotconv_s3_fwd.hip), whose waves need nothing of each other.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdlib>
#include <type_traits>

#include "rotconv_bf16.h"
#include "rotconv_expand.h"
#include "rotconv_kernels.h"
#include "rotconv_p4.h"
#include "rotconv_p4_taps.h"
#include "rotconv_split3.h"

namespace rotconv {
namespace {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef f4 f4u __attribute__((aligned(4)));      // four floats at any float's address

// KC (template parameter): K-steps (of 4 channels) per prefetch chunk: 8 (channels padded to 32), or 1 for layers
// with at most 4 input channels (a network's first layer: channels padded to 4, an eighth of the matrix work)
// S3: bf16 parts of the operands (rotconv_split3.h), KC = 8 only; else fp32 instructions
int cin_pad_f32(int Cin) { return Cin <= 4 ? 4 : (Cin + 31) / 32 * 32; }

// 4-byte words of one 32-channel chunk of a 16-filter block: parts as matrix operands, else [channel][tap][filter]
constexpr int chunk_words(int CinPad, int s3) { return s3 ? kS3FwdChunk : (CinPad == 4 ? 4 : 32) * 144; }
constexpr int max_cper(int s3) { return s3 ? kS3FwdResident : 7; }      // chunks of a block that stay in LDS

// UNPOOLED: write every orientation (rotconv_fwd); else max + arg-max over the bank's rotations.
// FASTW:    W % 8 == 0 and no wave chain reaches beyond the row: no load masks, vector stores.  With bf16 parts always
//           (other rows: rotconv_s3_fwd.hip).
// STREAM:   the filter block does not fit LDS: stream it in 32-channel chunks.
template <int NWX, int NWY, bool UNPOOLED, bool FASTW, bool STREAM, bool S3, int KC>
__global__ __launch_bounds__(64 * NWX * NWY) void k_p4_fwd(const float* __restrict__ x, const float* __restrict__ wt,
                                                           const int32_t* __restrict__ rot_of,
                                                           float* __restrict__ out_val, uint8_t* __restrict__ out_idx,
                                                           P4Geom g) {
  constexpr int NW = NWX * NWY;
  constexpr int NT = 64 * NW;
  constexpr int CHF = S3 ? kS3FwdChunk : KC * 4 * 144;      // floats of one chunk of the filter block
  extern __shared__ float smem[];
  float* Wl = smem;                      // [chunks of the part, or 2 if streamed][CHF]; a chunk: parts [tap][part][lane][8 bf16],
                                         // fp32 [channel][tap][filter]
  float* EL = smem + (STREAM ? 2 * CHF : g.cper * CHF);    // [2][NW][8][16] left-edge values of every wave
  float* ER = EL + 2 * NW * 128;         // [2][NW][8][16] right-edge values

  // XCD-aware unit decode: consecutive units (same image rows, different filter
  // blocks / banks) go to the same XCD so they share its L2 copy of the input.
  const int per_xcd = (g.units + 7) / 8;
  int v = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
  if (v >= g.units) return;
  // Channel split (small maps with deep inputs): the workgroup contracts the 32-channel chunks [c_lo, c_hi) only and
  // writes its unpooled sums into part `sp`; the parts are added in order afterwards.  Without a split: all chunks.
  const int sp = v % g.csplit; v /= g.csplit;
  const int nchunk = g.CinPad / (4 * KC);
  const int c_lo = sp * g.cper, c_hi = min(nchunk, c_lo + g.cper);
  const int cb = v % g.CB; v /= g.CB;
  const int cbo = g.cb0 + cb;            // the block among the layer's
  const int q = v % g.Q; v /= g.Q;
  const int seg = v % g.nseg; v /= g.nseg;
  const int bg = v % g.nbg;
  const int n = v / g.nbg;

  const int tid = threadIdx.x;
  const float* wsrc = wt + (size_t)(q * g.CB + cb) * nchunk * CHF;
  // A streamed chunk goes through registers in two halves (at most two 16-byte pieces per thread in flight): one is
  // loaded at the chunk's first tap and written at its fifth, the other from there to the chunk's end.
  constexpr int WPT = ((CHF / 4 + NT - 1) / NT + 1) / 2;
  f4 wreg[STREAM ? WPT : 1];
  auto wload = [&](int c, int half) {
#pragma unroll
    for (int k = 0; k < WPT; ++k) {
      const unsigned e = threadIdx.x + (half * WPT + k) * NT;
      if (e < CHF / 4) wreg[k] = reinterpret_cast<const f4*>(wsrc + (size_t)c * CHF)[e];
    }
  };
  auto wstore = [&](int buf, int half) {
#pragma unroll
    for (int k = 0; k < WPT; ++k) {
      const unsigned e = threadIdx.x + (half * WPT + k) * NT;
      if (e < CHF / 4) reinterpret_cast<f4*>(Wl + buf * CHF)[e] = wreg[k];
    }
  };
  auto wstage = [&](int c, int buf) {      // both halves at once
    for (int half = 0; half < 2; ++half) {
      wload(c, half);
      wstore(buf, half);
    }
  };
  if (STREAM) {
    wstage(c_lo, 0);
  } else if (g.raw_w) {
    // wt is the caller's w[Cout][Cin][9]; zeros beyond Cout / Cin
    if constexpr (S3) {
      // a thread splits the nine taps of two channels of a filter (72 contiguous bytes); the four channel pairs and
      // sixteen filters of a wave's threads fill 256 contiguous bytes of each (tap, part)
      const int n = (c_hi - c_lo) * 256;
      uint32_t* Wu = reinterpret_cast<uint32_t*>(Wl);
      for (int i = tid; i < n; i += NT) {
        const int f = (i / 4) % 16, ci = c_lo * 32 + (i / 64) * 8 + (i % 4) * 2;
        const bool okf = cbo * 16 + f < g.Cout, ok0 = okf && ci < g.Cin, ok1 = okf && ci + 1 < g.Cin;
        const float* w0 = wt + ((size_t)(ok0 ? cbo * 16 + f : 0) * g.Cin + (ok0 ? ci : 0)) * 9;
        float v0[9], v1[9];
#pragma unroll
        for (int u = 0; u < 9; ++u) { v0[u] = ok0 ? w0[u] : 0.f; v1[u] = ok1 ? w0[9 + u] : 0.f; }
        uint32_t* dst = Wu + (i / 256) * kS3FwdChunk + i % 256;
#pragma unroll
        for (int u = 0; u < 9; ++u) {
          uint16_t a[3], b[3];
          s3_split_weight(v0[u], a[0], a[1], a[2]);
          s3_split_weight(v1[u], b[0], b[1], b[2]);
#pragma unroll
          for (int k = 0; k < 3; ++k) dst[(u * 3 + k) * 256] = ((uint32_t)a[k] | (uint32_t)b[k] << 16) ^ (s3_tap_turned(u) ? 0x80008000u : 0u);
        }
      }
    } else {
      // sixteen loads 9 Cin floats apart per (channel, tap) and one 64-byte row of the block
      const int pairs = (c_hi - c_lo) * (CHF / 16), e_lo = c_lo * (CHF / 16), e_end = g.Cin * 9;
      const float* wrow = wt + (size_t)cbo * 16 * e_end;
      for (int i = tid; i < pairs; i += NT) {
        const int e = e_lo + i;                    // ci * 9 + u
        f4 v[4];
#pragma unroll
        for (int f = 0; f < 16; ++f)
          v[f / 4][f % 4] = (e < e_end && cbo * 16 + f < g.Cout) ? wrow[(size_t)f * e_end + e] : 0.f;
#pragma unroll
        for (int k = 0; k < 4; ++k) reinterpret_cast<f4*>(Wl)[i * 4 + k] = v[k];
      }
    }
  } else {
    const f4* src = reinterpret_cast<const f4*>(wsrc + (size_t)c_lo * CHF);
    f4* dst = reinterpret_cast<f4*>(Wl);
    const int n4 = (c_hi - c_lo) * (CHF / 4);
    for (int i = tid; i < n4; i += NT) dst[i] = src[i];
  }
  __syncthreads();

  // the wave index as a scalar: everything derived from it (band, rows, validity) is wave-uniform and the
  // compiler can branch on it without masking lanes
  const int wave = __builtin_amdgcn_readfirstlane(tid / 64), lane = tid % 64;
  const int wx = wave % NWX, wy = wave / NWX;
  const int lg = lane / 16, lc = lane % 16;
  const int x0 = g.seg_xorg[seg] + wx * 32;
  const int out_lo = g.seg_lo[seg], out_hi = g.seg_hi[seg];
  const int y0 = (bg * NWY + wy) * g.TY;
  const bool live = y0 < g.H;                // else: a band below the image
  const int nsteps = g.TY + 2;
  const int HW = g.H * g.W;

  int rot[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) rot[s] = rot_of[q * 4 + s];

  // A-operand loads: lane (lc, lg) reads X[ci][h][x0 + 2*lc .. +1], ci = 8*lg + i of a chunk (bf16 parts: its slice of
  // the 32-channel contraction) or 4*kstep + lg.  The address is a
  // per-row lane pointer plus a 32-bit channel offset.  Products of rows outside the image are discarded,
  // channels beyond Cin meet zero filter taps, so both only need a valid address; pixels beyond W must
  // read as zero (only possible when W % 32 != 0).
  const int pxa = x0 + 2 * lc;
  const bool px_ok = pxa < g.W;
  const float* xn = x + (size_t)n * g.Cin * HW + (px_ok ? pxa : 0);
  uint32_t lgoff = (uint32_t)(S3 ? lg * 8 : lg) * (uint32_t)HW;
  asm volatile("" : "+v"(lgoff));   // opaque: keeps the K-step part of the offset scalar (no per-load vector multiply)
  const uint32_t off_last = (uint32_t)(g.Cin - 1) * (uint32_t)HW;   // channels beyond Cin read channel Cin-1
  auto row_ptr = [&](int t) -> const float* {
    const int h = min(max(y0 - 1 + t, 0), g.H - 1);
    return xn + (size_t)h * g.W;
  };
  auto load_a = [&](const float* rp, int c, int k) -> float2 {      // k-th load of chunk c
    const uint32_t off = min((uint32_t)(S3 ? c * 32 + k : (c * KC + k) * 4) * (uint32_t)HW + lgoff, off_last);
    const float2 v2 = *reinterpret_cast<const float2*>(rp + off);
    if (FASTW) return v2;
    return px_ok ? v2 : make_float2(0.f, 0.f);
  };

  float accA[4][8], accB[4][8];
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int j = 0; j < 8; ++j) { accA[s][j] = 0.f; accB[s][j] = 0.f; }

  // A operands of one 32-channel chunk, refilled for the next chunk (possibly of the next row): with parts as soon as
  // they are split, with fp32 instructions each slot right after its MFMAs.  The prefetch distance is one chunk.
  float2 a_cur[KC];
  {
    const float* rp = row_ptr(0);
#pragma unroll
    for (int ks = 0; ks < KC; ++ks) a_cur[ks] = load_a(rp, c_lo, ks);
    __builtin_amdgcn_s_waitcnt(0x0F70);
  }
  const float* wl_lane = S3 ? Wl + lane * 4 : Wl + lg * 144 + lc;
  int seq = 0;                           // chunk steps done (streaming: LDS buffer parity)

  for (int t = 0; t < nsteps; ++t) {
    const int h = y0 - 1 + t;
    const bool row_ok = h >= 0 && h < g.H;
    const float* rp_cur = row_ptr(t);
    const float* rp_nxt = row_ptr(t + 1);
    f4 P[9][2];   // written by the row's first K-step (accumulator input = constant zero), or zeroed below

    // One chunk: parts tap by tap, fp32 instructions K-step by K-step, the weights read from LDS one tap or K-step ahead.
    // The scheduling fences keep loads and LDS reads where they are issued; left alone the compiler sinks them next to
    // their first use and waits there.
    auto chunk = [&](int c, bool first) {
      if (STREAM) asm volatile("" : "+s"(c));      // opaque: addresses are formed where they are used, not kept (and spilled) per chunk
      const bool last = c + 1 == c_hi;
      const float* rp = last ? rp_nxt : rp_cur;
      const int cn = last ? c_lo : c + 1;
      if (STREAM) wload(cn, 0);
      const float* wc = STREAM ? wl_lane + (seq & 1) * CHF : wl_lane + (size_t)(c - c_lo) * CHF;
      if constexpr (S3) {
        // the chunk's sixteen values of this lane (eight channels x two pixels) as packed parts
        u32x4 ap[2][3];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const S3Pair lo = s3_split2(a_cur[2 * i].x, a_cur[2 * i + 1].x), hi = s3_split2(a_cur[2 * i].y, a_cur[2 * i + 1].y);
#pragma unroll
          for (int k = 0; k < 3; ++k) { ap[0][k][i] = lo.p[k]; ap[1][k][i] = hi.p[k]; }
        }
#pragma unroll
        for (int k = 0; k < KC; ++k) a_cur[k] = load_a(rp, cn, k);
        const u32x4* wu = reinterpret_cast<const u32x4*>(wc);
        u32x4 bw[2][3];
#pragma unroll
        for (int k = 0; k < 3; ++k) bw[0][k] = wu[k * 64];
#pragma unroll
        for (int u = 0; u < 9; ++u) {
          if (u + 1 < 9) {
#pragma unroll
            for (int k = 0; k < 3; ++k) bw[(u + 1) & 1][k] = wu[((u + 1) * 3 + k) * 64];
          }
          if (STREAM && u == 4) {
            wstore((seq + 1) & 1, 0);
            wload(cn, 1);
          }
          __builtin_amdgcn_sched_barrier(0);
          const u32x4* b = bw[u & 1];
          // The smallest products first, their sum from zero: only the chunk's total meets the running sum, where one
          // chain through all chunks is cut six times a chunk (4x512 -> 512, 32x32: 204 against 195 us; error 8.4e-8 of the
          // norm, 1.3e-7 on the fp32 instructions; 8x64 -> 64, 256x256: 5.9e-8, 9.7e-8).
#pragma unroll
          for (int t = 0; t < 2; ++t) {
            f4 s = s3_mfma(ap[t][2], b[0], f4{0.f, 0.f, 0.f, 0.f});
            s = s3_mfma(ap[t][0], b[2], s);
            s = s3_mfma(ap[t][1], b[1], s);
            s = s3_mfma(ap[t][1], b[0], s);
            s = s3_mfma(ap[t][0], b[1], s);
            s = s3_mfma(ap[t][0], b[0], s);
            if (first) P[u][t] = s;
            else P[u][t] += s;
            asm volatile("" : "+v"(P[u][t]));       // here and not later: eighteen such sums at once do not fit the registers
            __builtin_amdgcn_sched_barrier(0);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      } else {
        float bw[2][9];
#pragma unroll
        for (int u = 0; u < 9; ++u) bw[0][u] = wc[u * 16];
#pragma unroll
        for (int ks = 0; ks < KC; ++ks) {
          if (ks + 1 < KC) {
#pragma unroll
            for (int u = 0; u < 9; ++u) bw[(ks + 1) & 1][u] = wc[(ks + 1) * 4 * 144 + u * 16];
          }
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int u = 0; u < 9; ++u) {
            const f4 zero = f4{0.f, 0.f, 0.f, 0.f};
            P[u][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a_cur[ks].x, bw[ks & 1][u], first && ks == 0 ? zero : P[u][0], 0, 0, 0);
            P[u][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a_cur[ks].y, bw[ks & 1][u], first && ks == 0 ? zero : P[u][1], 0, 0, 0);
          }
          a_cur[ks] = load_a(rp, cn, ks);
          if (STREAM && ks == KC / 2) {
            wstore((seq + 1) & 1, 0);
            wload(cn, 1);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      if (STREAM) {
        wstore((seq + 1) & 1, 1);
        __syncthreads();
      }
      ++seq;
    };
    // A row above / below the image (first and last band only) is multiplied like any other, from the clamped
    // row's values, and its products are then discarded: zeroing them ahead of the branch instead would put
    // 72 register moves on every row's path.  A wave whose whole band lies below the image (the workgroup's bands
    // need not divide H) multiplies nothing: it only keeps the workgroup's barriers and filter stages in step.
    if (live) {
      chunk(c_lo, true);
      for (int c = c_lo + 1; c < c_hi; ++c) chunk(c, false);
    } else if (STREAM) {
      for (int c = c_lo; c < c_hi; ++c) {
        wstage(c + 1 == c_hi ? c_lo : c + 1, (seq + 1) & 1);
        __syncthreads();
        ++seq;
      }
    }
    if (!row_ok || !live) {
      asm volatile("" ::: "memory");       // keeps this a branch
#pragma unroll
      for (int u = 0; u < 9; ++u) { P[u][0] = f4{0.f, 0.f, 0.f, 0.f}; P[u][1] = f4{0.f, 0.f, 0.f, 0.f}; }
    }

    // ---- neighbour values across lane groups and waves --------------------------
    // Lane (lg, lc) holds filter lc, pixels x0 + 8*lg + j, j = 2*i + b for P[u][b][i].
    float nbL[9], nbR[9];  // P_u at pixel (first - 1) resp. (last + 1) of this lane's 8 pixels
    const int par = t & 1;
    float* el = EL + (par * NW + wave) * 128 + lc;
    float* er = ER + (par * NW + wave) * 128 + lc;
    if (lg == 0) {
#pragma unroll
      for (int u = 0; u < 9; ++u)
        if (u != 4) el[edge_slot(u) * 16] = P[u][0][0];
    }
    if (lg == 3) {
#pragma unroll
      for (int u = 0; u < 9; ++u)
        if (u != 4) er[edge_slot(u) * 16] = P[u][1][3];
    }
    const int addr_up = ((lane + 16) & 63) * 4, addr_dn = ((lane + 48) & 63) * 4;
#pragma unroll
    for (int u = 0; u < 9; ++u) {
      if (u == 4) { nbL[u] = 0.f; nbR[u] = 0.f; continue; }
      // The sources are pinned in VGPRs of their own first: handing an element of the
      // accumulator vector straight to the cross-lane read picked the wrong element.
      float first_px = P[u][0][0], last_px = P[u][1][3];
      asm volatile("" : "+v"(first_px), "+v"(last_px));
      nbR[u] = __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(addr_up, __builtin_bit_cast(int, first_px)));
      nbL[u] = __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(addr_dn, __builtin_bit_cast(int, last_px)));
    }
    __syncthreads();
    if (NWX > 1) {
      // all lanes read both neighbour-wave slots (in bounds for every wave), then select; a chain
      // end has no neighbour: zero, which is right at an image border (other ends are not stored)
      const float* eln = EL + (par * NW + wave + 1) * 128 + lc;  // right neighbour's left edge
      const float* erp = ER + (par * NW + wave - 1) * 128 + lc;  // left neighbour's right edge
      const bool at_r = lg == 3, at_l = lg == 0;
      const bool has_r = wx + 1 < NWX, has_l = wx > 0;
#pragma unroll
      for (int u = 0; u < 9; ++u) {
        if (u == 4) continue;
        const float vr = has_r ? eln[edge_slot(u) * 16] : 0.f;
        const float vl = has_l ? erp[edge_slot(u) * 16] : 0.f;
        nbR[u] = at_r ? vr : nbR[u];
        nbL[u] = at_l ? vl : nbL[u];
      }
    } else {
#pragma unroll
      for (int u = 0; u < 9; ++u) {
        nbR[u] = lg == 3 ? 0.f : nbR[u];
        nbL[u] = lg == 0 ? 0.f : nbL[u];
      }
    }

    // ---- place the row of products at the rotated positions (Eq. 8) --------------
    const int y = h - 1;                       // output row completed by this step
    const int px0 = x0 + 8 * lg;               // first of this lane's 8 pixels
    const int co = cbo * 16 + lc;
    const bool fin = t >= 2 && y < g.H && co < g.Cout && px0 >= out_lo && px0 < out_hi;
    float best[8];
    uint32_t pk[2] = {0u, 0u};                 // arg-max bytes of the lane's 8 pixels
    int grp_r = 0;                             // any rotation of the bank (its pool group)
    bool first = true;
    auto place = [&](int s, int j, float& yfin) {
      // three taps per filter row; a sum starts from its first term (0 + v is an instruction: it is not v for v = -0), with
      // parts from one that is not turned (every row of every turn has one)
      float tr[3] = {0.f, 0.f, 0.f};
      bool begun[3] = {false, false, false};
#pragma unroll
      for (int k = 0; k < 9; ++k) {
        const int u = !S3 ? k : k < 5 ? 2 * k : 2 * (k - 5) + 1;
        const int jj = j + tap_j(s, u) - 1;
        const float val = jj < 0 ? nbL[u] : jj > 7 ? nbR[u] : P[u][jj & 1][jj >> 1];
        const int ti = tap_i(s, u);
        tr[ti] = !begun[ti] ? val : S3 && s3_tap_turned(u) ? tr[ti] - val : tr[ti] + val;
        begun[ti] = true;
      }
      const float t0 = tr[0], t1 = tr[1], t2 = tr[2];
      yfin = accA[s][j] + t2;         // rows h-2, h-1, h are in: output row h-1 done
      accA[s][j] = accB[s][j] + t1;   // output row h has rows h-1, h
      accB[s][j] = t0;                // output row h+1 has row h
    };
    if (UNPOOLED) {
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        float yfin[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) place(s, j, yfin[j]);
        if (fin && rot[s] >= 0) {
          float* o = out_val + ((((size_t)sp * g.N + n) * g.Cout + co) * g.R + rot[s]) * HW + (size_t)y * g.W + px0;
          if (FASTW) {
            reinterpret_cast<f4*>(o)[0] = f4{yfin[0], yfin[1], yfin[2], yfin[3]};
            reinterpret_cast<f4*>(o)[1] = f4{yfin[4], yfin[5], yfin[6], yfin[7]};
          } else {
#pragma unroll
            for (int j = 0; j < 8; ++j)
              if (px0 + j < min(g.W, out_hi)) o[j] = yfin[j];
          }
        }
      }
    } else {
      // pixel by pixel: the four rotations' values, their max and arg-max (smallest r wins ties)
#pragma unroll
      for (int s = 0; s < 4; ++s)
        if (rot[s] >= 0) { grp_r = rot[s]; first = false; }
      // all four quarter turns in the orientation set (every closed set; wave-uniform): plain compare chain
      const bool allrot = (rot[0] | rot[1] | rot[2] | rot[3]) >= 0;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        float bv = 0.f;
        int bi = 0;
        float yv[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) place(s, j, yv[s]);
        if (allrot) {
          bv = yv[0];
          bi = rot[0];
#pragma unroll
          for (int s = 1; s < 4; ++s) {
            const bool gt = yv[s] > bv;
            bv = gt ? yv[s] : bv;
            bi = gt ? rot[s] : bi;
          }
        } else {
          bool have = false;
#pragma unroll
          for (int s = 0; s < 4; ++s) {
            if (rot[s] >= 0) {
              const bool gt = !have || yv[s] > bv;
              bv = gt ? yv[s] : bv;
              bi = gt ? rot[s] : bi;
              have = true;
            }
          }
        }
        best[j] = bv;
        pk[j >> 2] |= (uint32_t)bi << (8 * (j & 3));
      }
    }
    if (!UNPOOLED && g.relu) {      // fused ReLU (pooled output only): dead elements get idx 255
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const bool dead = best[j] <= 0.f;      // a NaN stays one
        best[j] = dead ? 0.f : best[j];
        pk[j >> 2] |= dead ? 0xffu << (8 * (j & 3)) : 0u;
      }
    }
    if (!UNPOOLED && fin && !first) {
      size_t chan;
      if (g.out_mode == kOutPooled) {
        // every rotation of this bank lies in pool group (r mod ng); pooled channel = co*ng + group
        chan = (size_t)n * g.Cout * g.ng + (size_t)co * g.ng + (grp_r % g.ng);
      } else {  // kOutPartial: per-bank candidates [Q][N][Cout][H][W]
        chan = ((size_t)q * g.N + n) * g.Cout + co;
      }
      const size_t off = chan * HW + (size_t)y * g.W + px0;
      if (FASTW) {
        f4* o = reinterpret_cast<f4*>(out_val + off);
        o[0] = f4{best[0], best[1], best[2], best[3]};
        o[1] = f4{best[4], best[5], best[6], best[7]};
        *reinterpret_cast<uint2*>(out_idx + off) = make_uint2(pk[0], pk[1]);
      } else {
#pragma unroll
        for (int j = 0; j < 8; ++j)
          if (px0 + j < min(g.W, out_hi)) {
            out_val[off + j] = best[j];
            out_idx[off + j] = (uint8_t)(pk[j >> 2] >> (8 * (j & 3)));
          }
      }
    }
  }
}

// Max over the per-bank candidates of a pool group that spans several banks.
// Candidates [Q][N][Cout][HW]; group g of filter co collects banks q with (r mod ng) == g.
__global__ __launch_bounds__(256) void k_p4_combine(const float* __restrict__ pv, const uint8_t* __restrict__ pi,
                                                    const int32_t* __restrict__ rot_of, float* __restrict__ ypool,
                                                    uint8_t* __restrict__ idx, int N, int Cout, int HW, int Q, int ng,
                                                    int relu) {
  const int p = blockIdx.x * 256 + threadIdx.x;
  if (p >= HW) return;
  const int chan = blockIdx.y, n = blockIdx.z;  // chan = co*ng + grp
  const int co = chan / ng, grp = chan % ng;
  float best = 0.f;
  int bi = 255;
  for (int q = 0; q < Q; ++q) {
    int r0 = -1;
    for (int s = 0; s < 4; ++s)
      if (rot_of[q * 4 + s] >= 0) { r0 = rot_of[q * 4 + s]; break; }
    if (r0 < 0 || r0 % ng != grp) continue;
    const size_t o = (((size_t)q * N + n) * Cout + co) * HW + p;
    const float vq = pv[o];
    const int iq = pi[o];
    if (bi == 255 || vq > best || (vq == best && iq < bi)) { best = vq; bi = iq; }
  }
  const size_t o = ((size_t)n * Cout * ng + chan) * HW + p;
  const bool dead = relu && best <= 0.f;
  ypool[o] = dead ? 0.f : best;
  idx[o] = dead ? (uint8_t)255 : (uint8_t)bi;
}

// Channel split: y = sum of the parts, ascending (four elements per thread, scalar tail), in fp32 or, for the shares of the one
// contraction, in 64 bits (1x512 -> 128, 16x16 in sixteen shares: the error 9.8e-8 in fp32, 6.6e-8 so, in no more time).  The parts lie on
// 16 bytes only where n_elem is a multiple of four, and y of odd rows anywhere.
template <typename A>
__global__ __launch_bounds__(256) void k_p4_sum_parts(const float* __restrict__ part, float* __restrict__ y,
                                                      size_t n_elem, int nparts) {
  // (in 64 bits from zero: eight loads at a time of the first eight parts too, 15.1 -> 13.5 us; in fp32 that would lose a part's -0)
  constexpr int K0 = std::is_same_v<A, float> ? 1 : 0;
  const size_t n4 = n_elem / 4;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n4; i += (size_t)gridDim.x * 256) {
    A a[4] = {0, 0, 0, 0};
    if constexpr (K0) {
      const f4 first = reinterpret_cast<const f4u*>(part)[i];
#pragma unroll
      for (int e = 0; e < 4; ++e) a[e] = first[e];
    }
#pragma unroll 8
    for (int k = K0; k < nparts; ++k) {
      const f4 v = reinterpret_cast<const f4u*>(part + (size_t)k * n_elem)[i];
#pragma unroll
      for (int e = 0; e < 4; ++e) a[e] += v[e];
    }
    reinterpret_cast<f4u*>(y)[i] = f4{(float)a[0], (float)a[1], (float)a[2], (float)a[3]};
  }
  for (size_t e = n4 * 4 + (size_t)blockIdx.x * 256 + threadIdx.x; e < n_elem; e += (size_t)gridDim.x * 256) {
    A v = part[e];
    for (int k = 1; k < nparts; ++k) v += part[(size_t)k * n_elem + e];
    y[e] = (float)v;
  }
}

// Channel split, pooled: every orientation's sum over the parts (ascending), then max / arg-max over the pool
// group (first maximum wins) and the fused activation.  One thread per pooled element of the C filters from c0 on.
__global__ __launch_bounds__(256) void k_p4_sum_pool(const float* __restrict__ part, float* __restrict__ ypool,
                                                     uint8_t* __restrict__ idx, size_t n_elem, int nparts, int N, int C,
                                                     int c0, int Cout, int R, int ng, int HW, int relu) {
  const size_t total = (size_t)N * C * ng * HW;
  const size_t e = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= total) return;
  const int px = (int)(e % HW);
  const int grp = (int)((e / HW) % ng);
  const size_t nc = e / ((size_t)HW * ng);
  const float* yb = part + nc * R * HW + px;
  float best = 0.f;
  int bi = -1;
  for (int r = grp; r < R; r += ng) {
    float v = yb[(size_t)r * HW];
#pragma unroll 8
    for (int k = 1; k < nparts; ++k) v += yb[(size_t)k * n_elem + (size_t)r * HW];
    if (bi < 0 || v > best) { best = v; bi = r; }
  }
  size_t o = e;
  if (C != Cout) o += ((size_t)((uint32_t)nc / (uint32_t)C) * (Cout - C) + c0) * ng * HW;      // a slice (a division less, 0.1 us)
  const bool dead = relu && best <= 0.f;
  ypool[o] = dead ? 0.f : best;
  idx[o] = dead ? (uint8_t)255 : (uint8_t)bi;
}

// base bank(s) -> Q first-quadrant banks in the LDS image layout: [Q][CB][CinPad][9][16] fp32, or
// [Q][CB][chunk][tap][part][lane][8] bf16 parts; zero for padded filters / channels.
// nq > 1: the banks are folded into the sixteen filters of a block (column n = bank n % nq of filter n / nq): [CB']...
// One thread per (bank, filter, channel or pair of channels) and three taps (blockIdx.y).
template <bool S3>
__global__ __launch_bounds__(256) void k_p4_pack_fwd(const float* __restrict__ w, float* __restrict__ wt, ExpandTables tab,
                                                     int Q, int CB, int CinPad, int Cin, int Cout, int round16, int nq,
                                                     int cb0) {
  constexpr int CPT = S3 ? 2 : 1;                   // channels per thread
  const int per = CinPad * 16 / CPT;                // threads per block of sixteen filters
  const int total = (nq > 1 ? 1 : Q) * CB * per;
  const int e = blockIdx.x * 256 + threadIdx.x, u0 = blockIdx.y * 3;
  if (e >= total) return;
  const int blk = e / per, i = e % per;
  const int c16 = S3 ? (i / 4) % 16 : i % 16;
  const int ci = S3 ? (i / 64) * 8 + (i % 4) * 2 : i / 16;
  const int cb = cb0 + blk % CB;
  const int fpb = 16 / nq;
  const int q = nq > 1 ? c16 % nq : blk / CB;
  const int co = nq > 1 ? cb * fpb + c16 / nq : cb * 16 + c16;
  const size_t bank_stride = (size_t)Cout * Cin * 9;
  if constexpr (S3) {
    const bool in0 = co < Cout && ci < Cin, in1 = co < Cout && ci + 1 < Cin;
    const float* s0 = w + ((size_t)(in0 ? co : 0) * Cin + (in0 ? ci : 0)) * 9;
    const float* s1 = w + ((size_t)(in1 ? co : 0) * Cin + (in1 ? ci + 1 : 0)) * 9;
    uint32_t* dst = reinterpret_cast<uint32_t*>(wt) + ((size_t)blk * (CinPad / 32) + i / 256) * kS3FwdChunk + i % 256;
    float va[3], vb[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      va[j] = expand_tap(s0, bank_stride, 9, q, u0 + j, in0, tab, round16);
      vb[j] = expand_tap(s1, bank_stride, 9, q, u0 + j, in1, tab, round16);
    }
#pragma unroll
    for (int j = 0; j < 3; ++j) {
      uint16_t a[3], b[3];
      s3_split_weight(va[j], a[0], a[1], a[2]);
      s3_split_weight(vb[j], b[0], b[1], b[2]);
      const uint32_t turn = s3_tap_turned(u0 + j) ? 0x80008000u : 0u;
#pragma unroll
      for (int k = 0; k < 3; ++k) dst[((u0 + j) * 3 + k) * 256] = ((uint32_t)a[k] | (uint32_t)b[k] << 16) ^ turn;
    }
  } else {
    const bool in = co < Cout && ci < Cin;
    const float* src = w + (size_t)(in ? co * Cin + ci : 0) * 9;
    float* dst = wt + (size_t)(e / 16) * 144 + c16;
    float v[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) v[j] = expand_tap(src, bank_stride, 9, q, u0 + j, in, tab, round16);
#pragma unroll
    for (int j = 0; j < 3; ++j) dst[(u0 + j) * 16] = v[j];
  }
}

template <int NWX, int NWY, bool UNPOOLED, bool FASTW, bool STREAM, bool S3 = false, int KC = 8>
void launch_i(const P4Geom& g, const float* x, const float* wt, const int32_t* rot_of, float* ov, uint8_t* oi,
              hipStream_t st) {
  const size_t wfl = (size_t)(STREAM ? 2 : g.cper) * chunk_words(g.CinPad, S3);
  const size_t lds = (wfl + 4 * NWX * NWY * 128) * sizeof(float);
  const int grid = (g.units + 7) / 8 * 8;
  auto kern = k_p4_fwd<NWX, NWY, UNPOOLED, FASTW, STREAM, S3, KC>;
  (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  hipLaunchKernelGGL(kern, dim3(grid), dim3(64 * NWX * NWY), lds, st, x, wt, rot_of, ov, oi, g);
}

template <int NWX, int NWY>
void launch_t(const P4Geom& g, bool fastw, bool stream, const float* x, const float* wt, const int32_t* rot_of,
              float* ov, uint8_t* oi, hipStream_t st) {
  const bool unp = g.out_mode == kOutUnpooled;
  if (g.s3) {               // whole rows only (p4_fwd_geoms, s3_rows)
    if (unp && stream) launch_i<NWX, NWY, true, true, true, true>(g, x, wt, rot_of, ov, oi, st);
    else if (unp) launch_i<NWX, NWY, true, true, false, true>(g, x, wt, rot_of, ov, oi, st);
    else if (stream) launch_i<NWX, NWY, false, true, true, true>(g, x, wt, rot_of, ov, oi, st);
    else launch_i<NWX, NWY, false, true, false, true>(g, x, wt, rot_of, ov, oi, st);
    return;
  }
  if (g.CinPad == 4) {      // at most 4 input channels: one K-step per row
    if (unp && fastw) launch_i<NWX, NWY, true, true, false, false, 1>(g, x, wt, rot_of, ov, oi, st);
    else if (unp) launch_i<NWX, NWY, true, false, false, false, 1>(g, x, wt, rot_of, ov, oi, st);
    else if (fastw) launch_i<NWX, NWY, false, true, false, false, 1>(g, x, wt, rot_of, ov, oi, st);
    else launch_i<NWX, NWY, false, false, false, false, 1>(g, x, wt, rot_of, ov, oi, st);
    return;
  }
  if (unp) {
    if (stream) launch_i<NWX, NWY, true, false, true>(g, x, wt, rot_of, ov, oi, st);   // deep inputs: streamed block
    else if (fastw) launch_i<NWX, NWY, true, true, false>(g, x, wt, rot_of, ov, oi, st);
    else launch_i<NWX, NWY, true, false, false>(g, x, wt, rot_of, ov, oi, st);
  } else if (stream) {
    if (fastw) launch_i<NWX, NWY, false, true, true>(g, x, wt, rot_of, ov, oi, st);
    else launch_i<NWX, NWY, false, false, true>(g, x, wt, rot_of, ov, oi, st);   // a wave chain overhangs the row
  } else if (fastw) {
    launch_i<NWX, NWY, false, true, false>(g, x, wt, rot_of, ov, oi, st);
  } else {
    launch_i<NWX, NWY, false, false, false>(g, x, wt, rot_of, ov, oi, st);
  }
}

// Is a part's share of a block of 16 filters too large to stay in LDS next to the edge arrays?
bool needs_stream(const rotconv_plan* p, int csplit = 1) {
  const int nchunk = cin_pad_f32(p->d.Cin) == 4 ? 1 : cin_pad_f32(p->d.Cin) / 32;
  return (nchunk + csplit - 1) / csplit > max_cper(p->fwd_s3);
}

}  // namespace

bool p4_fwd_parts_wanted(const rotconv_plan* p) {
  return cin_pad_f32(p->d.Cin) > 4 && p->opt.bf16_parts >= 0 && s3_fwd_supported(p);
}

bool p4_fwd_f32_rows(const rotconv_plan* p) {
  // whole pixel pairs; segmented rows need whole-lane validity
  return !(p->d.W & 1) && (p->d.W <= 256 || !(p->d.W & 31));
}

bool p4_fwd_supported(const rotconv_plan* p) {
  const rotconv_desc& d = p->d;
  if (d.k != 3 || d.stride != 1 || d.pad != 1) return false;   // bf16 plans run these kernels on widened copies
  if (p4_fwd_f32_rows(p)) return true;
  // The kernel on bf16 parts takes rows of any width.  Not where the pool group spans several banks: there the padded rows'
  // base products (k_p4_fwd_base) are one contraction instead of one per bank.  bf16 tensors: on padded rows their own kernel.
  return d.dtype == ROTCONV_F32 && p4_fwd_parts_wanted(p) && p4_fwd_pool_mode(p) != kOutPartial;
}

namespace {
// Time of a launch plan, the sum of its launches' band costs, in 0.1 us; a negative value where there is none.
double plan_cost_p4(const rotconv_plan* p, int out_mode, int csplit) {
  if (p->fwd_s3 && ((p->d.W & 7) || !p4_fwd_f32_rows(p))) return -1;
  P4Geom gs[4];
  const int n = p4_fwd_geoms(p, out_mode, gs, 4, csplit);
  double c = 0;
  for (int i = 0; i < n; ++i) {
    if (p->fwd_s3 && !gs[i].inside) return -1;      // with parts: only rows that the wave chains cover exactly
    c += gs[i].cost;
  }
  return n < 0 ? -1 : c;
}
// With bf16 parts: does the kernel of chained waves run, or the one whose waves are on their own (rotconv_s3_fwd.hip)?  The
// chain multiplies no column twice, the other one leaves no lane idle on other rows and divides the line of bands where it
// likes.  Where both can run, the smaller modelled time.  130 layers of 12 to 300 rows, 12 to 600 channels and filters: on their
// own 0.87 of the chain's time in the mean on rows of 32 to 256 pixels (3x18 -> 295, 71x128 77 -> 43 us, 8x160 -> 288, 37x64 177
// -> 130), the chain ahead where its bands fit (8x64 -> 64, 256x256 219 / 236 us, 4x512 -> 512, 32x32 189 / 221); rows with
// masks in the chain took twice its time (2x55 -> 213, 294x204 400 -> 181 us).
bool chained(const rotconv_plan* p, int out_mode, int csplit, int nq) {
  if (!p->fwd_s3) return true;
  if (nq > 1) return false;
  const double c = plan_cost_p4(p, out_mode, csplit);
  return c >= 0 && c < s3_fwd_geom(p, out_mode, csplit, nq).cost;
}
double plan_cost(const rotconv_plan* p, int out_mode, int csplit, int nq) {
  return chained(p, out_mode, csplit, nq) ? plan_cost_p4(p, out_mode, csplit) : s3_fwd_geom(p, out_mode, csplit, nq).cost;
}
}  // namespace

void p4_fwd_choose_launches(rotconv_plan* p) {
  for (int pooled = 0; pooled < 2; ++pooled) {
    rotconv_plan::FwdLaunch& l = p->fwd_launch[pooled];
    const int mode = pooled ? p4_fwd_pool_mode(p) : kOutUnpooled;
    l.csplit = p->fwd_csplit[pooled];
    l.nq = l.csplit == 1 && mode == kOutPartial ? p4_fwd_fold(p) : 1;
    l.out_mode = l.csplit > 1 ? kOutUnpooled : l.nq > 1 ? kOutPooled : mode;
    l.chain = chained(p, l.out_mode, l.csplit, l.nq);
    if (l.chain) continue;
    const S3FwdGeom g = s3_fwd_geom(p, l.out_mode, l.csplit, l.nq);
    l.ty = g.TY;
    l.nw = g.nw;
  }
}

// Parts the channel contraction is split into (1: no split).  Small maps with deep inputs give the (filter block,
// band) decomposition too few workgroups, each with a long serial contraction; splitting the 32-channel chunks over
// workgroups (at most max_cper chunks each, so the filter share stays LDS-resident) costs one unpooled fp32 part per split
// and an ordered sum.  `pooled`: the caller wants the pooled output (the alternative is the fused pooled kernel,
// with the banks folded where the plan allows it).
int p4_fwd_csplit(const rotconv_plan* p, bool pooled) {
  const rotconv_desc& d = p->d;
  const int CinPad = cin_pad_f32(d.Cin);
  if (CinPad == 4 || d.W > 256) return 1;
  const int nchunk = CinPad / 32;
  if (nchunk < 2) return 1;
  const int s3 = p->fwd_s3, most = max_cper(s3);
  // Plan option fwd_csplit: 1 keeps the contraction whole, n >= 2 asks for n parts of equal size (as many whole chunks
  // as that takes, at most 32 parts); 0: the model, which only looks at parts that stay in LDS.
  const int forced = p->opt.fwd_csplit;
  if (forced == 1) return 1;
  if (forced >= 2) {
    const int cper = std::max((nchunk + forced - 1) / forced, (nchunk + 31) / 32);
    return (nchunk + cper - 1) / cper;
  }
  const int mode = pooled ? p4_fwd_pool_mode(p) : kOutUnpooled;
  const int nq = pooled && mode == kOutPartial ? p4_fwd_fold(p) : 1;
  double best = plan_cost(p, nq > 1 ? kOutPooled : mode, 1, nq);
  int best_s = 1;
  const double part_bytes = (double)d.N * d.Cout * d.R * d.H * d.W * 4.0;
  for (int s = 2; s <= 32; s *= 2) {
    const int cper = (nchunk + s - 1) / s;
    if (cper > most) continue;
    const int s_eff = (nchunk + cper - 1) / cper;
    if (s_eff < 2) break;
    // parts written and read once at about 4 TB/s, and a dependent launch
    const double over = (s3 ? 80. : 120.) + s_eff * part_bytes / 0.2e6;
    const double c = plan_cost(p, kOutUnpooled, s_eff, 1) + over;
    if (c < best) { best = c; best_s = s_eff; }
    if (cper == 1) break;
  }
  // rotconv_pool_fwd_static takes what its array holds.  Where that is not the modelled split, a smaller one of up to
  // seven chunks a part (streamed) is taken if it is: 7x1504 -> 128, 9x8 pixels: 8 parts instead of 16.
  auto fits = [&](int s) {
    return (double)p4_fwd_least_pack_bytes(p, 1, s) + s * part_bytes <= (double)ROTCONV_STATIC_SCRATCH_BYTES;
  };
  if (pooled && s3 && best_s > 1 && !fits(best_s)) {
    for (int cper = (nchunk + best_s - 1) / best_s + 1; cper <= 7; ++cper) {
      const int s = (nchunk + cper - 1) / cper;
      if (s > 1 && fits(s)) return s;
    }
  }
  return best_s;
}

// The unpooled forward's modelled time, us; negative where there is none.  (With a channel split 0.78 of the models' sum.)
double p4_fwd_us(const rotconv_plan* p) {
  const int cs = p->fwd_csplit[0];
  const double c = plan_cost(p, kOutUnpooled, cs, 1), parts = 4.0 * cs * p->d.N * p->d.Cout * p->d.R * p->d.H * p->d.W;
  return c < 0 ? c : cs > 1 ? 0.078 * (c + 80. + parts / 0.2e6) : 0.1 * c;
}

// Are the chained waves alone (rows that they overhang masked) no faster with a split, pooled?  In units of 0.3 us: four per
// 32-channel chunk and row step of a wave and three for the placing; a split's parts at 4 TB/s and 8 us of launches.
bool p4_fwd_chain_whole(const rotconv_plan* p) {
  const rotconv_desc& d = p->d;
  const int nchunk = cin_pad_f32(d.Cin) / 32, mode = p4_fwd_pool_mode(p);
  auto cost = [&](int out_mode, int csplit, int nq) {
    P4Geom gs[4];
    const int n = p4_fwd_geoms(p, out_mode, gs, 4, csplit, nq);
    long c = 0;
    for (int i = 0; i < n; ++i) c += gs[i].rows * (4 * gs[i].cper + 3) / 4;
    return n < 0 ? -1L : c;
  };
  // banks fold into a chain's columns where the block stays in LDS or the chain fits the row
  int nq = mode == kOutPartial ? p4_fwd_fold(p) : 1;
  if (needs_stream(p) && ((d.W & 31) || (d.W <= 256 && (d.W & (d.W - 1))))) nq = 1;
  const long whole = cost(nq > 1 ? kOutPooled : mode, 1, nq);
  const double part_bytes = (double)d.N * d.Cout * d.R * d.H * d.W * 4.0;
  for (int s = 2; s <= 32; s *= 2) {
    const int cper = (nchunk + s - 1) / s, s_eff = (nchunk + cper - 1) / cper;
    if (cper > max_cper(1)) continue;
    if (s_eff < 2) break;
    if (cost(kOutUnpooled, s_eff, 1) + 28 + (long)(s_eff * part_bytes / 0.6e6) < whole) return false;
    if (cper == 1) break;
  }
  return true;
}

// Cut the row into segments of at most 256 product columns; all segments of one launch share nwx.  nq: banks folded into
// the filters of a block.  Returns the number of launches (geoms) written.
int p4_fwd_geoms(const rotconv_plan* p, int out_mode, P4Geom* out, int max_out, int csplit, int nq) {
  const rotconv_desc& d = p->d;
  P4Geom base{};
  {
    const int CinPad = cin_pad_f32(d.Cin), nchunk = CinPad == 4 ? 1 : CinPad / 32;
    base.cper = (nchunk + csplit - 1) / csplit;
    base.csplit = (nchunk + base.cper - 1) / base.cper;
  }
  base.N = d.N; base.Cin = d.Cin; base.CinPad = cin_pad_f32(d.Cin); base.H = d.H; base.W = d.W;
  base.Cout = d.Cout; base.CB = (d.Cout + 15) / 16; base.R = d.R; base.Q = p->host.Q; base.ng = p->ng;
  base.out_mode = out_mode;
  base.s3 = p->fwd_s3;
  base.relu = out_mode == kOutPooled && d.activation == ROTCONV_ACT_RELU;
  int ng = 0;
  int pos = 0;
  while (pos < d.W) {
    int xorg, nwx;
    if (pos == 0) {
      xorg = 0;
      nwx = 1;
      while (nwx * 32 < d.W && nwx < 8) nwx *= 2;
    } else {
      const int need = d.W - (pos - 8);      // product columns from the pixel left of `pos` to the border
      nwx = 1;
      while (nwx * 32 < need && nwx < 8) nwx *= 2;
      // the last segment ends exactly at the right border (W % 32 == 0 here), others start 8 px early
      xorg = nwx * 32 >= need ? d.W - nwx * 32 : pos - 8;
    }
    const int chain_end = xorg + nwx * 32;
    const int hi = chain_end >= d.W ? d.W : chain_end - 8;
    int gi = -1;
    for (int i = 0; i < ng; ++i)
      if (out[i].nwx == nwx && out[i].nseg < 4) gi = i;
    if (gi < 0) {
      if (ng >= max_out) return -1;
      gi = ng++;
      out[gi] = base;
      out[gi].nwx = nwx;
      out[gi].nseg = 0;
      out[gi].inside = 1;
    }
    P4Geom& g = out[gi];
    g.seg_xorg[g.nseg] = xorg; g.seg_lo[g.nseg] = pos; g.seg_hi[g.nseg] = hi;
    if (chain_end > d.W) g.inside = 0;
    g.nseg++;
    pos = hi;
  }
  for (int i = 0; i < ng; ++i) {
    P4Geom& g = out[i];
    const int nwy = 8 / g.nwx;
    long best_cost = -1;
    // Rows per band: short bands cost halo rows (a band of ty rows computes ty + 2 rows of products) but give
    // more workgroups when the problem is small.  Cost of a choice = rounds of workgroups over the 256 CUs x row
    // steps per wave x how many waves share a SIMD (a workgroup whose bands reach beyond the image leaves waves idle).
    for (int ty : {1, 2, 4, 8, 16, 32, 64}) {
      const int nbg = (d.H + nwy * ty - 1) / (nwy * ty);
      const long units = (long)d.N * (nq > 1 ? (d.Cout * nq + 15) / 16 : g.Q * g.CB) * nbg * g.nseg * g.csplit;
      const int bands = nbg > 1 ? nwy : std::min(nwy, (d.H + ty - 1) / ty);
      const long cost = ((units + 255) / 256) * (ty + 2) * std::max(4, g.nwx * bands);
      if (best_cost < 0 || cost <= best_cost) { best_cost = cost; g.TY = ty; g.nbg = nbg; g.units = (int)units; }
    }
    g.rows = best_cost;
    // in 0.1 us; best_cost counts the rows of a wave alone on its SIMD as four, of two that share one as eight
    g.cost = g.s3 ? best_cost * (28.7 * g.cper + 13.) / 8. + 30. + 8. * g.cper : 5. * best_cost * g.cper;
  }
  return ng;
}

// Banks folded into a wave's sixteen filters for the pooled forward: the plan pools all R = 4 Q orientations of a filter
// together, Q is 2 or 4, every bank has its four quarter turns, and the products are those of bf16 parts (1: no folding).
int p4_fwd_fold(const rotconv_plan* p) {
  const int Q = p->host.Q;
  if ((Q != 2 && Q != 4) || p->ng != 1 || !p->fwd_s3 || (p->d.W & 1)) return 1;      // (odd rows: p4_fwd_supported pads them)
  for (int i = 0; i < Q * 4; ++i)
    if (p->rot_of[i] < 0) return 1;
  return Q;
}

namespace {
int fwd_blocks(const rotconv_plan* p, int nq) { return nq > 1 ? (p->d.Cout * nq + 15) / 16 : (p->d.Cout + 15) / 16; }
// words of the packed image of one filter block (of every bank, unless they are folded into its columns)
size_t block_words(const rotconv_plan* p, int nq) {
  const int CinPad = cin_pad_f32(p->d.Cin);
  return (size_t)(nq > 1 ? 1 : p->host.Q) * (CinPad == 4 ? 1 : CinPad / 32) * chunk_words(CinPad, p->fwd_s3);
}
}  // namespace

size_t p4_fwd_weights(const rotconv_plan* p) {
  return (size_t)p->host.Q * fwd_blocks(p, 1) * cin_pad_f32(p->d.Cin) * 144;
}

size_t p4_fwd_pack_floats(const rotconv_plan* p) { return block_words(p, 1) * fwd_blocks(p, 1); }

size_t p4_fwd_least_pack_bytes(const rotconv_plan* p, int nq, int csplit) {
  return p4_fwd_raw_weights(p, nq, csplit) ? 0 : block_words(p, nq) * sizeof(float);
}

// How the bank kernel delivers its result for this plan's pooling.
int p4_fwd_pool_mode(const rotconv_plan* p) {
  // every bank must fall into a single pool group: all its rotations share r mod ng
  for (int q = 0; q < p->host.Q; ++q) {
    int grp = -1;
    for (int s = 0; s < 4; ++s) {
      const int r = p->rot_of[q * 4 + s];
      if (r < 0) continue;
      if (grp < 0) grp = r % p->ng;
      else if (grp != r % p->ng) return kOutUnpooled;
    }
  }
  // does a group collect more than one bank?
  return (p->host.Q > p->ng) ? kOutPartial : kOutPooled;
}

bool p4_fwd_raw_weights(const rotconv_plan* p, int nq, int csplit) {
  return p->d.dtype == ROTCONV_F32 && p->base_bank && nq == 1 && !needs_stream(p, csplit);
}

namespace {
// The blocks [b0, b1) of sixteen filters, as a layer of these filters alone; out_val holds no others.
void launch_blocks(const rotconv_plan* p, int b0, int b1, int out_mode, const float* x, const float* w, float* pack,
                   size_t pack_bytes, float* out_val, uint8_t* out_idx, hipStream_t st, int nq, int csplit) {
  const rotconv_plan::FwdLaunch* l = nullptr;
  for (const auto& c : p->fwd_launch)
    if (c.out_mode == out_mode && c.csplit == csplit && c.nq == nq) l = &c;
  const bool s3 = p->fwd_s3, chain = l ? l->chain : chained(p, out_mode, csplit, nq);
  P4Geom gs[4];
  const int ng = chain ? p4_fwd_geoms(p, out_mode, gs, 4, csplit) : 0;
  const bool stream = needs_stream(p, csplit);
  const int raw = p4_fwd_raw_weights(p, nq, csplit) ? 1 : 0;
  const int CinPad = cin_pad_f32(p->d.Cin);
  const int Cout = std::min(p->d.Cout, b1 * 16) - b0 * 16;      // (b0 > 0: banks not folded)
  const size_t fit = raw ? b1 - b0 : pack_bytes / (block_words(p, nq) * sizeof(float));
  const int slice = (int)std::max<size_t>(1, std::min<size_t>(b1 - b0, fit));
  for (int cb0 = b0; cb0 < b1; cb0 += slice) {
    const int ncb = std::min(slice, b1 - cb0);
    if (!raw) {
      const int total = (nq > 1 ? 1 : p->host.Q) * ncb * CinPad * (s3 ? 8 : 16);
      auto kern = s3 ? k_p4_pack_fwd<true> : k_p4_pack_fwd<false>;
      hipLaunchKernelGGL(kern, dim3((total + 255) / 256, 3), dim3(256), 0, st, w, pack, expand_tables(p), p->host.Q, ncb,
                         CinPad, p->d.Cin, p->d.Cout, p->d.dtype == ROTCONV_BF16 ? 1 : 0, nq, cb0);
    }
    const float* wt = raw ? w + (size_t)b0 * 16 * p->d.Cin * 9 : pack;
    if (!chain) {
      S3FwdGeom g = s3_fwd_geom(p, out_mode, csplit, nq, l ? l->ty : 0, l ? l->nw : 0);
      g.raw_w = raw;
      g.units = g.units / g.CB * ncb;
      g.CB = ncb;
      g.cb0 = cb0 - b0;
      g.Cout = Cout;
      launch_s3_fwd(g, x, wt, p->dev.rot_of, out_val, out_idx, st);
    }
    for (int i = 0; i < ng; ++i) {
      P4Geom g = gs[i];
      g.raw_w = raw;
      g.units = g.units / g.CB * ncb;
      g.CB = ncb;
      g.cb0 = cb0 - b0;
      g.Cout = Cout;
      const bool fastw = (p->d.W & 7) == 0 && g.inside;   // no lane reaches beyond the row: no masks, vector stores
      switch (g.nwx) {
        case 1: launch_t<1, 8>(g, fastw, stream, x, wt, p->dev.rot_of, out_val, out_idx, st); break;
        case 2: launch_t<2, 4>(g, fastw, stream, x, wt, p->dev.rot_of, out_val, out_idx, st); break;
        case 4: launch_t<4, 2>(g, fastw, stream, x, wt, p->dev.rot_of, out_val, out_idx, st); break;
        default: launch_t<8, 1>(g, fastw, stream, x, wt, p->dev.rot_of, out_val, out_idx, st); break;
      }
    }
  }
}

}  // namespace

void launch_p4_fwd(const rotconv_plan* p, int out_mode, const float* x, const float* w, float* pack, size_t pack_bytes,
                   float* out_val, uint8_t* out_idx, hipStream_t st, int nq, int csplit) {
  launch_blocks(p, 0, fwd_blocks(p, nq), out_mode, x, w, pack, pack_bytes, out_val, out_idx, st, nq, csplit);
}

void launch_p4_fwd_parts(const rotconv_plan* p, int b0, int b1, const float* x, const float* w, float* pack, size_t pack_bytes,
                         float* out_val, hipStream_t st, int csplit) {
  launch_blocks(p, b0, b1, kOutUnpooled, x, w, pack, pack_bytes, out_val, nullptr, st, 1, csplit);
}

void launch_p4_sum_parts(const rotconv_plan* p, const float* part, int nparts, float* y, hipStream_t st, bool wide) {
  const size_t n_elem = (size_t)p->d.N * p->d.Cout * p->d.R * p->Ho * p->Wo;
  const unsigned blocks = (unsigned)std::max<size_t>(1, std::min<size_t>((n_elem / 4 + 255) / 256, 4096));
  if (wide) hipLaunchKernelGGL(k_p4_sum_parts<double>, dim3(blocks), dim3(256), 0, st, part, y, n_elem, nparts);
  else hipLaunchKernelGGL(k_p4_sum_parts<float>, dim3(blocks), dim3(256), 0, st, part, y, n_elem, nparts);
}

void launch_p4_sum_pool(const rotconv_plan* p, const float* part, int nparts, float* ypool, uint8_t* idx, int c0, int nc,
                        hipStream_t st) {
  const int HW = p->Ho * p->Wo;
  const size_t n_elem = (size_t)p->d.N * nc * p->d.R * HW;
  const size_t total = (size_t)p->d.N * nc * p->ng * HW;
  hipLaunchKernelGGL(k_p4_sum_pool, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, part, ypool, idx, n_elem,
                     nparts, p->d.N, nc, c0, p->d.Cout, p->d.R, p->ng, HW, p->d.activation == ROTCONV_ACT_RELU ? 1 : 0);
}

void launch_p4_combine(const rotconv_plan* p, const float* pv, const uint8_t* pi, float* ypool, uint8_t* idx,
                       hipStream_t st) {
  const int HW = p->d.H * p->d.W;
  dim3 grid((HW + 255) / 256, p->d.Cout * p->ng, p->d.N);
  hipLaunchKernelGGL(k_p4_combine, grid, dim3(256), 0, st, pv, pi, p->dev.rot_of, ypool, idx, p->d.N, p->d.Cout, HW,
                     p->host.Q, p->ng, p->d.activation == ROTCONV_ACT_RELU ? 1 : 0);
}

}  // namespace rotconv
