// Fast input-gradient kernel for 3x3, stride 1, pad 1 (fp32 tensors), fused with the orientation max-pool backward
// (paper Eq. 12, 13, 15 in shared-product form), on the bf16 matrix cores with operands split into three bf16 parts
// (rotconv_split3.h).
//
//   dX[ci,h,x] = sum_q sum_u sum_co F_q[co,ci,u] * D^q_u[co,h,x]
//   D^q_u[co,h,x] = sum_s Delta_(q,s)[co, h+1-i_s(u), x+1-j_s(u)],   (i_s,j_s) = R_s(u),   Delta_r = G * 1[idx == r]
//
// The routed gradients of a bank's four quarter turns are summed at the rotated tap positions first, in the operand's
// layout, then ONE contraction over (filter, tap) runs on the matrix cores.
//
// A lane owns one pixel column: M = 32 input channels, N = 32 pixels, K = 16 filters, eight of which are the lane's.  The
// neighbour columns are the neighbour lanes' registers, read by the additions themselves through whole-wave lane shifts,
// so a (G, idx) value is routed once per row it serves and no neighbourhood is loaded.  For that the rows of an image are
// laid end to end as padded rows of W + 2 slots (x = -1 .. W): a wave takes 32 consecutive slots, of which the inner 30
// are outputs, whatever W is.  Loads go through a buffer descriptor of the image: positions outside it get an offset
// beyond the descriptor's size and read as zero, which routes nothing.
//
// What bounds it: per K-step and 32 slots a wave spends about 900 vector instructions on D and its three parts (1.5 ns
// each) and 54 matrix instructions of 32 x 32 x 16 per 32 channels (19 ns each); 64 channels per workgroup are what two
// waves of a SIMD have registers for, so the two together are 4.1 us of matrix and 2.7 us of vector work a K-step.  They
// are kept half a K-step apart, one building its operands while the other multiplies: the first four waves of a workgroup
// meet the K-step's barrier before they build, the last four after (all before: 342 against 285 us at 8x64 -> 64, 256x256).
// Against the kernels on fp32 matrix cores (the same card, us): 8x64 -> 64, 256x256 391 -> 286, 4x512 -> 512, 32x32
// 211 -> 165, 4x128 -> 128, 128x128 187 -> 164, 8x512 -> 512, 16x16 209 -> 104.
//
#include <hip/hip_runtime.h>

#include <algorithm>

#include "rotconv_expand.h"
#include "rotconv_kernels.h"
#include "rotconv_p4.h"
#include "rotconv_p4_taps.h"
#include "rotconv_split3.h"

namespace rotconv {
namespace {

constexpr int NW = 8;                  // waves per workgroup
constexpr int NT = 64 * NW;
constexpr int KS = 16;                 // filters per K-step
constexpr int BLK4 = 9 * 3 * 64;       // 16-byte operands of one K-step and 32-channel block: [tap][part][lane]

struct S3BwdGeom {
  int N, Cin, H, W, Cout, Q, ng;
  int tiles;     // 30-slot tiles per image
  int ntile;     // N * tiles
  int ncg;       // groups of 32 * TB input channels
  int nkb, nk;   // K-steps per bank and in all
  int ksplit, kper;
  int units;
};

// Filters of a K-step: f0 + half * hoff + min(i, Cout - 1), always inside the bank: the last K-step of a ragged bank starts
// early, and with fewer than sixteen filters the lane halves overlap.  A filter met twice has zero weights the second time
// (s3_takes); its gradients reach the same pixels either way.
__host__ __device__ constexpr int s3_first_filter(int kb, int Cout) {
  const int last = Cout > KS ? Cout - KS : 0;
  return kb * KS < last ? kb * KS : last;
}
__host__ __device__ constexpr int s3_half_off(int Cout) { return Cout >= 16 ? 8 : Cout > 8 ? Cout - 8 : 0; }
__host__ __device__ constexpr int s3_filter(int kb, int half, int i, int Cout) {
  return s3_first_filter(kb, Cout) + half * s3_half_off(Cout) + (i < Cout - 1 ? i : Cout - 1);
}
__host__ __device__ constexpr bool s3_takes(int kb, int half, int i, int Cout) {
  const int f = s3_filter(kb, half, i, Cout);
  return f >= kb * KS && i < Cout && (half == 0 || f >= s3_first_filter(kb, Cout) + 8);
}

// the value of the lane to the left / right (slot - 1 / slot + 1)
__device__ __forceinline__ float from_left(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x138, 0xf, 0xf, true));
}
__device__ __forceinline__ float from_right(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x130, 0xf, 0xf, true));
}

// TB: 32-channel blocks per workgroup (the weights of a K-step fill one of two LDS buffers).
// LAST: the main products of all nine taps after the small ones of all, else tap by tap (see s3_mains_last).
template <int TB, bool LAST>
__global__ __launch_bounds__(NT, 2) void k_s3_bwd_data(const float* __restrict__ gpool, const uint8_t* __restrict__ idx,
                                                       const u32x4* __restrict__ wp, const int32_t* __restrict__ rot_of,
                                                       float* __restrict__ dx, S3BwdGeom g) {
  constexpr int PRE = 4;                       // filters of the next K-step whose (G, idx) are loaded during the
                                               // multiplication; the others' when the build begins
  constexpr int STG = TB * BLK4;               // 16-byte pieces of a K-step's weights
  extern __shared__ float smem[];
  u32x4* Wl = reinterpret_cast<u32x4*>(smem);  // [2][STG]
  // A workgroup takes unit after unit of its XCD's share, the workgroups of an XCD side by side (they share (G, idx)
  // rows in its L2).  Units follow each other without a gap: the next one's weights and (G, idx) are on their way while
  // the last K-step multiplies.
  const int per_xcd = (g.units + 7) / 8, stride = gridDim.x / 8;
  int v = (blockIdx.x % 8) * per_xcd + blockIdx.x / 8;
  const int vend = min(g.units, (int)(blockIdx.x % 8 + 1) * per_xcd);
  if (v >= vend) return;

  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid / 64), lane = tid % 64;
  const int half = lane / 32, l31 = lane % 32;
  const int HW = g.H * g.W;
  const uint32_t plane = (uint32_t)g.ng * (uint32_t)HW;      // elements from a filter to the next
  const size_t gimg = (size_t)g.Cout * plane;
  auto tile_of = [&](int u) { return (u / (g.ksplit * g.ncg)) * NW + wave; };
  __amdgpu_buffer_rsrc_t rg, ri;
  uint32_t og[3], oi[3];   // offsets of the lane's pixel of G and idx in rows h-1, h, h+1 of its first filter
  auto set_tile = [&](int u) {
    const int tile = min(tile_of(u), g.ntile - 1);
    const int n = tile / g.tiles, slot = (tile % g.tiles) * 30 + l31;
    const int h = slot / (g.W + 2), x = slot % (g.W + 2) - 1;
    const bool in = x >= 0 && x < g.W && h < g.H;
    rg = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(gpool + (size_t)n * gimg), 0, (int)(uint32_t)(gimg * 4), 0x27000);
    ri = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(idx + (size_t)n * gimg), 0, (int)(uint32_t)gimg, 0x27000);
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const int hr = h + d - 1;
      const bool ok = in && hr >= 0 && hr < g.H;
      const uint32_t o = (uint32_t)(half * s3_half_off(g.Cout)) * plane + (uint32_t)(hr * g.W + x);
      og[d] = ok ? o * 4u : kOutside;
      oi[d] = ok ? o : kOutside;
    }
  };

  float gr[8][3];          // G and idx of the lane's eight filters on the three rows
  uint32_t ir[8][3];
  auto load_raw = [&](int k, int i0, int i1) {      // filters [i0, i1) of the lane's eight
    const int q = k / g.nkb, f0 = s3_first_filter(k % g.nkb, g.Cout);
    int grp = 0;
    if (g.ng > 1) {
#pragma unroll
      for (int s = 3; s >= 0; --s) grp = rot_of[q * 4 + s] >= 0 ? rot_of[q * 4 + s] : grp;
      grp %= g.ng;
    }
    const uint32_t base = (uint32_t)f0 * plane + (uint32_t)grp * (uint32_t)HW;
#pragma unroll
    for (int i = i0; i < i1; ++i) {
      const uint32_t so = base + (uint32_t)min(i, g.Cout - 1) * plane;
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        gr[i][d] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rg, og[d], so * 4u, 0));
        ir[i][d] = __builtin_amdgcn_raw_buffer_load_b8(ri, oi[d], so, 0);
      }
    }
  };

  u32x4 op[9][3];          // the K-step's D operands: [tap][part], eight filters of the lane's pixel
  // D of one filter (all nine taps) on the lane's pixel
  auto build_one = [&](int i, const int (&rot)[4], int q, float (&D)[9]) {
    float m[4][3];       // routed gradient per quarter turn and row
#pragma unroll
    for (int d = 0; d < 3; ++d)
#pragma unroll
      for (int s = 0; s < 4; ++s) m[s][d] = ir[i][d] == (uint32_t)rot[s] ? gr[i][d] : 0.f;
#pragma unroll
    for (int u = 0; u < 9; ++u) {
      float t = 0.f;
      bool begun = false;
      // the terms of the lane's own column first: a shifted term folds into its addition
#pragma unroll
      for (int pass = 0; pass < 2; ++pass)
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const float mv = m[s][2 - tap_i(s, u)];
          const int c = 1 - tap_j(s, u);
          if ((c == 0) != (pass == 0)) continue;
          const float val = c == 0 ? mv : c < 0 ? from_left(mv) : from_right(mv);
          t = begun ? t + val : val;
          begun = true;
        }
      D[u] = t;
    }
  };
  auto build = [&](int k) {
    const int q = k / g.nkb;
    int rot[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) rot[s] = rot_of[q * 4 + s];     // -1 (absent) matches no byte
    load_raw(k, PRE, 8);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float Da[9], Db[9];
      build_one(2 * i, rot, q, Da);
      build_one(2 * i + 1, rot, q, Db);
#pragma unroll
      for (int u = 0; u < 9; ++u) {
        const S3Pair p = s3_split2(Da[u], Db[u]);
#pragma unroll
        for (int e = 0; e < 3; ++e) op[u][e][i] = p.p[e];
      }
      // the operands are first used in the multiplication: without an opaque use here the compiler moves all of the
      // arithmetic there and keeps its inputs instead
#pragma unroll
      for (int u = 0; u < 9; ++u)
#pragma unroll
        for (int e = 0; e < 3; ++e) asm volatile("" : "+v"(reinterpret_cast<uint32_t*>(&op[u][e])[i]));
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  // weights of a K-step -> LDS, in pieces of PC 16-byte loads per thread
  constexpr int PER = (STG + NT - 1) / NT;         // 16-byte pieces per thread and stage
  constexpr int PC = 2, NP = (PER + PC - 1) / PC, STEP = TB * 9 / (NP + 1) + 1;
  u32x4 wreg[PC];
  auto wsrc = [&](int u, int k) { return wp + ((size_t)(u / g.ksplit % g.ncg) * g.nk + k) * STG; };
  auto wload = [&](const u32x4* src, int p) {
#pragma unroll
    for (int j = 0; j < PC; ++j) {
      const unsigned e = threadIdx.x + (p * PC + j) * NT;
      if (p * PC + j < PER && e < STG) wreg[j] = src[e];
    }
  };
  auto wstore = [&](int buf, int p) {
#pragma unroll
    for (int j = 0; j < PC; ++j) {
      const unsigned e = threadIdx.x + (p * PC + j) * NT;
      if (p * PC + j < PER && e < STG) Wl[buf * STG + e] = wreg[j];
    }
  };

  s3_f16 acc[TB];
#pragma unroll
  for (int j = 0; j < TB; ++j)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[j][r] = 0.f;

  auto first_k = [&](int u) { return (u % g.ksplit) * g.kper; };
  int k = first_k(v), k1 = min(g.nk, k + g.kper);
  set_tile(v);
  load_raw(k, 0, PRE);
  for (int p = 0; p < NP; ++p) {
    wload(wsrc(v, k), p);
    wstore(0, p);
  }
  const bool early = wave < NW / 2;
  int buf = 0;
  while (true) {
    const bool last = k + 1 == k1;                       // the unit's last K-step
    const int vn = last ? v + stride : v, kn = last ? first_k(vn) : k + 1;
    const bool next = vn < vend;
    if (early) __syncthreads();
    build(k);
    if (!early) __syncthreads();
    const u32x4* nsrc = wsrc(vn, kn);
    const u32x4* wl = Wl + buf * STG + lane;
    u32x4 wv[2][3];
    [[maybe_unused]] u32x4 w0[2];
#pragma unroll
    for (int e = 0; e < 3; ++e) wv[0][e] = wl[e * 64];
#pragma unroll
    for (int b = 0; b < TB; ++b) {
      s3_f16 t;      // a K-step's sum starts from zero and is added to the running one
#pragma unroll
      for (int r = 0; r < 16; ++r) t[r] = 0.f;
#pragma unroll
      for (int u = 0; u < 9; ++u) {
        const int st = b * 9 + u;
        if (st % STEP == 0 && st / STEP <= NP && next) {
          if (st > 0) wstore(buf ^ 1, st / STEP - 1);
          if (st / STEP < NP) wload(nsrc, st / STEP);
        }
        if (LAST ? u + 1 < 9 : st + 1 < TB * 9) {
#pragma unroll
          for (int e = 0; e < 3; ++e) wv[(LAST ? u + 1 : st + 1) & 1][e] = wl[((st + 1) * 3 + e) * 64];
        } else if (LAST) {
          w0[0] = wl[b * 27 * 64];
        }
        if (st == TB * 9 - 5 && next) {
          if (last) set_tile(vn);
          load_raw(kn, 0, PRE);
        }
        __builtin_amdgcn_sched_barrier(0);
        // the smallest products first
        const u32x4* w = wv[(LAST ? u : st) & 1];
        t = s3_mfma32(w[2], op[u][0], t);
        t = s3_mfma32(w[0], op[u][2], t);
        t = s3_mfma32(w[1], op[u][1], t);
        t = s3_mfma32(w[0], op[u][1], t);
        t = s3_mfma32(w[1], op[u][0], t);
        if constexpr (!LAST) t = s3_mfma32(w[0], op[u][0], t);
      }
      if constexpr (LAST) {      // the first parts of the weights once more
#pragma unroll
        for (int u = 0; u < 9; ++u) {
          if (u + 1 < 9) {
            w0[(u + 1) & 1] = wl[(b * 9 + u + 1) * 3 * 64];
          } else if (b + 1 < TB) {
#pragma unroll
            for (int e = 0; e < 3; ++e) wv[0][e] = wl[((b + 1) * 27 + e) * 64];
          }
          __builtin_amdgcn_sched_barrier(0);
          t = s3_mfma32(w0[u & 1], op[u][0], t);
        }
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[b][r] += t[r];
    }
    static_assert(STEP * NP < TB * 9, "a K-step's pieces are written inside it");
    buf ^= 1;
    if (last) {
      // lane: pixel l31 of the tile; accumulator element r: channel 8 (r / 4) + 4 half + r % 4 of its block
      const int tile = tile_of(v), n = tile / g.tiles, slot = (tile % g.tiles) * 30 + l31;
      const int h = slot / (g.W + 2), x = slot % (g.W + 2) - 1;
      const int c0 = (v / g.ksplit % g.ncg) * TB * 32 + 4 * half;
      if (tile < g.ntile && x >= 0 && x < g.W && h < g.H && l31 >= 1 && l31 <= 30) {
        float* o = dx + (((size_t)(v % g.ksplit) * g.N + n) * g.Cin + c0) * HW + (size_t)(h * g.W + x);
#pragma unroll
        for (int j = 0; j < TB; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int c = j * 32 + 8 * (r / 4) + r % 4;
            if (c0 + c < g.Cin) o[(size_t)c * HW] = acc[j][r];
          }
      }
#pragma unroll
      for (int j = 0; j < TB; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[j][r] = 0.f;
      if (!next) break;
      k1 = min(g.nk, kn + g.kper);
    }
    v = vn;
    k = kn;
  }
}

// banks -> [channel group][K-step (bank, 16 filters)][32-channel block of the group][tap][part][lane][8 filters].
// One thread per (block, K-step, channel, pair of filters) and three taps (blockIdx.y).
__global__ __launch_bounds__(256) void k_s3_pack_bwd(const float* __restrict__ w, uint32_t* __restrict__ wp, ExpandTables tab,
                                                     int nblk, int bpg, int nk, int nkb, int Cin, int Cout, int round16) {
  const size_t total = (size_t)nblk * nk * 256;
  const size_t e = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= total) return;
  const int i = (int)(e % 256), cp = i % 4, l = i / 4, u0 = blockIdx.y * 3;
  const int k = (int)(e / 256 % nk), blk = (int)(e / 256 / nk);
  const int ci = blk * 32 + l % 32, half = l / 32, kb = k % nkb, q = k / nkb;
  const int co0 = s3_filter(kb, half, cp * 2, Cout), co1 = s3_filter(kb, half, cp * 2 + 1, Cout);
  const size_t bank_stride = (size_t)Cout * Cin * 9;
  const bool in0 = ci < Cin && s3_takes(kb, half, cp * 2, Cout), in1 = ci < Cin && s3_takes(kb, half, cp * 2 + 1, Cout);
  const float* s0 = w + ((size_t)(in0 ? co0 : 0) * Cin + (in0 ? ci : 0)) * 9;
  const float* s1 = w + ((size_t)(in1 ? co1 : 0) * Cin + (in1 ? ci : 0)) * 9;
  uint32_t* dst = wp + (((size_t)(blk / bpg) * nk + k) * bpg + blk % bpg) * (BLK4 * 4) + i;
  float a[3], b[3];
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    a[j] = expand_tap(s0, bank_stride, 9, q, u0 + j, in0, tab, round16);
    b[j] = expand_tap(s1, bank_stride, 9, q, u0 + j, in1, tab, round16);
  }
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    uint16_t pa[3], pb[3];
    s3_split_weight(a[j], pa[0], pa[1], pa[2]);
    s3_split_weight(b[j], pb[0], pb[1], pb[2]);
#pragma unroll
    for (int z = 0; z < 3; ++z) dst[((u0 + j) * 3 + z) * 256] = (uint32_t)pa[z] | (uint32_t)pb[z] << 16;
  }
}

// The matrix instruction cuts its sums, up to 54 times a K-step and channel block at the sum's full size when each tap's six
// products are added in turn; with the small products of all taps first, nine times.  Error of the norm, fp32 instructions /
// tap by tap / mains last: 9 filters 1.38e-7 / 1.55e-7 / below 6e-8, 24 filters 1.32e-7 / 1.56e-7 / 5.6e-8, 32 filters
// 2.2e-7 / 1.7e-7 / 5.9e-8, 64 2.8e-7 / 1.7e-7 / 6.6e-8, 512 3.9e-7 / 1.9e-7 / 9.2e-8, 2048 (64 channels) 2.47e-7 / 2.48e-7 / 1.64e-7.
// The second reading of the weights' first parts costs 3 % (8x64 -> 64, 256x256: 275.5 / 283.7 us, 4x128 -> 128, 128x128
// 160.4 / 164.1): it is taken where the shorter form would be less precise than the fp32 instructions.  That is also so on
// small layers, for which the kernel on fp32 instructions shares the contraction out in short sums (1x112 -> 240, 17x61: fp32
// instructions 1.59e-7, tap by tap 1.9e-7, mains last 9.2e-8; no time lost that could be measured, 42.6 / 43.0 us both gradients).
double s3_bwd_data_flop(const rotconv_plan* p) {
  return 18.0 * p->host.Q * p->d.N * p->d.Cin * p->d.Cout * p->d.H * p->d.W;
}
bool s3_mains_last(const rotconv_plan* p, int ksplit) {
  const double flop = s3_bwd_data_flop(p);
  return p->d.Cout < 32 || p->d.Cout > 1024 || flop < 1.2e9 || (flop < 4e9 && ksplit > 1);
}

struct S3BwdPlan { S3BwdGeom g; int TB; };

// Channel blocks per workgroup and split of the contraction, by the time they are modelled to take: rounds of
// workgroups over the 256 CUs x K-steps x (54 matrix instructions per block for each of the SIMD's two waves, 19 ns each,
// or the two waves' operand builds where those are longer), the partial sums' traffic at 4 TB/s and the launch that adds
// them.
S3BwdPlan s3_bwd_plan(const rotconv_plan* p) {
  const rotconv_desc& d = p->d;
  S3BwdGeom g{};
  g.N = d.N; g.Cin = d.Cin; g.H = d.H; g.W = d.W; g.Cout = d.Cout; g.ng = p->ng;
  g.Q = p->host.Q;
  g.tiles = (int)(((long)d.H * (d.W + 2) - 2 + 29) / 30);
  g.ntile = d.N * g.tiles;
  g.nkb = (d.Cout + KS - 1) / KS;
  g.nk = g.Q * g.nkb;
  const int nwg = (g.ntile + NW - 1) / NW, nblk = (d.Cin + 31) / 32;
  const double dx_bytes = 4.0 * d.N * d.Cin * d.H * d.W;
  const double build = 1.4;      // us
  S3BwdPlan best{};
  double best_t = -1;
  for (int per = 1; per <= 2; ++per) {
    const int ncg = (nblk + per - 1) / per;
    const double mul = 54 * 0.019 * per * 2;
    const double kt = std::max(mul, 2 * build) + 0.3;
    for (int s = 1; s <= g.nk && s <= 64; ++s) {
      const int kper = (g.nk + s - 1) / s, ks = (g.nk + kper - 1) / kper;
      if (ks != s || (s > 1 && s * dx_bytes > 268435456.0)) continue;
      const long units = (long)nwg * ncg * s;
      const double t = ((units + 255) / 256) * (kper * kt + 2.0) + (s > 1 ? 6.0 + (s + 1) * dx_bytes / 4.0e6 : 0.0);
      if (best_t < 0 || t < best_t) {
        best_t = t;
        best.TB = per;
        g.ncg = ncg; g.ksplit = s; g.kper = kper; g.units = (int)units;
        best.g = g;
      }
    }
  }
  return best;
}

}  // namespace

// The fp32 instructions only where the launch is too short for the packing of the weights' parts to pay and their blocks of 64
// channels are filled.  Fp32 instructions / bf16 parts on 170 random layers of 12 to 300 rows and columns, from 0.02 GFLOP: up
// to 32 channels never longer on parts (nor, with up to four, below: 1x3 -> 8, 64x64 16 / 13 us); with more, below 0.3 GFLOP,
// 0.8 to 1.2 times the time; above it one layer of 145 took longer (1x96 -> 51, 122x64 26.0 / 27.4 us), the mean 0.62 of the
// time (5x32 -> 384, 262x12 220 / 55, 8x64 -> 64, 32x32 26 / 24, 2x256 -> 256, 32x32 40 / 39).  Odd rows always: the fp32 instructions take them through
// copies to padded rows.  For other turns than quarter turns D is a sum over table entries and the fp32 table kernels stay
// the faster ones (4x128 -> 128, 128x128, 16 turns: 214 / 226).
bool s3_bwd_data_supported(const rotconv_plan* p) {
  if (!p4_bwd_data_layer(p) || p4_bwd_lut(p) || p->opt.bf16_parts < 0) return false;
  const rotconv_desc& d = p->d;
  // a descriptor's size has to stay at or below the offset that stands for "outside"
  if ((size_t)d.Cout * p->ng * d.H * d.W * 4 > kOutside) return false;
  const double flop = s3_bwd_data_flop(p);
  return p->opt.bf16_parts > 0 || (d.W & 1) || d.Cin <= 4 || flop >= (d.Cin <= 32 ? 0.02e9 : 0.3e9);
}

size_t s3_bwd_data_pack_bytes(const rotconv_plan* p) {
  const S3BwdPlan b = s3_bwd_plan(p);
  return (size_t)b.g.ncg * b.TB * b.g.nk * BLK4 * 16;
}

size_t s3_bwd_data_part_floats(const rotconv_plan* p) {
  const S3BwdPlan b = s3_bwd_plan(p);
  return b.g.ksplit > 1 ? (size_t)b.g.ksplit * p->d.N * p->d.Cin * p->d.H * p->d.W : 0;
}

void launch_s3_bwd_data(const rotconv_plan* p, const float* gpool, const uint8_t* idx, const float* w, void* pack,
                        float* dx_out, float* part, hipStream_t st) {
  const S3BwdPlan b = s3_bwd_plan(p);
  const S3BwdGeom& g = b.g;
  const int bpg = b.TB, nblk = g.ncg * bpg;
  const size_t total = (size_t)nblk * g.nk * 256;
  hipLaunchKernelGGL(k_s3_pack_bwd, dim3((unsigned)((total + 255) / 256), 3), dim3(256), 0, st, w,
                     static_cast<uint32_t*>(pack), expand_tables(p), nblk, bpg, g.nk, g.nkb, g.Cin, g.Cout,
                     p->d.dtype == ROTCONV_BF16 ? 1 : 0);
  float* dx = g.ksplit > 1 ? part : dx_out;
  const size_t lds = (size_t)2 * b.TB * BLK4 * 16;
  auto go = [&](auto kern) {
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL(kern, dim3(std::min(256, (g.units + 7) / 8 * 8)), dim3(NT), lds, st, gpool, idx, static_cast<const u32x4*>(pack),
                       p->dev.rot_of, dx, g);
  };
  if (s3_mains_last(p, g.ksplit)) {
    if (b.TB == 1) go(k_s3_bwd_data<1, true>); else go(k_s3_bwd_data<2, true>);
  } else {
    if (b.TB == 1) go(k_s3_bwd_data<1, false>); else go(k_s3_bwd_data<2, false>);
  }
  if (g.ksplit > 1) launch_p4_sum_dx(part, dx_out, (size_t)p->d.N * p->d.Cin * p->d.H * p->d.W, g.ksplit, st);
}

}  // namespace rotconv
