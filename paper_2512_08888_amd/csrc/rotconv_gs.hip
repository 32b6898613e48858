// Matrix-multiply + scatter family (fp32) for the layers the register-resident kernels do not take (k != 3,
// stride != 1, pad != 1, and the unfused gradient calls): the two-step organisation of the paper's Sec. IV on the
// matrix cores.
//
//   forward   P[(q,co,u)][pixel] = sum_ci F_q[co,ci,u] X[ci,pixel]        one GEMM per image, M = Q Cout k^2
//             Y_r[co,yo,xo] = sum_u P[(q,co,u)][yo s + i - pad, xo s + j - pad],  (i,j) = where quarter turn s_r puts
//             base tap u (Eq. 8), then max / arg-max over the pool group (Eq. 10)      -- the scatter, as a gather
//             (P of odd u is stored with its sign turned, see tap_sign)
//   gradients D[(q,co,u)][pixel] = sum_s Delta_(q,s)[co, (y + pad - i)/s, (x + pad - j)/s]   (Eq. 12 routed, or a dense dy)
//             dX = F^T D (one GEMM per image, Eq. 13/15);  dF = D X^T (one GEMM per image, split along the pixels,
//             parts added in order, Eq. 14/16), then the transposed first-quadrant expansion.
//
// The products / routed gradients of a few images at a time live in the workspace (k^2 Q Cout H W floats per image).
// The multiplications are shared by the quarter turns exactly as in the register-resident kernels; what this family
// gives up is their on-chip placement: every product goes through memory once.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdlib>

#include "glue_internal.h"
#include "rotconv_bf16.h"
#include "rotconv_expand.h"
#include "rotconv_gs.h"

namespace rotconv {
namespace {

struct GsGeom {
  int N, Cin, H, W, Cout, k, kk, R, Q, ng, stride, pad, Ho, Wo, relu;
};

GsGeom gs_geom(const rotconv_plan* p) {
  GsGeom g;
  g.N = p->d.N; g.Cin = p->d.Cin; g.H = p->d.H; g.W = p->d.W; g.Cout = p->d.Cout; g.k = p->d.k; g.kk = p->kk;
  g.R = p->d.R; g.Q = p->host.Q; g.ng = p->ng; g.stride = p->d.stride; g.pad = p->d.pad; g.Ho = p->Ho; g.Wo = p->Wo;
  g.relu = 0;
  return g;
}

size_t align256(size_t v) { return (v + 255) / 256 * 256; }

// In the forward the products of every other tap are formed with their sign turned and subtracted where they are placed.  The
// matrix instruction on bf16 parts cuts its sums towards minus infinity, an offset of one sign in each product that would
// grow with the k^2 taps while their sum grows with k: up to 32 channels a product is one such sum (15 x 15 taps, 8
// channels: offset 1.5e-7 of the norm and error 2.96e-7 without the signs, no offset and 2.54e-7 with them, 2.57e-7 on the
// fp32 instruction).
__device__ __forceinline__ constexpr float tap_sign(int u) { return u % 2 ? -1.f : 1.f; }

// base bank(s) -> the GEMM operand [(q, co, u)][ci] (first-quadrant banks, Sec. III-D / Eq. 17); one thread per
// (q, co, ci), every gridDim.y-th of its k^2 taps.  turned: with the signs of the forward
__global__ __launch_bounds__(256) void k_gs_pack(const float* __restrict__ w, float* __restrict__ a, ExpandTables tab, int Q,
                                                 int Cout, int Cin, int kk, int round16, int turned) {
  const int total = Q * Cout * Cin;
  const int e = blockIdx.x * 256 + threadIdx.x;
  if (e >= total) return;
  const int ci = e % Cin, co = (e / Cin) % Cout, q = e / (Cin * Cout);
  const float* src = w + ((size_t)co * Cin + ci) * kk;
  for (int u = blockIdx.y; u < kk; u += gridDim.y)
    a[((size_t)(q * Cout + co) * kk + u) * Cin + ci] =
        (turned ? tap_sign(u) : 1.f) * expand_tap(src, (size_t)Cout * Cin * kk, kk, q, u, true, tab, round16);
}

constexpr int kMaxKK = 225;      // k <= 15

constexpr int TS = 32;           // the tiles of the two kernels below are TS x TS pixels
constexpr int TP = 3;            // taps of products in LDS at a time

// Forward placement (Eq. 8), every orientation (!FUSED) or pooled over all of them (one pool group).  A workgroup places a
// filter's products on a tile of output pixels: the products that the four turns of a bank read there are staged in LDS once,
// TP taps at a time (the next ones' loads on their way meanwhile: one tap at a time waits for them 44 us long), a thread adds
// them up for four pixels of a column and four turns.
// (k_gs_place reads every product once per turn, through bounds of its own each time: 48 us for 32 filters of 5 x 5 taps on
// 2 x 96 x 96 pixels; 33 so.)
template <bool FUSED>
__global__ __launch_bounds__(256) void k_gs_place_tile(const float* __restrict__ P, const int32_t* __restrict__ rot_of,
                                                       const int32_t* __restrict__ turn_tap, float* __restrict__ yout,
                                                       uint8_t* __restrict__ idx, GsGeom g, int n0, int tx, int ext) {
  extern __shared__ float buf[];                         // [2][TP][ext][ext]: rows oy0 * stride - pad on; [4][kk] offsets
  const int oy0 = blockIdx.x / tx * TS, ox0 = blockIdx.x % tx * TS;
  const int co = blockIdx.y, b = blockIdx.z, n = n0 + b;
  const int Pi = g.H * g.W, Po = g.Ho * g.Wo, ext2 = ext * ext, stage = TP * ext2;
  int* off = reinterpret_cast<int*>(buf + 2 * stage);
  for (int i = threadIdx.x; i < 4 * g.kk; i += 256) off[i] = turn_tap[i] / g.k * ext + turn_tap[i] % g.k;
  const int iy0 = oy0 * g.stride - g.pad, ix0 = ox0 * g.stride - g.pad;
  const int lx = threadIdx.x % TS, ly = threadIdx.x / TS;      // pixels (ly + 8 m, lx), m = 0 .. 3
  const int lane_at = (ly * ext + lx) * g.stride, row8 = 8 * g.stride * ext;
  constexpr int NS = 18;                                 // values a thread has on their way
  // where value i of a stage lies behind the stage's first product (-1: outside the image)
  auto place_of = [&](int i) {
    const int tap = i / ext2, e = i - tap * ext2, y = iy0 + e / ext, x = ix0 + e % ext;
    return i < stage && (unsigned)y < (unsigned)g.H && (unsigned)x < (unsigned)g.W ? tap * Pi + y * g.W + x : -1;
  };
  int from[NS];
#pragma unroll
  for (int k = 0; k < NS; ++k) from[k] = place_of(threadIdx.x + 256 * k);
  float best[4] = {0.f, 0.f, 0.f, 0.f};
  int best_r[4] = {-1, -1, -1, -1};
  for (int q = 0; q < g.Q; ++q) {
    const float* Pq = P + ((size_t)b * g.Q * g.Cout + q * g.Cout + co) * g.kk * Pi;
    int rot[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) rot[s] = rot_of[q * 4 + s];
    float acc[4][4];
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int m = 0; m < 4; ++m) acc[s][m] = 0.f;
    float v[NS];
    // what lies outside is read at the stage's first product and dropped when it is written to LDS
    auto load = [&](int u0, int e0) {
      const float* src = Pq + (size_t)u0 * Pi;
      const unsigned end = min(g.kk - u0, TP) * Pi;
#pragma unroll
      for (int k = 0; k < NS; ++k) {
        const unsigned at = e0 ? place_of(e0 + threadIdx.x + 256 * k) : from[k];
        v[k] = src[at < end ? at : 0u];
      }
    };
    auto put = [&](float* d, int u0, int e0) {
      const unsigned end = min(g.kk - u0, TP) * Pi;
#pragma unroll
      for (int k = 0; k < NS; ++k) {
        const int i = e0 + threadIdx.x + 256 * k;
        const unsigned at = e0 ? place_of(i) : from[k];
        if (i < stage) d[i] = at < end ? v[k] : 0.f;
      }
    };
    load(0, 0);
    int par = 0;
    for (int u0 = 0; u0 < g.kk; u0 += TP, par ^= 1) {
      float* cur = buf + par * stage;
      put(cur, u0, 0);
      for (int e0 = NS * 256; e0 < stage; e0 += NS * 256) {      // larger filters and strides
        load(u0, e0);
        put(cur, u0, e0);
      }
      __syncthreads();                                   // (the other buffer was read before the last of these)
      if (u0 + TP < g.kk) load(u0 + TP, 0);
#pragma unroll
      for (int t = 0; t < TP; ++t) {                     // a tap beyond the last one reads zeros
        const int u = min(u0 + t, g.kk - 1);
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const float* src = cur + t * ext2 + off[s * g.kk + u] + lane_at;
#pragma unroll
          for (int m = 0; m < 4; ++m) acc[s][m] = src[m * row8] - acc[s][m];      // the taps' signs in turn
        }
      }
    }
    __syncthreads();
    const float sign = tap_sign((g.kk + TP - 1) / TP * TP - 1);      // of the last one
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int r = rot[s];
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        const int oy = oy0 + ly + 8 * m, ox = ox0 + lx;
        if (FUSED) {                                     // ties go to the smallest orientation
          const float v = fmaf(sign, acc[s][m], 0.f);      // (no negative zeros)
          const bool take = (r >= 0) & ((best_r[m] < 0) | (v > best[m]) | ((v == best[m]) & (r < best_r[m])));
          best[m] = take ? v : best[m];
          best_r[m] = take ? r : best_r[m];
        } else if (r >= 0 && oy < g.Ho && ox < g.Wo) {
          yout[(((size_t)n * g.Cout + co) * g.R + r) * Po + oy * g.Wo + ox] = fmaf(sign, acc[s][m], 0.f);
        }
      }
    }
  }
  if (FUSED) {
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const int oy = oy0 + ly + 8 * m, ox = ox0 + lx;
      if (oy >= g.Ho || ox >= g.Wo) continue;
      const size_t o = ((size_t)n * g.Cout + co) * Po + oy * g.Wo + ox;
      const bool dead = g.relu && best[m] <= 0.f;
      yout[o] = dead ? 0.f : best[m];
      idx[o] = dead ? (uint8_t)255 : (uint8_t)best_r[m];
    }
  }
}

// Forward placement (Eq. 8) as a gather over the products of `nb` images, then Eq. 10.  One thread per output pixel
// of a pooled channel (FUSED) or of a filter (all its orientations are written).  The tap offsets of the four
// quarter turns sit in LDS; a product outside the image is read from a valid address and dropped.
template <bool FUSED>
__global__ __launch_bounds__(256) void k_gs_place(const float* __restrict__ P, const int32_t* __restrict__ rq_of_r,
                                                  const int32_t* __restrict__ turn_tap, float* __restrict__ yout,
                                                  uint8_t* __restrict__ idx, GsGeom g, int n0) {
  __shared__ int siy[4 * kMaxKK], six[4 * kMaxKK];
  for (int i = threadIdx.x; i < 4 * g.kk; i += 256) {
    const int t = turn_tap[i];
    siy[i] = t / g.k - g.pad;
    six[i] = t % g.k - g.pad;
  }
  __syncthreads();
  const int Po = g.Ho * g.Wo, Pi = g.H * g.W;
  const int p = blockIdx.x * 256 + threadIdx.x;
  if (p >= Po) return;
  const int oy = (p / g.Wo) * g.stride, ox = (p % g.Wo) * g.stride;
  const int b = blockIdx.z, n = n0 + b;
  const int rstep = FUSED ? g.ng : 1;
  const float* Pb = P + (size_t)b * g.Q * g.Cout * g.kk * Pi;
  const int nchan = FUSED ? g.Cout * g.ng : g.Cout;
  for (int chan = blockIdx.y; chan < nchan; chan += gridDim.y) {
    const int co = FUSED ? chan / g.ng : chan, grp = FUSED ? chan % g.ng : 0;
    float best = 0.f;
    int best_r = -1;
    for (int r = grp; r < g.R; r += rstep) {
      const int rq = rq_of_r[r], q = rq >> 2, s = rq & 3;
      const float* Pq = Pb + (size_t)(q * g.Cout + co) * g.kk * Pi;
      const int* ty = siy + s * g.kk;
      const int* tx = six + s * g.kk;
      float acc = 0.f;
#pragma unroll 4
      for (int u = 0; u < g.kk; ++u) {
        const int yi = oy + ty[u], xi = ox + tx[u];
        const bool ok = (unsigned)yi < (unsigned)g.H && (unsigned)xi < (unsigned)g.W;
        const float v = Pq[(size_t)u * Pi + (ok ? yi * g.W + xi : 0)];
        acc = (ok ? v : 0.f) - acc;      // the taps' signs in turn
      }
      acc = fmaf(tap_sign(g.kk - 1), acc, 0.f);      // (no negative zeros)
      if (FUSED) {
        if (best_r < 0 || acc > best) { best = acc; best_r = r; }
      } else {
        yout[(((size_t)n * g.Cout + co) * g.R + r) * Po + p] = acc;
      }
    }
    if (FUSED) {
      const size_t o = ((size_t)n * g.Cout * g.ng + chan) * Po + p;
      const bool dead = g.relu && best <= 0.f;
      yout[o] = dead ? 0.f : best;
      idx[o] = dead ? (uint8_t)255 : (uint8_t)best_r;
    }
  }
}

// D[(q,co,u)][input pixel] of `nb` images: the gradient reaching input pixel (y, x) through base tap u of bank q,
// summed over the bank's quarter turns.  ROUTED: from the pooled gradient and idx (Eq. 12); else from a dense dy.
// A workgroup takes a tile of input pixels of a (bank, filter): the gradients of the four turns that its taps reach are
// routed into LDS once, on the grid of the input (zero between the outputs of a stride), and a thread adds up four values
// per tap for four pixels of a column.  (Each value read and routed once per tap and turn: 51 us for 32 filters of 5 x 5 taps
// on 2 x 96 x 96 pixels; 20 so, of which 13 are the 59 MB it writes.)
template <bool ROUTED>
__global__ __launch_bounds__(256) void k_gs_route(const float* __restrict__ gsrc, const uint8_t* __restrict__ idx,
                                                  const int32_t* __restrict__ rot_of,
                                                  const int32_t* __restrict__ turn_tap, float* __restrict__ D, GsGeom g,
                                                  int n0, int tx, int ext) {
  extern __shared__ float plane[];                       // [4][ext][ext]: rows y0 + pad - (k - 1) on; [kk][4] offsets
  int* off = reinterpret_cast<int*>(plane + 4 * ext * ext);
  for (int i = threadIdx.x; i < 4 * g.kk; i += 256)
    off[i % g.kk * 4 + i / g.kk] = i / g.kk * ext * ext - (turn_tap[i] / g.k * ext + turn_tap[i] % g.k);
  const int y0 = blockIdx.x / tx * TS, x0 = blockIdx.x % tx * TS;
  const int b = blockIdx.z, n = n0 + b;
  const int Po = g.Ho * g.Wo, Pi = g.H * g.W, ext2 = ext * ext;
  const int ny0 = y0 + g.pad - (g.k - 1), nx0 = x0 + g.pad - (g.k - 1);
  for (int qc = blockIdx.y; qc < g.Q * g.Cout; qc += gridDim.y) {      // qc = q * Cout + co
    const int co = qc % g.Cout, q = qc / g.Cout;
    if (qc != (int)blockIdx.y) __syncthreads();
    int rot[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) rot[s] = rot_of[q * 4 + s];
    for (int e = threadIdx.x; e < ext2; e += 256) {
      const int ny = ny0 + e / ext, nx = nx0 + e % ext;
      int oy = ny, ox = nx;
      bool ok = ny >= 0 && nx >= 0;
      if (g.stride != 1) {
        oy = ny / g.stride; ox = nx / g.stride;
        ok = ok && oy * g.stride == ny && ox * g.stride == nx;
      }
      ok = ok && oy < g.Ho && ox < g.Wo;
      const int o = ok ? oy * g.Wo + ox : 0;
      float v[4];
      int r[4];
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int rs = max(rot[s], 0);
        const size_t at = (ROUTED ? ((size_t)n * g.Cout + co) * g.ng + rs % g.ng : ((size_t)n * g.Cout + co) * g.R + rs) * Po + o;
        v[s] = gsrc[at];
        r[s] = ROUTED ? idx[at] : rot[s];
      }
#pragma unroll
      for (int s = 0; s < 4; ++s) plane[s * ext2 + e] = ok && rot[s] >= 0 && r[s] == rot[s] ? v[s] : 0.f;
    }
    __syncthreads();
    const int lx = threadIdx.x % TS, ly = threadIdx.x / TS;      // pixels (ly + 8 m, lx), m = 0 .. 3
    const int x = x0 + lx;
    float* Dq = D + ((size_t)b * g.Q * g.Cout + qc) * g.kk * Pi + (size_t)(y0 + ly) * g.W + x;
    const float* at = plane + (ly + g.k - 1) * ext + lx + g.k - 1;
#pragma unroll 2
    for (int u = 0; u < g.kk; ++u) {
      float acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const float* src = at + off[u * 4 + s];
#pragma unroll
        for (int m = 0; m < 4; ++m) acc[m] += src[8 * m * ext];
      }
#pragma unroll
      for (int m = 0; m < 4; ++m)
        if (x < g.W && y0 + ly + 8 * m < g.H) Dq[(size_t)u * Pi + (size_t)(8 * m) * g.W] = acc[m];
    }
  }
}

// acc[e] = (first ? 0 : acc[e]) + sum of the parts, ascending.
__global__ __launch_bounds__(256) void k_gs_sum_acc(const float* __restrict__ part, float* __restrict__ acc, size_t n,
                                                    int nparts, int first) {
  const size_t e = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= n) return;
  float s = first ? 0.f : acc[e];
  for (int z = 0; z < nparts; ++z) s += part[(size_t)z * n + e];
  acc[e] = s;
}

// dw[b][co][ci][t] = sum over the transposed first-quadrant expansion's row (b, t) of coef * dF[(q, co, u)][ci]
// (Eq. 16 / the chain rule through Eq. 17), fixed order.
__global__ __launch_bounds__(256) void k_gs_reduce_w(const float* __restrict__ dF, float* __restrict__ dw,
                                                     const int32_t* __restrict__ ptr, const int32_t* __restrict__ col,
                                                     const float* __restrict__ coef, int B, int Cout, int Cin, int kk) {
  const int total = B * Cout * Cin;
  const int e = blockIdx.x * 256 + threadIdx.x;
  if (e >= total) return;
  const int ci = e % Cin, co = (e / Cin) % Cout, b = e / (Cin * Cout);
  for (int t = blockIdx.y; t < kk; t += gridDim.y) {
    float acc = 0.f;
    for (int z = ptr[b * kk + t]; z < ptr[b * kk + t + 1]; ++z) {
      const int q = col[z] / kk, u = col[z] % kk;
      acc += coef[z] * dF[((size_t)(q * Cout + co) * kk + u) * Cin + ci];
    }
    dw[(((size_t)b * Cout + co) * Cin + ci) * kk + t] = acc;
  }
}

// images whose products / routed gradients are held at once: at most 512 MiB of them, at least one image
int chunk_images(const rotconv_plan* p) {
  const double per = 4.0 * p->host.Q * p->d.Cout * p->kk * p->d.H * p->d.W;
  return (int)std::max(1.0, std::min((double)p->d.N, (double)p->gs_chunk_bytes / per));
}

// split of the weight gradient's pixel contraction: enough workgroups to fill the chip, at least 256 pixels each
int bwdw_splitk(const rotconv_plan* p, int nb) {
  const int M = p->host.Q * p->d.Cout * p->kk;
  const long tiles = (long)((M + 127) / 128) * ((p->d.Cin + 127) / 128) * nb;
  const long want = (768 + tiles - 1) / tiles;
  const long cap = std::max(1, p->d.H * p->d.W / 256);
  return (int)std::max(1L, std::min({want, cap, 64L}));
}

struct GsLayout { size_t a, pd, part, dF, total; };
GsLayout gs_layout(const rotconv_plan* p) {
  const size_t M = (size_t)p->host.Q * p->d.Cout * p->kk;
  const int nb = chunk_images(p);
  GsLayout L;
  L.a = 0;
  L.pd = align256(M * p->d.Cin * 4);
  L.part = L.pd + align256((size_t)nb * M * p->d.H * p->d.W * 4);
  L.dF = L.part + align256((size_t)nb * bwdw_splitk(p, nb) * M * p->d.Cin * 4);
  L.total = L.dF + align256(M * p->d.Cin * 4);
  return L;
}

// the taps of a small kernel's threads over blockIdx.y, up to a few hundred workgroups
unsigned tap_groups(unsigned blocks, int kk) { return std::max(1u, std::min((unsigned)kk, 512u / blocks)); }

void pack(const rotconv_plan* p, const float* w, float* a, bool turned, hipStream_t st) {
  const int total = p->host.Q * p->d.Cout * p->d.Cin;
  const unsigned nb = (total + 255) / 256;
  hipLaunchKernelGGL(k_gs_pack, dim3(nb, tap_groups(nb, p->kk)), dim3(256), 0, st, w, a, expand_tables(p), p->host.Q, p->d.Cout,
                     p->d.Cin, p->kk, p->d.dtype == ROTCONV_BF16 ? 1 : 0, turned ? 1 : 0);
}

// The product of a pass (0 forward, 1 input gradient, 2 weight gradient) for nb images.
GemmArgs gemm_args(const rotconv_plan* p, int pass, int nb) {
  const int M = p->host.Q * p->d.Cout * p->kk, Pi = p->d.H * p->d.W, Cin = p->d.Cin;
  const size_t products = (size_t)M * Pi, image = (size_t)Cin * Pi;
  GemmArgs a{};
  a.batch = nb; a.splitk = 1;
  a.parts = p->opt.bf16_parts;
  if (pass == 0) {               // P[m][pixel] = sum_ci A[m][ci] X[ci][pixel]
    a.M = M; a.N = Pi; a.K = Cin; a.lda = Cin; a.ldb = Pi; a.ldc = Pi;
    a.strideB = image; a.strideC = products;
  } else if (pass == 1) {        // dX[ci][pixel] = sum_m A[m][ci] D[m][pixel]
    a.M = Cin; a.N = Pi; a.K = M; a.transA = 1; a.lda = Cin; a.ldb = Pi; a.ldc = Pi;
    a.strideB = products; a.strideC = image;
  } else {                       // dF[m][ci] = sum_pixel D[m][pixel] X[ci][pixel]
    a.M = M; a.N = Cin; a.K = Pi; a.transB = 1; a.lda = Pi; a.ldb = Pi; a.ldc = Cin;
    a.splitk = bwdw_splitk(p, chunk_images(p)); a.strideA = products; a.strideB = image; a.strideC = (size_t)M * Cin;
  }
  return a;
}

void forward(const rotconv_plan* p, bool fused, const float* x, const float* w, float* yout, uint8_t* idx, void* ws,
             hipStream_t st) {
  GsGeom g = gs_geom(p);
  g.relu = fused && p->d.activation == ROTCONV_ACT_RELU;
  const GsLayout L = gs_layout(p);
  char* c = static_cast<char*>(ws);
  float* A = reinterpret_cast<float*>(c + L.a);
  float* P = reinterpret_cast<float*>(c + L.pd);
  pack(p, w, A, true, st);
  const int Pi = g.H * g.W, Po = g.Ho * g.Wo;
  const int nbmax = chunk_images(p);
  for (int n0 = 0; n0 < g.N; n0 += nbmax) {
    const int nb = std::min(nbmax, g.N - n0);
    launch_gemm(gemm_args(p, 0, nb), A, x + (size_t)n0 * g.Cin * Pi, P, st);
    // one pool group (or none), the tiles' products within the LDS of a workgroup
    const int ext = (TS - 1) * g.stride + g.k, tx = (g.Wo + TS - 1) / TS;
    const size_t lds = ((size_t)2 * TP * ext * ext + 4 * g.kk) * sizeof(float);
    if ((!fused || g.ng == 1) && lds <= 163840 && g.Cout <= 65535) {
      dim3 tiles(tx * ((g.Ho + TS - 1) / TS), g.Cout, nb);
      auto go = [&](auto kern) {
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        hipLaunchKernelGGL(kern, tiles, dim3(256), lds, st, P, p->dev.rot_of, p->dev.turn_tap, yout, idx, g, n0, tx, ext);
      };
      if (fused) go(k_gs_place_tile<true>); else go(k_gs_place_tile<false>);
      continue;
    }
    dim3 grid((Po + 255) / 256, std::min(fused ? g.Cout * g.ng : g.Cout, 65535), nb);
    if (fused) hipLaunchKernelGGL(k_gs_place<true>, grid, dim3(256), 0, st, P, p->dev.rq_of_r, p->dev.turn_tap, yout, idx, g, n0);
    else hipLaunchKernelGGL(k_gs_place<false>, grid, dim3(256), 0, st, P, p->dev.rq_of_r, p->dev.turn_tap, yout, idx, g, n0);
  }
}

void route(const rotconv_plan* p, const GsGeom& g, bool routed, const float* gsrc, const uint8_t* idx, float* D, int n0,
           int nb, hipStream_t st) {
  const int ext = TS + g.k - 1, tx = (g.W + TS - 1) / TS;
  const size_t lds = (size_t)4 * (ext * ext + g.kk) * sizeof(float);      // k <= 15: 38 KB
  dim3 grid(tx * ((g.H + TS - 1) / TS), std::min(g.Q * g.Cout, 65535), nb);
  if (routed) hipLaunchKernelGGL(k_gs_route<true>, grid, dim3(256), lds, st, gsrc, idx, p->dev.rot_of, p->dev.turn_tap, D, g, n0, tx, ext);
  else hipLaunchKernelGGL(k_gs_route<false>, grid, dim3(256), lds, st, gsrc, idx, p->dev.rot_of, p->dev.turn_tap, D, g, n0, tx, ext);
}

void backward_data(const rotconv_plan* p, bool routed, const float* gsrc, const uint8_t* idx, const float* w, float* dx,
                   void* ws, hipStream_t st) {
  const GsGeom g = gs_geom(p);
  const GsLayout L = gs_layout(p);
  char* c = static_cast<char*>(ws);
  float* A = reinterpret_cast<float*>(c + L.a);
  float* D = reinterpret_cast<float*>(c + L.pd);
  pack(p, w, A, false, st);
  const int Pi = g.H * g.W;
  const int nbmax = chunk_images(p);
  for (int n0 = 0; n0 < g.N; n0 += nbmax) {
    const int nb = std::min(nbmax, g.N - n0);
    route(p, g, routed, gsrc, idx, D, n0, nb, st);
    launch_gemm(gemm_args(p, 1, nb), A, D, dx + (size_t)n0 * g.Cin * Pi, st);
  }
}

void backward_weight(const rotconv_plan* p, bool routed, const float* x, const float* gsrc, const uint8_t* idx,
                     float* dw, void* ws, hipStream_t st) {
  const GsGeom g = gs_geom(p);
  const GsLayout L = gs_layout(p);
  char* c = static_cast<char*>(ws);
  float* D = reinterpret_cast<float*>(c + L.pd);
  float* part = reinterpret_cast<float*>(c + L.part);
  float* dF = reinterpret_cast<float*>(c + L.dF);
  const int M = g.Q * g.Cout * g.kk, Pi = g.H * g.W;
  const int nbmax = chunk_images(p);
  const size_t nF = (size_t)M * g.Cin;
  for (int n0 = 0; n0 < g.N; n0 += nbmax) {
    const int nb = std::min(nbmax, g.N - n0);
    route(p, g, routed, gsrc, idx, D, n0, nb, st);
    const GemmArgs a = gemm_args(p, 2, nb);
    launch_gemm(a, D, x + (size_t)n0 * g.Cin * Pi, part, st);
    if (nbmax >= g.N) launch_sum_parts(part, dF, nF, nb * a.splitk, nF, st);
    else hipLaunchKernelGGL(k_gs_sum_acc, dim3((unsigned)((nF + 255) / 256)), dim3(256), 0, st, part, dF, nF, nb * a.splitk,
                            n0 == 0 ? 1 : 0);
  }
  const unsigned rb = (p->B * g.Cout * g.Cin + 255) / 256;
  hipLaunchKernelGGL(k_gs_reduce_w, dim3(rb, tap_groups(rb, g.kk)), dim3(256), 0, st, dF, dw, p->dev.fqt_ptr, p->dev.fqt_col,
                     p->dev.fqt_coef, p->B, g.Cout, g.Cin, g.kk);
}

}  // namespace

// Worth it from about a megaflop of products per call (measured: 16 x 16 maps with 8 -> 8 channels and 5 x 5 filters
// already break even); below that the single generic kernel wins on launches.
// Plan option gs = -1 / 1 switches the family off / on for every shape it can run.
bool gs_wanted(const rotconv_plan* p) {
  if (p->d.pool_op == ROTCONV_POOL_AVG) return false;
  if ((double)p->host.Q * p->d.Cout * p->kk * p->d.H * p->d.W * 4.0 > 3.0e9) return false;   // one image's products
  if (p->opt.gs) return p->opt.gs > 0;
  const double flops = 2.0 * p->d.N * p->d.H * p->d.W * p->d.Cin * p->d.Cout * p->kk * p->host.Q;
  return flops >= 1.0e6;
}

// The budget for the products of the images held at once (plan option gs_chunk_mb).
size_t gs_chunk_budget(const rotconv_plan* p) {
  if (p->opt.gs_chunk_mb > 0) return (size_t)p->opt.gs_chunk_mb << 20;
  if (p->opt.gs_chunk_mb < 0) return 0;       // one image at a time
  return (size_t)512 << 20;
}

size_t gs_ws_bytes(const rotconv_plan* p) { return gs_layout(p).total; }

// (the last images may be fewer than the others at a time)
bool gs_on_parts(const rotconv_plan* p, int pass) {
  const int nb = std::min(chunk_images(p), p->d.N), rest = p->d.N % nb;
  return gemm_on_parts(gemm_args(p, pass, nb)) || (rest && gemm_on_parts(gemm_args(p, pass, rest)));
}

void launch_gs_fwd(const rotconv_plan* p, const float* x, const float* w, float* y, void* ws, hipStream_t st) {
  forward(p, false, x, w, y, nullptr, ws, st);
}
void launch_gs_pool_fwd(const rotconv_plan* p, const float* x, const float* w, float* ypool, uint8_t* idx, void* ws,
                        hipStream_t st) {
  forward(p, true, x, w, ypool, idx, ws, st);
}
void launch_gs_bwd_data(const rotconv_plan* p, const float* dy, const float* w, float* dx, void* ws, hipStream_t st) {
  backward_data(p, false, dy, nullptr, w, dx, ws, st);
}
void launch_gs_pool_bwd_data(const rotconv_plan* p, const float* gpool, const uint8_t* idx, const float* w, float* dx,
                             void* ws, hipStream_t st) {
  backward_data(p, true, gpool, idx, w, dx, ws, st);
}
void launch_gs_bwd_weight(const rotconv_plan* p, const float* x, const float* dy, float* dw, void* ws, hipStream_t st) {
  backward_weight(p, false, x, dy, nullptr, dw, ws, st);
}
void launch_gs_pool_bwd_weight(const rotconv_plan* p, const float* x, const float* gpool, const uint8_t* idx, float* dw,
                               void* ws, hipStream_t st) {
  backward_weight(p, true, x, gpool, idx, dw, ws, st);
}

}  // namespace rotconv
