// Learned gauge-covariant smoother: parallel-transport convolution (PTC)
// layers out_a = sum_p W_p[a][b] T_p in_b over the identity and the eight
// nearest-neighbour transports, their weight and input gradients, full-batch
// Adam, and the training-pair generation from multigrid solves.
//
// Layout: channel-major like the fine spinors, element
// ((channel * 3 + colour) * V + site) * nrhs + rhs, FP32 complex.
#include "net.h"
#include "fine_dev.h"

#include <chrono>
#include <cmath>
#include <random>

namespace mgm {

// ------------------------------------------------------------ transports
//
// T_p in_b at site s: p = 0 identity, 1 + mu: U_mu(s) in(s + mu); 5 + mu:
// U_mu(s - mu)^H in(s - mu); the hop across the time boundary carries the
// antiperiodic sign.

__device__ __forceinline__ void site_coords(const Geom& g, int64_t s, int c[4]) {
  int64_t q = s;
  c[0] = (int)(q % g.X);
  q /= g.X;
  c[1] = (int)(q % g.Y);
  q /= g.Y;
  c[2] = (int)(q % g.Z);
  c[3] = (int)(q / g.Z);
}

// ------------------------------------------------------- matrix-core forms
//
// The channel mixes run on the FP32 matrix cores.  v_mfma_f32_4x4x1_16b computes
// D[i][n] = A[i] B[n] + D[i][n] for sixteen independent 4 x 4 blocks with one fused
// multiply-add per entry (checked on the device against fmaf, subnormals and
// NaN included), so a chain of them gives bit for bit the sums of the same chain of
// scalar FMAs, at twice their rate.  Lane l holds A row l % 4 and B column
// l % 4 of block l / 4, and the four rows of its own column of D.
typedef float f4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ f4_t mfma4(float a, float b, f4_t c) {
  return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, 0, 0, 0);
}

// out = sum_p W_p T_p in ; W [9][co][ci].  A lane is one element (site, rhs): it
// forms the transport of its own element (the links of a path loaded once for
// all input channels) and supplies it as the B column; the weights of output
// channels a0 + 4 g + l % 4 are the A rows, from an LDS copy in that order.  A
// workgroup computes the 4 NG output channels from a0 = 4 NG blockIdx.y.
// Bound by the lines of the nine neighbour reads (all miss L1) and the matrix
// cores: layers 4-16-16-16-4 on 16^3 x 32 at 4 rhs 1.17 ms (74 TFLOP/s), 3.19 ms
// with scalar FMAs and the links re-read per input channel.  Twelve loads in
// flight per wave; prefetching the next twelve spills or halves the occupancy
// (1.71 ms), and so does one colour per wave (2.2 ms).
template <int NG, class O>
__global__ __launch_bounds__(256) void k_ptc_layer(float2* __restrict__ out, const float2* __restrict__ in,
                                                   const float2* __restrict__ U, const float2* __restrict__ W,
                                                   Geom g, int co, int ci, int nrhs) {
  extern __shared__ __align__(16) float2 sW[];  // [path][input channel][l % 4][g]
  const int a0 = 4 * NG * (int)blockIdx.y;
  for (int i = threadIdx.x; i < kNetPaths * ci * 4 * NG; i += 256) {
    const int gg = i % NG, l4 = (i / NG) % 4, pb = i / (4 * NG), p = pb / ci, b = pb - p * ci;
    sW[i] = W[(p * co + a0 + 4 * gg + l4) * ci + b];
  }
  __syncthreads();
  const int64_t V = g.V, N = V * nrhs;
  const int64_t e = xcd_block(blockIdx.x, gridDim.x) * 256 + threadIdx.x;
  // every lane of a wave supplies weight rows: lanes past the end work on the
  // last element and store nothing
  const int64_t tid = e < N ? e : N - 1;
  const int64_t s = tid / nrhs;
  const int r = (int)(tid - s * nrhs);
  int c[4];
  site_coords(g, s, c);
  f4_t ar[3][NG], ai[3][NG];
#pragma unroll
  for (int cc = 0; cc < 3; cc++)
#pragma unroll
    for (int q = 0; q < NG; q++) ar[cc][q] = ai[cc][q] = (f4_t){0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
  for (int p = 0; p < kNetPaths; p++) {
    int64_t sn = s;
    const bool fwd = p <= 4;
    float ph = 1.f;
    cx<float> u[3][3];  // the transport matrix
    if (p > 0) {
      const int mu = (p - 1) & 3;
      const int cm = mu == 0 ? c[0] : mu == 1 ? c[1] : mu == 2 ? c[2] : c[3];
      const int ex = mu == 0 ? g.X : mu == 1 ? g.Y : mu == 2 ? g.Z : g.T;
      const int64_t sd = mu == 0 ? 1 : mu == 1 ? (int64_t)g.X : mu == 2 ? (int64_t)g.X * g.Y : (int64_t)g.X * g.Y * g.Z;
      const bool wrap = fwd ? (cm == ex - 1) : (cm == 0);
      const int64_t span = (int64_t)(ex - 1) * sd;
      sn = fwd ? (wrap ? s - span : s + sd) : (wrap ? s + span : s - sd);
      ph = (mu == 3 && wrap && g.antiperiodic) ? -1.f : 1.f;
      const uint32_t sl = (uint32_t)(fwd ? s : sn);
#pragma unroll
      for (int cc = 0; cc < 3; cc++)
#pragma unroll
        for (int k = 0; k < 3; k++) {
          const float2 w = link_entry<F32>(U, V, mu, fwd ? 3 * cc + k : 3 * k + cc, sl);
          u[cc][k] = {w.x, fwd ? w.y : -w.y};  // (U^H)_{ak} = conj(U_{ka})
        }
    }
    const O src = ((O)sn * (O)nrhs + (O)r) * (O)sizeof(float2);  // byte offset in a plane
    const float2* wp = sW + (p * ci * 4 + (threadIdx.x & 3)) * NG;
    // four input channels at a time (c_in is a multiple of 4): twelve loads in
    // flight
#pragma unroll 1
    for (int b0 = 0; b0 < ci; b0 += 4) {
      float2 raw[4][3];
#pragma unroll
      for (int j = 0; j < 4; j++)
#pragma unroll
        for (int k = 0; k < 3; k++) raw[j][k] = *at_byte(in + ((b0 + j) * 3 + k) * N, src);
#pragma unroll
      for (int j = 0; j < 4; j++) {
        cx<float> t[3];
        if (p == 0) {
#pragma unroll
          for (int cc = 0; cc < 3; cc++) t[cc] = {raw[j][cc].x, raw[j][cc].y};
        } else {
          cx<float> v[3];
#pragma unroll
          for (int k = 0; k < 3; k++) v[k] = {ph * raw[j][k].x, ph * raw[j][k].y};
#pragma unroll
          for (int cc = 0; cc < 3; cc++) {
            t[cc] = {0.f, 0.f};
#pragma unroll
            for (int k = 0; k < 3; k++) fma_(t[cc], u[cc][k], v[k]);
          }
        }
        float2 w[NG];
#pragma unroll
        for (int q = 0; q < NG; q++) w[q] = wp[(b0 + j) * 4 * NG + q];
        // acc.re += w.re t.re - w.im t.im, acc.im += w.re t.im + w.im t.re, each
        // as two chained products in this order
#pragma unroll
        for (int cc = 0; cc < 3; cc++)
#pragma unroll
          for (int q = 0; q < NG; q++) {
            ar[cc][q] = mfma4(w[q].x, t[cc].re, ar[cc][q]);
            ai[cc][q] = mfma4(w[q].x, t[cc].im, ai[cc][q]);
          }
#pragma unroll
        for (int cc = 0; cc < 3; cc++)
#pragma unroll
          for (int q = 0; q < NG; q++) {
            ar[cc][q] = mfma4(w[q].y, -t[cc].im, ar[cc][q]);
            ai[cc][q] = mfma4(w[q].y, t[cc].re, ai[cc][q]);
          }
      }
    }
  }
  if (e >= N) return;
#pragma unroll
  for (int q = 0; q < NG; q++)
#pragma unroll
    for (int i = 0; i < 4; i++)
#pragma unroll
      for (int cc = 0; cc < 3; cc++)
        out[(int64_t)((a0 + 4 * q + i) * 3 + cc) * N + tid] = make_float2(ar[cc][q][i], ai[cc][q][i]);
}

// Weight gradient of one layer: part[blk][p][a][b] = sum over the block's
// elements of gout_a conj(T_p in_b), summed over colours (grid nblk x 9).
// Elements are summed in tiles of kWE = 32 consecutive ones: within a tile in
// FP32 (element by element, colour by colour, each product pair
// fma(g.re, x.re, g.im x.im) added to the sum), over tiles in FP64.
// A block of four waves stages the gradients and transports of NTB tiles, ES
// elements of each at a time, in LDS; a wave owns output channels 4 ag .. + 3 and
// one set of NTL tiles, and an MFMA covers 4 x 4 pairs of (NTL tiles) x (input
// channel groups).  The loads of a step are in flight during the products of
// the one before.  A 16 x 16 layer of 32768 elements takes 81 us (111 without the
// loads ahead; 566 with two LDS reads for every pair and product); bound by the
// additions of the product pairs, as many vector as matrix cycles.
constexpr int kWE = 32;  // elements per tile
template <int CO, int CI>
struct WgradShape {
  static constexpr int NA = CO / 4, NB = CI / 4;
  static constexpr int NBp = NB <= 2 ? NB : 4;             // input groups per MFMA
  static constexpr int NTL = 16 / NBp;                     // tiles per MFMA
  static constexpr int WPS = NA <= 2 ? NA : 4;             // waves per tile set
  static constexpr int SETS = 4 / WPS, NTB = NTL * SETS;   // tiles per block
  static constexpr int per = (CO + CI) * 3 * NTB * 8;      // LDS bytes per staged element
  static constexpr int ES = per * 18 <= 57344 ? 16 : per * 10 <= 57344 ? 8 : per * 6 <= 57344 ? 4 : 2;
  static constexpr int ESP = ES + 2;  // rows 36 words (20, 12, 8) apart
  static constexpr size_t lds = (size_t)(CO + CI) * 3 * NTB * ESP * 8;
};
template <int CO, int CI>
__global__ __launch_bounds__(256) void k_ptc_wgrad(const float2* __restrict__ gout, const float2* __restrict__ in,
                                                   const float2* __restrict__ U, Geom g, int nrhs,
                                                   int64_t per_block, double2* __restrict__ part) {
  using S = WgradShape<CO, CI>;
  constexpr int ES = S::ES, ESP = S::ESP, NTB = S::NTB, NEL = NTB * ES;
  extern __shared__ __align__(16) float2 smem[];
  float2* sG = smem;                           // [CO * 3][NTB][ESP]
  float2* sX = smem + CO * 3 * NTB * ESP;      // [CI * 3][NTB][ESP]
  const int p = blockIdx.y;
  const int64_t V = g.V, N = V * nrhs;
  const int64_t e0 = (int64_t)blockIdx.x * per_block;
  const int64_t e1 = e0 + per_block < N ? e0 + per_block : N;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int ag = wave % S::WPS, set = wave / S::WPS;  // output group, tile set of this wave
  const int l4 = lane & 3, blk = lane >> 2, bg = blk % S::NBp, tl = blk / S::NBp;
  const bool work = ag < S::NA;  // three output groups: the fourth wave only stages
  const float2* pg = sG + (((work ? 4 * ag : 0) + l4) * 3 * NTB + set * S::NTL + tl) * ESP;
  const float2* px = sX + (((bg < S::NB ? 4 * bg : 0) + l4) * 3 * NTB + set * S::NTL + tl) * ESP;
  const int mu = (p - 1) & 3;
  const bool fwd = p <= 4;
  const int ex = mu == 0 ? g.X : mu == 1 ? g.Y : mu == 2 ? g.Z : g.T;
  const int64_t sd = mu == 0 ? 1 : mu == 1 ? (int64_t)g.X : mu == 2 ? (int64_t)g.X * g.Y : (int64_t)g.X * g.Y * g.Z;
  // staging: GI gradient entries and XI elements (a quarter of their input
  // channels each, sharing the links) per thread
  constexpr int GI = CO * 3 * NEL / 256, XI = 4 * NEL / 256;
  float2 gr[GI], vr[XI][S::NB][3], ur[XI][9];
  float ph[XI];
  auto elem = [&](int64_t k, int q) {  // element of staged slot q in step k
    return e0 + (k / (kWE / ES)) * (NTB * kWE) + (q / ES) * kWE + (k % (kWE / ES)) * ES + q % ES;
  };
  auto load = [&](int64_t k) {
#pragma unroll
    for (int i = 0; i < GI; i++) {
      const int j = t + 256 * i, row = j / NEL;
      const int64_t el = elem(k, j % NEL);
      gr[i] = el < e1 ? gout[(int64_t)row * N + el] : make_float2(0.f, 0.f);
    }
#pragma unroll
    for (int i = 0; i < XI; i++) {
      const int j = t + 256 * i, b0 = j / NEL;
      const int64_t el = elem(k, j % NEL);
      ph[i] = 1.f;
      if (el >= e1) {
#pragma unroll
        for (int b = 0; b < S::NB; b++)
#pragma unroll
          for (int cc = 0; cc < 3; cc++) vr[i][b][cc] = make_float2(0.f, 0.f);
        continue;  // the links of an earlier step times zero
      }
      const float2* src = in + el;
      if (p > 0) {
        const int64_t s = el / nrhs;
        const int r = (int)(el - s * nrhs);
        int c[4];
        site_coords(g, s, c);
        const int cm = mu == 0 ? c[0] : mu == 1 ? c[1] : mu == 2 ? c[2] : c[3];
        const bool wrap = fwd ? (cm == ex - 1) : (cm == 0);
        const int64_t span = (int64_t)(ex - 1) * sd;
        const int64_t sn = fwd ? (wrap ? s - span : s + sd) : (wrap ? s + span : s - sd);
        if (mu == 3 && wrap && g.antiperiodic) ph[i] = -1.f;
        link_load<F32>(U, V, mu, (uint32_t)(fwd ? s : sn), ur[i]);
        src = in + sn * nrhs + r;
      }
#pragma unroll
      for (int b = 0; b < S::NB; b++)
#pragma unroll
        for (int cc = 0; cc < 3; cc++) vr[i][b][cc] = src[(int64_t)((b0 + 4 * b) * 3 + cc) * N];
    }
  };
  auto store = [&]() {
#pragma unroll
    for (int i = 0; i < GI; i++) {
      const int j = t + 256 * i, row = j / NEL, q = j % NEL;
      sG[(row * NTB + q / ES) * ESP + q % ES] = gr[i];
    }
#pragma unroll
    for (int i = 0; i < XI; i++) {
      const int j = t + 256 * i, b0 = j / NEL, q = j % NEL;
      float2* dst = sX + (q / ES) * ESP + q % ES;
#pragma unroll
      for (int b = 0; b < S::NB; b++) {
        cx<float> v[3];
#pragma unroll
        for (int k = 0; k < 3; k++) v[k] = {ph[i] * vr[i][b][k].x, ph[i] * vr[i][b][k].y};
#pragma unroll
        for (int a = 0; a < 3; a++) {
          cx<float> x = {0.f, 0.f};
          if (p == 0) {
            x = v[a];
          } else {
#pragma unroll
            for (int k = 0; k < 3; k++) {
              const float2 w = ur[i][fwd ? 3 * a + k : 3 * k + a];
              fma_(x, cx<float>{w.x, fwd ? w.y : -w.y}, v[k]);  // (U^H)_{ak} = conj(U_{ka})
            }
          }
          dst[((b0 + 4 * b) * 3 + a) * NTB * ESP] = make_float2(x.re, x.im);
        }
      }
    }
  };
#pragma unroll
  for (int i = 0; i < XI; i++)
#pragma unroll
    for (int k = 0; k < 9; k++) ur[i][k] = make_float2(0.f, 0.f);
  double dr[4] = {0, 0, 0, 0}, di[4] = {0, 0, 0, 0};
  f4_t fr = {0.f, 0.f, 0.f, 0.f}, fi = {0.f, 0.f, 0.f, 0.f};
  const f4_t zero = {0.f, 0.f, 0.f, 0.f};
  const int64_t nstep = (e1 - e0 + NTB * kWE - 1) / (NTB * kWE) * (kWE / ES);
  load(0);
#pragma unroll 1
  for (int64_t k = 0; k < nstep; k++) {
    __syncthreads();  // the previous step's tiles consumed
    store();
    __syncthreads();
    if (k + 1 < nstep) load(k + 1);  // in flight during the products
    if (!work) continue;
#pragma unroll 2
    for (int ee = 0; ee < ES; ee += 2) {
      float4 gv[3], xv[3];  // two elements
#pragma unroll
      for (int cc = 0; cc < 3; cc++) {
        gv[cc] = *reinterpret_cast<const float4*>(pg + cc * NTB * ESP + ee);
        xv[cc] = *reinterpret_cast<const float4*>(px + cc * NTB * ESP + ee);
      }
#pragma unroll
      for (int o = 0; o < 2; o++)
#pragma unroll
        for (int cc = 0; cc < 3; cc++) {
          const float gx = o ? gv[cc].z : gv[cc].x, gy = o ? gv[cc].w : gv[cc].y;
          const float xx = o ? xv[cc].z : xv[cc].x, xy = o ? xv[cc].w : xv[cc].y;
          // g conj(x)
          fr += mfma4(gx, xx, mfma4(gy, xy, zero));
          fi += mfma4(gy, xx, mfma4(-gx, xy, zero));
        }
    }
    if ((k + 1) % (kWE / ES) == 0) {
#pragma unroll
      for (int i = 0; i < 4; i++) {
        dr[i] += (double)fr[i];
        di[i] += (double)fi[i];
      }
      fr = fi = zero;
    }
  }
  // tiles of the wave by a fixed shuffle tree, then the sets in order
#pragma unroll
  for (int off = 4 * S::NBp; off < 64; off <<= 1)
#pragma unroll
    for (int i = 0; i < 4; i++) {
      dr[i] += __shfl_xor(dr[i], off, 64);
      di[i] += __shfl_xor(di[i], off, 64);
    }
  __syncthreads();
  double2* sD = reinterpret_cast<double2*>(smem);  // [SETS][CO][CI]
  if (work && tl == 0 && bg < S::NB) {
#pragma unroll
    for (int i = 0; i < 4; i++)
      sD[(set * CO + 4 * ag + i) * CI + 4 * bg + l4] = make_double2(dr[i], di[i]);
  }
  __syncthreads();
  for (int k = t; k < CO * CI; k += 256) {
    double2 a = sD[k];
    for (int q = 1; q < S::SETS; q++) {
      a.x += sD[q * CO * CI + k].x;
      a.y += sD[q * CO * CI + k].y;
    }
    part[((int64_t)blockIdx.x * kNetPaths + p) * CO * CI + k] = a;
  }
}

// out[i] = sum_blk part[blk][i], one 64-lane wave per entry, fixed order
__global__ void k_ptc_wsum(const double2* __restrict__ part, int64_t nblk, int cnt, double2* __restrict__ out) {
  const int i = blockIdx.x;
  double a = 0, b = 0;
  for (int64_t k = threadIdx.x; k < nblk; k += 64) {
    const double2 v = part[k * cnt + i];
    a += v.x;
    b += v.y;
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    a += __shfl_down(a, off, 64);
    b += __shfl_down(b, off, 64);
  }
  if (threadIdx.x == 0) out[i] = make_double2(a, b);
}

// FP32 forward weights and backward weights W'_q = W_{opposite(q)}^H
// FP32 value rounded to the nearest BF16 value (ties to even), kept in FP32
__device__ __forceinline__ float round_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  u = (u + 0x7FFFu + ((u >> 16) & 1u)) & 0xFFFF0000u;
  return __uint_as_float(u);
}

// kernel weights from the master weights: FP32, or BF16-rounded when bf16
// (the layers then multiply BF16 weights and accumulate in FP32)
__global__ void k_ptc_wcopy(const double2* __restrict__ w64, float2* __restrict__ w32, float2* __restrict__ wadj,
                            int co, int ci, int bf16) {
  const int n = kNetPaths * co * ci;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    const int p = i / (co * ci), rem = i % (co * ci), a = rem / ci, b = rem % ci;
    const double2 w = w64[i];
    float wr = (float)w.x, wi = (float)w.y;
    if (bf16) {
      wr = round_bf16(wr);
      wi = round_bf16(wi);
    }
    w32[i] = make_float2(wr, wi);
    const int q = p == 0 ? 0 : (p <= 4 ? p + 4 : p - 4);
    wadj[(q * ci + b) * co + a] = make_float2(wr, -wi);
  }
}

// Adam on real and imaginary parts as separate parameters
__global__ void k_ptc_adam(double2* __restrict__ w, const double2* __restrict__ g, double2* __restrict__ m,
                           double2* __restrict__ v, int64_t n, double lr, double b1, double b2, double eps,
                           double c1, double c2) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const double2 gi = g[i];
    double2 mi = m[i], vi = v[i], wi = w[i];
    mi.x = b1 * mi.x + (1 - b1) * gi.x;
    mi.y = b1 * mi.y + (1 - b1) * gi.y;
    vi.x = b2 * vi.x + (1 - b2) * gi.x * gi.x;
    vi.y = b2 * vi.y + (1 - b2) * gi.y * gi.y;
    wi.x -= lr * (mi.x / c1) / (sqrt(vi.x / c2) + eps);
    wi.y -= lr * (mi.y / c1) / (sqrt(vi.y / c2) + eps);
    m[i] = mi;
    v[i] = vi;
    w[i] = wi;
  }
}

// loss = mean_j n2_j / e2_j and the per-rhs output-gradient scale 2 / (n e2_j)
__global__ void k_ptc_loss(const double* n2, const double* e2, int nrhs, double* scale, double* loss) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  double l = 0;
  for (int j = 0; j < nrhs; j++) {
    const double d = e2[j];
    l += d > 0 ? n2[j] / d : 0.0;
    scale[j] = d > 0 ? 2.0 / (nrhs * d) : 0.0;
  }
  *loss = l / nrhs;
}

// ------------------------------------------------------------------ host

static void launch_layer(Context* c, const FineOp* op, float2* out, const float2* in, const float2* W, int co,
                         int ci, int nrhs) {
  const int64_t N = op->g.V * nrhs;
  ProfScope ps(c, KC_NET, (double)op->g.V * (36.0 * 8 + (co + 9.0 * ci) * 3 * 8 * nrhs));
  const unsigned nb = nblocks_for(N, 256);
  // One workgroup computes all output channels, unless the lattice leaves CUs
  // idle: then the channels are split over workgroups (each repeats the
  // transports) as long as every CU gets at most one.  Network 4-16-16-16-4: 4096
  // elements 170 us whole, 141 in two and 129 in four parts; 32768 184, 154,
  // 160; 262144 571, 731, 1172.
  int ng = co / 4;
  if (ng == 3 && 3u * nb <= (unsigned)c->cu_count) ng = 1;
  while (ng % 2 == 0 && (unsigned)(co / (4 * ng)) * 2u * nb <= (unsigned)c->cu_count) ng /= 2;
  const dim3 grid(nb, co / (4 * ng)), tb(256);
  const size_t lds = (size_t)kNetPaths * ci * 4 * ng * sizeof(float2);
  auto launch = [&](auto* k) {
    hipLaunchKernelGGL(k, grid, tb, lds, c->stream, out, in, op->U32, W, op->g, co, ci, nrhs);
  };
  const bool wide = (double)N * sizeof(float2) > 4294967295.0;  // a channel plane past 32-bit byte offsets
  switch (ng) {
    case 1: launch(wide ? k_ptc_layer<1, int64_t> : k_ptc_layer<1, uint32_t>); break;
    case 2: launch(wide ? k_ptc_layer<2, int64_t> : k_ptc_layer<2, uint32_t>); break;
    case 3: launch(wide ? k_ptc_layer<3, int64_t> : k_ptc_layer<3, uint32_t>); break;
    case 4: launch(wide ? k_ptc_layer<4, int64_t> : k_ptc_layer<4, uint32_t>); break;
    default: throw Error(MGM_ERR_INVALID_ARG, "network widths must be 4, 8, 12 or 16");
  }
  MGM_LAUNCH_CHECK();
}

// blocks per path of the weight gradient: 256 elements each fill the chip
// from 32768 elements on (nine paths)
static int64_t wgrad_blocks(int64_t N) {
  int64_t nb = (N + 255) / 256;
  return nb < 1 ? 1 : (nb > 512 ? 512 : nb);
}

template <int CO, int CI>
static int64_t launch_wgrad_p(Context* c, const FineOp* op, const float2* gout, const float2* in, int nrhs,
                              double2* part) {
  using S = WgradShape<CO, CI>;
  const int64_t N = op->g.V * nrhs, nblk = wgrad_blocks(N), chunk = (int64_t)S::NTB * kWE;
  const int64_t per = ((N + nblk - 1) / nblk + chunk - 1) / chunk * chunk, nb = (N + per - 1) / per;
  const size_t lds = std::max(S::lds, (size_t)S::SETS * CO * CI * sizeof(double2));
  static_assert(S::lds <= 65536, "staged tiles exceed the default LDS of a workgroup");
  hipLaunchKernelGGL((k_ptc_wgrad<CO, CI>), dim3((unsigned)nb, kNetPaths), dim3(256), lds, c->stream, gout, in,
                     op->U32, op->g, nrhs, per, part);
  MGM_LAUNCH_CHECK();
  return nb;
}
// returns the number of block partials written to part[blk][path][co][ci]
static int64_t launch_wgrad(Context* c, const FineOp* op, const float2* gout, const float2* in, int co, int ci,
                            int nrhs, double2* part) {
#define MGM_WGRAD(A, B) \
  if (co == A && ci == B) return launch_wgrad_p<A, B>(c, op, gout, in, nrhs, part);
  MGM_WGRAD(4, 4) MGM_WGRAD(4, 8) MGM_WGRAD(4, 12) MGM_WGRAD(4, 16)
  MGM_WGRAD(8, 4) MGM_WGRAD(8, 8) MGM_WGRAD(8, 12) MGM_WGRAD(8, 16)
  MGM_WGRAD(12, 4) MGM_WGRAD(12, 8) MGM_WGRAD(12, 12) MGM_WGRAD(12, 16)
  MGM_WGRAD(16, 4) MGM_WGRAD(16, 8) MGM_WGRAD(16, 12) MGM_WGRAD(16, 16)
#undef MGM_WGRAD
  throw Error(MGM_ERR_INVALID_ARG, "network widths must be 4, 8, 12 or 16");
}

void Net::layout(Arena& a) {
  L = desc.nlayers;
  nw = 0;
  int wmax = 4, whid = 4;
  for (int l = 0; l <= L; l++) {
    width[l] = desc.width[l];
    wmax = std::max(wmax, width[l]);
    if (l > 0 && l < L) whid = std::max(whid, width[l]);
  }
  for (int l = 0; l < L; l++) {
    woff[l] = nw;
    nw += (int64_t)kNetPaths * width[l + 1] * width[l];
  }
  woff[L] = nw;
  w64 = a.take_n<double2>(nw);
  g64 = a.take_n<double2>(nw);
  m = a.take_n<double2>(nw);
  v = a.take_n<double2>(nw);
  w32 = a.take_n<float2>(nw);
  wadj = a.take_n<float2>(nw);
  const int64_t V = op->g.V;
  const int64_t na = (int64_t)whid * 3 * V * desc.max_nrhs;
  buf[0] = a.take_n<float2>(na);
  buf[1] = a.take_n<float2>(na);
  const int B = desc.train_nrhs;
  if (B > 0) {
    for (int l = 0; l <= L; l++) act[l] = a.take_n<float2>((size_t)width[l] * 3 * V * B);
    gbuf[0] = a.take_n<float2>((size_t)wmax * 3 * V * B);
    gbuf[1] = a.take_n<float2>((size_t)wmax * 3 * V * B);
    tr_e = a.take_n<float2>((size_t)12 * V * B);
    wpart_blocks = wgrad_blocks(V * B);
    wpart = a.take_n<double2>((size_t)wpart_blocks * kNetPaths * kNetMaxWidth * kNetMaxWidth);
    n2 = a.take_n<double>(B);
    e2 = a.take_n<double>(B);
    scale = a.take_n<double>(B);
    loss = a.take_n<double>(1);
    scratch.cap = (size_t)kRedBlocksMax * B;
    scratch.partial = a.take_n<double2>(scratch.cap);
  }
}

void Net::refresh() {
  for (int l = 0; l < L; l++) {
    const int co = width[l + 1], ci = width[l];
    hipLaunchKernelGGL(k_ptc_wcopy, dim3(nblocks_for((int64_t)kNetPaths * co * ci, 256)), dim3(256), 0,
                       ctx->stream, w64 + woff[l], w32 + woff[l], wadj + woff[l], co, ci, desc.bf16_weights ? 1 : 0);
  }
  MGM_LAUNCH_CHECK();
}

void Net::upload_weights(const std::vector<double>& host) {
  MGM_CHECK((int64_t)host.size() == 2 * nw, MGM_ERR_INVALID_ARG, "weight count mismatch");
  MGM_HIP(hipMemcpyAsync(w64, host.data(), sizeof(double2) * nw, hipMemcpyHostToDevice, ctx->stream));
  MGM_HIP(hipMemsetAsync(m, 0, sizeof(double2) * nw, ctx->stream));
  MGM_HIP(hipMemsetAsync(v, 0, sizeof(double2) * nw, ctx->stream));
  adam_step = 0;
  refresh();
  ctx->sync();  // host vector must outlive the copy
}

void Net::apply(const float2* r, float2* y, int nrhs) {
  MGM_CHECK(nrhs >= 1 && nrhs <= desc.max_nrhs, MGM_ERR_INVALID_ARG, "nrhs exceeds the network's max_nrhs");
  for (int l = 0; l < L; l++) {
    const float2* in = l == 0 ? r : buf[(l - 1) & 1];
    float2* out = l == L - 1 ? y : buf[l & 1];
    launch_layer(ctx, op, out, in, w32 + woff[l], width[l + 1], width[l], nrhs);
  }
}

double Net::loss_grad(const float2* r, const float2* e, int nrhs) {
  MGM_CHECK(desc.train_nrhs > 0 && nrhs >= 1 && nrhs <= desc.train_nrhs, MGM_ERR_INVALID_ARG,
            "nrhs exceeds the network's train_nrhs");
  Context* c = ctx;
  const int64_t V = op->g.V;
  auto in_of = [&](int l) { return l == 0 ? r : (const float2*)act[l]; };
  for (int l = 0; l < L; l++) launch_layer(c, op, act[l + 1], in_of(l), w32 + woff[l], width[l + 1], width[l], nrhs);
  // output gradient 2 (N(r) - e) / (n |e|^2), in place of the output
  Vec od;
  od.p = act[L];
  od.nsite = V;
  od.dof = 12;
  od.nrhs = nrhs;
  od.prec = MGM_PREC_F32;
  Vec ev = od.with((void*)e);
  b_axpy(c, nullptr, -1.0, ev, od);
  b_norm2(c, scratch, od, n2);
  b_norm2(c, scratch, ev, e2);
  hipLaunchKernelGGL(k_ptc_loss, dim3(1), dim3(1), 0, c->stream, n2, e2, nrhs, scale, loss);
  MGM_LAUNCH_CHECK();
  b_scale_rhs(c, od, scale);
  const float2* G = act[L];
  for (int l = L - 1; l >= 0; l--) {
    const int co = width[l + 1], ci = width[l];
    const int64_t nb = launch_wgrad(c, op, G, in_of(l), co, ci, nrhs, wpart);
    const int cnt = kNetPaths * co * ci;
    hipLaunchKernelGGL(k_ptc_wsum, dim3(cnt), dim3(64), 0, c->stream, wpart, nb, cnt, g64 + woff[l]);
    MGM_LAUNCH_CHECK();
    if (l > 0) {
      float2* Gn = gbuf[l & 1];
      // input gradient: sum_q T_q (W_{opposite q}^H G), a layer with c_out = ci
      launch_layer(c, op, Gn, G, wadj + woff[l], ci, co, nrhs);
      G = Gn;
    }
  }
  MGM_HIP(hipMemcpyAsync(pinned, loss, sizeof(double), hipMemcpyDeviceToHost, c->stream));
  c->sync();
  return pinned[0];
}

void Net::adam(double lr, double b1, double b2, double eps) {
  adam_step++;
  const double c1 = 1.0 - std::pow(b1, (double)adam_step), c2 = 1.0 - std::pow(b2, (double)adam_step);
  hipLaunchKernelGGL(k_ptc_adam, dim3(nblocks_for(nw, 256)), dim3(256), 0, ctx->stream, w64, g64, m, v, nw, lr, b1,
                     b2, eps, c1, c2);
  MGM_LAUNCH_CHECK();
  refresh();
}

void net_apply(Hier& H, Net& net, Vec r, Vec e) {
  MGM_CHECK(r.prec == MGM_PREC_F32 && e.prec == MGM_PREC_F32, MGM_ERR_INVALID_ARG,
            "the network smoother runs on FP32 vectors (solve kind NET)");
  MGM_CHECK(net.op == H.fine, MGM_ERR_INVALID_ARG, "network and hierarchy belong to different operators");
  net.apply((const float2*)r.p, (float2*)e.p, r.nrhs);
}

void net_train(Hier& H, Net& net, const mgm_train_desc& d, mgm_train_stats* st, double* history) {
  const auto t0 = std::chrono::steady_clock::now();
  const int B = net.desc.train_nrhs;
  MGM_CHECK(B > 0, MGM_ERR_INVALID_ARG, "network was created without training buffers (train_nrhs = 0)");
  MGM_CHECK(net.op == H.fine, MGM_ERR_INVALID_ARG, "network and hierarchy belong to different operators");
  MGM_CHECK(H.L >= 2 && B <= H.cap(0), MGM_ERR_INVALID_ARG, "hierarchy rhs capacity below train_nrhs");
  MGM_CHECK(d.steps >= 1 && d.lr > 0 && d.target_tol > 0, MGM_ERR_INVALID_ARG, "bad training parameters");
  Context* c = H.ctx;
  const int64_t V = H.g[0].V;
  // pairs: z (Z4), e_c = P D_c^-1 P^H z, r = z - D e_c, e = D^-1 r
  double2 *z = H.est.x[0], *ec = H.est.y[0], *rr = H.est.z[0], *ee = H.est.w[0];
  double2 *zc = H.est.x[1], *xc = H.est.y[1];
  draw_z4(c, d.seed, (uint32_t)(256 * 0 + 8), 0, B, V, 12, MGM_PREC_F64, z);
  SolveCfg sc;
  sc.tol = d.target_tol;
  sc.maxiter = 4000;
  sc.kind = MGM_SOLVE_MG;
  sc.smooth = 4;
  sc.coarse_iters = 8;
  MGM_CHECK(H.ws64[0].V != nullptr, MGM_ERR_INVALID_ARG, "training needs FP64 Krylov workspaces (mixed != 1)");
  H.T[0].restrict_(MGM_PREC_F64, z, zc, B);
  SolveOut so1, so0;
  solve(H, 1, sc, zc, xc, B, &so1);
  H.T[0].prolong(MGM_PREC_F64, xc, nullptr, ec, B, 0);
  H.apply(0, MGM_PREC_F64, ec, rr, B);
  Vec zv = H.vec(0, MGM_PREC_F64, z, B);
  b_xpay(c, zv, nullptr, -1.0, zv.with(rr));  // r = z - D e_c
  solve(H, 0, sc, rr, ee, B, &so0);
  MGM_CHECK(so0.converged && so1.converged, MGM_ERR_NOT_CONVERGED, "training-target solves did not converge");
  Vec r32 = H.vec(0, MGM_PREC_F32, net.act[0], B);
  b_copy(c, r32, zv.with(rr));
  b_copy(c, r32.with(net.tr_e), zv.with(ee));
  const double b1 = d.beta1 > 0 ? d.beta1 : 0.9, b2 = d.beta2 > 0 ? d.beta2 : 0.999;
  const double eps = d.eps > 0 ? d.eps : 1e-8;
  double first = 0, last = 0;
  for (int it = 0; it < d.steps; it++) {
    const double l = net.loss_grad(net.act[0], net.tr_e, B);
    MGM_CHECK(std::isfinite(l), MGM_ERR_NUMERIC, "non-finite training loss");
    if (it == 0) first = l;
    last = l;
    if (history) history[it] = l;
    net.adam(d.lr, b1, b2, eps);
  }
  c->sync();
  if (st) {
    st->loss_first = first;
    st->loss_last = last;
    st->steps = d.steps;
    st->seconds = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
  }
}

// initial weights: identity path with a 1/(4 + m0)-like scale on the first
// layer (the inverse of the Wilson diagonal), identity elsewhere, plus small
// Gaussian noise on every entry
std::vector<double> net_initial_weights(const Net& n, uint64_t seed) {
  std::mt19937_64 gen(seed);
  std::normal_distribution<double> nd(0.0, 1.0);
  std::vector<double> w(2 * n.nw, 0.0);
  for (int l = 0; l < n.L; l++) {
    const int co = n.width[l + 1], ci = n.width[l];
    const double noise = 0.01 / std::sqrt((double)kNetPaths * ci);
    for (int p = 0; p < kNetPaths; p++)
      for (int a = 0; a < co; a++)
        for (int b = 0; b < ci; b++) {
          const int64_t i = n.woff[l] + ((int64_t)p * co + a) * ci + b;
          double re = noise * nd(gen), im = noise * nd(gen);
          if (p == 0 && a == b) re += l == 0 ? 0.25 : 1.0;
          w[2 * i] = re;
          w[2 * i + 1] = im;
        }
  }
  return w;
}

}  // namespace mgm
