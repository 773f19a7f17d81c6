// Coarse stencil y(s) = sum_dir A_dir(s) x(nbr(s, dir)) on the matrix cores.
//
// Per coarse site the nine d x d complex blocks multiply d x nrhs neighbour
// blocks: a dense contraction over (dir, j), done by one wave per
// (site, 16 right-hand sides).  A is read once, from a fragment-packed copy
// in which every MFMA A-operand of a wave is one contiguous 1 KB chunk; the
// neighbour block is the B operand.  Complex products use real MFMAs:
//   Re y += Re A Re x - Im A Im x,   Im y += Re A Im x + Im A Re x.
// FP64 / FP32: v_mfma_{f64,f32}_16x16x4 (A[i][k]: lane = i%16 + 16 k;
// B[k][n]: lane = n + 16 k; D[i][n]: lane = n + 16 q with row i = 4 q + reg
// for FP32 and i = q + 4 reg for FP64 -- checked on the device).
// BF16 (mixed form): v_mfma_f32_16x16x16 bf16 with FP32 accumulation
// (A: lane holds k = 4 (lane/16) .. +3 of row lane%16; B likewise by column).
// BF16 values are rounded to nearest even from FP32.
#include "mg.h"

#include <type_traits>

namespace mgm {

typedef double d4_t __attribute__((ext_vector_type(4)));
typedef float f4_t __attribute__((ext_vector_type(4)));
typedef short s4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ void coords_c(const LGeom& g, int64_t s, int c[4]) {
  c[0] = (int)(s % g.dims[0]); s /= g.dims[0];
  c[1] = (int)(s % g.dims[1]); s /= g.dims[1];
  c[2] = (int)(s % g.dims[2]); s /= g.dims[2];
  c[3] = (int)s;
}
__device__ __forceinline__ int64_t nbr_c(const LGeom& g, const int c[4], int dir) {
  int cc[4] = {c[0], c[1], c[2], c[3]};
  if (dir > 0) {
    int mu = (dir - 1) & 3;
    cc[mu] += (dir <= 4) ? 1 : -1;
    cc[mu] = (cc[mu] + g.dims[mu]) % g.dims[mu];
  }
  return cc[0] + (int64_t)g.dims[0] * (cc[1] + (int64_t)g.dims[1] * (cc[2] + (int64_t)g.dims[2] * cc[3]));
}

struct MGeo {
  int d, MT, KC64, KC16;
};
static MGeo mgeo(int d) {
  MGeo m;
  m.d = d;
  m.MT = (d + 15) / 16;
  m.KC64 = (d + 3) / 4;
  m.KC16 = (d + 15) / 16;
  return m;
}

size_t mg_mfma_bytes(const CoarseOp& A) {
  MGeo m = mgeo(A.d);
  return (size_t)A.g.V * 9 * m.KC16 * m.MT * 2 * 64 * 4 * sizeof(uint16_t);
}
size_t mg_mfma64_bytes(const CoarseOp& A) {
  MGeo m = mgeo(A.d);
  return (size_t)A.g.V * 9 * m.KC64 * m.MT * 64 * sizeof(double2);
}

__device__ __forceinline__ uint16_t bf16_rne(float f) {
  uint32_t b = __float_as_uint(f);
  if ((b & 0x7fffffffu) > 0x7f800000u) return 0x7fc0;  // NaN
  b += 0x7fffu + ((b >> 16) & 1u);
  return (uint16_t)(b >> 16);
}

// ---------------------------------------------------------------- packing

__global__ void k_pack64(double2* __restrict__ out, const double2* __restrict__ A, LGeom g, MGeo m) {
  int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t per = (int64_t)9 * m.KC64 * m.MT * 64;
  if (e >= g.V * per) return;
  const int64_t s = e / per;
  int64_t q = e % per;
  const int lane = (int)(q % 64); q /= 64;
  const int mt = (int)(q % m.MT); q /= m.MT;
  const int kc = (int)(q % m.KC64);
  const int dir = (int)(q / m.KC64);
  const int i = 16 * mt + (lane & 15), k = 4 * kc + (lane >> 4);
  double2 v = make_double2(0, 0);
  if (i < m.d && k < m.d) v = A[((int64_t)(dir * m.d + i) * m.d + k) * g.V + s];
  out[e] = v;
}

__global__ void k_pack_bf16(uint16_t* __restrict__ out, const double2* __restrict__ A, LGeom g, MGeo m) {
  int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t per = (int64_t)9 * m.KC16 * m.MT * 2 * 64 * 4;
  if (e >= g.V * per) return;
  const int64_t s = e / per;
  int64_t q = e % per;
  const int el = (int)(q % 4); q /= 4;
  const int lane = (int)(q % 64); q /= 64;
  const int part = (int)(q % 2); q /= 2;  // 0: real, 1: imaginary
  const int mt = (int)(q % m.MT); q /= m.MT;
  const int kc = (int)(q % m.KC16);
  const int dir = (int)(q / m.KC16);
  const int i = 16 * mt + (lane & 15), k = 16 * kc + 4 * (lane >> 4) + el;
  float v = 0.0f;
  if (i < m.d && k < m.d) {
    double2 a = A[((int64_t)(dir * m.d + i) * m.d + k) * g.V + s];
    v = (float)(part ? a.y : a.x);
  }
  out[e] = bf16_rne(v);
}

void mg_mfma_pack(Context* c, CoarseOp& A) {
  MGeo m = mgeo(A.d);
  if (A.Abf) {
    int64_t n = A.g.V * 9 * m.KC16 * m.MT * 2 * 64 * 4;
    hipLaunchKernelGGL(k_pack_bf16, dim3(nblocks_for(n, 256)), dim3(256), 0, c->stream, (uint16_t*)A.Abf, A.A64,
                       A.g, m);
    MGM_LAUNCH_CHECK();
  }
}

void mg_mfma64_pack(Context* c, CoarseOp& A) {
  MGeo m = mgeo(A.d);
  int64_t n = A.g.V * 9 * m.KC64 * m.MT * 64;
  hipLaunchKernelGGL(k_pack64, dim3(nblocks_for(n, 256)), dim3(256), 0, c->stream, A.Ap64, A.A64, A.g, m);
  MGM_LAUNCH_CHECK();
}

// ---------------------------------------------------------------- apply

// 16x16x4 MFMA in FP64 or FP32 (same lane layout, one A and one B value per lane)
// Output row of accumulator register j in lane group q = lane/16 (column
// lane%16): FP64 interleaves rows (4 j + q), FP32 keeps them blocked (4 q + j).
struct M64 {
  using R = double;
  using C2 = double2;
  using V4 = d4_t;
  __device__ static V4 mfma(R a, R b, V4 c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
  __device__ static int row(int q, int j) { return 4 * j + q; }
};
struct M32 {
  using R = float;
  using C2 = float2;
  using V4 = f4_t;
  __device__ static V4 mfma(R a, R b, V4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
  __device__ static int row(int q, int j) { return 4 * q + j; }
};

template <class M, int MT, int MAXT = 256>
__global__ __launch_bounds__(MAXT) void k_coarse_mfma4(const typename M::C2* __restrict__ x,
                                                     typename M::C2* __restrict__ y,
                                                     const typename M::C2* __restrict__ Ap, LGeom g, int d, int KC,
                                                     int nrhs, int ntr, int wpb) {
  using R = typename M::R;
  using V4 = typename M::V4;
  using C2 = typename M::C2;
  // one workgroup per site and group of wpb 16-rhs tiles (one wave each):
  // the tiles of a site stream the same A fragments through the CU's caches
  // at the same time
  const int64_t s = blockIdx.x;
  const int nt = blockIdx.y * wpb + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (nt >= ntr) return;
  const int n = lane & 15, kq = lane >> 4;
  const int r = nt * 16 + n;
  const int64_t V = g.V;
  int c[4];
  coords_c(g, s, c);
  V4 yr[MT], yi[MT];
#pragma unroll
  for (int mt = 0; mt < MT; mt++) {
    yr[mt] = (V4){0, 0, 0, 0};
    yi[mt] = (V4){0, 0, 0, 0};
  }
  const C2* As = Ap + (int64_t)s * 9 * KC * MT * 64 + lane;
#pragma unroll 1
  for (int dir = 0; dir < 9; dir++) {
    const int64_t sn = nbr_c(g, c, dir);
    const C2* Ad = As + (int64_t)dir * KC * MT * 64;
#pragma unroll 4
    for (int kc = 0; kc < KC; kc++) {
      const int k = 4 * kc + kq;
      C2 xv = {0, 0};
      if (k < d && r < nrhs) xv = x[((int64_t)k * V + sn) * nrhs + r];
#pragma unroll
      for (int mt = 0; mt < MT; mt++) {
        const C2 a = Ad[(int64_t)(kc * MT + mt) * 64];
        yr[mt] = M::mfma(a.x, xv.x, yr[mt]);
        yr[mt] = M::mfma(-a.y, xv.y, yr[mt]);
        yi[mt] = M::mfma(a.x, xv.y, yi[mt]);
        yi[mt] = M::mfma(a.y, xv.x, yi[mt]);
      }
    }
  }
  if (r < nrhs) {
#pragma unroll
    for (int mt = 0; mt < MT; mt++)
#pragma unroll
      for (int j = 0; j < 4; j++) {
        const int i = 16 * mt + M::row(kq, j);
        if (i < d) y[((int64_t)i * V + s) * nrhs + r] = C2{(R)yr[mt][j], (R)yi[mt][j]};
      }
  }
}

template <int MT, int NT, int MAXT = 256>
__global__ __launch_bounds__(MAXT) void k_coarse_mfma_bf16(const float2* __restrict__ x, float2* __restrict__ y,
                                                         const uint16_t* __restrict__ Ap, LGeom g, int d,
                                                         int nrhs, int ntr, int wpb) {
  // K chunks of 16 = ceil(d / 16) = MT: the chunk loop unrolls completely so
  // every fragment load of a direction is in flight at once
  constexpr int KC = MT;
  // one workgroup per site and group of wpb waves, each wave NT consecutive
  // 16-rhs tiles: a wave loads every A fragment once for its NT tiles, and
  // the waves of a site stream the same fragments through the CU's caches
  const int64_t s = blockIdx.x;
  const int nt0 = (blockIdx.y * wpb + (threadIdx.x >> 6)) * NT;
  const int lane = threadIdx.x & 63;
  if (nt0 >= ntr) return;
  const int n = lane & 15, kq = lane >> 4;
  const int64_t V = g.V;
  int c[4];
  coords_c(g, s, c);
  f4_t yr[NT][MT], yi[NT][MT];
#pragma unroll
  for (int t = 0; t < NT; t++)
#pragma unroll
    for (int mt = 0; mt < MT; mt++) {
      yr[t][mt] = (f4_t){0, 0, 0, 0};
      yi[t][mt] = (f4_t){0, 0, 0, 0};
    }
  const uint16_t* As = Ap + (int64_t)s * 9 * KC * MT * 512 + lane * 4;
#pragma unroll 1
  for (int dir = 0; dir < 9; dir++) {
    const int64_t sn = nbr_c(g, c, dir);
    const uint16_t* Ad = As + (int64_t)dir * KC * MT * 512;
#pragma unroll
    for (int kc = 0; kc < KC; kc++) {
      s4_t ar[MT], ai[MT], nai[MT];
#pragma unroll
      for (int mt = 0; mt < MT; mt++) {
        const uint16_t* f = Ad + (int64_t)(kc * MT + mt) * 512;
        ar[mt] = *(const s4_t*)f;
        ai[mt] = *(const s4_t*)(f + 256);
        nai[mt] = ai[mt] ^ (s4_t){(short)0x8000, (short)0x8000, (short)0x8000, (short)0x8000};
      }
#pragma unroll
      for (int t = 0; t < NT; t++) {
        const int r = (nt0 + t) * 16 + n;
        s4_t br, bi;
#pragma unroll
        for (int el = 0; el < 4; el++) {
          const int k = 16 * kc + 4 * kq + el;
          float2 xv = make_float2(0.f, 0.f);
          if (k < d && r < nrhs) xv = x[((int64_t)k * V + sn) * nrhs + r];
          br[el] = (short)bf16_rne(xv.x);
          bi[el] = (short)bf16_rne(xv.y);
        }
#pragma unroll
        for (int mt = 0; mt < MT; mt++) {
          yr[t][mt] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(ar[mt], br, yr[t][mt], 0, 0, 0);
          yr[t][mt] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(nai[mt], bi, yr[t][mt], 0, 0, 0);
          yi[t][mt] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(ar[mt], bi, yi[t][mt], 0, 0, 0);
          yi[t][mt] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(ai[mt], br, yi[t][mt], 0, 0, 0);
        }
      }
    }
  }
#pragma unroll
  for (int t = 0; t < NT; t++) {
    const int r = (nt0 + t) * 16 + n;
    if (r < nrhs) {
#pragma unroll
      for (int mt = 0; mt < MT; mt++)
#pragma unroll
        for (int j = 0; j < 4; j++) {
          const int i = 16 * mt + 4 * kq + j;
          if (i < d) y[((int64_t)i * V + s) * nrhs + r] = make_float2(yr[t][mt][j], yi[t][mt][j]);
        }
    }
  }
}

// ------------------------------------------------ staged forms (d <= 64)
//
// One workgroup per site (and group of at most eight 16-rhs tiles): the A
// fragments of the site stream through two LDS buffers, copied there by
// direct-to-LDS loads one chunk ahead, so that they are read from memory once
// and from L2 once for all tiles (in the forms above every wave reads
// all of them: seven tiles of a 48-dof site moved 5.5 GB from L2 a launch, 1.3 of
// them needed); the neighbour values of the next chunk are loaded to registers
// meanwhile.  Sites go to the XCDs in contiguous ranges.

// 1 KB (64 lanes x 16 bytes) from global memory to LDS; the wave's own later
// vmcnt wait and a barrier make it visible
__device__ __forceinline__ void load_lds_1k(const void* g, void* l, int lane) {
  __builtin_amdgcn_global_load_lds(
      (const __attribute__((address_space(1))) void*)((const char*)g + lane * 16),
      (__attribute__((address_space(3))) void*)l, 16, 0, 0);
}
__device__ __forceinline__ void wait_vm0() { __builtin_amdgcn_s_waitcnt(0x0f70); }  // vmcnt(0) only

// Lane dir (0..8) of every wave holds that neighbour of s (V < 2^31); a uniform
// dir reads it with one lane read.
__device__ __forceinline__ int lane_nbr(const LGeom& g, int64_t s, int lane) {
  int c[4];
  coords_c(g, s, c);
  return (int)nbr_c(g, c, lane < 9 ? lane : 0);
}
// x at a uniform element offset plus a lane offset in bytes below 4 GiB
template <class C2>
__device__ __forceinline__ C2 ld_at(const C2* x, int64_t uniform, uint32_t lane_bytes) {
  return *reinterpret_cast<const C2*>(reinterpret_cast<const char*>(x + uniform) + lane_bytes);
}

// FP32 / FP64: wave w works on tile w / MS and the w % MS-th part of the MT row
// tiles.  KCH: (direction, k chunk) steps per staged chunk.
template <class M, int MT, int MS, int KCH>
__global__ __launch_bounds__(MS == 1 ? 512 : 1024) void k_coarse_staged4(const typename M::C2* __restrict__ x,
                                                             typename M::C2* __restrict__ y,
                                                             const typename M::C2* __restrict__ Ap, LGeom g, int d,
                                                             int KC, int nrhs, int ntr, int tpb) {
  using R = typename M::R;
  using V4 = typename M::V4;
  using C2 = typename M::C2;
  constexpr int MW = MT / MS;                                 // row tiles per wave
  constexpr int CB = KCH * MT * 64 * (int)sizeof(C2);         // bytes of a staged chunk
  static_assert(MT % MS == 0 && CB % 1024 == 0, "whole tiles per wave, whole 1 KB copies");
  __shared__ __align__(16) char sA[2][CB];
  const int64_t s = xcd_block(blockIdx.x, g.V);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, nw = blockDim.x >> 6;
  const int mh = wave % MS, nt = blockIdx.y * tpb + wave / MS;
  const int n = lane & 15, kq = lane >> 4;
  const bool live = nt < ntr;  // the other waves only stage
  const int r = (live ? nt : ntr - 1) * 16 + n, rl = r < nrhs ? r : nrhs - 1;
  const int64_t V = g.V, vn = V * nrhs;
  const int nb9 = lane_nbr(g, s, lane);
  const bool ragged = (d & 3) != 0;
  const uint32_t off = (uint32_t)((kq * vn + rl) * sizeof(C2)), off0 = (uint32_t)(rl * sizeof(C2));
  const int Q = 9 * KC, nchunk = (Q + KCH - 1) / KCH;
  const char* As = (const char*)(Ap + s * Q * MT * 64);
  const int64_t abytes = (int64_t)Q * MT * 64 * sizeof(C2);
  auto stage = [&](int c) {
    for (int u = wave; u < CB / 1024; u += nw) {
      const int64_t o = (int64_t)c * CB + u * 1024;
      if (o + lane * 16 < abytes) load_lds_1k(As + o, &sA[c & 1][u * 1024], lane);
    }
  };
  stage(0);
  C2 xn[KCH];
  int fd = 0, fk = 0;  // direction and k chunk of the next step to load
  auto fetch = [&]() {
#pragma unroll
    for (int i = 0; i < KCH; i++) {
      // beyond d the last valid row (the fragments are zero there)
      const uint32_t o = ragged && 4 * fk + kq >= d ? off0 : off;
      xn[i] = ld_at(x, 4 * fk * vn + (int64_t)__builtin_amdgcn_readlane(nb9, fd) * nrhs, o);
      if (++fk == KC) {
        fk = 0;
        fd = fd < 8 ? fd + 1 : 8;
      }
    }
  };
  fetch();
  V4 yr[MW], yi[MW];
#pragma unroll
  for (int m = 0; m < MW; m++) {
    yr[m] = (V4){0, 0, 0, 0};
    yi[m] = (V4){0, 0, 0, 0};
  }
#pragma unroll 1
  for (int c = 0; c < nchunk; c++) {
    wait_vm0();
    __syncthreads();  // chunk c staged by every wave; the other buffer consumed
    C2 xv[KCH];
#pragma unroll
    for (int i = 0; i < KCH; i++) xv[i] = xn[i];
    if (ragged) {  // a finite zero: x may hold anything
#pragma unroll
      for (int i = 0; i < KCH; i++)
        if (4 * ((c * KCH + i) % KC) + kq >= d) xv[i] = C2{0, 0};
    }
    if (c + 1 < nchunk) {
      stage(c + 1);
      fetch();
    }
    const C2* A = reinterpret_cast<const C2*>(sA[c & 1]) + mh * MW * 64 + lane;
#pragma unroll
    for (int i = 0; i < KCH; i++) {
      if (c * KCH + i < Q) {
#pragma unroll
        for (int m = 0; m < MW; m++) {
          const C2 a = A[(i * MT + m) * 64];
          yr[m] = M::mfma(a.x, xv[i].x, yr[m]);
          yi[m] = M::mfma(a.x, xv[i].y, yi[m]);
          yr[m] = M::mfma(-a.y, xv[i].y, yr[m]);
          yi[m] = M::mfma(a.y, xv[i].x, yi[m]);
        }
      }
    }
  }
  if (live && r < nrhs) {
#pragma unroll
    for (int m = 0; m < MW; m++)
#pragma unroll
      for (int j = 0; j < 4; j++) {
        const int i = 16 * (mh * MW + m) + M::row(kq, j);
        if (i < d) y[((int64_t)i * V + s) * nrhs + r] = C2{(R)yr[m][j], (R)yi[m][j]};
      }
  }
}

// four FP32 values rounded to nearest even by the conversion instruction
typedef __bf16 bf2_t __attribute__((ext_vector_type(2)));
typedef float fl2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ s4_t bf16x4(float a, float b, float c, float d) {
  const bf2_t lo = __builtin_convertvector((fl2_t){a, b}, bf2_t), hi = __builtin_convertvector((fl2_t){c, d}, bf2_t);
  return __builtin_bit_cast(s4_t, make_uint2(__builtin_bit_cast(uint32_t, lo), __builtin_bit_cast(uint32_t, hi)));
}

// BF16: one tile per wave.  The default up to 64 dof, mostly (8192 sites, 48 dof, 100 rhs:
// 782 -> 488 us, of which the nine neighbour reads from L2 set the pace; 20 rhs 248
// -> 186; 512 sites, 64 dof, 80 rhs 72 -> 37; 256 sites, 16 dof, 25 rhs 9 -> 6).
template <int MT, int KCH>
__global__ __launch_bounds__(512) void k_coarse_staged_bf16(const float2* __restrict__ x, float2* __restrict__ y,
                                                            const uint16_t* __restrict__ Ap, LGeom g, int d, int nrhs,
                                                            int ntr, int tpb) {
  constexpr int Q = 9 * MT, nchunk = Q / KCH, CB = KCH * MT * 1024;
  static_assert(Q % KCH == 0, "whole chunks");
  __shared__ __align__(16) char sA[2][CB];
  const int64_t s = xcd_block(blockIdx.x, g.V);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, nw = blockDim.x >> 6;
  const int nt = blockIdx.y * tpb + wave, n = lane & 15, kq = lane >> 4;
  const bool live = nt < ntr;
  const int r = (live ? nt : ntr - 1) * 16 + n, rl = r < nrhs ? r : nrhs - 1;
  const int64_t V = g.V, vn = V * nrhs;
  const int nb9 = lane_nbr(g, s, lane);
  const bool ragged = (d & 15) != 0;
  const uint32_t off = (uint32_t)((4 * kq * vn + rl) * sizeof(float2));
  const char* As = (const char*)Ap + s * (int64_t)Q * MT * 1024;
  auto stage = [&](int c) {
    for (int u = wave; u < CB / 1024; u += nw) load_lds_1k(As + (int64_t)c * CB + u * 1024, &sA[c & 1][u * 1024], lane);
  };
  stage(0);
  float2 xn[KCH][4];
  auto fetch = [&](int c) {
#pragma unroll
    for (int i = 0; i < KCH; i++) {
      const int q = c * KCH + i, dir = q / MT, kc = q - dir * MT;
      const int64_t xs = (int64_t)__builtin_amdgcn_readlane(nb9, dir) * nrhs + 16 * kc * vn;
      if (ragged && 16 * kc + 16 > d) {  // beyond d the last valid row
#pragma unroll
        for (int el = 0; el < 4; el++) {
          const int k = 4 * kq + el, kl = 16 * kc + k < d ? k : d - 1 - 16 * kc;
          xn[i][el] = ld_at(x, xs, (uint32_t)((kl * vn + rl) * sizeof(float2)));
        }
      } else {
#pragma unroll
        for (int el = 0; el < 4; el++) xn[i][el] = ld_at(x, xs + el * vn, off);
      }
    }
  };
  fetch(0);
  f4_t yr[MT], yi[MT];
#pragma unroll
  for (int m = 0; m < MT; m++) {
    yr[m] = (f4_t){0, 0, 0, 0};
    yi[m] = (f4_t){0, 0, 0, 0};
  }
#pragma unroll 1
  for (int c = 0; c < nchunk; c++) {
    wait_vm0();
    __syncthreads();
    s4_t br[KCH], bi[KCH];
#pragma unroll
    for (int i = 0; i < KCH; i++) {
      if (ragged) {
        const int k0 = 16 * ((c * KCH + i) % MT) + 4 * kq;
#pragma unroll
        for (int el = 0; el < 4; el++)
          if (k0 + el >= d) xn[i][el] = make_float2(0.f, 0.f);
      }
      br[i] = bf16x4(xn[i][0].x, xn[i][1].x, xn[i][2].x, xn[i][3].x);
      bi[i] = bf16x4(xn[i][0].y, xn[i][1].y, xn[i][2].y, xn[i][3].y);
    }
    if (c + 1 < nchunk) {
      stage(c + 1);
      fetch(c + 1);
    }
    const uint16_t* A = reinterpret_cast<const uint16_t*>(sA[c & 1]) + lane * 4;
#pragma unroll
    for (int i = 0; i < KCH; i++)
#pragma unroll
      for (int m = 0; m < MT; m++) {
        const s4_t ar = *(const s4_t*)(A + (i * MT + m) * 512), ai = *(const s4_t*)(A + (i * MT + m) * 512 + 256);
        const s4_t nai = ai ^ (s4_t){(short)0x8000, (short)0x8000, (short)0x8000, (short)0x8000};
        yr[m] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(ar, br[i], yr[m], 0, 0, 0);
        yi[m] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(ar, bi[i], yi[m], 0, 0, 0);
        yr[m] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(nai, bi[i], yr[m], 0, 0, 0);
        yi[m] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(ai, br[i], yi[m], 0, 0, 0);
      }
  }
  if (live && r < nrhs) {
#pragma unroll
    for (int m = 0; m < MT; m++)
#pragma unroll
      for (int j = 0; j < 4; j++) {
        const int i = 16 * m + 4 * kq + j;
        if (i < d) y[((int64_t)i * V + s) * nrhs + r] = make_float2(yr[m][j], yi[m][j]);
      }
  }
}

#define MT_DISPATCH(MTV, ...)                       \
  switch (MTV) {                                    \
    case 1: { constexpr int MTc = 1; __VA_ARGS__; } break; \
    case 2: { constexpr int MTc = 2; __VA_ARGS__; } break; \
    case 3: { constexpr int MTc = 3; __VA_ARGS__; } break; \
    case 4: { constexpr int MTc = 4; __VA_ARGS__; } break; \
    case 5: { constexpr int MTc = 5; __VA_ARGS__; } break; \
    case 6: { constexpr int MTc = 6; __VA_ARGS__; } break; \
    case 7: { constexpr int MTc = 7; __VA_ARGS__; } break; \
    case 8: { constexpr int MTc = 8; __VA_ARGS__; } break; \
    case 9: { constexpr int MTc = 9; __VA_ARGS__; } break; \
    case 10: { constexpr int MTc = 10; __VA_ARGS__; } break; \
    case 11: { constexpr int MTc = 11; __VA_ARGS__; } break; \
    case 12: { constexpr int MTc = 12; __VA_ARGS__; } break; \
    case 13: { constexpr int MTc = 13; __VA_ARGS__; } break; \
    case 14: { constexpr int MTc = 14; __VA_ARGS__; } break; \
    case 15: { constexpr int MTc = 15; __VA_ARGS__; } break; \
    case 16: { constexpr int MTc = 16; __VA_ARGS__; } break; \
    default: throw Error(MGM_ERR_SHAPE, "coarse dof must be <= 256"); \
  }

// the 512-thread shapes and two tiles per wave exist up to eight row tiles
// (their registers)
#define MT_DISPATCH8(MTV, ...)                      \
  switch (MTV) {                                    \
    case 1: { constexpr int MTc = 1; __VA_ARGS__; } break; \
    case 2: { constexpr int MTc = 2; __VA_ARGS__; } break; \
    case 3: { constexpr int MTc = 3; __VA_ARGS__; } break; \
    case 4: { constexpr int MTc = 4; __VA_ARGS__; } break; \
    case 5: { constexpr int MTc = 5; __VA_ARGS__; } break; \
    case 6: { constexpr int MTc = 6; __VA_ARGS__; } break; \
    case 7: { constexpr int MTc = 7; __VA_ARGS__; } break; \
    case 8: { constexpr int MTc = 8; __VA_ARGS__; } break; \
    default: throw Error(MGM_ERR_INVALID_ARG, "coarse shape not built for more than eight row tiles"); \
  }

// Waves (16-rhs tiles) per workgroup of at most 256 threads: 4 by default
// (the autotuner also tries 2 and 1); v indexes the distinct candidates for
// ntr tiles.
static int wpb_of(int ntr, int v) {
  int cand[3] = {std::min(ntr, 4), std::min(ntr, 2), 1}, n = 0, out[3];
  for (int c : cand) {
    bool seen = false;
    for (int k = 0; k < n; k++) seen |= out[k] == c;
    if (!seen) out[n++] = c;
  }
  return out[v < n ? v : 0];
}
static int wpb_count(int ntr) { return ntr >= 4 ? 3 : ntr >= 2 ? 2 : 1; }
// FP64 / FP32 shapes: the wpb_of candidates, then (5 to 8 tiles) every tile
// of a site in one workgroup of up to 512 threads, so that the site's A
// fragments are read from HBM once and shared through the CU's cache
static int shapes4_count(int ntr, int mt) { return wpb_count(ntr) + (ntr > 4 && ntr <= 8 && mt <= 8 ? 1 : 0); }
static int wpb4_of(int ntr, int v) { return v < wpb_count(ntr) ? wpb_of(ntr, v) : ntr; }

// Staged forms: up to 64 dof, lane offsets into x below 4 GiB.  Tiles go in
// groups of at most `cap` per workgroup.
static bool staged_ok(const CoarseOp& A, int nrhs, size_t cb, int lane_rows) {
  return A.d <= 64 && ((double)lane_rows * A.g.V + 1.0) * nrhs * (double)cb < 4294967296.0;
}
static int staged_tpb(int ntr, int cap) {
  const int groups = (ntr + cap - 1) / cap;
  return (ntr + groups - 1) / groups;
}
// launch variants of the FP32 / FP64 form: row tiles split over ms waves
static std::vector<int> staged4_splits(const CoarseOp& A, int nrhs, size_t cb) {
  if (!staged_ok(A, nrhs, cb, 3)) return {};
  switch (mgeo(A.d).MT) {
    case 1: return {1};
    case 2: return {1, 2};
    case 3: return {1};
    default: return {1, 2, 4};
  }
}
// Index of the default among the launch variants (the `ns` forms of one wave
// per tile, then the staged ones).  Staging pays as soon as the tiles of a site
// share it (100 rhs, 48 dof, 8192 sites: FP32 1.84 -> 1.50 ms, FP64 3.50 ->
// 2.95; 80 rhs, 64 dof, 512 sites: FP64 417 -> 259 us; 20 rhs, 48 dof: 530 -> 478, 957
// -> 894), at two tiles with four row tiles split over two waves (20 rhs, 64 dof,
// 8192 sites: FP32 918 -> 823 us).  A single tile is bound by reading the
// fragments where the sites fill the chip (8 rhs, 48 dof, 8192 sites: 298 us against
// 337 staged); with few sites the split over all row tiles shortens the
// chain of a site (4 rhs, 64 dof, 512 sites: FP64 164 -> 88 us, FP32 90 -> 50).
// Times below are repeated launches / a launch after other work, whose fragments come from
// HBM.  More than four tiles in one workgroup leave CUs idle where the sites are half as many
// or fewer: four row tiles are split (100 rhs, 64 dof, 64 sites: FP64 138 / 167 us with one
// wave per tile, 162 / 177 staged, 109 / 114 split, FP32 82 / 116, 95 / 105, 70 / 75), three
// do not split and stay with one wave (48 dof: FP64 88 / 112 and 107 / 122; FP32 on 64 sites
// 42 / 81 and 59 / 68, on 128 58 / 83 and 61 / 69).  One row tile in FP64: the fragments of a
// site are few, and from 2048 sites on (1024 with more than four tiles) the chip is
// full without (16 dof, 20 rhs, 4096 sites: 57 / 83 us, 72 / 94 staged).
static int staged4_default(const CoarseOp& A, int ntr, int ns, const std::vector<int>& splits, bool f64) {
  if (splits.empty()) return 0;
  const int MT = mgeo(A.d).MT;
  const int64_t V = A.g.V, cus = A.ctx->cu_count;
  if (ntr > 4 && MT == 4 && 2 * V <= cus) return ns + (int)splits.size() - 1;
  if (ntr > 4 && MT == 3 && (f64 ? 2 : 4) * V <= cus) return 0;
  if (f64 && MT == 1 && V >= (ntr > 4 ? 1024 : 2048)) return 0;
  if (ntr == 1) return V < 1024 ? ns + (int)splits.size() - 1 : 0;
  return ntr == 2 && MT == 4 ? ns + 1 : ns;
}
// BF16: staged except for a single tile of an even number of row tiles where all sites fit
// the chip at once, about 2048 (24 dof, 4 rhs: 19 / 36 us with one wave per tile, 21 / 37
// staged; 64 dof, 8 rhs 66 / 120 and 67 / 125; on 4096 sites 24 dof, 12 rhs 43 / 75 and
// 36 / 69; 64 dof, 4 rhs on 64 sites 20 / 36 and 22 / 25).
static bool staged_bf16_default(const CoarseOp& A, int ntr) {
  return ntr > 1 || mgeo(A.d).MT % 2 != 0 || A.g.V < 2048 || A.g.V >= 4096;
}
template <class M>
static void launch_staged4(const CoarseOp& A, const typename M::C2* x, typename M::C2* y, const typename M::C2* Ap,
                           int nrhs, int ms) {
  const MGeo m = mgeo(A.d);
  const int ntr = (nrhs + 15) / 16, tpb = staged_tpb(ntr, std::min(8, 16 / ms));
  const dim3 nb((unsigned)A.g.V, (unsigned)((ntr + tpb - 1) / tpb));
  // steps per staged chunk: longer chunks hide more, shorter ones leave LDS for
  // more workgroups (48 dof, 20 rhs: two steps 478 us in FP32 and 894 in FP64,
  // four 523 and 1019; 33 rhs FP32 694 and 644)
  const int kch = m.MT == 1 ? 12 : m.MT == 3 && (ntr == 2 || std::is_same<M, M64>::value) ? 2 : 4;
#define MGM_ST4(T, S, K)                                                                                            \
  if (m.MT == T && ms == S && kch == K)                                                                             \
    hipLaunchKernelGGL((k_coarse_staged4<M, T, S, K>), nb, dim3(64 * tpb * S), 0, A.ctx->stream, x, y, Ap, A.g, A.d, \
                       m.KC64, nrhs, ntr, tpb);
  MGM_ST4(1, 1, 12) MGM_ST4(2, 1, 4) MGM_ST4(2, 2, 4) MGM_ST4(3, 1, 2) MGM_ST4(3, 1, 4)
  MGM_ST4(4, 1, 4) MGM_ST4(4, 2, 4) MGM_ST4(4, 4, 4)
#undef MGM_ST4
  MGM_LAUNCH_CHECK();
}

void coarse_apply_mfma64(const CoarseOp& A, const double2* x, double2* y, int nrhs) {
  MGeo m = mgeo(A.d);
  const int ntr = (nrhs + 15) / 16;
  const int ns = shapes4_count(ntr, m.MT);
  const std::vector<int> splits = staged4_splits(A, nrhs, 16);
  ProfScope ps(A.ctx, KC_COARSE_F64, A.bytes(MGM_PREC_F64, nrhs));
  A.ctx->choose("coarse64/" + std::to_string(A.g.V) + "/" + std::to_string(A.d) + "/" + std::to_string(nrhs),
                ns + (int)splits.size(), [&](int v) {
                  MGM_CHECK(v >= 0 && v < ns + (int)splits.size(), MGM_ERR_INVALID_ARG,
                            "coarse launch variant out of range");
                  if (v >= ns) {
                    launch_staged4<M64>(A, x, y, A.Ap64, nrhs, splits[v - ns]);
                    return;
                  }
                  const int wpb = wpb4_of(ntr, v);
                  const dim3 nb((unsigned)A.g.V, (unsigned)((ntr + wpb - 1) / wpb)), tb(64 * wpb);
                  if (wpb > 4) {
                    MT_DISPATCH8(m.MT, hipLaunchKernelGGL((k_coarse_mfma4<M64, MTc, 512>), nb, tb, 0, A.ctx->stream,
                                                         x, y, A.Ap64, A.g, A.d, m.KC64, nrhs, ntr, wpb));
                  } else {
                    MT_DISPATCH(m.MT, hipLaunchKernelGGL((k_coarse_mfma4<M64, MTc>), nb, tb, 0, A.ctx->stream, x,
                                                         y, A.Ap64, A.g, A.d, m.KC64, nrhs, ntr, wpb));
                  }
                  MGM_LAUNCH_CHECK();
                },
                staged4_default(A, ntr, ns, splits, true));
}

void coarse_apply_mfma32(const CoarseOp& A, const float2* x, float2* y, int nrhs) {
  MGeo m = mgeo(A.d);
  const int ntr = (nrhs + 15) / 16;
  const int ns = shapes4_count(ntr, m.MT);
  const std::vector<int> splits = staged4_splits(A, nrhs, 8);
  ProfScope ps(A.ctx, KC_COARSE_F32, A.bytes(MGM_PREC_F32, nrhs));
  A.ctx->choose("coarse32/" + std::to_string(A.g.V) + "/" + std::to_string(A.d) + "/" + std::to_string(nrhs),
                ns + (int)splits.size(), [&](int v) {
                  MGM_CHECK(v >= 0 && v < ns + (int)splits.size(), MGM_ERR_INVALID_ARG,
                            "coarse launch variant out of range");
                  if (v >= ns) {
                    launch_staged4<M32>(A, x, y, A.A32, nrhs, splits[v - ns]);
                    return;
                  }
                  const int wpb = wpb4_of(ntr, v);
                  const dim3 nb((unsigned)A.g.V, (unsigned)((ntr + wpb - 1) / wpb)), tb(64 * wpb);
                  if (wpb > 4) {
                    MT_DISPATCH8(m.MT, hipLaunchKernelGGL((k_coarse_mfma4<M32, MTc, 512>), nb, tb, 0, A.ctx->stream,
                                                         x, y, A.A32, A.g, A.d, m.KC64, nrhs, ntr, wpb));
                  } else {
                    MT_DISPATCH(m.MT, hipLaunchKernelGGL((k_coarse_mfma4<M32, MTc>), nb, tb, 0, A.ctx->stream, x,
                                                         y, A.A32, A.g, A.d, m.KC64, nrhs, ntr, wpb));
                  }
                  MGM_LAUNCH_CHECK();
                },
                staged4_default(A, ntr, ns, splits, false));
}

__global__ void k_pack32(float2* __restrict__ out, const double2* __restrict__ packed64, int64_t n) {
  int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e < n) out[e] = make_float2((float)packed64[e].x, (float)packed64[e].y);
}

size_t mg_mfma32_bytes(const CoarseOp& A) { return mg_mfma64_bytes(A) / 2; }

void mg_mfma32_pack(Context* c, CoarseOp& A) {
  MGeo m = mgeo(A.d);
  int64_t n = A.g.V * 9 * m.KC64 * m.MT * 64;
  hipLaunchKernelGGL(k_pack32, dim3(nblocks_for(n, 256)), dim3(256), 0, c->stream, A.A32, A.Ap64, n);
  MGM_LAUNCH_CHECK();
}

void coarse_apply_mfma(const CoarseOp& A, const float2* x, float2* y, int nrhs) {
  MGM_CHECK(A.Abf != nullptr, MGM_ERR_INVALID_ARG, "BF16 coarse stencil not built (mixed == 0)");
  MGeo m = mgeo(A.d);
  const int ntr = (nrhs + 15) / 16;
  ProfScope ps(A.ctx, KC_COARSE_BF16, A.bytes(MGM_PREC_BF16, nrhs));
  // shapes: one tile per wave with 4 / 2 / 1 waves per workgroup, then two
  // and four tiles per wave (fewer A fragment loads per rhs); with more than
  // four tiles, also every tile of a site in one workgroup of up to 8 waves
  // (one or two tiles per wave), so that the site's A fragments are read
  // from HBM once and shared through the CU's cache
  struct Shape {
    int wpb, nt;
  };
  std::vector<Shape> shapes;
  for (int v = 0; v < wpb_count(ntr); v++) shapes.push_back({wpb_of(ntr, v), 1});
  if (ntr >= 2 && m.MT <= 8) shapes.push_back({1, 2});
  if (ntr >= 4 && m.MT <= 8) shapes.push_back({2, 2});
  if (ntr >= 4 && m.MT <= 3) shapes.push_back({1, 4});
  if (ntr >= 8 && m.MT <= 3) shapes.push_back({2, 4});
  const size_t n_small = shapes.size();
  const int staged = staged_ok(A, nrhs, 8, 16) ? 1 : 0;
  if (ntr > 4 && ntr <= 8 && m.MT <= 8) shapes.push_back({ntr, 1});
  if (ntr > 4 && ntr <= 16 && m.MT <= 4) shapes.push_back({(ntr + 1) / 2, 2});
  A.ctx->choose("coarsebf16/" + std::to_string(A.g.V) + "/" + std::to_string(A.d) + "/" + std::to_string(nrhs),
                (int)shapes.size() + staged, [&](int v) {
                  MGM_CHECK(v >= 0 && v < (int)shapes.size() + staged, MGM_ERR_INVALID_ARG,
                            "coarse launch variant out of range");
                  if (v == (int)shapes.size()) {
                    const int tpb = staged_tpb(ntr, 8);
                    const dim3 nb((unsigned)A.g.V, (unsigned)((ntr + tpb - 1) / tpb)), tb(64 * tpb);
#define MGM_STB(T, K)                                                                                              \
  if (m.MT == T)                                                                                                   \
    hipLaunchKernelGGL((k_coarse_staged_bf16<T, K>), nb, tb, 0, A.ctx->stream, x, y, (const uint16_t*)A.Abf, A.g,   \
                       A.d, nrhs, ntr, tpb);
                    MGM_STB(1, 9) MGM_STB(2, 6) MGM_STB(3, 3) MGM_STB(4, 3)
#undef MGM_STB
                    MGM_LAUNCH_CHECK();
                    return;
                  }
                  const int wpb = shapes[v].wpb, tpw = shapes[v].nt;
                  const int groups = (ntr + tpw - 1) / tpw;
                  const dim3 nb((unsigned)A.g.V, (unsigned)((groups + wpb - 1) / wpb)), tb(64 * wpb);
                  if ((size_t)v >= n_small) {
                    // workgroups of up to 512 threads
                    if (tpw == 1) {
                      MT_DISPATCH8(m.MT, hipLaunchKernelGGL((k_coarse_mfma_bf16<MTc, 1, 512>), nb, tb, 0,
                                                           A.ctx->stream, x, y, (const uint16_t*)A.Abf, A.g, A.d,
                                                           nrhs, ntr, wpb));
                    } else {
                      switch (m.MT) {
                        case 1: hipLaunchKernelGGL((k_coarse_mfma_bf16<1, 2, 512>), nb, tb, 0, A.ctx->stream, x, y,
                                                   (const uint16_t*)A.Abf, A.g, A.d, nrhs, ntr, wpb); break;
                        case 2: hipLaunchKernelGGL((k_coarse_mfma_bf16<2, 2, 512>), nb, tb, 0, A.ctx->stream, x, y,
                                                   (const uint16_t*)A.Abf, A.g, A.d, nrhs, ntr, wpb); break;
                        case 3: hipLaunchKernelGGL((k_coarse_mfma_bf16<3, 2, 512>), nb, tb, 0, A.ctx->stream, x, y,
                                                   (const uint16_t*)A.Abf, A.g, A.d, nrhs, ntr, wpb); break;
                        default: hipLaunchKernelGGL((k_coarse_mfma_bf16<4, 2, 512>), nb, tb, 0, A.ctx->stream, x,
                                                    y, (const uint16_t*)A.Abf, A.g, A.d, nrhs, ntr, wpb); break;
                      }
                    }
                  } else if (tpw == 1) {
                    MT_DISPATCH(m.MT, hipLaunchKernelGGL((k_coarse_mfma_bf16<MTc, 1>), nb, tb, 0, A.ctx->stream, x,
                                                         y, (const uint16_t*)A.Abf, A.g, A.d, nrhs, ntr, wpb));
                  } else if (tpw == 2) {
                    MT_DISPATCH8(m.MT, hipLaunchKernelGGL((k_coarse_mfma_bf16<MTc, 2>), nb, tb, 0, A.ctx->stream, x,
                                                         y, (const uint16_t*)A.Abf, A.g, A.d, nrhs, ntr, wpb));
                  } else {
                    switch (m.MT) {
                      case 1: hipLaunchKernelGGL((k_coarse_mfma_bf16<1, 4>), nb, tb, 0, A.ctx->stream, x, y,
                                                 (const uint16_t*)A.Abf, A.g, A.d, nrhs, ntr, wpb); break;
                      case 2: hipLaunchKernelGGL((k_coarse_mfma_bf16<2, 4>), nb, tb, 0, A.ctx->stream, x, y,
                                                 (const uint16_t*)A.Abf, A.g, A.d, nrhs, ntr, wpb); break;
                      default: hipLaunchKernelGGL((k_coarse_mfma_bf16<3, 4>), nb, tb, 0, A.ctx->stream, x, y,
                                                  (const uint16_t*)A.Abf, A.g, A.d, nrhs, ntr, wpb); break;
                    }
                  }
                  MGM_LAUNCH_CHECK();
                },
                staged && staged_bf16_default(A, ntr) ? (int)shapes.size() : 0);
}

}  // namespace mgm
