// Aggregation-based transfers, block orthonormalisation of test vectors and
// the Galerkin coarse stencil (Sec. 2.2: R_l = P_l^H with unitary P_l,
// D_{l+1} = P_l^H D_l P_l).
#include "mg.h"

#include <type_traits>
#include "fine_dev.h"
#include "group.h"

namespace mgm {

// ----------------------------------------------------------------- geometry

LGeom coarse_geom(const LGeom& f, const int b[4], int ntv) {
  LGeom c;
  c.V = 1;
  for (int m = 0; m < 4; m++) {
    c.dims[m] = f.dims[m] / b[m];
    c.V *= c.dims[m];
  }
  c.dof = 2 * ntv;
  return c;
}

TGeom make_tgeom(const LGeom& f, const int b[4], int ntv) {
  TGeom t;
  t.f = f;
  for (int m = 0; m < 4; m++) t.b[m] = b[m];
  t.c = coarse_geom(f, b, ntv);
  t.ntv = ntv;
  t.bvol = b[0] * b[1] * b[2] * b[3];
  t.half = f.dof / 2;
  t.rows = t.bvol * t.half;
  return t;
}

__device__ __forceinline__ void coords_of(const LGeom& g, int64_t s, int c[4]) {
  c[0] = (int)(s % g.dims[0]); s /= g.dims[0];
  c[1] = (int)(s % g.dims[1]); s /= g.dims[1];
  c[2] = (int)(s % g.dims[2]); s /= g.dims[2];
  c[3] = (int)s;
}
__device__ __forceinline__ int64_t index_of(const LGeom& g, const int c[4]) {
  int x = (c[0] + g.dims[0]) % g.dims[0], y = (c[1] + g.dims[1]) % g.dims[1];
  int z = (c[2] + g.dims[2]) % g.dims[2], t = (c[3] + g.dims[3]) % g.dims[3];
  return x + (int64_t)g.dims[0] * (y + (int64_t)g.dims[1] * (z + (int64_t)g.dims[2] * t));
}
// fine site of local index loc inside aggregate a
__device__ __forceinline__ int64_t fine_site(const TGeom& t, int64_t a, int loc) {
  int ca[4], l[4], f[4];
  coords_of(t.c, a, ca);
  l[0] = loc % t.b[0]; loc /= t.b[0];
  l[1] = loc % t.b[1]; loc /= t.b[1];
  l[2] = loc % t.b[2]; loc /= t.b[2];
  l[3] = loc;
  for (int m = 0; m < 4; m++) f[m] = ca[m] * t.b[m] + l[m];
  return index_of(t.f, f);
}
// aggregate and local index of fine site s
__device__ __forceinline__ void agg_of(const TGeom& t, int64_t s, int64_t& a, int& loc) {
  int f[4], ca[4];
  coords_of(t.f, s, f);
  for (int m = 0; m < 4; m++) ca[m] = f[m] / t.b[m];
  a = index_of(t.c, ca);
  loc = (f[0] % t.b[0]) + t.b[0] * ((f[1] % t.b[1]) + t.b[1] * ((f[2] % t.b[2]) + t.b[2] * (f[3] % t.b[3])));
}

// ------------------------------------------------------------- agg map

__global__ void k_agg_map(TGeom t, int64_t* out) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t total = t.c.V * 2 * t.rows;
  if (i >= total) return;
  int row = (int)(i % t.rows);
  int64_t q = i / t.rows;
  int chi = (int)(q % 2);
  int64_t a = q / 2;
  int loc = row / t.half, j = row % t.half;
  int64_t s = fine_site(t, a, loc);
  out[i] = s * t.f.dof + chi * t.half + j;
}

void mg_agg_map(Context* c, const TGeom& t, int64_t* out) {
  int64_t total = t.c.V * 2 * t.rows;
  hipLaunchKernelGGL(k_agg_map, dim3(nblocks_for(total, 256)), dim3(256), 0, c->stream, t, out);
  MGM_LAUNCH_CHECK();
}

// ------------------------------------------------------------ transfers
//
// Both transfers are products with the aggregate's (rows x N_tv) block of P and
// run on the matrix cores: v_mfma 16x16x4 in FP32 or FP64, whose entries are
// chains of fused multiply-adds like the scalar ones (A[i][k]: lane i + 16 k,
// B[k][n]: lane n + 16 k; D[i][n]: lane n + 16 q, register j, row 4 q + j in
// FP32 and 4 j + q in FP64).  An aggregate and chirality is worked on by wpa
// waves of a 256-thread workgroup, four or one (transfer_split).  P streams from
// memory straight into the A operand; workgroups go to the XCDs in contiguous
// ranges, so that aggregates that share lines of the fine vector share an L2, and
// the tiles of one aggregate (right-hand sides, test vectors) follow each other there,
// as they share P and the lines at the ends of their column ranges: FP32
// prolongation of 33 rhs on 16^3 x 32 in 2^4 aggregates, 24 test vectors, 404 us with the
// tiles in separate passes over the lattice, 330 side by side.  Aggregates 4^4, 24 test
// vectors, 20 rhs on 16^3 x 32, first form (scalar FMAs on LDS tiles) -> now:
// restriction FP64 324 -> 259 us, FP32 176 -> 142, FP16 200 -> 50 (277 MB: at the
// rate of a copy); prolongation FP64 393 -> 251, FP32 203 -> 123, FP16 added
// 290 -> 155 (530 MB, 104 us at that rate).

typedef float f4_t __attribute__((ext_vector_type(4)));
typedef double d4_t __attribute__((ext_vector_type(4)));
template <typename R>
struct Mm;
template <>
struct Mm<float> {
  using V4 = f4_t;
  __device__ __forceinline__ static V4 mfma(float a, float b, V4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  __device__ __forceinline__ static int row(int q, int j) { return 4 * q + j; }
};
template <>
struct Mm<double> {
  using V4 = d4_t;
  __device__ __forceinline__ static V4 mfma(double a, double b, V4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  __device__ __forceinline__ static int row(int q, int j) { return 4 * j + q; }
};

// Entry of the fine vector (one rhs, one chirality) that row = loc * half + j of
// aggregate a stands for, j Vf + site(loc), into LDS: half * Vf < 2^32, as a
// level's vectors and operator have to fit the device.
__device__ __forceinline__ void aggregate_rows(const TGeom& t, int64_t a, uint32_t* tab, int i0, int step) {
  int ca[4];
  coords_of(t.c, a, ca);
  for (int row = i0; row < t.rows; row += step) {
    const int loc = row / t.half, j = row - loc * t.half;
    int rem = loc, f[4];
#pragma unroll
    for (int m = 0; m < 4; m++) {
      const int l = rem % t.b[m];
      rem /= t.b[m];
      f[m] = ca[m] * t.b[m] + l;
    }
    tab[row] = (uint32_t)(j * t.f.V + index_of(t.f, f));
  }
}
__host__ __device__ inline int row_words(int rows) { return (rows + 3) & ~3; }

// Tiles of a launch: ny groups of rhs from group y0 on, nz of test vectors.
struct Tiles {
  int ny, nz, y0;
};
struct TileAt {
  int64_t blk;
  int y, z;
};
__device__ __forceinline__ TileAt tile_at(const Tiles& p) {
  uint32_t q = (uint32_t)xcd_block(blockIdx.x, gridDim.x);
  const uint32_t z = q % (uint32_t)p.nz;
  q /= (uint32_t)p.nz;
  const uint32_t y = q % (uint32_t)p.ny;
  return {(int64_t)(q / (uint32_t)p.ny), p.y0 + (int)y, (int)z};
}

// the value of the lane beside this one (l ^ 1)
__device__ __forceinline__ float lane_pair(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0xB1, 0xf, 0xf, true));
}
__device__ __forceinline__ double lane_pair(double v) {
  const int2 a = __builtin_bit_cast(int2, v);
  return __builtin_bit_cast(double, make_int2(__builtin_amdgcn_update_dpp(0, a.x, 0xB1, 0xf, 0xf, true),
                                              __builtin_amdgcn_update_dpp(0, a.y, 0xB1, 0xf, 0xf, true)));
}

// y_c[chi k][a][r] = sum_rows conj(P[a][chi][row][k]) x[chi half + j][site(loc)][r]
// As real products: the test vectors are the A tiles, MT of them from
// 16 MT at.z on, the 2 nr columns (re, im of each rhs side by side) the B
// tiles, NT of them from rhs 8 NT at.y on.  Wave w of wpa sums the row
// quadruples w, w + wpa, ..., four in a chain, the chains then one after the other
// (a chain of a whole share was up to 1.8 times further from FP64 sums), and
// the wpa partial tiles are added in order through LDS.
template <class P, class PM, int MT, int NT>
__global__ __launch_bounds__(256) void k_restrict(const typename P::S* __restrict__ x, typename P::S* __restrict__ yc,
                                                  const typename PM::S* __restrict__ Pm, TGeom t, int nrhs, int wpa,
                                                  Tiles tiles) {
  using R = typename P::R;
  using MM = Mm<R>;
  using V4 = typename MM::V4;
  extern __shared__ __align__(16) char smem[];
  const TileAt at = tile_at(tiles);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, n = lane & 15, kq = lane >> 4;
  const int sub = wave / wpa, w = wave - sub * wpa;  // block of P of this wave, its share of the rows
  const int64_t ac = at.blk * (4 / wpa) + sub;
  const bool live = ac < 2 * t.c.V;
  const int64_t a = live ? ac >> 1 : 0;
  const int chi = live ? (int)(ac & 1) : 0;
  const int K = t.ntv, rows = t.rows;
  const int64_t Vc = t.c.V;
  uint32_t* tab = reinterpret_cast<uint32_t*>(smem) + sub * row_words(rows);
  aggregate_rows(t, a, tab, w * 64 + lane, wpa * 64);
  __syncthreads();
  V4 tot[MT][NT], acc[MT][NT];
#pragma unroll
  for (int m = 0; m < MT; m++)
#pragma unroll
    for (int s = 0; s < NT; s++) tot[m][s] = acc[m][s] = (V4){0, 0, 0, 0};
  const typename PM::S* pb = Pm + ((a * 2 + chi) * rows) * (int64_t)K;
  // This lane's rows of the A tiles and columns of the B tiles.  Loads are
  // unconditional (the last valid test vector or rhs instead of one beyond:
  // those rows and columns of the result are not stored), so that they stay in
  // flight together.
  int ka[MT];
  const typename P::S* xb[NT];
#pragma unroll
  for (int m = 0; m < MT; m++) {
    const int k = 16 * (MT * at.z + m) + n;
    ka[m] = k < K ? k : K - 1;
  }
  const int part = n & 1;
#pragma unroll
  for (int s = 0; s < NT; s++) {
    const int r = 8 * (NT * at.y + s) + (n >> 1);
    xb[s] = x + (int64_t)chi * t.half * t.f.V * nrhs + (r < nrhs ? r : nrhs - 1);
  }
  const int quads = (rows + 3) >> 2;
  // quadruples in flight: four where the registers hold them (1 rhs on 16^3 x 32 in 4^4
  // aggregates, 28 test vectors, FP32 72 us with two, 62 with four)
  constexpr int H = NT == 1 || std::is_same<R, float>::value ? 4 : 2;
  int nchain = 0;  // steps summed in acc
#pragma unroll 1
  for (int u0 = w; u0 < quads; u0 += H * wpa) {
    typename PM::S praw[H][MT];
    typename P::S xraw[H][NT];
    bool in[H];
#pragma unroll
    for (int h = 0; h < H; h++) {
      const int row = 4 * (u0 + h * wpa) + kq;
      in[h] = row < rows;
      const int rw = in[h] ? row : 0;
      const int64_t off = (int64_t)tab[rw] * nrhs;
#pragma unroll
      for (int m = 0; m < MT; m++) praw[h][m] = pb[rw * K + ka[m]];
#pragma unroll
      for (int s = 0; s < NT; s++) xraw[h][s] = xb[s][off];
    }
#pragma unroll
    for (int h = 0; h < H; h++) {
      // conj(P) x: re = Pre xre + Pim xim, im = Pre xim - Pim xre
      R b1[NT], b2[NT];
#pragma unroll
      for (int s = 0; s < NT; s++) {
        const cx<R> v = P::ld(&xraw[h][s], 0);
        b1[s] = part ? v.im : v.re;
        b2[s] = part ? -v.re : v.im;
        if (!in[h]) b1[s] = b2[s] = 0;
      }
#pragma unroll
      for (int m = 0; m < MT; m++) {
        const cx<typename PM::R> v = PM::ld(&praw[h][m], 0);
        const R a1 = in[h] ? (R)v.re : (R)0, a2 = in[h] ? (R)v.im : (R)0;
#pragma unroll
        for (int s = 0; s < NT; s++) acc[m][s] = MM::mfma(a1, b1[s], acc[m][s]);
#pragma unroll
        for (int s = 0; s < NT; s++) acc[m][s] = MM::mfma(a2, b2[s], acc[m][s]);
      }
    }
    if (++nchain == 4 / H || u0 + H * wpa >= quads) {
#pragma unroll
      for (int m = 0; m < MT; m++)
#pragma unroll
        for (int s = 0; s < NT; s++) {
          tot[m][s] += acc[m][s];
          acc[m][s] = (V4){0, 0, 0, 0};
        }
      nchain = 0;
    }
  }
  if (wpa > 1) {
    // [w - 1][MT][NT][lane] partial tiles; the first wave adds them in order
    V4* sT = reinterpret_cast<V4*>(smem + sizeof(uint32_t) * (4 / wpa) * row_words(rows)) +
             sub * (wpa - 1) * MT * NT * 64;
    if (w > 0) {
#pragma unroll
      for (int m = 0; m < MT; m++)
#pragma unroll
        for (int s = 0; s < NT; s++) sT[(((w - 1) * MT + m) * NT + s) * 64 + lane] = tot[m][s];
    }
    __syncthreads();
    if (w > 0) return;
    for (int o = 1; o < wpa; o++)
#pragma unroll
      for (int m = 0; m < MT; m++)
#pragma unroll
        for (int s = 0; s < NT; s++) tot[m][s] += sT[(((o - 1) * MT + m) * NT + s) * 64 + lane];
  }
  if (!live) return;
#pragma unroll
  for (int s = 0; s < NT; s++) {
    const int r = 8 * (NT * at.y + s) + (n >> 1);
    if (r >= nrhs) continue;
#pragma unroll
    for (int m = 0; m < MT; m++)
#pragma unroll
      for (int j = 0; j < 4; j++) {
        const int k = 16 * (MT * at.z + m) + MM::row(kq, j);
        if (k < K)
          reinterpret_cast<R*>(yc)[2 * (((int64_t)(chi * K + k) * Vc + a) * nrhs + r) + part] = tot[m][s][j];
      }
  }
}

// The restriction of FP16 vectors, y_c = xs (P^H x16): products of FP16 operands
// are exact in FP32, so they run on v_mfma_f32_16x16x16_f16 (FP32 sums) without a
// conversion, and the scale is applied to the sums.  Lane (n, kq) holds rows
// 4 kq .. 4 kq + 3 of the sixteen of a step: of test vector and part n (A), of
// rhs n (B).
typedef _Float16 h4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ h4_t pick4(const uint32_t (&v)[4], bool hi) {
  const uint32_t sel = hi ? 0x07060302u : 0x05040100u;  // upper or lower halves of two words
  const uint2 o = make_uint2(__builtin_amdgcn_perm(v[1], v[0], sel), __builtin_amdgcn_perm(v[3], v[2], sel));
  return __builtin_bit_cast(h4_t, o);
}
template <int MT, int NT>
__global__ __launch_bounds__(256) void k_restrict16(const uint32_t* __restrict__ x, float2* __restrict__ yc,
                                                    const uint32_t* __restrict__ Pm, TGeom t, int nrhs, int wpa,
                                                    const double* __restrict__ xs, int xgs, Tiles tiles) {
  extern __shared__ __align__(16) char smem[];
  const TileAt at = tile_at(tiles);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, n = lane & 15, kq = lane >> 4;
  const int sub = wave / wpa, w = wave - sub * wpa;
  const int64_t ac = at.blk * (4 / wpa) + sub;
  const bool live = ac < 2 * t.c.V;
  const int64_t a = live ? ac >> 1 : 0;
  const int chi = live ? (int)(ac & 1) : 0;
  const int K = t.ntv, half = t.half, rows = t.rows;
  const int64_t Vc = t.c.V, Vf = t.f.V;
  uint32_t* tab = reinterpret_cast<uint32_t*>(smem) + sub * row_words(rows);
  aggregate_rows(t, a, tab, w * 64 + lane, wpa * 64);
  __syncthreads();
  f4_t acc[MT][NT];
#pragma unroll
  for (int m = 0; m < MT; m++)
#pragma unroll
    for (int s = 0; s < NT; s++) acc[m][s] = (f4_t){0, 0, 0, 0};
  const uint32_t* pb = Pm + ((a * 2 + chi) * rows) * (int64_t)K;
  int ka[MT], rb[NT];
#pragma unroll
  for (int m = 0; m < MT; m++) {
    const int k = 8 * (MT * at.z + m) + (n >> 1);
    ka[m] = k < K ? k : K - 1;
  }
  const bool im = n & 1;
  const uint32_t flip = im ? 0x80008000u : 0u;
  const uint32_t* xb[NT];
#pragma unroll
  for (int s = 0; s < NT; s++) {
    const int r = 16 * (NT * at.y + s) + n;
    rb[s] = r < nrhs ? r : nrhs - 1;
    xb[s] = x + grouped_index(chi * half * Vf, rb[s], nrhs, xgs, 2 * half * Vf);
  }
  const int nstep = (rows + 15) >> 4;
#pragma unroll 1
  for (int u = w; u < nstep; u += wpa) {
    const int row0 = 16 * u + 4 * kq;
    uint32_t pv[MT][4], xv[NT][4];
#pragma unroll
    for (int e = 0; e < 4; e++) {
      const int rw = row0 + e < rows ? row0 + e : rows - 1;
      const int64_t off = (int64_t)tab[rw] * xgs;
#pragma unroll
      for (int m = 0; m < MT; m++) pv[m][e] = pb[rw * K + ka[m]];
#pragma unroll
      for (int s = 0; s < NT; s++) xv[s][e] = xb[s][off];
    }
    if (16 * u + 16 > rows) {  // last step of a row count not divisible by 16
#pragma unroll
      for (int e = 0; e < 4; e++)
        if (row0 + e >= rows) {
#pragma unroll
          for (int m = 0; m < MT; m++) pv[m][e] = 0;
#pragma unroll
          for (int s = 0; s < NT; s++) xv[s][e] = 0;
        }
    }
    h4_t xr[NT], xi[NT];
#pragma unroll
    for (int s = 0; s < NT; s++) {
      xr[s] = pick4(xv[s], false);
      xi[s] = pick4(xv[s], true);
    }
    // conj(P) x: re = Pre xre + Pim xim, im = -Pim xre + Pre xim
#pragma unroll
    for (int m = 0; m < MT; m++) {
      const uint2 b1 = __builtin_bit_cast(uint2, pick4(pv[m], im));
      const h4_t a1 = __builtin_bit_cast(h4_t, make_uint2(b1.x ^ flip, b1.y ^ flip)), a2 = pick4(pv[m], !im);
#pragma unroll
      for (int s = 0; s < NT; s++) acc[m][s] = __builtin_amdgcn_mfma_f32_16x16x16f16(a1, xr[s], acc[m][s], 0, 0, 0);
#pragma unroll
      for (int s = 0; s < NT; s++) acc[m][s] = __builtin_amdgcn_mfma_f32_16x16x16f16(a2, xi[s], acc[m][s], 0, 0, 0);
    }
  }
  if (wpa > 1) {
    f4_t* sT = reinterpret_cast<f4_t*>(smem + sizeof(uint32_t) * (4 / wpa) * row_words(rows)) +
               sub * (wpa - 1) * MT * NT * 64;
    if (w > 0) {
#pragma unroll
      for (int m = 0; m < MT; m++)
#pragma unroll
        for (int s = 0; s < NT; s++) sT[(((w - 1) * MT + m) * NT + s) * 64 + lane] = acc[m][s];
    }
    __syncthreads();
    if (w > 0) return;
    for (int o = 1; o < wpa; o++)
#pragma unroll
      for (int m = 0; m < MT; m++)
#pragma unroll
        for (int s = 0; s < NT; s++) acc[m][s] += sT[(((o - 1) * MT + m) * NT + s) * 64 + lane];
  }
  if (!live) return;
#pragma unroll
  for (int s = 0; s < NT; s++) {
    const int r = 16 * (NT * at.y + s) + n;
    if (r >= nrhs) continue;
    const float sc = (float)xs[r];
#pragma unroll
    for (int m = 0; m < MT; m++)
#pragma unroll
      for (int j = 0; j < 4; j += 2) {
        const int k = 8 * (MT * at.z + m) + ((4 * kq + j) >> 1);
        if (k < K)
          yc[((int64_t)(chi * K + k) * Vc + a) * nrhs + r] = make_float2(sc * acc[m][s][j], sc * acc[m][s][j + 1]);
      }
  }
}

// y = P x_c (mode 0), x - P x_c (mode 1), y + P x_c (mode 2), or
// xs * x + P x_c (mode 3, x stored as PX, scaled per rhs by xs and in column
// groups of xgs right-hand sides)
// As real products: rows of P are the A tiles, two tiles of 16 at a time per
// wave, the 2 nr columns (re, im of each rhs side by side, nr rhs from
// 8 NT at.y on) the B tiles, from an LDS copy of the aggregate's coarse
// values.  VK consecutive test vectors per A load (4 VK divides N_tv where VK > 1).
// ALL: the entries of P of 32 test vectors (FP64: 16) are loaded together, so that the lines
// of a row are read once before other waves replace them in L1, and their latency is paid
// once (FP16 added, 24 test vectors: 20 rhs on 24^3 x 48 in 4^4 aggregates 742 us to 688, 12 rhs on
// 16^3 x 32 in 2^4 133 to 119, with cold caches 164 to 144); else in steps, with fewer registers: one
// wave an aggregate with four tiles of rhs and more, FP64 three (FP32, 32 rhs on 16^4, 12 test
// vectors, 55 us in steps, 85 with all; FP64 50 rhs 260, 282 with all).
template <class P, class PM, class PX, int NT, int VK, bool ALL>
__global__ __launch_bounds__(256) void k_prolong(const typename P::S* __restrict__ xc, const typename P::S* __restrict__ x,
                                                 typename P::S* __restrict__ y, const typename PM::S* __restrict__ Pm,
                                                 TGeom t, int nrhs, int mode, int wpa,
                                                 const typename PX::S* __restrict__ xq, const double* __restrict__ xs,
                                                 int xgs, Tiles tiles) {
  using R = typename P::R;
  using MM = Mm<R>;
  using V4 = typename MM::V4;
  constexpr int MT = 2, NC = 8 * NT;  // row tiles per step, rhs per workgroup
  extern __shared__ __align__(16) char smem[];
  const TileAt at = tile_at(tiles);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, n = lane & 15, kq = lane >> 4;
  const int sub = wave / wpa, w = wave - sub * wpa;
  const int64_t ac = at.blk * (4 / wpa) + sub;
  const bool live = ac < 2 * t.c.V;
  const int64_t a = live ? ac >> 1 : 0;
  const int chi = live ? (int)(ac & 1) : 0;
  const int K = t.ntv, half = t.half, rows = t.rows, r0 = NC * at.y;
  const int Kp = (K + 4 * VK - 1) / (4 * VK) * (4 * VK);
  const int64_t Vc = t.c.V, Vf = t.f.V;
  uint32_t* tab = reinterpret_cast<uint32_t*>(smem) + sub * row_words(t.rows);
  cx<R>* sC = reinterpret_cast<cx<R>*>(smem + sizeof(uint32_t) * (4 / wpa) * row_words(t.rows)) +
              sub * Kp * NC;  // [Kp][NC] coarse values
  aggregate_rows(t, a, tab, w * 64 + lane, wpa * 64);
  for (int i = w * 64 + lane; i < Kp * NC; i += wpa * 64) {
    const int k = i / NC, r = r0 + i - k * NC;
    cx<R> v = {0, 0};
    if (k < K && r < nrhs) v = P::ld(xc, ((int64_t)(chi * K + k) * Vc + a) * nrhs + r);
    sC[i] = v;
  }
  __syncthreads();
  if (!live) return;
  const typename PM::S* pb = Pm + ((a * 2 + chi) * rows) * (int64_t)K;
  const int part = n & 1;
  // as in the restriction, loads are unconditional: rows and columns beyond the
  // last read the last and are not stored
  R sc[NT];
  int rb[NT];
  int64_t xo[NT];
#pragma unroll
  for (int s = 0; s < NT; s++) {
    const int r = r0 + 8 * s + (n >> 1);
    rb[s] = r < nrhs ? r : nrhs - 1;
    sc[s] = mode == 3 ? (R)xs[rb[s]] : (R)1;
    xo[s] = mode == 3 ? grouped_index(0, rb[s], nrhs, xgs, 2 * half * Vf) : (int64_t)rb[s];
  }
  const typename P::S* src = mode == 1 ? x : y;
  const int ntile = (rows + 15) >> 4;
#pragma unroll 1
  for (int t0 = MT * w; t0 < ntile; t0 += MT * wpa) {
    // The two lanes of a column hold re and im of four rows; each loads and stores whole
    // entries of two of them (rows j = 2 e + part): half the memory instructions
    // of a part each (FP32, 33 rhs on 16^4 in 2^4 aggregates, 28 test vectors, 190 us to 174)
    V4 acc[MT][NT];
    int64_t frow[MT][2];
#pragma unroll
    for (int m = 0; m < MT; m++)
#pragma unroll
      for (int e = 0; e < 2; e++) {
        const int row = 16 * (t0 + m) + MM::row(kq, 2 * e + part), rw = row < rows ? row : rows - 1;
        frow[m][e] = chi * half * Vf + tab[rw];
      }
    if (mode == 0) {
#pragma unroll
      for (int m = 0; m < MT; m++)
#pragma unroll
        for (int s = 0; s < NT; s++) acc[m][s] = (V4){0, 0, 0, 0};
    } else {
      cx<R> v[MT][2][NT];
      if (mode == 3) {
        typename PX::S raw[MT][2][NT];
#pragma unroll
        for (int m = 0; m < MT; m++)
#pragma unroll
          for (int e = 0; e < 2; e++)
#pragma unroll
            for (int s = 0; s < NT; s++) raw[m][e][s] = xq[frow[m][e] * xgs + xo[s]];
#pragma unroll
        for (int m = 0; m < MT; m++)
#pragma unroll
          for (int e = 0; e < 2; e++)
#pragma unroll
            for (int s = 0; s < NT; s++) {
              const cx<typename PX::R> u = PX::ld(&raw[m][e][s], 0);
              v[m][e][s] = {sc[s] * (R)u.re, sc[s] * (R)u.im};
            }
      } else {
        typename P::S raw[MT][2][NT];
#pragma unroll
        for (int m = 0; m < MT; m++)
#pragma unroll
          for (int e = 0; e < 2; e++)
#pragma unroll
            for (int s = 0; s < NT; s++) raw[m][e][s] = src[frow[m][e] * nrhs + xo[s]];
#pragma unroll
        for (int m = 0; m < MT; m++)
#pragma unroll
          for (int e = 0; e < 2; e++)
#pragma unroll
            for (int s = 0; s < NT; s++) {
              const cx<R> u = P::ld(&raw[m][e][s], 0);
              v[m][e][s] = mode == 1 ? cx<R>{-u.re, -u.im} : u;
            }
      }
#pragma unroll
      for (int m = 0; m < MT; m++)
#pragma unroll
        for (int e = 0; e < 2; e++)
#pragma unroll
          for (int s = 0; s < NT; s++) {
            const cx<R> u = v[m][e][s];
            const R other = lane_pair(part ? u.re : u.im);
            acc[m][s][2 * e] = part ? other : u.re;
            acc[m][s][2 * e + 1] = part ? u.im : other;
          }
    }
    // acc holds -x (mode 1), y (mode 2), xs x (mode 3) or 0; the sum over k is
    // added on top and the sign restored for mode 1
    const typename PM::S* pr[MT];
#pragma unroll
    for (int m = 0; m < MT; m++) {
      const int row = 16 * (t0 + m) + n;
      pr[m] = pb + (row < rows ? row : rows - 1) * K;
    }
    constexpr int CK = !ALL ? 4 * VK : std::is_same<R, float>::value ? 32 : 16, U = CK / (4 * VK);
    struct alignas(VK * sizeof(typename PM::S)) Entries {
      typename PM::S v[VK];
    };
#pragma unroll(ALL ? 1 : 2)
    for (int kc = 0; kc < K; kc += CK) {
      Entries raw[MT][U];
#pragma unroll
      for (int u = 0; u < U; u++) {
        if (kc + 4 * VK * u >= K) break;
        const int kl = kc + 4 * VK * u + VK * kq;  // this lane's first test vector
#pragma unroll
        for (int m = 0; m < MT; m++) raw[m][u] = *reinterpret_cast<const Entries*>(pr[m] + (kl < K ? kl : 0));
      }
#pragma unroll
      for (int u = 0; u < U; u++) {
        if (kc + 4 * VK * u >= K) break;
        const int kl = kc + 4 * VK * u + VK * kq;
        const bool in = VK > 1 || kl < K;  // VK > 1 only where 4 VK divides K
#pragma unroll
        for (int e = 0; e < VK; e++) {
          cx<R> pv[MT];
#pragma unroll
          for (int m = 0; m < MT; m++) {
            const cx<typename PM::R> v = PM::ld(raw[m][u].v, e);
            pv[m] = in ? cx<R>{(R)v.re, (R)v.im} : cx<R>{0, 0};
          }
#pragma unroll
          for (int s = 0; s < NT; s++) {
            const cx<R> c = sC[(kl + e) * NC + 8 * s + (n >> 1)];
            const R b1 = part ? c.im : c.re, b2 = part ? c.re : -c.im;
#pragma unroll
            for (int m = 0; m < MT; m++) acc[m][s] = MM::mfma(pv[m].re, b1, acc[m][s]);
#pragma unroll
            for (int m = 0; m < MT; m++) acc[m][s] = MM::mfma(pv[m].im, b2, acc[m][s]);
          }
        }
      }
    }
#pragma unroll
    for (int m = 0; m < MT; m++)
#pragma unroll
      for (int e = 0; e < 2; e++) {
        const bool row_in = 16 * (t0 + m) + MM::row(kq, 2 * e + part) < rows;
#pragma unroll
        for (int s = 0; s < NT; s++) {
          const R a = acc[m][s][2 * e], b = acc[m][s][2 * e + 1], other = lane_pair(part ? a : b);
          const cx<R> v = part ? cx<R>{other, b} : cx<R>{a, other};
          if (row_in && r0 + 8 * s + (n >> 1) < nrhs)
            P::st(y, frow[m][e] * nrhs + rb[s], mode == 1 ? cx<R>{-v.re, -v.im} : v);
        }
      }
  }
}

double Transfer::bytes(mgm_prec p, int nrhs) const {
  double w = (double)prec_bytes(p);
  return (double)t.c.V * 2 * t.rows * t.ntv * w + (double)t.f.V * t.f.dof * nrhs * w +
         (double)t.c.V * t.c.dof * nrhs * w;
}

static void check_transfer(const TGeom& t) {
  MGM_CHECK(t.ntv <= 128 && t.bvol <= 1024 && t.rows <= 4096, MGM_ERR_SHAPE,
            "transfers support at most 128 test vectors and 1024 sites per aggregate");
}

// Waves per aggregate and chirality (one or four), and tiles of rhs per workgroup.  One
// wave where the rows are few (2^4 aggregates of the fine level have 96, six steps of
// four waves: FP16 restriction, 12 test vectors, 12 rhs on 16^4, 20 us with one, 26 with
// four), in even groups of at most one_max tiles, if a CU gets cu_waves waves; else four
// (8 test vectors on 4^4, FP64 restriction of 33 rhs 15.7 us with one, 7.4 with four; 40 test
// vectors in 2^3 x 4 aggregates on 8^4, FP32 restriction of one 15.5 and 9.6), in even groups of
// at most four_max tiles, or of fewer until every CU has a workgroup (24 test vectors, 16
// aggregates 4^4, FP64 restriction of 33 rhs 75 us with three tiles, 32 with one).
struct TransferSplit {
  int wpa, nt;
};
static TransferSplit transfer_split(const Context* c, const TGeom& t, int tiles, int one_max, int four_max,
                                    int cu_waves) {
  auto groups = [&](int nt) { return (tiles + nt - 1) / nt; };
  auto even = [&](int most) { return groups(groups(most)); };
  const int one = even(one_max);
  if (t.rows < 256 && 2 * t.c.V * groups(one) >= (int64_t)cu_waves * c->cu_count) return {1, one};
  int nt = even(four_max);
  while (nt > 1 && 2 * t.c.V * groups(nt) < c->cu_count) nt--;
  return {4, nt};
}
// one launch, or several of whole rhs groups where one would pass 2^31 threads
template <class F>
static void launch_tiles(int64_t blocks, int ny, int nz, F launch) {
  const int most = (int)std::max<int64_t>(1, (1 << 23) / (blocks * nz));
  for (int y0 = 0; y0 < ny; y0 += most) {
    const Tiles p{std::min(most, ny - y0), nz, y0};
    launch(dim3((unsigned)(blocks * p.ny * nz)), p);
    MGM_LAUNCH_CHECK();
  }
}
static int64_t transfer_blocks(const TGeom& t, int wpa) { return (2 * t.c.V * wpa + 3) / 4; }

template <class P, class PM, int MT, int NT>
static void launch_restrict_nt(Context* c, const TGeom& t, const typename P::S* x, typename P::S* yc,
                               const typename PM::S* Pm, int nrhs, int wpa) {
  const size_t lds = sizeof(uint32_t) * (4 / wpa) * row_words(t.rows) +
                     (size_t)(4 / wpa) * (wpa - 1) * MT * NT * 64 * sizeof(typename Mm<typename P::R>::V4);
  launch_tiles(transfer_blocks(t, wpa), (nrhs + 8 * NT - 1) / (8 * NT), (t.ntv + 16 * MT - 1) / (16 * MT),
               [&](dim3 nb, Tiles p) {
                 hipLaunchKernelGGL((k_restrict<P, PM, MT, NT>), nb, dim3(256), lds, c->stream, x, yc, Pm, t, nrhs,
                                    wpa, p);
               });
}
// Tiles of rhs.  FP64: up to three whole, more one by one, whose registers hold four
// quadruples in flight (12 test vectors on 16^4 in 2^4 aggregates, 50 rhs, 335 us in twos, 199
// one by one; 17 rhs 88 us whole, 96).  FP32: up to five whole (24 test vectors on 16^3 x 32 in 2^4
// aggregates, 33 rhs, 282 us in threes, 230 in one), more in even groups of at most four;
// with four waves an aggregate at most three.
template <class P, class PM, int MT>
static void launch_restrict_mt(Context* c, const TGeom& t, const typename P::S* x, typename P::S* yc,
                               const typename PM::S* Pm, int nrhs) {
  constexpr bool f64 = std::is_same<P, F64>::value;
  const int tiles = (nrhs + 7) / 8, most = f64 && tiles > 3 ? 1 : 3;
  const TransferSplit q = transfer_split(c, t, tiles, f64 ? most : tiles <= 5 ? 5 : 4, most, 4);
  switch (q.nt) {
    case 1: launch_restrict_nt<P, PM, MT, 1>(c, t, x, yc, Pm, nrhs, q.wpa); break;
    case 2: launch_restrict_nt<P, PM, MT, 2>(c, t, x, yc, Pm, nrhs, q.wpa); break;
    case 3: launch_restrict_nt<P, PM, MT, 3>(c, t, x, yc, Pm, nrhs, q.wpa); break;
    case 4: if constexpr (!f64) launch_restrict_nt<P, PM, MT, 4>(c, t, x, yc, Pm, nrhs, q.wpa); break;
    default: if constexpr (!f64) launch_restrict_nt<P, PM, MT, 5>(c, t, x, yc, Pm, nrhs, q.wpa); break;
  }
}
template <class P, class PM>
static void launch_restrict(Context* c, const TGeom& t, const typename P::S* x, typename P::S* yc,
                            const typename PM::S* Pm, int nrhs) {
  check_transfer(t);
  if (t.ntv <= 16)
    launch_restrict_mt<P, PM, 1>(c, t, x, yc, Pm, nrhs);
  else
    launch_restrict_mt<P, PM, 2>(c, t, x, yc, Pm, nrhs);
}

// Tiles of rhs: FP64 even groups of at most three (one wave an aggregate) or four; FP32
// up to five whole (24 test vectors on 16^3 x 32 in 2^4 aggregates, 33 rhs, 292 us in threes, 272
// in one), more in even groups of at most four.
template <class P, class PM, class PX, int VK>
static void launch_prolong_vk(Context* c, const TGeom& t, const typename P::S* xc, const typename P::S* x,
                              typename P::S* y, const typename PM::S* Pm, int nrhs, int mode,
                              const typename PX::S* xq, const double* xs, int xgs) {
  constexpr bool f64 = std::is_same<P, F64>::value;
  const int tiles = (nrhs + 7) / 8;
  const size_t cb = sizeof(typename P::S);
  const int Kp = (t.ntv + 4 * VK - 1) / (4 * VK) * (4 * VK);
  TransferSplit q = transfer_split(c, t, tiles, f64 ? 3 : tiles <= 5 ? 5 : 4, 4, 8);
  // coarse values of more than 64 KiB: fewer rhs per workgroup, or one
  // aggregate and chirality (four waves) instead of four
  auto need = [&](int nt) {
    return sizeof(uint32_t) * (4 / q.wpa) * row_words(t.rows) + (size_t)(4 / q.wpa) * Kp * 8 * nt * cb;
  };
  while (q.nt > 2 && need(q.nt) > 65536) q.nt--;
  if (need(q.nt) > 65536) q.wpa = 4;
  while (q.nt > 1 && need(q.nt) > 65536) q.nt--;
  const size_t lds = need(q.nt);
  auto launch = [&](auto* k) {
    launch_tiles(transfer_blocks(t, q.wpa), (tiles + q.nt - 1) / q.nt, 1, [&](dim3 nb, Tiles p) {
      hipLaunchKernelGGL(k, nb, dim3(256), lds, c->stream, xc, x, y, Pm, t, nrhs, mode, q.wpa, xq, xs, xgs, p);
    });
  };
  const bool all = q.wpa == 4;
  switch (q.nt) {
    case 1: launch(k_prolong<P, PM, PX, 1, VK, true>); break;
    case 2: launch(k_prolong<P, PM, PX, 2, VK, true>); break;
    case 3: launch(all || !f64 ? k_prolong<P, PM, PX, 3, VK, true> : k_prolong<P, PM, PX, 3, VK, false>); break;
    case 4: launch(all || f64 ? k_prolong<P, PM, PX, 4, VK, true> : k_prolong<P, PM, PX, 4, VK, false>); break;
    default:
      if constexpr (!f64) launch(k_prolong<P, PM, PX, 5, VK, false>);  // one wave an aggregate
  }
}
template <class P, class PM, class PX>
static void launch_prolong(Context* c, const TGeom& t, const typename P::S* xc, const typename P::S* x,
                           typename P::S* y, const typename PM::S* Pm, int nrhs, int mode,
                           const typename PX::S* xq, const double* xs, int xgs) {
  check_transfer(t);
  // two test vectors (8 bytes of FP16) per A load where the rows are so aligned
  if (std::is_same<PM, F16>::value && t.ntv % 8 == 0)
    launch_prolong_vk<P, PM, PX, 2>(c, t, xc, x, y, Pm, nrhs, mode, xq, xs, xgs);
  else
    launch_prolong_vk<P, PM, PX, 1>(c, t, xc, x, y, Pm, nrhs, mode, xq, xs, xgs);
}

void Transfer::restrict_(mgm_prec p, const void* x, void* yc, int nrhs) const {
  ProfScope ps(ctx, KC_TRANSFER, bytes(p, nrhs));
  if (p == MGM_PREC_F64)
    launch_restrict<F64, F64>(ctx, t, (const double2*)x, (double2*)yc, P64, nrhs);
  else if (p == MGM_PREC_F32)
    launch_restrict<F32, F16>(ctx, t, (const float2*)x, (float2*)yc, P16, nrhs);
  else
    throw Error(MGM_ERR_INVALID_ARG, "restrict: precision must be F64 or F32");
}

void Transfer::prolong(mgm_prec p, const void* xc, const void* x, void* y, int nrhs, int mode) const {
  ProfScope ps(ctx, KC_TRANSFER, bytes(p, nrhs));
  if (p == MGM_PREC_F64)
    launch_prolong<F64, F64, F64>(ctx, t, (const double2*)xc, (const double2*)x, (double2*)y, P64, nrhs, mode, nullptr,
                                  nullptr, nrhs);
  else if (p == MGM_PREC_F32)
    launch_prolong<F32, F16, F32>(ctx, t, (const float2*)xc, (const float2*)x, (float2*)y, P16, nrhs, mode, nullptr,
                                  nullptr, nrhs);
  else
    throw Error(MGM_ERR_INVALID_ARG, "prolong: precision must be F64 or F32");
}

void Transfer::restrict16(const __half2* x16, const double* xs, float2* yc, int nrhs, int xgs) const {
  ProfScope ps(ctx, KC_TRANSFER, bytes(MGM_PREC_F32, nrhs));
  check_transfer(t);
  MGM_CHECK(P16 != nullptr && xs != nullptr, MGM_ERR_INVALID_ARG, "FP16 transfer input needs P16 and scales");
  if (xgs <= 0) xgs = nrhs;
  MGM_CHECK(nrhs % xgs == 0, MGM_ERR_INVALID_ARG, "column groups must divide the rhs count");
  const int mt = (t.ntv + 7) / 8, MT = mt <= 4 ? mt : (mt + 3) / 4 * 4 <= (mt + 2) / 3 * 3 ? 4 : 3;
  const TransferSplit q = transfer_split(ctx, t, (nrhs + 15) / 16, 4, 4, 4);
  const size_t lds = sizeof(uint32_t) * (4 / q.wpa) * row_words(t.rows) +
                     (size_t)(4 / q.wpa) * (q.wpa - 1) * MT * q.nt * 64 * sizeof(f4_t);
  auto launch = [&](auto* k) {
    launch_tiles(transfer_blocks(t, q.wpa), (nrhs + 16 * q.nt - 1) / (16 * q.nt), (mt + MT - 1) / MT,
                 [&](dim3 nb, Tiles p) {
                   hipLaunchKernelGGL(k, nb, dim3(256), lds, ctx->stream, (const uint32_t*)x16, yc,
                                      (const uint32_t*)P16, t, nrhs, q.wpa, xs, xgs, p);
                 });
  };
#define MGM_R16(M, N) \
  if (MT == M && q.nt == N) launch(k_restrict16<M, N>);
  MGM_R16(1, 1) MGM_R16(1, 2) MGM_R16(1, 3) MGM_R16(1, 4) MGM_R16(2, 1) MGM_R16(2, 2) MGM_R16(2, 3) MGM_R16(2, 4)
  MGM_R16(3, 1) MGM_R16(3, 2) MGM_R16(3, 3) MGM_R16(3, 4) MGM_R16(4, 1) MGM_R16(4, 2) MGM_R16(4, 3) MGM_R16(4, 4)
#undef MGM_R16
}

void Transfer::prolong16(const float2* xc, const __half2* x16, const double* xs, float2* y, int nrhs,
                         int xgs) const {
  ProfScope ps(ctx, KC_TRANSFER, bytes(MGM_PREC_F32, nrhs));
  check_transfer(t);
  MGM_CHECK(P16 != nullptr && xs != nullptr, MGM_ERR_INVALID_ARG, "FP16 transfer input needs P16 and scales");
  if (xgs <= 0) xgs = nrhs;
  MGM_CHECK(nrhs % xgs == 0, MGM_ERR_INVALID_ARG, "column groups must divide the rhs count");
  launch_prolong<F32, F16, F16>(ctx, t, xc, (const float2*)nullptr, y, P16, nrhs, 3, x16, xs, xgs);
}

// ------------------------------------------------------------ block QR

__device__ double2 block_sum2(double2 v, double2* red) {
  const int t = threadIdx.x;
  red[t] = v;
  __syncthreads();
  for (int s = blockDim.x / 2; s > 0; s >>= 1) {
    if (t < s) red[t] = make_double2(red[t].x + red[t + s].x, red[t].y + red[t + s].y);
    __syncthreads();
  }
  double2 out = red[0];
  __syncthreads();
  return out;
}

// Modified Gram-Schmidt over the columns of every (aggregate, chirality)
// block, each column orthogonalised twice against the previous ones.
__global__ void k_block_mgs2(const double2* __restrict__ tv, double2* __restrict__ Pm, TGeom t, int* flag) {
  extern __shared__ double2 w[];
  __shared__ double2 red[256];
  const int64_t a = blockIdx.x >> 1;
  const int chi = blockIdx.x & 1;
  const int tid = threadIdx.x, nt = blockDim.x;
  const int ntv = t.ntv;
  double2* Pb = Pm + (a * 2 + chi) * (int64_t)t.rows * ntv;
  for (int k = 0; k < ntv; k++) {
    double n0 = 0;
    for (int row = tid; row < t.rows; row += nt) {
      int loc = row / t.half, j = row % t.half;
      int64_t s = fine_site(t, a, loc);
      double2 v = tv[((int64_t)(chi * t.half + j) * t.f.V + s) * ntv + k];
      w[row] = v;
      n0 += v.x * v.x + v.y * v.y;
    }
    n0 = block_sum2(make_double2(n0, 0), red).x;
    for (int pass = 0; pass < 2; pass++)
      for (int jj = 0; jj < k; jj++) {
        cx<double> h = {0, 0};
        for (int row = tid; row < t.rows; row += nt) {
          double2 qv = Pb[(int64_t)row * ntv + jj];
          fmac_(h, cx<double>{qv.x, qv.y}, cx<double>{w[row].x, w[row].y});
        }
        double2 hs = block_sum2(make_double2(h.re, h.im), red);
        for (int row = tid; row < t.rows; row += nt) {
          double2 qv = Pb[(int64_t)row * ntv + jj];
          cx<double> wv = {w[row].x, w[row].y};
          wv = wv - cx<double>{hs.x, hs.y} * cx<double>{qv.x, qv.y};
          w[row] = make_double2(wv.re, wv.im);
        }
        __syncthreads();
      }
    double nn = 0;
    for (int row = tid; row < t.rows; row += nt) nn += w[row].x * w[row].x + w[row].y * w[row].y;
    nn = block_sum2(make_double2(nn, 0), red).x;
    double nrm = sqrt(nn);
    double inv = 1.0 / nrm;
    if (!(n0 > 0.0) || !(nrm >= 1e-12 * sqrt(n0))) {
      inv = 0.0;
      if (tid == 0) *flag = 1;
    }
    for (int row = tid; row < t.rows; row += nt)
      Pb[(int64_t)row * ntv + k] = make_double2(w[row].x * inv, w[row].y * inv);
    __syncthreads();
  }
}

void mg_block_mgs2(Context* c, const TGeom& t, const double2* tv, double2* P, int* flag) {
  size_t sh = (size_t)t.rows * sizeof(double2);
  MGM_CHECK(sh <= 64 * 1024, MGM_ERR_SHAPE, "aggregate too large for LDS column");
  hipLaunchKernelGGL(k_block_mgs2, dim3((unsigned)(t.c.V * 2)), dim3(256), sh, c->stream, tv, P, t, flag);
  MGM_LAUNCH_CHECK();
}

// ------------------------------------------------------------ Galerkin

// Which stencil direction of the aggregate a fine hop k from local
// coordinates l contributes to (0 when it stays inside).
__device__ __forceinline__ int hop_target(int k, const int l[4], const int b[4]) {
  if (k == 0) return 0;
  int mu = (k - 1) & 3;
  if (k <= 4) return l[mu] == b[mu] - 1 ? k : 0;
  return l[mu] == 0 ? k : 0;
}

// One Wilson-clover block of D (12 x 12 at site s, direction k) applied to a
// single spinor p; y is the neighbour site of the hop.
__device__ void wilson_block(const FineOp& op, int k, int64_t s, int64_t y, const int fc[4],
                             const cx<double>* p, cx<double>* out) {
  const Geom& g = op.g;
  if (k == 0) {
    // entry by entry: a whole block in registers spills here
    for (int chi = 0; chi < 2; chi++) {
      auto c = [&](int j) { return op.C64[clover_pos<F64>(g.V, 36 * chi + j, s)]; };
      const cx<double>* x = p + 6 * chi;
      cx<double>* y = out + 6 * chi;
      for (int i = 0; i < 6; i++) y[i] = c(i) * x[i];
      int q = 0;
      for (int i = 1; i < 6; i++)
        for (int j = 0; j < i; j++, q++) {
          const cx<double> cij = {c(6 + 2 * q), c(7 + 2 * q)};
          fma_(y[i], cij, x[j]);
          fmac_(y[j], cij, x[i]);
        }
    }
    return;
  }
  const bool fwd = k <= 4;
  const int mu = (k - 1) & 3;
  const int ext[4] = {g.X, g.Y, g.Z, g.T};
  double ph = 1.0;
  if (mu == 3 && g.antiperiodic && ((fwd && fc[3] == ext[3] - 1) || (!fwd && fc[3] == 0))) ph = -1.0;
  const int64_t ls = fwd ? s : y;  // site owning the link U_mu
  cx<double> U[3][3];
  for (int q = 0; q < 9; q++) {
    double2 v = op.U64[link_pos<F64>(g.V, mu, q, ls)];
    U[q / 3][q % 3] = {v.x, v.y};
  }
  cx<double> h[2][3];
  for (int a = 0; a < 3; a++) {
    cx<double> a0, a1;
    A_times(mu, p[6 + a], p[9 + a], a0, a1);
    h[0][a] = fwd ? p[a] - a0 : p[a] + a0;
    h[1][a] = fwd ? p[3 + a] - a1 : p[3 + a] + a1;
  }
  const double f = -0.5 * ph;
  for (int a = 0; a < 3; a++) {
    cx<double> g0 = {0, 0}, g1 = {0, 0};
    for (int b = 0; b < 3; b++) {
      if (fwd) {
        fma_(g0, U[a][b], h[0][b]);
        fma_(g1, U[a][b], h[1][b]);
      } else {
        fmac_(g0, U[b][a], h[0][b]);
        fmac_(g1, U[b][a], h[1][b]);
      }
    }
    g0 = f * g0;
    g1 = f * g1;
    cx<double> d0, d1;
    Ad_times(mu, g0, g1, d0, d1);
    out[a] = g0;
    out[3 + a] = g1;
    out[6 + a] = fwd ? (-1.0) * d0 : d0;
    out[9 + a] = fwd ? (-1.0) * d1 : d1;
  }
}

__device__ __forceinline__ int64_t hop_neighbour(const LGeom& g, const int c[4], int k) {
  if (k == 0) return index_of(g, c);
  int mu = (k - 1) & 3;
  int cc[4] = {c[0], c[1], c[2], c[3]};
  cc[mu] += (k <= 4) ? 1 : -1;
  return index_of(g, cc);
}

constexpr int kGalPairs = 16;  // (i, j) pairs per thread: d * jc <= 256 * kGalPairs

// Both Galerkin kernels run one workgroup per (coarse site, stencil
// direction, chunk of jc coarse columns j).  For every fine site x of the
// aggregate, the sum over the hops k of x that land in that direction of
// B[x, k] P(y_k) (the chunk's columns) is staged in LDS, and each thread
// accumulates up to kGalPairs entries (i, j) of P(x)^H times that sum.
__global__ void k_galerkin_fine(FineOp op, TGeom t, const double2* __restrict__ Pm, double2* __restrict__ Ac,
                                int jc) {
  extern __shared__ double2 T[];  // [12][jc] hop sums, then [2][6][ntv] rows of P(x)
  const int64_t a = blockIdx.x;
  const int tgt = blockIdx.y;
  const int j0 = blockIdx.z * jc;
  const int d = 2 * t.ntv, ntv = t.ntv, tid = threadIdx.x;
  const int nj = d - j0 < jc ? d - j0 : jc;
  double2* PX = T + 12 * jc;
  cx<double> acc[kGalPairs];
  for (int q = 0; q < kGalPairs; q++) acc[q] = {0, 0};
  int ca[4];
  coords_of(t.c, a, ca);
  for (int loc = 0; loc < t.bvol; loc++) {
    int l[4], rem = loc, fc[4];
    l[0] = rem % t.b[0]; rem /= t.b[0];
    l[1] = rem % t.b[1]; rem /= t.b[1];
    l[2] = rem % t.b[2]; rem /= t.b[2];
    l[3] = rem;
    bool any = false;
    for (int k = 0; k < 9; k++) any |= hop_target(k, l, t.b) == tgt;
    if (!any) continue;  // uniform over the workgroup
    for (int m = 0; m < 4; m++) fc[m] = ca[m] * t.b[m] + l[m];
    const int64_t s = index_of(t.f, fc);
    if (tid < nj) {
      const int j = j0 + tid, chij = j / ntv, kk = j % ntv;
      cx<double> sum[12];
      for (int m = 0; m < 12; m++) sum[m] = {0, 0};
      for (int k = 0; k < 9; k++) {
        if (hop_target(k, l, t.b) != tgt) continue;
        const int64_t y = hop_neighbour(t.f, fc, k);
        int64_t ay;
        int locy;
        agg_of(t, y, ay, locy);
        cx<double> p[12];
        for (int m = 0; m < 12; m++) p[m] = {0, 0};
        for (int m = 0; m < 6; m++) {
          double2 v = Pm[((ay * 2 + chij) * t.rows + locy * 6 + m) * (int64_t)ntv + kk];
          p[6 * chij + m] = {v.x, v.y};
        }
        cx<double> o[12];
        wilson_block(op, k, s, y, fc, p, o);
        for (int m = 0; m < 12; m++) sum[m] = sum[m] + o[m];
      }
      for (int m = 0; m < 12; m++) T[m * jc + tid] = make_double2(sum[m].re, sum[m].im);
    }
    for (int e = tid; e < 12 * ntv; e += blockDim.x) {
      const int chi = e / (6 * ntv), r = e - chi * 6 * ntv;  // r = m ntv + k
      PX[e] = Pm[((a * 2 + chi) * t.rows + loc * 6) * (int64_t)ntv + r];
    }
    __syncthreads();
    for (int q = 0; q < kGalPairs; q++) {
      int pidx = tid + q * blockDim.x;
      if (pidx >= d * nj) break;
      int i = pidx / nj, jj = pidx % nj;
      int chii = i / ntv, ki = i % ntv;
      const double2* pr = PX + chii * 6 * ntv + ki;
      for (int m = 0; m < 6; m++) {
        double2 pv = pr[m * ntv];
        double2 tv = T[(6 * chii + m) * jc + jj];
        fmac_(acc[q], cx<double>{pv.x, pv.y}, cx<double>{tv.x, tv.y});
      }
    }
    __syncthreads();
  }
  const int64_t Vc = t.c.V;
  for (int q = 0; q < kGalPairs; q++) {
    int pidx = tid + q * blockDim.x;
    if (pidx >= d * nj) break;
    int i = pidx / nj, j = j0 + pidx % nj;
    Ac[((int64_t)(tgt * d + i) * d + j) * Vc + a] = make_double2(acc[q].re, acc[q].im);
  }
}

__global__ void k_galerkin_coarse(CoarseOp op, TGeom t, const double2* __restrict__ Pm, double2* __restrict__ Ac,
                                  int jc) {
  extern __shared__ double2 T[];  // [dl][jc]
  const int64_t a = blockIdx.x;
  const int tgt = blockIdx.y;
  const int j0 = blockIdx.z * jc;
  const int d = 2 * t.ntv, ntv = t.ntv, tid = threadIdx.x;
  const int nj = d - j0 < jc ? d - j0 : jc;
  const int dl = t.f.dof, hl = t.half;
  const int64_t Vl = t.f.V;
  cx<double> acc[kGalPairs];
  for (int q = 0; q < kGalPairs; q++) acc[q] = {0, 0};
  int ca[4];
  coords_of(t.c, a, ca);
  for (int loc = 0; loc < t.bvol; loc++) {
    int l[4], rem = loc, fc[4];
    l[0] = rem % t.b[0]; rem /= t.b[0];
    l[1] = rem % t.b[1]; rem /= t.b[1];
    l[2] = rem % t.b[2]; rem /= t.b[2];
    l[3] = rem;
    bool any = false;
    for (int k = 0; k < 9; k++) any |= hop_target(k, l, t.b) == tgt;
    if (!any) continue;  // uniform over the workgroup
    for (int m = 0; m < 4; m++) fc[m] = ca[m] * t.b[m] + l[m];
    const int64_t s = index_of(t.f, fc);
    // entries (i2, jj) of the chunk's hop sum, one per thread at a time
    for (int e = tid; e < dl * nj; e += blockDim.x) {
      const int i2 = e / nj, jj = e - i2 * nj;
      const int j = j0 + jj, chij = j / ntv, kk = j % ntv;
      cx<double> o = {0, 0};
      for (int k = 0; k < 9; k++) {
        if (hop_target(k, l, t.b) != tgt) continue;
        const int64_t y = hop_neighbour(t.f, fc, k);
        int64_t ay;
        int locy;
        agg_of(t, y, ay, locy);
        const double2* py = Pm + ((ay * 2 + chij) * t.rows + locy * hl) * (int64_t)ntv + kk;
        const double2* Arow = op.A64 + ((int64_t)(k * dl + i2) * dl + chij * hl) * Vl + s;
        for (int mm = 0; mm < hl; mm++) {
          double2 av = Arow[(int64_t)mm * Vl];
          double2 pv = py[(int64_t)mm * ntv];
          fma_(o, cx<double>{av.x, av.y}, cx<double>{pv.x, pv.y});
        }
      }
      T[i2 * jc + jj] = make_double2(o.re, o.im);
    }
    __syncthreads();
    for (int q = 0; q < kGalPairs; q++) {
      int pidx = tid + q * blockDim.x;
      if (pidx >= d * nj) break;
      int i = pidx / nj, jj = pidx % nj;
      int chii = i / ntv, ki = i % ntv;
      const double2* pr = Pm + ((a * 2 + chii) * t.rows + loc * hl) * (int64_t)ntv + ki;
      for (int mm = 0; mm < hl; mm++) {
        double2 pv = pr[(int64_t)mm * ntv];
        double2 tv = T[(chii * hl + mm) * jc + jj];
        fmac_(acc[q], cx<double>{pv.x, pv.y}, cx<double>{tv.x, tv.y});
      }
    }
    __syncthreads();
  }
  const int64_t Vc = t.c.V;
  for (int q = 0; q < kGalPairs; q++) {
    int pidx = tid + q * blockDim.x;
    if (pidx >= d * nj) break;
    int i = pidx / nj, j = j0 + pidx % nj;
    Ac[((int64_t)(tgt * d + i) * d + j) * Vc + a] = make_double2(acc[q].re, acc[q].im);
  }
}

// columns per Galerkin workgroup: all d when the pairs and the staged rows
// fit, else the largest power of two that does
static int galerkin_jc(int d, int rows_staged) {
  int jc = d;
  while (jc > 1 && ((size_t)d * jc > (size_t)256 * kGalPairs || (size_t)rows_staged * jc * sizeof(double2) > 65536))
    jc = (jc + 1) / 2;
  return jc;
}

void mg_galerkin_fine(Context* c, const FineOp& op, const Transfer& T, CoarseOp& out) {
  const TGeom& t = T.t;
  const int d = 2 * t.ntv;
  MGM_CHECK(d <= 256, MGM_ERR_SHAPE, "too many test vectors");
  const int jc = galerkin_jc(d, 12);
  const size_t sh = (size_t)12 * (jc + t.ntv) * sizeof(double2);
  hipLaunchKernelGGL(k_galerkin_fine, dim3((unsigned)t.c.V, 9, (unsigned)((d + jc - 1) / jc)), dim3(256), sh,
                     c->stream, op, t, T.P64, out.A64, jc);
  MGM_LAUNCH_CHECK();
}

void mg_galerkin_coarse(Context* c, const CoarseOp& op, const Transfer& T, CoarseOp& out) {
  const TGeom& t = T.t;
  const int d = 2 * t.ntv;
  MGM_CHECK(d <= 256 && t.f.dof <= 256, MGM_ERR_SHAPE, "too many test vectors");
  const int jc = galerkin_jc(d, t.f.dof);
  const size_t sh = (size_t)t.f.dof * jc * sizeof(double2);
  hipLaunchKernelGGL(k_galerkin_coarse, dim3((unsigned)t.c.V, 9, (unsigned)((d + jc - 1) / jc)), dim3(256), sh,
                     c->stream, op, t, T.P64, out.A64, jc);
  MGM_LAUNCH_CHECK();
}

// ------------------------------------------------------- coarse stencil

// y(s) = sum_dir A[dir](s) x(nbr(s, dir)) runs on the matrix cores
// (coarse_mfma.hip): FP64 and FP32 with 16x16x4 MFMAs, BF16 operands with
// FP32 accumulation for the mixed-precision preconditioner.

double CoarseOp::bytes(mgm_prec p, int nrhs) const {
  // algorithmic bytes: nine complex d x d blocks once, x and y once
  double wa = p == MGM_PREC_F64 ? 16.0 : p == MGM_PREC_F32 ? 8.0 : 4.0;
  double wv = p == MGM_PREC_F64 ? 16.0 : 8.0;
  return (double)g.V * (9.0 * d * d * wa + 2.0 * d * nrhs * wv);
}

void CoarseOp::apply(mgm_prec p, const void* x, void* y, int nrhs) const {
  if (p == MGM_PREC_F64) {
    coarse_apply_mfma64(*this, (const double2*)x, (double2*)y, nrhs);
  } else if (p == MGM_PREC_F32) {
    MGM_CHECK(A32 != nullptr, MGM_ERR_INVALID_ARG, "FP32 coarse stencil not built (mixed == 0)");
    coarse_apply_mfma32(*this, (const float2*)x, (float2*)y, nrhs);
  } else if (p == MGM_PREC_BF16) {
    coarse_apply_mfma(*this, (const float2*)x, (float2*)y, nrhs);
  } else {
    throw Error(MGM_ERR_INVALID_ARG, "coarse apply: unsupported precision");
  }
}

// ---------------------------------------------------------- conversions

// P entries are O(1/sqrt(rows)), well inside the FP16 range
__global__ void k_c64_to_c16(__half2* o, const double2* in, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) o[i] = __floats2half2_rn((float)in[i].x, (float)in[i].y);
}

void mg_convert_P(Context* c, Transfer& T) {
  int64_t n = T.t.c.V * 2 * (int64_t)T.t.rows * T.t.ntv;
  hipLaunchKernelGGL(k_c64_to_c16, dim3(nblocks_for(n, 256)), dim3(256), 0, c->stream, T.P16, T.P64, n);
  MGM_LAUNCH_CHECK();
}

void mg_convert_A(Context* c, CoarseOp& A) { mg_mfma32_pack(c, A); }

}  // namespace mgm
