// Device helpers of the Wilson-clover stencil shared by the dslash and the
// Galerkin coarse-operator construction.
#pragma once
#include "fine.h"

#include <type_traits>

namespace mgm {

// Layout of the operator's fields.  A lane loads the entries of its own site, so
// consecutive entries are stored side by side in groups of 16 bytes (8 for the FP16
// clover): a link is 5 loads in FP32 and 3 in FP16 instead of 9, the clover 18
// instead of 72 (FP64: 36), consecutive sites still read consecutive groups, and a
// short run of sites fills whole cache lines.
//   links: entries 0..7 of the matrix in groups of LG, plane mu * 8 / LG + k / LG, then
//   the ninth entries [mu][V] (FP64, one entry to 16 bytes: [mu][9][V]);
//   clover: 72 / CG planes of CG reals.
template <class P>
struct FieldGroup;
template <>
struct FieldGroup<F64> {
  static constexpr int LG = 1, CG = 2;
};
template <>
struct FieldGroup<F32> {
  static constexpr int LG = 2, CG = 4;
};
template <>
struct FieldGroup<F16> {
  static constexpr int LG = 4, CG = 4;
};
// position of entry k of U_mu, and of real j of the clover, of site s
template <class P>
__host__ __device__ __forceinline__ int64_t link_pos(int64_t V, int mu, int k, int64_t s) {
  constexpr int LG = FieldGroup<P>::LG;
  if (LG == 1) return (int64_t)(mu * 9 + k) * V + s;
  if (k == 8) return (int64_t)(32 + mu) * V + s;
  return (int64_t)(mu * 8 + k / LG * LG) * V + s * LG + k % LG;
}
template <class P>
__host__ __device__ __forceinline__ int64_t clover_pos(int64_t V, int j, int64_t s) {
  constexpr int CG = FieldGroup<P>::CG;
  return (int64_t)(j / CG * CG) * V + s * CG + j % CG;
}
template <class T, int N>
struct alignas(N * sizeof(T)) Pack {
  T v[N];
};
// base + byte offset: with a uniform base and a 32-bit offset the address takes
// one register and no vector arithmetic
template <class T, class O>
__device__ __forceinline__ T* at_byte(T* base, O off) {
  using C = typename std::conditional<std::is_const<T>::value, const char, char>::type;
  return reinterpret_cast<T*>(reinterpret_cast<C*>(base) + off);
}
// the nine stored entries of U_mu(s) (16 s fits 32 bits: the fields of 2^28 sites in
// the three formats would take 541 GB)
template <class P>
__device__ __forceinline__ void link_load(const typename P::S* __restrict__ U, int64_t V, int mu, uint32_t s,
                                          typename P::S (&w)[9]) {
  using S = typename P::S;
  constexpr int LG = FieldGroup<P>::LG;
  if constexpr (LG == 1) {
#pragma unroll
    for (int k = 0; k < 9; k++) w[k] = *at_byte(U + (int64_t)(mu * 9 + k) * V, s * (uint32_t)sizeof(S));
  } else {
#pragma unroll
    for (int c = 0; c < 8 / LG; c++) {
      const Pack<S, LG> v = *reinterpret_cast<const Pack<S, LG>*>(
          at_byte(U + (int64_t)(mu * 8 + c * LG) * V, s * (uint32_t)(LG * sizeof(S))));
#pragma unroll
      for (int j = 0; j < LG; j++) w[c * LG + j] = v.v[j];
    }
    w[8] = *at_byte(U + (int64_t)(32 + mu) * V, s * (uint32_t)sizeof(S));
  }
}
// one of them, of an entry that is the same in every lane
template <class P>
__device__ __forceinline__ typename P::S link_entry(const typename P::S* __restrict__ U, int64_t V, int mu, int k,
                                                    uint32_t s) {
  constexpr uint32_t LG = FieldGroup<P>::LG, B = sizeof(typename P::S);
  return *at_byte(U + link_pos<P>(V, mu, k, 0), s * (LG == 1 || k == 8 ? B : LG * B));
}
template <class P>
__device__ __forceinline__ void clover_load(const typename P::RS* __restrict__ C, int64_t V, uint32_t s, int chi,
                                            typename P::R (&c)[36]) {
  using T = typename P::RS;
  constexpr int CG = FieldGroup<P>::CG;
#pragma unroll
  for (int k = 0; k < 36; k += CG) {
    const Pack<T, CG> v = *reinterpret_cast<const Pack<T, CG>*>(
        at_byte(C + (int64_t)(36 * chi + k) * V, s * (uint32_t)(CG * sizeof(T))));
#pragma unroll
    for (int j = 0; j < CG; j++) c[k + j] = P::ldr(v.v, j);
  }
}

// Hermitian 6x6 block times a 6-vector, block packed as 6 diagonal reals
// followed by the 15 complex entries below the diagonal.
template <class R>
__device__ __forceinline__ void clover_mul(const R (&c)[36], const cx<R>* x, cx<R>* y) {
#pragma unroll
  for (int i = 0; i < 6; i++) y[i] = c[i] * x[i];
  int q = 0;
#pragma unroll
  for (int i = 1; i < 6; i++)
#pragma unroll
    for (int j = 0; j < i; j++, q++) {
      const cx<R> cij = {c[6 + 2 * q], c[7 + 2 * q]};
      fma_(y[i], cij, x[j]);
      fmac_(y[j], cij, x[i]);
    }
}
// A_mu l (per colour) for the chiral basis, and A_mu^H g.
template <typename R>
__device__ __forceinline__ void A_times(int mu, cx<R> l0, cx<R> l1, cx<R>& o0, cx<R>& o1) {
  switch (mu) {
    case 0: o0 = times_mi(l1); o1 = times_mi(l0); break;        // -i s1
    case 1: o0 = (R)-1 * l1;   o1 = l0; break;                  // -i s2
    case 2: o0 = times_mi(l0); o1 = times_i(l1); break;         // -i s3
    default: o0 = l0; o1 = l1; break;                           // 1
  }
}
template <typename R>
__device__ __forceinline__ void Ad_times(int mu, cx<R> g0, cx<R> g1, cx<R>& o0, cx<R>& o1) {
  switch (mu) {
    case 0: o0 = times_i(g1); o1 = times_i(g0); break;
    case 1: o0 = g1; o1 = (R)-1 * g0; break;
    case 2: o0 = times_i(g0); o1 = times_mi(g1); break;
    default: o0 = g0; o1 = g1; break;
  }
}

}  // namespace mgm
