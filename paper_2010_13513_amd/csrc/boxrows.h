// Stencil rows on boxes in LDS by discretisation (include after
// generated/stencils.inc).
#pragma once

namespace hhg {
namespace {

template <int DISC>
struct BoxRows;
template <>
struct BoxRows<1> {
  template <typename T, int GR, int S1, int S2, int SG, typename P>
  static __device__ __forceinline__ T A(P u) {
    return gen::p1_As<T, GR, S1, S2, SG>(u);
  }
  template <typename T, int GR, int S1, int S2, typename P>
  static __device__ __forceinline__ T BT(P p, int d) {
    return gen::p1_BTs<T, GR, S1, S2>(p, d);
  }
  // the same over three planes of a ring
  template <typename T, int GR, int S1, int SG, typename P>
  static __device__ __forceinline__ T Ar(const P (&u)[3]) {
    return gen::p1_Ar<T, GR, S1, SG>(u);
  }
  template <typename T, int GR, int S1, typename P>
  static __device__ __forceinline__ T BTr(const P (&p)[3], int d) {
    return gen::p1_BTr<T, GR, S1>(p, d);
  }
  // element-wise row of the variable-viscosity A (units of h): u the site's
  // word, nu the viscosity of the site's P1 index
  template <typename T, int GR, int S1, int S2, int SG>
  static __device__ __forceinline__ T Anu(const T* u, const T* nu) {
    T a0 = 0, a1 = 0, a2 = 0;
    gen::p1_Anu_g0<T>(u, u, u, nu, 0, 0, S1, S2, SG, a0, a1, a2);
    return a0;
  }
  static constexpr int denA = gen::p1_zm_den[0], denT = gen::p1_zm_den[1];
};
template <>
struct BoxRows<8> {
  template <typename T, int GR, int S1, int S2, int SG, typename P>
  static __device__ __forceinline__ T A(P u) {
    return gen::p2_As<T, GR, S1, S2, SG>(u);
  }
  template <typename T, int GR, int S1, int S2, typename P>
  static __device__ __forceinline__ T BT(P p, int d) {
    return gen::p2_BTs<T, GR, S1, S2>(p, d);
  }
  template <typename T, int GR, int S1, int SG, typename P>
  static __device__ __forceinline__ T Ar(const P (&u)[3]) {
    return gen::p2_Ar<T, GR, S1, SG>(u);
  }
  template <typename T, int GR, int S1, typename P>
  static __device__ __forceinline__ T BTr(const P (&p)[3], int d) {
    return gen::p2_BTr<T, GR, S1>(p, d);
  }
  template <typename T, int GR, int S1, int S2, int SG>
  static __device__ __forceinline__ T Anu(const T* u, const T* nu) {
    T a0 = 0, a1 = 0, a2 = 0;
    if constexpr (GR == 0) gen::p2_Anu_g0<T>(u, u, u, nu, 0, 0, S1, S2, SG, a0, a1, a2);
    if constexpr (GR == 1) gen::p2_Anu_g1<T>(u, u, u, nu, 0, 0, S1, S2, SG, a0, a1, a2);
    if constexpr (GR == 2) gen::p2_Anu_g2<T>(u, u, u, nu, 0, 0, S1, S2, SG, a0, a1, a2);
    if constexpr (GR == 3) gen::p2_Anu_g3<T>(u, u, u, nu, 0, 0, S1, S2, SG, a0, a1, a2);
    if constexpr (GR == 4) gen::p2_Anu_g4<T>(u, u, u, nu, 0, 0, S1, S2, SG, a0, a1, a2);
    if constexpr (GR == 5) gen::p2_Anu_g5<T>(u, u, u, nu, 0, 0, S1, S2, SG, a0, a1, a2);
    if constexpr (GR == 6) gen::p2_Anu_g6<T>(u, u, u, nu, 0, 0, S1, S2, SG, a0, a1, a2);
    if constexpr (GR == 7) gen::p2_Anu_g7<T>(u, u, u, nu, 0, 0, S1, S2, SG, a0, a1, a2);
    return a0;
  }
  static constexpr int denA = gen::p2_zm_den[0], denT = gen::p2_zm_den[1];
};
constexpr int gdir(int G, int g, int axis) {
  return G == 1 ? 0 : ((axis == 0 ? 0xB2 : (axis == 1 ? 0xD4 : 0xE8)) >> g) & 1;
}

}  // namespace
}  // namespace hhg
