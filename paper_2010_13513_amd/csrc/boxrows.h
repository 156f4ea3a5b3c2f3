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
  static constexpr int denA = gen::p2_zm_den[0], denT = gen::p2_zm_den[1];
};
constexpr int gdir(int G, int g, int axis) {
  return G == 1 ? 0 : ((axis == 0 ? 0xB2 : (axis == 1 ? 0xD4 : 0xE8)) >> g) & 1;
}

}  // namespace
}  // namespace hhg
