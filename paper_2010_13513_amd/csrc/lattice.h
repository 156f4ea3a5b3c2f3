// Index helpers of the lattice layout shared by the kernel files (include
// inside a .hip file after kernels.h).
#pragma once
#include "kernels.h"

namespace hhg {
namespace {

constexpr int kBlock = 256;

__device__ __forceinline__ void decode(int t, int n1, int& i, int& j, int& k) {
  i = t % n1;
  const int r = t / n1;
  j = r % n1;
  k = r / n1;
}
// parity class of velocity group g (0: vertex, 1..7: edge directions)
__device__ __forceinline__ int gdx(int g) { return (0xB2 >> g) & 1; }
__device__ __forceinline__ int gdy(int g) { return (0xD4 >> g) & 1; }
__device__ __forceinline__ int gdz(int g) { return (0xE8 >> g) & 1; }

template <int G>
__device__ __forceinline__ bool vel_interior(int g, int i, int j, int k, int N) {
  const int dx = G == 1 ? 0 : gdx(g), dy = G == 1 ? 0 : gdy(g), dz = G == 1 ? 0 : gdz(g);
  return i >= 1 - dx && j >= 1 - dy && k >= 1 - dz && i <= N - 1 && j <= N - 1 && k <= N - 1;
}
// velocity site exists (not padding): doubled position 2(i,j,k) + dir inside [0, 2N]
template <int G>
__device__ __forceinline__ bool vel_exists(int g, int i, int j, int k, int N) {
  if (G == 1) return true;
  return i + gdx(g) <= N && j + gdy(g) <= N && k + gdz(g) <= N;
}
__device__ __forceinline__ int bcls3(int c, int N) { return c == 0 ? 0 : (c == N ? 2 : 1); }

// Faces of the cube a velocity site lies on (bit f as in Geom::nf), from its
// position in site units (doubled for P2).
__device__ __forceinline__ int site_faces(int X, int Y, int Z, int M) {
  return (X == 0) | ((X == M) << 1) | ((Y == 0) << 2) | ((Y == M) << 3) | ((Z == 0) << 4) | ((Z == M) << 5);
}
// The velocity site is an unknown: it exists and lies on no Dirichlet face
// (interior sites, and sites whose faces are all outflow faces).
template <int G>
__device__ __forceinline__ bool vel_unknown(const Geom& g, int gr, int i, int j, int k) {
  if (!vel_exists<G>(gr, i, j, k, g.N)) return false;
  const int f = G == 1 ? site_faces(i, j, k, g.N)
                       : site_faces(2 * i + gdx(gr), 2 * j + gdy(gr), 2 * k + gdz(gr), 2 * g.N);
  return (f & ~g.nf) == 0;
}

// Velocity value of the finest level at site (i, j, k) of group gr of a level
// `up` refinements below it (a vertex there): its slot in a component.
template <int G>
__device__ __forceinline__ int finest_slot(int gr, int i, int j, int k, int n1, int up) {
  const int u = G == 1 ? up : up - 1;
  const int X = (G == 1 ? i : 2 * i + gdx(gr)) << u, Y = (G == 1 ? j : 2 * j + gdy(gr)) << u,
            Z = (G == 1 ? k : 2 * k + gdz(gr)) << u;
  return X + n1 * (Y + n1 * Z);
}

}  // namespace
}  // namespace hhg
