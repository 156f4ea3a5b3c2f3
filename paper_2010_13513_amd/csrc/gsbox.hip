// Gauss-Seidel sweeps on boxes of the lattice held in LDS (gfx950).
#include <climits>
#include <type_traits>

#include "kernels.h"
#include "lanes.h"
#include "lattice.h"

#include "generated/stencils.inc"
#include "boxrows.h"

namespace hhg {
namespace {

// ------------------------------------------- Gauss-Seidel runs on boxes
// A run of colours (a generated sequence Q) of one velocity component on a box
// of the lattice held in LDS: the tile's sites plus the layers around them
// that the run's later colours read.  The layers are recomputed by every tile
// that needs them (same rows, same order, hence the same values), so one
// launch does what took one launch per colour.  Tiles run in any order: they
// read the groups of this run from one buffer and write them to the other.
// Bound by latency on these sizes: a launch, the box's loads in one batch and
// a barrier and an LDS round trip per colour (Taylor-Hood, N = 16: 5 - 7 us
// per run of four or five colours against 3.3 us per colour launch).
template <typename Q, int TX, int TY, int TZ, int NT, bool VAR>
struct BoxShape {
  static constexpr int BX = TX + Q::bhi[0] - Q::blo[0], BY = TY + Q::bhi[1] - Q::blo[1],
                       BZ = TZ + Q::bhi[2] - Q::blo[2];
  static constexpr int S1 = BX, S2 = BX * BY, SG = BX * BY * BZ;
  static constexpr int arrays = Q::G + (VAR ? 2 : 1);  // velocity groups, pressure, viscosity
  static constexpr int words = SG * arrays;
  static constexpr int loads = (SG + NT - 1) / NT;
  // step s: box of updated sites; the vertex colours take every other i
  static constexpr int grp(int s) { return Q::col[s] < kGsVertexColours ? 0 : Q::col[s] - kGsVertexColours + 1; }
  static constexpr bool half(int s) { return Q::col[s] < kGsVertexColours; }
  static constexpr int W(int s) { return (TX + Q::hi[s][0] - Q::lo[s][0] + (half(s) ? 1 : 0)) / (half(s) ? 2 : 1); }
  static constexpr int H(int s) { return TY + Q::hi[s][1] - Q::lo[s][1]; }
  static constexpr int D(int s) { return TZ + Q::hi[s][2] - Q::lo[s][2]; }
  static constexpr int passes(int s) { return (W(s) * H(s) * D(s) + NT - 1) / NT; }
  static constexpr int first(int s) { return s == 0 ? 0 : first(s - 1) + passes(s - 1); }
  static constexpr int total = first(Q::n);
};

// Tile of a block: consecutive blocks of an XCD take 4 x 4 x 4 groups of tiles,
// so the layers that neighbouring tiles share stay in that XCD's L2.  All
// counts are powers of two.
struct TileGrid {
  int lx, ly, lz;  // log2 of the tile counts
};
__device__ __forceinline__ void tile_of(const TileGrid& tg, int& tx, int& ty, int& tz, int& comp) {
  const int lt = tg.lx + tg.ly + tg.lz;
  const int lin = (int)(blockIdx.x & 7) * (int)(gridDim.x >> 3) + (int)(blockIdx.x >> 3);
  comp = lin >> lt;
  int r = lin & ((1 << lt) - 1);
  const int cx = min(tg.lx, 2), cy = min(tg.ly, 2), cz = min(tg.lz, 2);
  tx = r & ((1 << cx) - 1), r >>= cx;
  ty = r & ((1 << cy) - 1), r >>= cy;
  tz = r & ((1 << cz) - 1), r >>= cz;
  tx |= (r & ((1 << (tg.lx - cx)) - 1)) << cx, r >>= tg.lx - cx;
  ty |= (r & ((1 << (tg.ly - cy)) - 1)) << cy, r >>= tg.ly - cy;
  tz |= r << cz;
}

template <typename T, typename Q, int TX, int TY, int TZ, int NT, bool VAR>
__global__ void __launch_bounds__(NT) k_gs_box(Geom g, LevelConst<T> lc, const T* x, const T* alt, T* xw, T* altw,
                                               const T* __restrict__ pv, const T* __restrict__ b, unsigned in_alt,
                                               TileGrid tg) {
  using Sh = BoxShape<Q, TX, TY, TZ, NT, VAR>;
  using R = BoxRows<Q::G>;
  constexpr int G = Q::G, S1 = Sh::S1, S2 = Sh::S2, SG = Sh::SG;
  __shared__ T box[Sh::words];
  const int N = g.N, n1 = g.n1, n2 = g.n1 * g.n1, nn = g.nn;
  const int tid = threadIdx.x;
  int x0, y0, z0, d;
  tile_of(tg, x0, y0, z0, d);
  x0 *= TX, y0 *= TY, z0 *= TZ;
  const size_t dv = (size_t)d * g.vstride;
  T v[Sh::loads][Sh::arrays];
#pragma unroll
  for (int q = 0; q < Sh::loads; ++q) {
    const int c = tid + q * NT;
    const int bx = c % S1, by = (c / S1) % Sh::BY, bz = c / S2;
    const int i = min(max(x0 + Q::blo[0] + bx, 0), N), j = min(max(y0 + Q::blo[1] + by, 0), N),
              k = min(max(z0 + Q::blo[2] + bz, 0), N);
    const int at = i + n1 * j + n2 * k;
#pragma unroll
    for (int gr = 0; gr < G; ++gr) v[q][gr] = (((in_alt >> gr) & 1u) ? alt : x)[dv + gr * nn + at];
    v[q][G] = pv[at];
    if constexpr (VAR) v[q][G + 1] = lc.nu[at];
  }
  // the sites this thread updates: box position (-1: none) and f
  int lp[Sh::total];
  T f[Sh::total], ai[VAR ? Sh::total : 1];
  auto each = [&](auto&& fn) {
    auto go = [&](auto self, auto sc) {
      constexpr int s = decltype(sc)::value;
      if constexpr (s < Q::n) {
        fn(sc);
        self(self, std::integral_constant<int, s + 1>{});
      }
    };
    go(go, std::integral_constant<int, 0>{});
  };
  each([&](auto sc) {
    constexpr int s = decltype(sc)::value, gr = Sh::grp(s), W = Sh::W(s), H = Sh::H(s);
#pragma unroll
    for (int q = 0; q < Sh::passes(s); ++q) {
      const int c = tid + q * NT;
      const int w = c % W, h = (c / W) % H, dd = c / (W * H);
      const int j = y0 + Q::lo[s][1] + h, k = z0 + Q::lo[s][2] + dd;
      int bx = Q::lo[s][0] - Q::blo[0] + (Sh::half(s) ? 2 * w : w);
      if (Sh::half(s)) bx += (x0 + Q::lo[s][0] + j + k + Q::col[s]) & 1;
      const int i = x0 + Q::blo[0] + bx;
      const bool on = dd < Sh::D(s) && bx < TX + Q::hi[s][0] - Q::blo[0] && vel_interior<G>(gr, i, j, k, N);
      lp[Sh::first(s) + q] =
          on ? bx + S1 * (Q::lo[s][1] - Q::blo[1] + h) + S2 * (Q::lo[s][2] - Q::blo[2] + dd) : -1;
      const int at = gr * nn + i + n1 * j + n2 * k;
      f[Sh::first(s) + q] = on ? b[dv + at] : T(0);
      if constexpr (VAR) ai[Sh::first(s) + q] = on ? lc.ainv_site[at] : T(0);
    }
  });
#pragma unroll
  for (int q = 0; q < Sh::loads; ++q) {
    const int c = tid + q * NT;
    if (c < SG) {
#pragma unroll
      for (int gr = 0; gr < Sh::arrays; ++gr) box[gr * SG + c] = v[q][gr];
    }
  }
  __syncthreads();
  const T sa = lc.a / T(R::denA), sb = lc.b / T(R::denT);
  each([&](auto sc) {  // f - B^T p, fixed during the run
    constexpr int s = decltype(sc)::value, gr = Sh::grp(s);
#pragma unroll
    for (int q = 0; q < Sh::passes(s); ++q) {
      const int l = lp[Sh::first(s) + q];
      if (l >= 0) f[Sh::first(s) + q] -= sb * R::template BT<T, gr, S1, S2>(box + G * SG + l, d);
    }
  });
  each([&](auto sc) {
    constexpr int s = decltype(sc)::value, gr = Sh::grp(s);
#pragma unroll
    for (int q = 0; q < Sh::passes(s); ++q) {
      const int l = lp[Sh::first(s) + q];
      if (l >= 0) {
        T* u = box + gr * SG + l;
        if constexpr (VAR)
          *u += (f[Sh::first(s) + q] - lc.a * R::template Anu<T, gr, S1, S2, SG>(u, box + (G + 1) * SG + l)) *
                ai[Sh::first(s) + q];
        else
          *u += (f[Sh::first(s) + q] - sa * R::template A<T, gr, S1, S2, SG>(u)) * lc.ainv[gr];
      }
    }
    __syncthreads();
  });
  // the tile's words of the run's groups, boundary values and padding included
  // (the last tiles with the boundary layer)
  const int wx = x0 + TX == N ? TX + 1 : TX, wy = y0 + TY == N ? TY + 1 : TY, wz = z0 + TZ == N ? TZ + 1 : TZ;
  constexpr int cells = (TX + 1) * (TY + 1) * (TZ + 1);
#pragma unroll
  for (int q = 0; q < (cells + NT - 1) / NT; ++q) {
    const int c = tid + q * NT;
    const int cx = c % (TX + 1), cy = (c / (TX + 1)) % (TY + 1), cz = c / ((TX + 1) * (TY + 1));
    if (cx < wx && cy < wy && cz < wz) {
      const int at = x0 + cx + n1 * (y0 + cy) + n2 * (z0 + cz);
      const int l = cx - Q::blo[0] + S1 * (cy - Q::blo[1]) + S2 * (cz - Q::blo[2]);
#pragma unroll
      for (int gr = 0; gr < G; ++gr)
        if (Q::wr[gr]) ((in_alt >> gr) & 1u ? xw : altw)[dv + gr * nn + at] = box[gr * SG + l];
    }
  }
}

// The velocity sweeps of one Uzawa iteration on a small level, one workgroup
// per component: the component lives in LDS with compile-time strides, every
// thread owns its sites of each colour (their f - B^T p stays in registers,
// p being fixed), and a colour is a barrier apart from the next instead of a
// launch apart.  Bound by the chain of colours: Taylor-Hood, N = 8, three
// sweeps: 27 launches of 3.2 us before, 20.6 us in one launch now (0.6 us per
// colour); P1, N = 16, three sweeps: 6 x 3.1 -> 12.6 us.
template <typename T, int G, int N, int NT, bool VAR>
__global__ void __launch_bounds__(NT) k_gs_level(LevelConst<T> lc, T* __restrict__ x, const T* __restrict__ pv,
                                                 const T* __restrict__ b, int xi, int sym) {
  using R = BoxRows<G>;
  constexpr int S1 = N + 1, S2 = S1 * S1, nn = S2 * S1, VS = G * nn, NC = gs_colours(G);
  __shared__ T box[VS + nn + (VAR ? nn : 0)];
  const int tid = threadIdx.x, d = blockIdx.x;
  T* __restrict__ xd = x + d * VS;
  const T* __restrict__ bd = b + d * VS;
  for (int c = tid; c < VS; c += NT) box[c] = xd[c];
  for (int c = tid; c < nn; c += NT) box[VS + c] = pv[c];
  if constexpr (VAR)
    for (int c = tid; c < nn; c += NT) box[VS + nn + c] = lc.nu[c];
  constexpr auto grp = [](int c) constexpr { return c < kGsVertexColours ? 0 : c - kGsVertexColours + 1; };
  constexpr auto dim = [](int c, int axis) constexpr {
    const int g = c < kGsVertexColours ? 0 : c - kGsVertexColours + 1;
    return N - 1 + gdir(G, g, axis);
  };
  // sites of colour c: (i, j, k) over the group's interior box; a vertex
  // colour takes every other i of a row
  constexpr auto count = [](int c) constexpr {
    const int g = c < kGsVertexColours ? 0 : c - kGsVertexColours + 1;
    const int w = N - 1 + gdir(G, g, 0);
    return (c < kGsVertexColours ? (w + 1) / 2 : w) * (N - 1 + gdir(G, g, 1)) * (N - 1 + gdir(G, g, 2));
  };
  constexpr int PV = (count(0) + NT - 1) / NT, PE = (count(NC - 1) + NT - 1) / NT;
  constexpr int P = PV > PE ? PV : PE;
  static_assert(G == 1 || PE * NT >= N * N * (N - 1), "passes cover every edge group");
  int lp[NC][P];
  T f[NC][P], ai[VAR ? NC : 1][P];
  auto colours = [&](auto&& fn) {
    auto go = [&](auto self, auto cc) {
      constexpr int c = decltype(cc)::value;
      if constexpr (c < NC) {
        fn(cc);
        self(self, std::integral_constant<int, c + 1>{});
      }
    };
    go(go, std::integral_constant<int, 0>{});
  };
  colours([&](auto cc) {
    constexpr int c = decltype(cc)::value, g = grp(c);
    constexpr bool half = c < kGsVertexColours;
    constexpr int W = half ? (dim(c, 0) + 1) / 2 : dim(c, 0), H = dim(c, 1);
#pragma unroll
    for (int q = 0; q < P; ++q) {
      const int t = tid + q * NT;
      const int w = t % W, r = t / W;
      const int j = 1 - gdir(G, g, 1) + r % H, k = 1 - gdir(G, g, 2) + r / H;
      const int i = half ? 1 + ((c + 1 + j + k) & 1) + 2 * w : 1 - gdir(G, g, 0) + w;
      const bool on = t < count(c) && i <= N - 1;
      const int l = g * nn + i + S1 * j + S2 * k;
      lp[c][q] = on ? l : -1;
      f[c][q] = on ? bd[l] : T(0);
      if constexpr (VAR) ai[c][q] = on ? lc.ainv_site[l] : T(0);
    }
  });
  __syncthreads();
  const T sa = lc.a / T(R::denA), sb = lc.b / T(R::denT);
  colours([&](auto cc) {
    constexpr int c = decltype(cc)::value, g = grp(c);
#pragma unroll
    for (int q = 0; q < P; ++q)
      if (lp[c][q] >= 0) f[c][q] -= sb * R::template BT<T, g, S1, S2>(box + VS - g * nn + lp[c][q], d);
  });
  auto relax = [&](auto cc) {
    constexpr int c = decltype(cc)::value, g = grp(c);
#pragma unroll
    for (int q = 0; q < P; ++q)
      if (lp[c][q] >= 0) {
        T* u = box + lp[c][q];
        if constexpr (VAR)
          *u += (f[c][q] - lc.a * R::template Anu<T, g, S1, S2, nn>(u, box + VS + nn + lp[c][q] - g * nn)) * ai[c][q];
        else
          *u += (f[c][q] - sa * R::template A<T, g, S1, S2, nn>(u)) * lc.ainv[g];
      }
    __syncthreads();
  };
#pragma unroll 1
  for (int s = 0; s < xi; ++s) {
    colours(relax);
    // the turn's colour is idempotent and not repeated
    if (sym)
      colours([&](auto cc) {
        if constexpr (decltype(cc)::value > 0) relax(std::integral_constant<int, NC - 1 - decltype(cc)::value>{});
      });
  }
  for (int c = tid; c < VS; c += NT) xd[c] = box[c];
}

// ------------------------------------------- Gauss-Seidel runs along k
// The same runs on the large levels: a workgroup owns a tile of columns (and a
// range of planes) and marches along k with a ring of the last planes in LDS.
// Each wavefront belongs to one colour of the run; at iteration q colour s
// updates plane q - skew[s], far enough behind the earlier colours that all of
// them run in the same iteration, one barrier per plane.  Planes are loaded
// kMarchDepth iterations ahead into registers, so that an iteration does not
// wait for memory (loaded within it: N = 64 586 against 381 us, three ahead
// the same as two), and a word is read once per run for the tile's own columns
// (and by the neighbour tiles that need it in their layers, from the L2).
// N = 256 is bound by the memory: 1.7 - 1.9 ms per run in float64 for 27 arrays
// read with 1.2 times the words and the right-hand sides and results of its
// groups (4.4 TB/s by the L2's misses), and three runs pass over the arrays
// instead of nine launches.  N = 64 is bound by the plane's latency: LDS reads,
// arithmetic and a barrier, 0.9 us.  Tiles of 16 x 8: with 8 x 8 two
// workgroups fit a CU and the layers grow (N = 256 7.8 -> 9.0 ms, N = 64 381 ->
// 438 us); larger ones exceed the LDS or the 1024 threads.
constexpr int kMarchDepth = 2;
constexpr int kCUs = 256;

template <typename Q, int TX, int TY>
struct MarchShape {
  static constexpr int G = Q::G;
  static constexpr int BX = TX + Q::bhi[0] - Q::blo[0], BY = TY + Q::bhi[1] - Q::blo[1];
  static constexpr int cells = BX * BY, PS = cells * (G + 1);
  static constexpr int last = Q::skew[Q::n - 1], W = last + 4;  // planes q - last - 1 .. q + 2
  static constexpr int words = PS * W;
  static constexpr int grp(int s) { return Q::col[s] < kGsVertexColours ? 0 : Q::col[s] - kGsVertexColours + 1; }
  static constexpr bool half(int s) { return Q::col[s] < kGsVertexColours; }
  static constexpr int SX(int s) { return (TX + Q::hi[s][0] - Q::lo[s][0] + (half(s) ? 1 : 0)) / (half(s) ? 2 : 1); }
  static constexpr int SY(int s) { return TY + Q::hi[s][1] - Q::lo[s][1]; }
  // lanes per row: the box's pitch for whole rows, so that a wavefront's words
  // are contiguous in LDS and meet no bank twice
  static constexpr int PX(int s) { return half(s) ? SX(s) : BX; }
  static constexpr int waves(int s) { return (PX(s) * SY(s) + 63) / 64; }
  static constexpr int first(int s) { return s == 0 ? 0 : first(s - 1) + waves(s - 1); }
  static constexpr int NT = 64 * first(Q::n);
  static constexpr int SW = (PS + NT - 1) / NT;  // words of a plane per thread
  static constexpr int nwr() {
    int n = 0;
    for (int gr = 0; gr < G; ++gr) n += Q::wr[gr];
    return n;
  }
  static constexpr int wgroup(int a) {  // the a-th written group
    int gr = 0;
    for (;; ++gr)
      if (Q::wr[gr] && a-- == 0) return gr;
  }
  static constexpr int OC = (TX + 1) * (TY + 1), OW = (nwr() * OC + NT - 1) / NT;
  // first iteration with a plane to update, relative to the first output plane
  static constexpr int q0() {
    int q = Q::lo[0][2] + Q::skew[0];
    for (int s = 1; s < Q::n; ++s) q = q < Q::lo[s][2] + Q::skew[s] ? q : Q::lo[s][2] + Q::skew[s];
    return q;
  }
  static constexpr int pro = q0() + 2 - Q::blo[2];  // planes in the ring before it
  // what the ring's length and the write-back rely on: no step is further behind
  // than the last, and the planes before the first iteration fit the ring
  static constexpr int most() {
    int m = 0;
    for (int s = 0; s < Q::n; ++s) m = m > Q::skew[s] ? m : Q::skew[s];
    return m;
  }
  static_assert(last == most() && pro >= 1 && pro <= W, "ring of planes");
};

// The march of the wavefronts of colour s.
template <typename T, typename Q, int TX, int TY, int d, int s>
__device__ __forceinline__ void march(const Geom& g, const LevelConst<T>& lc, const T* x, const T* alt, T* out,
                                      const T* __restrict__ pv, const T* __restrict__ b, unsigned in_alt, int x0,
                                      int y0, int za, int zb, T* ring) {
  using Sh = MarchShape<Q, TX, TY>;
  using R = BoxRows<Q::G>;
  constexpr int G = Q::G, S1 = Sh::BX, SG = Sh::cells, W = Sh::W, PS = Sh::PS, D = kMarchDepth;
  constexpr int gr = Sh::grp(s), Z = Q::skew[s];
  constexpr bool half = Sh::half(s);
  const int N = g.N, n1 = g.n1, n2 = g.n1 * g.n1, nn = g.nn;
  const int tid = threadIdx.x;
  const size_t dv = (size_t)d * g.vstride;
  // words of a plane: tid, tid + NT, ... of [array][cell]
  const T* src[Sh::SW];
#pragma unroll
  for (int i = 0; i < Sh::SW; ++i) {
    const int w = min(tid + i * Sh::NT, PS - 1), a = w / SG, cell = w - a * SG, cy = cell / S1;
    const int ci = min(max(x0 + Q::blo[0] + cell - cy * S1, 0), N), cj = min(max(y0 + Q::blo[1] + cy, 0), N);
    src[i] = (a == G ? pv : (((in_alt >> a) & 1u) ? alt : x) + dv + (size_t)a * nn) + ci + n1 * cj;
  }
  auto load = [&](T(&v)[Sh::SW], int plane) {
    const size_t at = (size_t)n2 * (unsigned)min(max(plane, 0), N);
#pragma unroll
    for (int i = 0; i < Sh::SW; ++i) v[i] = src[i][at];
  };
  auto store = [&](const T(&v)[Sh::SW], int slot) {
    T* to = ring + slot * PS + tid;
#pragma unroll
    for (int i = 0; i < Sh::SW; ++i)
      if ((i + 1) * Sh::NT <= PS || tid + i * Sh::NT < PS) to[i * Sh::NT] = v[i];
  };
  // this thread's site of colour s: box column bx (+ 1 by the parity of the
  // plane for the vertex colours), by
  const T sa = lc.a / T(R::denA), sb = lc.b / T(R::denT), ai = lc.ainv[gr];
  const int c = tid - 64 * Sh::first(s);
  const int bx = Q::lo[s][0] - Q::blo[0] + (half ? 2 : 1) * (c % Sh::PX(s));
  const int by = Q::lo[s][1] - Q::blo[1] + c / Sh::PX(s);
  const int i0 = x0 + Q::blo[0] + bx, j0 = y0 + Q::blo[1] + by;
  const int par = x0 + Q::lo[s][0] + j0 + Q::col[s];
  // rows of the plane's interior in x and y (bit 1: one step in x further)
  unsigned ok = 0;
#pragma unroll
  for (int e = 0; e < (half ? 2 : 1); ++e)
    if (c < Sh::PX(s) * Sh::SY(s) && bx + e < TX + Q::hi[s][0] - Q::blo[0] &&
        i0 + e >= 1 - gdir(G, gr, 0) && i0 + e < N && j0 >= 1 - gdir(G, gr, 1) && j0 < N)
      ok |= 1u << e;
  const T* const fb = b + dv + (size_t)gr * nn + min(max(i0, 0), N - 1) + n1 * min(max(j0, 0), N);
  const int klo = max(za + Q::lo[s][2], 1 - gdir(G, gr, 2)), khi = min(zb + Q::hi[s][2], N);
  auto load_f = [&](int q) {
    const int k = min(max(q - Z, 0), N);
    const int e = half ? (par + k) & 1 : 0;
    return fb[(size_t)n2 * (unsigned)k + e];
  };
  // the words this thread writes of a finished plane
  int ol[Sh::OW];
  T* dst[Sh::OW];
  const int wx = x0 + TX == N ? TX + 1 : TX, wy = y0 + TY == N ? TY + 1 : TY;
#pragma unroll
  for (int i = 0; i < Sh::OW; ++i) {
    const int t = tid + i * Sh::NT, a = t / Sh::OC, o = t - a * Sh::OC, oy = o / (TX + 1), ox = o - oy * (TX + 1);
    int og = 0;
#pragma unroll
    for (int w = 0; w < Sh::nwr(); ++w)
      if (a == w) og = Sh::wgroup(w);
    ol[i] = a < Sh::nwr() && ox < wx && oy < wy ? og * SG + ox - Q::blo[0] + S1 * (oy - Q::blo[1]) : -1;
    dst[i] = out + dv + (size_t)og * nn + x0 + ox + n1 * (y0 + oy);
  }
  // planes up to the first iteration's, then D ahead
  const int qa = za + Sh::q0(), qe = zb + Sh::last;
  {
    T v[Sh::pro][Sh::SW];
#pragma unroll
    for (int p = 0; p < Sh::pro; ++p) load(v[p], za + Q::blo[2] + p);
#pragma unroll
    for (int p = 0; p < Sh::pro; ++p) store(v[p], p % W);
  }
  int slot = Sh::pro % W;  // ring slot of plane q + 2
  T v[D][Sh::SW], f[D];
#pragma unroll
  for (int u = 0; u < D; ++u) {
    load(v[u], qa + 2 + u);
    f[u] = load_f(qa + u);
  }
  __syncthreads();
  auto step = [&](int q, T(&vu)[Sh::SW], T& fu) {
    store(vu, slot);
    load(vu, q + 2 + D);
    const int k = q - Z;
    if (k >= klo && k < khi) {
      const int e = half ? (par + k) & 1 : 0;
      if ((ok >> e) & 1u) {
        const int l = bx + e + S1 * by;
        T* u[3];
        const T* p[3];
#pragma unroll
        for (int dk = -1; dk <= 1; ++dk) {
          int sl = slot - (Z + 2 - dk);
          sl = sl < 0 ? sl + W : sl;
          u[dk + 1] = ring + sl * PS + gr * SG + l;
          p[dk + 1] = ring + sl * PS + G * SG + l;
        }
        const T r = fu - sb * R::template BTr<T, gr, S1>(p, d) - sa * R::template Ar<T, gr, S1, SG>(u);
        u[1][0] += r * ai;
        // the row's LDS reads first, then its arithmetic
        __builtin_amdgcn_sched_group_barrier(0x100, 80, 0);
        __builtin_amdgcn_sched_group_barrier(0x2, 200, 0);
      }
    }
    fu = load_f(q + D);
    // the plane that every colour has passed
    const int ko = q - 1 - Sh::last;
    if (ko >= za && ko < zb) {
      int sl = slot - (Sh::last + 3);
      sl = sl < 0 ? sl + W : sl;
#pragma unroll
      for (int i = 0; i < Sh::OW; ++i)
        if (ol[i] >= 0) dst[i][(size_t)n2 * (unsigned)ko] = ring[sl * PS + ol[i]];
    }
    slot = slot + 1 == W ? 0 : slot + 1;
    __syncthreads();
  };
#pragma unroll 1
  for (int q = qa; q <= qe; q += D) {
#pragma unroll
    for (int u = 0; u < D; ++u) step(q + u, v[u], f[u]);
  }
}

template <typename T, typename Q, int TX, int TY>
__global__ void __launch_bounds__((MarchShape<Q, TX, TY>::NT))
    k_gs_march(Geom g, LevelConst<T> lc, const T* x, const T* alt, T* out, const T* __restrict__ pv,
               const T* __restrict__ b, unsigned in_alt, int ltx, int lty, int kc) {
  using Sh = MarchShape<Q, TX, TY>;
  __shared__ T ring[Sh::words];
  // block -> (tile x, tile y, component, planes), x fastest, a contiguous
  // range per XCD
  const int lin = (int)(blockIdx.x & 7) * (int)(gridDim.x >> 3) + (int)(blockIdx.x >> 3);
  const int x0 = (lin & ((1 << ltx) - 1)) * TX, y0 = ((lin >> ltx) & ((1 << lty) - 1)) * TY;
  const int rest = lin >> (ltx + lty);
  const int d = rest % 3, za = (rest / 3) * kc, zb = min(za + kc, g.n1);
  if (za >= g.n1) return;  // grid padding: whole workgroup
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / 64);
  auto go = [&](auto self, auto dc, auto sc) {
    constexpr int s = decltype(sc)::value;
    if constexpr (s < Q::n) {
      if (s == Q::n - 1 || wave < Sh::first(s) + Sh::waves(s))
        march<T, Q, TX, TY, decltype(dc)::value, s>(g, lc, x, alt, out, pv, b, in_alt, x0, y0, za, zb, ring);
      else
        self(self, dc, std::integral_constant<int, s + 1>{});
    }
  };
  const std::integral_constant<int, 0> first{};
  if (d == 0)
    go(go, std::integral_constant<int, 0>{}, first);
  else if (d == 1)
    go(go, std::integral_constant<int, 1>{}, first);
  else
    go(go, std::integral_constant<int, 2>{}, first);
}

}  // namespace

// Sites of colour c (the timer's work units): a vertex colour has the sites of
// one parity, (i + j + k) mod 2 = c, of an odd number per axis.
double colour_sites(const Geom& g, int c) {
  const int gr = c < kGsVertexColours ? 0 : c - kGsVertexColours + 1;
  double n = 1.0;
  for (int a = 0; a < 3; ++a) n *= g.N - 1 + gdir(g.G, gr, a);
  return c < kGsVertexColours ? (n + 2 * c - 1) / 2 : n;
}
template <typename Q>
double run_sites(const Geom& g) {
  double sites = 0;
  for (int q = 0; q < Q::n; ++q) sites += colour_sites(g, Q::col[q]);
  return sites;
}

// One run of colours, from the buffers that hold their groups to the others.
template <typename T, typename Q, int TX, int TY, int TZ, int NT>
void launch_gs_run(hipStream_t s, const Geom& g, const LevelConst<T>& lc, T* x, T* alt, const T* p, const T* b,
                   unsigned& in_alt) {
  auto log2i = [](int v) {
    int l = 0;
    while ((1 << l) < v) ++l;
    return l;
  };
  KScope ks(s, Q::G == 1 ? KF_GS_VERTEX : KF_GS_EDGE, run_sites<Q>(g), true);
  const TileGrid tg{log2i(g.N / TX), log2i(g.N / TY), log2i(g.N / TZ)};
  const dim3 grid(3 << (tg.lx + tg.ly + tg.lz));
  constexpr bool with_nu = !(Q::G == 1 && Q::n > 3);  // no run of four with a viscosity
  HHG_REQUIRE(with_nu || !lc.nu, HHG_ERR_STATE, "internal: no kernel for a run of colours");
  if (with_nu && lc.nu)
    launch_timed(ks, k_gs_box<T, Q, TX, TY, TZ, NT, with_nu>, grid, dim3(NT), s, g, lc, x, alt, x, alt, p, b, in_alt,
                 tg);
  else
    launch_timed(ks, k_gs_box<T, Q, TX, TY, TZ, NT, false>, grid, dim3(NT), s, g, lc, x, alt, x, alt, p, b, in_alt,
                 tg);
  for (int gr = 0; gr < Q::G; ++gr) in_alt ^= (unsigned)Q::wr[gr] << gr;
}

template <typename T, typename Q, int TX, int TY>
void launch_gs_march(hipStream_t s, const Geom& g, const LevelConst<T>& lc, T* x, T* alt, const T* p, const T* b,
                     unsigned& in_alt) {
  using Sh = MarchShape<Q, TX, TY>;
  static_assert(Sh::NT <= 1024 && Sh::words * sizeof(T) <= 160 * 1024, "one workgroup");
  auto log2i = [](int v) {
    int l = 0;
    while ((1 << l) < v) ++l;
    return l;
  };
  KScope ks(s, Q::G == 1 ? KF_GS_VERTEX : KF_GS_EDGE, run_sites<Q>(g), true);
  const int ltx = log2i(g.N / TX), lty = log2i(g.N / TY);
  // planes per workgroup: the fewest iterations in turn, with the planes that
  // a range marches besides its own (a workgroup per CU; where LDS holds two,
  // they share its bandwidth).  N = 64: 2 ranges 380 us (1: 609, 4: 443), N =
  // 128: 2 (float64 1115 us, 4: 1199; float32 640, 1: 726, 4: 680), N = 256: 1
  // (7.8 ms, 2: 8.0)
  const int tiles = 3 << (ltx + lty), extra = Sh::last + Sh::pro;
  int kc = g.n1, best = INT_MAX;
  for (int ch = 1; ch <= 8; ++ch) {
    const int planes = (g.n1 + ch - 1) / ch, cost = (tiles * ch + kCUs - 1) / kCUs * (planes + extra);
    if (cost < best) best = cost, kc = planes;
  }
  const int nch = (g.n1 + kc - 1) / kc, blocks = (tiles * nch + 7) & ~7;
  // the groups a run writes are all in the same buffer
  unsigned wr = 0;
  for (int gr = 0; gr < Q::G; ++gr) wr |= (unsigned)Q::wr[gr] << gr;
  HHG_REQUIRE((in_alt & wr) == 0 || (in_alt & wr) == wr, HHG_ERR_STATE, "internal: groups of a run in two buffers");
  T* out = (in_alt >> Sh::wgroup(0)) & 1u ? x : alt;
  launch_timed(ks, k_gs_march<T, Q, TX, TY>, dim3(blocks), dim3(Sh::NT), s, g, lc, x, alt, out, p, b, in_alt, ltx, lty,
               kc);
  in_alt ^= wr;
}

template <typename T>
bool gs_runs_supported(const Geom& g, bool varnu, int iters, int xi, bool sym) {
  if (g.nf != 0) return false;
  const bool sweeps = xi * (sym ? 2 : 1) > 1;
  if (g.G == 1) {
    // one float64 iteration of forward sweeps with a viscosity gains less than
    // its copy back costs (below)
    if (varnu && sizeof(T) == 8 && iters == 1 && !sym && (g.N == 64 || (g.N == 128 && xi == 1))) return false;
    return g.N == 32 || (g.N == 64 && sweeps) || g.N > 64;
  }
  return g.N == 16 || g.N == 32 || (!varnu && (g.N > 64 || (g.N == 64 && sizeof(T) == 8 && sweeps)));
}

// Taylor-Hood.  Variable viscosity takes the same runs (float32 V(3,3) with three
// sweeps to N = 64: 4.29 -> 3.00 ms).  Measured per Uzawa iteration with three
// forward sweeps (float64 / float32, constant coefficients), against a launch
// per colour: N = 16 105 -> 49 / 100 -> 42 us with two runs on 4^3 tiles (three
// runs: 53 / 48; 8 x 4 x 4 tiles: 57 / 48), N = 32 125 -> 101 / 110 -> 77 us with
// three runs on 8^3 tiles (4^3 tiles: 130 / 102; 8 x 8 x 4: 117 / 79).  From N =
// 64 on the layers recomputed around boxes cost what the saved passes over
// memory give (three runs on 8^3 tiles 524 us, a launch per colour 410 us);
// there the runs go along k, constant viscosity only: N = 64 float64 410 -> 381
// us, N = 128 with one sweep 1355 -> 1115 / 678 -> 640, symmetric (float32) 1199
// -> 936, N = 256 29.4 -> 18.2 ms (float32, one sweep 6.3 -> 5.1).  A launch per
// colour stays where that is no gain: one sweep at N = 64 (160 against 165 us,
// the copy back included), float32 at N = 64 (250 against 280).
// P1: the colours of the sweeps alternate, a colour next to itself (the turn of
// a symmetric sweep) being idempotent; they are cut into runs of nearly equal
// length.  Smoothing calls with three sweeps, a launch per colour -> now, us
// (float64 / float32): N = 32 28.0 -> 20.6 / 24.5 -> 17.8 (8^3 boxes, runs of
// three; of two 22.6 / 20.2), N = 64 53.7 -> 49.6 / 45.7 -> 36.4 (16 x 8 x 8
// boxes, runs of two / four: with 4-byte words four fit two workgroups per
// CU), N = 128 302 -> 226 / 200 -> 160 and N = 256 2842 -> 1878 / 1836 -> 1049
// (along k on 16 x 16 / 32 x 8 tiles, runs of two at N = 128 in float64, else
// of three; boxes 246 / 170 and 2406 / 1384).  One forward sweep at N = 64 is
// two launches either way with the copy back (28.1 against 28.6 us): a launch
// per colour there.  Variable viscosity: on boxes at every size, the runs of at
// most three from N = 64 on in float32 (with the viscosity a run of four fills
// the LDS and the registers: two sweeps at N = 128, a launch per colour 177 us,
// one run of four 222, two of two 156).  One float64 iteration of forward
// sweeps at N = 64 (three: 61.9 against 65.3 us) and of one at N = 128 (171
// against 179) keeps a launch per colour, two and more (124 against 120) do not.
template <typename T>
void launch_gs_runs(hipStream_t s, const Geom& g, const LevelConst<T>& lc, T* x, T* alt, const T* p, const T* b,
                    int xi, bool sym, unsigned& in_alt) {
#define HHG_RUN(Q, ...) launch_gs_run<T, gen::Q, __VA_ARGS__>(s, g, lc, x, alt, p, b, in_alt)
#define HHG_MARCH(Q, ...) launch_gs_march<T, gen::Q, __VA_ARGS__>(s, g, lc, x, alt, p, b, in_alt)
  if (g.G == 1) {
    const bool along_k = g.N > 64 && !lc.nu;
    const int total = sym ? 2 * xi + 1 : 2 * xi;
    const bool f64 = sizeof(T) == 8;
    const int most = g.N == 32 ? 3 : (along_k ? (f64 && g.N == 128 ? 2 : 3) : (f64 ? 2 : (lc.nu ? 3 : 4)));
    const int runs = (total + most - 1) / most;
    for (int done = 0, r = 0; r < runs; ++r) {
      const int len = (total - done + runs - r - 1) / (runs - r);
      // the runs that the cuts make (those of one colour start at colour 0, those
      // of four too)
      bool launched = false;
#define HHG_P1(S_, L_)                                                                  \
  if ((done & 1) == S_ && len == L_) {                                                  \
    if (along_k) {                                                                      \
      if constexpr (L_ <= 3 && (L_ > 1 || sizeof(T) == 8))                              \
        launched = true, HHG_MARCH(P1Seq##S_##L_, 128 / (int)sizeof(T), 2 * (int)sizeof(T)); \
    } else if (g.N == 32) {                                                             \
      if constexpr (L_ == 2 || L_ == 3) launched = true, HHG_RUN(P1Seq##S_##L_, 8, 8, 8, 512); \
    } else {                                                                            \
      if constexpr (sizeof(T) == 8 ? S_ == 0 && L_ <= 2 : L_ > 1)                       \
        launched = true, HHG_RUN(P1Seq##S_##L_, 16, 8, 8, 512);                         \
    }                                                                                   \
  }
      HHG_P1(0, 1) HHG_P1(0, 2) HHG_P1(0, 3) HHG_P1(0, 4) HHG_P1(1, 2) HHG_P1(1, 3)
#undef HHG_P1
      HHG_REQUIRE(launched, HHG_ERR_STATE, "internal: no kernel for a run of colours");
      done += len;
    }
    return;
  }
  for (int sw = 0; sw < xi * (sym ? 2 : 1); ++sw) {
    const bool backward = sym && (sw & 1);
    if (g.N >= 64) {
      if (!backward) {
        HHG_MARCH(P2Fwd01, 16, 8);
        HHG_MARCH(P2Fwd24, 16, 8);
        HHG_MARCH(P2Fwd58, 16, 8);
      } else {
        HHG_MARCH(P2Bwd85, 16, 8);
        HHG_MARCH(P2Bwd42, 16, 8);
        HHG_MARCH(P2Bwd10, 16, 8);
      }
      continue;
    }
    if (g.N == 16) {
      if (!backward) {
        HHG_RUN(P2Fwd03, 4, 4, 4, 512);
        HHG_RUN(P2Fwd48, 4, 4, 4, 512);
      } else {
        HHG_RUN(P2Bwd84, 4, 4, 4, 512);
        HHG_RUN(P2Bwd30, 4, 4, 4, 512);
      }
    } else {
      if (!backward) {
        HHG_RUN(P2Fwd01, 8, 8, 8, 1024);
        HHG_RUN(P2Fwd24, 8, 8, 8, 1024);
        HHG_RUN(P2Fwd58, 8, 8, 8, 1024);
      } else {
        HHG_RUN(P2Bwd85, 8, 8, 8, 1024);
        HHG_RUN(P2Bwd42, 8, 8, 8, 1024);
        HHG_RUN(P2Bwd10, 8, 8, 8, 1024);
      }
    }
  }
#undef HHG_RUN
#undef HHG_MARCH
}

// Taylor-Hood N <= 8 and P1 N <= 16; P1 N = 16 with one sweep of two colours
// costs less as two launches than the load and write-back around it (smoothing
// call 14.6 against 17.6 us; two sweeps 21.5 against 15.6 us).  With a viscosity
// its element rows on 1024 threads gain in float32 from three sweeps on (call
// 27.2 -> 23.8 us; two sweeps three times 54.7 -> 57.1), in float64 never (three
// sweeps 29.7 -> 32.8, symmetric 19.1 -> 24.5).
template <typename T>
bool gs_level_supported(const Geom& g, bool varnu, int xi, bool sym) {
  if (g.nf != 0) return false;
  if (g.G == 8) return g.N == 4 || g.N == 8;
  const int sweeps = xi * (sym ? 2 : 1);
  return g.N == 8 || (g.N == 16 && (varnu ? sizeof(T) == 4 && sweeps > 2 : sweeps > 1));
}
template <typename T>
void launch_gs_level(hipStream_t s, const Geom& g, const LevelConst<T>& lc, T* x, const T* p, const T* b, int xi,
                     bool sym) {
  const int last = gs_colours(g.G) - 1;  // taken once by a symmetric sweep
  double sweep = sym ? -colour_sites(g, last) : 0.0;
  for (int c = 0; c <= last; ++c) sweep += (sym ? 2 : 1) * colour_sites(g, c);
  KScope ks(s, g.G == 1 ? KF_GS_VERTEX : KF_GS_EDGE, sweep * xi, true);
#define HHG_LEVEL(G_, N_, NT_)                                                                              \
  if (g.G == G_ && g.N == N_) {                                                                             \
    constexpr bool with_nu = !(G_ == 1 && N_ == 16 && sizeof(T) == 8); /* gs_level_supported */             \
    if (with_nu && lc.nu)                                                                                   \
      launch_timed(ks, k_gs_level<T, G_, N_, NT_, with_nu>, dim3(3), dim3(NT_), s, lc, x, p, b, xi, (int)sym); \
    else                                                                                                    \
      launch_timed(ks, k_gs_level<T, G_, N_, NT_, false>, dim3(3), dim3(NT_), s, lc, x, p, b, xi, (int)sym); \
  }
  HHG_LEVEL(8, 8, 512)
  HHG_LEVEL(8, 4, 128)
  HHG_LEVEL(1, 8, 192)
  HHG_LEVEL(1, 16, 1024)
#undef HHG_LEVEL
}

#define HHG_INSTANTIATE(T)                                                                                          \
  template bool gs_runs_supported<T>(const Geom&, bool, int, int, bool);                                            \
  template bool gs_level_supported<T>(const Geom&, bool, int, bool);                                                \
  template void launch_gs_level<T>(hipStream_t, const Geom&, const LevelConst<T>&, T*, const T*, const T*, int,    \
                                   bool);                                                                           \
  template void launch_gs_runs<T>(hipStream_t, const Geom&, const LevelConst<T>&, T*, T*, const T*, const T*, int,  \
                                  bool, unsigned&);

HHG_INSTANTIATE(double)
HHG_INSTANTIATE(float)

}  // namespace hhg
