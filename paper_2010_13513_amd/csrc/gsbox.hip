// Gauss-Seidel sweeps on boxes of the lattice held in LDS (gfx950).
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
    if (sym)
      colours([&](auto cc) { relax(std::integral_constant<int, NC - 1 - decltype(cc)::value>{}); });
  }
  for (int c = tid; c < VS; c += NT) xd[c] = box[c];
}

}  // namespace

// Sites that a run updates (the timer's work units).
template <typename Q>
double run_sites(const Geom& g) {
  double sites = 0;
  for (int q = 0; q < Q::n; ++q) {
    const int gr = Q::col[q] < kGsVertexColours ? 0 : Q::col[q] - kGsVertexColours + 1;
    double n = Q::col[q] < kGsVertexColours ? 0.5 : 1.0;
    for (int a = 0; a < 3; ++a) n *= g.N - 1 + gdir(Q::G, gr, a);
    sites += n;
  }
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
  KScope ks(s, Q::G == 1 ? KF_GS_VERTEX : KF_GS_EDGE, run_sites<Q>(g));
  const TileGrid tg{log2i(g.N / TX), log2i(g.N / TY), log2i(g.N / TZ)};
  const dim3 grid(3 << (tg.lx + tg.ly + tg.lz));
  if (lc.nu)
    hipLaunchKernelGGL((k_gs_box<T, Q, TX, TY, TZ, NT, true>), grid, dim3(NT), 0, s, g, lc, x, alt, x, alt, p, b,
                       in_alt, tg);
  else
    hipLaunchKernelGGL((k_gs_box<T, Q, TX, TY, TZ, NT, false>), grid, dim3(NT), 0, s, g, lc, x, alt, x, alt, p, b,
                       in_alt, tg);
  for (int gr = 0; gr < Q::G; ++gr) in_alt ^= (unsigned)Q::wr[gr] << gr;
}

bool gs_runs_supported(const Geom& g, int xi, bool sym) {
  if (g.nf != 0) return false;
  return g.G == 8 ? g.N == 16 || g.N == 32 : g.N == 32 || (g.N == 64 && xi * (sym ? 2 : 1) > 1) || g.N > 64;
}

// Taylor-Hood.  Variable viscosity takes the same runs (float32 V(3,3) with three
// sweeps to N = 64: 4.29 -> 3.15 ms).  Measured per Uzawa iteration with three
// forward sweeps (float64 / float32, constant coefficients), against a launch
// per colour: N = 16 105 -> 49 / 100 -> 42 us with two runs on 4^3 tiles (three
// runs: 53 / 48; 8 x 4 x 4 tiles: 57 / 48), N = 32 125 -> 101 / 110 -> 77 us with
// three runs on 8^3 tiles (4^3 tiles: 130 / 102; 8 x 8 x 4: 117 / 79).  From N =
// 64 on the layers recomputed around the tiles cost what the saved passes over
// memory give (three runs on 8^3 tiles 524 us, a launch per colour 410 us), so
// a colour stays a launch there.
// P1: the colours of the sweeps alternate, a colour next to itself (the turn of
// a symmetric sweep) being idempotent; they are cut into runs of nearly equal
// length.  Smoothing calls with three sweeps, a launch per colour -> now, us
// (float64 / float32): N = 32 28.0 -> 20.6 / 24.5 -> 17.8 (8^3 tiles, runs of
// three; of two 22.6 / 20.2), N = 64 53.7 -> 49.6 / 45.7 -> 36.4, N = 128 302 ->
// 246 / 200 -> 170, N = 256 2842 -> 2406 / 1836 -> 1384 (16 x 8 x 8 tiles;
// 8^3: 264 / 200 at N = 128).  Runs of four are better where a tile is 4-byte
// words (N = 64 39.7, N = 256 1489 with two) and not with 8 (one workgroup per
// CU then; N = 256 2427).  One forward sweep at N = 64 is two launches either
// way with the copy back (28.1 against 28.6): a launch per colour there.
template <typename T>
void launch_gs_runs(hipStream_t s, const Geom& g, const LevelConst<T>& lc, T* x, T* alt, const T* p, const T* b,
                    int xi, bool sym, unsigned& in_alt) {
#define HHG_RUN(Q, ...) launch_gs_run<T, gen::Q, __VA_ARGS__>(s, g, lc, x, alt, p, b, in_alt)
  if (g.G == 1) {
    const int total = sym ? 2 * xi + 1 : 2 * xi, most = g.N == 32 ? 3 : (sizeof(T) == 4 ? 4 : 2);
    const int runs = (total + most - 1) / most;
    for (int done = 0, r = 0; r < runs; ++r) {
      const int len = (total - done + runs - r - 1) / (runs - r);
#define HHG_P1(S_, L_)                                                                        \
  if ((done & 1) == S_ && len == L_) {                                                        \
    if (g.N == 32) {                                                                          \
      if constexpr (L_ <= 3) HHG_RUN(P1Seq##S_##L_, 8, 8, 8, 512);                            \
    } else {                                                                                  \
      if constexpr (L_ <= 2 || sizeof(T) == 4) HHG_RUN(P1Seq##S_##L_, 16, 8, 8, 512);         \
    }                                                                                         \
  }
      HHG_P1(0, 1) HHG_P1(0, 2) HHG_P1(0, 3) HHG_P1(0, 4)
      HHG_P1(1, 1) HHG_P1(1, 2) HHG_P1(1, 3) HHG_P1(1, 4)
#undef HHG_P1
      done += len;
    }
    return;
  }
  for (int sw = 0; sw < xi * (sym ? 2 : 1); ++sw) {
    const bool backward = sym && (sw & 1);
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
}

// Taylor-Hood N <= 8 and P1 N <= 16; P1 N = 16 with one sweep of two colours
// costs less as two launches than the load and write-back around it (smoothing
// call 14.6 against 17.6 us; two sweeps 21.5 against 15.6 us).
bool gs_level_supported(const Geom& g, int xi, bool sym) {
  if (g.nf != 0) return false;
  return g.G == 8 ? g.N == 4 || g.N == 8 : g.N == 8 || (g.N == 16 && xi * (sym ? 2 : 1) > 1);
}
template <typename T>
void launch_gs_level(hipStream_t s, const Geom& g, const LevelConst<T>& lc, T* x, const T* p, const T* b, int xi,
                     bool sym) {
  const double m = (g.G == 1 ? g.N : 2 * g.N) - 1;
  KScope ks(s, KF_GS_EDGE, m * m * m * xi * (sym ? 2 : 1));
#define HHG_LEVEL(G_, N_, NT_)                                                                                      \
  if (g.G == G_ && g.N == N_) {                                                                                     \
    if (lc.nu)                                                                                                      \
      hipLaunchKernelGGL((k_gs_level<T, G_, N_, NT_, true>), dim3(3), dim3(NT_), 0, s, lc, x, p, b, xi, (int)sym); \
    else                                                                                                            \
      hipLaunchKernelGGL((k_gs_level<T, G_, N_, NT_, false>), dim3(3), dim3(NT_), 0, s, lc, x, p, b, xi, (int)sym); \
  }
  HHG_LEVEL(8, 8, 512)
  HHG_LEVEL(8, 4, 128)
  HHG_LEVEL(1, 8, 192)
  HHG_LEVEL(1, 16, 1024)
#undef HHG_LEVEL
}

#define HHG_INSTANTIATE(T)                                                                                          \
  template void launch_gs_level<T>(hipStream_t, const Geom&, const LevelConst<T>&, T*, const T*, const T*, int,    \
                                   bool);                                                                           \
  template void launch_gs_runs<T>(hipStream_t, const Geom&, const LevelConst<T>&, T*, T*, const T*, const T*, int,  \
                                  bool, unsigned&);

HHG_INSTANTIATE(double)
HHG_INSTANTIATE(float)

}  // namespace hhg
