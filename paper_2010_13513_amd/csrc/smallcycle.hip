// The V-cycle over the smallest levels in one workgroup, specialised on the
// lattice size (gfx950).
//
// On these levels (P1-P1 up to 8, P2-P1 up to 4 intervals per edge) the whole
// cycle is a chain of short phases, so what counts is the time of one phase:
// every vector lives in LDS with compile-time strides (a stencil entry is an
// immediate offset of one address, no address arithmetic), the sites a thread
// updates and their f - B^T p stay in registers over the sweeps of an Uzawa
// iteration, and the boundary classes of the pressure rows are a weight table
// in LDS.  Per-phase cost is then a barrier, the LDS latency and one row.
#include <type_traits>

#include "kernels.h"
#include "lanes.h"
#include "lattice.h"

#include "generated/stencils.inc"
#include "boxrows.h"

namespace hhg {
namespace {

// Entries and weights of the pressure rows (all boundary classes).
template <int G>
struct PRows;
template <>
struct PRows<1> {
  static constexpr int n = gen::p1_Pn, m = 4;
  static constexpr const int (&off)[gen::p1_Pn][4] = gen::p1_Poff;
  static __device__ __forceinline__ const double* w() { return gen::p1_Pw; }
};
template <>
struct PRows<8> {
  static constexpr int n = gen::p2_Pn, m = 3;
  static constexpr const int (&off)[gen::p2_Pn][4] = gen::p2_Poff;
  static __device__ __forceinline__ const double* w() { return gen::p2_Pw; }
};

template <int G, int N>
struct Shape {
  static constexpr int S1 = N + 1, S2 = S1 * S1, nn = S2 * S1, VS = G * nn, words = 3 * VS + nn;
  static constexpr int NC = gs_colours(G);
  static constexpr int grp(int c) { return c < kGsVertexColours ? 0 : c - kGsVertexColours + 1; }
  static constexpr int dim(int g, int axis) { return N - 1 + gdir(G, g, axis); }
  static constexpr int width(int c) {
    return c < kGsVertexColours ? (dim(0, 0) + 1) / 2 : dim(grp(c), 0);
  }
  static constexpr int count(int c) { return width(c) * dim(grp(c), 1) * dim(grp(c), 2); }
  static constexpr int most() {
    int m = 0;
    for (int c = 0; c < NC; ++c) m = m > count(c) ? m : count(c);
    return m;
  }
  // wavefronts per velocity component in the sweeps (every colour in one pass)
  static constexpr int waves = most() == 0 ? 1 : (most() + 63) / 64;
};
// Intervals of the smallest lattice of a hierarchy (Taylor-Hood on one interval
// is refused at creation).
template <int G>
constexpr int kSmallest = G == 1 ? 1 : 2;
// LDS layout: the weight table, then [x | b] (and the vertex viscosities when
// they vary) of every level from the top down to the smallest lattice, then one
// residual vector of the top level's size.
template <int G, int NTOP, bool VAR>
struct Layout {
  static constexpr int NMIN = kSmallest<G>;
  static constexpr int table = 27 * PRows<G>::n * PRows<G>::m;
  template <int N>
  static constexpr int xoff() {
    if constexpr (N >= NTOP) return table;
    else return xoff<2 * N>() + 2 * Shape<G, 2 * N>::words + (VAR ? Shape<G, 2 * N>::nn : 0);
  }
  static constexpr int roff = xoff<NMIN>() + 2 * Shape<G, NMIN>::words + (VAR ? Shape<G, NMIN>::nn : 0);
  static constexpr int words = roff + Shape<G, NTOP>::words;
};

template <typename T, int G, int NTOP, int NT, bool VAR>
struct Cycle {
  using L = Layout<G, NTOP, VAR>;
  using R = BoxRows<G>;
  using PR = PRows<G>;
  static constexpr int NW = NT / 64;
  const SmallLevel<T>* lv;
  const SmallCycle<T>& sc;
  T* box;
  double* red;  // max(2 NW, NT) doubles
  int tid, wave, lane;

  template <int N>
  __device__ __forceinline__ T* X() const { return box + L::template xoff<N>(); }
  template <int N>
  __device__ __forceinline__ T* B() const { return box + L::template xoff<N>() + Shape<G, N>::words; }
  template <int N>
  __device__ __forceinline__ T* Nu() const { return box + L::template xoff<N>() + 2 * Shape<G, N>::words; }
  __device__ __forceinline__ T* Rv() const { return box + L::roff; }

  // A's row of group g at velocity word l of component d; sa: unit of the
  // integer weights (or, with a viscosity, of the element rows).
  template <int N, int g>
  __device__ __forceinline__ T arow(T sa, const T* x, int l, int d) const {
    using S = Shape<G, N>;
    if constexpr (VAR)
      return sa * R::template Anu<T, g, S::S1, S::S2, S::nn>(x + l, Nu<N>() + l - d * S::VS - g * S::nn);
    else
      return sa * R::template A<T, g, S::S1, S::S2, S::nn>(x + l);
  }

  // Slice s of the pressure row at node t: B's component s, or (P1, s = 3)
  // the C row; weights at h = 1, table [entry][slice][class] (lanes of
  // different classes read different banks).  An entry outside the cube
  // weighs zero and meets a word that is finite unless one that some row uses
  // is not: x's own, the table or the level above's viscosity or right-hand side
  // of the pressure below them, for P1's C rows b's boundary sites above them
  // (staged as zero).
  template <int N>
  __device__ __forceinline__ T prow_slice(const T* x, int t, int s) const {
    using S = Shape<G, N>;
    const int i = t % S::S1, j = (t / S::S1) % S::S1, k = t / S::S2;
    const T* w = box + (bcls3(i, N) + 3 * bcls3(j, N) + 9 * bcls3(k, N)) + 27 * s;
    const T* u = x + s * S::VS + t;
    T a = 0, c = 0;
#pragma unroll
    for (int e = 0; e < PR::n; ++e) {
      T& acc = e & 1 ? c : a;
      acc = fma(w[e * PR::m * 27],
                u[PR::off[e][0] * S::nn + PR::off[e][1] + PR::off[e][2] * S::S1 + PR::off[e][3] * S::S2], acc);
    }
    return a + c;
  }
  // Every slice of every pressure row into part[slice][node]; then a barrier.
  template <int N>
  __device__ __forceinline__ void prow_parts(const T* x, T* part) const {
    using S = Shape<G, N>;
#pragma unroll 1
    for (int t = tid; t < PR::m * S::nn; t += NT) {
      const int s = t / S::nn;
      part[t] = prow_slice<N>(x, t - s * S::nn, s);
    }
    __syncthreads();
  }
  template <int N>
  __device__ __forceinline__ T prow_residual(const LevelConst<T>& lc, const T* b, const T* part, int t) const {
    using S = Shape<G, N>;
    T y = lc.b * (part[t] + part[S::nn + t] + part[2 * S::nn + t]);
    if (G == 1) y -= lc.c * part[(PR::m - 1) * S::nn + t];
    return b[3 * S::VS + t] - y;
  }

  // Order the LDS accesses of one component's wavefronts between two colours:
  // one wavefront runs them in program order, more need the barrier.
  template <int N>
  __device__ __forceinline__ void colour_sync() const {
    if constexpr (Shape<G, N>::waves == 1) {
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    } else {
      __syncthreads();
    }
  }

  // iters >= 0 Uzawa iterations on x, then (want_r) r = b - calA x, boundary
  // velocity rows zero.  The sweeps of component d run on wavefronts d W ..
  // d W + W - 1 (W = Shape::waves), one site per thread and colour.
  template <int N>
  __device__ __forceinline__ void smooth(int q, int iters, bool want_r) const {
    using S = Shape<G, N>;
    constexpr int W = S::waves;
    static_assert(3 * W <= NW, "a component's wavefronts");
    const LevelConst<T>& lc = lv[q].lc;
    T* x = X<N>();
    const T* b = B<N>();
    T* r = Rv();
    const T sa = VAR ? lc.a : lc.a / T(R::denA), sb = lc.b / T(R::denT);
    const int d = wave / W;
    const bool act = d < 3;
    const int ct = tid - d * (64 * W);
    auto colours = [&](auto&& fn) {
      auto go = [&](auto self, auto cc) {
        constexpr int c = decltype(cc)::value;
        if constexpr (c < S::NC) {
          fn(cc);
          self(self, std::integral_constant<int, c + 1>{});
        }
      };
      go(go, std::integral_constant<int, 0>{});
    };
    int lp[S::NC];
    T f[S::NC], ai[S::NC];
    colours([&](auto cc) {
      constexpr int c = decltype(cc)::value, g = S::grp(c), M = S::count(c);
      constexpr bool half = c < kGsVertexColours;
      lp[c] = -1;
      f[c] = 0;
      ai[c] = VAR ? T(0) : lc.ainv[g];
      if constexpr (M > 0) {
        constexpr int Wd = S::width(c), H = S::dim(g, 1);
        const int w = ct % Wd, rr = ct / Wd;
        const int j = 1 - gdir(G, g, 1) + rr % H, k = 1 - gdir(G, g, 2) + rr / H;
        const int i = half ? 1 + ((c + 1 + j + k) & 1) + 2 * w : 1 - gdir(G, g, 0) + w;
        if (act && ct < M && i <= N - 1) {
          const int at = g * S::nn + i + S::S1 * j + S::S2 * k;
          lp[c] = d * S::VS + at;
          if constexpr (VAR) ai[c] = lc.ainv_site[at];
        }
      }
    });
    constexpr int PP = (S::nn + NT - 1) / NT;
    T dn[PP];
#pragma unroll
    for (int p = 0; p < PP; ++p) dn[p] = tid + p * NT < S::nn ? lv[q].dinv[tid + p * NT] : T(0);
    if (want_r)
      for (int t = tid; t < 3 * S::VS; t += NT) r[t] = T(0);
    // the last pass (it == iters) is the residual alone
    const int passes = iters + (want_r ? 1 : 0);
#pragma unroll 1
    for (int it = 0; it < passes; ++it) {
      const bool last = it == iters;
      if (act) {
        const T* pd = x + 3 * S::VS - d * S::VS;
        colours([&](auto cc) {
          constexpr int c = decltype(cc)::value, g = S::grp(c);
          if (lp[c] >= 0) f[c] = b[lp[c]] - sb * R::template BT<T, g, S::S1, S::S2>(pd + lp[c] - g * S::nn, d);
        });
      }
      if (last) {
        if (act)
          colours([&](auto cc) {
            constexpr int c = decltype(cc)::value, g = S::grp(c);
            if (lp[c] >= 0) f[c] -= arow<N, g>(sa, x, lp[c], d);
          });
      } else {
        auto relax = [&](auto cc) {
          constexpr int c = decltype(cc)::value, g = S::grp(c);
          if constexpr (S::count(c) > 0) {
            if (lp[c] >= 0) x[lp[c]] += (f[c] - arow<N, g>(sa, x, lp[c], d)) * ai[c];
            colour_sync<N>();
          }
        };
        if (W > 1 || act) {
#pragma unroll 1
          for (int s = 0; s < sc.xi; ++s) {
            colours(relax);
            // the turn's colour is idempotent and not repeated
            if (sc.gs_sym)
              colours([&](auto cc) {
                if constexpr (decltype(cc)::value > 0)
                  relax(std::integral_constant<int, S::NC - 1 - decltype(cc)::value>{});
              });
          }
        }
        __syncthreads();
      }
      // pressure rows: r_p = g - B u + C p; the step p -= omega D^{-1} r_p,
      // or (last) r_p stored.  The partial sums go where r is not needed:
      // before the residual, r itself; then the coarse level's vectors are
      // still unused.
      T* part = last ? scratch<N>() : r;
      prow_parts<N>(x, part);
#pragma unroll
      for (int p = 0; p < PP; ++p) {
        const int t = tid + p * NT;
        if (t < S::nn) {
          const T rp = prow_residual<N>(lc, b, part, t);
          if (last)
            r[3 * S::VS + t] = rp;
          else
            x[3 * S::VS + t] -= sc.omega * dn[p] * rp;
        }
      }
      if (last && act)
        colours([&](auto cc) {
          constexpr int c = decltype(cc)::value;
          if (lp[c] >= 0) r[lp[c]] = f[c];
        });
      if (!last && it + 1 == iters && want_r) {  // r held partial sums: clear them
        __syncthreads();
        for (int t = tid; t < PR::m * S::nn && t < 3 * S::VS; t += NT) r[t] = T(0);
      }
      __syncthreads();
    }
  }
  // Partial sums of the residual's pressure rows: 3 nn (4 nn for P1) words.
  // Taylor-Hood: the next level's vectors, still unused.  P1: the spare words.
  template <int N>
  __device__ __forceinline__ T* scratch() const {
    if constexpr (G == 8) {
      static_assert(3 * Shape<8, N>::nn <= 2 * Shape<8, N / 2>::words, "fits the coarse vectors");
      return X<N / 2>();
    } else {
      return box + L::words;
    }
  }

  // p -= sum_k w_k p_k / sum_k w_k, w_k = int psi_k (mode 0) or 1 (mode 1).
  template <int N>
  __device__ __forceinline__ void shift(int q, T* p, int mode) const {
    using S = Shape<G, N>;
    double a = 0.0, m = 0.0;
    for (int t = tid; t < S::nn; t += NT) {
      double w = 1.0;
      if (mode == 0)
        w = (double)lv[q].tb->mclass[bcls3(t % S::S1, N) + 3 * bcls3((t / S::S1) % S::S1, N) + 9 * bcls3(t / S::S2, N)];
      a += w * (double)p[t];
      m += w;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      a += __shfl_xor(a, o);
      m += __shfl_xor(m, o);
    }
    if (lane == 0) {
      red[2 * wave] = a;
      red[2 * wave + 1] = m;
    }
    __syncthreads();
    double sa = 0.0, sm = 0.0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      sa += red[2 * w];
      sm += red[2 * w + 1];
    }
    const double mean = sa / sm;
    for (int t = tid; t < S::nn; t += NT) p[t] = (T)((double)p[t] - mean);
    __syncthreads();
  }

  // b of the coarse level = R r with the pressure shifted to zero sum; x = 0.
  // Taylor-Hood: a wavefront per group (one gather's code each).
  template <int N>
  __device__ __forceinline__ void restrict_to(int q) const {
    using F = Shape<G, N>;
    constexpr int NC = N / 2;
    using C = Shape<G, NC>;
    const T* r = Rv();
    T* cb = B<NC>();
    T* cx = X<NC>();
    for (int t = tid; t < C::words; t += NT) cx[t] = T(0);
    auto site = [&](int t, int& i, int& j, int& k) {
      i = t % C::S1, j = (t / C::S1) % C::S1, k = t / C::S2;
      return 2 * i + F::S1 * 2 * j + F::S2 * 2 * k;
    };
    static_assert(G == 1 || NW >= 8, "a wavefront per group");
    const int g = G == 1 ? 0 : wave;
    if (g < G) {
#pragma unroll 1
      for (int t = G == 1 ? tid : lane; t < 3 * C::nn; t += G == 1 ? NT : 64) {
        const int d = t / C::nn, c = t - d * C::nn;
        int i, j, k;
        const int fb = site(c, i, j, k);
        const T* rd = r + d * F::VS;
        T a0 = 0, a1 = 0, a2 = 0;
        if (vel_interior<G>(g, i, j, k, NC)) {
          if constexpr (G == 1) {
            gen::p1_R_g0<T>(rd, fb, F::S1, F::S2, F::nn, 0, a0, a1, a2);
          } else {
            switch (g) {
              case 0: gen::p2_R_g0<T>(rd, fb, F::S1, F::S2, F::nn, 0, a0, a1, a2); break;
              case 1: gen::p2_R_g1<T>(rd, fb, F::S1, F::S2, F::nn, 0, a0, a1, a2); break;
              case 2: gen::p2_R_g2<T>(rd, fb, F::S1, F::S2, F::nn, 0, a0, a1, a2); break;
              case 3: gen::p2_R_g3<T>(rd, fb, F::S1, F::S2, F::nn, 0, a0, a1, a2); break;
              case 4: gen::p2_R_g4<T>(rd, fb, F::S1, F::S2, F::nn, 0, a0, a1, a2); break;
              case 5: gen::p2_R_g5<T>(rd, fb, F::S1, F::S2, F::nn, 0, a0, a1, a2); break;
              case 6: gen::p2_R_g6<T>(rd, fb, F::S1, F::S2, F::nn, 0, a0, a1, a2); break;
              default: gen::p2_R_g7<T>(rd, fb, F::S1, F::S2, F::nn, 0, a0, a1, a2); break;
            }
          }
        }
        (void)a1, (void)a2;
        cb[d * C::VS + g * C::nn + c] = a0;
      }
    }
#pragma unroll 1
    for (int t = NT - 1 - tid; t < C::nn; t += NT) {
      int i, j, k;
      const int fb = site(t, i, j, k);
      const T* pf = r + 3 * F::VS;
      cb[3 * C::VS + t] = G == 1 ? gen::p1_RP<T>(pf, fb, 2 * i, 2 * j, 2 * k, N, F::S1, F::S2)
                                 : gen::p2_RP<T>(pf, fb, 2 * i, 2 * j, 2 * k, N, F::S1, F::S2);
    }
    __syncthreads();
    shift<NC>(q - 1, cb + 3 * C::VS, 1);
  }

  // x += I x_coarse on interior velocity sites and every pressure node, by
  // coarse cubes: the cube's coarse words, then the eight fine sites of one
  // fine group (Taylor-Hood: a wavefront per group).
  template <int N>
  __device__ __forceinline__ void prolong_from() const {
    using F = Shape<G, N>;
    constexpr int NC = N / 2;
    using C = Shape<G, NC>;
    const T* xc = X<NC>();
    T* x = X<N>();
    auto cube = [&](int t, int d, int g, bool pres) {
      const int i = t % C::S1, j = (t / C::S1) % C::S1, k = t / C::S2;
      const int oi = i < NC ? 1 : 0, oj = j < NC ? C::S1 : 0, ok = k < NC ? C::S2 : 0;
      const T* src = xc + d * C::VS + t;
      T c[27], v[8];
      if (G == 8 && !pres) {
#pragma unroll
        for (int e = 0; e < 27; ++e) {
          const int a = e % 3, bb = (e / 3) % 3, ee = e / 9;
          constexpr int kGroupOfParity[8] = {0, 1, 2, 4, 3, 5, 6, 7};
          c[e] = src[kGroupOfParity[(a & 1) + 2 * (bb & 1) + 4 * (ee & 1)] * C::nn + (a == 2 ? oi : 0) +
                     (bb == 2 ? oj : 0) + (ee == 2 ? ok : 0)];
        }
        if constexpr (G == 8) gen::p2_Pc<T>(g, c, v);
      } else {
#pragma unroll
        for (int e = 0; e < 27; ++e) {
          const int a = e % 3, bb = (e / 3) % 3, ee = e / 9;
          c[e] = (a == 1 || bb == 1 || ee == 1) ? T(0) : src[(a ? oi : 0) + (bb ? oj : 0) + (ee ? ok : 0)];
        }
        gen::p1_Pc_g0<T>(c, v);
      }
      T* dst = x + d * F::VS + g * F::nn + 2 * i + F::S1 * 2 * j + F::S2 * 2 * k;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int fi = 2 * i + (e & 1), fj = 2 * j + ((e >> 1) & 1), fk = 2 * k + (e >> 2);
        const bool in = pres ? fi <= N && fj <= N && fk <= N : vel_interior<G>(g, fi, fj, fk, N);
        if (in) dst[(e & 1) + F::S1 * ((e >> 1) & 1) + F::S2 * (e >> 2)] += v[e];
      }
    };
    if constexpr (G == 1) {
#pragma unroll 1
      for (int t = tid; t < 4 * C::nn; t += NT) cube(t % C::nn, t / C::nn, 0, t >= 3 * C::nn);
    } else {
      if (wave < 8)
#pragma unroll 1
        for (int t = lane; t < 3 * C::nn; t += 64) cube(t % C::nn, t / C::nn, wave, false);
#pragma unroll 1
      for (int t = NT - 1 - tid; t < C::nn; t += NT) cube(t, 3, 0, true);
    }
    __syncthreads();
  }

  // Coarsest level, reached with x = 0: x = K^+ b on the unknowns, zero
  // pressure mean.  K^+ is symmetric: row `row` is read as a column, so
  // consecutive threads read consecutive words; the threads beyond the rows
  // share them, part by part.
  template <int N>
  __device__ __forceinline__ void coarse() const {
    using S = Shape<G, N>;
    T* x = X<N>();
    const T* b = B<N>();
    const int n = sc.nunk;
    const int parts = NT / n > 8 ? 8 : NT / n;  // n <= NT (host-checked)
    const int part = tid / n, row = tid - part * n;
    double acc = 0.0;
    if (part < parts) {
      const int c0 = n * part / parts, c1 = n * (part + 1) / parts;
      double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
      int c = c0;
      for (; c + 4 <= c1; c += 4) {
        a0 += sc.Kp[(size_t)c * n + row] * (double)b[sc.unk[c]];
        a1 += sc.Kp[(size_t)(c + 1) * n + row] * (double)b[sc.unk[c + 1]];
        a2 += sc.Kp[(size_t)(c + 2) * n + row] * (double)b[sc.unk[c + 2]];
        a3 += sc.Kp[(size_t)(c + 3) * n + row] * (double)b[sc.unk[c + 3]];
      }
      for (; c < c1; ++c) a0 += sc.Kp[(size_t)c * n + row] * (double)b[sc.unk[c]];
      acc = (a0 + a1) + (a2 + a3);
    }
    red[tid] = acc;
    __syncthreads();
    if (tid < n) {
      double v = 0.0;
      for (int p = 0; p < parts; ++p) v += red[p * n + tid];
      x[sc.unk[tid]] = (T)v;
    }
    __syncthreads();
    shift<N>(0, x + 3 * S::VS, 0);
  }

  template <int N>
  __device__ __forceinline__ void run(int q) const {
    const int below = sc.nlev - 1 - q;
    smooth<N>(q, sc.pre0 + below * sc.inc, true);
    restrict_to<N>(q);
    if constexpr (N / 2 == kSmallest<G>) {
      coarse<N / 2>();  // q == 1 (host-checked)
    } else {
      if (q == 1)
        coarse<N / 2>();
      else
        run<N / 2>(q - 1);
    }
    prolong_from<N>();
    smooth<N>(q, sc.post0 + below * sc.inc, false);
  }
};

template <typename T, int G, int NTOP, int NT, bool VAR>
__global__ void __launch_bounds__(NT) k_cycle_small(const SmallLevel<T>* __restrict__ lv, SmallCycle<T> sc) {
  using L = Layout<G, NTOP, VAR>;
  using S = Shape<G, NTOP>;
  constexpr int spare = G == 1 ? 4 * S::nn : 0;  // Cycle::scratch
  __shared__ T box[L::words + spare];
  __shared__ double red[NT];
  const int tid = threadIdx.x;
  constexpr int n = PRows<G>::n, m = PRows<G>::m;
#pragma unroll 4
  for (int t = tid; t < L::table; t += NT) {  // [class][entry][slice] -> [entry][slice][class]
    const int cls = t / (n * m), es = t - cls * (n * m);
    box[es * 27 + cls] = (T)PRows<G>::w()[t];
  }
  // b's word t; P1: zero for the words up to (0, 1, 1) of the first component, all
  // on the boundary: no row uses them, and the C rows' entries above the cube
  // meet them (Cycle::prow_slice; from the last pressure one step in i, j and k)
  auto rhs = [&](int t) { return G == 1 && t <= S::S2 + S::S1 ? T(0) : sc.b[t]; };
  if (sc.xc) {
    // an FMG step: boundary values, zero elsewhere, and the level below, whose
    // interpolation is added after the barrier
    using C = Shape<G, NTOP / 2>;
    T* const xc = box + L::template xoff<NTOP / 2>();
#pragma unroll 4
    for (int t = tid; t < S::words; t += NT) {
      const int d = t / S::VS, r = t - d * S::VS, g = r / S::nn, q = r - g * S::nn;
      const int i = q % S::S1, j = (q / S::S1) % S::S1, k = q / S::S2;
      const bool bnd = d < 3 && vel_exists<G>(g, i, j, k, NTOP) && !vel_interior<G>(g, i, j, k, NTOP);
      const T* from = sc.fx ? sc.fx + (size_t)d * sc.fvs + finest_slot<G>(g, i, j, k, sc.fn1, sc.fup) : sc.x + t;
      box[L::table + t] = bnd ? *from : T(0);
      box[L::table + S::words + t] = rhs(t);
    }
#pragma unroll 4
    for (int t = tid; t < C::words; t += NT) xc[t] = sc.xc[t];
  } else {
#pragma unroll 4
    for (int t = tid; t < S::words; t += NT) {
      box[L::table + t] = sc.x[t];
      box[L::table + S::words + t] = rhs(t);
    }
  }
  if constexpr (VAR) {  // every level's viscosity above the coarsest
    auto load = [&](auto self, auto nc, int q) {
      constexpr int N = decltype(nc)::value;
      T* nu = box + L::template xoff<N>() + 2 * Shape<G, N>::words;
      for (int t = tid; t < Shape<G, N>::nn; t += NT) nu[t] = lv[q].lc.nu[t];
      if constexpr (N / 2 > kSmallest<G>)
        if (q > 1) self(self, std::integral_constant<int, N / 2>{}, q - 1);
    };
    load(load, std::integral_constant<int, NTOP>{}, sc.nlev - 1);
  }
  __syncthreads();
  const Cycle<T, G, NTOP, NT, VAR> cy{lv, sc, box, red, tid, __builtin_amdgcn_readfirstlane(tid / 64), tid % 64};
  if (sc.xc) cy.template prolong_from<NTOP>();
  cy.template run<NTOP>(sc.nlev - 1);
  __syncthreads();
  if (sc.mean) cy.template shift<NTOP>(sc.nlev - 1, box + L::table + 3 * S::VS, 0);
  for (int t = tid; t < S::words; t += NT) sc.x[t] = box[L::table + t];
}

}  // namespace

// False (nothing launched) where the general kernel is needed: bfloat16
// levels, a viscosity on some of the levels only (nu: 0 none, 1 all above the
// coarsest, 2 mixed), other lattice sizes, more unknowns than threads, a count of
// smoothing steps below zero on some level (taken as none there).
template <typename T>
bool launch_cycle_small(hipStream_t s, const SmallLevel<T>* lv, const SmallCycle<T>& sc, int ntop, int nu) {
  const int inc = min(0, (sc.nlev - 2) * sc.inc);  // of the lowest level above the coarsest
  if (nu > 1 || sc.q16 > 0 || sc.nlev < 2 || sc.pre0 + inc < 0 || sc.post0 + inc < 0) return false;
  if ((ntop >> (sc.nlev - 1)) < (sc.G == 1 ? kSmallest<1> : kSmallest<8>)) return false;  // run's recursion
#define HHG_SMALL(G_, N_, NT_)                                                                  \
  if (sc.G == G_ && ntop == N_ && sc.nunk <= NT_) {                                             \
    KScope ks(s, KF_SMALL, sc.nlev);                                                            \
    if (nu)                                                                                     \
      hipLaunchKernelGGL((k_cycle_small<T, G_, N_, NT_, true>), dim3(1), dim3(NT_), 0, s, lv, sc); \
    else                                                                                        \
      hipLaunchKernelGGL((k_cycle_small<T, G_, N_, NT_, false>), dim3(1), dim3(NT_), 0, s, lv, sc); \
    return true;                                                                                \
  }
  HHG_SMALL(8, 4, 512)
  HHG_SMALL(1, 8, 768)
  HHG_SMALL(1, 4, 256)
  HHG_SMALL(1, 2, 192)
#undef HHG_SMALL
  return false;
}
template bool launch_cycle_small<double>(hipStream_t, const SmallLevel<double>*, const SmallCycle<double>&, int, int);
template bool launch_cycle_small<float>(hipStream_t, const SmallLevel<float>*, const SmallCycle<float>&, int, int);

}  // namespace hhg
