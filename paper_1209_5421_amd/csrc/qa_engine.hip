// Specialised persistent small-level engine (gfx950).
//
// Below a few thousand cells the K-cycle (Algorithm 2.2, with the nonlinear PCG of Algorithm 2.1 as the coarse
// solver of every level) is a chain of dependent steps on small vectors, run by one workgroup. k_engine in
// qa_solve.hip interprets a generic step list against a level table read at run time. This file holds the variant
// for the common shape of those levels, in which every level size, LDS offset and color of a step is a compile-time
// constant:
//  - the coarsest level is the 64-cell level k = 3, one smoothing sweep, two inner steps of Algorithm 2.1;
//  - on the engine's levels no coupling reaches beyond one cell, so no two cells of one color are coupled;
//  - the top level is k = KT (4, 5 or 6).
//
// What bounds it is the latency of its chain of steps on one CU, so a step is kept to an LDS round trip, the nine
// products of a row and a barrier:
//  - a thread owns whole super-cells (the four cells of one parent, one per color) of a level, two on the 4,096-cell
//    level and one below, and keeps their operator rows, the reciprocals of their diagonals and their entries of
//    f, q0, p0 and the current B^ output u in registers for the whole launch. Global memory is read once, in the
//    prologue. The 1,024-cell level belongs to wavefronts 4 to 7 and the 256-cell level to wavefront 0 of the
//    512-thread workgroup (k = 6), so the two share one set of registers;
//  - LDS holds only what neighbours read: u, one plane per color over the super-cells in row-major order with a ring
//    of zeros around the grid. A neighbour is then a compile-time distance from the super-cell's own place, an
//    immediate offset of the LDS load: no index arithmetic and no test for the grid's edge (an absent slot holds 0
//    and reads the ring or a cell of the ring's row padding). The row stride is 8 mod 16 super-cells, so that a
//    wavefront's 8 x 8 Morton block of super-cells touches every bank alike;
//  - the presmoothing sweep starts from zero, so a phase skips the slots of colors not yet relaxed (their products
//    are zero); the prolongation is folded into the first post-smoothing phase, which reads u + P e_c of its
//    neighbours formed from the presmoothing planes and the coarse correction's plane and writes a second set of
//    planes; quotients by the diagonal take Markstein's correction of numerator x reciprocal (the correctly rounded
//    quotient for a correctly rounded reciprocal) in three instructions; a system with a diagonal too small for its
//    reciprocal takes k_engine_div, the same with divisions;
//  - A p1 is formed for the second inner step instead of A (p1 + beta p0): with (p0, q0), (g, p0), (p1, q0),
//    (p1, A p1), (r, p1) and (r, p0) Algorithm 2.1's beta and alpha1 follow, so a level needs one reduction per inner
//    step. The error of one FP32 preconditioner application against FP64, geometric mean over 120 systems of 256 to
//    1,044,484 unknowns, is 1.31e-6 this way and 1.43e-6 with A (p1 + beta p0);
//  - the whole of B~ on the 256-cell level k = 4, with the coarsest solve below it, runs in a single wavefront: its
//    steps are ordered by the wavefront's in-order LDS accesses, with no workgroup barrier between them.
//  - the FP64 coarsest solve is shared by four wavefronts, the three others holding their columns of the inverse in
//    registers that no level of theirs uses.
// Before, with operators and vectors of the levels below the top in LDS, neighbours by index arithmetic, two
// reductions per second inner step and the coarsest solve in one wavefront, a launch took 71.6 us (FP32, k = 6) and
// 27.3 us (FP64, k = 5); now 31.8 and 15.3 us. Of the FP32 launch's 39 us with a clock read after every step, the
// prologue takes 4, the 4,096-cell level 9, the 1,024-cell level 9 and the eight B^ of the 256-cell level 17, where a
// color phase is 0.1 us (one LDS round trip, nine products), the coarsest solve 0.45 and a reduction 0.25 us.

#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <algorithm>
#include <mutex>
#include <type_traits>
#include <utility>
#include <vector>

#include "qa_internal.hpp"
#include "qa_launch.hpp"
#include "qa_wave.hpp"

namespace qa {

namespace {

constexpr int kFeCoarse = 64;                 // cells of the coarsest level k = 3
constexpr int kFeRedWaves = 8;                // wavefronts of the largest level

template <int C>
using IC = std::integral_constant<int, C>;

// neighbour offsets of Section 4.4 as constants: self, E, NE, N, NW, W, SW, S, SE
constexpr int fe_dx(int s) { return (s == 1 || s == 2 || s == 8) ? 1 : ((s == 4 || s == 5 || s == 6) ? -1 : 0); }
constexpr int fe_dy(int s) { return (s == 2 || s == 3 || s == 4) ? 1 : ((s == 6 || s == 7 || s == 8) ? -1 : 0); }

// the slot S neighbour of the color-C cell of a super-cell: its color and the offset of its super-cell
template <int C, int S>
struct FeNbr {
  static constexpr int ux = (C & 1) + fe_dx(S), uy = (C >> 1) + fe_dy(S);
  static constexpr int color = (ux & 1) | ((uy & 1) << 1);
  static constexpr int ox = ux < 0 ? -1 : (ux > 1 ? 1 : 0), oy = uy < 0 ? -1 : (uy > 1 ? 1 : 0);
};

// geometry of level k: S x S super-cells, padded row stride P, cells per plane PP
template <int K>
struct FeGeo {
  static constexpr int S = 1 << (K - 1), N4 = S * S, N = 4 * N4;
  static constexpr int P = K == 6 ? 40 : 24;
  static constexpr int PP = (S + 2) * P;
};

// LDS of one configuration. In doubles: the first 16 columns of the coarsest inverse (pairs of entries of a lane's row
// side by side), the coarsest right-hand side, the helpers' partial sums and the wavefront sums of the reductions. Then
// in units of T, for every level k = KT .. 4: the presmoothing planes (4), the post-smoothing planes (4) and the plane
// of the next level's correction, and the right-hand side handed to the next level (k > 4; color-major).
template <int KT>
struct FeLayout {
  static constexpr int kAinv = 0, kG3 = 16 * kFeCoarse, kPart = kG3 + kFeCoarse, kRed = kPart + 4 * kFeCoarse,
                       kDoubles = kRed + 2 * 4 * kFeRedWaves;
  __host__ __device__ static constexpr int planes(int k) {  // offset of level k's planes
    int o = 0;
    if (k < 6 && KT >= 6) o += 9 * FeGeo<6>::PP + FeGeo<5>::N;
    if (k < 5 && KT >= 5) o += 9 * FeGeo<5>::PP + FeGeo<4>::N;
    return o;
  }
  static constexpr int t_units = planes(4) + 9 * FeGeo<4>::PP;
  static constexpr int TR = KT == 6 ? 2 : 1;               // super-cells per thread of the top level
  static constexpr int threads = KT == 6 ? 512 : KT == 5 ? 320 : 256;
  template <class T>
  static constexpr size_t bytes() {
    return sizeof(double) * kDoubles + sizeof(T) * static_cast<size_t>(t_units);
  }
};

// a thread's super-cells of one level
template <class T, int TR>
struct FeRows {
  T a[TR][4][9];   // operator rows by color, slot order
  T rd[TR][4];     // 1 / diagonal
  T f[TR][4], q0[TR][4], p0[TR][4], u[TR][4];
};

template <class T>
struct FeArgs {
  Ptr<const double> ainv;       // coarsest inverse, 64 x 64, storage numbering (bitwise symmetric: Y^t Y in one order)
  Ptr<const T> ax[3];           // 9 x n operator of each engine level from the top down (global)
  Ptr<const T> g;               // the top level's right-hand side and result (global)
  Ptr<T> e;
};

template <class F>
__device__ __forceinline__ void for_slots(F f) {
  f(IC<0>{}); f(IC<1>{}); f(IC<2>{}); f(IC<3>{}); f(IC<4>{}); f(IC<5>{}); f(IC<6>{}); f(IC<7>{}); f(IC<8>{});
}

template <class F>
__device__ __forceinline__ void for_colors(F f) {
  f(IC<0>{});
  f(IC<1>{});
  f(IC<2>{});
  f(IC<3>{});
}

template <class F>
__device__ __forceinline__ void for_16(F f) {
  f(IC<0>{}); f(IC<1>{}); f(IC<2>{}); f(IC<3>{}); f(IC<4>{}); f(IC<5>{}); f(IC<6>{}); f(IC<7>{});
  f(IC<8>{}); f(IC<9>{}); f(IC<10>{}); f(IC<11>{}); f(IC<12>{}); f(IC<13>{}); f(IC<14>{}); f(IC<15>{});
}

// the thread index, opaque to the optimiser: places derived from it on the lower levels are formed when such a level
// begins rather than kept in registers across the launch
__device__ __forceinline__ int fe_tid() {
  int t;
  asm volatile("v_mov_b32 %0, %1" : "=v"(t) : "v"(static_cast<int>(threadIdx.x)));
  return t;
}

// Order between the sub-steps of the one-wavefront B~: a wavefront's LDS accesses are performed in issue order, so
// keeping the compiler from moving memory accesses across this point is all that is needed.
__device__ __forceinline__ void fe_wsync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  asm volatile("" ::: "memory");
}

template <bool WAVE>
__device__ __forceinline__ void fe_sync() {
  if constexpr (WAVE) fe_wsync();
  else __syncthreads();
}

// four sums over the level's W wavefronts, the same in every thread: each wavefront's sums as above, then the
// wavefronts' sums added in pairs
template <int W, bool WAVE>
__device__ __forceinline__ void fe_reduce4(double (&v)[4], double *red, bool act, int wl) {
  const int lane = static_cast<int>(threadIdx.x & 63);
  if constexpr (WAVE) {
    const double k = wave_sum4(v);
#pragma unroll
    for (int j = 0; j < 4; j++) v[sum4_of(j)] = readlane_f64(k, j);
  } else {
    if (act) {
      const double k = wave_sum4(v);
      if (lane < 4) red[sum4_of(lane) * kFeRedWaves + wl] = k;
    }
    __syncthreads();
    if (act) {  // lanes 8 j .. 8 j + 7 hold the wavefronts' sums of v[j]
      double r = (lane & 7) < W ? red[((lane >> 3) & 3) * kFeRedWaves + (lane & 7)] : 0.0;
      r += dpp_f64<0xb1>(r);
      r += dpp_f64<0x4e>(r);
      if constexpr (W > 4) r += dpp_f64<0x141>(r);  // row_half_mirror
#pragma unroll
      for (int j = 0; j < 4; j++) v[j] = readlane_f64(r, 8 * j);
    }
  }
}

// sum over the nine slots of the color-C row: own values from registers, the others from the planes at `pl` (the
// super-cell's place less one row and one column). PRE: in a sweep from zero, the slots of colors not relaxed yet
// (and the row itself) hold zero and are left out.
template <class T, int K, int C, bool PRE>
__device__ __forceinline__ T fe_row(const T (&a)[9], const T (&own)[4], const T *pl) {
  using G = FeGeo<K>;
  T acc = 0;
  for_slots([&](auto ss) {
    constexpr int s = decltype(ss)::value;
    using Nb = FeNbr<C, s>;
    if constexpr (!PRE || Nb::color < C) {
      T x;
      if constexpr (Nb::ox == 0 && Nb::oy == 0) x = own[Nb::color];
      else x = pl[Nb::color * G::PP + (Nb::oy + 1) * G::P + Nb::ox + 1];
      acc += a[s] * x;
    }
  });
  return acc;
}

// B~ of Algorithm 2.1 (n = 2) on level k = K, its B^ (Algorithm 2.2, one sweep) around the next level's child(). R.f
// holds the right-hand side; out(t, c, e) takes the result's entry of color c of the thread's super-cell t. A, B, E:
// the level's pre- and post-smoothing planes and the correction's plane at the thread's place (less one row and one
// column); a thread's second super-cell lies 16 rows on. `act`: the thread belongs to the level (all threads call,
// or, for a level of one wavefront, its threads). TOP: the reciprocals of the diagonals are formed on the way, each
// when its rows are first needed. DIV: divisions in place of reciprocals. put(t, g) hands the restricted residual to the
// next level, child(half) runs that.
template <class T, int K, int TR, int W, bool WAVE, bool TOP, bool DIV, class Put, class Child, class Out>
__device__ __forceinline__ void fe_btilde(FeRows<T, TR> &R, T *A, T *B, const T *E, bool act, int wl, double *red,
                                          Put put, Child child, Out out) {
  using G = FeGeo<K>;
  constexpr int own = G::P + 1, second = 16 * G::P;
  double d0 = 0.0, rd0 = 0.0;
  T a0 = 0;
  auto quot = [](T n, T d, T rd) -> T {
    if constexpr (DIV) return n / d;
    else return quotient(n, d, rd);
  };
  auto relax = [&](auto cc, auto pre, T *pl, int half) {  // x += (f - A x) / diag on the color's rows
    constexpr int c = decltype(cc)::value;
    constexpr bool p = decltype(pre)::value != 0;
    if (act)
#pragma unroll
      for (int t = 0; t < TR; t++) {
        if constexpr (TOP && p)
          if (half == 0) R.rd[t][c] = T(1) / R.a[t][c][0];
        const T acc = fe_row<T, K, c, p>(R.a[t][c], R.u[t], pl + t * second);
        const T dl = quot(R.f[t][c] - acc, R.a[t][c][0], R.rd[t][c]);
        if constexpr (p) R.u[t][c] = dl;
        else R.u[t][c] += dl;
        pl[t * second + c * G::PP + own] = R.u[t][c];
      }
    fe_sync<WAVE>();
  };
#pragma unroll 1
  for (int half = 0; half < 2; half++) {
    if (act)
#pragma unroll
      for (int t = 0; t < TR; t++) {
        if constexpr (TOP)
          if (half == 0) R.rd[t][0] = T(1) / R.a[t][0][0];
        R.u[t][0] = quot(R.f[t][0], R.a[t][0][0], R.rd[t][0]);
        A[t * second + own] = R.u[t][0];
      }
    fe_sync<WAVE>();
    relax(IC<1>{}, IC<1>{}, A, half);
    relax(IC<2>{}, IC<1>{}, A, half);
    relax(IC<3>{}, IC<1>{}, A, half);
    if (act)
#pragma unroll
      for (int t = 0; t < TR; t++) {  // residual, summed over the children in the order 0, 1, 3, 2 (Section 4.3)
        const T *pl = A + t * second;
        const T r0 = R.f[t][0] - fe_row<T, K, 0, false>(R.a[t][0], R.u[t], pl);
        const T r1 = R.f[t][1] - fe_row<T, K, 1, false>(R.a[t][1], R.u[t], pl);
        const T r3 = R.f[t][3] - fe_row<T, K, 3, false>(R.a[t][3], R.u[t], pl);
        const T r2 = R.f[t][2] - fe_row<T, K, 2, false>(R.a[t][2], R.u[t], pl);
        T acc = 0;
        acc += r0;
        acc += r1;
        acc += r3;
        acc += r2;
        put(t, acc);
      }
    fe_sync<WAVE>();
    child(half);
    if (act)
#pragma unroll
      for (int t = 0; t < TR; t++) {  // u += P e_c, and color 3 relaxed against its neighbours' u + P e_c
        const T *pl = A + t * second, *el = E + t * second;
        const T em = el[own];
        for_colors([&](auto cc) { R.u[t][decltype(cc)::value] += em; });
        T acc = 0;
        for_slots([&](auto ss) {
          constexpr int s = decltype(ss)::value;
          using Nb = FeNbr<3, s>;
          T x;
          if constexpr (Nb::ox == 0 && Nb::oy == 0) {
            x = R.u[t][Nb::color];
          } else {
            constexpr int o = (Nb::oy + 1) * G::P + Nb::ox + 1;
            x = pl[Nb::color * G::PP + o] + el[o];
          }
          acc += R.a[t][3][s] * x;
        });
        R.u[t][3] += quot(R.f[t][3] - acc, R.a[t][3][0], R.rd[t][3]);
        T *ql = B + t * second + own;
        for_colors([&](auto cc) {
          constexpr int c = decltype(cc)::value;
          ql[c * G::PP] = R.u[t][c];
        });
      }
    fe_sync<WAVE>();
    relax(IC<2>{}, IC<0>{}, B, half);
    relax(IC<1>{}, IC<0>{}, B, half);
    relax(IC<0>{}, IC<0>{}, B, half);
    double v[4] = {0.0, 0.0, 0.0, 0.0};
    if (act)
#pragma unroll
      for (int t = 0; t < TR; t++) {  // A u with (u, A u), (f, u) and, in the second step, (u, q0), (f, p0)
        if (t > 0) __builtin_amdgcn_sched_barrier(0);  // one super-cell at a time (register pressure)
        T y[4];
        const T *pl = B + t * second;
        for_colors([&](auto cc) {
          constexpr int c = decltype(cc)::value;
          y[c] = fe_row<T, K, c, false>(R.a[t][c], R.u[t], pl);
        });
        for_colors([&](auto cc) {
          constexpr int c = decltype(cc)::value;
          const double ud = static_cast<double>(R.u[t][c]), fd = static_cast<double>(R.f[t][c]);
          v[0] += ud * static_cast<double>(y[c]);
          v[1] += fd * ud;
          if (half) {
            v[2] += ud * static_cast<double>(R.q0[t][c]);
            v[3] += fd * static_cast<double>(R.p0[t][c]);
          }
        });
        if (!half)
          for_colors([&](auto cc) {
            constexpr int c = decltype(cc)::value;
            R.q0[t][c] = y[c];
            R.p0[t][c] = R.u[t][c];
          });
      }
    fe_reduce4<W, WAVE>(v, red, act, wl);
    if (act) {
      const bool first = half == 0;
      if (first) {  // alpha0, r = g - alpha0 q0
        d0 = v[0];
        a0 = static_cast<T>(readlane_f64((d0 > 0.0) ? v[1] / d0 : 0.0, 0));  // uniform: kept in scalar registers
        rd0 = readlane_f64(1.0 / d0, 0);  // ready before the second step's beta waits for it
#pragma unroll
        for (int t = 0; t < TR; t++)
          for_colors([&](auto cc) {
            constexpr int c = decltype(cc)::value;
            R.f[t][c] = R.f[t][c] - a0 * R.q0[t][c];
          });
      } else {  // direction d = p1 + beta p0: (d, A d) and (r, d) from the inner products at hand
        const bool stop = !(d0 > 0.0);
        double bd = -v[2] * rd0;
        if (d0 < 1e-290) bd = -v[2] / d0;  // 1 / d0 may overflow
        const T bt = static_cast<T>(stop ? 0.0 : bd);
        const double b = static_cast<double>(bt);
        const double d1 = v[0] + b * (2.0 * v[2] + b * d0);
        const T a1 = static_cast<T>((stop || !(d1 > 0.0)) ? 0.0 : (v[1] + b * v[3]) / d1);
#pragma unroll
        for (int t = 0; t < TR; t++)
          for_colors([&](auto cc) {
            constexpr int c = decltype(cc)::value;
            T e = a0 * R.p0[t][c];
            e += a1 * (R.u[t][c] + bt * R.p0[t][c]);
            out(t, cc, e);
          });
      }
    }
  }
}

// operator rows of the level's super-cells j, j + step, ... into registers, in the order the presmoothing sweep and the
// residual need them: color 0's diagonal, the rows of colors 1 to 3, the rest of color 0
template <class T, int K, int TR>
__device__ __forceinline__ void fe_load_rows(FeRows<T, TR> &R, const T *__restrict__ ax, int j, int step) {
  using G = FeGeo<K>;
  auto load = [&](auto cc, auto ss) {
    constexpr int c = decltype(cc)::value, s = decltype(ss)::value;
#pragma unroll
    for (int t = 0; t < TR; t++) R.a[t][c][s] = ax[s * G::N + c * G::N4 + j + t * step];
  };
  load(IC<0>{}, IC<0>{});
  for_slots([&](auto ss) { load(IC<1>{}, ss); });
  for_slots([&](auto ss) { load(IC<2>{}, ss); });
  for_slots([&](auto ss) { load(IC<3>{}, ss); });
  for_slots([&](auto ss) {
    if constexpr (decltype(ss)::value > 0) load(IC<0>{}, ss);
  });
}
template <class T, int TR>
__device__ __forceinline__ void fe_recip(FeRows<T, TR> &R) {
#pragma unroll
  for (int t = 0; t < TR; t++)
    for_colors([&](auto cc) {
      constexpr int c = decltype(cc)::value;
      R.rd[t][c] = T(1) / R.a[t][c][0];
    });
}

template <class T, int KT, bool DIV = false>
__device__ __forceinline__ void k_engine_fast_body(FeArgs<T> A) {
  using Lay = FeLayout<KT>;
  constexpr int NT = Lay::threads, TR = Lay::TR;
  // wavefronts of the levels: the top level from wavefront 0; k = 5 below it from 4; k = 4 below those in one; the
  // coarsest solve in that one and three others from wh on
  constexpr int w5 = KT == 6 ? 4 : 0, w4 = KT == 5 ? 4 : 0, wh = KT == 5 ? 0 : 1;
  extern __shared__ __align__(16) unsigned char smem[];
  double *D = reinterpret_cast<double *>(smem);
  T *S = reinterpret_cast<T *>(smem + sizeof(double) * Lay::kDoubles);
  const int tid = static_cast<int>(threadIdx.x), lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // R: the top level's rows. X: those of the levels below it (k = 5 and k = 4 belong to different wavefronts; below a
  // top level k = 5, which leaves wavefront 4 free, X is R).
  FeRows<T, TR> R;
  FeRows<T, 1> below;
  auto &X = [&]() -> FeRows<T, 1> & {
    if constexpr (KT == 5) return R;
    else return below;
  }();
  const bool act_top = KT == 5 ? wave < 4 : (KT == 4 ? wave == 0 : true);
  const bool act5 = KT == 6 && wave >= w5, act4 = KT > 4 && wave == w4;
  const int part = (wave >= wh && wave < wh + 3) ? wave - wh + 1 : 0;  // helper of the coarsest solve (1 to 3) or 0
  const int jt = tid, j5 = tid - 64 * w5, j4 = lane;
  constexpr int step = KT == 6 ? 512 : 0;
  // a helper's 16 entries of its lane's row of the coarsest inverse; k = 6: in the registers of X, which its
  // wavefronts do not use otherwise
  double hrow[KT == 6 ? 1 : 16];
  static_assert(KT != 6 || sizeof(T) == 4, "two registers of X to a double");
  auto hset = [&](auto ii, double v) {
    constexpr int i = decltype(ii)::value;
    if constexpr (KT == 6) {
      const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
      X.a[0][i / 9][i % 9] = __builtin_bit_cast(float, static_cast<unsigned>(u));
      X.a[0][2 + i / 9][i % 9] = __builtin_bit_cast(float, static_cast<unsigned>(u >> 32));
    } else {
      hrow[i] = v;
    }
  };
  auto hget = [&](auto ii) -> double {
    constexpr int i = decltype(ii)::value;
    if constexpr (KT == 6) {
      const unsigned lo = __builtin_bit_cast(unsigned, static_cast<float>(X.a[0][i / 9][i % 9]));
      const unsigned hi = __builtin_bit_cast(unsigned, static_cast<float>(X.a[0][2 + i / 9][i % 9]));
      return __builtin_bit_cast(double, (static_cast<unsigned long long>(hi) << 32) | lo);
    } else {
      return hrow[i];
    }
  };
  const int q3 = static_cast<int>(q_of_m(static_cast<uint32_t>(lane), 3));  // lane's cell of the coarsest level
  // Loads in the order of their first use; each is waited for only there. The entries of the coarsest inverse for LDS
  // come first, as they pass through registers.
  double a16[16];
  if (wave == w4)
#pragma unroll
    for (int i = 0; i < 16; i++) a16[i] = A.ainv[i * kFeCoarse + q3];
  if (act_top) {
#pragma unroll
    for (int t = 0; t < TR; t++)
      for_colors([&](auto cc) {
        constexpr int c = decltype(cc)::value;
        R.f[t][c] = A.g[c * FeGeo<KT>::N4 + jt + t * step];
      });
    fe_load_rows<T, KT, TR>(R, A.ax[0], jt, step);
  }
  if constexpr (KT == 6) {
    if (act5) fe_load_rows<T, 5, 1>(X, A.ax[1], j5, 0);
  }
  if constexpr (KT > 4) {
    if (act4) fe_load_rows<T, 4, 1>(X, A.ax[KT - 4], j4, 0);
  }
  if (part)  // row q3 of the symmetric inverse read as a column
    for_16([&](auto ii) { hset(ii, A.ainv[(16 * part + decltype(ii)::value) * kFeCoarse + q3]); });
  {
    constexpr int nz = Lay::t_units * static_cast<int>(sizeof(T)) / 16;
    static_assert(Lay::t_units * sizeof(T) % 16 == 0, "whole 16-byte stores");
    float4 *Z = reinterpret_cast<float4 *>(S);  // the planes' rings are read and never written
    for (int i = tid; i < nz; i += NT) Z[i] = make_float4(0.f, 0.f, 0.f, 0.f);
  }
  if (wave == w4)
#pragma unroll
    for (int p = 0; p < 8; p++)
      reinterpret_cast<double2 *>(D + Lay::kAinv)[p * 64 + lane] = make_double2(a16[2 * p], a16[2 * p + 1]);
  __syncthreads();

  // the thread's place in the planes of level k, for its super-cell of Morton index j
  auto place = [](int j, int p) {
    return static_cast<int>(compact_bits(static_cast<uint32_t>(j) >> 1)) * p +
           static_cast<int>(compact_bits(static_cast<uint32_t>(j)));
  };
  // where a cell (2 X + cx, 2 Y + cy) of level k lies in the parent's correction plane: the place of (X, Y)'s first
  // cell, then cy rows and cx columns on
  auto parent_place = [](int j, int p) {
    return (2 * static_cast<int>(compact_bits(static_cast<uint32_t>(j) >> 1)) + 1) * p +
           2 * static_cast<int>(compact_bits(static_cast<uint32_t>(j))) + 1;
  };

  // the 256-cell level in one wavefront (act), e to the caller's out. Its coarsest solve e3 = A_3^{-1} g3 in FP64
  // takes a quarter of the columns in each of four wavefronts: one FMA chain per i mod 4, added pairwise, then the
  // four wavefronts' sums.
  auto level4 = [&](FeRows<T, 1> &Y, bool act, auto top, auto out) {
    using G = FeGeo<4>;
    T *S4 = S + Lay::planes(4);
    const int lane = fe_tid() & 63, q3 = static_cast<int>(q_of_m(static_cast<uint32_t>(lane), 3));
    const int pl = place(lane, G::P);
    double *g3 = D + Lay::kG3, *ps = D + Lay::kPart;
    if (act) {
      fe_btilde<T, 4, 1, 1, true, decltype(top)::value != 0, DIV>(
          Y, S4 + pl, S4 + 4 * G::PP + pl, S4 + 8 * G::PP + pl, true, 0, nullptr,
          [&](int, T acc) { g3[q3] = static_cast<double>(acc); },
          [&](int) {
            __syncthreads();
            const double2 *Ai = reinterpret_cast<const double2 *>(D + Lay::kAinv) + lane;
            const double gr = g3[lane & 15];
            double acc[4] = {0.0, 0.0, 0.0, 0.0};
            for_16([&](auto nn) {
              constexpr int n = decltype(nn)::value;
              if constexpr (n % 2 == 0) {
                const double2 x = Ai[(n / 2) * 64];
                acc[n % 4] += x.x * bcast_of<n, 16>(gr);
                acc[n % 4 + 1] += x.y * bcast_of<n + 1, 16>(gr);
              }
            });
            const double mine = (acc[0] + acc[1]) + (acc[2] + acc[3]);
            __syncthreads();
            S4[8 * G::PP + pl + G::P + 1] =
                static_cast<T>((mine + ps[64 + lane]) + (ps[128 + lane] + ps[192 + lane]));
            fe_wsync();
          },
          out);
    } else {
#pragma unroll 1
      for (int half = 0; half < 2; half++) {
        __syncthreads();
        if (part) {
          const double gr = g3[16 * part + (lane & 15)];
          double acc[4] = {0.0, 0.0, 0.0, 0.0};
          for_16([&](auto nn) {
            constexpr int n = decltype(nn)::value;
            acc[n % 4] += hget(nn) * bcast_of<n, 16>(gr);
          });
          ps[64 * part + lane] = (acc[0] + acc[1]) + (acc[2] + acc[3]);
        }
        __syncthreads();
      }
    }
  };
  // result entries of the top level to global memory
  auto to_global = [&](int t, auto cc, T e) {
    A.e[decltype(cc)::value * FeGeo<KT>::N4 + jt + t * step] = e;
  };

  if constexpr (KT == 4) {
    level4(R, act_top, IC<1>{}, to_global);
  } else {
    // the right-hand side handed to the next level lies behind this level's planes (color-major)
    auto level5 = [&](auto &Y, bool act, auto top, auto out) {
      using G = FeGeo<5>;
      const int t5 = fe_tid(), j = t5 - 64 * w5, j4 = t5 & 63;
      T *S5 = S + Lay::planes(5);
      T *g4 = S5 + 9 * G::PP;
      const int pl = place(j & (G::N4 - 1), G::P), e4 = parent_place(j4, G::P);
      fe_btilde<T, 5, 1, 4, false, decltype(top)::value != 0, DIV>(
          Y, S5 + pl, S5 + 4 * G::PP + pl, S5 + 8 * G::PP + pl, act, wave - w5, D + Lay::kRed,
          [&](int, T acc) { g4[(j & 3) * FeGeo<4>::N4 + (j >> 2)] = acc; },
          [&](int half) {
            if constexpr (decltype(top)::value != 0)
              if (act4 && half == 0) fe_recip(X);
            if (act4)
              for_colors([&](auto cc) {
                constexpr int c = decltype(cc)::value;
                X.f[0][c] = g4[c * FeGeo<4>::N4 + j4];
              });
            level4(X, act4, IC<0>{}, [&](int, auto cc, T e) {
              constexpr int c = decltype(cc)::value;
              S5[8 * G::PP + e4 + (c >> 1) * G::P + (c & 1)] = e;
            });
            __syncthreads();
          },
          out);
    };
    if constexpr (KT == 5) {
      level5(R, act_top, IC<1>{}, to_global);
    } else {
      using G = FeGeo<6>;
      T *S6 = S + Lay::planes(6);
      T *g5 = S6 + 9 * G::PP;
      const int pl = place(jt, G::P);
      fe_btilde<T, 6, 2, 8, false, true, DIV>(
          R, S6 + pl, S6 + 4 * G::PP + pl, S6 + 8 * G::PP + pl, true, wave, D + Lay::kRed + 4 * kFeRedWaves,
          [&](int t, T acc) { g5[(jt & 3) * FeGeo<5>::N4 + (jt >> 2) + t * (step / 4)] = acc; },
          [&](int half) {
            if (half == 0 && (act5 || act4)) fe_recip(X);
            const int j5 = (fe_tid() - 64 * w5) & (FeGeo<5>::N4 - 1), e5 = parent_place(j5, G::P);
            if (act5)
              for_colors([&](auto cc) {
                constexpr int c = decltype(cc)::value;
                X.f[0][c] = g5[c * FeGeo<5>::N4 + j5];
              });
            level5(X, act5, IC<0>{}, [&, e5](int, auto cc, T e) {
              constexpr int c = decltype(cc)::value;
              S6[8 * G::PP + e5 + (c >> 1) * G::P + (c & 1)] = e;
            });
            __syncthreads();
          },
          to_global);
    }
  }
}
template <class T, int KT>
__global__ void __launch_bounds__(FeLayout<KT>::threads) k_engine_fast(FeArgs<T> A) {
  k_engine_fast_body<T, KT>(A);
}
template <class T, int KT>
__device__ __forceinline__ void k_engine_div_body(FeArgs<T> A) {
  k_engine_fast_body<T, KT, true>(A);
}
template <class T, int KT>
__global__ void __launch_bounds__(FeLayout<KT>::threads) k_engine_div(FeArgs<T> A) {
  k_engine_div_body<T, KT>(A);
}

// ---- host side ----

// steps of one launch (a step ends with a barrier; B~ of the 256-cell level is one): per inner step of a level four
// presmoothing phases, the restriction, the next level's steps, four post-smoothing phases and the reduction
constexpr int fe_steps(int kt) { return kt == 4 ? 1 : 2 * (10 + fe_steps(kt - 1)); }

// configuration ids: FP32 k = 6, 5, 4; FP64 k = 5, 4 (the operators of the 4,096-cell level in FP64 alone are 288 KB,
// and with its vectors exceed the registers and LDS of a CU)
struct FeCfg {
  int pi, kt;
};
constexpr FeCfg kFeCfgs[] = {{1, 6}, {1, 5}, {1, 4}, {0, 5}, {0, 4}};

size_t fe_cfg_bytes(int id) {
  switch (id) {
    case 0: return FeLayout<6>::bytes<float>();
    case 1: return FeLayout<5>::bytes<float>();
    case 2: return FeLayout<4>::bytes<float>();
    case 3: return FeLayout<5>::bytes<double>();
    default: return FeLayout<4>::bytes<double>();
  }
}

template <class T, int KT>
const void *fe_kernel_of(bool div) {
  return div ? reinterpret_cast<const void *>(k_engine_div<T, KT>)
             : reinterpret_cast<const void *>(k_engine_fast<T, KT>);
}
const void *fe_kernel(int id, bool div) {
  switch (id) {
    case 0: return fe_kernel_of<float, 6>(div);
    case 1: return fe_kernel_of<float, 5>(div);
    case 2: return fe_kernel_of<float, 4>(div);
    case 3: return fe_kernel_of<double, 5>(div);
    default: return fe_kernel_of<double, 4>(div);
  }
}

amg_status fe_lds_limits(int device, size_t lds_max) {
  static std::once_flag once[64];
  if (device < 0 || device >= 64) return AMG_ERR_DEVICE;
  amg_status st = AMG_OK;
  std::call_once(once[device], [&]() {
    for (int id = 0; id < 10; id++)
      if (hipFuncSetAttribute(fe_kernel(id % 5, id >= 5), hipFuncAttributeMaxDynamicSharedMemorySize,
                              static_cast<int>(lds_max)) != hipSuccess)
        st = AMG_ERR_DEVICE;
  });
  return st;
}

template <class T>
std::vector<LevelWork<T>> &fe_work(amg_hierarchy *h) {
  if constexpr (std::is_same<T, float>::value) return h->w32;
  else return h->w64;
}
template <class T>
const T *fe_level_ax(const QuadLevel &Q) {
  if constexpr (std::is_same<T, float>::value) return Q.ax32;
  else return Q.ax64;
}

template <class T, int KT>
void fe_launch(amg_hierarchy *h, int pi) {
  FeArgs<T> A{};
  const int top = h->engine_top[pi];
  A.ainv = h->ainv;
  for (int i = 0; i < 3; i++) A.ax[i] = top + i < h->nlev ? fe_level_ax<T>(h->lev[top + i]) : nullptr;
  const LevelWork<T> &w = fe_work<T>(h)[top];
  A.g = w.g;
  A.e = w.e;
  const size_t lds = FeLayout<KT>::template bytes<T>();
  Timing &t = h->timing;
  const int kind = pi ? KK_ENGINE32 : KK_ENGINE64;
  if (!h->recording && t.kind == kind && t.used + 2 <= t.ev.size()) {  // dispatch-stamped start / stop
    hipExtLaunchKernelGGL(h->tiny_diag[pi] ? k_engine_div<T, KT> : k_engine_fast<T, KT>, dim3(1),
                          dim3(FeLayout<KT>::threads), lds, h->stream, t.ev[t.used], t.ev[t.used + 1], 0, A);
    t.used += 2;
  } else if (h->tiny_diag[pi]) {
    QA_RUN(h, FeLayout<KT>::threads, 1, lds, k_engine_div, QA_T(T, KT), A);
  } else {
    QA_RUN(h, FeLayout<KT>::threads, 1, lds, k_engine_fast, QA_T(T, KT), A);
  }
}

}  // namespace

// The configuration a precision's small levels have the shape of, or -1: the top is the largest level the registers
// allow, k = min(L, 6) in FP32, min(L, 5) in FP64.
int engine_fast_config(const amg_hierarchy *h, int pi) {
  if (h->use_engine != 1 || h->nlev < 3 || h->L < 4 || h->lev[h->nlev - 1].k != 3 || h->nc != kFeCoarse ||
      h->opt.sweeps != 1 || h->opt.inner_iters != 2)
    return -1;
  for (int id = 0; id < 5; id++) {
    const FeCfg c = kFeCfgs[id];
    if (c.pi != pi || std::min(h->L, pi ? 6 : 5) != c.kt) continue;
    if (fe_cfg_bytes(id) > h->lds_max) return -1;
    for (int l = 1 + (h->L - c.kt); l + 1 < h->nlev; l++)
      if (h->lev[l].ovf_nnz != 0 || h->lev[l].same_color_ovf) return -1;
    return id;
  }
  return -1;
}

amg_status plan_engine_fast(amg_hierarchy *h) {
  for (int pi = 0; pi < 2; pi++) {
    const int id = h->fe_cfg[pi] = engine_fast_config(h, pi);
    if (id < 0) continue;
    const int kt = kFeCfgs[id].kt, top = 1 + (h->L - kt);  // hierarchy index of level k = kt
    h->engine_top[pi] = top;
    h->engine_lds_top[pi] = top;
    h->engine_lds[pi] = fe_cfg_bytes(id);
    h->engine_nops[pi] = fe_steps(kt);
  }
  if (h->fe_cfg[0] >= 0 || h->fe_cfg[1] >= 0) QA_TRY(fe_lds_limits(h->device, h->lds_max));
  return AMG_OK;
}

void launch_engine_fast(amg_hierarchy *h, int pi) {
  switch (h->fe_cfg[pi]) {
    case 0: fe_launch<float, 6>(h, pi); break;
    case 1: fe_launch<float, 5>(h, pi); break;
    case 2: fe_launch<float, 4>(h, pi); break;
    case 3: fe_launch<double, 5>(h, pi); break;
    case 4: fe_launch<double, 4>(h, pi); break;
    default: break;
  }
}

}  // namespace qa
