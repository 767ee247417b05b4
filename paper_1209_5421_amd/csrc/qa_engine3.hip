// Persistent engine of the small octree levels (gfx950): B~ (Algorithm 2.1 with n = 2) of the 4,096-cell level k = 4, or
// of the 512-cell level k = 3 where that is the finest tree level, and everything below it in one launch of one
// 512-thread workgroup. The coarsest level is the 64-cell level k = 2; one smoothing sweep.
//
// Like the quadtree's engine it is bound by the latency of its chain of steps on one CU; in 3D by the operator as well,
// which at 27 entries a row (432 KB on the 4,096-cell level in FP32) exceeds the registers and LDS of a CU:
//  - u lies in LDS as the plain lattice of the level's cells with a ring of zeros around it, so that every neighbour of
//    every color is the same compile-time distance away: an immediate offset of the LDS load, no index arithmetic (the
//    Morton rule for 27 neighbours is about 700 instructions a row) and no edge tests. The strides let a wavefront's
//    4 x 4 x 4 block of cells of one color touch every second bank twice;
//  - on level 4 a thread owns a super-cell (the eight cells of one parent, one per color): its f, q0 and p0 stay in
//    registers, and the rows stream from L2, each row's entries loaded one or two rows ahead of their use and across the
//    barriers (kAhead); the presmoothing sweep starts from zero, so it neither loads nor reads the slots of colors not
//    relaxed yet;
//  - on level 3 eight threads share the rows of a super-cell, each holding four of the 27 slots of all eight in registers,
//    so that the 64 rows of a color phase are spread over every wavefront;
//  - A p1 with (p1, A p1), (r, p1), (p1, q0) and (r, p0) replaces A (p1 + beta p0), as in the quadtree's engine: one
//    reduction per inner step;
//  - the FP64 coarsest solve takes eight columns per thread.
// On the top level couplings beyond one cell are allowed (OVF): rows that have some are marked once, and coupled rows of
// one color see the values from before their phase.
// One launch takes 84 us (FP32) and 139 us (FP64) on level 4, where B~ of that level took 30 launches and about 390 us.
// Of the FP32 launch the sixteen color phases of level 4 take 1.0 us each (0.5 without the operator's loads: a CU reads
// 35 to 50 bytes per clock from L2), a color phase of level 3 0.24 us (0.4 with the 64 rows in one wavefront).
// Taken alone the kernel brought an FP32-preconditioned solve of the heat step with 1,020,100 unknowns from 28.0 to
// 15.2 ms, one in FP64 with 8,820 from 6.1 to 3.5 ms.

#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <mutex>
#include <type_traits>
#include <utility>
#include <vector>

#include "qa_internal.hpp"
#include "qa_launch.hpp"
#include "qa_wave.hpp"

namespace qa {

namespace {

constexpr int kO3Threads = 512;

template <int C>
using IC = std::integral_constant<int, C>;

template <int... I, class F>
__device__ __forceinline__ void o3_each(std::integer_sequence<int, I...>, F f) {
  (f(IC<I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void o3_for(F f) {
  o3_each(std::make_integer_sequence<int, N>{}, f);
}

// offsets of slot s: the nine plane offsets of Section 4.4 (self, E, NE, N, NW, W, SW, S, SE) at dz = 0, +1, -1
constexpr int o3_dx(int s) {
  const int p = s % 9;
  return (p == 1 || p == 2 || p == 8) ? 1 : ((p == 4 || p == 5 || p == 6) ? -1 : 0);
}
constexpr int o3_dy(int s) {
  const int p = s % 9;
  return (p == 2 || p == 3 || p == 4) ? 1 : ((p == 6 || p == 7 || p == 8) ? -1 : 0);
}
constexpr int o3_dz(int s) { return s < 9 ? 0 : (s < 18 ? 1 : -1); }
// color of the slot's neighbour of a color-c cell
constexpr int o3_color(int c, int s) {
  return c ^ ((o3_dx(s) & 1) | ((o3_dy(s) & 1) << 1) | ((o3_dz(s) & 1) << 2));
}
// restriction order of the children: (0, 1, 3, 2) on either layer
constexpr int o3_child(int i) { return (i & 4) | ((i & 3) == 2 ? 3 : ((i & 3) == 3 ? 2 : (i & 3))); }

// lattice of level k: side 2^k with a ring around it
template <int K>
struct O3Geo {
  static constexpr int S = 1 << K, n = S * S * S, N8 = n / 8;
  static constexpr int SY = K == 4 ? 20 : 12, SZ = SY * (S + 2), cells = SZ * (S + 2);
  // distance of a slot's neighbour from the cell's corner place (one row, column and layer back)
  static constexpr int off(int s) { return (1 + o3_dz(s)) * SZ + (1 + o3_dy(s)) * SY + 1 + o3_dx(s); }
  static constexpr int own = SZ + SY + 1;
  static constexpr int child(int c) { return (c >> 2) * SZ + ((c >> 1) & 1) * SY + (c & 1); }
};

// LDS. In doubles: the coarsest inverse (rows 66 apart, so that eight rows read at once use different banks), its
// right-hand side, the wavefront sums of the reductions. In units of T: the two lattices and, in FP64, p0 of level 4.
struct O3Lay {
  static constexpr int kAinvRow = 66;
  static constexpr int kAinv = 0, kG2 = 64 * kAinvRow, kRed = kG2 + 64, kDoubles = kRed + 32;
  static constexpr int kLat4 = 0, kLat3 = O3Geo<4>::cells, kP0 = kLat3 + O3Geo<3>::cells;
  template <class T>
  static constexpr int units() {
    return kP0 + (sizeof(T) == 8 ? O3Geo<4>::n : 0);
  }
  template <class T>
  static constexpr size_t bytes() {
    return sizeof(double) * kDoubles + sizeof(T) * units<T>();
  }
};

template <class T>
struct O3Args {
  const double *ainv;             // coarsest inverse, 64 x 64, storage numbering (bitwise symmetric)
  const T *ax4, *ax3;             // 27 x n operators
  const T *g;                     // the top level's right-hand side and result
  T *e;
  const int32_t *optr, *ocol;     // the top level's overflow couplings (OVF)
  const T *oval;
};

// place of the cell with color-major index q on level k's lattice (its corner)
template <int K>
__device__ __forceinline__ int o3_place(uint32_t q) {
  using G = O3Geo<K>;
  const uint32_t m = m_of_q3(q, K);
  return static_cast<int>(compact3(m >> 2)) * G::SZ + static_cast<int>(compact3(m >> 1)) * G::SY +
         static_cast<int>(compact3(m));
}

// sum of a row's overflow couplings times u (added behind its 27 slots). ZERO: in the sweep from zero, entries of colors
// not relaxed yet (the row's own among them) hold zero.
template <class T, int K, bool ZERO>
__device__ __forceinline__ T o3_ovf(const O3Args<T> &A, T acc, uint32_t q, int c, const T *lat) {
  for (int32_t e = A.optr[q]; e < A.optr[q + 1]; e++) {
    const uint32_t i = static_cast<uint32_t>(A.ocol[e]);
    if (ZERO && static_cast<int>(i / O3Geo<K>::N8) >= c) continue;
    acc += A.oval[e] * lat[o3_place<K>(i) + O3Geo<K>::own];
  }
  return acc;
}

// between two rows: the finished row's sum is formed here, not later, nothing is loaded further ahead, and no lattice
// value is kept for the next row (any of it would spill)
template <class T>
__device__ __forceinline__ void o3_done(T &sum) {
  asm volatile("" : "+v"(sum) : : "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// entry `at` (compile-time part) + lane offset of an operator, by a buffer load: the slot's distance is a scalar operand.
// The lane's byte offset passes through o3_opaque for every row: the optimiser would otherwise hoist the loads out of the
// loop over the inner steps, or keep one step's entries for the next, and spill them.
__device__ __forceinline__ int o3_opaque(int x) {
  asm volatile("" : "+v"(x));
  return x;
}
template <class T>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t o3_rsrc(const T *p, int count) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<T *>(p), 0, count * static_cast<int>(sizeof(T)), 0x00027000);
}
template <class T>
__device__ __forceinline__ T o3_load(__amdgpu_buffer_rsrc_t r, int lane_bytes, int at) {
  if constexpr (sizeof(T) == 4) {
    return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, lane_bytes, at * 4, 0));
  } else {
    return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, lane_bytes, at * 8, 0));
  }
}

// a lane's value moved by a DPP lane pattern
template <int Ctrl>
__device__ __forceinline__ double o3_dpp(double x) {
  return dpp_f64<Ctrl>(x);
}
template <int Ctrl>
__device__ __forceinline__ float o3_dpp(float x) {
  return __builtin_bit_cast(
      float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), Ctrl, 0xf, 0xf, false));
}
// sum over the eight lanes 8 k .. 8 k + 7, the same in each
template <class X>
__device__ __forceinline__ X o3_sum8(X x) {
  x += o3_dpp<0xb1>(x);   // quad_perm [1, 0, 3, 2]
  x += o3_dpp<0x4e>(x);   // quad_perm [2, 3, 0, 1]
  x += o3_dpp<0x141>(x);  // row_half_mirror
  return x;
}
// eight sums over the eight lanes 8 k .. 8 k + 7, sum g in lane g: in each step a lane hands its partner the half of its
// values that the partner keeps
template <class T>
__device__ __forceinline__ T o3_sum8_own(const T (&v)[8], int g) {
  const bool b0 = g & 1, b1 = g & 2, b2 = g & 4;
  T h[4];
#pragma unroll
  for (int i = 0; i < 4; i++) h[i] = (b2 ? v[4 + i] : v[i]) + o3_dpp<0x141>(b2 ? v[i] : v[4 + i]);
  const T k0 = (b0 ? h[1] : h[0]) + o3_dpp<0xb1>(b0 ? h[0] : h[1]);
  const T k1 = (b0 ? h[3] : h[2]) + o3_dpp<0xb1>(b0 ? h[2] : h[3]);
  return (b1 ? k1 : k0) + o3_dpp<0x4e>(b1 ? k0 : k1);
}

template <class T>
struct O3Row {
  T a[27];
};

// Algorithm 2.1's scalars of one level between its two steps
template <class T>
struct O3Scal {
  double d0 = 0.0;
  T a0 = 0;
};

template <class T>
struct O3 {
  const O3Args<T> &A;
  double *D;
  T *S;
  int tid;

  // (u, A u), (f, u), (u, q0), (f, p0) over the workgroup -> alpha0 (first) or beta and alpha1, uniform
  __device__ __forceinline__ void first_scalars(double (&v)[4], O3Scal<T> &Z) const {
    block_sum4<kO3Threads>(v, reinterpret_cast<double(*)[8]>(D + O3Lay::kRed));
    Z.d0 = v[0];
    Z.a0 = static_cast<T>(readlane_f64((v[0] > 0.0) ? v[1] / v[0] : 0.0, 0));
  }
  __device__ __forceinline__ void second_scalars(double (&v)[4], const O3Scal<T> &Z, T &bt, T &a1) const {
    block_sum4<kO3Threads>(v, reinterpret_cast<double(*)[8]>(D + O3Lay::kRed));
    const bool stop = !(Z.d0 > 0.0);
    bt = static_cast<T>(stop ? 0.0 : -v[2] / Z.d0);
    const double b = static_cast<double>(bt);
    const double d1 = v[0] + b * (2.0 * v[2] + b * Z.d0);
    a1 = static_cast<T>((stop || !(d1 > 0.0)) ? 0.0 : (v[1] + b * v[3]) / d1);
  }

  // ---- level 3: eight threads to a super-cell j = tid >> 3; thread g = tid & 7 of them owns row g 64 + j and holds the
  // slots 4 g .. 4 g + 3 of all eight rows, so that a color phase is spread over every wavefront ----

  // B~ with right-hand side f of the thread's row; returns the row's result. (A thread's row is the level-4 super-cell
  // of the same Morton index: right-hand side and result pass between the levels in registers.)
  template <bool TOP, bool OVF>
  __device__ __forceinline__ T level3(T f) const {
    using G = O3Geo<3>;
    const int t = o3_opaque(tid), j = t >> 3, g = t & 7;
    const uint32_t q = static_cast<uint32_t>(g * G::N8 + j);
    const T *lat0 = S + O3Lay::kLat3;
    T *lat = S + O3Lay::kLat3 + o3_place<3>(static_cast<uint32_t>(j));  // color 0's corner
    T a[8][4];
    const T *at[4];
    {
      const __amdgpu_buffer_rsrc_t r = o3_rsrc(A.ax3, 27 * G::n);
      const int lb = (4 * g * G::n + j) * static_cast<int>(sizeof(T));  // slot 27 lies behind the operator: reads 0
#pragma unroll
      for (int c = 0; c < 8; c++)
#pragma unroll
        for (int i = 0; i < 4; i++) a[c][i] = o3_load<T>(r, lb, i * G::n + c * G::N8);
#pragma unroll
      for (int i = 0; i < 4; i++) {
        const int s = 4 * g + i, p = s % 9, z = s / 9;
        const int dx = ((0x106 >> p) & 1) - ((0x70 >> p) & 1), dy = ((0x1c >> p) & 1) - ((0x1c0 >> p) & 1);
        const int dz = z == 1 ? 1 : (z == 2 ? -1 : 0);
        at[i] = lat + (s < 27 ? (1 + dz) * G::SZ + (1 + dy) * G::SY + 1 + dx : static_cast<int>(G::own));
      }
    }
    T *own = lat + ((g >> 2) * G::SZ + ((g >> 1) & 1) * G::SY + (g & 1)) + G::own;
    const T dg = A.ax3[q];
    bool far = false;
    if constexpr (TOP && OVF) far = A.optr[q + 1] > A.optr[q];
    double *g2 = D + O3Lay::kG2;
    const int q2 = static_cast<int>(q_of_m3(static_cast<uint32_t>(j), 2));
    auto part = [&](auto cc) -> T {  // this thread's four products of color c's row
      constexpr int c = decltype(cc)::value;
      T acc = a[c][0] * at[0][G::child(c)];
#pragma unroll
      for (int i = 1; i < 4; i++) acc += a[c][i] * at[i][G::child(c)];
      return acc;
    };
    auto row = [&]() -> T {  // (A u) of the own row
      T v[8];
      o3_for<8>([&](auto cc) { v[decltype(cc)::value] = part(cc); });
      T acc = o3_sum8_own(v, g);
      if constexpr (TOP && OVF)
        if (far) acc = o3_ovf<T, 3, false>(A, acc, q, 0, lat0);
      return acc;
    };
    auto phase = [&](auto cc, T &u) {  // x += (f - A x) / diag on color c's rows
      constexpr int c = decltype(cc)::value;
      T acc = o3_sum8(part(cc));
      if (g == c) {
        if constexpr (TOP && OVF)
          if (far) acc = o3_ovf<T, 3, false>(A, acc, q, 0, lat0);
        u += (f - acc) / dg;
      }
      if constexpr (TOP && OVF) __syncthreads();
      if (g == c) *own = u;
      __syncthreads();
    };
    O3Scal<T> Z;
    T q0 = 0, p0 = 0, e = 0;
#pragma unroll 1
    for (int half = 0; half < 2; half++) {
      T u = 0;
      *own = T(0);  // colors not relaxed yet (and coupled rows of the phase's color) hold zero
      __syncthreads();
      o3_for<8>([&](auto cc) { phase(cc, u); });
      const T r = o3_sum8(f - row());  // residual, summed over the children
      if (g == 0) g2[q2] = static_cast<double>(r);
      __syncthreads();
      {  // e2 = A_2^{-1} g2: thread g takes the columns 8 g .. 8 g + 7 of the super-cell's row
        const double2 *Ai = reinterpret_cast<const double2 *>(D + O3Lay::kAinv + q2 * O3Lay::kAinvRow + 8 * g);
        const double2 *gv = reinterpret_cast<const double2 *>(g2 + 8 * g);
        double acc[2] = {0.0, 0.0};
#pragma unroll
        for (int i = 0; i < 4; i++) {
          const double2 x = Ai[i], y = gv[i];
          acc[0] += x.x * y.x;
          acc[1] += x.y * y.y;
        }
        u += static_cast<T>(o3_sum8(acc[0] + acc[1]));
        *own = u;
      }
      __syncthreads();
      o3_for<8>([&](auto cc) { phase(IC<7 - decltype(cc)::value>{}, u); });
      const T y = row();
      const double ud = static_cast<double>(u), fd = static_cast<double>(f);
      double v[4] = {ud * static_cast<double>(y), fd * ud, 0.0, 0.0};
      if (half == 0) {
        first_scalars(v, Z);
        q0 = y, p0 = u;
        f = f - Z.a0 * q0;
      } else {
        v[2] = ud * static_cast<double>(q0);
        v[3] = fd * static_cast<double>(p0);
        T bt, a1;
        second_scalars(v, Z, bt, a1);
        e = Z.a0 * p0;
        e += a1 * (u + bt * p0);
      }
    }
    return e;
  }

  // ---- level 4: thread = super-cell j, rows c 512 + j ----

  // jobs of the two stages between which the next level runs. Stage 0: the presmoothing phases of colors 0 .. 7, then
  // the residuals of the children in restriction order; stage 1: the post-smoothing phases of colors 7 .. 0, then A u.
  static constexpr int job_color(int stage, int i) {
    return stage == 0 ? (i < 8 ? i : o3_child(i - 8)) : (i < 8 ? 7 - i : i - 8);
  }
  // entries of the job's row: in the sweep from zero the diagonal and the slots of colors relaxed already
  template <int STAGE, int I>
  __device__ __forceinline__ void job_load(O3Row<T> &b) const {
    constexpr int c = job_color(STAGE, I);
    constexpr bool pre = STAGE == 0 && I < 8;
    const __amdgpu_buffer_rsrc_t r = o3_rsrc(A.ax4, 27 * O3Geo<4>::n);
    const int lb = o3_opaque(tid * static_cast<int>(sizeof(T)));
    o3_for<27>([&](auto ss) {
      constexpr int s = decltype(ss)::value;
      if constexpr (!pre || s == 0 || o3_color(c, s) < c)
        b.a[s] = o3_load<T>(r, lb, s * O3Geo<4>::n + c * O3Geo<4>::N8);
    });
  }
  template <int STAGE, int I, bool OVF>
  __device__ __forceinline__ T job_sum(const O3Row<T> &b, const T *lat, const T *lat0, unsigned far) const {
    using G = O3Geo<4>;
    constexpr int c = job_color(STAGE, I);
    constexpr bool pre = STAGE == 0 && I < 8;
    T acc = 0;
    o3_for<27>([&](auto ss) {
      constexpr int s = decltype(ss)::value;
      if constexpr (!pre || o3_color(c, s) < c) acc += b.a[s] * lat[G::child(c) + G::off(s)];
    });
    if constexpr (OVF)
      if ((far >> c) & 1u) acc = o3_ovf<T, 4, pre>(A, acc, static_cast<uint32_t>(c * G::N8 + tid), c, lat0);
    // the next rows' loads between this row's products: issued in one run, they hold a wavefront up for as long as the
    // products take
    o3_for<27>([&](auto) {
      __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);  // a load
      __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);  // two VALU instructions
    });
    o3_done(acc);
    return acc;
  }

  template <bool OVF>
  __device__ __forceinline__ void level4() const {
    using G = O3Geo<4>;
    constexpr int kAhead = sizeof(T) == 4 ? 2 : 1;  // rows loaded ahead (FP64: two would exceed the registers)
    constexpr int NB = kAhead + 1;
    const int corner = o3_place<4>(static_cast<uint32_t>(tid));  // color 0's
    T *lat0 = S + O3Lay::kLat4, *lat = lat0 + corner;
    T f[8], q0[8], p0r[sizeof(T) == 4 ? 8 : 1];
    auto p0 = [&](int c) -> T & {  // FP64: in LDS, to save registers
      if constexpr (sizeof(T) == 4) return p0r[c];
      else return S[O3Lay::kP0 + c * G::N8 + tid];
    };
    unsigned far = 0;
    o3_for<8>([&](auto cc) {
      constexpr int c = decltype(cc)::value;
      f[c] = A.g[c * G::N8 + tid];
      q0[c] = p0(c) = T(0);
      if constexpr (OVF)
        if (A.optr[c * G::N8 + tid + 1] > A.optr[c * G::N8 + tid]) far |= 1u << c;
    });
    O3Scal<T> Z;
#pragma unroll 1
    for (int half = 0; half < 2; half++) {
      O3Row<T> b[NB];
      o3_for<kAhead>([&](auto ii) { job_load<0, decltype(ii)::value>(b[decltype(ii)::value]); });
      T gsum = 0;
      o3_for<16>([&](auto ii) {
        constexpr int i = decltype(ii)::value, c = job_color(0, i);
        if constexpr (i + kAhead < 16) job_load<0, i + kAhead>(b[(i + kAhead) % NB]);
        const O3Row<T> &r = b[i % NB];
        const T d = f[c] - job_sum<0, i, OVF>(r, lat, lat0, far);
        if constexpr (i < 8) {
          lat[G::child(c) + G::own] = T(0) + d / r.a[0];
          __syncthreads();
        } else {
          gsum += d;
        }
      });
      const T em = level3<false, false>(gsum);
      o3_for<kAhead>([&](auto ii) { job_load<1, decltype(ii)::value>(b[decltype(ii)::value]); });
      o3_for<8>([&](auto cc) { lat[G::child(decltype(cc)::value) + G::own] += em; });
      __syncthreads();
      double v[4] = {0.0, 0.0, 0.0, 0.0};
      o3_for<16>([&](auto ii) {
        constexpr int i = decltype(ii)::value, c = job_color(1, i);
        if constexpr (i + kAhead < 16) job_load<1, i + kAhead>(b[(i + kAhead) % NB]);
        const O3Row<T> &r = b[i % NB];
        const T s = job_sum<1, i, OVF>(r, lat, lat0, far);
        T *own = lat + G::child(c) + G::own;
        if constexpr (i < 8) {
          const T u = *own + (f[c] - s) / r.a[0];
          if constexpr (OVF) __syncthreads();
          *own = u;
          __syncthreads();
        } else {
          const double ud = static_cast<double>(*own), fd = static_cast<double>(f[c]);
          v[0] += ud * static_cast<double>(s);
          v[1] += fd * ud;
          v[2] += ud * static_cast<double>(q0[c]);  // zero in the first step
          v[3] += fd * static_cast<double>(p0(c));
          q0[c] = half ? q0[c] : s;
          p0(c) = half ? p0(c) : *own;
        }
      });
      if (half == 0) {
        first_scalars(v, Z);
        o3_for<8>([&](auto cc) {
          constexpr int c = decltype(cc)::value;
          f[c] = f[c] - Z.a0 * q0[c];
        });
      } else {
        T bt, a1;
        second_scalars(v, Z, bt, a1);
        o3_for<8>([&](auto cc) {
          constexpr int c = decltype(cc)::value;
          T e = Z.a0 * p0(c);
          e += a1 * (lat[G::child(c) + G::own] + bt * p0(c));
          A.e[c * G::N8 + tid] = e;
        });
      }
    }
  }
};

template <class T, int KT, bool OVF>
__global__ void __launch_bounds__(kO3Threads) k_engine_oct(O3Args<T> A) {
  extern __shared__ __align__(16) unsigned char smem[];
  double *D = reinterpret_cast<double *>(smem);
  T *S = reinterpret_cast<T *>(smem + sizeof(double) * O3Lay::kDoubles);
  const int tid = static_cast<int>(threadIdx.x);
  double ai[8];
#pragma unroll
  for (int k = 0; k < 8; k++) ai[k] = A.ainv[tid + k * kO3Threads];
  for (int i = tid; i < O3Lay::units<T>(); i += kO3Threads) S[i] = T(0);  // the lattices' rings are read, never written
#pragma unroll
  for (int k = 0; k < 8; k++) {
    const int i = tid + k * kO3Threads;
    D[O3Lay::kAinv + (i >> 6) * O3Lay::kAinvRow + (i & 63)] = ai[k];
  }
  __syncthreads();
  const O3<T> E{A, D, S, tid};
  if constexpr (KT == 4) {
    E.template level4<OVF>();
  } else {
    const int q = (tid & 7) * O3Geo<3>::N8 + (tid >> 3);
    A.e[q] = E.template level3<true, OVF>(A.g[q]);
  }
}

template <class T>
const void *o3_kernel(int kt, bool ovf) {
  if (kt == 4)
    return ovf ? reinterpret_cast<const void *>(k_engine_oct<T, 4, true>)
               : reinterpret_cast<const void *>(k_engine_oct<T, 4, false>);
  return ovf ? reinterpret_cast<const void *>(k_engine_oct<T, 3, true>)
             : reinterpret_cast<const void *>(k_engine_oct<T, 3, false>);
}

amg_status o3_lds_limits(int device) {
  static std::once_flag once[64];
  if (device < 0 || device >= 64) return AMG_ERR_DEVICE;
  amg_status st = AMG_OK;
  std::call_once(once[device], [&]() {
    for (int kt : {3, 4})
      for (bool ovf : {false, true})
        for (bool dbl : {false, true}) {
          const void *k = dbl ? o3_kernel<double>(kt, ovf) : o3_kernel<float>(kt, ovf);
          const int b = static_cast<int>(dbl ? O3Lay::bytes<double>() : O3Lay::bytes<float>());
          if (hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, b) != hipSuccess) st = AMG_ERR_DEVICE;
        }
  });
  return st;
}

template <class T>
void o3_launch(amg_hierarchy *h, const LevelWork<T> &w, const T *ax4, const T *ax3, const T *oval) {
  const QuadLevel &Q = h->lev[h->oct_top];
  const O3Args<T> A{h->ainv, ax4, ax3, w.g, w.e, Q.optr, Q.ocol, oval};
  const size_t lds = O3Lay::bytes<T>();
  const bool ovf = Q.ovf_nnz != 0;
  const auto kernel = Q.k == 4 ? (ovf ? k_engine_oct<T, 4, true> : k_engine_oct<T, 4, false>)
                               : (ovf ? k_engine_oct<T, 3, true> : k_engine_oct<T, 3, false>);
  if (refuse_recording(h)) return;
  Timing &t = h->timing;
  if (t.kind == (sizeof(T) == 4 ? KK_ENGINE32 : KK_ENGINE64) && t.used + 2 <= t.ev.size()) {
    hipExtLaunchKernelGGL(kernel, dim3(1), dim3(kO3Threads), lds, h->stream, t.ev[t.used], t.ev[t.used + 1], 0, A);
    t.used += 2;
  } else {
    kernel<<<1, kO3Threads, lds, h->stream>>>(A);
  }
}

// steps of one launch (a step ends with a barrier): per inner step of a level eight presmoothing phases, the restriction,
// the next level's steps (one for the coarsest solve), eight post-smoothing phases and the reduction
constexpr int o3_steps(int kt) { return 2 * (18 + (kt == 3 ? 1 : o3_steps(kt - 1))); }

// algorithmic floating-point operations of one launch: each add, multiply or divide counts one (a fused multiply-add
// two), once per value; a row of 27 slots is 54
double o3_flops(int kt) {
  const double n = static_cast<double>(1 << (3 * kt)), n8 = n / 8;
  const double child = kt == 3 ? 2.0 * 64 * 64 : o3_flops(kt - 1);
  // color 0 from zero, seven phases, residuals and their sums, prolongation, eight phases, A u and two inner products
  const double step = n8 + 7 * n8 * 57 + n * 56 + child + n + 8 * n8 * 57 + n * 58;
  return 2 * step + 3 * n + 2 * n + 2 * n + 4 * n;  // first update, beta, direction, last update
}

}  // namespace

// Selects the octree engine's top level: k = min(L, 4), where the coarsest level is k = 2 with 64 cells, the cycle has
// one sweep and two inner steps, and the level below the top holds no couplings beyond one cell.
amg_status plan_engine_oct(amg_hierarchy *h) {
  h->oct_top = -1;
  if (h->dim != 3 || h->opt.engine == 0 || h->nlev < 3 || h->L < 3 || h->lev[h->nlev - 1].k != 2 || h->nc != 64 ||
      h->opt.sweeps != 1 || h->opt.inner_iters != 2)
    return AMG_OK;
  const int kt = h->L < 4 ? h->L : 4, top = 1 + (h->L - kt);
  for (int l = top + 1; l + 1 < h->nlev; l++)
    if (h->lev[l].ovf_nnz != 0 || h->lev[l].same_color_ovf) return AMG_OK;
  int lds = 0;
  QA_HIP(hipDeviceGetAttribute(&lds, hipDeviceAttributeMaxSharedMemoryPerBlock, h->device));
  if (O3Lay::bytes<double>() > static_cast<size_t>(lds)) return AMG_OK;
  QA_TRY(o3_lds_limits(h->device));
  h->oct_top = top;
  for (int pi = 0; pi < 2; pi++) {
    h->engine_top[pi] = top;
    h->engine_lds_top[pi] = kt == 4 ? top + 1 : top;  // the 512-cell level's rows lie in registers during its visits
    h->engine_nops[pi] = o3_steps(kt);
    h->engine_lds[pi] = pi ? O3Lay::bytes<float>() : O3Lay::bytes<double>();
    h->engine_flops[pi] = o3_flops(kt);
  }
  return AMG_OK;
}

void launch_engine_oct(amg_hierarchy *h, int precision) {
  const int top = h->oct_top;
  const bool four = h->lev[top].k == 4;
  const QuadLevel &Q = h->lev[top], &Q3 = h->lev[four ? top + 1 : top];
  if (precision) o3_launch<float>(h, h->w32[top], four ? Q.ax32 : nullptr, Q3.ax32, Q.oval32);
  else o3_launch<double>(h, h->w64[top], four ? Q.ax64 : nullptr, Q3.ax64, Q.oval64);
}

}  // namespace qa
