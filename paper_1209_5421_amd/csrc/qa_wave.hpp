// Wavefront reductions of doubles (gfx950, 64 lanes), shared by the engine and the tree-level kernels. Fixed trees: a
// sum depends only on the lanes' values.
#pragma once

#include <hip/hip_runtime.h>

namespace qa {

__host__ __device__ __forceinline__ float fma_of(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__host__ __device__ __forceinline__ double fma_of(double a, double b, double c) { return __builtin_fma(a, b, c); }

// n / d from rd = 1 / d rounded to nearest: q = n rd, then q + (n - q d) rd with fused multiply-adds (Markstein, IBM
// Journal of Research and Development 34, 1990). For d from the smallest normal number up; below about a quarter of that
// rd is infinite, and systems with such diagonals (amg_hierarchy::tiny_diag) take the division.
template <class T>
__host__ __device__ __forceinline__ T quotient(T n, T d, T rd) {
  const T q = n * rd;
  return fma_of(fma_of(-q, d, n), rd, q);
}

// lane N's value in every lane of each row of 16 lanes (row_newbcast); with G = 8, lane N's of each half row
template <int N, int G>
__device__ __forceinline__ float bcast_of(float x) {
  const int u = __builtin_bit_cast(int, x);
  int r = __builtin_amdgcn_update_dpp(0, u, 0x150 + N, 0xf, 0xf, true);
  if constexpr (G == 8) r = __builtin_amdgcn_update_dpp(r, u, 0x158 + N, 0xf, 0xc, false);
  return __builtin_bit_cast(float, r);
}
template <int N, int G>
__device__ __forceinline__ double bcast_of(double x) {
  const long u = __builtin_bit_cast(long, x);
  long r = __builtin_amdgcn_update_dpp(0L, u, 0x150 + N, 0xf, 0xf, true);
  if constexpr (G == 8) r = __builtin_amdgcn_update_dpp(r, u, 0x158 + N, 0xf, 0xc, false);
  return __builtin_bit_cast(double, r);
}

// a lane's double moved by a DPP lane pattern (two 32-bit moves)
template <int Ctrl>
__device__ __forceinline__ double dpp_f64(double x) {
  const unsigned long long u = __builtin_bit_cast(unsigned long long, x);
  const int lo = __builtin_amdgcn_update_dpp(0, static_cast<int>(u & 0xffffffffu), Ctrl, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, static_cast<int>(u >> 32), Ctrl, 0xf, 0xf, false);
  return __builtin_bit_cast(double, (static_cast<unsigned long long>(static_cast<unsigned>(hi)) << 32) |
                                        static_cast<unsigned>(lo));
}
__device__ __forceinline__ double readlane_f64(double x, int lane) {
  const unsigned long long u = __builtin_bit_cast(unsigned long long, x);
  const unsigned lo = static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(u & 0xffffffffu), lane));
  const unsigned hi = static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(u >> 32), lane));
  return __builtin_bit_cast(double, (static_cast<unsigned long long>(hi) << 32) | lo);
}

// the sum of x over the lanes i, i + 16, i + 32, i + 48 of a wavefront, in every one of them: rows of 16 lanes added in
// pairs, then the two halves
__device__ __forceinline__ double rows_sum(double x) {
  const unsigned long long u = __builtin_bit_cast(unsigned long long, x);
  const auto l0 = __builtin_amdgcn_permlane16_swap(static_cast<unsigned>(u), static_cast<unsigned>(u), false, false);
  const auto h0 =
      __builtin_amdgcn_permlane16_swap(static_cast<unsigned>(u >> 32), static_cast<unsigned>(u >> 32), false, false);
  x = __builtin_bit_cast(double, (static_cast<unsigned long long>(h0[0]) << 32) | l0[0]) +
      __builtin_bit_cast(double, (static_cast<unsigned long long>(h0[1]) << 32) | l0[1]);
  const unsigned long long w = __builtin_bit_cast(unsigned long long, x);
  const auto l1 = __builtin_amdgcn_permlane32_swap(static_cast<unsigned>(w), static_cast<unsigned>(w), false, false);
  const auto h1 =
      __builtin_amdgcn_permlane32_swap(static_cast<unsigned>(w >> 32), static_cast<unsigned>(w >> 32), false, false);
  return __builtin_bit_cast(double, (static_cast<unsigned long long>(h1[0]) << 32) | l1[0]) +
         __builtin_bit_cast(double, (static_cast<unsigned long long>(h1[1]) << 32) | l1[1]);
}

// four sums over one wavefront at once: in two steps of pairs each lane hands over the half of its values that its
// partner keeps, so that one value per lane is left (lane i holds a part of sum sum4_of(i & 3)), which is then added
// over the lanes of equal i & 3. A fixed tree: the result depends only on the lanes' values.
__device__ __forceinline__ constexpr int sum4_of(int i) { return (i & 1) * 2 + (i >> 1); }
__device__ __forceinline__ double wave_sum4(const double (&v)[4]) {
  const bool b0 = threadIdx.x & 1, b1 = threadIdx.x & 2;
  const double k0 = (b0 ? v[2] : v[0]) + dpp_f64<0xb1>(b0 ? v[0] : v[2]);  // quad_perm [1, 0, 3, 2]
  const double k1 = (b0 ? v[3] : v[1]) + dpp_f64<0xb1>(b0 ? v[1] : v[3]);
  double k = (b1 ? k1 : k0) + dpp_f64<0x4e>(b1 ? k0 : k1);                 // quad_perm [2, 3, 0, 1]
  k += dpp_f64<0x124>(k);                                                  // row_ror 4
  k += dpp_f64<0x128>(k);                                                  // row_ror 8
  return rows_sum(k);
}

// four sums over a workgroup of NT threads (at most 512), the same in every thread (all call): each wavefront's sums as
// above, then the wavefronts' added in pairs. red: 4 x 8 doubles of LDS, not in use before the next barrier but one.
template <int NT>
__device__ __forceinline__ void block_sum4(double (&v)[4], double (*red)[8]) {
  const int lane = static_cast<int>(threadIdx.x & 63), w = static_cast<int>(threadIdx.x >> 6);
  const double k = wave_sum4(v);
  if (lane < 4) red[sum4_of(lane)][w] = k;
  __syncthreads();
  double r = (lane & 7) < NT / 64 ? red[(lane >> 3) & 3][lane & 7] : 0.0;  // lanes 8 j .. 8 j + 7: the waves' v[j]
  r += dpp_f64<0xb1>(r);
  r += dpp_f64<0x4e>(r);
  r += dpp_f64<0x141>(r);
#pragma unroll
  for (int j = 0; j < 4; j++) v[j] = readlane_f64(r, 8 * j);
}

}  // namespace qa
