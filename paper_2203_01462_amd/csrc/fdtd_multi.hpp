// fdtd_multi.hpp -- what the several-step kernels of the two 2D polarizations
// share: region limits, lane shifts, address-space pointers and the launch's
// parameters.
#pragma once

#include "fdtd_2d.hpp"

namespace fdtd {

constexpr int MX = 64;          // columns of a region: one wavefront
constexpr int MKMAX = 12;       // most steps per launch
constexpr int MWMAX = 16;       // most wavefronts per workgroup

template <typename T>
using cptr = const __attribute__((address_space(4))) T *;
template <typename T>
using gptr = __attribute__((address_space(1))) T *;

__device__ __forceinline__ bool pml_e2(int i, int n, int P) { return P > 0 && (i < P || i > n - 1 - P); }
__device__ __forceinline__ bool pml_h2(int i, int n, int P) { return P > 0 && (i < P || i >= n - 1 - P); }

// The value of lane - 1 (wave_shr:1) / lane + 1 (wave_shl:1); 0 in the lane
// without one, which only feeds nodes outside the exact middle.
template <int CTRL>
__device__ __forceinline__ float lane_shift(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ double lane_shift(double v) {
  const long long b = __double_as_longlong(v);
  const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffll), CTRL, 0xf, 0xf, true);
  const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xf, 0xf, true);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
template <typename T>
__device__ __forceinline__ T lane_left(T v) { return lane_shift<0x138>(v); }
template <typename T>
__device__ __forceinline__ T lane_right(T v) { return lane_shift<0x130>(v); }

// What a launch does: `steps` steps from step number n0 on (ascending, or
// descending in the adjoint), copy rd read and copy rd ^ 1 written.
struct MultiStep {
  int n0, steps, rd;
  void *hist;  // history buffer (null: the instance's own, every step kept)
  int hist_base, hist_on;
};

// Regions a launch needs over one grid.
inline int multi_regions(int nx, int ny, const MultiTile &g) {
  const int W = MX - 2 * g.K, H = g.R * g.nw - 2 * g.K;
  return ((nx + W - 1) / W) * ((ny + H - 1) / H);
}

}  // namespace fdtd
