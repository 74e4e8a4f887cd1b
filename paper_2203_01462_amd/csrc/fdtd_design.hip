// fdtd_design.hip -- per-element kernels of the design-update loop: the
// open-close density filter of eq. (26) with its transposed Jacobian for the
// chain rule of eq. (27), one step of the method of moving asymptotes for a
// box-constrained objective (with the sums of its globally convergent
// variant), and the non-discreteness / optimality statistics.
//
// Sums are deterministic: every reduction writes one FP64 partial per
// workgroup (wavefront shuffles, then the four wavefronts in order), and the
// workgroup that finishes last adds the partials in a fixed order and writes
// the sums to host memory, so that a reduction is one launch.
#include <algorithm>
#include <cmath>
#include <map>
#include <string>
#include <vector>

#include "fdtd_design.h"
#include "fdtd_internal.hpp"

using namespace fdtd;

namespace {

thread_local std::string g_err;

constexpr int BS = 256;   // threads per workgroup (4 wavefronts)
constexpr int RS = 1024;  // ... of a reduction, at most

// A reduction's workgroups: their arrivals are served one at a time, about 20 ns
// each, so there are at most 256 and their threads take several elements
// (512 x 512 cells: mma_begin with its wait 42 us with 1024 workgroups of 256, 26
// with 256 of 1024, 27 as three launches), of 256 threads while that is one
// element each (128 x 128: 17.5 us, 19.5 with 1024).
constexpr int kReduceBlocks = 256;

template <typename F>
fdtd_status dguard(F &&f) {
  try {
    f();
    return FDTD_OK;
  } catch (const Error &e) {
    g_err = e.msg;
    return e.code;
  } catch (const std::bad_alloc &) {
    g_err = "host out of memory";
    return FDTD_ENOMEM;
  }
}

// ---------------------------------------------------------------- reductions
// Sums of the NQ values over the workgroup, for thread 0: wavefront shuffles,
// then the first wavefront over the wavefronts' sums (a fixed order).
template <int NQ>
__device__ __forceinline__ void block_sums(double (&v)[NQ]) {
  __shared__ double lds[NQ][RS / 64];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    for (int o = 32; o > 0; o >>= 1) v[q] += __shfl_down(v[q], o, 64);
    if (lane == 0) lds[q][w] = v[q];
  }
  __syncthreads();
  if (w == 0) {
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      double s = lane < (int)blockDim.x / 64 ? lds[q][lane] : 0;
      for (int o = RS / 128; o > 0; o >>= 1) s += __shfl_down(s, o, 64);
      v[q] = s;
    }
  }
  __syncthreads();
}

// The end of a reduction of the threads' v: the workgroup's sums go to
// part[block * NQ + q]; the workgroup that arrives last adds all partials into
// out (host memory) and rearms the counter.
template <int NQ>
__device__ __forceinline__ void finish_block(double (&v)[NQ], double *part, unsigned *count, double *out) {
  __shared__ bool last;
  block_sums(v);
  if (threadIdx.x == 0) {
    for (int q = 0; q < NQ; ++q) part[(size_t)blockIdx.x * NQ + q] = v[q];
    __threadfence();
    last = atomicAdd(count, 1u) == gridDim.x - 1;
  }
  __syncthreads();
  if (!last) return;
  __threadfence();
  for (int q = 0; q < NQ; ++q) v[q] = threadIdx.x < gridDim.x ? part[(size_t)threadIdx.x * NQ + q] : 0;
  block_sums(v);
  if (threadIdx.x == 0) {
    for (int q = 0; q < NQ; ++q) out[q] = v[q];
    *count = 0;
  }
}

int nblocks(int64_t n) { return (int)((n + BS - 1) / BS); }
int rthreads(int64_t n) { return n <= (int64_t)BS * kReduceBlocks ? BS : RS; }
int rblocks(int64_t n) { return (int)std::min<int64_t>((n + rthreads(n) - 1) / rthreads(n), kReduceBlocks); }

// Partials, arrival counter and the sums of a reduction.  The sums are pinned
// host memory that the kernel writes: read after the stream has drained.
struct Reduction {
  DevBuf part, count;
  double *sums = nullptr;
  void alloc() {
    part.alloc(kReduceBlocks * 2 * sizeof(double));
    if (!sums) {
      count.alloc(sizeof(unsigned));
      FDTD_HIP(hipMemset(count.p, 0, sizeof(unsigned)));
      FDTD_HIP(hipStreamSynchronize(nullptr));
      FDTD_HIP(hipHostMalloc((void **)&sums, 2 * sizeof(double), hipHostMallocDefault));
    }
  }
  Reduction() = default;
  Reduction(const Reduction &) = delete;
  Reduction &operator=(const Reduction &) = delete;
  ~Reduction() {
    if (sums) (void)hipHostFree(sums);
  }
};

// ---------------------------------------------------------------- filter
// Cell coordinates of linear index i in an nx x ny x nz box (x fastest).
__device__ __forceinline__ void coords(int64_t i, int nx, int ny, int &ix, int &iy, int &iz) {
  ix = (int)(i % nx);
  iy = (int)((i / nx) % ny);
  iz = (int)(i / ((int64_t)nx * ny));
}

// 1 / sum_j w_ij over the box (the weights are symmetric: w_ij = w_ji).
__global__ void __launch_bounds__(BS) winv_kernel(double *winv, int nx, int ny, int nz, double r, int R, int Rz) {
  const int64_t i = (int64_t)blockIdx.x * BS + threadIdx.x;
  if (i >= (int64_t)nx * ny * nz) return;
  int ix, iy, iz;
  coords(i, nx, ny, ix, iy, iz);
  double s = 0;
  for (int dz = -Rz; dz <= Rz; ++dz)
    for (int dy = -R; dy <= R; ++dy)
      for (int dx = -R; dx <= R; ++dx) {
        const int jx = ix + dx, jy = iy + dy, jz = iz + dz;
        if (jx < 0 || jx >= nx || jy < 0 || jy >= ny || jz < 0 || jz >= nz) continue;
        const double w = r - sqrt((double)(dx * dx + dy * dy + dz * dz));
        if (w > 0) s += w;
      }
  winv[i] = 1.0 / s;
}

// One fW-mean stage: e_i = f^-1(sum_j w_ij f(u_j) * winv_i), f(u) = 1/(u+alpha);
// erosion (dual = 0): u = x, y = e; dilation (dual = 1): u = 1-x, y = 1-e.
template <typename TI, typename TO>
__global__ void __launch_bounds__(BS) stage_kernel(const TI *__restrict__ x, TO *__restrict__ y,
                                                  const double *__restrict__ winv, int nx, int ny, int nz, double r,
                                                  int R, int Rz, double alpha, int dual) {
  const int64_t i = (int64_t)blockIdx.x * BS + threadIdx.x;
  if (i >= (int64_t)nx * ny * nz) return;
  int ix, iy, iz;
  coords(i, nx, ny, ix, iy, iz);
  double s = 0;
  for (int dz = -Rz; dz <= Rz; ++dz)
    for (int dy = -R; dy <= R; ++dy)
      for (int dx = -R; dx <= R; ++dx) {
        const int jx = ix + dx, jy = iy + dy, jz = iz + dz;
        if (jx < 0 || jx >= nx || jy < 0 || jy >= ny || jz < 0 || jz >= nz) continue;
        const double w = r - sqrt((double)(dx * dx + dy * dy + dz * dz));
        if (w <= 0) continue;
        const double xj = (double)x[((int64_t)jz * ny + jy) * nx + jx];
        const double u = dual ? 1.0 - xj : xj;
        s += w / (u + alpha);
      }
  const double e = 1.0 / (s * winv[i]) - alpha;
  // an fW-mean of values in [0,1] lies in [0,1]; clamp off the rounding
  // (all-void or all-metal neighbourhoods land within an ulp of the bounds)
  y[i] = (TO)fmin(fmax(dual ? 1.0 - e : e, 0.0), 1.0);
}

// Transpose of one stage at input x, output y: with e = (dual ? 1-y : y),
// u = (dual ? 1-x : x): h_i = gy_i winv_i (e_i+alpha)^2 and
// gx_j = (u_j+alpha)^-2 sum_i w_ij h_i.  (The two sign flips of the dual
// stage cancel.)
template <typename TG, typename TY>
__global__ void __launch_bounds__(BS) stage_h_kernel(const TG *__restrict__ gy, const TY *__restrict__ y,
                                                    const double *__restrict__ winv, int64_t n, double alpha, int dual,
                                                    double *__restrict__ h) {
  const int64_t i = (int64_t)blockIdx.x * BS + threadIdx.x;
  if (i >= n) return;
  const double yi = (double)y[i];
  const double e = dual ? 1.0 - yi : yi;
  h[i] = (double)gy[i] * winv[i] * (e + alpha) * (e + alpha);
}

template <typename TX, typename TO>
__global__ void __launch_bounds__(BS) stage_gather_kernel(const double *__restrict__ h, const TX *__restrict__ x,
                                                         TO *__restrict__ gx, int nx, int ny, int nz, double r, int R,
                                                         int Rz, double alpha, int dual) {
  const int64_t j = (int64_t)blockIdx.x * BS + threadIdx.x;
  if (j >= (int64_t)nx * ny * nz) return;
  int jx, jy, jz;
  coords(j, nx, ny, jx, jy, jz);
  double s = 0;
  for (int dz = -Rz; dz <= Rz; ++dz)
    for (int dy = -R; dy <= R; ++dy)
      for (int dx = -R; dx <= R; ++dx) {
        const int ix = jx + dx, iy = jy + dy, iz = jz + dz;
        if (ix < 0 || ix >= nx || iy < 0 || iy >= ny || iz < 0 || iz >= nz) continue;
        const double w = r - sqrt((double)(dx * dx + dy * dy + dz * dz));
        if (w <= 0) continue;
        s += w * h[((int64_t)iz * ny + iy) * nx + ix];
      }
  const double xj = (double)x[j];
  const double u = dual ? 1.0 - xj : xj;
  gx[j] = (TO)(s / ((u + alpha) * (u + alpha)));
}

// What bounds these stages is latency: a thread a cell that forms each weight
// (a square root) and each f(u) (a division) again from global memory took
// 12.7 us a stage on 128 x 128 cells and 10.6 + 3.9 us a transposed stage.
// Tiled forms: a workgroup forms f(u) (or h) once per cell of its tile and halo
// into LDS and walks a list of taps (offset in the LDS tile, weight; the order
// of the loops above, cells outside the box hold zero), which every lane reads
// at the same address.
struct Tap {
  double w;
  int off, pad;
};
constexpr int CB = 32;                       // side of the cells a cascade workgroup computes
constexpr int CMAXR = 3;                     // (its stored tile, CB - 6 R, is a fifth of them at R = 3)

// w_ij-weighted sum around LDS cell `at`.
__device__ __forceinline__ double tap_sum(const double *f, int at, const Tap *__restrict__ taps, int nt) {
  double s = 0;
#pragma unroll 16
  for (int t = 0; t < nt; ++t) s += taps[t].w * f[at + taps[t].off];
  return s;
}

template <typename T>
struct Cascade {
  const T *x;      // input of the first stage
  T *xs[5];        // stage inputs and output, kept for the transpose
  T *out;
  const double *winv;
  const Tap *taps;
  int nt, nx, ny, R;
  double alpha;
};

// All four stages on a 2D box: thread (tx, ty) of a workgroup computes cell
// (x0 - 3 R + tx, y0 - 3 R + ty) in every stage, whose valid cells shrink by R
// a side, and the middle CB - 6 R squared are stored.  A stage's output is
// rounded to T before the next reads it.  128 x 128 FP32, R = 3: four stages
// and two copies 53 us -> 9.0.
template <typename T>
__global__ void __launch_bounds__(CB * CB) cascade_kernel(const Cascade<T> c) {
  __shared__ double f[2][(CB + 2 * CMAXR) * (CB + 2 * CMAXR)];
  const int R = c.R, side = CB + 2 * R, tile = CB - 6 * R;
  const int tx = threadIdx.x & (CB - 1), ty = threadIdx.x / CB;
  const int x0 = blockIdx.x * tile - 4 * R, y0 = blockIdx.y * tile - 4 * R;  // corner of the LDS tile
  const int ix = x0 + R + tx, iy = y0 + R + ty, at = (R + ty) * side + R + tx;
  const bool in = ix >= 0 && ix < c.nx && iy >= 0 && iy < c.ny;
  const int64_t i = in ? (int64_t)iy * c.nx + ix : 0;
  const bool keep = in && tx >= 3 * R && tx < 3 * R + tile && ty >= 3 * R && ty < 3 * R + tile;
  const double winv = c.winv[i];
  if (keep) c.xs[0][i] = c.x[i];
  for (int k = threadIdx.x; k < side * side; k += CB * CB) {
    const int r = k / side, q = k - r * side, jx = x0 + q, jy = y0 + r;
    const bool ok = jx >= 0 && jx < c.nx && jy >= 0 && jy < c.ny;
    f[0][k] = ok ? 1.0 / ((double)c.x[(int64_t)jy * c.nx + jx] + c.alpha) : 0.0;
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const bool dual = k == 1 || k == 2, next = k == 0 || k == 1;  // (of the stage after this one)
    const int m = R * k;
    if (tx >= m && tx < CB - m && ty >= m && ty < CB - m) {
      const double e = 1.0 / (tap_sum(f[k & 1], at, c.taps, c.nt) * winv) - c.alpha;
      const T y = (T)fmin(fmax(dual ? 1.0 - e : e, 0.0), 1.0);
      if (keep) c.xs[k + 1][i] = y;
      if (k == 3) {
        if (keep) c.out[i] = y;
      } else {
        const double u = next ? 1.0 - (double)y : (double)y;
        f[(k & 1) ^ 1][at] = in ? 1.0 / (u + c.alpha) : 0.0;
      }
    }
    if (k < 3) __syncthreads();
  }
}

template <typename T>
struct CascadeBack {
  const T *gy;
  const T *xs[5];
  T *gx;
  const double *winv;
  const Tap *taps;
  int nt, nx, ny, R;
  double alpha;
};

// The transposed cascade on the same cells: h of stage 3 over the LDS tile,
// then per stage the gather and the next stage's h; the gradients between the
// stages stay in FP64.  128 x 128 FP32, R = 3: eight launches 49 us -> 8.8.
template <typename T>
__global__ void __launch_bounds__(CB * CB) cascade_back_kernel(const CascadeBack<T> c) {
  __shared__ double h[2][(CB + 2 * CMAXR) * (CB + 2 * CMAXR)];
  const int R = c.R, side = CB + 2 * R, tile = CB - 6 * R;
  const int tx = threadIdx.x & (CB - 1), ty = threadIdx.x / CB;
  const int x0 = blockIdx.x * tile - 4 * R, y0 = blockIdx.y * tile - 4 * R;
  const int ix = x0 + R + tx, iy = y0 + R + ty, at = (R + ty) * side + R + tx;
  const bool in = ix >= 0 && ix < c.nx && iy >= 0 && iy < c.ny;
  const int64_t i = in ? (int64_t)iy * c.nx + ix : 0;
  const bool keep = in && tx >= 3 * R && tx < 3 * R + tile && ty >= 3 * R && ty < 3 * R + tile;
  const double winv = c.winv[i];
  double xk[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) xk[k] = (double)c.xs[k][i];
  for (int k = threadIdx.x; k < side * side; k += CB * CB) {
    const int r = k / side, q = k - r * side, jx = x0 + q, jy = y0 + r;
    const bool ok = jx >= 0 && jx < c.nx && jy >= 0 && jy < c.ny;
    const int64_t j = ok ? (int64_t)jy * c.nx + jx : 0;
    const double e = (double)c.xs[4][j];
    h[0][k] = ok ? (double)c.gy[j] * c.winv[j] * (e + c.alpha) * (e + c.alpha) : 0.0;
  }
  __syncthreads();
#pragma unroll
  for (int k = 3; k >= 0; --k) {
    const bool dual = k == 1 || k == 2, next = k == 3 || k == 2;  // (of stage k - 1)
    const int m = R * (3 - k), b = (3 - k) & 1;
    if (tx >= m && tx < CB - m && ty >= m && ty < CB - m) {
      const double u = dual ? 1.0 - xk[k] : xk[k];
      const double g = tap_sum(h[b], at, c.taps, c.nt) / ((u + c.alpha) * (u + c.alpha));
      if (k == 0) {
        if (keep) c.gx[i] = (T)g;
      } else {
        const double e = next ? 1.0 - xk[k] : xk[k];
        h[b ^ 1][at] = in ? g * winv * (e + c.alpha) * (e + c.alpha) : 0.0;
      }
    }
    if (k > 0) __syncthreads();
  }
}

// The cell and LDS layout of a tiled single stage: a tile of tx x ty x tz
// cells (a thread each) in a box with a halo of Rx, Ry, Rz cells.
struct Tile {
  int nx, ny, nz, Rx, Ry, Rz, tx, ty, tz;
  __host__ __device__ __forceinline__ int sx() const { return tx + 2 * Rx; }
  __host__ __device__ __forceinline__ int sy() const { return ty + 2 * Ry; }
  __host__ __device__ __forceinline__ int sz() const { return tz + 2 * Rz; }
};

// Calls fill(cell, k) -> value for every LDS cell k inside the box (cell: its
// linear index), zero elsewhere.
template <typename F>
__device__ __forceinline__ void fill_tile(const Tile &g, double *lds, F &&fill) {
  const int sx = g.sx(), sy = g.sy(), cells = sx * sy * g.sz();
  for (int k = threadIdx.x; k < cells; k += blockDim.x) {
    const int r = k / sx, q = k - r * sx, p = r / sy;
    const int jx = (int)blockIdx.x * g.tx - g.Rx + q, jy = (int)blockIdx.y * g.ty - g.Ry + (r - p * sy),
              jz = (int)blockIdx.z * g.tz - g.Rz + p;
    const bool ok = jx >= 0 && jx < g.nx && jy >= 0 && jy < g.ny && jz >= 0 && jz < g.nz;
    lds[k] = ok ? fill(((int64_t)jz * g.ny + jy) * g.nx + jx) : 0.0;
  }
}

// The thread's cell (false: outside the box) and its LDS cell.
__device__ __forceinline__ bool tile_cell(const Tile &g, int64_t &i, int &at) {
  const int t = threadIdx.x, lx = t % g.tx, ly = (t / g.tx) % g.ty, lz = t / (g.tx * g.ty);
  const int ix = blockIdx.x * g.tx + lx, iy = blockIdx.y * g.ty + ly, iz = blockIdx.z * g.tz + lz;
  i = ((int64_t)iz * g.ny + iy) * g.nx + ix;
  at = ((lz + g.Rz) * g.sy() + ly + g.Ry) * g.sx() + lx + g.Rx;
  return ix < g.nx && iy < g.ny && iz < g.nz;
}

// One stage on tiles (any 2D box; 3D up to R = 4); copy (if set) keeps the
// input.  64 x 64 x 16 FP64, R = 3: 60 us a stage with the kernel above -> 9.4.
template <typename T>
__global__ void __launch_bounds__(1024) stage_tile_kernel(const Tile g, const T *__restrict__ x, T *__restrict__ copy,
                                                         T *__restrict__ y, T *__restrict__ y2,
                                                         const double *__restrict__ winv,
                                                         const Tap *__restrict__ taps, int nt, double alpha,
                                                         int dual) {
  extern __shared__ double f[];
  fill_tile(g, f, [&](int64_t j) {
    const double xj = (double)x[j];
    return 1.0 / ((dual ? 1.0 - xj : xj) + alpha);
  });
  __syncthreads();
  int64_t i;
  int at;
  if (!tile_cell(g, i, at)) return;
  const double e = 1.0 / (tap_sum(f, at, taps, nt) * winv[i]) - alpha;
  const T v = (T)fmin(fmax(dual ? 1.0 - e : e, 0.0), 1.0);
  if (copy) copy[i] = x[i];
  y[i] = v;
  if (y2) y2[i] = v;
}

// Its transpose: h over the tile and its halo, then the gather.
template <typename TG, typename T, typename TO>
__global__ void __launch_bounds__(1024) stage_back_tile_kernel(const Tile g, const TG *__restrict__ gy,
                                                              const T *__restrict__ y, const T *__restrict__ x,
                                                              TO *__restrict__ gx, const double *__restrict__ winv,
                                                              const Tap *__restrict__ taps, int nt, double alpha,
                                                              int dual) {
  extern __shared__ double h[];
  fill_tile(g, h, [&](int64_t j) {
    const double yj = (double)y[j], e = dual ? 1.0 - yj : yj;
    return (double)gy[j] * winv[j] * (e + alpha) * (e + alpha);
  });
  __syncthreads();
  int64_t i;
  int at;
  if (!tile_cell(g, i, at)) return;
  const double xj = (double)x[i], u = dual ? 1.0 - xj : xj;
  gx[i] = (TO)(tap_sum(h, at, taps, nt) / ((u + alpha) * (u + alpha)));
}

// ---------------------------------------------------------------- MMA
struct MmaArgs {
  double xmin, xmax, move, asyinit, asyincr, asydecr;
};

// Asymptotes and move limits of an outer iteration (k = accepted iterations
// so far); partial sums of |df0| for the initial curvature weight.
template <typename T>
__global__ void __launch_bounds__(RS) mma_begin_kernel(const T *__restrict__ xin, const T *__restrict__ dfin, int64_t n,
                                                      int k, MmaArgs a, double *__restrict__ x, double *__restrict__ df,
                                                      const double *__restrict__ xo1, const double *__restrict__ xo2,
                                                      double *__restrict__ L, double *__restrict__ U,
                                                      double *__restrict__ lo, double *__restrict__ hi,
                                                      double *part, unsigned *count, double *out) {
  double s[1] = {0};
  for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < n; j += (int64_t)gridDim.x * blockDim.x) {
    const double xj = (double)xin[j], dj = (double)dfin[j], dx = a.xmax - a.xmin;
    double l, u;
    if (k < 2) {
      l = xj - a.asyinit * dx;
      u = xj + a.asyinit * dx;
    } else {
      const double t = (xj - xo1[j]) * (xo1[j] - xo2[j]);
      const double g = t < 0 ? a.asydecr : (t > 0 ? a.asyincr : 1.0);
      l = xj - g * (xo1[j] - L[j]);
      u = xj + g * (U[j] - xo1[j]);
      l = fmin(fmax(l, xj - 10.0 * dx), xj - 0.01 * dx);
      u = fmax(fmin(u, xj + 10.0 * dx), xj + 0.01 * dx);
    }
    x[j] = xj;
    df[j] = dj;
    L[j] = l;
    U[j] = u;
    lo[j] = fmax(fmax(a.xmin, l + 0.1 * (xj - l)), xj - a.move * dx);
    hi[j] = fmin(fmin(a.xmax, u - 0.1 * (u - xj)), xj + a.move * dx);
    s[0] += fabs(dj) * dx;
  }
  finish_block(s, part, count, out);
}

// Minimizer of the separable approximation with curvature weight rho:
// p = (U-x)^2 (1.001 g+ + 0.001 g- + rho/dx), q = (x-L)^2 (0.001 g+ + 1.001 g- + rho/dx),
// x* = clamp((sqrt(p) L + sqrt(q) U) / (sqrt(p) + sqrt(q)), lo, hi); partial sums
// of the change of p/(U-.) + q/(.-L) from x to x* (formed per element as
// (x*-x) [p/((U-x*)(U-x)) - q/((x*-L)(x-L))], so large rho does not cancel)
// and of the distance measure.
template <typename T>
__global__ void __launch_bounds__(RS) mma_solve_kernel(const double *__restrict__ x, const double *__restrict__ df,
                                                      const double *__restrict__ L, const double *__restrict__ U,
                                                      const double *__restrict__ lo, const double *__restrict__ hi,
                                                      int64_t n, double rho, MmaArgs a, T *__restrict__ xnew,
                                                      double *part, unsigned *count, double *out) {
  double s[2] = {0, 0};
  for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < n; j += (int64_t)gridDim.x * blockDim.x) {
    const double xj = x[j], d = df[j], l = L[j], u = U[j], dx = a.xmax - a.xmin;
    const double gp = fmax(d, 0.0), gm = fmax(-d, 0.0);
    const double p = (u - xj) * (u - xj) * (1.001 * gp + 0.001 * gm + rho / dx);
    const double q = (xj - l) * (xj - l) * (0.001 * gp + 1.001 * gm + rho / dx);
    const double sp = sqrt(p), sq = sqrt(q);
    double xs = (sp * l + sq * u) / (sp + sq);
    xs = fmin(fmax(xs, lo[j]), hi[j]);
    const T xt = (T)xs;
    xnew[j] = xt;
    const double xr = (double)xt;  // the value the caller evaluates
    s[0] += (xr - xj) * (p / ((u - xr) * (u - xj)) - q / ((xr - l) * (xj - l)));
    s[1] += (u - l) * (xr - xj) * (xr - xj) / ((u - xr) * (xr - l) * dx);
  }
  finish_block(s, part, count, out);
}

template <typename T>
__global__ void __launch_bounds__(BS) mma_accept_kernel(const T *__restrict__ xnew, int64_t n, double *__restrict__ x,
                                                       double *__restrict__ xo1, double *__restrict__ xo2) {
  const int64_t j = (int64_t)blockIdx.x * BS + threadIdx.x;
  if (j >= n) return;
  xo2[j] = xo1[j];
  xo1[j] = x[j];
  x[j] = (double)xnew[j];
}

// ---------------------------------------------------------------- stats
template <typename T>
__global__ void __launch_bounds__(RS) stats_kernel(const T *__restrict__ x, const T *__restrict__ g, int64_t n,
                                                  double xmin, double xmax, double *part, unsigned *count,
                                                  double *out) {
  double s[2] = {0, 0};
  for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < n; j += (int64_t)gridDim.x * blockDim.x) {
    const double xj = (double)x[j];
    s[0] += 4.0 * xj * (1.0 - xj);
    if (g) {
      const double r = xj - fmin(fmax(xj - (double)g[j], xmin), xmax);
      s[1] += r * r;
    }
  }
  finish_block(s, part, count, out);
}

// Workspace of design_stats, a few KiB per thread and device, freed with the
// thread: a call returns with its stream drained, so the next call of the
// thread finds it idle whatever stream it uses.
Reduction &stats_work() {
  thread_local std::map<int, Reduction> work;
  int dev = 0;
  FDTD_HIP(hipGetDevice(&dev));
  Reduction &r = work[dev];
  if (!r.sums) r.alloc();
  return r;
}

hipStream_t own_or(void *s, bool &own) {
  if (s) {
    own = false;
    return (hipStream_t)s;
  }
  hipStream_t t;
  FDTD_HIP(hipStreamCreate(&t));
  own = true;
  return t;
}

}  // namespace

struct fdtd_filter {
  int nx = 1, ny = 1, nz = 1, prec = 64, R = 0, Rz = 0;
  int64_t n = 0;
  double r = 0, alpha = 0;
  bool applied = false, own = false;
  hipStream_t s = nullptr;
  DevBuf winv, xs[5], h, g[2];  // stage inputs x0..x3 and output x4; transpose scratch
  // the route by box and radius: all stages in one launch, one launch a stage
  // on tiles, or (3D beyond R = 4, whose halo exceeds the LDS, and boxes with
  // more tiles than a grid has room for) the plain kernels
  enum { kCascade, kTiled, kPlain } route = kPlain;
  Tile tile{};
  int nt = 0;
  DevBuf taps;
  ~fdtd_filter() {
    if (s) (void)hipStreamSynchronize(s);
    if (own && s) (void)hipStreamDestroy(s);
  }
};

struct fdtd_mma {
  int64_t n = 0;
  int prec = 64, k = 0;
  bool begun = false, own = false;
  double f0 = 0;
  MmaArgs a{};
  hipStream_t s = nullptr;
  DevBuf x, df, xo1, xo2, L, U, lo, hi;
  Reduction red;
  ~fdtd_mma() {
    if (s) (void)hipStreamSynchronize(s);
    if (own && s) (void)hipStreamDestroy(s);
  }
};

namespace {

// Forward stage k of the cascade: erode, dilate, dilate, erode.
constexpr int kDual[4] = {0, 1, 1, 0};

bool overlap(const void *a, const void *b, size_t bytes) {
  const auto x = (uintptr_t)a, y = (uintptr_t)b;
  return x < y + bytes && y < x + bytes;
}

dim3 tile_grid(const Tile &g) {
  return dim3((g.nx + g.tx - 1) / g.tx, (g.ny + g.ty - 1) / g.ty, (g.nz + g.tz - 1) / g.tz);
}
size_t tile_lds(const Tile &g) {
  return (size_t)g.sx() * g.sy() * g.sz() * sizeof(double);
}

template <typename T>
void filter_apply(fdtd_filter *f, const void *rho, void *out, double alpha) {
  const dim3 g(nblocks(f->n)), b(BS);
  const T *x = (const T *)rho;
  if (f->route == fdtd_filter::kPlain || overlap(rho, out, f->n * sizeof(T))) {
    FDTD_HIP(hipMemcpyAsync(f->xs[0].p, rho, f->n * sizeof(T), hipMemcpyDeviceToDevice, f->s));
    x = f->xs[0].as<T>();
  }
  if (f->route == fdtd_filter::kCascade) {
    Cascade<T> c{x, {}, (T *)out, f->winv.as<double>(), f->taps.as<Tap>(), f->nt, f->nx, f->ny, f->R, alpha};
    for (int k = 0; k < 5; ++k) c.xs[k] = f->xs[k].as<T>();
    const int t = CB - 6 * f->R;
    hipLaunchKernelGGL(cascade_kernel<T>, dim3((f->nx + t - 1) / t, (f->ny + t - 1) / t), dim3(CB * CB), 0, f->s, c);
  } else if (f->route == fdtd_filter::kTiled) {
    for (int k = 0; k < 4; ++k)
      hipLaunchKernelGGL(stage_tile_kernel<T>, tile_grid(f->tile), dim3(f->tile.tx * f->tile.ty * f->tile.tz), tile_lds(f->tile), f->s, f->tile,
                         k ? f->xs[k].as<T>() : x, k || x == f->xs[0].as<T>() ? nullptr : f->xs[0].as<T>(),
                         f->xs[k + 1].as<T>(), k == 3 ? (T *)out : nullptr, f->winv.as<double>(), f->taps.as<Tap>(),
                         f->nt, alpha, kDual[k]);
  } else {
    for (int k = 0; k < 4; ++k)
      hipLaunchKernelGGL((stage_kernel<T, T>), g, b, 0, f->s, f->xs[k].as<T>(), f->xs[k + 1].as<T>(),
                         f->winv.as<double>(), f->nx, f->ny, f->nz, f->r, f->R, f->Rz, alpha, kDual[k]);
    FDTD_HIP(hipMemcpyAsync(out, f->xs[4].p, f->n * sizeof(T), hipMemcpyDeviceToDevice, f->s));
  }
  FDTD_HIP(hipGetLastError());
}

template <typename T>
void filter_transpose(fdtd_filter *f, const void *gf, void *gout) {
  const dim3 g(nblocks(f->n)), b(BS);
  const double a = f->alpha;
  if (f->route == fdtd_filter::kCascade) {
    const T *gy = (const T *)gf;
    if (overlap(gf, gout, f->n * sizeof(T))) {
      FDTD_HIP(hipMemcpyAsync(f->h.p, gf, f->n * sizeof(T), hipMemcpyDeviceToDevice, f->s));
      gy = f->h.as<T>();
    }
    CascadeBack<T> c{gy, {}, (T *)gout, f->winv.as<double>(), f->taps.as<Tap>(), f->nt, f->nx, f->ny, f->R, a};
    for (int k = 0; k < 5; ++k) c.xs[k] = f->xs[k].as<T>();
    const int t = CB - 6 * f->R;
    hipLaunchKernelGGL(cascade_back_kernel<T>, dim3((f->nx + t - 1) / t, (f->ny + t - 1) / t), dim3(CB * CB), 0,
                       f->s, c);
    FDTD_HIP(hipGetLastError());
    return;
  }
  if (f->route == fdtd_filter::kTiled) {
    const dim3 tg = tile_grid(f->tile), tb(f->tile.tx * f->tile.ty * f->tile.tz);
    const size_t lds = tile_lds(f->tile);
    double *ga = f->g[0].as<double>(), *gb = f->g[1].as<double>();
    const double *wi = f->winv.as<double>();
    const Tap *tp = f->taps.as<Tap>();
    hipLaunchKernelGGL((stage_back_tile_kernel<T, T, double>), tg, tb, lds, f->s, f->tile, (const T *)gf,
                       f->xs[4].as<T>(), f->xs[3].as<T>(), ga, wi, tp, f->nt, a, kDual[3]);
    hipLaunchKernelGGL((stage_back_tile_kernel<double, T, double>), tg, tb, lds, f->s, f->tile, ga, f->xs[3].as<T>(),
                       f->xs[2].as<T>(), gb, wi, tp, f->nt, a, kDual[2]);
    hipLaunchKernelGGL((stage_back_tile_kernel<double, T, double>), tg, tb, lds, f->s, f->tile, gb, f->xs[2].as<T>(),
                       f->xs[1].as<T>(), ga, wi, tp, f->nt, a, kDual[1]);
    hipLaunchKernelGGL((stage_back_tile_kernel<double, T, T>), tg, tb, lds, f->s, f->tile, ga, f->xs[1].as<T>(),
                       f->xs[0].as<T>(), (T *)gout, wi, tp, f->nt, a, kDual[0]);
    FDTD_HIP(hipGetLastError());
    return;
  }
  // stage 3 (erode, x3 -> x4) from the caller's gradient; intermediate
  // gradients in FP64
  hipLaunchKernelGGL((stage_h_kernel<T, T>), g, b, 0, f->s, (const T *)gf, f->xs[4].as<T>(), f->winv.as<double>(),
                     f->n, a, kDual[3], f->h.as<double>());
  int cur = 0;
  for (int k = 3; k >= 0; --k) {
    if (k < 3)
      hipLaunchKernelGGL((stage_h_kernel<double, T>), g, b, 0, f->s, f->g[cur ^ 1].as<double>(), f->xs[k + 1].as<T>(),
                         f->winv.as<double>(), f->n, a, kDual[k], f->h.as<double>());
    if (k > 0)
      hipLaunchKernelGGL((stage_gather_kernel<T, double>), g, b, 0, f->s, f->h.as<double>(), f->xs[k].as<T>(),
                         f->g[cur].as<double>(), f->nx, f->ny, f->nz, f->r, f->R, f->Rz, a, kDual[k]);
    else
      hipLaunchKernelGGL((stage_gather_kernel<T, T>), g, b, 0, f->s, f->h.as<double>(), f->xs[0].as<T>(), (T *)gout,
                         f->nx, f->ny, f->nz, f->r, f->R, f->Rz, a, kDual[0]);
    cur ^= 1;
  }
  FDTD_HIP(hipGetLastError());
}

// The route of a filter and its taps at the LDS strides of that route.  A
// cascade's workgroups compute five cells for each they store (R = 3), so the
// single launch wins while three rounds of the CUs hold it (us per filter, cascade
// against tiles: 300^2 14 / 22, 512^2 35 / 24).  Tiles of 256 cells where those of
// 1024 would leave half of the CUs idle (100^2, R = 8:
// 70 -> 47 us a filter).  Along an axis of few cells the tile is as short as the box
// and longer along the others, and halo and taps keep inside the box (us per filter,
// square tiles / these / the plain kernels, forward and transpose: 4000000 x 1,
// R = 2 4922 / 248 / 461; 1000000 x 2, R = 3 1343 / 194 / 444).
void filter_route(fdtd_filter *f) {
  const bool flat = f->nz == 1;
  if (!flat && f->R > 4) return;
  const int side = CB - 6 * f->R;  // (used up to R = 3)
  const bool cascade = flat && f->R <= CMAXR &&
                       (int64_t)((f->nx + side - 1) / side) * ((f->ny + side - 1) / side) <= 768;
  const bool small = f->n <= 131072;
  const int n[3] = {f->nx, f->ny, f->nz}, R[3] = {std::min(f->R, f->nx - 1), std::min(f->R, f->ny - 1),
                                                  std::min(f->Rz, f->nz - 1)};
  int t[3] = {flat ? (small ? 16 : 32) : (small ? 8 : 16), flat ? (small ? 16 : 32) : 8, flat ? 1 : (small ? 4 : 8)};
  int spare = 1;
  for (int d = 0; d < 3; ++d)
    while (t[d] > 1 && t[d] / 2 >= n[d]) {
      t[d] /= 2;
      spare *= 2;
    }
  auto cells = [&] { return (t[0] + 2 * R[0]) * (t[1] + 2 * R[1]) * (t[2] + 2 * R[2]); };
  for (int d = 0; d < 3; ++d)
    while (spare > 1 && t[d] < n[d]) {
      t[d] *= 2;
      if (cells() > 8192) {  // 64 KiB of LDS
        t[d] /= 2;
        break;
      }
      spare /= 2;
    }
  f->tile = Tile{f->nx, f->ny, f->nz, R[0], R[1], R[2], t[0], t[1], t[2]};
  const dim3 g = tile_grid(f->tile);
  // (what a grid has room for: 65535 tiles along y and z, 2^32 threads along x)
  const bool fits = g.y <= 65535 && g.z <= 65535 && (uint64_t)g.x * (t[0] * t[1] * t[2]) < (1ull << 32);
  if (!cascade && !fits) return;
  f->route = cascade ? fdtd_filter::kCascade : fdtd_filter::kTiled;
  const int sx = cascade ? CB + 2 * f->R : f->tile.sx(), sy = f->tile.sy();
  std::vector<Tap> taps;
  for (int dz = -R[2]; dz <= R[2]; ++dz)
    for (int dy = -R[1]; dy <= R[1]; ++dy)
      for (int dx = -R[0]; dx <= R[0]; ++dx) {
        const double w = f->r - std::sqrt((double)(dx * dx + dy * dy + dz * dz));
        if (w > 0) taps.push_back(Tap{w, (dz * sy + dy) * sx + dx, 0});
      }
  f->nt = (int)taps.size();
  f->taps.alloc(taps.size() * sizeof(Tap));
  FDTD_HIP(hipMemcpy(f->taps.p, taps.data(), taps.size() * sizeof(Tap), hipMemcpyHostToDevice));
}

}  // namespace

extern "C" {

const char *fdtd_design_last_error(void) { return g_err.c_str(); }

fdtd_status fdtd_filter_create(const int32_t n[3], double radius, int32_t precision, void *stream, fdtd_filter **out) {
  if (!out) return FDTD_EINVAL;
  *out = nullptr;
  auto f = new fdtd_filter();
  const fdtd_status st = dguard([&] {
    if (!n || n[0] < 1 || n[1] < 1 || n[2] < 1) throw Error{FDTD_EINVAL, "filter box must have positive size"};
    if (!(radius > 0) || radius > 16) throw Error{FDTD_EINVAL, "filter radius must lie in (0, 16] cells"};
    if (precision != 32 && precision != 64) throw Error{FDTD_EINVAL, "precision must be 32 or 64"};
    f->nx = n[0]; f->ny = n[1]; f->nz = n[2];
    f->n = (int64_t)n[0] * n[1] * n[2];
    f->prec = precision;
    f->r = radius;
    f->R = (int)std::ceil(radius);
    f->Rz = f->nz > 1 ? f->R : 0;
    f->s = own_or(stream, f->own);
    const size_t es = precision == 32 ? 4 : 8;
    f->winv.alloc(f->n * sizeof(double));
    for (auto &x : f->xs) x.alloc(f->n * es);
    f->h.alloc(f->n * sizeof(double));
    for (auto &x : f->g) x.alloc(f->n * sizeof(double));
    filter_route(f);
    hipLaunchKernelGGL(winv_kernel, dim3(nblocks(f->n)), dim3(BS), 0, f->s, f->winv.as<double>(), f->nx, f->ny, f->nz,
                       f->r, f->R, f->Rz);
    FDTD_HIP(hipGetLastError());
    FDTD_HIP(hipStreamSynchronize(f->s));
  });
  if (st != FDTD_OK) {
    delete f;
    return st;
  }
  *out = f;
  return FDTD_OK;
}

fdtd_status fdtd_filter_apply(fdtd_filter *f, const void *rho, void *rho_f, double alpha) {
  if (!f) return FDTD_EINVAL;
  return dguard([&] {
    if (!rho || !rho_f) throw Error{FDTD_EINVAL, "null filter buffer"};
    if (!(alpha > 0)) throw Error{FDTD_EINVAL, "filter alpha must be > 0"};
    if (f->prec == 32) filter_apply<float>(f, rho, rho_f, alpha); else filter_apply<double>(f, rho, rho_f, alpha);
    f->alpha = alpha;
    f->applied = true;
  });
}

fdtd_status fdtd_filter_transpose(fdtd_filter *f, const void *g_f, void *g) {
  if (!f) return FDTD_EINVAL;
  return dguard([&] {
    if (!f->applied) throw Error{FDTD_ESTATE, "filter transpose before apply"};
    if (!g_f || !g) throw Error{FDTD_EINVAL, "null filter buffer"};
    if (f->prec == 32) filter_transpose<float>(f, g_f, g); else filter_transpose<double>(f, g_f, g);
  });
}

fdtd_status fdtd_filter_destroy(fdtd_filter *f) {
  delete f;
  return FDTD_OK;
}

fdtd_status fdtd_mma_create(int64_t n, int32_t precision, double xmin, double xmax, double move, double asyinit,
                            double asyincr, double asydecr, void *stream, fdtd_mma **out) {
  if (!out) return FDTD_EINVAL;
  *out = nullptr;
  auto m = new fdtd_mma();
  const fdtd_status st = dguard([&] {
    if (n < 1) throw Error{FDTD_EINVAL, "mma needs n >= 1"};
    if (precision != 32 && precision != 64) throw Error{FDTD_EINVAL, "precision must be 32 or 64"};
    if (!(xmax > xmin) || !(move > 0) || !(asyinit > 0) || !(asyincr >= 1) || !(asydecr > 0 && asydecr <= 1))
      throw Error{FDTD_EINVAL, "invalid mma parameters"};
    m->n = n;
    m->prec = precision;
    m->a = MmaArgs{xmin, xmax, move, asyinit, asyincr, asydecr};
    m->s = own_or(stream, m->own);
    for (DevBuf *b : {&m->x, &m->df, &m->xo1, &m->xo2, &m->L, &m->U, &m->lo, &m->hi}) b->alloc(n * sizeof(double));
    m->red.alloc();
  });
  if (st != FDTD_OK) {
    delete m;
    return st;
  }
  *out = m;
  return FDTD_OK;
}

fdtd_status fdtd_mma_begin(fdtd_mma *m, const void *x, double f0, const void *df0, double *rho0) {
  if (!m) return FDTD_EINVAL;
  return dguard([&] {
    if (!x || !df0) throw Error{FDTD_EINVAL, "null mma buffer"};
    const int nb = rblocks(m->n);
    if (m->prec == 32)
      hipLaunchKernelGGL(mma_begin_kernel<float>, dim3(nb), dim3(rthreads(m->n)), 0, m->s, (const float *)x, (const float *)df0,
                         m->n, m->k, m->a, m->x.as<double>(), m->df.as<double>(), m->xo1.as<double>(),
                         m->xo2.as<double>(), m->L.as<double>(), m->U.as<double>(), m->lo.as<double>(),
                         m->hi.as<double>(), m->red.part.as<double>(), m->red.count.as<unsigned>(), m->red.sums);
    else
      hipLaunchKernelGGL(mma_begin_kernel<double>, dim3(nb), dim3(rthreads(m->n)), 0, m->s, (const double *)x, (const double *)df0,
                         m->n, m->k, m->a, m->x.as<double>(), m->df.as<double>(), m->xo1.as<double>(),
                         m->xo2.as<double>(), m->L.as<double>(), m->U.as<double>(), m->lo.as<double>(),
                         m->hi.as<double>(), m->red.part.as<double>(), m->red.count.as<unsigned>(), m->red.sums);
    FDTD_HIP(hipGetLastError());
    FDTD_HIP(hipStreamSynchronize(m->s));
    const double sum = m->red.sums[0];
    m->f0 = f0;
    m->begun = true;
    if (rho0) *rho0 = std::max(1e-6, 0.1 * sum / (double)m->n);
  });
}

fdtd_status fdtd_mma_solve(fdtd_mma *m, double rho, void *xnew, double *approx, double *dist) {
  if (!m) return FDTD_EINVAL;
  return dguard([&] {
    if (!m->begun) throw Error{FDTD_ESTATE, "mma solve before begin"};
    if (!xnew) throw Error{FDTD_EINVAL, "null mma buffer"};
    if (!(rho >= 0)) throw Error{FDTD_EINVAL, "mma rho must be >= 0"};
    const int nb = rblocks(m->n);
    if (m->prec == 32)
      hipLaunchKernelGGL(mma_solve_kernel<float>, dim3(nb), dim3(rthreads(m->n)), 0, m->s, m->x.as<double>(), m->df.as<double>(),
                         m->L.as<double>(), m->U.as<double>(), m->lo.as<double>(), m->hi.as<double>(), m->n, rho, m->a,
                         (float *)xnew, m->red.part.as<double>(), m->red.count.as<unsigned>(), m->red.sums);
    else
      hipLaunchKernelGGL(mma_solve_kernel<double>, dim3(nb), dim3(rthreads(m->n)), 0, m->s, m->x.as<double>(), m->df.as<double>(),
                         m->L.as<double>(), m->U.as<double>(), m->lo.as<double>(), m->hi.as<double>(), m->n, rho, m->a,
                         (double *)xnew, m->red.part.as<double>(), m->red.count.as<unsigned>(), m->red.sums);
    FDTD_HIP(hipGetLastError());
    FDTD_HIP(hipStreamSynchronize(m->s));
    const double *t = m->red.sums;
    if (approx) *approx = m->f0 + t[0];
    if (dist) *dist = t[1];
  });
}

fdtd_status fdtd_mma_accept(fdtd_mma *m, const void *xnew) {
  if (!m) return FDTD_EINVAL;
  return dguard([&] {
    if (!m->begun) throw Error{FDTD_ESTATE, "mma accept before begin"};
    if (!xnew) throw Error{FDTD_EINVAL, "null mma buffer"};
    const int nb = nblocks(m->n);
    if (m->prec == 32)
      hipLaunchKernelGGL(mma_accept_kernel<float>, dim3(nb), dim3(BS), 0, m->s, (const float *)xnew, m->n,
                         m->x.as<double>(), m->xo1.as<double>(), m->xo2.as<double>());
    else
      hipLaunchKernelGGL(mma_accept_kernel<double>, dim3(nb), dim3(BS), 0, m->s, (const double *)xnew, m->n,
                         m->x.as<double>(), m->xo1.as<double>(), m->xo2.as<double>());
    FDTD_HIP(hipGetLastError());
    FDTD_HIP(hipStreamSynchronize(m->s));
    m->k += 1;
    m->begun = false;
  });
}

fdtd_status fdtd_mma_destroy(fdtd_mma *m) {
  delete m;
  return FDTD_OK;
}

fdtd_status fdtd_design_stats(int64_t n, int32_t precision, const void *x, const void *g, double xmin, double xmax,
                              void *stream, double out[2]) {
  return dguard([&] {
    if (n < 1 || !x || !out) throw Error{FDTD_EINVAL, "design stats need n >= 1, x and out"};
    if (precision != 32 && precision != 64) throw Error{FDTD_EINVAL, "precision must be 32 or 64"};
    bool own = false;
    hipStream_t s = own_or(stream, own);
    const int nb = rblocks(n);
    Reduction &red = stats_work();
    if (precision == 32)
      hipLaunchKernelGGL(stats_kernel<float>, dim3(nb), dim3(rthreads(n)), 0, s, (const float *)x, (const float *)g, n, xmin,
                         xmax, red.part.as<double>(), red.count.as<unsigned>(), red.sums);
    else
      hipLaunchKernelGGL(stats_kernel<double>, dim3(nb), dim3(rthreads(n)), 0, s, (const double *)x, (const double *)g, n, xmin,
                         xmax, red.part.as<double>(), red.count.as<unsigned>(), red.sums);
    FDTD_HIP(hipGetLastError());
    FDTD_HIP(hipStreamSynchronize(s));
    out[0] = red.sums[0] / (double)n;
    out[1] = std::sqrt(red.sums[1]);
    if (own) (void)hipStreamDestroy(s);
  });
}

}  // extern "C"
