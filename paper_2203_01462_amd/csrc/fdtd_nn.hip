// fdtd_nn.hip -- kernels of the surrogate network: 3x3 convolutions as
// implicit GEMMs on the BF16 matrix cores (v_mfma_f32_16x16x16_bf16, FP32
// accumulation), their data and weight gradients, and the elementwise,
// pooling, head, loss and optimizer kernels around them.
//
// GEMM tiling: a workgroup (4 wavefronts) owns a 64 x 64 output tile and
// walks the reduction dimension in steps of 16, staging both operand tiles
// in LDS (the im2col gather of the 3x3 window happens while staging); each
// wavefront owns 16 output rows and issues four 16x16x16 MFMAs per step.
// MFMA operand layout (wave64): lane l holds A[l%16][4(l/16)+j],
// B[4(l/16)+j][l%16] and returns D[4(l/16)+j][l%16], j = 0..3.
#include <cstdint>
#include <map>
#include <mutex>
#include <string>
#include <type_traits>

#include "fdtd_internal.hpp"
#include "fdtd_nn.h"

using namespace fdtd;

namespace {

typedef short s4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));

constexpr int BS = 256;
constexpr int TM = 64, TN = 64, TK = 16, PAD = 4;

// Workgroups go round-robin over the 8 XCDs, each with its own L2; neighbouring
// work items (tiles that share 128-byte lines of a row, output-channel blocks of
// one tile) belong on one XCD.  Item of workgroup b of a grid of xcd_grid(items):
// XCD b % 8 takes items (b % 8) * grid / 8 onwards, in order.
__device__ __forceinline__ int xcd_item(int b, int grid) { return (b & 7) * (grid >> 3) + (b >> 3); }
unsigned xcd_grid(int64_t items) { return (unsigned)((items + 7) / 8 * 8); }
// A launch takes fewer than 2^32 work items along an axis: so many workgroups of BS
// at most in such a grid.
constexpr int64_t MAX_XCD = ((int64_t)1 << 32) / BS - 8;

// IEEE binary32 -> bfloat16, round to nearest even (NaN kept quiet).
__device__ __forceinline__ uint16_t f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float bf2f(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

// The BF16 output of a convolution: relu(v) in the forward pass; with a mask
// (the BF16 output of the ReLU that produced this convolution's input, in a
// data-gradient pass) the pre-activation gradient v * (mask > 0), the same
// value as the separate ReLU backward of the FP32 v.
__device__ __forceinline__ uint16_t store_a(float v, const uint16_t *__restrict__ mask, size_t o) {
  return mask ? f2bf(bf2f(mask[o]) > 0.f ? v : 0.f) : f2bf(fmaxf(v, 0.f));
}

// Mask values of one 16-channel block of a tiled kernel's outputs: rows
// `row0 + s` (s < 4, pix0 = the first row's pixel offset) at the lane's
// column, channels co0 + 4 kq + j.
__device__ __forceinline__ void load_mask16(uint16_t (&mk)[4][4], int co0, int cout, int kq, size_t pix0, int w,
                                            size_t cs, const uint16_t *__restrict__ mask) {
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int co = co0 + 4 * kq + j;
      mk[s][j] = co < cout ? mask[(size_t)co * cs + pix0 + (size_t)s * w] : (uint16_t)0;
    }
}

// Output of that block: z = v (FP32) and/or a = relu(v) (BF16), or with a
// mask (mk loaded by load_mask16) a = v * (mask > 0) (BF16).  The values are
// formed first and stored back to back (a store between loads and arithmetic
// that reuse its registers would wait for it to complete).
__device__ __forceinline__ void tile_out16(const f4 (&acc)[4], const uint16_t (&mk)[4][4], bool masked, int co0,
                                           int cout, int kq, size_t pix0, int w, size_t cs,
                                           const float *__restrict__ bias, float *__restrict__ z,
                                           uint16_t *__restrict__ a) {
  // the lane's four biases, loaded together ahead of the stores
  float bv[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) bv[j] = (bias && co0 + 4 * kq + j < cout) ? bias[co0 + 4 * kq + j] : 0.f;
  float v[4][4];
  uint16_t b[4][4];
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      v[s][j] = acc[s][j] + bv[j];
      b[s][j] = masked ? f2bf(bf2f(mk[s][j]) > 0.f ? v[s][j] : 0.f) : f2bf(fmaxf(v[s][j], 0.f));
    }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int co = co0 + 4 * kq + j;
    if (co >= cout) continue;
    const size_t o = (size_t)co * cs + pix0;
    if (z) {
#pragma unroll
      for (int s = 0; s < 4; ++s) z[o + (size_t)s * w] = v[s][j];
    }
    if (a) {
#pragma unroll
      for (int s = 0; s < 4; ++s) a[o + (size_t)s * w] = b[s][j];
    }
  }
}

// Elements xs .. xs + 7 (xs >= 0) of a row of w elements at any address, zero beyond
// the row: one 16-byte load (the type says 2-byte alignment) that starts early
// enough to end inside the row (raw8), shifted down when it is used (cut8); rows
// of less than 8 element by element.  row must be readable also where the caller
// discards the result.
__device__ __forceinline__ uint4 raw8(const uint16_t *row, int xs, int w) {
  struct __attribute__((packed, aligned(2))) V {
    uint32_t v[4];
  };
  if (w >= 8) {
    const V v = *(const V *)(row + min(xs, w - 8));
    return uint4{v.v[0], v.v[1], v.v[2], v.v[3]};
  }
  uint32_t e[8];
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    e[q] = row[min(xs + q, w - 1)];
    if (xs + q >= w) e[q] = 0u;
  }
  return uint4{e[0] | (e[1] << 16), e[2] | (e[3] << 16), e[4] | (e[5] << 16), e[6] | (e[7] << 16)};
}
__device__ __forceinline__ uint4 cut8(uint4 v, int xs, int w, bool ok) {
  const int past = w >= 8 ? min(max(xs - (w - 8), 0), 8) : 0;  // elements to drop
  uint64_t lo = (uint64_t)v.x | ((uint64_t)v.y << 32), hi = (uint64_t)v.z | ((uint64_t)v.w << 32);
  if (past >= 4) {
    lo = hi;
    hi = 0;
  }
  const int d = 16 * (past & 3);
  lo = (lo >> d) | ((hi << 1) << (63 - d));
  hi >>= d;
  if (!ok || past == 8) lo = hi = 0;
  return uint4{(uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32)};
}

__device__ __forceinline__ double block_sum(double v, double *lds) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
  if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = v;
  __syncthreads();
  double s = 0;
  if (threadIdx.x == 0)
    for (int k = 0; k < BS / 64; ++k) s += lds[k];
  __syncthreads();
  return s;
}

// One 16-step of the K loop: wavefront `wave` multiplies its 16 rows of As
// with the four 16-column blocks of Bs.
__device__ __forceinline__ void mfma_step(const uint16_t (*As)[TK + PAD], const uint16_t (*Bs)[TN + PAD], int wave,
                                          int lane, f4 acc[4]) {
  s4 a;
#pragma unroll
  for (int j = 0; j < 4; ++j) a[j] = (short)As[16 * wave + (lane & 15)][4 * (lane >> 4) + j];
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    s4 b;
#pragma unroll
    for (int j = 0; j < 4; ++j) b[j] = (short)Bs[4 * (lane >> 4) + j][16 * s + (lane & 15)];
    acc[s] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, acc[s], 0, 0, 0);
  }
}

// z[co][n][p] = bias[co] + sum_k w[co][k] xhat[k][n][p], k = (ky, kx, ci),
// xhat = the zero-padded 3x3 window of x[ci][n].  Writes z (FP32) and/or
// a = bf16(max(z, 0)).  grid (ceil(HW/64), ceil(cout/64), n).
__global__ void __launch_bounds__(BS) conv_fwd_kernel(int cin, int cout, int h, int w, const uint16_t *__restrict__ x,
                                                     const uint16_t *__restrict__ wt, const float *__restrict__ bias,
                                                     float *__restrict__ z, uint16_t *__restrict__ a,
                                                     const uint16_t *__restrict__ mask) {
  __shared__ uint16_t As[TM][TK + PAD];
  __shared__ uint16_t Bs[TK][TN + PAD];
  const int n = blockIdx.z, nimg = gridDim.z, HW = h * w, K = cin * 9;
  const int p0 = blockIdx.x * TN, co0 = blockIdx.y * TM;
  const int t = threadIdx.x, wave = t >> 6, lane = t & 63;
  const size_t cs = (size_t)nimg * HW;  // channel stride
  const uint16_t *xn = x + (size_t)n * HW;
  f4 acc[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) acc[s] = f4{0.f, 0.f, 0.f, 0.f};
  for (int k0 = 0; k0 < K; k0 += TK) {
    {
      const int r = t >> 2, c = (t & 3) * 4, co = co0 + r;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int k = k0 + c + j;
        As[r][c + j] = (co < cout && k < K) ? wt[(size_t)co * K + k] : (uint16_t)0;
      }
    }
    {
      const int kk = t >> 4, c = (t & 15) * 4, k = k0 + kk;
      const int tap = k / cin, ci = k - tap * cin, ky = tap / 3, kx = tap - ky * 3;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int p = p0 + c + j;
        uint16_t v = 0;
        if (k < K && p < HW) {
          const int y = p / w, xx = p - y * w, iy = y + ky - 1, ix = xx + kx - 1;
          if (iy >= 0 && iy < h && ix >= 0 && ix < w) v = xn[(size_t)ci * cs + iy * w + ix];
        }
        Bs[kk][c + j] = v;
      }
    }
    __syncthreads();
    mfma_step(As, Bs, wave, lane, acc);
    __syncthreads();
  }
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int co = co0 + 16 * wave + 4 * (lane >> 4) + j, p = p0 + 16 * s + (lane & 15);
      if (co < cout && p < HW) {
        const float v = acc[s][j] + (bias ? bias[co] : 0.f);
        const size_t o = (size_t)co * cs + (size_t)n * HW + p;
        if (z) z[o] = v;
        if (a) a[o] = store_a(v, mask, o);
      }
    }
}

// The same convolution, LDS-tiled for cin % 32 == 0, h, w multiples of 16 and
// 16-byte aligned weights (ODD: x at any address, the same bits), on v_mfma_f32_16x16x32_bf16.  A workgroup owns
// 32 output channels x 16 x 16 pixels of one image; per chunk of 32 input
// channels it stages the 18 x 18 halo tile channel-last in LDS (eight channels of
// one pixel are one 16-byte LDS read) and the weights of all nine taps, then each
// wavefront (four pixel rows) runs nine taps x 2 x 4 matrix instructions.  What
// bounds it is the wait for the staged data: all of a chunk's loads are issued
// together, the next chunk's before the current one's matrix instructions.  A
// thread loads a halo row of two channels (the channel pairs of a row on
// neighbouring lanes: their LDS writes fall into one pixel's row); the last two
// rows, which 256 threads leave over, go by 16-byte pieces.  One chunk (ONE) holds
// 96 registers instead of 198: three workgroups a CU.  32 images of 128^2:
// 32 -> 32 channels 40 us and 9 to 14 for a channel-last copy -> 28;
// 16^2, 256 -> 256 35 us and 5 -> 22 (blocks of 64 channels left half of the CUs
// idle there, and at 64^2, 64 -> 192 took 92 us against 70).
// One-dimensional grid of xcd_grid((h/16) * (w/16) * ceil(cout / 32) * n).
constexpr int CC = 32;                  // input channels per chunk
constexpr int MT = 2;                   // output channels of a workgroup / 16
constexpr int XST = 40;                 // LDS stride between staged pixels (80 B: conflict-free 16 B reads)
constexpr int WST = 40;                 // LDS stride between staged (tap, co) weight rows
constexpr int TT = 16, HT = TT + 2;     // output tile side, halo tile side

// Elements sh (0 .. 7) onwards of u, two a word.
template <int N>
__device__ __forceinline__ void shift_down(uint32_t (&u)[N], int sh) {
  const uint32_t two = sh & 4 ? ~0u : 0u, one = sh & 2 ? ~0u : 0u;
#pragma unroll
  for (int k = 0; k + 2 < N; ++k) u[k] ^= (u[k] ^ u[k + 2]) & two;
#pragma unroll
  for (int k = 0; k + 1 < N; ++k) u[k] ^= (u[k] ^ u[k + 1]) & one;
#pragma unroll
  for (int k = 0; k + 1 < N; ++k) u[k] = __builtin_amdgcn_alignbit(u[k + 1], u[k], 16 * (sh & 1));
}

template <bool ONE, bool ODD>
__global__ void __launch_bounds__(BS) conv_fwd_mfma_kernel(int cin, int cout, int h, int w,
                                                               const uint16_t *__restrict__ x,
                                                               const uint16_t *__restrict__ wt,
                                                               const float *__restrict__ bias,
                                                               float *__restrict__ z, uint16_t *__restrict__ a,
                                                               const uint16_t *__restrict__ mask, const int nimg) {
  __shared__ __attribute__((aligned(16))) uint16_t Xs[HT * HT * XST];
  __shared__ __attribute__((aligned(16))) uint16_t Ws[9 * 16 * MT * WST];
  constexpr int NWV = (9 * 16 * MT * 4 + BS - 1) / BS;   // 16-byte weight vectors per thread
  const int HW = h * w;
  const int tilesx = w / TT, tiles = (h / TT) * tilesx, cot = (cout + 16 * MT - 1) / (16 * MT);
  const int item = xcd_item(blockIdx.x, gridDim.x), n = item / (cot * tiles);
  if (n >= nimg) return;
  const int tile = item / cot % tiles, steps = ONE ? 1 : cin / CC;
  const int co0 = item % cot * 16 * MT;
  const int t = threadIdx.x, wave = t >> 6, lane = t & 63, l16 = lane & 15, kq = lane >> 4;
  const size_t cs = (size_t)nimg * HW;
  // x off a 16-byte address by sh elements, the same for every row (w is a multiple of
  // 16): aligned vectors, each with an element of the row in it, shifted when they
  // are used
  constexpr int NV = ODD ? 3 : 2;
  const int sh = ODD ? __builtin_amdgcn_readfirstlane((int)((uintptr_t)x >> 1) & 7) : 0;
  uint4 xv[2 * NV], xt[2] = {}, wr[NWV];
  uint32_t xe[4], te2 = 0;  // halo columns
  // rows 0 .. 15: channels c, c + 1 of row r; rows 16, 17: 8 pixels of channel tc
  const int c = 2 * (t & 15), r = t >> 4, tc = (t >> 1) & 31, tr = 16 + (t >> 6), th = t & 1;
  int lx0 = 0, ly0 = 0;  // the loaded tile's origin
  // global -> registers for the chunk at channel c0; registers -> LDS after the barrier
  auto load_x = [&](int c0) {
    ly0 = (tile / tilesx) * TT;
    lx0 = (tile % tilesx) * TT;
    const int xl = max(lx0 - 1, 0), xr = min(lx0 + TT, w - 1);
    const uint16_t *r0 = x + (size_t)(c0 + c) * cs + (size_t)n * HW + (size_t)max(ly0 - 1 + r, 0) * w;
    const uint16_t *r1 = r0 + cs;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      xv[k] = *(const uint4 *)(r0 - sh + lx0 + 8 * k);
      xv[NV + k] = *(const uint4 *)(r1 - sh + lx0 + 8 * k);
    }
    xe[0] = r0[xl];
    xe[1] = r1[xl];
    xe[2] = r0[xr];
    xe[3] = r1[xr];
    if (t < 128) {
      const uint16_t *rt = x + (size_t)(c0 + tc) * cs + (size_t)n * HW + (size_t)min(ly0 - 1 + tr, h - 1) * w;
      xt[0] = *(const uint4 *)(rt - sh + lx0 + 8 * th);
      if (ODD) xt[1] = *(const uint4 *)(rt - sh + lx0 + 8 * th + 8);
      te2 = rt[th ? xr : xl];
    }
  };
  auto store_x = [&]() {
    const bool ok = ly0 - 1 + r >= 0, left = lx0 > 0, right = lx0 + TT < w;
    uint32_t u0[4 * NV], u1[4 * NV];
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      u0[4 * k] = xv[k].x; u0[4 * k + 1] = xv[k].y; u0[4 * k + 2] = xv[k].z; u0[4 * k + 3] = xv[k].w;
      u1[4 * k] = xv[NV + k].x; u1[4 * k + 1] = xv[NV + k].y; u1[4 * k + 2] = xv[NV + k].z; u1[4 * k + 3] = xv[NV + k].w;
    }
    if constexpr (ODD) {
      shift_down(u0, sh);
      shift_down(u1, sh);
    }
    uint16_t *d = Xs + r * HT * XST + c;
    *(uint32_t *)d = ok && left ? xe[0] | (xe[1] << 16) : 0u;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      *(uint32_t *)(d + (2 * q + 1) * XST) = ok ? (u0[q] & 0xffffu) | (u1[q] << 16) : 0u;
      *(uint32_t *)(d + (2 * q + 2) * XST) = ok ? (u0[q] >> 16) | (u1[q] & 0xffff0000u) : 0u;
    }
    *(uint32_t *)(d + (TT + 1) * XST) = ok && right ? xe[2] | (xe[3] << 16) : 0u;
    if (t < 128) {
      const bool okt = ly0 - 1 + tr < h;
      uint16_t *p = Xs + (tr * HT + 8 * th + 1) * XST + tc;
      uint32_t v[8] = {xt[0].x, xt[0].y, xt[0].z, xt[0].w, xt[1].x, xt[1].y, xt[1].z, xt[1].w};
      if constexpr (ODD) shift_down(v, sh);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        p[2 * q * XST] = okt ? (uint16_t)v[q] : (uint16_t)0;
        p[(2 * q + 1) * XST] = okt ? (uint16_t)(v[q] >> 16) : (uint16_t)0;
      }
      Xs[(tr * HT + (th ? TT + 1 : 0)) * XST + tc] = okt && (th ? right : left) ? (uint16_t)te2 : (uint16_t)0;
    }
  };
  auto load_w = [&](int c0) {
#pragma unroll
    for (int k = 0; k < NWV; ++k) {
      const int v = t + k * BS;
      const int part = v & 3, row = v >> 2;
      const int tap = row / (16 * MT), col = row - tap * (16 * MT), co = co0 + col;
      wr[k] = uint4{0u, 0u, 0u, 0u};
      if (v < 9 * 16 * MT * 4 && co < cout) wr[k] = *(const uint4 *)(wt + ((size_t)co * 9 + tap) * cin + c0 + 8 * part);
    }
  };
  auto store_w = [&]() {
#pragma unroll
    for (int k = 0; k < NWV; ++k) {
      const int v = t + k * BS;
      if (v < 9 * 16 * MT * 4) *(uint4 *)(Ws + (v >> 2) * WST + 8 * (v & 3)) = wr[k];
    }
  };
  f4 acc[MT][4];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int s = 0; s < 4; ++s) acc[m][s] = f4{0.f, 0.f, 0.f, 0.f};
  load_w(0);
  load_x(0);
  const bool masked = a && mask;
  const size_t pix0 = (size_t)n * HW + (size_t)((tile / tilesx) * TT + 4 * wave) * w + (tile % tilesx) * TT + l16;
  uint16_t mk[2][4][4];
  for (int st = 0; st < steps; ++st) {
    store_w();
    store_x();
    __syncthreads();
    if (st + 1 < steps) {  // the next chunk's loads fly while the matrix cores work
      load_w((st + 1) * CC);
      load_x((st + 1) * CC);
    } else if (masked) {   // a data-gradient pass's mask values, ahead of the stores
      load_mask16(mk[0], co0, cout, kq, pix0, w, cs, mask);
    }
#pragma unroll
    for (int tap = 0; tap < 9; ++tap) {
      const int ky = tap / 3, kx = tap - 3 * ky;
      bf8 av[MT], bv[4];
#pragma unroll
      for (int m = 0; m < MT; ++m) av[m] = *(const bf8 *)(Ws + (tap * 16 * MT + 16 * m + l16) * WST + 8 * kq);
#pragma unroll
      for (int s = 0; s < 4; ++s) bv[s] = *(const bf8 *)(Xs + ((4 * wave + s + ky) * HT + l16 + kx) * XST + 8 * kq);
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int s = 0; s < 4; ++s) acc[m][s] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[m], bv[s], acc[m][s], 0, 0, 0);
    }
    if (st + 1 < steps) __syncthreads();
  }
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    if (masked && m + 1 < MT) load_mask16(mk[(m + 1) & 1], co0 + 16 * (m + 1), cout, kq, pix0, w, cs, mask);
    tile_out16(acc[m], mk[m & 1], masked, co0 + 16 * m, cout, kq, pix0, w, cs, bias, z, a);
  }
}

// The convolution for any shape with at most CP <= 384 input channels (padded to a
// multiple of 16): a workgroup owns 64 output channels x 8 x 8 pixels, stages the
// 10 x 10 halo with all its channels once (channel-last, zeros outside the image
// and beyond cin), and its wavefronts walk k = (tap, channel) in steps of 16 as
// conv_fwd_kernel does - the same matrix instructions in the same order, so for
// cin % 16 == 0 the same bits - with the weights' fragments read ahead from
// global memory.  That kernel's time is its staging (an index division and a
// 2-byte load per element and tap), which it is still the better one for where this
// one would pad much (conv_packs).  4 x 48 x 50 x 75 -> 80 channels:
// 62 us -> 15.5.
constexpr int GT = 8, GH = GT + 2, AHEAD = 9;  // 9 divides the steps

template <int CP, bool VEC>
__global__ void __launch_bounds__(BS) conv_gen_kernel(int cin, int cout, int h, int w, const uint16_t *__restrict__ x,
                                                     const uint16_t *__restrict__ wt, const float *__restrict__ bias,
                                                     float *__restrict__ z, uint16_t *__restrict__ a,
                                                     const uint16_t *__restrict__ mask, int nimg) {
  constexpr int S = CP + 4;  // LDS stride between pixels
  __shared__ __attribute__((aligned(16))) uint16_t Xs[GH * GH * S];
  const int HW = h * w, K = cin * 9;
  const int tilesx = (w + GT - 1) / GT, tiles = tilesx * ((h + GT - 1) / GT), cot = (cout + TM - 1) / TM;
  const int item = xcd_item(blockIdx.x, gridDim.x), n = item / (cot * tiles), tile = item / cot % tiles;
  if (n >= nimg) return;
  const int y0 = (tile / tilesx) * GT, x0 = (tile % tilesx) * GT, co0 = item % cot * TM;
  const int t = threadIdx.x, wave = t >> 6, lane = t & 63, l16 = lane & 15, kq = lane >> 4;
  const size_t cs = (size_t)nimg * HW;
  const uint16_t *xn = x + (size_t)n * HW;
  const int steps = (cin + 15) >> 4;  // a tap
  // the lane's row of weights: channels 16 st + 4 kq .. + 3 of a tap, read where
  // they are (or, past the last channel, from inside the row) AHEAD steps before
  // they are used, zeroed past the last channel when they are used
  const uint16_t *wr = wt + (size_t)min(co0 + 16 * wave + l16, cout - 1) * K;
  auto load_a = [&](int tap, int st) {
    const int c = 16 * st + 4 * kq;
    if constexpr (VEC) {
      return *(const uint2 *)(wr + min(tap, 8) * cin + min(c, cin - 4));
    } else {
      uint32_t e[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) e[j] = wr[min(tap, 8) * cin + min(c + j, cin - 1)];
      return uint2{e[0] | (e[1] << 16), e[2] | (e[3] << 16)};
    }
  };
  auto use_a = [&](uint2 v, int st) {
    const int left = cin - (16 * st + 4 * kq);  // channels from here on
    v.x = left >= 2 ? v.x : left == 1 ? v.x & 0xffffu : 0u;
    v.y = left >= 4 ? v.y : left == 3 ? v.y & 0xffffu : 0u;
    return __builtin_bit_cast(s4, v);
  };
  uint2 ar[AHEAD];
  int ft = 0, fs = 0;  // the fragment to fetch next
#pragma unroll
  for (int u = 0; u < AHEAD; ++u) {
    ar[u] = load_a(ft, fs);
    if (++fs == steps) {
      fs = 0;
      ++ft;
    }
  }
  // the lane's outputs (channels co4 .. + 3 of four pixels), their biases and mask
  // values, read first: a load between the stores below would wait for them
  const int co4 = co0 + 16 * wave + 4 * kq;
  size_t pix[4];
  bool okp[4];
  float bv4[4];
  uint16_t mk[4][4];
#pragma unroll
  for (int j = 0; j < 4; ++j) bv4[j] = bias ? bias[min(co4 + j, cout - 1)] : 0.f;
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const int p = 16 * s + l16, y = y0 + (p >> 3), xx = x0 + (p & 7);
    okp[s] = y < h && xx < w;
    pix[s] = okp[s] ? (size_t)n * HW + (size_t)y * w + xx : 0;
    if (a && mask) {
#pragma unroll
      for (int j = 0; j < 4; ++j) mk[s][j] = mask[(size_t)min(co4 + j, cout - 1) * cs + pix[s]];
    }
  }
  // a halo row of two channels per thread and turn
  for (int e = t; e < GH * 8 * steps; e += BS) {
    const int c = 2 * (e / GH), r = e % GH, iy = y0 - 1 + r;
    const bool ok = iy >= 0 && iy < h;
    const uint16_t *r0 = xn + (size_t)min(c, cin - 1) * cs + (size_t)(ok ? iy : 0) * w;
    const uint16_t *r1 = xn + (size_t)min(c + 1, cin - 1) * cs + (size_t)(ok ? iy : 0) * w;
    uint4 v0 = raw8(r0, x0, w), v1 = raw8(r1, x0, w);
    const int xl = max(x0 - 1, 0), xr = min(x0 + GT, w - 1);
    const uint32_t l0 = r0[xl], l1 = r1[xl], e0 = r0[xr], e1 = r1[xr];
    v0 = cut8(v0, x0, w, true);
    v1 = cut8(v1, x0, w, true);
    const uint32_t m0 = ok && c < cin ? 0xffffu : 0u, m1 = ok && c + 1 < cin ? 0xffff0000u : 0u;
    uint16_t *d = Xs + r * GH * S + c;
    *(uint32_t *)d = x0 > 0 ? (l0 & m0) | ((l1 << 16) & m1) : 0u;
    const uint32_t u0[4] = {v0.x, v0.y, v0.z, v0.w}, u1[4] = {v1.x, v1.y, v1.z, v1.w};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      *(uint32_t *)(d + (2 * q + 1) * S) = (u0[q] & m0) | ((u1[q] << 16) & m1);
      *(uint32_t *)(d + (2 * q + 2) * S) = ((u0[q] >> 16) & m0) | (u1[q] & m1);
    }
    *(uint32_t *)(d + (GT + 1) * S) = x0 + GT < w ? (e0 & m0) | ((e1 << 16) & m1) : 0u;
  }
  __syncthreads();
  f4 acc[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) acc[s] = f4{0.f, 0.f, 0.f, 0.f};
  const uint16_t *xb[4];  // pixel 16 s + l16 of the tile
#pragma unroll
  for (int s = 0; s < 4; ++s) xb[s] = Xs + ((2 * s + (l16 >> 3)) * GH + (l16 & 7)) * S + 4 * kq;
  // the next step's pixels are read while this step multiplies
  uint2 bn[4];
  int st = 0, off = 0, kx = 0;
#pragma unroll
  for (int s = 0; s < 4; ++s) bn[s] = *(const uint2 *)xb[s];
  for (int it = 0; it < steps; ++it) {
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) {
      const s4 av = use_a(ar[u], st);
      uint2 b[4];
#pragma unroll
      for (int s = 0; s < 4; ++s) b[s] = bn[s];
      off += 16;
      if (++st == steps) {
        st = 0;
        off += S - 16 * steps;
        if (++kx == 3) {
          kx = 0;
          off += (GH - 3) * S;
        }
      }
      const int o = u == AHEAD - 1 && it == steps - 1 ? 0 : off;
#pragma unroll
      for (int s = 0; s < 4; ++s) bn[s] = *(const uint2 *)(xb[s] + o);
      ar[u] = load_a(ft, fs);
      if (++fs == steps) {
        fs = 0;
        ++ft;
      }
#pragma unroll
      for (int s = 0; s < 4; ++s)
        acc[s] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(av, __builtin_bit_cast(s4, b[s]), acc[s], 0, 0, 0);
    }
  }
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float v = acc[s][j] + bv4[j];
      if (!(okp[s] && co4 + j < cout)) continue;
      const size_t o = (size_t)(co4 + j) * cs + pix[s];
      if (z) z[o] = v;
      if (a) a[o] = mask ? f2bf(bf2f(mk[s][j]) > 0.f ? v : 0.f) : f2bf(fmaxf(v, 0.f));
    }
}

// The convolution of a one-channel input (cout <= 64): a workgroup of 64 x 4
// pixels stages its 66 x 6 input halo and the weights in LDS; each thread
// forms its pixel's cout outputs as FP32 sums over the taps in order (plus
// the bias), written as z and/or a (store_a).  grid (ceil(w/64), ceil(h/4), n).
__global__ void __launch_bounds__(BS) conv1_fwd_kernel(int cout, int h, int w, const uint16_t *__restrict__ x,
                                                      const uint16_t *__restrict__ wt, const float *__restrict__ bias,
                                                      float *__restrict__ z, uint16_t *__restrict__ a,
                                                      const uint16_t *__restrict__ mask) {
  __shared__ float xs[6][66];
  __shared__ float ws[64 * 9];
  const int n = blockIdx.z, nimg = gridDim.z, HW = h * w;
  const int x0 = blockIdx.x * 64, y0 = blockIdx.y * 4;
  const int t = threadIdx.x, lx = t & 63, ly = t >> 6;
  for (int i = t; i < 6 * 66; i += BS) {
    const int r = i / 66, q = i - r * 66, iy = y0 - 1 + r, ix = x0 - 1 + q;
    xs[r][q] = (iy >= 0 && iy < h && ix >= 0 && ix < w) ? bf2f(x[(size_t)n * HW + (size_t)iy * w + ix]) : 0.f;
  }
  for (int i = t; i < cout * 9; i += BS) ws[i] = bf2f(wt[i]);
  __syncthreads();
  const int xx = x0 + lx, yy = y0 + ly;
  if (xx >= w || yy >= h) return;
  float xn[9];
#pragma unroll
  for (int tp = 0; tp < 9; ++tp) xn[tp] = xs[ly + tp / 3][lx + tp % 3];
  const size_t cs = (size_t)nimg * HW, pix = (size_t)n * HW + (size_t)yy * w + xx;
  for (int co = 0; co < cout; ++co) {
    float v = 0.f;
#pragma unroll
    for (int tp = 0; tp < 9; ++tp) v = fmaf(ws[co * 9 + tp], xn[tp], v);
    v += bias ? bias[co] : 0.f;
    const size_t o = (size_t)co * cs + pix;
    if (z) z[o] = v;
    if (a) a[o] = store_a(v, mask, o);
  }
}

// Which of the two kernels for any shape?  conv_fwd_kernel packs the pixels of an
// image and the taps' channels: ceil(9 cin / 16) steps on ceil(hw / 64) blocks, each
// step staged element by element.  conv_gen_kernel pads both: nine times
// ceil(cin / 16) much cheaper steps, after a halo, on whole 8 x 8 tiles; channel
// counts that are no multiple of 4 load its weights element by element.  The costs
// below, in steps of the former, were fitted to 2011 measured layers (1 to 384
// channels, 1 to 192 out, images from one pixel over rows and columns to 333 x 517):
// the slower kernel is taken by more than 10% in 24 of them.  us, conv_fwd_kernel
// against conv_gen_kernel: 32 x (3 -> 16) x 127^2 35 / 55, 32 x (1 -> 128) x 50^2
// 16 / 33, 8 x (48 -> 80) x 4000 x 1 48 / 69; 4 x (48 -> 80) x 16^2 38 / 8.
bool conv_packs(int n, int cin, int cout, int h, int w) {
  if (cin > 384) return true;  // (its halo does not fit the LDS)
  const double images = (double)n * ((cout + TM - 1) / TM);
  const double packed = images * (((int64_t)h * w + TN - 1) / TN);
  const double tiled = images * ((h + GT - 1) / GT) * ((w + GT - 1) / GT);
  const int steps = (9 * cin + 15) / 16, padded = 9 * ((cin + 15) / 16);
  if (tiled > (double)MAX_XCD) return true;  // (more tiles than a one-dimensional grid takes)
  const double step = cin % 4 == 0 ? 0.115 : cout > 32 ? 0.4 : 0.21;
  return std::max(1.0, packed / 896) * (steps + 0.4) < std::max(1.0, tiled / 512) * (0.6 + step * padded);
}

// A copy of device memory that lives until the stream has used it.
struct StreamCopy {
  void *p = nullptr;
  hipStream_t s;
  StreamCopy(const void *src, size_t bytes, hipStream_t stream) : s(stream) {
    FDTD_HIP(hipMallocAsync(&p, bytes, s));
    const hipError_t e = hipMemcpyAsync(p, src, bytes, hipMemcpyDeviceToDevice, s);
    if (e != hipSuccess) {
      (void)hipFreeAsync(p, s);
      FDTD_HIP(e);
    }
  }
  StreamCopy(const StreamCopy &) = delete;
  StreamCopy &operator=(const StreamCopy &) = delete;
  ~StreamCopy() { (void)hipFreeAsync(p, s); }
};

bool overlap(const void *a, size_t na, const void *b, size_t nb) {
  return a && b && (uintptr_t)a < (uintptr_t)b + nb && (uintptr_t)b < (uintptr_t)a + na;
}

// One forward convolution launch: the LDS-tiled kernel where the shape and
// the weights' alignment allow it, else one of the two for any shape.
void launch_conv(int n, int cin, int cout, int h, int w, const uint16_t *x, const uint16_t *wt, const float *bias,
                 float *z, uint16_t *a, const uint16_t *mask, hipStream_t s) {
  if (cin == 1 && cout <= 64) {
    hipLaunchKernelGGL(conv1_fwd_kernel, dim3((w + 63) / 64, (h + 3) / 4, n), dim3(BS), 0, s, cout, h, w, x, wt, bias,
                       z, a, mask);
    return;
  }
  const int64_t items = (int64_t)(h / TT) * (w / TT) * ((cout + 16 * MT - 1) / (16 * MT)) * n;
  if (cin % CC == 0 && h % TT == 0 && w % TT == 0 && ((uintptr_t)wt & 15) == 0 && items <= MAX_XCD) {
    const dim3 g(xcd_grid(items));
    const bool odd = (uintptr_t)x & 15;
    const size_t nx = (size_t)cin * n * h * w, ny = (size_t)cout * n * h * w;
    // in place: neighbouring tiles still read what this one writes
    if (overlap(x, nx * sizeof(uint16_t), z, ny * sizeof(float)) ||
        overlap(x, nx * sizeof(uint16_t), a, ny * sizeof(uint16_t))) {
      const StreamCopy c(x, nx * sizeof(uint16_t), s);
      launch_conv(n, cin, cout, h, w, (const uint16_t *)c.p, wt, bias, z, a, mask, s);
      return;
    }
    auto *k = cin == CC ? (odd ? &conv_fwd_mfma_kernel<true, true> : &conv_fwd_mfma_kernel<true, false>)
                        : (odd ? &conv_fwd_mfma_kernel<false, true> : &conv_fwd_mfma_kernel<false, false>);
    hipLaunchKernelGGL(k, g, dim3(BS), 0, s, cin, cout, h, w, x, wt, bias, z, a, mask, n);
    return;
  }
  if (!conv_packs(n, cin, cout, h, w)) {
    const dim3 g(xcd_grid((int64_t)((h + GT - 1) / GT) * ((w + GT - 1) / GT) * ((cout + TM - 1) / TM) * n));
    auto pick = [&](auto vec) {
      constexpr bool V = decltype(vec)::value;
      return cin <= 64 ? &conv_gen_kernel<64, V> : cin <= 128 ? &conv_gen_kernel<128, V>
             : cin <= 256 ? &conv_gen_kernel<256, V> : &conv_gen_kernel<384, V>;
    };
    auto *k = cin % 4 == 0 && ((uintptr_t)wt & 7) == 0 ? pick(std::true_type()) : pick(std::false_type());
    hipLaunchKernelGGL(k, g, dim3(BS), 0, s, cin, cout, h, w, x, wt, bias, z, a, mask, n);
    return;
  }
  const dim3 g((h * w + TN - 1) / TN, (cout + TM - 1) / TM, n);
  hipLaunchKernelGGL(conv_fwd_kernel, g, dim3(BS), 0, s, cin, cout, h, w, x, wt, bias, z, a, mask);
}

// Partial weight gradients over one range of pixels q = (n, p) of the batch:
// part[split][co][k] = sum_q dz[co][q] xhat[k][q], and with bpart the bias sums
// bpart[split][co] = sum_q dz[co][q].  For images that would fill less than a
// quarter of the 8 x 16-pixel tiles of the kernel below: here the pixels of all
// images follow one another, at an index division per element.  us with / without
// (64 -> 64 channels): 4096 images of 1 x 1 34 / 1187, 1024 of 4 x 4 59 / 93, 512 of
// 5 x 5 51 / 69, 8 of 4000 x 1 76 / 242; the other way 512 of 6 x 6 62 / 57, of
// 7 x 7 73 / 54.  grid (ceil(K/64), ceil(cout/64), splits).
__global__ void __launch_bounds__(BS) conv_wgrad_kernel(int nimg, int cin, int cout, int h, int w,
                                                       const uint16_t *__restrict__ x, const uint16_t *__restrict__ dz,
                                                       float *__restrict__ part, int chunk,
                                                       double *__restrict__ bpart) {
  __shared__ uint16_t As[TM][TK + PAD];  // dz: co x q
  __shared__ uint16_t Bs[TK][TN + PAD];  // xhat: q x k
  const int HW = h * w, K = cin * 9;
  const int64_t P = (int64_t)nimg * HW;
  const int k0 = blockIdx.x * TN, co0 = blockIdx.y * TM, split = blockIdx.z;
  const int64_t qb = (int64_t)split * chunk, qe = min(P, qb + chunk);
  const int t = threadIdx.x, wave = t >> 6, lane = t & 63;
  f4 acc[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) acc[s] = f4{0.f, 0.f, 0.f, 0.f};
  const bool with_bias = bpart != nullptr && k0 == 0;
  double bsum = 0;
  for (int64_t q0 = qb; q0 < qe; q0 += TK) {
    {
      const int r = t >> 2, c = (t & 3) * 4, co = co0 + r;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int64_t q = q0 + c + j;
        As[r][c + j] = (co < cout && q < qe) ? dz[(size_t)co * P + q] : (uint16_t)0;
        if (with_bias) bsum += bf2f(As[r][c + j]);
      }
    }
    {
      const int qq = t >> 4, c = (t & 15) * 4;
      const int64_t q = q0 + qq;
      const bool qok = q < qe;
      const int64_t n = qok ? q / HW : 0;
      const int p = qok ? (int)(q - n * HW) : 0;
      const int y = p / w, xx = p - y * w;
      const uint16_t *xn = x + (size_t)n * HW;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int k = k0 + c + j;
        uint16_t v = 0;
        if (qok && k < K) {
          const int tap = k / cin, ci = k - tap * cin, ky = tap / 3, kx = tap - ky * 3;
          const int iy = y + ky - 1, ix = xx + kx - 1;
          if (iy >= 0 && iy < h && ix >= 0 && ix < w) v = xn[(size_t)ci * P + iy * w + ix];
        }
        Bs[qq][c + j] = v;
      }
    }
    __syncthreads();
    mfma_step(As, Bs, wave, lane, acc);
    __syncthreads();
  }
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int co = co0 + 16 * wave + 4 * (lane >> 4) + j, k = k0 + 16 * s + (lane & 15);
      if (co < cout && k < K) part[((size_t)split * cout + co) * K + k] = acc[s][j];
    }
  if (with_bias) {
    bsum += __shfl_xor(bsum, 1, 64);
    bsum += __shfl_xor(bsum, 2, 64);
    if ((t & 3) == 0 && co0 + (t >> 2) < cout) bpart[(size_t)split * cout + co0 + (t >> 2)] = bsum;
  }
}

// Weight gradient, LDS-tiled for cin % 32 == 0, h % 8 == 0, w % 16 == 0 and
// 16-byte aligned x and dz:
// part[split][co][tap][ci] = sum over the split's pixel tiles of
// dz[co][q] x[ci][q shifted by tap] (rows `stride` floats apart).  A
// workgroup owns CT (64 or 32) output channels x 32 input channels x 9 taps
// and walks 8 x 16 pixel tiles; the reduction runs over pixels (32 per
// matrix instruction), so both operands are staged pixel-contiguous: dz rows
// as they are, and the input tile three times, shifted by kx = 0, 1, 2, so
// every 16-byte fragment read stays aligned.  CT = 64: wavefront w owns
// output channels 16w..16w+15 and both 16-channel halves of the input chunk
// (2 x 9 accumulator tiles); CT = 32 (layers with at most 32 output
// channels): output channels 16(w & 1).. and input half w >> 1 (1 x 9).
// With bpart, the workgroups of the first input chunk also write the
// split's bias partial sums: the sum of dz[co][q] over its tiles, as float
// bpart[split * stride + co], with RAG as double bpart[split * cout + co].  One-dimensional grid of xcd_grid(ceil(cout/CT) * ceil(cin/32) *
// splits): with the items of neighbouring tiles on one XCD, 96 -> 32 channels on 32
// images of 128^2 takes 101 us (146 when they went round-robin), 64 -> 64 at 64^2
// 36 (46).
// RAG: any shape and alignment: tiles and channels may hang over (zeros there),
// rows are loaded by raw8, and the bias sums stay in FP64 until all of them are
// added.  The
// kernel it replaces formed an index by division per element and matrix step:
// 4 x (48 -> 80) x 50 x 75 46 us -> 19.
constexpr int GY = 8, GX = 16, GP = GY * GX;  // pixel tile
constexpr int DST = GP + 8;                   // LDS stride of staged dz rows
constexpr int XCI = (GY + 2) * GX + 8;        // LDS stride per input channel of a shifted copy

template <int CT, bool RAG>
__global__ void __launch_bounds__(BS) conv_wgrad_mfma_kernel(int nimg, int cin, int cout, int h, int w,
                                                            const uint16_t *__restrict__ x,
                                                            const uint16_t *__restrict__ dz,
                                                            float *__restrict__ part, int64_t stride,
                                                            int tiles_per_split, void *__restrict__ bpart,
                                                            int splits) {
  constexpr int NT = CT / 32;           // 16-channel input halves per wavefront
  constexpr int DV = CT * GY * 2 / BS;  // 16-byte dz vectors per thread and tile
  __shared__ __attribute__((aligned(16))) uint16_t Ds[CT * DST];
  __shared__ __attribute__((aligned(16))) uint16_t Xs[3 * 32 * XCI];
  const int HW = h * w;
  const size_t P = (size_t)nimg * HW;
  // items: output blocks fastest, then input chunks, then splits (neighbours read
  // the same tiles)
  const int gx = (cout + CT - 1) / CT, gy = (cin + 31) / 32, item = xcd_item(blockIdx.x, gridDim.x);
  const int co0 = item % gx * CT, ci0 = item / gx % gy * 32, split = item / (gx * gy);
  if (split >= splits) return;
  const int tx_n = (w + GX - 1) / GX, tiles_img = ((h + GY - 1) / GY) * tx_n, tiles = nimg * tiles_img;
  const int T0 = split * tiles_per_split, T1 = min(tiles, T0 + tiles_per_split);
  const int t = threadIdx.x, wave = t >> 6, lane = t & 63, l16 = lane & 15, kq = lane >> 4;
  const int cw = CT == 64 ? wave : (wave & 1), nb = CT == 64 ? 0 : (wave >> 1);
  const bool with_bias = bpart != nullptr && ci0 == 0;
  f4 acc[NT][9];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
#pragma unroll
    for (int tp = 0; tp < 9; ++tp) acc[nt][tp] = f4{0.f, 0.f, 0.f, 0.f};
  using B = std::conditional_t<RAG, double, float>;
  B bacc[DV];
#pragma unroll
  for (int k = 0; k < DV; ++k) bacc[k] = 0;
  // A tile's global loads, issued together into registers: the dz rows (CT
  // channels x 8 rows x 16 pixels as 16-byte vectors) and the input halo
  // rows y0-1 .. y0+8 of the 32 channels (one row per thread and pass: the
  // 16 interior pixels as two 16-byte vectors plus the two halo pixels).
  // The next tile's loads fly while the current tile's matrix instructions run.
  constexpr int XR = (32 * (GY + 2) + BS - 1) / BS;
  uint4 dv[DV], xa[XR], xb[XR];
  uint32_t xl[XR], xr[XR];
  bool okd[DV], okx[XR];  // RAG: the row exists; the loaded rows are cut when they are stored
  int cx0 = 0, cy0 = 0;
  auto load_tile = [&](int T) {
    const int n = T / tiles_img, rem = T - n * tiles_img;
    const int y0 = (rem / tx_n) * GY, x0 = (rem % tx_n) * GX;
    cx0 = x0;
    cy0 = y0;
#pragma unroll
    for (int k = 0; k < DV; ++k) {
      const int v = t + k * BS;
      const int half = v & 1, r = (v >> 1) & (GY - 1), co = co0 + (v >> 4);
      dv[k] = uint4{0u, 0u, 0u, 0u};
      if constexpr (RAG) {
        const bool ok = co < cout && y0 + r < h;
        const uint16_t *row = dz + (ok ? (size_t)co * P + (size_t)n * HW + (size_t)(y0 + r) * w : 0);
        dv[k] = raw8(row, x0 + 8 * half, w);
        okd[k] = ok;
      } else if (co < cout) dv[k] = *(const uint4 *)(dz + (size_t)co * P + (size_t)n * HW + (size_t)(y0 + r) * w + x0 + 8 * half);
    }
#pragma unroll
    for (int q = 0; q < XR; ++q) {
      const int rr = t + q * BS;
      xa[q] = xb[q] = uint4{0u, 0u, 0u, 0u};
      xl[q] = xr[q] = 0u;
      const int c = rr / (GY + 2), r = rr - c * (GY + 2), iy = y0 - 1 + r;
      if constexpr (RAG) {
        const bool ok = rr < 32 * (GY + 2) && ci0 + c < cin && iy >= 0 && iy < h;
        const uint16_t *row = x + (ok ? (size_t)(ci0 + c) * P + (size_t)n * HW + (size_t)iy * w : 0);
        xa[q] = raw8(row, x0, w);
        xb[q] = raw8(row, x0 + 8, w);
        xl[q] = row[max(x0 - 1, 0)];
        xr[q] = row[min(x0 + GX, w - 1)];
        okx[q] = ok;
      } else if (rr < 32 * (GY + 2) && iy >= 0 && iy < h) {
        const uint16_t *row = x + (size_t)(ci0 + c) * P + (size_t)n * HW + (size_t)iy * w;
        xa[q] = *(const uint4 *)(row + x0);
        xb[q] = *(const uint4 *)(row + x0 + 8);
        if (x0 > 0) xl[q] = row[x0 - 1];
        if (x0 + GX < w) xr[q] = row[x0 + GX];
      }
    }
  };
  // ... and their LDS copies: dz rows as they are, the input rows three
  // times, shifted by kx (copy kx, pixel q = input column x0 - 1 + q + kx)
  auto store_tile = [&]() {
    if constexpr (RAG) {
#pragma unroll
      for (int k = 0; k < DV; ++k) dv[k] = cut8(dv[k], cx0 + 8 * (t & 1), w, okd[k]);
#pragma unroll
      for (int q = 0; q < XR; ++q) {
        xa[q] = cut8(xa[q], cx0, w, okx[q]);
        xb[q] = cut8(xb[q], cx0 + 8, w, okx[q]);
        xl[q] = okx[q] && cx0 > 0 ? xl[q] : 0u;
        xr[q] = okx[q] && cx0 + GX < w ? xr[q] : 0u;
      }
    }
#pragma unroll
    for (int k = 0; k < DV; ++k) {
      const int v = t + k * BS;
      const int half = v & 1, r = (v >> 1) & (GY - 1), c = v >> 4;
      *(uint4 *)(Ds + c * DST + r * GX + 8 * half) = dv[k];
      if (with_bias) {
        const uint32_t u[4] = {dv[k].x, dv[k].y, dv[k].z, dv[k].w};
        B s8 = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) s8 += (B)bf2f((uint16_t)(u[j] & 0xffffu)) + (B)bf2f((uint16_t)(u[j] >> 16));
        bacc[k] += s8;
      }
    }
#pragma unroll
    for (int q = 0; q < XR; ++q) {
      const int rr = t + q * BS;
      if (rr >= 32 * (GY + 2)) continue;
      const int c = rr / (GY + 2), r = rr - c * (GY + 2);
      const uint32_t W[8] = {xa[q].x, xa[q].y, xa[q].z, xa[q].w, xb[q].x, xb[q].y, xb[q].z, xb[q].w};
      uint32_t S0[8], S2[8];
      S0[0] = xl[q] | (W[0] << 16);
#pragma unroll
      for (int k = 1; k < 8; ++k) S0[k] = (W[k - 1] >> 16) | (W[k] << 16);
#pragma unroll
      for (int k = 0; k < 7; ++k) S2[k] = (W[k] >> 16) | (W[k + 1] << 16);
      S2[7] = (W[7] >> 16) | (xr[q] << 16);
      uint16_t *d0 = Xs + (0 * 32 + c) * XCI + r * GX;
      uint16_t *d1 = Xs + (1 * 32 + c) * XCI + r * GX;
      uint16_t *d2 = Xs + (2 * 32 + c) * XCI + r * GX;
      *(uint4 *)d0 = uint4{S0[0], S0[1], S0[2], S0[3]};
      *(uint4 *)(d0 + 8) = uint4{S0[4], S0[5], S0[6], S0[7]};
      *(uint4 *)d1 = uint4{W[0], W[1], W[2], W[3]};
      *(uint4 *)(d1 + 8) = uint4{W[4], W[5], W[6], W[7]};
      *(uint4 *)d2 = uint4{S2[0], S2[1], S2[2], S2[3]};
      *(uint4 *)(d2 + 8) = uint4{S2[4], S2[5], S2[6], S2[7]};
      if (RAG) d0[w - cx0 < GX ? w - cx0 : (GY + 2 - r) * GX] = 0;  // (else behind the channel's rows)
    }
  };
  // taps of kernel rows k0 .. k1 - 1 over the tile
  auto multiply = [&](auto k0, auto k1) {
#pragma unroll
    for (int ks = 0; ks < GP / 32; ++ks) {
      const int py = 2 * ks + (kq >> 1), px = 8 * (kq & 1);
      const bf8 av = *(const bf8 *)(Ds + (16 * cw + l16) * DST + 32 * ks + 8 * kq);
#pragma unroll
      for (int tp = 3 * decltype(k0)::value; tp < 3 * decltype(k1)::value; ++tp) {
        const int ky = tp / 3, kx = tp - 3 * ky;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          const bf8 bv = *(const bf8 *)(Xs + (kx * 32 + 16 * (nb + nt) + l16) * XCI + (py + ky) * GX + px);
          acc[nt][tp] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bv, acc[nt][tp], 0, 0, 0);
        }
      }
    }
  };
  using C0 = std::integral_constant<int, 0>;
  using C1 = std::integral_constant<int, 1>;
  using C3 = std::integral_constant<int, 3>;
  if (T0 < T1) load_tile(T0);
  for (int T = T0; T < T1; ++T) {
    store_tile();
    __syncthreads();
    // A tile that hangs over the image: the gradients beyond it are zero, and where a
    // tap pairs them with the image's last column (kx = 0) or last row (ky = 0) the
    // input has to be zero too, since zero times an infinite input is not zero.  That
    // column of the copy shifted by kx = 0 serves no other pair (zeroed when the row
    // is stored); the row does, so the other taps go first.
    const int py1 = h - cy0;  // rows inside the image
    if (T + 1 < T1) load_tile(T + 1);
    if constexpr (RAG) {
      multiply(C1{}, C3{});
      if (py1 < GY) {
        __syncthreads();
        if (t < 192) *(uint4 *)(Xs + (t >> 1) * XCI + py1 * GX + 8 * (t & 1)) = uint4{0u, 0u, 0u, 0u};
        __syncthreads();
      }
      multiply(C0{}, C1{});
    } else {
      multiply(C0{}, C3{});
    }
    __syncthreads();
  }
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
#pragma unroll
    for (int tp = 0; tp < 9; ++tp)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int co = co0 + 16 * cw + 4 * kq + j, ci = ci0 + 16 * (nb + nt) + l16;
        if (co < cout && (!RAG || ci < cin)) part[(size_t)split * stride + ((size_t)co * 9 + tp) * cin + ci] = acc[nt][tp][j];
      }
  if (with_bias) {
    // the 16 consecutive lanes that staged one channel's rows, summed in a
    // fixed butterfly order
#pragma unroll
    for (int k = 0; k < DV; ++k) {
      B v = bacc[k];
#pragma unroll
      for (int o = 8; o > 0; o >>= 1) v += __shfl_xor(v, o, 16);
      const int co = co0 + (t >> 4) + 16 * k;
      if ((t & 15) != 0 || co >= cout) continue;
      if (!RAG) ((float *)bpart)[(size_t)split * stride + co] = (float)v;
      else ((double *)bpart)[(size_t)split * cout + co] = v;
    }
  }
}

// Weight gradient of a layer with one input channel and at most 32 output
// channels (the network's first layer), h % 8 == 0, w % 64 == 0:
// part[split * stride + co * 9 + tap] = sum over the split's 8 x 64 pixel
// tiles of dz[co][q] x[q shifted by tap], bpart[split * stride + co] = the
// sum of dz[co][q] (FP32).  Wavefront wv owns channels 8 wv .. 8 wv + 7, its
// lanes the tile's columns; a fixed butterfly combines the lanes' sums.
// grid (splits).
constexpr int C1Y = 8;
__global__ void __launch_bounds__(BS) conv1_wgrad_kernel(int nimg, int cout, int h, int w,
                                                        const uint16_t *__restrict__ x, const uint16_t *__restrict__ dz,
                                                        float *__restrict__ part, int64_t stride, int tiles_per_split,
                                                        float *__restrict__ bpart) {
  __shared__ float xs[C1Y + 2][66];
  const int HW = h * w;
  const size_t P = (size_t)nimg * HW;
  const int tx = w / 64, tiles_img = (h / C1Y) * tx, tiles = nimg * tiles_img;
  const int split = blockIdx.x, T0 = split * tiles_per_split, T1 = min(tiles, T0 + tiles_per_split);
  const int t = threadIdx.x, wv = t >> 6, lane = t & 63;
  float acc[8][9], bacc[8];
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    bacc[c] = 0.f;
#pragma unroll
    for (int tp = 0; tp < 9; ++tp) acc[c][tp] = 0.f;
  }
  for (int T = T0; T < T1; ++T) {
    const int n = T / tiles_img, rem = T - n * tiles_img;
    const int y0 = (rem / tx) * C1Y, x0 = (rem % tx) * 64;
    __syncthreads();  // the previous tile's rows are read
    for (int i = t; i < (C1Y + 2) * 66; i += BS) {
      const int r = i / 66, q = i - r * 66, iy = y0 - 1 + r, ix = x0 - 1 + q;
      xs[r][q] = (iy >= 0 && iy < h && ix >= 0 && ix < w) ? bf2f(x[(size_t)n * HW + (size_t)iy * w + ix]) : 0.f;
    }
    __syncthreads();
#pragma unroll 2
    for (int r = 0; r < C1Y; ++r) {
      float xn[9];
#pragma unroll
      for (int tp = 0; tp < 9; ++tp) xn[tp] = xs[r + tp / 3][lane + tp % 3];
      const size_t pix = (size_t)n * HW + (size_t)(y0 + r) * w + x0 + lane;
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        const int co = 8 * wv + c;
        const float d = co < cout ? bf2f(dz[(size_t)co * P + pix]) : 0.f;
        bacc[c] += d;
#pragma unroll
        for (int tp = 0; tp < 9; ++tp) acc[c][tp] = fmaf(d, xn[tp], acc[c][tp]);
      }
    }
  }
  // The 80 sums over the lanes: each exchange halves the sums a lane carries on
  // (85 exchanges instead of a butterfly per sum, 480: 32 images of 128^2 52 -> 44
  // us).  The additions are the butterflies', so the bits are too.
  float v[80];
#pragma unroll
  for (int c = 0; c < 8; ++c) {
#pragma unroll
    for (int tp = 0; tp < 9; ++tp) v[10 * c + tp] = acc[c][tp];
    v[10 * c + 9] = bacc[c];
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int o = 32 >> k, half = 40 >> k;
    const bool up = lane & o;
#pragma unroll
    for (int i = 0; i < half; ++i) {
      const float give = up ? v[i] : v[i + half], keep = up ? v[i + half] : v[i];
      v[i] = keep + __shfl_xor(give, o, 64);
    }
  }
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    v[i] += __shfl_xor(v[i], 2, 64);
    v[i] += __shfl_xor(v[i], 1, 64);
  }
  if ((lane & 3) == 0) {
    const int first = (lane & 32 ? 40 : 0) + (lane & 16 ? 20 : 0) + (lane & 8 ? 10 : 0) + (lane & 4 ? 5 : 0);
    const int co = 8 * wv + first / 10;
    if (co < cout) {
#pragma unroll
      for (int i = 0; i < 5; ++i) {
        const int k = first % 10 + i;
        if (k < 9) part[(size_t)split * stride + co * 9 + k] = v[i];
        else if (bpart) bpart[(size_t)split * stride + co] = v[i];
      }
    }
  }
}

// Split plan of the weight gradient: which kernel, how many partial sums, pixel
// tiles per split.
struct WgradPlan {
  bool tiled, c1, packed;  // 16-byte loads of whole tiles; one-input-channel kernel; pixels packed
  int splits, chunk;       // (chunk: tiles, packed: pixels)
};

// Output-channel tile of the tiled weight gradient.
inline int wgrad_ct(int cout) { return cout <= 32 ? 32 : 64; }

// The most splits a ragged shape takes: 768 workgroups of 64 x 64 weights, at least
// 256 pixels each (fewer partial sums than that per pixel cost more than they give).
int wgrad_splits(int n, int cin, int cout, int h, int w) {
  const int64_t P = (int64_t)n * h * w;
  const int64_t groups = (int64_t)((cin * 9 + TN - 1) / TN) * ((cout + TM - 1) / TM);
  const int64_t want = std::max<int64_t>(1, (768 + groups - 1) / groups);
  const int splits = (int)std::min<int64_t>(want, std::max<int64_t>(1, (P + 255) / 256));
  int64_t chunk = (P + splits - 1) / splits;
  chunk = (chunk + TK - 1) / TK * TK;
  return (int)((P + chunk - 1) / chunk);
}

// About 768 workgroups in flight (three per CU), at least two pixel tiles
// per tiled workgroup so the partial sums stay few.
WgradPlan wgrad_plan(int n, int cin, int cout, int h, int w) {
  WgradPlan pl{};
  if (cin == 1 && cout <= 32 && h % C1Y == 0 && w % 64 == 0) {
    const int tiles = n * (h / C1Y) * (w / 64);
    pl.c1 = true;
    pl.chunk = std::min(2, tiles);
    pl.splits = (tiles + pl.chunk - 1) / pl.chunk;
    return pl;
  }
  if (cin % 32 == 0 && h % GY == 0 && w % GX == 0) {
    const int ct = wgrad_ct(cout);
    const int groups = ((cout + ct - 1) / ct) * (cin / 32);
    const int tiles = n * (h / GY) * (w / GX);
    const int want = std::max(1, (768 + groups - 1) / groups);
    const int per = std::max(std::min(2, tiles), (tiles + want - 1) / want);
    pl.tiled = true;
    pl.chunk = per;
    pl.splits = (tiles + per - 1) / per;
    return pl;
  }
  const int64_t tiles = (int64_t)n * ((h + GY - 1) / GY) * ((w + GX - 1) / GX), P = (int64_t)n * h * w;
  if (4 * P < tiles * GP) {
    pl.packed = true;
    pl.splits = wgrad_splits(n, cin, cout, h, w);
    pl.chunk = (int)((P + pl.splits - 1) / pl.splits + TK - 1) / TK * TK;
    return pl;
  }
  // ragged shapes: as many workgroups, at most the splits of wgrad_splits
  const int ct = wgrad_ct(cout);
  const int64_t groups = (int64_t)((cout + ct - 1) / ct) * ((cin + 31) / 32);
  const int64_t want = std::max<int64_t>(1, std::min<int64_t>((768 + groups - 1) / groups, wgrad_splits(n, cin, cout, h, w)));
  pl.chunk = (int)((tiles + want - 1) / want);
  pl.splits = (int)((tiles + pl.chunk - 1) / pl.chunk);
  return pl;
}

// out[i] = sum over k < splits of part[k * stride + i], i < m.  G groups of
// consecutive splits per output, each summed in split order (the unrolled
// loads are issued ahead; the additions keep their order), then the G group
// sums in group order: a fixed order for a given split count, with G
// wavefronts' loads in flight per output row when the splits are many.
// grid ceil(m / 64), 64 G threads.
template <int G>
__device__ __forceinline__ void split_sum(const float *__restrict__ part, int splits, int64_t stride, int64_t m,
                                          float *__restrict__ out) {
  __shared__ float red[G][64];
  const int o = threadIdx.x & 63, g = threadIdx.x >> 6;
  const int64_t i = (int64_t)blockIdx.x * 64 + o;
  const int k0 = (int)((int64_t)splits * g / G), k1 = (int)((int64_t)splits * (g + 1) / G);
  float s = 0.f;
  if (i < m) {
#pragma unroll 8
    for (int k = k0; k < k1; ++k) s += part[(size_t)k * stride + i];
  }
  if constexpr (G == 1) {
    if (i < m) out[i] = s;
  } else {
    red[g][o] = s;
    __syncthreads();
    if (g == 0 && i < m) {
      float r = red[0][o];
#pragma unroll
      for (int q = 1; q < G; ++q) r += red[q][o];
      out[i] = r;
    }
  }
}

template <int G>
__global__ void __launch_bounds__(64 * G) split_sum_kernel(const float *__restrict__ part, int splits, int64_t stride,
                                                          int64_t m, float *__restrict__ out) {
  split_sum<G>(part, splits, stride, m, out);
}

// The same with the bias sums db[co] of bpart[split][cout], in FP64 up to their one
// rounding, in the blocks after the weights': 64 channels a block or, of a layer with
// fewer, the next power of two, the threads left over taking more groups of splits
// (pairwise sums of the groups: a fixed order).
template <int G>
__global__ void __launch_bounds__(64 * G) split_sum2_kernel(const float *__restrict__ part, int splits, int64_t m,
                                                           float *__restrict__ dw, const double *__restrict__ bpart,
                                                           int cout, float *__restrict__ db) {
  const int nb = (int)((m + 63) / 64), b = (int)blockIdx.x - nb;
  if (b < 0) {
    split_sum<G>(part, splits, m, m, dw);
    return;
  }
  __shared__ double red[64 * G];
  int cp = 64;
  while (cp / 2 >= cout) cp /= 2;
  const int t = threadIdx.x, co = 64 * b + (t & (cp - 1)), g = t / cp, ng = 64 * G / cp;
  const int k0 = (int)((int64_t)splits * g / ng), k1 = (int)((int64_t)splits * (g + 1) / ng);
  double s = 0;
  if (co < cout) {
#pragma unroll 8
    for (int k = k0; k < k1; ++k) s += bpart[(size_t)k * cout + co];
  }
  red[t] = s;
  for (int w = 32 * G; w >= cp; w >>= 1) {
    __syncthreads();
    if (t < w) red[t] += red[t + w];
  }
  if (t < cp && co < cout) db[co] = (float)red[t];
}

void launch_split_sum2(const float *part, int splits, int64_t m, float *dw, const double *bpart, int cout, float *db,
                       hipStream_t s) {
  const dim3 g((unsigned)((m + 63) / 64 + (cout + 63) / 64));
  if (splits >= 64)
    hipLaunchKernelGGL(split_sum2_kernel<16>, g, dim3(64 * 16), 0, s, part, splits, m, dw, bpart, cout, db);
  else if (splits >= 16)
    hipLaunchKernelGGL(split_sum2_kernel<4>, g, dim3(64 * 4), 0, s, part, splits, m, dw, bpart, cout, db);
  else
    hipLaunchKernelGGL(split_sum2_kernel<1>, g, dim3(64), 0, s, part, splits, m, dw, bpart, cout, db);
}

void launch_split_sum(const float *part, int splits, int64_t stride, int64_t m, float *out, hipStream_t s) {
  const dim3 g((unsigned)((m + 63) / 64));
  if (splits >= 64)
    hipLaunchKernelGGL(split_sum_kernel<16>, g, dim3(64 * 16), 0, s, part, splits, stride, m, out);
  else if (splits >= 16)
    hipLaunchKernelGGL(split_sum_kernel<4>, g, dim3(64 * 4), 0, s, part, splits, stride, m, out);
  else
    hipLaunchKernelGGL(split_sum_kernel<1>, g, dim3(64), 0, s, part, splits, stride, m, out);
}

// wrot[ci][ky][kx][co] = w[co][2-ky][2-kx][ci]: the data gradient is the
// forward convolution of dz with these weights.
__global__ void __launch_bounds__(BS) rot_kernel(int cin, int cout, const uint16_t *__restrict__ w,
                                                uint16_t *__restrict__ wrot) {
  const int64_t i = (int64_t)blockIdx.x * BS + threadIdx.x;
  if (i >= (int64_t)cin * cout * 9) return;
  const int ci = (int)(i % cin), tap = (int)((i / cin) % 9), co = (int)(i / (9 * (int64_t)cin));
  wrot[((size_t)ci * 9 + (8 - tap)) * cout + co] = w[i];
}

// Every layer of a table in one launch: the turned, transposed layout of
// rot_kernel at wrot + off[l] from layer l's weights at w + off[l] (layout
// [cout][3][3][cin]).  Thread i writes element k of layer l's output (so the
// stores are contiguous and the scattered accesses are the reads); it finds
// its layer by scanning the prefix counts (at most kRotLayers entries).
constexpr int kRotLayers = 32;
struct RotTable {
  int n;
  int cin[kRotLayers], cout[kRotLayers];
  int64_t off[kRotLayers], first[kRotLayers + 1];
};

__global__ void __launch_bounds__(BS) rot_all_kernel(const RotTable t, const uint16_t *__restrict__ w,
                                                    uint16_t *__restrict__ wrot) {
  const int64_t i = (int64_t)blockIdx.x * BS + threadIdx.x;
  if (i >= t.first[t.n]) return;
  int l = 0;
  while (l + 1 < t.n && i >= t.first[l + 1]) ++l;
  const int64_t k = i - t.first[l];
  const int cin = t.cin[l], cout = t.cout[l];
  const int co = (int)(k % cout), rtap = (int)((k / cout) % 9), ci = (int)(k / (9 * (int64_t)cout));
  wrot[t.off[l] + k] = w[t.off[l] + ((int64_t)co * 9 + (8 - rtap)) * cin + ci];
}

__global__ void __launch_bounds__(BS) relu_kernel(int64_t n, const float *__restrict__ z, uint16_t *__restrict__ a) {
  const int64_t i = (int64_t)blockIdx.x * BS + threadIdx.x;
  if (i < n) a[i] = f2bf(fmaxf(z[i], 0.f));
}

__global__ void __launch_bounds__(BS) relu_back_kernel(int64_t n, const uint16_t *__restrict__ a,
                                                      const float *__restrict__ da, uint16_t *__restrict__ dz) {
  const int64_t i = (int64_t)blockIdx.x * BS + threadIdx.x;
  if (i < n) dz[i] = f2bf(bf2f(a[i]) > 0.f ? da[i] : 0.f);
}

// The same on eight elements per thread (count % 8 == 0, 16-byte aligned).
__global__ void __launch_bounds__(BS) relu_back8_kernel(int64_t n8, const uint4 *__restrict__ a,
                                                       const float4 *__restrict__ da, uint4 *__restrict__ dz) {
  const int64_t i = (int64_t)blockIdx.x * BS + threadIdx.x;
  if (i >= n8) return;
  const uint4 av = a[i];
  const float4 d0 = da[2 * i], d1 = da[2 * i + 1];
  const uint32_t aw[4] = {av.x, av.y, av.z, av.w};
  const float dv[8] = {d0.x, d0.y, d0.z, d0.w, d1.x, d1.y, d1.z, d1.w};
  uint32_t o[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const uint16_t lo = f2bf(bf2f((uint16_t)(aw[k] & 0xffffu)) > 0.f ? dv[2 * k] : 0.f);
    const uint16_t hi = f2bf(bf2f((uint16_t)(aw[k] >> 16)) > 0.f ? dv[2 * k + 1] : 0.f);
    o[k] = (uint32_t)lo | ((uint32_t)hi << 16);
  }
  dz[i] = uint4{o[0], o[1], o[2], o[3]};
}

__global__ void __launch_bounds__(BS) to_bf16_kernel(int64_t n, const float *__restrict__ x, uint16_t *__restrict__ y) {
  const int64_t i = (int64_t)blockIdx.x * BS + threadIdx.x;
  if (i < n) y[i] = f2bf(x[i]);
}

__global__ void __launch_bounds__(BS) from_bf16_kernel(int64_t n, const uint16_t *__restrict__ x, float *__restrict__ y) {
  const int64_t i = (int64_t)blockIdx.x * BS + threadIdx.x;
  if (i < n) y[i] = bf2f(x[i]);
}

// y[plane][i][j] = mean of x[plane][2i..2i+1][2j..2j+1]
__global__ void __launch_bounds__(BS) pool2_kernel(int64_t planes, int h, int w, const uint16_t *__restrict__ x,
                                                  uint16_t *__restrict__ y) {
  const int ho = h / 2, wo = w / 2;
  const int64_t i = (int64_t)blockIdx.x * BS + threadIdx.x;
  if (i >= planes * ho * wo) return;
  const int64_t pl = i / ((int64_t)ho * wo);
  const int r = (int)(i % ((int64_t)ho * wo)), yi = r / wo, xi = r - yi * wo;
  const uint16_t *b = x + (size_t)pl * h * w + (size_t)(2 * yi) * w + 2 * xi;
  y[i] = f2bf(0.25f * (bf2f(b[0]) + bf2f(b[1]) + bf2f(b[w]) + bf2f(b[w + 1])));
}

__global__ void __launch_bounds__(BS) pool2_back_kernel(int64_t planes, int h, int w, const float *__restrict__ dy,
                                                       float *__restrict__ dx) {
  const int64_t i = (int64_t)blockIdx.x * BS + threadIdx.x;
  if (i >= planes * h * w) return;
  const int64_t pl = i / ((int64_t)h * w);
  const int r = (int)(i % ((int64_t)h * w)), yi = r / w, xi = r - yi * w;
  dx[i] = 0.25f * dy[(size_t)pl * (h / 2) * (w / 2) + (size_t)(yi / 2) * (w / 2) + xi / 2];
}

// The gradients that meet at a pooled and skipped activation a, through its ReLU:
// dz = bf16((0.25 dy[plane][i/2][j/2] + skip[plane][i][j]) * (a > 0)), the values of
// pool2_back, axpy and relu_back one after another.  V elements of a row per thread
// (8: 16-byte accesses; w % 8 == 0, aligned).  What bounds it is its bytes: the
// three levels of 32 images of 128^2 took 119 us as three passes each, 49 in one.
template <int V>
__global__ void __launch_bounds__(BS) pool2_back_join_kernel(int64_t planes, int h, int w, const float *__restrict__ dy,
                                                            const float *__restrict__ skip,
                                                            const uint16_t *__restrict__ a,
                                                            uint16_t *__restrict__ dz) {
  const int wv = w / V;
  const int64_t i = (int64_t)blockIdx.x * BS + threadIdx.x;
  if (i >= planes * h * wv) return;
  const int64_t pl = i / ((int64_t)h * wv);
  const int r = (int)(i % ((int64_t)h * wv)), yi = r / wv, xi = V * (r - yi * wv);
  const float *g = dy + (size_t)pl * (h / 2) * (w / 2) + (size_t)(yi / 2) * (w / 2) + xi / 2;
  const size_t o = (size_t)pl * h * w + (size_t)yi * w + xi;
  if constexpr (V == 8) {
    const float4 q = *(const float4 *)g, s0 = *(const float4 *)(skip + o), s1 = *(const float4 *)(skip + o + 4);
    const uint4 av = *(const uint4 *)(a + o);
    const uint32_t aw[4] = {av.x, av.y, av.z, av.w};
    const float gv[4] = {q.x, q.y, q.z, q.w}, sv[8] = {s0.x, s0.y, s0.z, s0.w, s1.x, s1.y, s1.z, s1.w};
    uint32_t u[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const float p = 0.25f * gv[k];
      const uint16_t lo = f2bf(bf2f((uint16_t)(aw[k] & 0xffffu)) > 0.f ? __fadd_rn(p, sv[2 * k]) : 0.f);
      const uint16_t hi = f2bf(bf2f((uint16_t)(aw[k] >> 16)) > 0.f ? __fadd_rn(p, sv[2 * k + 1]) : 0.f);
      u[k] = (uint32_t)lo | ((uint32_t)hi << 16);
    }
    *(uint4 *)(dz + o) = uint4{u[0], u[1], u[2], u[3]};
  } else {
    dz[o] = f2bf(bf2f(a[o]) > 0.f ? __fadd_rn(0.25f * g[0], skip[o]) : 0.f);
  }
}

// y[plane][2i+a][2j+b] = x[plane][i][j]
__global__ void __launch_bounds__(BS) up2_kernel(int64_t planes, int h, int w, const uint16_t *__restrict__ x,
                                                uint16_t *__restrict__ y) {
  const int64_t i = (int64_t)blockIdx.x * BS + threadIdx.x;
  if (i >= planes * 4 * h * w) return;
  const int64_t pl = i / (4 * (int64_t)h * w);
  const int r = (int)(i % (4 * (int64_t)h * w)), yi = r / (2 * w), xi = r - yi * (2 * w);
  y[i] = x[(size_t)pl * h * w + (size_t)(yi / 2) * w + xi / 2];
}

// Vector forms for w % 4 == 0: pool2_back writes four outputs of each of
// two rows from two gradients; up2 copies four inputs to eight outputs of
// each of two rows (16-byte stores).
__global__ void __launch_bounds__(BS) pool2_back4_kernel(int64_t planes, int h, int w, const float *__restrict__ dy,
                                                        float *__restrict__ dx) {
  const int wq = w / 4, ho = h / 2;
  const int64_t i = (int64_t)blockIdx.x * BS + threadIdx.x;
  if (i >= planes * ho * wq) return;
  const int64_t pl = i / ((int64_t)ho * wq);
  const int r = (int)(i % ((int64_t)ho * wq)), yo = r / wq, xq = r - yo * wq;
  const float2 g = *(const float2 *)(dy + (size_t)pl * ho * (w / 2) + (size_t)yo * (w / 2) + 2 * xq);
  const float4 v = {0.25f * g.x, 0.25f * g.x, 0.25f * g.y, 0.25f * g.y};
  float *b = dx + (size_t)pl * h * w + (size_t)(2 * yo) * w + 4 * xq;
  *(float4 *)b = v;
  *(float4 *)(b + w) = v;
}

__global__ void __launch_bounds__(BS) up2x4_kernel(int64_t planes, int h, int w, const uint16_t *__restrict__ x,
                                                  uint16_t *__restrict__ y) {
  const int wq = w / 4;
  const int64_t i = (int64_t)blockIdx.x * BS + threadIdx.x;
  if (i >= planes * h * wq) return;
  const int64_t pl = i / ((int64_t)h * wq);
  const int r = (int)(i % ((int64_t)h * wq)), yi = r / wq, xq = r - yi * wq;
  const uint2 v = *(const uint2 *)(x + (size_t)pl * h * w + (size_t)yi * w + 4 * xq);
  const uint32_t e[4] = {v.x & 0xffffu, v.x >> 16, v.y & 0xffffu, v.y >> 16};
  const uint4 o = {e[0] | (e[0] << 16), e[1] | (e[1] << 16), e[2] | (e[2] << 16), e[3] | (e[3] << 16)};
  uint16_t *b = y + (size_t)pl * 4 * h * w + (size_t)(2 * yi) * (2 * w) + 8 * xq;
  *(uint4 *)b = o;
  *(uint4 *)(b + 2 * w) = o;
}

// up2_back on two outputs per thread (w % 2 == 0): two 16-byte row reads.
__global__ void __launch_bounds__(BS) up2_back2_kernel(int64_t planes, int h, int w, const float *__restrict__ dy,
                                                      float *__restrict__ dx) {
  const int wh = w / 2;
  const int64_t i = (int64_t)blockIdx.x * BS + threadIdx.x;
  if (i >= planes * h * wh) return;
  const int64_t pl = i / ((int64_t)h * wh);
  const int r = (int)(i % ((int64_t)h * wh)), yi = r / wh, xh = r - yi * wh;
  const float *b = dy + (size_t)pl * 4 * h * w + (size_t)(2 * yi) * (2 * w) + 4 * xh;
  const float4 u = *(const float4 *)b, d = *(const float4 *)(b + 2 * w);
  *(float2 *)(dx + (size_t)pl * h * w + (size_t)yi * w + 2 * xh) = float2{u.x + u.y + d.x + d.y, u.z + u.w + d.z + d.w};
}

__global__ void __launch_bounds__(BS) up2_back_kernel(int64_t planes, int h, int w, const float *__restrict__ dy,
                                                     float *__restrict__ dx) {
  const int64_t i = (int64_t)blockIdx.x * BS + threadIdx.x;
  if (i >= planes * h * w) return;
  const int64_t pl = i / ((int64_t)h * w);
  const int r = (int)(i % ((int64_t)h * w)), yi = r / w, xi = r - yi * w;
  const float *b = dy + (size_t)pl * 4 * h * w + (size_t)(2 * yi) * (2 * w) + 2 * xi;
  dx[i] = b[0] + b[1] + b[2 * w] + b[2 * w + 1];
}

__global__ void __launch_bounds__(BS) adam_kernel(int64_t n, float *__restrict__ p, float *__restrict__ m,
                                                 float *__restrict__ v, const float *__restrict__ g,
                                                 uint16_t *__restrict__ pb, float lr, float b1, float b2, float eps,
                                                 float c1, float c2) {
  const int64_t i = (int64_t)blockIdx.x * BS + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.f - b1) * gi;
  const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  const float pi = p[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
  p[i] = pi;
  if (pb) pb[i] = f2bf(pi);
}

__global__ void __launch_bounds__(BS) axpy_kernel(int64_t n, float a, const float *__restrict__ x, float *__restrict__ y) {
  const int64_t i = (int64_t)blockIdx.x * BS + threadIdx.x;
  if (i < n) y[i] += a * x[i];
}

__global__ void __launch_bounds__(BS) axpy4_kernel(int64_t n4, float a, const float4 *__restrict__ x,
                                                  float4 *__restrict__ y) {
  const int64_t i = (int64_t)blockIdx.x * BS + threadIdx.x;
  if (i >= n4) return;
  const float4 u = x[i];
  float4 v = y[i];
  v.x += a * u.x;
  v.y += a * u.y;
  v.z += a * u.z;
  v.w += a * u.w;
  y[i] = v;
}

// grad = 2 (pred - target) * scale; partial sums of (pred - target)^2
__global__ void __launch_bounds__(BS) mse_kernel(int64_t n, const float *__restrict__ pred,
                                                const float *__restrict__ target, float scale,
                                                float *__restrict__ grad, double *__restrict__ part) {
  __shared__ double lds[BS / 64];
  const int64_t i = (int64_t)blockIdx.x * BS + threadIdx.x;
  double e2 = 0;
  if (i < n) {
    const float d = pred[i] - target[i];
    if (grad) grad[i] = 2.f * d * scale;
    e2 = (double)d * d;
  }
  const double s = block_sum(e2, lds);
  if (threadIdx.x == 0) part[blockIdx.x] = s;
}

__global__ void __launch_bounds__(BS) sum_kernel(const double *__restrict__ part, int nb, double *__restrict__ out) {
  __shared__ double lds[BS / 64];
  double v = 0;
  for (int b = threadIdx.x; b < nb; b += BS) v += part[b];
  const double s = block_sum(v, lds);
  if (threadIdx.x == 0) out[0] = s;
}

// da[c][n][p] = dout[n] wl[c] / hw
__global__ void __launch_bounds__(BS) gap_linear_back_a_kernel(int nimg, int c, int hw, const float *__restrict__ dout,
                                                              const float *__restrict__ wl, float *__restrict__ da) {
  const int64_t i = (int64_t)blockIdx.x * BS + threadIdx.x;
  if (i >= (int64_t)c * nimg * hw) return;
  const int64_t cn = i / hw;
  const int ch = (int)(cn / nimg), n = (int)(cn - (int64_t)ch * nimg);
  da[i] = dout[n] * wl[ch] / (float)hw;
}

// out[n] = bl + sum_c wl[c] mean_p a[c][n][p]: a workgroup per image (or several, one
// after another), FP64 sums in a fixed order.  Q = 1: a wavefront takes a channel, then
// the next one, its lanes the pixels lane + 64 k; Q = 4 (64 to 255 pixels): four
// channels at a time, for loads in flight; Q = 0 (fewer): L lanes a channel and 64 / L
// channels side by side.  256 channels of 13 x 13 pixels, 32 images: 8 us (40 with 256
// threads that divide an index per element); 64 channels of one pixel, 4096 images:
// 8 (21 with 64 lanes per channel), of 10 x 10 pixels 24 (Q = 1 36); 256 channels of
// 16 x 16, 1024 images: Q = 4 53, Q = 1 31.
template <int Q>
__global__ void __launch_bounds__(1024) gap_linear_kernel(int nimg, int c, int hw, int L, const uint16_t *__restrict__ a,
                                                           const float *__restrict__ wl, const float *__restrict__ bl,
                                                           float *__restrict__ out) {
  __shared__ double lds[16];
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63, waves = blockDim.x >> 6;
  for (int n = blockIdx.x; n < nimg; n += gridDim.x) {
    double v = 0;
    if constexpr (Q == 0) {
      const int side = 64 / L, p = lane & (L - 1);
      if (p < hw) {
#pragma unroll 4
        for (int ch = wv * side + lane / L; ch < c; ch += waves * side)
          v += (double)wl[ch] * (double)bf2f(a[((size_t)ch * nimg + n) * hw + p]);
      }
    } else if constexpr (Q == 1) {
      for (int ch = wv; ch < c; ch += waves) {
        const uint16_t *row = a + ((size_t)ch * nimg + n) * hw;
        double sp = 0;
#pragma unroll 4
        for (int p = lane; p < hw; p += 64) sp += bf2f(row[p]);
        v += (double)wl[ch] * sp;
      }
    } else {
      for (int ch = wv; ch < c; ch += Q * waves) {
        const uint16_t *row[Q];
        double sp[Q] = {};
#pragma unroll
        for (int q = 0; q < Q; ++q) row[q] = a + ((size_t)std::min(ch + q * waves, c - 1) * nimg + n) * hw;
        for (int p = lane; p < hw; p += 64)
#pragma unroll
          for (int q = 0; q < Q; ++q) sp[q] += bf2f(row[q][p]);
#pragma unroll
        for (int q = 0; q < Q; ++q)
          if (ch + q * waves < c) v += (double)wl[ch + q * waves] * sp[q];
      }
    }
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
    if (lane == 0) lds[wv] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
      double s = 0;
      for (int k = 0; k < waves; ++k) s += lds[k];
      out[n] = (float)(s / hw + bl[0]);
    }
    if (n + (int)gridDim.x < nimg) __syncthreads();
  }
}

// dwl[c] = sum_n dout[n] mean_p a[c][n][p]; dbl = sum_n dout[n].  One workgroup per channel (+1 for the bias).
__global__ void __launch_bounds__(BS) gap_linear_back_w_kernel(int nimg, int c, int hw, const uint16_t *__restrict__ a,
                                                              const float *__restrict__ dout, float *__restrict__ dwl,
                                                              float *__restrict__ dbl) {
  __shared__ double lds[BS / 64];
  const int ch = blockIdx.x;
  double v = 0;
  if (ch < c) {
    for (int64_t i = threadIdx.x; i < (int64_t)nimg * hw; i += BS)
      v += (double)dout[i / hw] * bf2f(a[(size_t)ch * nimg * hw + i]);
  } else {
    for (int n = threadIdx.x; n < nimg; n += BS) v += dout[n];
  }
  const double s = block_sum(v, lds);
  if (threadIdx.x == 0) {
    if (ch < c) dwl[ch] = (float)(s / hw);
    else dbl[0] = (float)s;
  }
}

int nb_of(int64_t n) { return (int)((n + BS - 1) / BS); }
bool aligned(const void *p, uintptr_t b) { return ((uintptr_t)p & (b - 1)) == 0; }

thread_local std::string g_err;

template <typename F>
fdtd_status nguard(F &&f) {
  try {
    f();
    return FDTD_OK;
  } catch (const Error &e) {
    g_err = e.msg;
    return e.code;
  } catch (const std::exception &e) {
    g_err = e.what();
    return FDTD_EDEVICE;
  }
}

void need(bool ok) {
  if (!ok) throw Error{FDTD_EINVAL, "invalid sizes or missing pointer"};
}


}  // namespace

extern "C" {

fdtd_status fdtd_nn_conv3x3(int32_t n, int32_t cin, int32_t cout, int32_t h, int32_t w, const uint16_t *x,
                            const uint16_t *wt, const float *bias, float *z, uint16_t *a, void *stream) {
  return nguard([&] {
    need(n > 0 && n <= 65535 && cin > 0 && cout > 0 && h > 0 && w > 0 && x && wt && (z || a));
    launch_conv(n, cin, cout, h, w, x, wt, bias, z, a, nullptr, (hipStream_t)stream);
    FDTD_HIP(hipGetLastError());
  });
}

fdtd_status fdtd_nn_conv3x3_dgrad(int32_t n, int32_t cin, int32_t cout, int32_t h, int32_t w, const uint16_t *dz,
                                  const uint16_t *wt, uint16_t *wrot, float *dx, void *stream) {
  return nguard([&] {
    need(n > 0 && n <= 65535 && cin > 0 && cout > 0 && h > 0 && w > 0 && dz && wrot && dx);
    hipStream_t s = (hipStream_t)stream;
    if (wt) hipLaunchKernelGGL(rot_kernel, dim3(nb_of((int64_t)cin * cout * 9)), dim3(BS), 0, s, cin, cout, wt, wrot);
    launch_conv(n, cout, cin, h, w, dz, wrot, nullptr, dx, nullptr, nullptr, s);
    FDTD_HIP(hipGetLastError());
  });
}

fdtd_status fdtd_nn_conv3x3_dgrad_relu(int32_t n, int32_t cin, int32_t cout, int32_t h, int32_t w, const uint16_t *dz,
                                       const uint16_t *wt, uint16_t *wrot, const uint16_t *a, uint16_t *dza,
                                       void *stream) {
  return nguard([&] {
    need(n > 0 && n <= 65535 && cin > 0 && cout > 0 && h > 0 && w > 0 && dz && wrot && a && dza);
    hipStream_t s = (hipStream_t)stream;
    if (wt) hipLaunchKernelGGL(rot_kernel, dim3(nb_of((int64_t)cin * cout * 9)), dim3(BS), 0, s, cin, cout, wt, wrot);
    launch_conv(n, cout, cin, h, w, dz, wrot, nullptr, nullptr, dza, a, s);
    FDTD_HIP(hipGetLastError());
  });
}

fdtd_status fdtd_nn_rot_weights(int32_t nlayers, const int32_t *cin, const int32_t *cout, const int64_t *off,
                                const uint16_t *w, uint16_t *wrot, void *stream) {
  return nguard([&] {
    need(nlayers >= 1 && nlayers <= kRotLayers && cin && cout && off && w && wrot);
    RotTable t{};
    t.n = nlayers;
    t.first[0] = 0;
    for (int l = 0; l < nlayers; ++l) {
      need(cin[l] > 0 && cout[l] > 0 && off[l] >= 0);
      t.cin[l] = cin[l];
      t.cout[l] = cout[l];
      t.off[l] = off[l];
      t.first[l + 1] = t.first[l] + (int64_t)cin[l] * cout[l] * 9;
    }
    need(t.first[nlayers] <= (int64_t)INT32_MAX * BS);
    hipLaunchKernelGGL(rot_all_kernel, dim3(nb_of(t.first[nlayers])), dim3(BS), 0, (hipStream_t)stream, t, w, wrot);
    FDTD_HIP(hipGetLastError());
  });
}

int64_t fdtd_nn_wgrad_work(int32_t n, int32_t cin, int32_t cout, int32_t h, int32_t w) {
  if (n <= 0 || cin <= 0 || cout <= 0 || h <= 0 || w <= 0) return 0;
  const WgradPlan pl = wgrad_plan(n, cin, cout, h, w);
  // splits rows of cout * cin * 9 weight and cout bias sums, the latter FP64 (and
  // 8-byte aligned) in the kernel for any shape and alignment
  const int64_t m = (int64_t)cout * cin * 9;
  return pl.c1 ? pl.splits * (m + cout) : pl.splits * (m + 2 * cout) + 1;
}

}  // extern "C"

// Scratch of the allocation-free weight gradient: one array per device,
// held until the process ends (72 MiB: the largest workspace the split plan
// asks for, about 768 partial sums of a 64 x 32 x 9 block, is 55 MiB).  In
// host code `scratch` names a host-side stand-in, never the device memory:
// kernels get the address hipGetSymbolAddress returns on each device.
static constexpr int64_t kScratchFloats = int64_t(18) << 20;
static __device__ __align__(256) float scratch[kScratchFloats];

namespace {

// The weight and bias gradients with partial sums in `work` (at least
// fdtd_nn_wgrad_work floats; every slot the reductions read is written first).
void wgrad_run(int32_t n, int32_t cin, int32_t cout, int32_t h, int32_t w, const uint16_t *x, const uint16_t *dz,
               float *dw, float *db, float *work, hipStream_t s) {
    const int64_t m = (int64_t)cout * cin * 9, stride = m + cout;
    const WgradPlan pl = wgrad_plan(n, cin, cout, h, w);
    // partial rows [split][m weight sums | cout bias sums]
    float *bp = db ? work + m : nullptr;
    const int ct = wgrad_ct(cout);
    const int64_t blocks = (int64_t)((cout + ct - 1) / ct) * ((cin + 31) / 32);
    if (pl.c1) {
      hipLaunchKernelGGL(conv1_wgrad_kernel, dim3(pl.splits), dim3(BS), 0, s, n, cout, h, w, x, dz, work, stride,
                         pl.chunk, bp);
    } else if (pl.tiled && (((uintptr_t)dz | (uintptr_t)x) & 15) == 0) {
      auto *k = ct == 32 ? &conv_wgrad_mfma_kernel<32, false> : &conv_wgrad_mfma_kernel<64, false>;
      hipLaunchKernelGGL(k, dim3(xcd_grid(blocks * pl.splits)), dim3(BS), 0, s, n, cin, cout, h, w, x, dz, work, stride,
                         pl.chunk, (void *)bp, pl.splits);
    } else {
      // any shape, any address: partial rows [split][m weight sums], then (8-byte
      // aligned) the bias sums [split][cout] in FP64
      double *b64 = (double *)(((uintptr_t)(work + pl.splits * m) + 7) & ~(uintptr_t)7);
      if (pl.packed) {
        const dim3 g((cin * 9 + TN - 1) / TN, (cout + TM - 1) / TM, pl.splits);
        hipLaunchKernelGGL(conv_wgrad_kernel, g, dim3(BS), 0, s, n, cin, cout, h, w, x, dz, work, pl.chunk,
                           db ? b64 : nullptr);
      } else {
        auto *k = ct == 32 ? &conv_wgrad_mfma_kernel<32, true> : &conv_wgrad_mfma_kernel<64, true>;
        hipLaunchKernelGGL(k, dim3(xcd_grid(blocks * pl.splits)), dim3(BS), 0, s, n, cin, cout, h, w, x, dz, work, m,
                           pl.chunk, db ? (void *)b64 : nullptr, pl.splits);
      }
      if (db) launch_split_sum2(work, pl.splits, m, dw, b64, cout, db, s);
      else launch_split_sum(work, pl.splits, m, m, dw, s);
      FDTD_HIP(hipGetLastError());
      return;
    }
    if (db && db == dw + m) {  // contiguous weight and bias gradients: one reduction
      launch_split_sum(work, pl.splits, stride, m + cout, dw, s);
    } else {
      launch_split_sum(work, pl.splits, stride, m, dw, s);
      if (db) launch_split_sum(work + m, pl.splits, stride, cout, db, s);
    }
    FDTD_HIP(hipGetLastError());
}

// Device address of `scratch` on the current device, looked up once per
// device with that device current.
float *scratch_on_current_device() {
  int dev = 0;
  FDTD_HIP(hipGetDevice(&dev));
  static std::mutex mu;
  static std::map<int, float *> ptrs;
  std::lock_guard<std::mutex> lock(mu);
  auto it = ptrs.find(dev);
  if (it != ptrs.end()) return it->second;
  void *p = nullptr;
  const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
  if (e != hipSuccess || !p) {
    (void)hipGetLastError();
    throw Error{FDTD_EDEVICE, std::string("hipGetSymbolAddress(scratch) failed: ") + hipGetErrorString(e)};
  }
  ptrs[dev] = static_cast<float *>(p);
  return ptrs[dev];
}

}  // namespace

extern "C" {

fdtd_status fdtd_nn_conv3x3_wgrad(int32_t n, int32_t cin, int32_t cout, int32_t h, int32_t w, const uint16_t *x,
                                  const uint16_t *dz, float *dw, float *db, float *work, void *stream) {
  return nguard([&] {
    need(n > 0 && cin > 0 && cout > 0 && h > 0 && w > 0 && x && dz && dw && work);
    wgrad_run(n, cin, cout, h, w, x, dz, dw, db, work, (hipStream_t)stream);
  });
}

fdtd_status fdtd_nn_conv3x3_wgrad_noalloc(int32_t n, int32_t cin, int32_t cout, int32_t h, int32_t w,
                                          const uint16_t *x, const uint16_t *dz, float *dw, float *db, void *stream) {
  return nguard([&] {
    need(n > 0 && cin > 0 && cout > 0 && h > 0 && w > 0 && x && dz && dw);
    const int64_t want = fdtd_nn_wgrad_work(n, cin, cout, h, w);
    if (want > kScratchFloats)
      throw Error{FDTD_EINVAL, "weight gradient needs " + std::to_string(want) + " floats of scratch; the static array "
                               "holds " + std::to_string(kScratchFloats) + " (use fdtd_nn_conv3x3_wgrad with a workspace)"};
    wgrad_run(n, cin, cout, h, w, x, dz, dw, db, scratch_on_current_device(), (hipStream_t)stream);
  });
}

fdtd_status fdtd_nn_relu_bf16(int64_t count, const float *z, uint16_t *a, void *stream) {
  return nguard([&] {
    need(count > 0 && z && a);
    hipLaunchKernelGGL(relu_kernel, dim3(nb_of(count)), dim3(BS), 0, (hipStream_t)stream, count, z, a);
    FDTD_HIP(hipGetLastError());
  });
}

fdtd_status fdtd_nn_relu_bf16_backward(int64_t count, const uint16_t *a, const float *da, uint16_t *dz,
                                       void *stream) {
  return nguard([&] {
    need(count > 0 && a && da && dz);
    if (count % 8 == 0 && aligned(a, 16) && aligned(da, 16) && aligned(dz, 16))
      hipLaunchKernelGGL(relu_back8_kernel, dim3(nb_of(count / 8)), dim3(BS), 0, (hipStream_t)stream, count / 8,
                         (const uint4 *)a, (const float4 *)da, (uint4 *)dz);
    else
      hipLaunchKernelGGL(relu_back_kernel, dim3(nb_of(count)), dim3(BS), 0, (hipStream_t)stream, count, a, da, dz);
    FDTD_HIP(hipGetLastError());
  });
}

fdtd_status fdtd_nn_to_bf16(int64_t count, const float *x, uint16_t *y, void *stream) {
  return nguard([&] {
    need(count > 0 && x && y);
    hipLaunchKernelGGL(to_bf16_kernel, dim3(nb_of(count)), dim3(BS), 0, (hipStream_t)stream, count, x, y);
    FDTD_HIP(hipGetLastError());
  });
}

fdtd_status fdtd_nn_from_bf16(int64_t count, const uint16_t *x, float *y, void *stream) {
  return nguard([&] {
    need(count > 0 && x && y);
    hipLaunchKernelGGL(from_bf16_kernel, dim3(nb_of(count)), dim3(BS), 0, (hipStream_t)stream, count, x, y);
    FDTD_HIP(hipGetLastError());
  });
}

fdtd_status fdtd_nn_pool2(int64_t planes, int32_t h, int32_t w, const uint16_t *x, uint16_t *y, void *stream) {
  return nguard([&] {
    need(planes > 0 && h > 1 && w > 1 && h % 2 == 0 && w % 2 == 0 && x && y);
    hipLaunchKernelGGL(pool2_kernel, dim3(nb_of(planes * (h / 2) * (w / 2))), dim3(BS), 0, (hipStream_t)stream,
                       planes, h, w, x, y);
    FDTD_HIP(hipGetLastError());
  });
}

fdtd_status fdtd_nn_pool2_backward(int64_t planes, int32_t h, int32_t w, const float *dy, float *dx, void *stream) {
  return nguard([&] {
    need(planes > 0 && h > 1 && w > 1 && h % 2 == 0 && w % 2 == 0 && dy && dx);
    if (w % 4 == 0 && aligned(dy, 8) && aligned(dx, 16))
      hipLaunchKernelGGL(pool2_back4_kernel, dim3(nb_of(planes * (h / 2) * (w / 4))), dim3(BS), 0,
                         (hipStream_t)stream, planes, h, w, dy, dx);
    else
      hipLaunchKernelGGL(pool2_back_kernel, dim3(nb_of(planes * h * w)), dim3(BS), 0, (hipStream_t)stream, planes, h,
                         w, dy, dx);
    FDTD_HIP(hipGetLastError());
  });
}

fdtd_status fdtd_nn_pool2_backward_join(int64_t planes, int32_t h, int32_t w, const float *dy, const float *skip,
                                        const uint16_t *a, uint16_t *dz, void *stream) {
  return nguard([&] {
    need(planes > 0 && h > 1 && w > 1 && h % 2 == 0 && w % 2 == 0 && dy && skip && a && dz);
    hipStream_t s = (hipStream_t)stream;
    if (w % 8 == 0 && aligned(dy, 16) && aligned(skip, 16) && aligned(a, 16) && aligned(dz, 16))
      hipLaunchKernelGGL(pool2_back_join_kernel<8>, dim3(nb_of(planes * h * (w / 8))), dim3(BS), 0, s, planes, h, w, dy,
                         skip, a, dz);
    else
      hipLaunchKernelGGL(pool2_back_join_kernel<1>, dim3(nb_of(planes * h * w)), dim3(BS), 0, s, planes, h, w, dy, skip,
                         a, dz);
    FDTD_HIP(hipGetLastError());
  });
}

fdtd_status fdtd_nn_up2(int64_t planes, int32_t h, int32_t w, const uint16_t *x, uint16_t *y, void *stream) {
  return nguard([&] {
    need(planes > 0 && h > 0 && w > 0 && x && y);
    if (w % 4 == 0 && aligned(x, 8) && aligned(y, 16))
      hipLaunchKernelGGL(up2x4_kernel, dim3(nb_of(planes * h * (w / 4))), dim3(BS), 0, (hipStream_t)stream, planes, h,
                         w, x, y);
    else
      hipLaunchKernelGGL(up2_kernel, dim3(nb_of(planes * 4 * h * w)), dim3(BS), 0, (hipStream_t)stream, planes, h, w,
                         x, y);
    FDTD_HIP(hipGetLastError());
  });
}

fdtd_status fdtd_nn_up2_backward(int64_t planes, int32_t h, int32_t w, const float *dy, float *dx, void *stream) {
  return nguard([&] {
    need(planes > 0 && h > 0 && w > 0 && dy && dx);
    if (w % 2 == 0 && aligned(dy, 16) && aligned(dx, 8))
      hipLaunchKernelGGL(up2_back2_kernel, dim3(nb_of(planes * h * (w / 2))), dim3(BS), 0, (hipStream_t)stream,
                         planes, h, w, dy, dx);
    else
      hipLaunchKernelGGL(up2_back_kernel, dim3(nb_of(planes * h * w)), dim3(BS), 0, (hipStream_t)stream, planes, h,
                         w, dy, dx);
    FDTD_HIP(hipGetLastError());
  });
}

fdtd_status fdtd_nn_adam(int64_t count, float *p, float *m, float *v, const float *g, uint16_t *pb, float lr,
                         float beta1, float beta2, float eps, int32_t t, void *stream) {
  return nguard([&] {
    need(count > 0 && p && m && v && g && t >= 1);
    const float c1 = 1.f - std::pow(beta1, (float)t), c2 = 1.f - std::pow(beta2, (float)t);
    hipLaunchKernelGGL(adam_kernel, dim3(nb_of(count)), dim3(BS), 0, (hipStream_t)stream, count, p, m, v, g, pb, lr,
                       beta1, beta2, eps, c1, c2);
    FDTD_HIP(hipGetLastError());
  });
}

fdtd_status fdtd_nn_axpy(int64_t count, float a, const float *x, float *y, void *stream) {
  return nguard([&] {
    need(count > 0 && x && y);
    if (count % 4 == 0 && aligned(x, 16) && aligned(y, 16))
      hipLaunchKernelGGL(axpy4_kernel, dim3(nb_of(count / 4)), dim3(BS), 0, (hipStream_t)stream, count / 4, a,
                         (const float4 *)x, (float4 *)y);
    else
      hipLaunchKernelGGL(axpy_kernel, dim3(nb_of(count)), dim3(BS), 0, (hipStream_t)stream, count, a, x, y);
    FDTD_HIP(hipGetLastError());
  });
}

int64_t fdtd_nn_mse_work(int64_t count) { return count > 0 ? nb_of(count) : 0; }

fdtd_status fdtd_nn_mse(int64_t count, const float *pred, const float *target, float scale, float *grad,
                        double *work, double *sum_sq, void *stream) {
  return nguard([&] {
    need(count > 0 && pred && target && work && sum_sq);
    hipStream_t s = (hipStream_t)stream;
    const int nb = nb_of(count);
    hipLaunchKernelGGL(mse_kernel, dim3(nb), dim3(BS), 0, s, count, pred, target, scale, grad, work);
    hipLaunchKernelGGL(sum_kernel, dim3(1), dim3(BS), 0, s, work, nb, sum_sq);
    FDTD_HIP(hipGetLastError());
  });
}

fdtd_status fdtd_nn_gap_linear(int32_t n, int32_t c, int32_t hw, const uint16_t *a, const float *wl, const float *bl,
                               float *out, void *stream) {
  return nguard([&] {
    need(n > 0 && c > 0 && hw > 0 && a && wl && bl && out);
    int L = 1;
    while (L < 64 && L < hw) L *= 2;
    const dim3 grid(std::min(n, 1 << 21));
    // while two workgroups a CU hold the images, the more wavefronts the better; beyond,
    // their number costs, unless each still has much to do (4096 images of 64 channels:
    // 9 pixels 22 us with 1024 threads, 8 with 256; 100 pixels 28 with 512, 24 with 256;
    // 1024 images of 256 channels, 169 pixels 27 with 512, 42 with 256; 256 pixels 33
    // with 1024, 31 with 512)
    const int most = n <= 512 ? 1024 : hw >= 256 || (hw >= 64 && c > 64) ? 512 : 256;
    const int threads = (int)std::min<int64_t>(most, ((int64_t)c * L + 63) / 64 * 64);
    auto *k = hw < 64 ? &gap_linear_kernel<0> : hw < 256 ? &gap_linear_kernel<4> : &gap_linear_kernel<1>;
    hipLaunchKernelGGL(k, grid, dim3(threads), 0, (hipStream_t)stream, n, c, hw, L, a, wl, bl, out);
    FDTD_HIP(hipGetLastError());
  });
}

fdtd_status fdtd_nn_gap_linear_backward(int32_t n, int32_t c, int32_t hw, const uint16_t *a, const float *wl,
                                        const float *dout, float *da, float *dwl, float *dbl, void *stream) {
  return nguard([&] {
    need(n > 0 && c > 0 && hw > 0 && a && wl && dout && da && dwl && dbl);
    hipStream_t s = (hipStream_t)stream;
    const int64_t total = (int64_t)n * c * hw;
    hipLaunchKernelGGL(gap_linear_back_a_kernel, dim3(nb_of(total)), dim3(BS), 0, s, n, c, hw, dout, wl, da);
    hipLaunchKernelGGL(gap_linear_back_w_kernel, dim3(c + 1), dim3(BS), 0, s, n, c, hw, a, dout, dwl, dbl);
    FDTD_HIP(hipGetLastError());
  });
}

const char *fdtd_nn_last_error(void) { return g_err.c_str(); }

}  // extern "C"
