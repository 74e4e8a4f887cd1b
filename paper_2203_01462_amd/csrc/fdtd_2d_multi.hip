// fdtd_2d_multi.hip -- several time steps per launch of the 2D TMz solve and
// of its adjoint, for every kind of node (background, absorber, walls,
// injection lines, design, gap).
//
// The per-step kernels of fdtd_2d.hip spend a launch on every step: a small
// grid's step is one chain of dependent loads and stores (200^2 in FP64: 12 us
// per step, whatever the bandwidth), a large grid moves its state through
// memory once per step.  Here a workgroup loads a region of 64 x (R nw) nodes
// into registers, advances it up to K steps and stores the (64 - 2K) x (R nw -
// 2K) nodes in its middle: a step spoils one more node on every side (E needs
// H one node below and left, H needs E one node above and right), so after K
// steps the middle is exact.  Regions overlap by their halos; every array a
// halo reads, the Drude current included, has a read and a write copy, and
// launches alternate between them.
//
// What bounds it: a small grid, the chain launch - parameter loads - field
// loads - K steps - stores, with one region per CU; a large one, the regions'
// loads and stores (per node and step about a third of the per-step kernels'
// bytes) and the vector instructions of the steps, which overlap only as far
// as the registers let two workgroups share a CU.  2048^2 FP32: 18.7 us per
// step with two steps per launch on the background only, 6.9 / 6.4 us now.
//
// A wavefront holds 64 columns and R consecutive rows per lane, wavefronts
// stack along y.  Along x the neighbours come from the adjacent lanes (DPP
// wave shifts), along y from the lane's own registers; only the first and last
// row of a wavefront go through LDS, double-buffered, so a step costs one
// barrier.  The H_x row below a wavefront's first is recomputed in it (from the
// exchanged E row), which saves a second exchange.  Absorber memories, Drude
// coefficients and currents and the FP64 sensitivity sums stay in registers
// for the K steps; what a step reads from memory (history, adjoint source) is
// loaded one step ahead, the incident line's values are staged in LDS first.
//
// The arithmetic of a node is that of step_general / step_bulk in
// fdtd_2d.hip, with the roundings of the graded and Drude terms written out in
// both, so the results are the per-step kernels' to the last bit in FP64.
// Outside the absorber the grading tables
// hold the identity (b = 1, a = 0, 1/kappa = 1) and the memories are zero, so
// a graded difference needs no per-lane choice.
#include <algorithm>

#include "fdtd_multi.hpp"

namespace fdtd {
namespace {

// LDS of a workgroup: the exchanged rows [2][waves][2][64] and, where the
// region meets an injection line, the incident values of the launch's steps:
// E at every region row [K][rows], E and H at the two horizontal lines [K][4].
template <typename T, int R>
struct MultiLds {
  T x[2 * MWMAX * 2 * MX];
  T ei[MKMAX * 64];
  T ab[MKMAX * 4];
};

// One region with origin (x0, y0); its nodes [K, 64 - K) x [K, R nw - K) are
// stored.  PX, PY: the absorber or the walls along x / y are in reach; TF: an
// injection line is; DES: the design or the gap box is.  The parameter block
// stays in memory and is read with scalar loads where it is needed (kept in
// registers it would spill into the step loop).
template <typename T, bool ADJ, bool PX, bool PY, bool TF, bool DES, int R>
__device__ __forceinline__ void multi_body(cptr<Multi2D<T>> m, const MultiStep st, const int K, const int nw,
                                           const int x0, const int y0, MultiLds<T, R> &lds) {
  const int nx = m->s.nx, ny = m->s.ny, P = m->s.P;
  const int pitch = m->s.pitch, rd = st.rd;
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i = x0 + lane, jb = y0 + wv * R;
  const T ch = m->s.chx, ce_s = m->s.ce_s;
  // Every load below is unconditional, from a row and column clamped to the
  // grid (or box).  What a node outside the grid holds besides E = 0 does not
  // matter: it reaches only E on the walls, which is never updated.
  const int ic = PX ? min(max(i, 0), nx - 1) : i;
  auto jc = [&](int j) { return PY ? min(max(j, 0), ny - 1) : j; };
  auto ld = [](const T *q, int at) { return ((gptr<const T>)q)[at]; };

  // ------------------------------------------------------------ loads
  T e[R], hy[R], hx[R + 1];  // hx[r]: row jb - 1 + r
  {
    const T *ez = m->s.ez[rd], *fx = m->s.hx[rd], *fy = m->s.hy[rd];
#pragma unroll
    for (int r = 0; r <= R; ++r) hx[r] = ld(fx + jc(jb - 1 + r) * pitch, ic);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      e[r] = ld(ez + jc(jb + r) * pitch, ic);
      hy[r] = ld(fy + jc(jb + r) * pitch, ic);
    }
  }
  // E update factor: 0 on the walls and outside the grid, where E stays 0
  T ce[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    ce[r] = ce_s;
    if (PX) ce[r] = i >= 1 && i <= nx - 2 ? ce[r] : T(0);
    if (PY) ce[r] = jb + r >= 1 && jb + r <= ny - 2 ? ce[r] : T(0);
  }
  // absorber along x (per lane) and along y (do the wavefront's rows reach
  // it?); the memories are zero off their strips
  bool py = false;
  T bxe = T(1), axe = T(0), ikxe = T(1), bxh = T(1), axh = T(0), ikxh = T(1);
  T bye[R], aye[R], ikye[R], byh[R + 1], ayh[R + 1], ikyh[R + 1];
  T pex[R], pey[R], phx[R + 1], phy[R];
  if constexpr (PX) {
    bxe = ld(m->s.bxe, ic); axe = ld(m->s.axe, ic); ikxe = ld(m->s.ikxe, ic);
    bxh = ld(m->s.bxh, ic); axh = ld(m->s.axh, ic); ikxh = ld(m->s.ikxh, ic);
    const T *q0 = m->s.pex[rd], *q1 = m->s.phy[rd];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      pex[r] = ld(q0 + jc(jb + r) * pitch, ic);
      phy[r] = ld(q1 + jc(jb + r) * pitch, ic);
    }
  }
  if constexpr (PY) {
    py = P > 0 && (jb - 1 < P || jb + R - 1 >= ny - 1 - P);
    const cptr<T> tbe = (cptr<T>)m->s.bye, tae = (cptr<T>)m->s.aye, tie = (cptr<T>)m->s.ikye;
    const cptr<T> tbh = (cptr<T>)m->s.byh, tah = (cptr<T>)m->s.ayh, tih = (cptr<T>)m->s.ikyh;
    const T *q0 = m->s.pey[rd], *q1 = m->s.phx[rd];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int j = jc(jb + r);
      bye[r] = tbe[j]; aye[r] = tae[j]; ikye[r] = tie[j];
      pey[r] = ld(q0 + j * pitch, ic);
    }
#pragma unroll
    for (int r = 0; r <= R; ++r) {
      const int j = jc(jb - 1 + r);
      byh[r] = tbh[j]; ayh[r] = tah[j]; ikyh[r] = tih[j];
      phx[r] = ld(q1 + j * pitch, ic);
    }
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    if (PX) e[r] = i >= 0 && i < nx ? e[r] : T(0);
    if (PY) e[r] = jb + r >= 0 && jb + r < ny ? e[r] : T(0);
  }
  const bool ownx = lane >= K && lane < MX - K && i < nx;
  const int row0 = wv * R;  // the wavefront's first row in the region
  auto owny = [&](int r) { return row0 + r >= K && row0 + r < R * nw - K && jb + r < ny; };
  // Design and gap.  A Drude node's update e0 + inv q, q = dt/dx curl - (..) J
  // - bs e0, and a plain node's e0 + ce curl are one form: a plain node has
  // factor ce, dt/dx replaced by 1, and no J, bs and beta.
  T J[R], fq[R], bs[R], beta[R], gb[R], gc[R], Em[R];
  double gacc[R];
  const int nd = m->s.dnx * m->s.dny, ng = m->s.ng, dnx = m->s.dnx, gnx = m->s.gnx;
  const int dx0 = m->s.dx0, dy0 = m->s.dy0, dny = m->s.dny, gx0 = m->s.gx0, gy0 = m->s.gy0, gny = m->s.gny;
  const int dic = min(max(i - dx0, 0), dnx - 1), gic = min(max(i - gx0, 0), gnx - 1);
  const bool lind = i >= dx0 && i < dx0 + dnx, ling = i >= gx0 && i < gx0 + gnx;  // lane in the box's columns
  auto rind = [&](int r) { return jb + r >= dy0 && jb + r < dy0 + dny; };          // row in the box's rows
  auto ring = [&](int r) { return jb + r >= gy0 && jb + r < gy0 + gny; };
  auto drow = [&](int r) { return min(max(jb + r - dy0, 0), dny - 1) * dnx; };
  auto grow = [&](int r) { return min(max(jb + r - gy0, 0), gny - 1) * gnx; };
  T dthJ = T(0), kpm1 = T(0), ga = T(0);
  T *hist = nullptr;
  bool gw = false;      // does the wavefront hold gap nodes?
  bool staged = false;  // adjoint source values of the launch's steps in LDS
  if constexpr (DES) {
    const T *rho = m->s.rho, *Jr = m->J[rd];
    const T A0 = m->s.A0, A1 = m->s.A1, B0 = m->s.B0, B1 = m->s.B1, Sg = m->s.Sg, dt = m->s.dt_, ce_g = m->s.ce_g;
    const T rs = m->s.rs, gsm = m->s.gsm, dtdx = m->s.dtdx;
    hist = st.hist ? (T *)st.hist : m->s.hist;
    gw = x0 + MX > gx0 && x0 < gx0 + gnx && jb + R > gy0 && jb < gy0 + gny;
    T x[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      x[r] = ld(rho + drow(r), dic);
      J[r] = ld(Jr + drow(r), dic);
      if constexpr (ADJ) {
        gacc[r] = ((gptr<const double>)(m->s.grad + drow(r)))[dic];
        Em[r] = ld(hist + (int64_t)(st.n0 - 1 - st.hist_base) * nd + drow(r), dic);
      }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const bool gap = ling && ring(r), drude = lind && rind(r) && !gap;
      ce[r] = gap ? ce_g : ce[r];
      const T eps2 = fma1(x[r], A1, A0);
      const T be = fma1(x[r], B1, B0);
      const T b = fma1(be, dt, Sg * x[r] * (T(1) - x[r]));
      const T inv = T(2) / (eps2 + b);
      ce[r] = drude ? inv : ce[r];
      fq[r] = drude ? dtdx : T(1);
      bs[r] = drude ? b : T(0);
      beta[r] = drude ? be : T(0);
      J[r] = drude ? J[r] : T(0);
      if constexpr (ADJ) {
        gc[r] = -(T(1) - rs) / (T(2) * (rs + x[r] * (T(1) - rs)));
        gb[r] = gsm * (T(1) - T(2) * x[r]);
      }
    }
    dthJ = m->s.dthJ;
    kpm1 = m->s.kpm1;
    ga = m->s.ga;
    if constexpr (ADJ) {
      // values of every gap node for the launch's steps, where they fit
      staged = st.steps * ng <= MKMAX * 64;
      if (staged && x0 + MX > gx0 && x0 < gx0 + gnx && y0 + R * nw > gy0 && y0 < gy0 + gny) {
        for (int q = threadIdx.x; q < st.steps * ng; q += 64 * nw) {
          const int s = q / ng;
          lds.ei[q] = ((gptr<const T>)(m->s.asrc + (int64_t)(st.n0 - s) * ng))[q - s * ng];
        }
        __syncthreads();
      }
    }
  }
  // incident values of the launch's steps; the factors that add them
  int ja = 0, jt = 0;
  T tcx = T(0), tcy = T(0);  // at the vertical lines (H_y), between them (H_x)
  bool tfrow = false, tfcol = false;
  if constexpr (TF) {
    const int ia = m->s.ia, ib = m->s.ib, jref = m->s.jref, L = m->s.L, ry = R * nw;
    const T *einc = m->s.einc, *hinc = m->s.hinc;
    ja = m->s.ja;
    jt = m->s.jb;
    tcx = i == ia - 1 ? -ch : i == ib ? ch : T(0);
    tcy = i >= ia && i <= ib ? ch : T(0);
    tfcol = (ia - 1 >= x0 && ia - 1 < x0 + MX) || (ib >= x0 && ib < x0 + MX);
    auto hit = [&](int v) { return v >= jb - 1 && v < jb + R; };
    tfrow = hit(ja - 1) || hit(ja) || hit(jt);
    if (tfcol)
      for (int q = threadIdx.x; q < st.steps * ry; q += 64 * nw) {
        const int s = q / ry, j = y0 + q - s * ry;
        const bool on = j >= ja && j <= jt;
        const T v = ((gptr<const T>)einc)[(int64_t)(st.n0 + s) * L + (on ? j - jref : 0)];
        lds.ei[q] = on ? v : T(0);
      }
    if ((int)threadIdx.x < 4 * st.steps) {
      const int s = threadIdx.x >> 2, w = threadIdx.x & 3;
      const int at = w == 0 ? ja : w == 2 ? ja - 1 : jt;
      lds.ab[threadIdx.x] = ((gptr<const T>)(w < 2 ? einc : hinc))[(int64_t)(st.n0 + s) * L + (at - jref)];
    }
    __syncthreads();
  }

  // ------------------------------------------------------------ steps
#pragma unroll 1
  for (int s = 0; s < st.steps; ++s) {
    const int n = ADJ ? st.n0 - s : st.n0 + s;
    T Emn[R];
    if constexpr (DES && ADJ) {  // the next step's forward field
      const T *h = hist + (int64_t)(max(n - 1, st.hist_base + 1) - 1 - st.hist_base) * nd;
#pragma unroll
      for (int r = 0; r < R; ++r) Emn[r] = ld(h + drow(r), dic);
    }
    // the E rows the curls act on: graded along y in the adjoint
    T gy[R];
#pragma unroll
    for (int r = 0; r < R; ++r) gy[r] = e[r];
    if constexpr (PY && ADJ) {
      if (py) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
          pey[r] = mem1(bye[r], pey[r], aye[r], e[r]);
          gy[r] = fma1(e[r], ikye[r], pey[r]);
        }
      }
    }
    T *xb = lds.x + (s & 1) * (MWMAX * 2 * MX);
    xb[(2 * wv) * MX + lane] = gy[0];
    xb[(2 * wv + 1) * MX + lane] = gy[R - 1];
    // H_y (needs no row exchange); hyc: what E's curl reads, graded along x in
    // the adjoint
    T hyc[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if constexpr (!ADJ) {
        T dE = lane_right(e[r]) - e[r];
        if constexpr (PX) {
          phy[r] = mem1(bxh, phy[r], axh, dE);
          dE = fma1(dE, ikxh, phy[r]);
        }
        hy[r] = fma1(ch, dE, hy[r]);
      } else {
        T gx = e[r];
        if constexpr (PX) {
          pex[r] = mem1(bxe, pex[r], axe, e[r]);
          gx = fma1(e[r], ikxe, pex[r]);
        }
        hy[r] = fma1(ch, lane_right(gx) - gx, hy[r]);
      }
    }
    if constexpr (TF && !ADJ) {
      if (tfcol) {
#pragma unroll
        for (int r = 0; r < R; ++r) hy[r] = fma1(tcx, lds.ei[s * (R * nw) + row0 + r], hy[r]);
      }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      hyc[r] = hy[r];
      if constexpr (ADJ && PX) {
        phy[r] = mem1(bxh, phy[r], axh, hy[r]);
        hyc[r] = fma1(hy[r], ikxh, phy[r]);
      }
    }
    __syncthreads();
    const T gdn = wv > 0 ? xb[(2 * wv - 1) * MX + lane] : T(0);
    const T gup = wv + 1 < nw ? xb[(2 * wv + 2) * MX + lane] : T(0);
    // H_x; hxc as hyc
    T hxc[R + 1];
#pragma unroll
    for (int r = 0; r <= R; ++r) hxc[r] = (r < R ? gy[r] : gup) - (r > 0 ? gy[r - 1] : gdn);
    if constexpr (PY && !ADJ) {
      if (py) {
#pragma unroll
        for (int r = 0; r <= R; ++r) {
          phx[r] = mem1(byh[r], phx[r], ayh[r], hxc[r]);
          hxc[r] = fma1(hxc[r], ikyh[r], phx[r]);
        }
      }
    }
#pragma unroll
    for (int r = 0; r <= R; ++r) hx[r] = fma1(-ch, hxc[r], hx[r]);
    T hA = T(0), hB = T(0);
    if constexpr (TF && !ADJ) {
      if (tfrow) {
        const T eA = lds.ab[4 * s], eB = lds.ab[4 * s + 1];
        hA = tcy != T(0) ? lds.ab[4 * s + 2] : T(0);
        hB = tcy != T(0) ? lds.ab[4 * s + 3] : T(0);
#pragma unroll
        for (int r = 0; r <= R; ++r) {
          if (jb - 1 + r == ja - 1) hx[r] += mul1(tcy, eA);
          if (jb - 1 + r == jt) hx[r] -= mul1(tcy, eB);
        }
      }
    }
#pragma unroll
    for (int r = 0; r <= R; ++r) hxc[r] = hx[r];
    if constexpr (PY && ADJ) {
      if (py) {
#pragma unroll
        for (int r = 0; r <= R; ++r) {
          phx[r] = mem1(byh[r], phx[r], ayh[r], hx[r]);
          hxc[r] = fma1(hx[r], ikyh[r], phx[r]);
        }
      }
    }
    // E and J
    T cx[R], cy[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      cx[r] = hyc[r] - lane_left(hyc[r]);
      cy[r] = hxc[r + 1] - hxc[r];
      if constexpr (PX && !ADJ) {
        pex[r] = mem1(bxe, pex[r], axe, cx[r]);
        cx[r] = fma1(cx[r], ikxe, pex[r]);
      }
    }
    if constexpr (PY && !ADJ) {
      if (py) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
          pey[r] = mem1(bye[r], pey[r], aye[r], cy[r]);
          cy[r] = fma1(cy[r], ikye[r], pey[r]);
        }
      }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) cx[r] = cx[r] - cy[r];
    if constexpr (TF && !ADJ) {
      if (tfrow) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
          if (jb + r == ja) cx[r] += hA;
          if (jb + r == jt) cx[r] -= hB;
        }
      }
    }
    if constexpr (DES && ADJ) {
      if (gw) {  // the adjoint source
#pragma unroll
        for (int r = 0; r < R; ++r)
          if (ring(r)) {
            const T v = staged ? lds.ei[s * ng + grow(r) + gic] : ld(m->s.asrc + (int64_t)n * ng + grow(r), gic);
            cx[r] = ling ? cx[r] + v : cx[r];
          }
      }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if constexpr (!DES) {
        e[r] = fma1(ce[r], cx[r], e[r]);
      } else {
        const T e0 = e[r], Jo = J[r];
        const T q = fma1(-bs[r], e0, fma1(fq[r], cx[r], -(dthJ * Jo)));
        const T e1 = fma1(ce[r], q, e0);
        const T Jn = Jo + fma1(kpm1, Jo, beta[r] * (e0 + e1));
        J[r] = Jn;
        e[r] = e1;
        if constexpr (ADJ) {  // (stored on the Drude nodes only)
          const T t = fma1(gc[r], Jn + Jo, fma1(ga, ce[r] * q, gb[r] * (e0 + e1)));
          gacc[r] = sens1(gacc[r], Em[r], t);
          Em[r] = Emn[r];
        }
      }
    }
    if constexpr (DES && !ADJ) {
      if (st.hist_on && ownx && lind) {
        T *h = hist + (int64_t)(n - st.hist_base) * nd;
#pragma unroll
        for (int r = 0; r < R; ++r)
          if (owny(r) && rind(r)) ((gptr<T>)(h + drow(r)))[dic] = e[r];
      }
      if (gw && ownx && ling) {
        double *g = m->s.gapE + (int64_t)(n + 1) * ng;
#pragma unroll
        for (int r = 0; r < R; ++r)
          if (owny(r) && ring(r)) ((gptr<double>)(g + grow(r)))[gic] = (double)e[r];
      }
    }
  }

  // ------------------------------------------------------------ stores
  asm volatile("" : "+s"(m));  // the write pointers are read here, not kept over the steps
  {
    const int wr = rd ^ 1;
    if (ownx) {
      T *ez = m->s.ez[wr], *fx = m->s.hx[wr], *fy = m->s.hy[wr];
#pragma unroll
      for (int r = 0; r < R; ++r)
        if (owny(r)) {
          const int64_t q = (int64_t)(jb + r) * pitch;
          ((gptr<T>)(ez + q))[i] = e[r];
          ((gptr<T>)(fx + q))[i] = hx[r + 1];
          ((gptr<T>)(fy + q))[i] = hy[r];
        }
    }
    if constexpr (PX) {
      T *q0 = m->s.pex[wr], *q1 = m->s.phy[wr];
      if (ownx && pml_e2(i, nx, P))
#pragma unroll
        for (int r = 0; r < R; ++r)
          if (owny(r)) ((gptr<T>)(q0 + (int64_t)(jb + r) * pitch))[i] = pex[r];
      if (ownx && pml_h2(i, nx, P))
#pragma unroll
        for (int r = 0; r < R; ++r)
          if (owny(r)) ((gptr<T>)(q1 + (int64_t)(jb + r) * pitch))[i] = phy[r];
    }
    if constexpr (PY) {
      if (py && ownx) {
        T *q0 = m->s.pey[wr], *q1 = m->s.phx[wr];
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const int j = jb + r;
          if (owny(r) && pml_e2(j, ny, P)) ((gptr<T>)(q0 + (int64_t)j * pitch))[i] = pey[r];
          if (owny(r) && pml_h2(j, ny, P)) ((gptr<T>)(q1 + (int64_t)j * pitch))[i] = phx[r + 1];
        }
      }
    }
    if constexpr (DES) {
      if (ownx && lind) {
        T *Jw = m->J[wr];
#pragma unroll
        for (int r = 0; r < R; ++r)
          if (owny(r) && rind(r) && !(ling && ring(r))) {
            ((gptr<T>)(Jw + drow(r)))[dic] = J[r];
            if constexpr (ADJ) ((gptr<double>)(m->s.grad + drow(r)))[dic] = gacc[r];
          }
      }
    }
  }
}

// Workgroups first[k] .. first[k+1] - 1 take the regions of instance k (a
// single context is a batch of one).  Which body a region needs follows from
// what its nodes touch.
template <typename T, bool ADJ, int R>
__global__ void __launch_bounds__(64 * MWMAX)
    step2d_multi(const Multi2D<T> *ms, const int *first, const int ninst, const MultiStep st, const MultiTile g) {
  __shared__ MultiLds<T, R> lds;
  const int b = blockIdx.x;
  int lo = 0, hi = ninst - 1, f0 = 0;
  if (ninst > 1) {
    const cptr<int> f = (cptr<int>)first;
    while (lo < hi) {  // last k with first[k] <= b
      const int mid = (lo + hi + 1) >> 1;
      if (f[mid] <= b) lo = mid; else hi = mid - 1;
    }
    f0 = f[lo];
  }
  const cptr<Multi2D<T>> m = (cptr<Multi2D<T>>)(ms + lo);
  const int nx = m->s.nx, ny = m->s.ny, P = m->s.P;
  const int lb = b - f0;
  const int K = g.K, nw = g.nw, W = MX - 2 * K, ntx = (nx + W - 1) / W, H = R * nw - 2 * K, nty = (ny + H - 1) / H;
  const int tx = lb % ntx, ty = lb / ntx;
  if (ty >= nty) return;
  const int x0 = tx * W - K, y0 = ty * H - K;
  const int x1 = x0 + MX - 1, y1 = y0 + R * nw - 1;
  const bool px = x0 < P + 1 || x1 > nx - 3 - P, py = y0 < P + 1 || y1 > ny - 3 - P;
  bool tf = false;
  if (!ADJ && m->s.tf_on) {
    const int ia = m->s.ia, ib = m->s.ib, ja = m->s.ja, jt = m->s.jb;
    auto hit = [](int lo, int hi, int v) { return v >= lo && v <= hi; };
    tf = hit(x0, x1, ia - 1) || hit(x0, x1, ib) || hit(y0 - 1, y1, ja - 1) || hit(y0, y1, ja) || hit(y0 - 1, y1, jt);
  }
  auto meets = [&](int bx, int by, int bnx, int bny) {
    return x1 >= bx && x0 < bx + bnx && y1 >= by && y0 < by + bny;
  };
  const bool des = meets(m->s.dx0, m->s.dy0, m->s.dnx, m->s.dny) || meets(m->s.gx0, m->s.gy0, m->s.gnx, m->s.gny);
  constexpr bool F = !ADJ;
  if (des) {
    if (px || py || tf) multi_body<T, ADJ, true, true, F, true, R>(m, st, K, nw, x0, y0, lds);
    else multi_body<T, ADJ, false, false, false, true, R>(m, st, K, nw, x0, y0, lds);
  } else if (F && tf) {
    if (px && py) multi_body<T, ADJ, true, true, F, false, R>(m, st, K, nw, x0, y0, lds);
    else if (px) multi_body<T, ADJ, true, false, F, false, R>(m, st, K, nw, x0, y0, lds);
    else if (py) multi_body<T, ADJ, false, true, F, false, R>(m, st, K, nw, x0, y0, lds);
    else multi_body<T, ADJ, false, false, F, false, R>(m, st, K, nw, x0, y0, lds);
  } else {
    if (px && py) multi_body<T, ADJ, true, true, false, false, R>(m, st, K, nw, x0, y0, lds);
    else if (px) multi_body<T, ADJ, true, false, false, false, R>(m, st, K, nw, x0, y0, lds);
    else if (py) multi_body<T, ADJ, false, true, false, false, R>(m, st, K, nw, x0, y0, lds);
    else multi_body<T, ADJ, false, false, false, false, R>(m, st, K, nw, x0, y0, lds);
  }
}

}  // namespace

int step2d_multi_blocks(int nx, int ny, const MultiTile &g) { return multi_regions(nx, ny, g); }

// Regions by size.  While one round of the 256 CUs holds them all, a launch
// takes one region's time: the flattest region that still fits wins (fewer
// instructions per step and wavefront, and more steps per launch pay for the
// launch and the loads), so the candidates are tried in that order.  Beyond
// one round the work per exact node counts, and the bytes of the halos: 64 x 64
// nodes in FP32, 64 x 32 in FP64.  (FP64 at R = 4 spills, 46 registers forward and
// 138 adjoint; compiled for 8 wavefronts at most it does not, but then one
// workgroup is on a CU instead of two: 2048^2 10.8 / 11.8 -> 15.7 / 15.7.)
// Measured on square grids with a side/4 design box, us per forward / adjoint
// step (R, nw, K), where the neighbouring choices cross:
//   FP32 333^2: 2,16,10 1.10 / 1.04; 4,8,8 1.26 / 1.23; 4,16,12 1.32 / 1.48
//        400^2: 2,16,10 1.63 / 1.45; 4,8,8 1.28 / 1.25; 4,16,12 1.36 / 1.42
//        512^2: 4,8,8   1.52 / 1.40; 4,16,12 1.42 / 1.47; 4,16,10 1.58 / 1.62
//        700^2: 4,16,12 2.01 / 1.74; 4,16,10 1.60 / 1.68
//       1448^2: 4,16,10 4.47 / 4.29; 4,16,8 4.73 / 4.59
//       2048^2: 4,16,10 6.99 / 6.65; 4,16,8 6.85 / 6.43; 4,8,8 7.74 / 7.48
//   FP64 333^2: 2,16,10 1.47 / 1.24; 2,16,8 1.71 / 1.48
//        400^2: 2,16,10 2.09 / 1.85; 2,16,8 1.67 / 1.49
//        512^2: 2,16,8  2.37 / 2.11; 4,8,8 2.01 / 2.17; 4,12,8 2.06 / 2.56
//       2048^2: 2,16,8  16.0 / 15.4; 4,8,8 10.7 / 11.7; 4,12,8 11.2 / 12.3
// (the per-step kernels: 333^2 FP32 7.2 / 7.2, 512^2 7.6 / 7.7, 2048^2 25.0 /
// 27.3; 200^2 FP64 11.9 / 10.8, here 1.49 / 1.57).
MultiTile multi2d_tile(const int (*n)[2], int count, int precision) {
  static const MultiTile f32[] = {{2, 16, 10}, {4, 8, 8}, {4, 16, 12}, {4, 16, 10}};
  static const MultiTile f64[] = {{2, 16, 10}, {2, 16, 8}};
  auto fits = [&](const MultiTile &g) {
    int64_t t = 0;
    for (int k = 0; k < count; ++k) t += step2d_multi_blocks(n[k][0], n[k][1], g);
    return t <= 256;
  };
  if (precision == 64) {
    for (const MultiTile &g : f64)
      if (fits(g)) return g;
    return {4, 8, 8};
  }
  for (const MultiTile &g : f32)
    if (fits(g)) return g;
  int64_t nodes = 0;
  for (int k = 0; k < count; ++k) nodes += (int64_t)n[k][0] * n[k][1];
  return nodes < 3000000 ? MultiTile{4, 16, 10} : MultiTile{4, 16, 8};
}

template <typename T, bool ADJ>
static void launch_multi(const Multi2D<T> *ms, const int *first, int ninst, int nblocks, const MultiStep &st,
                         const MultiTile &g, hipStream_t s) {
  const dim3 grid(nblocks), block(64 * g.nw);
  if (g.R == 2) hipLaunchKernelGGL((step2d_multi<T, ADJ, 2>), grid, block, 0, s, ms, first, ninst, st, g);
  else hipLaunchKernelGGL((step2d_multi<T, ADJ, 4>), grid, block, 0, s, ms, first, ninst, st, g);
}

template <typename T>
void launch_step2d_multi(const Multi2D<T> *ms, const int *first, int ninst, int nblocks, int n0, int steps,
                         const MultiTile &g, int rd, bool adjoint, void *hist, int hist_base, int hist_on,
                         hipStream_t s) {
  const MultiStep st{n0, steps, rd, hist, hist_base, hist_on};
  if (adjoint) launch_multi<T, true>(ms, first, ninst, nblocks, st, g, s);
  else launch_multi<T, false>(ms, first, ninst, nblocks, st, g, s);
}

template void launch_step2d_multi<float>(const Multi2D<float> *, const int *, int, int, int, int, const MultiTile &,
                                         int, bool, void *, int, int, hipStream_t);
template void launch_step2d_multi<double>(const Multi2D<double> *, const int *, int, int, int, int, const MultiTile &,
                                          int, bool, void *, int, int, hipStream_t);

}  // namespace fdtd
