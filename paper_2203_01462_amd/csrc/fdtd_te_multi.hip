// fdtd_te_multi.hip -- several time steps per launch of the 2D TEz solve (E_x,
// E_y, H_z) and of its adjoint, for every kind of node.
//
// The regions, the register and LDS scheme and the exactness argument are
// those of fdtd_2d_multi.hip; the roles of E and H are swapped: H_z needs E_x
// one row above and E_y one column right, E_x needs H_z one row below, E_y H_z
// one column left, so a step again spoils one node per side.  The H_z row below
// a wavefront's first is recomputed in it, from the E_x and E_y rows it gets
// from the wavefront below (in the adjoint graded, as the curls read them).
//
// What bounds it is what bounds the TMz kernel.  A launch per step before
// (fdtd_te.hip): 384^2 FP32 11.7 / 13.4 us per forward / adjoint step, now 1.5 /
// 1.75; 1024^2 FP32 18.5, now 3.7.  The sums are that kernel's, up to the rounding
// of separately compiled code.
#include <algorithm>

#include "fdtd_multi.hpp"

namespace fdtd {
namespace {

// LDS of a workgroup: the exchanged rows [2][waves][3][64] (E_x first, E_x
// last, E_y last); the incident H at every region row [K][rows] or, in the
// adjoint, the gap's source values; E and H at the two horizontal lines [K][4].
template <typename T>
struct TeLds {
  T x[2 * MWMAX * 3 * MX];
  T ei[MKMAX * 64];
  T ab[MKMAX * 4];
};

// One edge family (0: E_x, 1: E_y) of a lane's R edges in the design: the form
// e0 + c q, q = fq curl - dthJ J - bs e0 of fdtd_2d_multi.hip.
template <typename T, bool ADJ, int R>
struct TeEdges {
  T J[R], fq[R], bs[R], beta[R], gb[R], gc[R], Em[R];
  double gacc[R];
};

template <typename T, bool ADJ, bool PX, bool PY, bool TF, bool DES, int R>
__device__ __forceinline__ void te_multi_body(cptr<Multi2D<T>> m, const MultiStep st, const int K, const int nw,
                                              const int x0, const int y0, TeLds<T> &lds) {
  const int nx = m->s.nx, ny = m->s.ny, P = m->s.P;
  const int pitch = m->s.pitch, rd = st.rd;
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i = x0 + lane, jb = y0 + wv * R;
  const T ch = m->s.chx, ce_s = m->s.ce_s;
  // unconditional loads from clamped positions (see fdtd_2d_multi.hip)
  const int ic = PX ? min(max(i, 0), nx - 1) : i;
  auto jc = [&](int j) { return PY ? min(max(j, 0), ny - 1) : j; };
  auto ld = [](const T *q, int at) { return ((gptr<const T>)q)[at]; };

  // ------------------------------------------------------------ loads
  T ex[R], ey[R], hz[R + 1];  // hz[r]: row jb - 1 + r
  {
    const T *fx = m->s.ez[rd], *fy = m->s.hx[rd], *fz = m->s.hy[rd];
#pragma unroll
    for (int r = 0; r <= R; ++r) hz[r] = ld(fz + jc(jb - 1 + r) * pitch, ic);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      ex[r] = ld(fx + jc(jb + r) * pitch, ic);
      ey[r] = ld(fy + jc(jb + r) * pitch, ic);
    }
  }
  // update factors, 0 on the walls and outside the grid, where E stays 0
  T cx[R], cy[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int j = jb + r;
    cx[r] = cy[r] = ce_s;
    if (PX) {
      cx[r] = i >= 0 && i <= nx - 2 ? cx[r] : T(0);
      cy[r] = i >= 1 && i <= nx - 2 ? cy[r] : T(0);
    }
    if (PY) {
      cx[r] = j >= 1 && j <= ny - 2 ? cx[r] : T(0);
      cy[r] = j >= 0 && j <= ny - 2 ? cy[r] : T(0);
    }
  }
  // absorber tables and memories: H_z along x (mhx) and y (mhy), E_x along y
  // (mex), E_y along x (mey); zero off their strips
  bool py = false;
  T bxe = T(1), axe = T(0), ikxe = T(1), bxh = T(1), axh = T(0), ikxh = T(1);
  T bye[R], aye[R], ikye[R], byh[R + 1], ayh[R + 1], ikyh[R + 1];
  T mhx[R + 1], mhy[R + 1], mex[R], mey[R];
  if constexpr (PX) {
    bxe = ld(m->s.bxe, ic); axe = ld(m->s.axe, ic); ikxe = ld(m->s.ikxe, ic);
    bxh = ld(m->s.bxh, ic); axh = ld(m->s.axh, ic); ikxh = ld(m->s.ikxh, ic);
    const T *q0 = m->s.pex[rd], *q1 = m->s.phy[rd];
#pragma unroll
    for (int r = 0; r <= R; ++r) mhx[r] = ld(q0 + jc(jb - 1 + r) * pitch, ic);
#pragma unroll
    for (int r = 0; r < R; ++r) mey[r] = ld(q1 + jc(jb + r) * pitch, ic);
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
      mex[r] = ld(q1 + j * pitch, ic);
    }
#pragma unroll
    for (int r = 0; r <= R; ++r) {
      const int j = jc(jb - 1 + r);
      byh[r] = tbh[j]; ayh[r] = tah[j]; ikyh[r] = tih[j];
      mhy[r] = ld(q0 + j * pitch, ic);
    }
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const bool on = (!PX || (i >= 0 && i < nx)) && (!PY || (jb + r >= 0 && jb + r < ny));
    if (PX || PY) {
      ex[r] = on ? ex[r] : T(0);
      ey[r] = on ? ey[r] : T(0);
    }
  }
  const bool ownx = lane >= K && lane < MX - K && i < nx;
  const int row0 = wv * R;
  auto owny = [&](int r) { return row0 + r >= K && row0 + r < R * nw - K && jb + r < ny; };
  // Design and gap edges: family c spans dnx + c columns and dny + 1 - c rows
  // of the box, at density index off(c) + v (dnx + c) + u; the gap likewise.
  const int dnx = m->s.dnx, dny = m->s.dny, gnx = m->s.gnx, gny = m->s.gny, ng = m->s.ng;
  const int dx0 = m->s.dx0, dy0 = m->s.dy0, gx0 = m->s.gx0, gy0 = m->s.gy0;
  const int nd = dnx * (dny + 1) + (dnx + 1) * dny;
  const bool hasgap = gnx > 0 && gny > 0;
  auto lind = [&](int c) { return i >= dx0 && i < dx0 + dnx + c; };
  auto rind = [&](int c, int r) { return jb + r >= dy0 && jb + r < dy0 + dny + 1 - c; };
  auto ling = [&](int c) { return hasgap && i >= gx0 && i < gx0 + gnx + c; };
  auto ring = [&](int c, int r) { return hasgap && jb + r >= gy0 && jb + r < gy0 + gny + 1 - c; };
  auto dcol = [&](int c) { return min(max(i - dx0, 0), dnx + c - 1); };
  auto gcol = [&](int c) { return min(max(i - gx0, 0), max(gnx + c - 1, 0)); };
  auto drow = [&](int c, int r) {
    return (c ? dnx * (dny + 1) : 0) + min(max(jb + r - dy0, 0), dny - c) * (dnx + c);
  };
  auto grow = [&](int c, int r) {
    return (c ? gnx * (gny + 1) : 0) + min(max(jb + r - gy0, 0), gny - c) * (gnx + c);
  };
  TeEdges<T, ADJ, R> D[2];
  T dthJ = T(0), kpm1 = T(0), ga = T(0);
  T *hist = nullptr;
  bool gw = false, staged = false;
  if constexpr (DES) {
    const T *rho = m->s.rho, *Jr = m->J[rd];
    const T A0 = m->s.A0, A1 = m->s.A1, B0 = m->s.B0, B1 = m->s.B1, Sg = m->s.Sg, dt = m->s.dt_, ce_g = m->s.ce_g;
    const T rs = m->s.rs, gsm = m->s.gsm, dtdx = m->s.dtdx;
    hist = st.hist ? (T *)st.hist : m->s.hist;
    gw = hasgap && x0 + MX > gx0 && x0 <= gx0 + gnx && jb + R > gy0 && jb <= gy0 + gny;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      T x[R];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        x[r] = ld(rho + drow(c, r), dcol(c));
        D[c].J[r] = ld(Jr + drow(c, r), dcol(c));
        if constexpr (ADJ) {
          D[c].gacc[r] = ((gptr<const double>)(m->s.grad + drow(c, r)))[dcol(c)];
          D[c].Em[r] = ld(hist + (int64_t)(st.n0 - 1 - st.hist_base) * nd + drow(c, r), dcol(c));
        }
      }
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const bool gap = ling(c) && ring(c, r), drude = lind(c) && rind(c, r) && !gap;
        T &ce = c ? cy[r] : cx[r];
        ce = gap ? ce_g : ce;
        const T eps2 = fma1(x[r], A1, A0);
        const T be = fma1(x[r], B1, B0);
        const T b = fma1(be, dt, Sg * x[r] * (T(1) - x[r]));
        const T inv = T(2) / (eps2 + b);
        ce = drude ? inv : ce;
        D[c].fq[r] = drude ? dtdx : T(1);
        D[c].bs[r] = drude ? b : T(0);
        D[c].beta[r] = drude ? be : T(0);
        D[c].J[r] = drude ? D[c].J[r] : T(0);
        if constexpr (ADJ) {
          D[c].gc[r] = -(T(1) - rs) / (T(2) * (rs + x[r] * (T(1) - rs)));
          D[c].gb[r] = gsm * (T(1) - T(2) * x[r]);
        }
      }
    }
    dthJ = m->s.dthJ;
    kpm1 = m->s.kpm1;
    ga = m->s.ga;
    if constexpr (ADJ) {
      staged = st.steps * ng <= MKMAX * 64;
      if (staged && hasgap && x0 + MX > gx0 && x0 <= gx0 + gnx && y0 + R * nw > gy0 && y0 <= gy0 + gny) {
        for (int q = threadIdx.x; q < st.steps * ng; q += 64 * nw) {
          const int s = q / ng;
          lds.ei[q] = ((gptr<const T>)(m->s.asrc + (int64_t)(st.n0 - s) * ng))[q - s * ng];
        }
        __syncthreads();
      }
    }
  }
  // incident values of the launch's steps: H at the rows beside the vertical
  // lines, E and H at the horizontal ones
  int ja = 0, jt = 0;
  bool tfrow = false, tfcol = false, tfx = false;
  T tcl = T(0);  // E_y at the left line takes -H, at the right line +H
  if constexpr (TF) {
    const int ia = m->s.ia, ib = m->s.ib, jref = m->s.jref, L = m->s.L, ry = R * nw;
    const T *einc = m->s.einc, *hinc = m->s.hinc;
    ja = m->s.ja;
    jt = m->s.jb;
    tfx = i >= ia && i <= ib - 1;
    tcl = i == ia ? T(-1) : i == ib ? T(1) : T(0);
    tfcol = (ia >= x0 && ia < x0 + MX) || (ib >= x0 && ib < x0 + MX);
    auto hit = [&](int v) { return v >= jb - 1 && v < jb + R; };
    tfrow = hit(ja - 1) || hit(ja) || hit(jt);
    if (tfcol)
      for (int q = threadIdx.x; q < st.steps * ry; q += 64 * nw) {
        const int s = q / ry, j = y0 + q - s * ry;
        const bool on = j >= ja && j <= jt - 1;
        const T v = ((gptr<const T>)hinc)[(int64_t)(st.n0 + s) * L + (on ? j - jref : 0)];
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
    T Emn[2][R];
    if constexpr (DES && ADJ) {  // the next step's forward field
      const T *h = hist + (int64_t)(max(n - 1, st.hist_base + 1) - 1 - st.hist_base) * nd;
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int r = 0; r < R; ++r) Emn[c][r] = ld(h + drow(c, r), dcol(c));
    }
    // what H_z's curl reads: E_x and E_y, in the adjoint graded along y and x
    T gx[R], gy[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      gx[r] = ex[r];
      gy[r] = ey[r];
      if constexpr (ADJ && PX) {
        mey[r] = mem1(bxe, mey[r], axe, ey[r]);
        gy[r] = fma1(ey[r], ikxe, mey[r]);
      }
    }
    if constexpr (ADJ && PY) {
      if (py) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
          mex[r] = mem1(bye[r], mex[r], aye[r], ex[r]);
          gx[r] = fma1(ex[r], ikye[r], mex[r]);
        }
      }
    }
    T *xb = lds.x + (s & 1) * (MWMAX * 3 * MX);
    xb[(3 * wv) * MX + lane] = gx[0];
    xb[(3 * wv + 1) * MX + lane] = gx[R - 1];
    xb[(3 * wv + 2) * MX + lane] = gy[R - 1];
    __syncthreads();
    const T gxd = wv > 0 ? xb[(3 * wv - 2) * MX + lane] : T(0);
    const T gyd = wv > 0 ? xb[(3 * wv - 1) * MX + lane] : T(0);
    const T gxu = wv + 1 < nw ? xb[(3 * wv + 3) * MX + lane] : T(0);
    // H_z: dE_y/dx - dE_x/dy
    T dx[R + 1], dy[R + 1];
#pragma unroll
    for (int r = 0; r <= R; ++r) {
      const T g = r > 0 ? gy[r - 1] : gyd;
      dx[r] = lane_right(g) - g;
      dy[r] = (r < R ? gx[r] : gxu) - (r > 0 ? gx[r - 1] : gxd);
      if constexpr (!ADJ && PX) {
        mhx[r] = mem1(bxh, mhx[r], axh, dx[r]);
        dx[r] = fma1(dx[r], ikxh, mhx[r]);
      }
    }
    if constexpr (!ADJ && PY) {
      if (py) {
#pragma unroll
        for (int r = 0; r <= R; ++r) {
          mhy[r] = mem1(byh[r], mhy[r], ayh[r], dy[r]);
          dy[r] = fma1(dy[r], ikyh[r], mhy[r]);
        }
      }
    }
#pragma unroll
    for (int r = 0; r <= R; ++r) hz[r] = fma1(-ch, dx[r] - dy[r], hz[r]);
    T hA = T(0), hB = T(0);
    if constexpr (TF && !ADJ) {
      if (tfrow) {
        const T eA = tfx ? lds.ab[4 * s] : T(0), eB = tfx ? lds.ab[4 * s + 1] : T(0);
        hA = tfx ? lds.ab[4 * s + 2] : T(0);
        hB = tfx ? lds.ab[4 * s + 3] : T(0);
#pragma unroll
        for (int r = 0; r <= R; ++r) {
          if (jb - 1 + r == ja - 1) hz[r] = fma1(-ch, eA, hz[r]);
          if (jb - 1 + r == jt) hz[r] = fma1(ch, eB, hz[r]);
        }
      }
    }
    // what the E curls read: H_z, in the adjoint graded along x and y
#pragma unroll
    for (int r = 0; r <= R; ++r) {
      dx[r] = dy[r] = hz[r];
      if constexpr (ADJ && PX) {
        mhx[r] = mem1(bxh, mhx[r], axh, hz[r]);
        dx[r] = fma1(hz[r], ikxh, mhx[r]);
      }
    }
    if constexpr (ADJ && PY) {
      if (py) {
#pragma unroll
        for (int r = 0; r <= R; ++r) {
          mhy[r] = mem1(byh[r], mhy[r], ayh[r], hz[r]);
          dy[r] = fma1(hz[r], ikyh[r], mhy[r]);
        }
      }
    }
    // curls: E_x dH_z/dy, E_y -dH_z/dx
    T ux[R], uy[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      ux[r] = dy[r + 1] - dy[r];
      uy[r] = dx[r + 1] - lane_left(dx[r + 1]);
      if constexpr (!ADJ && PX) {
        mey[r] = mem1(bxe, mey[r], axe, uy[r]);
        uy[r] = fma1(uy[r], ikxe, mey[r]);
      }
      uy[r] = -uy[r];
    }
    if constexpr (!ADJ && PY) {
      if (py) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
          mex[r] = mem1(bye[r], mex[r], aye[r], ux[r]);
          ux[r] = fma1(ux[r], ikye[r], mex[r]);
        }
      }
    }
    if constexpr (TF && !ADJ) {
      if (tfrow) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
          if (jb + r == ja) ux[r] += hA;
          if (jb + r == jt) ux[r] -= hB;
        }
      }
      if (tfcol) {
#pragma unroll
        for (int r = 0; r < R; ++r) uy[r] = fma1(tcl, lds.ei[s * (R * nw) + row0 + r], uy[r]);
      }
    }
    if constexpr (DES && ADJ) {
      if (gw) {  // the adjoint source
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
          for (int r = 0; r < R; ++r)
            if (ring(c, r)) {
              const T v = staged ? lds.ei[s * ng + grow(c, r) + gcol(c)]
                                 : ld(m->s.asrc + (int64_t)n * ng + grow(c, r), gcol(c));
              T &u = c ? uy[r] : ux[r];
              u = ling(c) ? u + v : u;
            }
      }
    }
    // E and J
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int r = 0; r < R; ++r) {
        T &e = c ? ey[r] : ex[r];
        const T u = c ? uy[r] : ux[r], ce = c ? cy[r] : cx[r];
        if constexpr (!DES) {
          e = fma1(ce, u, e);
        } else {
          const T e0 = e, Jo = D[c].J[r];
          const T q = fma1(-D[c].bs[r], e0, fma1(D[c].fq[r], u, -(dthJ * Jo)));
          const T e1 = fma1(ce, q, e0);
          const T Jn = Jo + fma1(kpm1, Jo, D[c].beta[r] * (e0 + e1));
          D[c].J[r] = Jn;
          e = e1;
          if constexpr (ADJ) {  // (stored on the Drude edges only)
            const T t = fma1(D[c].gc[r], Jn + Jo, fma1(ga, ce * q, D[c].gb[r] * (e0 + e1)));
            D[c].gacc[r] = sens1(D[c].gacc[r], D[c].Em[r], t);
            D[c].Em[r] = Emn[c][r];
          }
        }
      }
    if constexpr (DES && !ADJ) {
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        if (st.hist_on && ownx && lind(c)) {
          T *h = hist + (int64_t)(n - st.hist_base) * nd;
#pragma unroll
          for (int r = 0; r < R; ++r)
            if (owny(r) && rind(c, r)) ((gptr<T>)(h + drow(c, r)))[dcol(c)] = c ? ey[r] : ex[r];
        }
        if (gw && ownx && ling(c)) {
          double *g = m->s.gapE + (int64_t)(n + 1) * ng;
#pragma unroll
          for (int r = 0; r < R; ++r)
            if (owny(r) && ring(c, r)) ((gptr<double>)(g + grow(c, r)))[gcol(c)] = (double)(c ? ey[r] : ex[r]);
        }
      }
    }
  }

  // ------------------------------------------------------------ stores
  asm volatile("" : "+s"(m));  // the write pointers are read here, not kept over the steps
  const int wr = rd ^ 1;
  auto put = [&](T *q, int r, T v) { ((gptr<T>)(q + (int64_t)(jb + r) * pitch))[i] = v; };
  if (ownx) {
    T *fx = m->s.ez[wr], *fy = m->s.hx[wr], *fz = m->s.hy[wr];
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (owny(r)) {
        put(fx, r, ex[r]);
        put(fy, r, ey[r]);
        put(fz, r, hz[r + 1]);
      }
  }
  if constexpr (PX) {
    T *q0 = m->s.pex[wr], *q1 = m->s.phy[wr];
    if (ownx && pml_h2(i, nx, P))
#pragma unroll
      for (int r = 0; r < R; ++r)
        if (owny(r)) put(q0, r, mhx[r + 1]);
    if (ownx && pml_e2(i, nx, P))
#pragma unroll
      for (int r = 0; r < R; ++r)
        if (owny(r)) put(q1, r, mey[r]);
  }
  if constexpr (PY) {
    if (py && ownx) {
      T *q0 = m->s.pey[wr], *q1 = m->s.phx[wr];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        if (owny(r) && pml_h2(jb + r, ny, P)) put(q0, r, mhy[r + 1]);
        if (owny(r) && pml_e2(jb + r, ny, P)) put(q1, r, mex[r]);
      }
    }
  }
  if constexpr (DES) {
    T *Jw = m->J[wr];
#pragma unroll
    for (int c = 0; c < 2; ++c)
      if (ownx && lind(c)) {
#pragma unroll
        for (int r = 0; r < R; ++r)
          if (owny(r) && rind(c, r) && !(ling(c) && ring(c, r))) {
            ((gptr<T>)(Jw + drow(c, r)))[dcol(c)] = D[c].J[r];
            if constexpr (ADJ) ((gptr<double>)(m->s.grad + drow(c, r)))[dcol(c)] = D[c].gacc[r];
          }
      }
  }
}

// Which body a region needs follows from what its nodes touch.
template <typename T, bool ADJ, int R>
__global__ void __launch_bounds__(64 * MWMAX)
    step_te_multi(const Multi2D<T> *mp, const MultiStep st, const MultiTile g) {
  __shared__ TeLds<T> lds;
  const cptr<Multi2D<T>> m = (cptr<Multi2D<T>>)mp;
  const int nx = m->s.nx, ny = m->s.ny, P = m->s.P;
  const int K = g.K, nw = g.nw, W = MX - 2 * K, ntx = (nx + W - 1) / W;
  const int x0 = (blockIdx.x % ntx) * W - K, y0 = (blockIdx.x / ntx) * (R * nw - 2 * K) - K;
  const int x1 = x0 + MX - 1, y1 = y0 + R * nw - 1;
  const bool px = x0 < P + 1 || x1 > nx - 3 - P, py = y0 < P + 1 || y1 > ny - 3 - P;
  auto hit = [](int lo, int hi, int v) { return v >= lo && v <= hi; };
  bool tf = false;
  if (!ADJ && m->s.tf_on) {
    const int ia = m->s.ia, ib = m->s.ib, ja = m->s.ja, jt = m->s.jb;
    tf = hit(x0, x1, ia) || hit(x0, x1, ib) || hit(y0 - 1, y1, ja - 1) || hit(y0, y1, ja) || hit(y0 - 1, y1, jt);
  }
  // a box of bnx x bny cells: nodes bx .. bx + bnx, by .. by + bny
  auto meets = [&](int bx, int by, int bnx, int bny) {
    return bnx > 0 && bny > 0 && x1 >= bx && x0 <= bx + bnx && y1 >= by && y0 <= by + bny;
  };
  const bool des = meets(m->s.dx0, m->s.dy0, m->s.dnx, m->s.dny) || meets(m->s.gx0, m->s.gy0, m->s.gnx, m->s.gny);
  constexpr bool F = !ADJ;
  if (des) {
    if (px || py || tf) te_multi_body<T, ADJ, true, true, F, true, R>(m, st, K, nw, x0, y0, lds);
    else te_multi_body<T, ADJ, false, false, false, true, R>(m, st, K, nw, x0, y0, lds);
  } else if (F && tf) {
    te_multi_body<T, ADJ, true, true, F, false, R>(m, st, K, nw, x0, y0, lds);
  } else {
    if (px && py) te_multi_body<T, ADJ, true, true, false, false, R>(m, st, K, nw, x0, y0, lds);
    else if (px) te_multi_body<T, ADJ, true, false, false, false, R>(m, st, K, nw, x0, y0, lds);
    else if (py) te_multi_body<T, ADJ, false, true, false, false, R>(m, st, K, nw, x0, y0, lds);
    else te_multi_body<T, ADJ, false, false, false, false, R>(m, st, K, nw, x0, y0, lds);
  }
}

}  // namespace

// Regions by size, as in fdtd_2d_multi.hip: the flattest that one round of the
// 256 CUs holds; beyond that 64 x 32 regions with fewer halo nodes, on half the
// wavefronts once the work per node counts more than the adjoint's spilled
// registers (91 in FP32 with R = 4; compiled without spills for 8 wavefronts at
// most the 2048^2 adjoint takes 13.1 us instead of 8.9).  us per forward / adjoint
// step (R, nw, K):
//   FP32  256^2: 2,16,10 1.30 / 1.58; 2,16,8 1.46 / 1.70
//         384^2: 2,16,10 1.78 / 1.59; 2,16,8 1.51 / 1.75; 4,8,8 1.92 / 2.29
//         700^2: 2,16,8  3.07 / 2.52; 4,8,8 2.56 / 3.31
//        1024^2: 2,16,8  5.19 / 4.39; 4,8,8 3.70 / 3.68; 4,16,8 3.58 / 3.89
//   FP64  256^2: 2,16,10 1.58 / 2.31; 2,16,8 1.77 / 2.46
//         700^2: 2,16,8  3.85 / 3.45; 2,16,6 3.91 / 3.69; 4,8,8 4.20 / 10.1
//        1024^2: 2,16,8  6.68 / 6.14; 2,16,6 6.34 / 6.01
// (the per-step kernels: 384^2 FP32 11.7 / 13.4, 1024^2 about 18.5).
MultiTile multi_te_tile(int nx, int ny, int precision) {
  const int64_t nodes = (int64_t)nx * ny;
  if (multi_regions(nx, ny, {2, 16, 10}) <= 256) return {2, 16, 10};
  if (precision == 64) return nodes < 800000 ? MultiTile{2, 16, 8} : MultiTile{2, 16, 6};
  return nodes < 500000 ? MultiTile{2, 16, 8} : MultiTile{4, 8, 8};
}

template <typename T>
void launch_step_te_multi(const Multi2D<T> *m, int nx, int ny, int n0, int steps, const MultiTile &g, int rd,
                          bool adjoint, void *hist, int hist_base, int hist_on, hipStream_t s) {
  const MultiStep st{n0, steps, rd, hist, hist_base, hist_on};
  const dim3 grid(multi_regions(nx, ny, g)), block(64 * g.nw);
  if (sizeof(T) == 8 || g.R == 2) {
    if (adjoint) hipLaunchKernelGGL((step_te_multi<T, true, 2>), grid, block, 0, s, m, st, g);
    else hipLaunchKernelGGL((step_te_multi<T, false, 2>), grid, block, 0, s, m, st, g);
  } else if constexpr (sizeof(T) == 4) {
    if (adjoint) hipLaunchKernelGGL((step_te_multi<T, true, 4>), grid, block, 0, s, m, st, g);
    else hipLaunchKernelGGL((step_te_multi<T, false, 4>), grid, block, 0, s, m, st, g);
  }
}

template void launch_step_te_multi<float>(const Multi2D<float> *, int, int, int, int, const MultiTile &, int, bool,
                                          void *, int, int, hipStream_t);
template void launch_step_te_multi<double>(const Multi2D<double> *, int, int, int, int, const MultiTile &, int, bool,
                                           void *, int, int, hipStream_t);

}  // namespace fdtd
