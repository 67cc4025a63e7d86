// af_scheme2d.hpp -- the pieces of the 2D stage that its kernels share: site
// and cell data, the limited face flux and the wall projection.  Kernels that
// evaluate the same expression of the same values round alike (multiply-adds
// are fused within one expression only), so all of them give the same bits.
#pragma once

#include <type_traits>

#include "af_device.hpp"
#include "af_internal.hpp"
#include "af_lattice.hpp"

namespace afd {

// (u, v, p, T, c) of state V, given 1/rho
template <typename R>
__device__ __forceinline__ void aux_of(const PhysT<R>& ph, const R* V, R ir, R* w) {
  const R p = ph.gm1 * (V[3] - R(0.5) * (V[1] * V[1] + V[2] * V[2]) * ir);
  w[0] = V[1] * ir;
  w[1] = V[2] * ir;
  w[2] = p;
  w[3] = p * ir;
  w[4] = root(ph.gam * w[3]);
}

// Simpson centre value from the cell average, the sum of the four edge
// points and the sum of the four corners (Sec. 2.2), scaled toward the
// average with the density-then-pressure rule when the centre limiter is on,
// and its (u, v, p, T, c).  A centre whose density and pressure are already
// at least eps keeps its value: the rule's parameter is 1 there (the rule is
// continuous at that threshold, so only round-off separates the two
// evaluations of the test).  The rule itself runs in FP64.
template <typename R>
__device__ __forceinline__ void centre_value(const PhysT<R>& ph, const Phys& phd, const R* Ub,
                                             const R* e, const R* c, R* V, R* w) {
#pragma unroll
  for (int k = 0; k < 4; ++k) V[k] = (R(36.0) * Ub[k] - R(4.0) * e[k] - c[k]) / R(16.0);
  R ir = rcp(V[0]);
  const R p = ph.gm1 * (V[3] - R(0.5) * (V[1] * V[1] + V[2] * V[2]) * ir);
  if ((ph.lim & LIM_CENTRE) && !(Ub[0] > R(0.0) && V[0] >= R(kPPEps) && p >= R(kPPEps))) {
    if (!(Ub[0] > R(0.0))) {
#pragma unroll
      for (int k = 0; k < 4; ++k) V[k] = Ub[k];
    } else {
      double Ud[4], Vd[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        Ud[k] = Ub[k];
        Vd[k] = V[k];
      }
      bool bad = false;
      const double th = theta_pair2(Ud, Vd, phd.gm1, bad, ph.lim & LIM_PEXACT);
      if (th < 1.0) {
        double Wd[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          Wd[k] = Ud[k] + th * (Vd[k] - Ud[k]);
          V[k] = R(Wd[k]);
        }
        if constexpr (!std::is_same<R, double>::value) {
          // FP32 stencils: the scaled centre's pressure may sit at eps, far
          // below the rounding of E - |m|^2 / (2 rho) in FP32, so its
          // (u, v, p, T, c) are taken from the FP64 value
          const double ird = rcp(Wd[0]);
          const double pd = phd.gm1 * (Wd[3] - 0.5 * (Wd[1] * Wd[1] + Wd[2] * Wd[2]) * ird);
          w[0] = R(Wd[1] * ird);
          w[1] = R(Wd[2] * ird);
          w[2] = R(pd);
          w[3] = R(pd * ird);
          w[4] = R(root(phd.gam * (pd * ird)));
          return;
        }
      }
    }
    ir = rcp(V[0]);
  }
  aux_of(ph, V, ir, w);
}

// (u, v, p, T, c) in R of the FP64 value V
template <typename R>
__device__ __forceinline__ void aux_of_fp64(const PhysT<double>& pd, const double* V, R* w) {
  const double ir = rcp(V[0]);
  const double p = pd.gm1 * (V[3] - 0.5 * (V[1] * V[1] + V[2] * V[2]) * ir);
  const double Tt = p * ir;
  w[0] = R(V[1] * ir);
  w[1] = R(V[2] * ir);
  w[2] = R(p);
  w[3] = R(Tt);
  w[4] = R(root(pd.gam * Tt));
}

// pressure of state V, given 1/rho
template <typename R>
__device__ __forceinline__ R pressure_r(const PhysT<R>& ph, const R* V, R ir) {
  return ph.gm1 * (V[3] - R(0.5) * (V[1] * V[1] + V[2] * V[2]) * ir);
}

// per-cell low-order data (Sec. 3.1):
//   o[0..3] F_x, o[4..7] F_y (total fluxes with S = central differences of
//   Z(average)), o[8] |u|+c, o[9] |v|+c, o[10] b_x, o[11] b_y, from the
//   averages of the cell, with its sound speed c0, and of its four neighbours
//   (ghost cells as boundary images)
//
// A cell average with its reciprocal density and pressure: neighbours enter
// by their momenta, 1/rho and p.
template <typename R>
struct CellAvg {
  R U[4], r, p;
};

// smoothness sensors phi1, phi2 of a cell (Sec. 3.2)
template <typename R>
__device__ __forceinline__ void cell_sensors(const G2& g, const CellAvg<R>& a0,
                                             const CellAvg<R>& xm, const CellAvg<R>& xp,
                                             const CellAvg<R>& ym, const CellAvg<R>& yp, R* phi) {
  const R *Cxm = xm.U, *Cxp = xp.U, *Cym = ym.U, *Cyp = yp.U;
  const R rxm = xm.r, rxp = xp.r, rym = ym.r, ryp = yp.r;
  const R p0 = a0.p, pxm = xm.p, pxp = xp.p, pym = ym.p, pyp = yp.p;
  const R i2x = R(1.0 / (2.0 * g.dx)), i2y = R(1.0 / (2.0 * g.dy));
  const R ux = (Cxp[1] * rxp - Cxm[1] * rxm) * i2x;
  const R vx = (Cxp[2] * rxp - Cxm[2] * rxm) * i2x;
  const R uy = (Cyp[1] * ryp - Cym[1] * rym) * i2y;
  const R vy = (Cyp[2] * ryp - Cym[2] * rym) * i2y;
  const R jx = fabs(pxp - R(2.0) * p0 + pxm) / fabs(pxp + R(2.0) * p0 + pxm);
  const R jy = fabs(pyp - R(2.0) * p0 + pym) / fabs(pyp + R(2.0) * p0 + pym);
  phi[0] = mx(jx, jy);
  const R div = ux + vy, curl = vx - uy;
  phi[1] = mx(-div / root(div * div + curl * curl + R(kDucros)), R(0.0));
}
template <typename R>
__device__ __forceinline__ void cell_low(const G2& g, const PhysT<R>& ph, const CellAvg<R>& a0,
                                         const CellAvg<R>& xm, const CellAvg<R>& xp,
                                         const CellAvg<R>& ym, const CellAvg<R>& yp, R c0, R* o) {
  const R *C0 = a0.U, *Cxm = xm.U, *Cxp = xp.U, *Cym = ym.U, *Cyp = yp.U;
  const R r0 = a0.r, rxm = xm.r, rxp = xp.r, rym = ym.r, ryp = yp.r;
  const R p0 = a0.p, pxm = xm.p, pxp = xp.p, pym = ym.p, pyp = yp.p;
  const R u0 = C0[1] * r0, v0 = C0[2] * r0;
  const R i2x = R(1.0 / (2.0 * g.dx)), i2y = R(1.0 / (2.0 * g.dy));
  const R ux = (Cxp[1] * rxp - Cxm[1] * rxm) * i2x;
  const R vx = (Cxp[2] * rxp - Cxm[2] * rxm) * i2x;
  const R Tx = (pxp * rxp - pxm * rxm) * i2x;
  const R uy = (Cyp[1] * ryp - Cym[1] * rym) * i2y;
  const R vy = (Cyp[2] * ryp - Cym[2] * rym) * i2y;
  const R Ty = (pyp * ryp - pym * rym) * i2y;
  R Fv[4];
  visc_flux2(0, u0, v0, ux, vx, Tx, uy, vy, Ty, ph, Fv);
  o[0] = C0[1] - Fv[0];
  o[1] = C0[1] * u0 + p0 - Fv[1];
  o[2] = C0[2] * u0 - Fv[2];
  o[3] = (C0[3] + p0) * u0 - Fv[3];
  visc_flux2(1, u0, v0, ux, vx, Tx, uy, vy, Ty, ph, Fv);
  o[4] = C0[2] - Fv[0];
  o[5] = C0[1] * v0 - Fv[1];
  o[6] = C0[2] * v0 + p0 - Fv[2];
  o[7] = (C0[3] + p0) * v0 - Fv[3];
  o[8] = fabs(u0) + c0;
  o[9] = fabs(v0) + c0;
  bvisc2_xy(p0, p0 * r0, ux, vx, Tx, uy, vy, Ty, ph, o[10], o[11]);
}

// total flux F_d = F^c_d - F^v_d of state (m1, m2, E) with velocity (u, v),
// pressure p and gradients gr = (u_x, v_x, T_x, u_y, v_y, T_y)
template <typename R>
__device__ __forceinline__ void tot_flux(int d, const R* U, R u, R v, R p, const R* gr,
                                         const PhysT<R>& ph, R* F) {
  R Fv[4];
  visc_flux2(d, u, v, gr[0], gr[1], gr[2], gr[3], gr[4], gr[5], ph, Fv);
  const R ud = d == 0 ? u : v;
  F[0] = U[1 + d] - Fv[0];
  F[1] = U[1] * ud + (d == 0 ? p : R(0.0)) - Fv[1];
  F[2] = U[2] * ud + (d == 1 ? p : R(0.0)) - Fv[2];
  F[3] = (U[3] + p) * ud - Fv[3];
}

// direction-D terms of the residual of a point, from the five sites of its line:
// the biased inviscid operators as central difference plus dissipation with
// alpha, compact D^{(d),2}(K_dd, Z), and the mixed terms from the derivatives
// across D of the velocities (ga along D, gb the other one; index 2 unused).
// at(v, o): value v of site o, in the line's frame: density, momentum along D
// and across, energy, velocity along D and across, pressure, temperature.  Rr:
// density, momentum along D and across, energy.
//
// Every factor is applied at its site.  With the constants after the differences
// and the form of B from differences the sum takes 120 of 3100 operations per row
// of a strip less (the stage at 2048 x 1024 351 us instead of 357, FP32 stencils
// 264 instead of 270), but rounds otherwise.  A step with FP32 stencils moves by up
// to 7e-9 of a smooth flow's state, a third of its distance from 64 bits.  One in
// FP64 moves by 4e-17, which was enough to keep SSP-RK54 in the opening transient of
// the 1000 x 500 tube: from t = 3.5e-4 on every step was halved some 36 times.
enum LineValue { kRho, kMd, kMo, kE, kVa, kVb, kP, kT };
template <typename R, typename At>
__device__ __forceinline__ void line_terms(const PhysT<R>& ph, double h, R alpha, At at,
                                           const R* ga, const R* gb, R* Rr) {
  const R i6h = R(1.0 / (6.0 * h));
  const R ai = alpha * i6h;
  R va[5], vb[5], Tt[5];
#pragma unroll
  for (int o = 0; o < 5; ++o) {
    va[o] = at(kVa, o);
    vb[o] = at(kVb, o);
    Tt[o] = at(kT, o);
  }
  // inviscid, one component at a time (short live ranges)
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    R f[5], w[5];
#pragma unroll
    for (int o = 0; o < 5; ++o) {
      w[o] = at(k == 0 ? kRho : (k == 1 ? kMd : (k == 2 ? kMo : kE)), o);
      f[o] = k == 0 ? at(kMd, o)
                    : (k == 1 ? w[o] * va[o] + at(kP, o)
                              : (k == 2 ? w[o] * va[o] : (w[o] + at(kP, o)) * va[o]));
    }
    Rr[k] = -(dc5(f[0], f[1], f[3], f[4], i6h) + ai * d4(w[0], w[1], w[2], w[3], w[4]));
  }
  // compact D^{(d),2}(K_dd, Z)
  const R s4 = R(4.0 / (h * h));
  const R mu = ph.mu, m43 = R(4.0 / 3.0) * ph.mu;
  Rr[1] += s4 * m43 * bcol(va);
  Rr[2] += s4 * mu * bcol(vb);
  Rr[3] += s4 * (m43 * bquad(va) + mu * bquad(vb) + ph.kap * bcol(Tt));
  // mixed
  R m1[5], m2[5], m3[5];
#pragma unroll
  for (int o = 0; o < 5; ++o) {
    if (o == 2) {
      m1[o] = m2[o] = m3[o] = R(0.0);
      continue;
    }
    m1[o] = -R(2.0 / 3.0) * mu * gb[o];
    m2[o] = mu * ga[o];
    m3[o] = mu * (vb[o] * ga[o] - R(2.0 / 3.0) * va[o] * gb[o]);
  }
  Rr[1] += dc5(m1[0], m1[1], m1[3], m1[4], i6h);
  Rr[2] += dc5(m2[0], m2[1], m2[3], m2[4], i6h);
  Rr[3] += dc5(m3[0], m3[1], m3[3], m3[4], i6h);
}

// wall projection of a point value (no-slip: zero momentum; symmetry: zero
// normal momentum; density and internal energy kept)
__device__ __forceinline__ void project(int kind, int ax, double* V) {
  if (kind == BC_NOSLIP) {
    V[3] -= (V[1] * V[1] + V[2] * V[2]) / (2.0 * V[0]);
    V[1] = 0.0;
    V[2] = 0.0;
  } else if (kind == BC_SYMMETRY) {
    V[3] -= V[1 + ax] * V[1 + ax] / (2.0 * V[0]);
    V[1 + ax] = 0.0;
  }
}

__device__ __forceinline__ int wall_of(int bc) {
  return (bc == BC_NOSLIP || bc == BC_SYMMETRY) ? bc : -1;
}

// what the limiter of a face reads of its cells a (minus) and b (plus): the
// FP64 averages, the low-order cell fluxes along the face's axis, the LLF
// flux, and the larger of the two cells' sensors
template <typename R>
struct FaceCells {
  double Ua[4], Ub[4];
  R Fa[4], Fb[4], FL[4], phi1, phi2;
};

// limited flux of face (i, j) of direction d (Sec. 3.2, 3.3) from its
// high-order flux FH.  blend: a coefficient per face that takes the place of
// theta^s, or NULL; ts_out: receives the coefficient used in its place per
// face, or NULL.  own: the face belongs to this workgroup (others are computed
// along, raise no flag and write nothing).  low: the flag raised where a low-order
// state is inadmissible.
template <typename R>
__device__ __forceinline__ void limit_face(const G2& g, const PhysT<R>& ph, const Phys& phd, int d,
                                           int i, int j, double dt, const FaceCells<R>& c,
                                           const R* FH, const float* blend, float* ts_out, bool own,
                                           unsigned* flags, unsigned low, R* F) {
  R ts = R(1.0);
  double tpp = 1.0;
  // the face's entries in per-face arrays: x-faces [n2][n1+1], then
  // y-faces [n2+1][n1]; a periodic axis's last face is its first again
  const bool use_blend = blend != nullptr;
  if (ph.lim & LIM_LOWONLY) {
    ts = R(0.0);
    tpp = 0.0;
  } else {
    if (use_blend) {
      // the given coefficient takes the place of theta^s
      const long nfx = (long)g.n2 * (g.n1 + 1);
      const int fi = (d == 0 && i == g.n1 && g.n1x == g.n1) ? 0 : i;
      const int fj = (d == 1 && j == g.n2 && g.n2y == g.n2) ? 0 : j;
      if (own) ts = R(blend[d == 0 ? (long)fj * (g.n1 + 1) + fi : nfx + (long)fj * g.n1 + fi]);
    } else if (ph.lim & LIM_SMOOTH) {
      ts = exp(-ph.Cs * c.phi1 * c.phi2);
    }
    if (ph.lim & LIM_PP) {
      // the density and pressure blend in FP64 (Sec. 3.3)
      const double m4 = 4.0 * dt / (d == 0 ? g.dx : g.dy);
      double ULp[4], UHp[4], ULm[4], UHm[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const double fl = c.FL[k], fh = FH[k], fca = c.Fa[k], fcb = c.Fb[k];
        const double Fs = fl + double(ts) * (fh - fl);
        ULp[k] = c.Ua[k] - m4 * (fl - fca);
        UHp[k] = c.Ua[k] - m4 * (Fs - fca);
        ULm[k] = c.Ub[k] - m4 * (fcb - fl);
        UHm[k] = c.Ub[k] - m4 * (fcb - Fs);
      }
      bool bad = false;
      const double pLp = pressure2(ULp[0], ULp[1], ULp[2], ULp[3], phd.gm1);
      const double pLm = pressure2(ULm[0], ULm[1], ULm[2], ULm[3], phd.gm1);
      if (keeps(ULp[0], pLp, UHp[0], pressure2(UHp[0], UHp[1], UHp[2], UHp[3], phd.gm1)) &&
          keeps(ULm[0], pLm, UHm[0], pressure2(UHm[0], UHm[1], UHm[2], UHm[3], phd.gm1))) {
        tpp = 1.0;  // as almost everywhere: see theta_pair2
      } else if (!(ULp[0] > 0.0) || !(ULm[0] > 0.0)) {
        tpp = 0.0;
        bad = true;
      } else {
        if (!(pLp > 0.0) || !(pLm > 0.0)) bad = true;
        const double tr = mn(theta_lin(ULp[0], UHp[0], mn(kPPEps, ULp[0])),
                             theta_lin(ULm[0], UHm[0], mn(kPPEps, ULm[0])));
        double Tp[4], Tm[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          Tp[k] = ULp[k] + tr * (UHp[k] - ULp[k]);
          Tm[k] = ULm[k] + tr * (UHm[k] - ULm[k]);
        }
        const bool ex = ph.lim & LIM_PEXACT;
        const double tp = mn(theta_p2(ULp, pLp, Tp, mn(kPPEps, pLp), phd.gm1, ex),
                             theta_p2(ULm, pLm, Tm, mn(kPPEps, pLm), phd.gm1, ex));
        tpp = tr * tp;
      }
      if (bad && own) raise_flag(flags, low);
    }
  }
  const double th = double(ts) * tpp;
  if (ts_out && own) {
    const long nfx = (long)g.n2 * (g.n1 + 1);
    ts_out[d == 0 ? (long)j * (g.n1 + 1) + i : nfx + (long)j * g.n1 + i] = float(ts);
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const double fl = c.FL[k], fh = FH[k];
    F[k] = R(fl + th * (fh - fl));
  }
}

}  // namespace afd
