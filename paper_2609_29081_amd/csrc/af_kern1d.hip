// af_kern1d.hip -- the 1D compact AF method (Sec. 2.1) on gfx950, FP64: one
// SSP-RK3 stage as one launch, and a whole step (SSP-RK3 or SSP-RK54) as one.
// Same pipeline as the 2D stage (lattice, gradients, per-cell low-order data,
// limited face fluxes, cell update, point update), with U = (rho, rho u, E),
// W = (rho, u, p), Z = (0, u, T) and
//   K(W) = [[0,0,0],[0,4mu/3,0],[0,4mu u/3,kappa]].
//
// The 1D problems are small (hundreds of cells), so a stage is bound by
// latency: launches, loads, and the chain of dependent FP64 operations.  A
// workgroup of three wave64s takes 61 cells and the points at their lower
// sides, and passes everything through LDS:
//   before a barrier  waves 0-1 one lattice site each (values, centres,
//                     primitives), wave 2 one cell each of the tile +- 1
//                     (low-order data)
//   after it          wave 0 one face each (limited flux), whose neighbours'
//                     fluxes come by a lane shift to the cell update; wave 1
//                     one point each
// 61 cells are the most for which sites (2 x 61 + 5), ring cells (63) and
// faces (62) fit one per lane.
//
// A step keeps its tile in LDS from stage to stage.  A stage's values depend
// on two cells at either side, so a tile's outer cells are computed along with
// those of its neighbours, two fewer at either side in each stage: 61 - 8 cells
// of a tile are its own in SSP-RK3, 61 - 16 in SSP-RK54.  That is 1.15 and 1.36
// times the work, and one launch, one read and one write of the state instead
// of three or five: a step of a run of 800 cells took 21.7 us with a launch per
// stage and takes 15.1, one of SSP-RK54 at 160 cells (af_step) 62 and 36.5.  The
// step kernel takes 197 VGPRs and spills 49 scalar registers (into lanes of
// vector ones, no memory): its arguments are held across the stages.
#include "af_device.hpp"
#include "af_internal.hpp"

using namespace afd;

namespace {

constexpr int kCells = 61, kThreads = 192;
constexpr int kSites = 2 * kCells + 5, kRing = kCells + 2;
static_assert(kSites <= 128 && kRing <= 64, "one site and one ring cell per lane");

struct G1 {
  int n, np;
  long off_pts;
  int bc0, bc1;
  double dx;
  double dl[3], dr[3];  // states of Dirichlet sides (x-low, x-high)
};

// a stage's launch (see StageCoef)
struct Stage1 {
  double ca, cb;
  int first, skip_flagged, stage;
  unsigned* flags;
  const double* dt_dev;
  double dt_host, dt_mul;
};

// a step's launch: its stages out = ca base + cb FE(in, mul dt), where base is
// the step's first state but in the last stage of SSP-RK54 (see rk54)
struct Step1 {
  int stages;
  double ca[5], cb[5], mul[5];
  double wa, wb, ga, gb;  // SSP-RK54's shared evaluation
  unsigned* flags;
  const double* dt_dev;
  double dt_host;
  afi::StepExtras1 x;
};

// the state a stage reads: in global memory, its ghosts the images of what
// axis_image says ...
struct Global1 {
  const double* __restrict__ U;
  __device__ __forceinline__ int image(const G1& g, int X, int& kind) const {
    return axis_image(X, 2 * g.n, g.bc0, g.bc1, kind);
  }
  __device__ __forceinline__ double cell(const G1& g, int i, int k) const {
    return U[(long)k * g.n + i];
  }
  __device__ __forceinline__ double point(const G1& g, int j, int k) const {
    if (j == g.n && g.np == g.n) j = 0;
    return U[g.off_pts + (long)k * g.np + j];
  }
};
// ... or in LDS: cells b - 2 .. b + 62 and points b - 1 .. b + 62, continued
// beyond periodic sides
struct Held1 {
  double C[3][kCells + 4], P[3][kCells + 3];
  int b;
  __device__ __forceinline__ int image(const G1& g, int X, int& kind) const {
    kind = -1;
    return g.bc0 == BC_PERIODIC ? X : axis_image(X, 2 * g.n, g.bc0, g.bc1, kind);
  }
  __device__ __forceinline__ double cell(const G1&, int i, int k) const { return C[k][i - b + 2]; }
  __device__ __forceinline__ double point(const G1&, int j, int k) const { return P[k][j - b + 1]; }
};

template <typename Src>
__device__ __forceinline__ void cell_image1(const G1& g, const Src& U, int i, double* V) {
  // beyond a Dirichlet side, its state
  if ((i < 0 && g.bc0 == BC_DIRICHLET) || (i >= g.n && g.bc1 == BC_DIRICHLET)) {
    const double* d = i < 0 ? g.dl : g.dr;
#pragma unroll
    for (int k = 0; k < 3; ++k) V[k] = d[k];
    return;
  }
  int kind;
  const int Xi = U.image(g, 2 * i + 1, kind);
  const double s = (kind == BC_NOSLIP || kind == BC_SYMMETRY) ? -1.0 : 1.0;
  const int ii = Xi >> 1;
  V[0] = U.cell(g, ii, 0);
  V[1] = s * U.cell(g, ii, 1);
  V[2] = U.cell(g, ii, 2);
}

// data of a tile in LDS
struct Tile1 {
  double U[3][kSites];   // lattice values (centres: Simpson, scaled)
  double A[4][kSites];   // u, p, T, c
  // cells of the tile +- 1: 0-2 F, 3 rs, 4 b, 5 phi1, 6 phi2, 7-9 average
  double C[10][kRing];
  double red[2][kThreads / 64];
  unsigned stop;
};

// velocity, pressure and temperature of a state, from one reciprocal: in a chain
// of dependent operations a division is three times as long
struct Prim1 {
  double u, p, T;
};
__device__ __forceinline__ Prim1 prim1(const Phys& ph, const double* V) {
  const double ir = rcp(V[0]), u = V[1] * ir, p = ph.gm1 * (V[2] - V[1] * V[1] * (0.5 * ir));
  return Prim1{u, p, p * ir};
}

// lattice site X into tile entry t
template <typename Src>
__device__ __forceinline__ void lattice_site(const G1& g, const Phys& ph, const Src& U, int X,
                                             int t, Tile1& S) {
  int kind;
  const int Xi = U.image(g, X, kind);
  const double s = (kind == BC_NOSLIP || kind == BC_SYMMETRY) ? -1.0 : 1.0;
  double V[3];
  if (Xi & 1) {
    const int i = Xi >> 1;
    double Ub[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      Ub[k] = U.cell(g, i, k);
      V[k] = (6.0 * Ub[k] - (U.point(g, i, k) + U.point(g, i + 1, k))) / 4.0;
    }
    if (ph.lim & LIM_CENTRE) {
      if (!(Ub[0] > 0.0)) {
#pragma unroll
        for (int k = 0; k < 3; ++k) V[k] = Ub[k];
      } else {
        bool bad = false;
        const double th = theta_pair1(Ub, V, ph.gm1, bad, ph.lim & LIM_PEXACT);
        if (th < 1.0) {
#pragma unroll
          for (int k = 0; k < 3; ++k) V[k] = Ub[k] + th * (V[k] - Ub[k]);
        }
      }
    }
  } else {
#pragma unroll
    for (int k = 0; k < 3; ++k) V[k] = U.point(g, Xi >> 1, k);
  }
  V[1] *= s;
  if ((X < 0 && g.bc0 == BC_DIRICHLET) || (X > 2 * g.n && g.bc1 == BC_DIRICHLET)) {
    const double* d = X < 0 ? g.dl : g.dr;
#pragma unroll
    for (int k = 0; k < 3; ++k) V[k] = d[k];
  }
  const Prim1 w = prim1(ph, V);
#pragma unroll
  for (int k = 0; k < 3; ++k) S.U[k][t] = V[k];
  S.A[0][t] = w.u;
  S.A[1][t] = w.p;
  S.A[2][t] = w.T;
  S.A[3][t] = root(ph.gam * w.T);
}

// low-order data of cell i (ghosts as boundary images) into ring entry t
template <typename Src>
__device__ __forceinline__ void cell_site(const G1& g, const Phys& ph, const Src& U, int i, int t,
                                          Tile1& S) {
  double C0[3], Cm[3], Cp[3];
  cell_image1(g, U, i, C0);
  cell_image1(g, U, i - 1, Cm);
  cell_image1(g, U, i + 1, Cp);
  const Prim1 w0 = prim1(ph, C0), wm = prim1(ph, Cm), wp = prim1(ph, Cp);
  const double p0 = w0.p, pm = wm.p, pp = wp.p, u0 = w0.u;
  const double i2 = 1.0 / (2.0 * g.dx);
  const double ux = (wp.u - wm.u) * i2;
  const double Tx = (wp.T - wm.T) * i2;
  const double tau = (4.0 / 3.0) * ph.mu * ux;
  S.C[0][t] = C0[1];
  S.C[1][t] = C0[1] * u0 + p0 - tau;
  S.C[2][t] = (C0[2] + p0) * u0 - (u0 * tau + ph.kap * Tx);
  S.C[3][t] = fabs(u0) + root(ph.gam * w0.T);
  S.C[4][t] = bvisc1(p0, w0.T, ux, Tx, ph);
  S.C[5][t] = fabs(pp - 2.0 * p0 + pm) / fabs(pp + 2.0 * p0 + pm);
  S.C[6][t] = mx(-ux / root(ux * ux + kDucros), 0.0);
#pragma unroll
  for (int k = 0; k < 3; ++k) S.C[7 + k][t] = C0[k];
}

// limited flux of the face between ring cells a and a + 1, at lattice entry q
__device__ __forceinline__ void face_flux(const G1& g, const Phys& ph, const Tile1& S, int a, int q,
                                          double dt, unsigned& raised, double* F) {
  const int b = a + 1;
  double FH[3];
  {
    const double i6 = 1.0 / (6.0 * g.dx);
    const double* uu = S.A[0];
    const double* TT = S.A[2];
    const double gu = dc5(uu[q - 2], uu[q - 1], uu[q + 1], uu[q + 2], i6);
    const double gT = dc5(TT[q - 2], TT[q - 1], TT[q + 1], TT[q + 2], i6);
    const double m = S.U[1][q], E = S.U[2][q];
    const double u = uu[q], p = S.A[1][q];
    const double tau = (4.0 / 3.0) * ph.mu * gu;
    FH[0] = m;
    FH[1] = m * u + p - tau;
    FH[2] = (E + p) * u - (u * tau + ph.kap * gT);
  }
  const int limc = ph.lim & (LIM_SMOOTH | LIM_PP | LIM_LOWONLY);
  if (!limc) {
#pragma unroll
    for (int k = 0; k < 3; ++k) F[k] = FH[k];
  } else {
    const double lam = mx(S.C[3][a], S.C[3][b]) + mx(S.C[4][a], S.C[4][b]);
    double FL[3], Ua[3], Ub[3], Fa[3], Fb[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      Ua[k] = S.C[7 + k][a];
      Ub[k] = S.C[7 + k][b];
      Fa[k] = S.C[k][a];
      Fb[k] = S.C[k][b];
      FL[k] = 0.5 * (Fa[k] + Fb[k]) - 0.5 * lam * (Ub[k] - Ua[k]);
    }
    double ts = 1.0, tpp = 1.0;
    if (ph.lim & LIM_LOWONLY) {
      ts = 0.0;
      tpp = 0.0;
    } else {
      if (ph.lim & LIM_SMOOTH)
        ts = exp(-ph.Cs * mx(S.C[5][a], S.C[5][b]) * mx(S.C[6][a], S.C[6][b]));
      if (ph.lim & LIM_PP) {
        const double m2 = 2.0 * dt / g.dx;
        double ULp[3], UHp[3], ULm[3], UHm[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          const double Fs = FL[k] + ts * (FH[k] - FL[k]);
          ULp[k] = Ua[k] - m2 * (FL[k] - Fa[k]);
          UHp[k] = Ua[k] - m2 * (Fs - Fa[k]);
          ULm[k] = Ub[k] - m2 * (Fb[k] - FL[k]);
          UHm[k] = Ub[k] - m2 * (Fb[k] - Fs);
        }
        bool bad = false;
        const double pLp = pressure1(ULp[0], ULp[1], ULp[2], ph.gm1);
        const double pLm = pressure1(ULm[0], ULm[1], ULm[2], ph.gm1);
        if (keeps(ULp[0], pLp, UHp[0], pressure1(UHp[0], UHp[1], UHp[2], ph.gm1)) &&
            keeps(ULm[0], pLm, UHm[0], pressure1(UHm[0], UHm[1], UHm[2], ph.gm1))) {
          tpp = 1.0;  // as almost everywhere: see theta_pair2
        } else if (!(ULp[0] > 0.0) || !(ULm[0] > 0.0)) {
          tpp = 0.0;
          bad = true;
        } else {
          if (!(pLp > 0.0) || !(pLm > 0.0)) bad = true;
          const double tr = mn(theta_lin(ULp[0], UHp[0], mn(kPPEps, ULp[0])),
                                 theta_lin(ULm[0], UHm[0], mn(kPPEps, ULm[0])));
          double Tp[3], Tm[3];
#pragma unroll
          for (int k = 0; k < 3; ++k) {
            Tp[k] = ULp[k] + tr * (UHp[k] - ULp[k]);
            Tm[k] = ULm[k] + tr * (UHm[k] - ULm[k]);
          }
          const bool ex = ph.lim & LIM_PEXACT;
          const double tp = mn(theta_p1(ULp, pLp, Tp, mn(kPPEps, pLp), ph.gm1, ex),
                               theta_p1(ULm, pLm, Tm, mn(kPPEps, pLm), ph.gm1, ex));
          tpp = tr * tp;
        }
        if (bad) raised |= STAGE_CELL_LOW;
      }
    }
    const double th = ts * tpp;
#pragma unroll
    for (int k = 0; k < 3; ++k) F[k] = FL[k] + th * (FH[k] - FL[k]);
  }
}

// low-order data of site o (1..3) of the five-site low-order point lattice
// V[0..4] (point, average, point, average, point): total flux with the
// central-difference gradient over its neighbours, |u|+c and b
__device__ __forceinline__ void lo_site1(const Phys& ph, const double (&V)[5][3],
                                         const double* u, const double* p, const double* T,
                                         const double* c, int o, double ih, double* F,
                                         double& r, double& b) {
  const double ux = (u[o + 1] - u[o - 1]) * ih, Tx = (T[o + 1] - T[o - 1]) * ih;
  const double tau = (4.0 / 3.0) * ph.mu * ux;
  F[0] = V[o][1];
  F[1] = V[o][1] * u[o] + p[o] - tau;
  F[2] = (V[o][2] + p[o]) * u[o] - (u[o] * tau + ph.kap * Tx);
  r = fabs(u[o]) + c[o];
  b = bvisc1(p[o], T[o], ux, Tx, ph);
}

// forward-Euler value of point k0 (lattice entry q, ring cells r0 and r0 + 1
// at its sides) into out
__device__ __forceinline__ void point_update(const G1& g, const Phys& ph, const Tile1& S, int k0,
                                             int q, int r0, double dt, unsigned& raised,
                                             double* out) {
  const int X = 2 * k0;
  const double i6h = 1.0 / (6.0 * g.dx);
  double Us[5][3], u[5], p[5], T[5];
  double alpha = 0.0;
#pragma unroll
  for (int o = 0; o < 5; ++o) {
    const int s = q + o - 2;
#pragma unroll
    for (int k = 0; k < 3; ++k) Us[o][k] = S.U[k][s];
    u[o] = S.A[0][s];
    p[o] = S.A[1][s];
    T[o] = S.A[2][s];
    alpha = mx(alpha, fabs(u[o]) + S.A[3][s]);
  }
  double Fc[5][3];
#pragma unroll
  for (int o = 0; o < 5; ++o) {
    Fc[o][0] = Us[o][1];
    Fc[o][1] = Us[o][1] * u[o] + p[o];
    Fc[o][2] = (Us[o][2] + p[o]) * u[o];
  }
  double R[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const double dF = dc5(Fc[0][k], Fc[1][k], Fc[3][k], Fc[4][k], i6h);
    const double dU = d4(Us[0][k], Us[1][k], Us[2][k], Us[3][k], Us[4][k]);
    R[k] = -(dF + alpha * i6h * dU);
  }
  const double s4 = 4.0 / (g.dx * g.dx);
  const double m43 = (4.0 / 3.0) * ph.mu;
  R[1] += s4 * m43 * bcol(u);
  R[2] += s4 * (m43 * bform(u, u) + ph.kap * bcol(T));
  double U0[3], UH[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    U0[k] = Us[2][k];
    out[k] = UH[k] = U0[k] + dt * R[k];
  }
  if (ph.lim & LIM_POINT) {
    // low-order LLF scheme on the lattice of point values (X-2, X, X+2) and
    // cell averages (X-1, X+1: ring cells k0 and k0+1), Sec. 3.4
    double V[5][3], lu[5], lp[5], lT[5], lc[5];
#pragma unroll
    for (int o = 0; o < 5; o += 2) {
#pragma unroll
      for (int k = 0; k < 3; ++k) V[o][k] = Us[o][k];
      lu[o] = u[o];
      lp[o] = p[o];
      lT[o] = T[o];
      lc[o] = S.A[3][q + o - 2];
    }
#pragma unroll
    for (int o = 1; o < 5; o += 2) {
#pragma unroll
      for (int k = 0; k < 3; ++k) V[o][k] = S.C[7 + k][r0 + (o >> 1)];
      const Prim1 w = prim1(ph, V[o]);
      lu[o] = w.u;
      lp[o] = w.p;
      lT[o] = w.T;
      lc[o] = root(ph.gam * lT[o]);
    }
    const double ih = 1.0 / g.dx;
    double F1[3], F2[3], F3[3], r1, r2, r3, b1, b2, b3;
    lo_site1(ph, V, lu, lp, lT, lc, 1, ih, F1, r1, b1);
    lo_site1(ph, V, lu, lp, lT, lc, 2, ih, F2, r2, b2);
    lo_site1(ph, V, lu, lp, lT, lc, 3, ih, F3, r3, b3);
    const double lp23 = mx(r2, r3) + mx(b2, b3), lm12 = mx(r1, r2) + mx(b1, b2);
    double Fp[3], Fm[3], UL[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      Fp[k] = 0.5 * (F2[k] + F3[k]) - 0.5 * lp23 * (V[3][k] - V[2][k]);
      Fm[k] = 0.5 * (F1[k] + F2[k]) - 0.5 * lm12 * (V[2][k] - V[1][k]);
    }
    const double c2 = 2.0 * dt / g.dx;
#pragma unroll
    for (int k = 0; k < 3; ++k) UL[k] = U0[k] - c2 * (Fp[k] - Fm[k]);
    bool lbad = false;
    double th = theta_pair1(UL, UH, ph.gm1, lbad, ph.lim & LIM_PEXACT);
    if (ph.lim & LIM_LOWONLY) th = 0.0;
    if (lbad) raised |= STAGE_POINT_LOW;
    if (th != 1.0) {
#pragma unroll
      for (int k = 0; k < 3; ++k) out[k] = UL[k] + th * (UH[k] - UL[k]);
    }
  }
  const int wl = (g.bc0 == BC_NOSLIP || g.bc0 == BC_SYMMETRY);
  const int wr = (g.bc1 == BC_NOSLIP || g.bc1 == BC_SYMMETRY);
  if ((X == 0 && wl) || (X == 2 * g.n && wr)) {
    out[2] -= out[1] * out[1] / (2.0 * out[0]);
    out[1] = 0.0;
  }
  // a point on a Dirichlet side keeps the prescribed state
  if ((X == 0 && g.bc0 == BC_DIRICHLET) || (X == 2 * g.n && g.bc1 == BC_DIRICHLET)) {
    const double* d = X == 0 ? g.dl : g.dr;
#pragma unroll
    for (int k = 0; k < 3; ++k) out[k] = d[k];
  }
}

__global__ void __launch_bounds__(kThreads) k_stage1(G1 g, Phys ph, Stage1 st,
                                                     const double* __restrict__ Un,
                                                     const double* __restrict__ Uk,
                                                     double* __restrict__ Uout) {
  __shared__ Tile1 S;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int i0 = blockIdx.x * kCells;
  const int nc = min(kCells, g.n - i0);        // cells of the tile (0: a last point alone)
  const int npt = min(kCells, g.np - i0);      // its points
  // inside a step attempt: stop if a stage before this one raised a flag (the
  // attempt is rejected and the output never read); for one of this stage's own a
  // late tile does not, since its flags may come before
  const int shift = attempt_shift(st.stage);
  if (tid == 0) S.stop = st.skip_flagged ? peek_flags(st.flags) & ((1u << shift) - 1u) : 0u;
  // entry t of the tile's lattice is site 2 i0 - 2 + t; ring entry t is cell
  // i0 - 1 + t
  const Global1 U{Uk};
  if (wave < 2) {
    if (tid < 2 * nc + 5) lattice_site(g, ph, U, 2 * i0 - 2 + tid, tid, S);
  } else if (lane < nc + 2) {
    cell_site(g, ph, U, i0 - 1 + lane, lane, S);
  }
  __syncthreads();
  if (S.stop) return;
  double dt = st.dt_dev ? *st.dt_dev : st.dt_host;
  if (st.dt_mul != 1.0) dt = st.dt_mul * dt;
  bool ok = true;
  unsigned raised = 0u;
  // RK combination of the forward-Euler value fe of DOF array element a
  auto combine = [&](long a, double fe) {
    const double o = st.first ? fe : st.ca * Un[a] + st.cb * fe;
    Uout[a] = o;
    ok &= (bool)isfinite(o);
  };
  if (wave == 0) {
    double F[3] = {0.0, 0.0, 0.0};
    if (nc > 0 && lane <= nc) face_flux(g, ph, S, lane, 2 * lane + 2, dt, raised, F);
    const double m = dt / g.dx;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const double Fp = __shfl_down(F[k], 1, 64);
      if (lane < nc) combine((long)k * g.n + i0 + lane, S.C[7 + k][lane + 1] - m * (Fp - F[k]));
    }
  } else if (wave == 1 && lane < npt) {
    double out[3];
    point_update(g, ph, S, i0 + lane, 2 * lane + 2, lane, dt, raised, out);
#pragma unroll
    for (int k = 0; k < 3; ++k) combine(g.off_pts + (long)k * g.np + i0 + lane, out[k]);
  }
  if (!ok) raised |= wave == 0 ? STAGE_CELLS_NONFINITE : STAGE_POINTS_NONFINITE;
  if (raised)
    raise_flag(st.flags, st.skip_flagged
                             ? raised << shift
                             : ((raised & STAGE_CELL_LOW) ? FLAG_CELL_LOW : 0u) |
                                   ((raised & STAGE_POINT_LOW) ? FLAG_POINT_LOW : 0u) |
                                   (ok ? 0u : FLAG_NONFINITE));
}

// a whole step from U to Uout (other memory: neighbouring tiles read U)
__global__ void __launch_bounds__(kThreads) k_step1(G1 g, Phys ph, Step1 st,
                                                    const double* __restrict__ U,
                                                    double* __restrict__ Uout) {
  __shared__ Tile1 S;
  __shared__ Held1 H;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int halo = 2 * (st.stages - 1), own = kCells - 2 * halo;
  const int b = (int)blockIdx.x * own - halo;  // first cell of the tile, and lane 0's
  const bool periodic = g.bc0 == BC_PERIODIC;
  if (tid == 0) {
    // A step of a run's block stops once one before it was rejected (the block is
    // redone).  Any other step is an attempt of its own, whose flag word was
    // cleared before the launch: what is up by now came from a faster tile, and a
    // tile that stopped for it would leave out flags of an earlier stage.
    S.stop = st.x.t_out ? peek_flags(st.flags) : 0u;
    H.b = b;
  }
  // the tile of the state.  Beyond periodic sides it goes on; beyond others
  // nothing is read from here (ghosts are images)
  auto within = [&](int i, int n) {
    if (!periodic) return i < 0 ? 0 : min(i, n - 1);
    const int r = i % n;
    return r < 0 ? r + n : r;
  };
  for (int e = tid; e < 3 * (kCells + 4); e += kThreads) {
    const int k = e / (kCells + 4), t = e % (kCells + 4);
    H.C[k][t] = U[(long)k * g.n + within(b - 2 + t, g.n)];
  }
  for (int e = tid; e < 3 * (kCells + 3); e += kThreads) {
    const int k = e / (kCells + 3), t = e % (kCells + 3);
    H.P[k][t] = U[g.off_pts + (long)k * g.np + within(b - 1 + t, g.np)];
  }
  // the step's dt (eq. cfl, as k_cfl takes it) from the averages of the whole
  // grid, each workgroup for itself: a few loads per thread on a small grid,
  // where a reduction as kernels of its own costs two launches
  if (st.x.cfl.on) {
    double ra = 0.0, rv = 0.0;
    for (int c = tid; c < g.n; c += kThreads) {
      const double r = U[c], m = U[g.n + c], E = U[2 * g.n + c];
      const double p = pressure1(r, m, E, ph.gm1);
      const double cs = root(ph.gam * p / r);
      ra = mx(ra, (fabs(m / r) + cs) * st.x.cfl.icx);
      rv = mx(rv, st.x.cfl.vcoef / r);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      ra = mx(ra, __shfl_xor(ra, o, 64));
      rv = mx(rv, __shfl_xor(rv, o, 64));
    }
    if (lane == 0) {
      S.red[0][wave] = ra;
      S.red[1][wave] = rv;
    }
  }
  __syncthreads();
  if (S.stop) return;
  double dt0;
  if (st.x.cfl.on) {
    const double a = mx(mx(S.red[0][0], S.red[0][1]), S.red[0][2]);
    const double v = mx(mx(S.red[1][0], S.red[1][1]), S.red[1][2]);
    const double t = *st.x.t_in;
    dt0 = 1.0 / (a + v);
    if (t + dt0 > st.x.cfl.t_final) dt0 = st.x.cfl.t_final - t;
    if (!(dt0 > 0.0)) dt0 = 0.0;
  } else {
    dt0 = st.dt_dev ? *st.dt_dev : st.dt_host;
  }
  // a run's step keeps the time (t_in is read by other workgroups too, so t_out
  // is other memory where dt comes from it)
  if (st.x.t_out && blockIdx.x == 0 && tid == 0) {
    const double t = *st.x.t_in;
    *st.x.t_out = dt0 > 0.0 ? t + dt0 : t;
    if (dt0 > 0.0) *st.x.steps = *st.x.steps + 1.0;
  }
  unsigned all = 0u;
  // the lane's cell (wave 0) or point (wave 1): the step's first state, and
  // SSP-RK54's second stage, which its last one builds on
  double un[3], u2[3] = {0.0, 0.0, 0.0}, now[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) now[k] = un[k] = wave == 0 ? H.C[k][lane < 61 ? lane + 2 : 0]
                                                        : H.P[k][lane < 62 ? lane + 1 : 0];
  const int j = b + lane;
  const bool real_face = periodic || (j >= 0 && j <= g.n);
  const bool real_cell = periodic || (j >= 0 && j < g.n);
  const bool real_point = periodic || (j >= 0 && j < g.np);
  for (int s = 0; s < st.stages; ++s) {
    // entry t of the lattice is site 2 b - 2 + t, of the ring cell b - 1 + t;
    // of the ghosts, those that faces and points of the grid reach
    if (wave < 2) {
      const int X = 2 * b - 2 + tid;
      if (tid < kSites && (periodic || (X >= -2 && X <= 2 * g.n + 2)))
        lattice_site(g, ph, H, X, tid, S);
    } else if (lane < kRing && (periodic || (j - 1 >= -1 && j - 1 <= g.n))) {
      cell_site(g, ph, H, j - 1, lane, S);
    }
    __syncthreads();
    double dt = dt0;
    if (st.mul[s] != 1.0) dt = st.mul[s] * dt;
    const double ca = st.ca[s], cb = st.cb[s];
    const bool first = ca == 0.0, five = st.stages == 5;
    unsigned raised = 0u;
    bool ok = true;
    // the stage's combinations for the forward-Euler value fe of component k
    auto combine = [&](int k, double fe) {
      const double base = five && s == 4 ? u2[k] : un[k];
      const double o = first ? fe : ca * base + cb * fe;
      ok &= (bool)isfinite(o);
      now[k] = o;
      if (five && s == 1) u2[k] = o;
      if (five && s == 3) {
        now[k] = st.wa * un[k] + st.wb * o;
        u2[k] = st.ga * u2[k] + st.gb * o;
      }
    };
    if (wave == 0) {
      double F[3] = {0.0, 0.0, 0.0};
      if (real_face && lane >= 2 * s && lane <= kCells - 2 * s)
        face_flux(g, ph, S, lane, 2 * lane + 2, dt, raised, F);
      const double m = dt / g.dx;
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const double Fp = __shfl_down(F[k], 1, 64);
        if (real_cell && lane >= 2 * s && lane < kCells - 2 * s) {
          combine(k, S.C[7 + k][lane + 1] - m * (Fp - F[k]));
          H.C[k][lane + 2] = now[k];
        }
      }
    } else if (wave == 1 && real_point && lane >= 2 * s && lane <= kCells - 2 * s) {
      double out[3];
      point_update(g, ph, S, j, 2 * lane + 2, lane, dt, raised, out);
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        combine(k, out[k]);
        H.P[k][lane + 1] = now[k];
      }
    }
    if (!ok) raised |= wave == 0 ? STAGE_CELLS_NONFINITE : STAGE_POINTS_NONFINITE;
    all |= raised << attempt_shift(s);
    __syncthreads();
  }
  if (lane >= halo && lane < halo + own) {
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      if (wave == 0 && j < g.n) Uout[(long)k * g.n + j] = now[k];
      if (wave == 1 && j < g.np) Uout[g.off_pts + (long)k * g.np + j] = now[k];
    }
  }
  if (all) raise_flag(st.flags, all);
}

G1 geo1(const afi::Geo& geo) {
  G1 g;
  g.n = geo.n1;
  g.np = geo.n1x;
  g.off_pts = geo.off_pts;
  g.bc0 = geo.bc[0];
  g.bc1 = geo.bc[1];
  g.dx = geo.dx;
  for (int k = 0; k < 3; ++k) {
    g.dl[k] = geo.bcstate[0][k];
    g.dr[k] = geo.bcstate[1][k];
  }
  return g;
}

}  // namespace

namespace afi {

// Every workgroup takes the maxima of the whole grid for itself, which costs less
// than a launch while the averages are few.  Measured, us a step of a run with dt
// in the step and in a launch before it (SSP-RK3; SSP-RK54):
//   400 cells    13.0, 14.3;  17.5, 18.7
//   800          13.9, 14.4;  18.4, 19.0
//   1200         14.8, 14.7;  19.2, 19.3
//   1600         15.5, 15.1;  19.8, 19.6
//   4096         20.1, 16.9;  24.3, 21.3
// (A single step saves its state in the launch that fixes dt, so that dt in the
// step itself gains it nothing: af_step of 400 cells takes 32.2 us so, 30.2 apart.)
bool step1d_takes_cfl(const Geo& g) { return g.dim == 1 && g.n1 <= 1200; }

hipError_t stage1d(const Geo& geo, const Phys& ph, const Work& w, const double* Un,
                   const double* Uk, double* Uout, const double* dt_dev, double dt_host,
                   StageCoef sc, hipStream_t s, Timer* tm) {
  const G1 g = geo1(geo);
  Stage1 st{};
  st.ca = sc.a;
  st.cb = sc.b;
  st.first = sc.first;
  st.skip_flagged = sc.skip_flagged;
  st.stage = sc.stage;
  st.flags = w.flags;
  st.dt_dev = dt_dev;
  st.dt_host = dt_host;
  st.dt_mul = sc.dt_mul;
  AFI_TIMED(tm, 0, s,
            hipLaunchKernelGGL(k_stage1, dim3((unsigned)((g.np + kCells - 1) / kCells)),
                               dim3(kThreads), 0, s, g, ph, st, Un, Uk, Uout));
  return hipGetLastError();
}

hipError_t step1d(const Geo& geo, const Phys& ph, const Work& w, const double* U, double* Uout,
                  const double* dt_dev, double dt_host, const StepCoef1& sc, const StepExtras1& x,
                  hipStream_t s, Timer* tm) {
  const G1 g = geo1(geo);
  Step1 st{};
  st.stages = sc.stages;
  for (int k = 0; k < sc.stages; ++k) {
    st.ca[k] = sc.a[k];
    st.cb[k] = sc.b[k];
    st.mul[k] = sc.mul[k];
  }
  st.wa = sc.wa;
  st.wb = sc.wb;
  st.ga = sc.ga;
  st.gb = sc.gb;
  st.flags = w.flags;
  st.dt_dev = dt_dev;
  st.dt_host = dt_host;
  st.x = x;
  const int own = kCells - 4 * (sc.stages - 1);
  AFI_TIMED(tm, 0, s,
            hipLaunchKernelGGL(k_step1, dim3((unsigned)((g.np + own - 1) / own)), dim3(kThreads),
                               0, s, g, ph, st, U, Uout));
  return hipGetLastError();
}

}  // namespace afi
