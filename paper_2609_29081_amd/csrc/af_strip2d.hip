// af_strip2d.hip -- one SSP-RK3 stage of the 2D compact AF method on gfx950
// as a pipeline of wavefronts that marches up a strip of the grid.
//
// The tile kernel (af_stage2d.hip) spends more than half of its vector
// instructions on index arithmetic and halo sites, and its waves wait for
// each other at seven barriers per tile.  Here a workgroup of twelve wave64s
// takes a strip of 60 cell columns (one per lane, two more on either side) and
// a range of rows, and each wave does one part of the scheme per step of the
// march, which takes it one row of cells further.  When row r is loaded,
//                 first half of the step         second half
//   wave_centre   centres of row r-1             gradients around row r-1
//   wave_edges    points ye of row r             low-order y terms of ye, r-2
//   wave_cells    averages of row r              low-order data of cells, r-1
//   wave_xface    limited x-face fluxes, r-3     smoothness sensors, r-1; gradients
//                                                at centres, r-2
//   wave_yface    limited y-face fluxes, r-2     averages updated, r-3
//   wave_xres0    x residual of co, r-2          x residual of ye, r-2
//   wave_xlow0    points co of row r             low-order x terms of co, ye, r-2
//   wave_xlow1    points xe of row r             low-order x terms of xe, r-2
//   wave_xe       x residual of xe, r-3          xe updated, r-3
//   wave_yres0    y residual of co, r-3          low-order y terms of co, xe, r-2
//   wave_yres1    y residual of xe, r-3          co updated, r-3
//   wave_ye       y residual of ye, r-3          ye updated, r-3
// (a strip's rows are finished three steps behind the march, which starts two
// rows early).  Everything is computed once per site and row (the columns at
// the sides of a strip and a few rows at its ends apart), lanes address LDS at
// unit stride, and directions are compile-time constants.  Rows pass through
// LDS rings of two to four slots (156 KB in FP64, so one workgroup fills a
// CU); what a wave needs again in the next row and the rings no longer hold
// stays in its registers.
//
// What bounds it: vector instructions and, in FP64, the power they take.  A step
// of a strip takes 5,110 cycles (FP32 stencils: 4,110) for 3,100 (3,010) vector
// instructions on four SIMDs, which are busy 64 % (75 %) of the time; LDS is
// busy 45 % and HBM a fifth.  An FP64 instruction takes 4.4 cycles of its SIMD
// whatever it depends on, and under a stream of them the clock falls from 2.4
// to about 2.05 GHz, so that large FP64 stages gain only from fewer
// instructions.  Small grids (few rows per strip) are bound by the chains of
// dependent work between two barriers.  So the parts are spread over the SIMDs
// to equal work in either half (of 85 other assignments none is better), what a
// half has to wait for is kept short, and three waves per SIMD, which FP64 at
// 168 registers a wave just allows, hide each other's waits.
//
// Measured, stage of the shock tube (tile kernel, this; the card's clock under
// this load differs from hour to hour, 87 to 101 us for the first):
//   1000 x 500   FP64 210, 88 us    FP32 stencils 157, 70 us
//   2048 x 1024  FP64 878, 343 us   FP32 stencils 670, 269 us
//   400 x 200    FP64 41, 26 us     FP32 stencils 40, 21 us
//   64 x 32      FP64 28, 12.8 us   FP32 stencils 42, 11.2 us
// On the way, at 1000 x 500 in FP64: 125 with eight waves (two per SIMD), 107
// with twelve, 103 with shorter maxima, square roots, limiters and addresses
// (all on one day, at the slower clock).
//
// The arithmetic is the tile kernel's, expression by expression, so the two
// give the same bits.  The tile kernel remains for batches (see strip_shapes, and
// the variants that af_batch_set_variant and af_batch_tune choose among) and for
// single grids of few columns and many rows (single_on_tiles).
#include <algorithm>

#include "af_scheme2d.hpp"

using namespace afd;

namespace {

constexpr int W = 64;                 // lanes: cell columns of a strip with its margins
constexpr int SX = afi::kStripColumns;  // cell columns a strip owns: lanes 2 .. 61
constexpr int NT = 768;               // twelve waves, three per SIMD
constexpr int CO = 0, YE = 1, XE = 2; // point types

template <typename R>
constexpr bool kFP64 = std::is_same<R, double>::value;

// LDS of a strip.  Column c of a row holds cell column i0 - 2 + c: its points
// co, xe at the column's lower side, ye and the average or centre at its
// middle.  A row's slot is its distance from the first loaded row, modulo the
// number of slots.
template <typename R>
struct Rings {
  R P[3][9][4][W];      // points: U (4), u, v, p, T, c; rows r .. r-3
  R Z[9][3][W];         // centres, rows r-1 .. r-3
  R GE0[6][2][W];       // gradients at co and ...
  R GO0[6][2][W];       // ... ye (but T_x): rows r-1, r-2
  R GE1[6][3][W];       // at xe (but T_y): rows r-1 .. r-3
  R GO1[4][2][W];       // at centres (u_x, v_x, u_y, v_y): rows r-2, r-3
  R AV[10][4][W];       // averages: U (4), u, v, p, T, c, 1/rho; rows r .. r-3
  R C[14][3][W];        // cell low-order data, rows r-1 .. r-3
  R FX[4][W];           // limited x-face fluxes, row r-3
  // residual and low-order terms on their way to the wave that updates the
  // point; written in one half of a row, read in the next half
  R XC[8][W], XY[8][W]; // x-direction, residual (4) and low-order: co, ye
  R LX[4][W];           // x-direction low-order terms of xe
  R LC[4][W], LE[4][W]; // y-direction low-order terms of co, xe ...
  R LO[4][W];           // ... and ye
  R RX[4][W], RC[4][W]; // y-direction residuals of xe, co
  // FP32 stencils: FP64 averages, and the low parts V - float(V) of the points
  double AVD[4][4][kFP64<R> ? 1 : W];
  float PL[3][4][4][kFP64<R> ? 1 : W];
  unsigned stop;
};

// one lattice site: U (4), u, v, p, T, c
template <typename R>
struct Site {
  R U[4], a[5];
};

template <typename R, int S>
__device__ __forceinline__ Site<R> site9(const R (&A)[9][S][W], int slot, int c) {
  Site<R> s;
#pragma unroll
  for (int k = 0; k < 4; ++k) s.U[k] = A[k][slot][c];
#pragma unroll
  for (int k = 0; k < 5; ++k) s.a[k] = A[4 + k][slot][c];
  return s;
}
template <typename R>
__device__ __forceinline__ Site<R> avg_site(const R (&A)[10][4][W], int slot, int c) {
  Site<R> s;
#pragma unroll
  for (int k = 0; k < 4; ++k) s.U[k] = A[k][slot][c];
#pragma unroll
  for (int k = 0; k < 5; ++k) s.a[k] = A[4 + k][slot][c];
  return s;
}

// (u, v, T) of a site
template <typename R>
struct Z3 {
  R u, v, T;
};
template <typename R, int Q, int S>
__device__ __forceinline__ Z3<R> z3(const R (&A)[Q][S][W], int slot, int c) {
  return Z3<R>{A[4][slot][c], A[5][slot][c], A[7][slot][c]};
}
template <typename R>
__device__ __forceinline__ Z3<R> z3(const Site<R>& s) {
  return Z3<R>{s.a[0], s.a[1], s.a[3]};
}

// value of x in the lane to the left (lane - 1) or right (lane + 1); the
// first or last lane keeps its own
template <int CTRL>
__device__ __forceinline__ int lane_shift(int x) {
  return __builtin_amdgcn_update_dpp(x, x, CTRL, 0xF, 0xF, false);
}
template <int CTRL>
__device__ __forceinline__ float lane_shift(float x) {
  return __int_as_float(lane_shift<CTRL>(__float_as_int(x)));
}
template <int CTRL>
__device__ __forceinline__ double lane_shift(double x) {
  const long long v = __double_as_longlong(x);
  const int lo = lane_shift<CTRL>((int)v), hi = lane_shift<CTRL>((int)(v >> 32));
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
template <typename R>
__device__ __forceinline__ R from_left(R x) { return lane_shift<0x138>(x); }   // wave_shr:1
template <typename R>
__device__ __forceinline__ R from_right(R x) { return lane_shift<0x130>(x); }  // wave_shl:1

// direction-D terms of the residual of a point, from the five sites s of its
// line and the derivatives across D of the velocities at them (see line_terms)
template <int D, typename R>
__device__ __forceinline__ void line_resid(const PhysT<R>& ph, double h, const Site<R>* const* s,
                                           const R* ga, const R* gb, R* Rd) {
  R sp[5];
#pragma unroll
  for (int o = 0; o < 5; ++o) sp[o] = fabs(s[o]->a[D]) + s[o]->a[4];
  R Rr[4];
  line_terms(
      ph, h, mx5(sp[0], sp[1], sp[2], sp[3], sp[4]),
      [&](LineValue v, int o) {
        return v == kRho  ? s[o]->U[0]
               : v == kMd ? s[o]->U[1 + D]
               : v == kMo ? s[o]->U[2 - D]
               : v == kE  ? s[o]->U[3]
               : v == kVa ? s[o]->a[D]
               : v == kVb ? s[o]->a[1 - D]
               : v == kP  ? s[o]->a[2]
                          : s[o]->a[3];
      },
      ga, gb, Rr);
  Rd[0] = Rr[0];
  Rd[1] = D ? Rr[2] : Rr[1];
  Rd[2] = D ? Rr[1] : Rr[2];
  Rd[3] = Rr[3];
}

// direction-D data of a site of the low-order point scheme (Sec. 3.4): total
// flux and b, from its central differences over the four neighbours
template <typename R>
struct LoFlux {
  R F[4], b;
};
template <int D, typename R>
__device__ __forceinline__ LoFlux<R> lo_flux(const PhysT<R>& ph, const Site<R>& s, const Z3<R>& xm,
                                             const Z3<R>& xp, const Z3<R>& ym, const Z3<R>& yp,
                                             R ihx, R ihy) {
  R gr[6];
  gr[0] = (xp.u - xm.u) * ihx;
  gr[1] = (xp.v - xm.v) * ihx;
  gr[2] = (xp.T - xm.T) * ihx;
  gr[3] = (yp.u - ym.u) * ihy;
  gr[4] = (yp.v - ym.v) * ihy;
  gr[5] = (yp.T - ym.T) * ihy;
  LoFlux<R> f;
  tot_flux(D, s.U, s.a[0], s.a[1], s.a[2], gr, ph, f.F);
  // the density component is the momentum itself
  f.F[0] = s.U[1 + D];
  f.b = bvisc2_dir(D, s.a[2], s.a[3], gr[0], gr[1], gr[2], gr[3], gr[4], gr[5], ph);
  return f;
}
// LLF flux between sites a (minus) and b (plus) of a line of direction D
template <int D, typename R>
__device__ __forceinline__ void lo_face(const Site<R>& a, const LoFlux<R>& fa, const Site<R>& b,
                                        const LoFlux<R>& fb, R* F) {
  const R ra = fabs(a.a[D]) + a.a[4], rb = fabs(b.a[D]) + b.a[4];
  const R lam = mx(ra, rb) + mx(fa.b, fb.b);
#pragma unroll
  for (int k = 0; k < 4; ++k)
    F[k] = R(0.5) * (fa.F[k] + fb.F[k]) - R(0.5) * lam * (b.U[k] - a.U[k]);
}

// what every wave of the workgroup knows
template <typename R>
struct Ctx {
  G2 g;
  Phys phd;
  PhysT<R> ph;
  const double* __restrict__ Uk;
  const double* __restrict__ Un;
  double* __restrict__ Uout;
  double dt, ca, cb;
  int first;
  unsigned* flags;
  int shift;           // of the flags raised (see kStageShift)
  const float* blend;  // see limit_face
  float* ts_out;
  int lane, i0;        // cell column of lane c: i0 - 2 + c
  int j0, j1;          // rows of the strip
  int rows;            // rows of the march: r = j0 - 2 .. j0 - 3 + rows
};

// ring slots of the rows around row r (k = r - (j0 - 2) >= 0)
__device__ __forceinline__ int slot4(int k) { return k & 3; }
__device__ __forceinline__ int slot2(int k) { return k & 1; }
__device__ __forceinline__ int slot3(int k) { return (k + 3) % 3; }

// p, known to point to global memory (loads through a pointer that came from
// memory would be flat ones)
template <typename T>
__device__ __forceinline__ T* in_global(T* p) {
  return (T*)(__attribute__((address_space(1))) T*)(uintptr_t)p;
}
// byte offset of element i >= 0 of a row of doubles, for at()
__device__ __forceinline__ unsigned element(unsigned i) {
  unsigned o = i * 8u;
  asm("" : "+v"(o));
  return o;
}
// element of the row at p, which is the same for the whole wave: its address is
// p in scalar registers and a 32-bit offset.  (Left to itself the compiler adds
// the two up per lane, an instruction more for every access; hence the asm here
// and above, which hides from it what they are.)
template <typename T>
__device__ __forceinline__ T& at(T* p, unsigned o) {
  asm("" : "+s"(p));
  using Byte = __attribute__((address_space(1))) char;
  return *(T*)((Byte*)(uintptr_t)p + o);
}

// the stage's update of a point from its residual Rs and low-order terms Ls
// (Sec. 2.2, 3.4), the RK combination, and the store
template <typename R>
__device__ __forceinline__ void point_finish(const Ctx<R>& X, int t, int i, int j, const double* U0,
                                             const R* Rs, const double* Ls, const double* un,
                                             bool own, bool& nonfinite) {
  const G2& g = X.g;
  double UH[4], out[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) out[k] = UH[k] = U0[k] + X.dt * double(Rs[k]);
  if (X.ph.lim & LIM_POINT) {
    double UL[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) UL[k] = U0[k] - Ls[k];
    bool lbad = false;
    double th = theta_pair2(UL, UH, X.phd.gm1, lbad, X.ph.lim & LIM_PEXACT);
    if (X.ph.lim & LIM_LOWONLY) th = 0.0;
    if (lbad && own) raise_flag(X.flags, FLAG_POINT_LOW << X.shift);
    if (th != 1.0) {
#pragma unroll
      for (int k = 0; k < 4; ++k) out[k] = UL[k] + th * (UH[k] - UL[k]);
    }
  }
  if (t != YE) {
    if (i == 0) project(wall_of(g.bc0), 0, out);
    if (i == g.n1) project(wall_of(g.bc1), 0, out);
  }
  if (t != XE) {
    if (j == 0) project(wall_of(g.bc2), 1, out);
    if (j == g.n2) project(wall_of(g.bc3), 1, out);
  }
  if (!own) return;
  const int ni = t == YE ? g.n1 : g.n1x, nj = t == XE ? g.n2 : g.n2y;
  const long np = (long)ni * nj;
  double* o = X.Uout + (t == XE ? g.off_xe : (t == YE ? g.off_ye : g.off_co)) + (long)j * ni;
  const unsigned e = element(i);
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const double v = X.first ? out[k] : X.ca * un[k] + X.cb * out[k];
    if (!isfinite(v)) nonfinite = true;
    at(o + k * np, e) = v;
  }
}

// U^n of point (i, j) of type t, or of cell average (i, j) (t = -1)
template <typename R>
__device__ __forceinline__ void load_un(const Ctx<R>& X, int t, int i, int j, bool own, double* un) {
  const G2& g = X.g;
#pragma unroll
  for (int k = 0; k < 4; ++k) un[k] = 0.0;
  if (X.first || !own) return;
  const int ni = (t == YE || t < 0) ? g.n1 : g.n1x, nj = (t == XE || t < 0) ? g.n2 : g.n2y;
  const long np = (long)ni * nj;
  const double* p =
      X.Un + (t < 0 ? 0L : (t == XE ? g.off_xe : (t == YE ? g.off_ye : g.off_co))) + (long)j * ni;
  const unsigned e = element(i);
#pragma unroll
  for (int k = 0; k < 4; ++k) un[k] = at(p + k * np, e);
}

// FP64 value of a point, from its LDS copy (and, with FP32 stencils, the low part)
template <typename R>
__device__ __forceinline__ void fp64_point(const Rings<R>& S, int t, int slot, int c, const R* U,
                                           double* U0) {
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if constexpr (kFP64<R>)
      U0[k] = U[k];
    else
      U0[k] = double(U[k]) + double(S.PL[t][k][slot][c]);
  }
}

#define STRIP_BARRIER() __syncthreads()

// the barrier in the middle of a row; true if the attempt was rejected meanwhile
template <typename R>
__device__ __forceinline__ bool mid_row(const Rings<R>& S) {
  STRIP_BARRIER();
  return __builtin_amdgcn_readfirstlane(S.stop) != 0u;
}

// ---- loads -------------------------------------------------------------------
// The lane's two lattice columns of the strip (E: co, xe; O: ye, averages):
// image columns and momentum flips.  Lanes beyond the grid's ghosts (strips at
// the upper side) read column 0.
struct Columns {
  unsigned cE, cO;  // columns of the DOF arrays
  int fE, fO;       // flips
  bool flips;       // any lane of the strip has one
};
template <typename R>
__device__ __forceinline__ Columns columns_of(const Ctx<R>& X) {
  const G2& g = X.g;
  const int Xlim = 2 * g.n1, x = 2 * (X.i0 - 2 + X.lane);
  int kE = -1, kO = -1;
  int iE = x <= Xlim + kMargin ? axis_image(x, Xlim, g.bc0, g.bc1, kE) : 0;
  const int iO = x + 1 <= Xlim + kMargin ? axis_image(x + 1, Xlim, g.bc0, g.bc1, kO) : 1;
  if (iE == Xlim && g.n1x == g.n1) iE = 0;
  const int fE = image_flips(kE, -1), fO = image_flips(kO, -1);
  return Columns{(unsigned)(iE >> 1), (unsigned)(iO >> 1), fE, fO, __ballot(fE | fO) != 0};
}
// image row and flips of the even (odd) lattice line of row r; rows past the
// last ghost are never used
template <typename R>
__device__ __forceinline__ int even_line(const Ctx<R>& X, int r, int& flip) {
  const G2& g = X.g;
  const int Ylim = 2 * g.n2;
  int ky;
  int y = axis_image(2 * r <= Ylim + kMargin ? 2 * r : Ylim, Ylim, g.bc2, g.bc3, ky);
  if (y == Ylim && g.n2y == g.n2) y = 0;
  flip = image_flips(-1, ky);
  return y >> 1;
}
template <typename R>
__device__ __forceinline__ int odd_line(const Ctx<R>& X, int r, int& flip) {
  const G2& g = X.g;
  const int Ylim = 2 * g.n2;
  int ky;
  const int y =
      axis_image(2 * r + 1 <= Ylim + kMargin ? 2 * r + 1 : Ylim - 1, Ylim, g.bc2, g.bc3, ky);
  flip = image_flips(-1, ky);
  return y >> 1;
}

// raw values of a site type in flight: CO, YE, XE, or AV (3) the averages
struct Raw {
  double v[4];
  int flip;
  bool flips;  // any lane's flip is not 0
};
template <int T, typename R>
__device__ __forceinline__ void issue(const Ctx<R>& X, const Columns& col, int r, Raw& q) {
  const G2& g = X.g;
  int fy;
  const int row = (T & 2) ? odd_line(X, r, fy) : even_line(X, r, fy);
  q.flip = fy ^ ((T & 1) ? col.fO : col.fE);
  q.flips = fy != 0 || col.flips;
  const int ni = (T & 1) ? g.n1 : g.n1x, nj = (T & 2) ? g.n2 : g.n2y;
  const double* b =
      X.Uk + (T == CO ? g.off_co : (T == YE ? g.off_ye : (T == XE ? g.off_xe : 0L))) + (long)row * ni;
  const long pl = (long)ni * nj;
  const unsigned e = element((T & 1) ? col.cO : col.cE);
#pragma unroll
  for (int k = 0; k < 4; ++k) q.v[k] = at(b + k * pl, e);
}
// their values with the image's signs
__device__ __forceinline__ void signed_values(const Raw& q, double* V) {
#pragma unroll
  for (int k = 0; k < 4; ++k) V[k] = q.v[k];
  if (q.flips) {  // rows and strips at a wall only
    V[1] = (q.flip & 1) ? -V[1] : V[1];
    V[2] = (q.flip & 2) ? -V[2] : V[2];
  }
}
// a point of type t into its ring
template <typename R>
__device__ __forceinline__ void store_point(Rings<R>& S, const Ctx<R>& X, int t, int s,
                                            const double* V) {
  const int lane = X.lane;
  R w[5];
  aux_of_fp64(X.phd, V, w);
#pragma unroll
  for (int k = 0; k < 4; ++k) S.P[t][k][s][lane] = R(V[k]);
#pragma unroll
  for (int k = 0; k < 5; ++k) S.P[t][4 + k][s][lane] = w[k];
  if constexpr (!kFP64<R>) {
#pragma unroll
    for (int k = 0; k < 4; ++k) S.PL[t][k][s][lane] = float(V[k] - double(float(V[k])));
  }
}

// ---- wave_centre -------------------------------------------------------------------
template <typename R>
__device__ __forceinline__ void wave_centre(Rings<R>& S, const Ctx<R>& X) {
  const G2& g = X.g;
  const int c = X.lane, cl = c > 0 ? c - 1 : 0, cr = c < W - 1 ? c + 1 : W - 1;
  const int Xlim = 2 * g.n1, Ylim = 2 * g.n2, n1 = g.n1, n1x = g.n1x, n2 = g.n2;
  const Columns col = columns_of(X);
  // a centre beyond a wall or outflow side takes the value of its image
  // column, which another lane of the strip holds
  const int xo = 2 * (X.i0 - 2 + c) + 1;
  const bool ghost_col =
      xo <= Xlim + kMargin && (xo < 0 || xo > Xlim) && g.bc0 != BC_PERIODIC;
  const int image_lane = (int)col.cO - X.i0 + 2;
  const bool has_ghost_col = g.bc0 != BC_PERIODIC && (X.i0 < 2 || 2 * (X.i0 + 62) > Xlim);
  // centre of the lane's cell of row r straight from the state (for the row
  // beyond a lower wall or outflow side, whose image the march has not reached)
  auto centre_of = [&](int r, R* V, R* w) {
    int kd;
    int iR = xo + 1 <= Xlim + kMargin ? axis_image(xo + 1, Xlim, g.bc0, g.bc1, kd) : 0;
    if (iR == Xlim && n1x == n1) iR = 0;
    const unsigned cR = (unsigned)(iR >> 1), cE = col.cE, cO = col.cO;
    R Ub[4], e[4], cc[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const double* co = X.Uk + g.off_co + (long)k * n1x * g.n2y + (long)r * n1x;
      const double* ye = X.Uk + g.off_ye + (long)k * n1 * g.n2y + (long)r * n1;
      const double* xe = X.Uk + g.off_xe + (long)k * n1x * n2 + (long)r * n1x;
      const double* av = X.Uk + (long)k * n1 * n2 + (long)r * n1;
      Ub[k] = R(av[cO]);
      e[k] = R(xe[cE]) + R(xe[cR]) + R(ye[cO]) + R(ye[n1 + cO]);
      cc[k] = R(co[cE]) + R(co[cR]) + R(co[n1x + cE]) + R(co[n1x + cR]);
    }
    centre_value(X.ph, X.phd, Ub, e, cc, V, w);
  };
  auto flipped = [](R v, bool neg) { return neg ? -v : v; };
  const R ihx = R(1.0 / (6.0 * g.dx)), ihy = R(1.0 / (6.0 * g.dy));

  // (co and ye of row r are loaded here too: their ring entries come in the same
  // half row)
  Raw nco, nye;
  issue<CO>(X, col, X.j0 - 2, nco);
  issue<YE>(X, col, X.j0 - 2, nye);
  R zv[4], zw[5];  // the latest centre
#pragma unroll
  for (int k = 0; k < 4; ++k) zv[k] = R(0.0);
#pragma unroll
  for (int k = 0; k < 5; ++k) zw[k] = R(0.0);
  R lowv[4], loww[5];
  const bool low_ghost = X.j0 == 0 && g.bc2 != BC_PERIODIC;
  if (low_ghost) centre_of(0, lowv, loww);

  for (int k = 0; k < X.rows; ++k) {
    const int r = X.j0 - 2 + k;
    double V[4];
    R co[4], ye[4];
    signed_values(nye, V);
#pragma unroll
    for (int n = 0; n < 4; ++n) ye[n] = R(V[n]);
    signed_values(nco, V);
    if (k + 1 < X.rows) {
      issue<CO>(X, col, r + 1, nco);
      issue<YE>(X, col, r + 1, nye);
    }
#pragma unroll
    for (int n = 0; n < 4; ++n) co[n] = R(V[n]);
    // centre of row r-1
    const int rc = r - 1;
    if (k >= 2) {
      int f = 0, ky;
      if (rc < 0 && low_ghost) {
        (void)axis_image(2 * rc + 1, Ylim, g.bc2, g.bc3, ky);
        f = image_flips(-1, ky);
#pragma unroll
        for (int n = 0; n < 4; ++n) zv[n] = lowv[n];
#pragma unroll
        for (int n = 0; n < 5; ++n) zw[n] = loww[n];
      } else if (rc >= n2 && g.bc2 != BC_PERIODIC) {
        // the row beyond the upper side: its image is the row below, whose
        // centre this lane computed last
        (void)axis_image(2 * rc + 1 <= Ylim + kMargin ? 2 * rc + 1 : Ylim, Ylim, g.bc2, g.bc3, ky);
        f = image_flips(-1, ky);
      } else {
        R Ub[4], e[4], cc[4];
        const int s1 = slot4(k - 1);
#pragma unroll
        for (int n = 0; n < 4; ++n) {
          Ub[n] = S.AV[n][s1][c];
          e[n] = S.P[XE][n][s1][c] + S.P[XE][n][s1][cr] + S.P[YE][n][s1][c] + ye[n];
          cc[n] = S.P[CO][n][s1][c] + S.P[CO][n][s1][cr] + co[n] + from_right(co[n]);
        }
        centre_value(X.ph, X.phd, Ub, e, cc, zv, zw);
      }
      const int sz = slot3(k - 1);
#pragma unroll
      for (int n = 0; n < 4; ++n) S.Z[n][sz][c] = zv[n];
#pragma unroll
      for (int n = 0; n < 5; ++n) S.Z[4 + n][sz][c] = zw[n];
      if (f) {
        S.Z[1][sz][c] = flipped(zv[1], f & 1);
        S.Z[4][sz][c] = flipped(zw[0], f & 1);
        S.Z[2][sz][c] = flipped(zv[2], f & 2);
        S.Z[5][sz][c] = flipped(zw[1], f & 2);
      }
      if (has_ghost_col) {
        __builtin_amdgcn_wave_barrier();
        if (ghost_col) {
          R z[9];
#pragma unroll
          for (int n = 0; n < 9; ++n) z[n] = S.Z[n][sz][image_lane];
#pragma unroll
          for (int n = 0; n < 9; ++n)
            S.Z[n][sz][c] = flipped(z[n], ((n == 1 || n == 4) && (col.fO & 1)) ||
                                              ((n == 2 || n == 5) && (col.fO & 2)));
        }
      }
    }
    if (mid_row(S)) return;
    if (k >= 2) {
      const int p0 = slot4(k), p1 = slot4(k - 1), p2 = slot4(k - 2);
      const int z1 = slot3(k - 1), z2 = slot3(k - 2);
      const int ge = slot2(k - 1), g1 = slot3(k - 1);
      const int src[3] = {4, 5, 7};  // u, v, T
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        const R (&co_)[4][W] = S.P[CO][src[q]];
        const R (&ye_)[4][W] = S.P[YE][src[q]];
        const R (&xe_)[4][W] = S.P[XE][src[q]];
        const R (&zz)[3][W] = S.Z[src[q]];
        S.GE0[q][ge][c] = dc5(co_[p1][cl], ye_[p1][cl], ye_[p1][c], co_[p1][cr], ihx);
        S.GE0[3 + q][ge][c] = dc5(co_[p2][c], xe_[p2][c], xe_[p1][c], co_[p0][c], ihy);
        if (q < 2) S.GO0[q][ge][c] = dc5(ye_[p1][cl], co_[p1][c], co_[p1][cr], ye_[p1][cr], ihx);
        S.GO0[3 + q][ge][c] = dc5(ye_[p2][c], zz[z2][c], zz[z1][c], ye_[p0][c], ihy);
        S.GE1[q][g1][c] = dc5(xe_[p1][cl], zz[z1][cl], zz[z1][c], xe_[p1][cr], ihx);
        if (q < 2)
          S.GE1[3 + q][g1][c] = dc5(xe_[p2][c], co_[p1][c], co_[p0][c], xe_[p0][c], ihy);
      }
    }
    STRIP_BARRIER();
  }
}

// ---- wave_edges --------------------------------------------------------------------
template <typename R>
__device__ __forceinline__ void wave_edges(Rings<R>& S, const Ctx<R>& X) {
  const G2& g = X.g;
  const int c = X.lane, cr = c < W - 1 ? c + 1 : W - 1;
  const R ihx = R(1.0 / g.dx), ihy = R(1.0 / g.dy);
  const R cL = R(2.0 * X.dt / g.dy);
  Site<R> y2{};     // ye of row r-2, its low-order data, and the LLF flux below it
  LoFlux<R> fy2{};
  R Fprev[4] = {};
  const Columns col = columns_of(X);
  Raw nye;
  issue<YE>(X, col, X.j0 - 2, nye);
  for (int k = 0; k < X.rows; ++k) {
    const int r = X.j0 - 2 + k;
    double V[4];
    signed_values(nye, V);
    if (k + 1 < X.rows) issue<YE>(X, col, r + 1, nye);
    store_point(S, X, YE, slot4(k), V);
    if (mid_row(S)) return;
    if (k >= 2 && (X.ph.lim & LIM_POINT)) {
      // the line ye, average, ye of the column
      const int s1 = slot4(k - 1), s2 = slot4(k - 2);
      const Site<R> A = avg_site(S.AV, s2, c), y1 = site9(S.P[YE], s1, c);
      const LoFlux<R> fA = lo_flux<1>(X.ph, A, z3(S.P[XE], s2, c), z3(S.P[XE], s2, cr), z3(y2),
                                      z3(y1), ihx, ihy);
      const LoFlux<R> fy1 = lo_flux<1>(X.ph, y1, z3(S.P[CO], s1, c), z3(S.P[CO], s1, cr), z3(A),
                                       z3(S.AV, s1, c), ihx, ihy);
      R Fya[4], Fay[4];
      lo_face<1>(y2, fy2, A, fA, Fya);
      lo_face<1>(A, fA, y1, fy1, Fay);
#pragma unroll
      for (int n = 0; n < 4; ++n) {
        S.LO[n][c] = cL * (Fya[n] - Fprev[n]);
        Fprev[n] = Fay[n];
      }
      y2 = y1;
      fy2 = fy1;
    }
    STRIP_BARRIER();
  }
}

// a cell average of the ring
template <typename R>
__device__ __forceinline__ CellAvg<R> ring_cell(const Rings<R>& S, int slot, int c) {
  CellAvg<R> a;
#pragma unroll
  for (int n = 0; n < 4; ++n) a.U[n] = S.AV[n][slot][c];
  a.p = S.AV[6][slot][c];
  a.r = S.AV[9][slot][c];
  return a;
}

// ---- wave_cells --------------------------------------------------------------------
template <typename R>
__device__ __forceinline__ void wave_cells(Rings<R>& S, const Ctx<R>& X, unsigned stop_for) {
  const G2& g = X.g;
  const int c = X.lane, cl = c > 0 ? c - 1 : 0, cr = c < W - 1 ? c + 1 : W - 1;
  const Columns col = columns_of(X);
  Raw nav;
  issue<3>(X, col, X.j0 - 2, nav);
  // inside a step attempt: stop once any workgroup has raised a flag of stop_for
  // (it is rejected and its output is never read).  The flag word of the row
  // before is the one that counts, so that nobody waits for its load.
  unsigned fl = 0u;
  for (int k = 0; k < X.rows; ++k) {
    const int r = X.j0 - 2 + k, s = slot4(k);
    if (c == 0) S.stop = fl;
    double V[4];
    signed_values(nav, V);
    if (k + 1 < X.rows) issue<3>(X, col, r + 1, nav);
    R C0[4];
#pragma unroll
    for (int n = 0; n < 4; ++n) C0[n] = R(V[n]);
    const R r0 = rcp(C0[0]);
    const R pr = pressure_r(X.ph, C0, r0);
#pragma unroll
    for (int n = 0; n < 4; ++n) S.AV[n][s][c] = C0[n];
    S.AV[4][s][c] = C0[1] * r0;
    S.AV[5][s][c] = C0[2] * r0;
    S.AV[6][s][c] = pr;
    S.AV[7][s][c] = pr * r0;
    S.AV[8][s][c] = root(X.ph.gam * pr * r0);
    S.AV[9][s][c] = r0;
    if constexpr (!kFP64<R>) {
#pragma unroll
      for (int n = 0; n < 4; ++n) S.AVD[n][s][c] = V[n];
    }
    if (mid_row(S)) return;
    if (stop_for) fl = peek_flags(X.flags) & stop_for;
    if (k >= 2) {
      const int p0 = slot4(k), p1 = slot4(k - 1), p2 = slot4(k - 2);
      R o[12];
      cell_low(g, X.ph, ring_cell(S, p1, c), ring_cell(S, p1, cl), ring_cell(S, p1, cr),
               ring_cell(S, p2, c), ring_cell(S, p0, c), S.AV[8][p1][c], o);
      const int sc = slot3(k - 1);
#pragma unroll
      for (int n = 0; n < 12; ++n) S.C[n][sc][c] = o[n];
    }
    STRIP_BARRIER();
  }
}

// what a face needs of one of its cells
template <typename R>
struct FaceCell {
  double U64[4];
  R U[4], F[4], rs, b, phi1, phi2;
};
template <typename R>
__device__ __forceinline__ FaceCell<R> face_cell(const Rings<R>& S, int d, int sc, int sa, int c) {
  FaceCell<R> f;
#pragma unroll
  for (int n = 0; n < 4; ++n) {
    f.U[n] = S.AV[n][sa][c];
    if constexpr (kFP64<R>)
      f.U64[n] = f.U[n];
    else
      f.U64[n] = S.AVD[n][sa][c];
    f.F[n] = S.C[4 * d + n][sc][c];
  }
  f.rs = S.C[8 + d][sc][c];
  f.b = S.C[10 + d][sc][c];
  f.phi1 = S.C[12][sc][c];
  f.phi2 = S.C[13][sc][c];
  return f;
}

template <typename R>
__device__ __forceinline__ void face_between(const Ctx<R>& X, int d, int i, int j,
                                             const FaceCell<R>& a, const FaceCell<R>& b, const R* FH,
                                             bool own, R* F) {
  const float* blend = X.blend;
  float* ts_out = X.ts_out;
  const int limc = (X.ph.lim & (LIM_SMOOTH | LIM_PP | LIM_LOWONLY)) | (blend ? 1 : 0);
  if (!limc) {
#pragma unroll
    for (int k = 0; k < 4; ++k) F[k] = FH[k];
    return;
  }
  FaceCells<R> fc;
  const R lam = mx(a.rs, b.rs) + mx(a.b, b.b);
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    fc.Ua[k] = a.U64[k];
    fc.Ub[k] = b.U64[k];
    fc.Fa[k] = a.F[k];
    fc.Fb[k] = b.F[k];
    fc.FL[k] = R(0.5) * (a.F[k] + b.F[k]) - R(0.5) * lam * (b.U[k] - a.U[k]);
  }
  fc.phi1 = mx(a.phi1, b.phi1);
  fc.phi2 = mx(a.phi2, b.phi2);
  limit_face(X.g, X.ph, X.phd, d, i, j, X.dt, fc, FH, blend, ts_out, own, X.flags,
             FLAG_CELL_LOW << X.shift, F);
}

// total flux of direction D at a point of type t, gradients gr
template <int D, typename R, int S1, int S2>
__device__ __forceinline__ void point_flux(const PhysT<R>& ph, const R (&P)[9][S1][W], int sp,
                                           const R (&G)[6][S2][W], int sg, int c, R* F) {
  R U[4], gr[6];
  U[0] = R(0.0);  // not read
#pragma unroll
  for (int k = 1; k < 4; ++k) U[k] = P[k][sp][c];
#pragma unroll
  for (int k = 0; k < 6; ++k) gr[k] = G[k][sg][c];
  tot_flux(D, U, P[4][sp][c], P[5][sp][c], P[6][sp][c], gr, ph, F);
}

// ---- wave_xface --------------------------------------------------------------------
template <typename R>
__device__ __forceinline__ void wave_xface(Rings<R>& S, const Ctx<R>& X) {
  const G2& g = X.g;
  const int c = X.lane, cl = c > 0 ? c - 1 : 0, cr = c < W - 1 ? c + 1 : W - 1;
  const int i = X.i0 - 2 + c;
  const bool own_col = c >= 2 && c <= SX + 2 && i <= g.n1;
  const R ihx = R(1.0 / (6.0 * g.dx)), ihy = R(1.0 / (6.0 * g.dy));
  R Fco[4], Fxe[4];  // fluxes at co and xe of the row before
#pragma unroll
  for (int n = 0; n < 4; ++n) Fco[n] = Fxe[n] = R(0.0);
  for (int k = 0; k < X.rows; ++k) {
    const int r = X.j0 - 2 + k;
    if (k >= 4) {
      R F0[4], F1[4];
      point_flux<0>(X.ph, S.P[CO], slot4(k - 2), S.GE0, slot2(k - 2), c, F0);
      point_flux<0>(X.ph, S.P[XE], slot4(k - 2), S.GE1, slot3(k - 2), c, F1);
      const int j = r - 3;
      if (j >= X.j0 && j < X.j1 && j < g.n2) {
        R FH[4], F[4];
#pragma unroll
        for (int n = 0; n < 4; ++n) FH[n] = (Fco[n] + R(4.0) * Fxe[n] + F0[n]) * R(1.0 / 6.0);
        const FaceCell<R> a = face_cell(S, 0, slot3(k - 3), slot4(k - 3), cl);
        const FaceCell<R> b = face_cell(S, 0, slot3(k - 3), slot4(k - 3), c);
        face_between(X, 0, i, j, a, b, FH, own_col, F);
#pragma unroll
        for (int n = 0; n < 4; ++n) S.FX[n][c] = F[n];
      }
#pragma unroll
      for (int n = 0; n < 4; ++n) {
        Fco[n] = F0[n];
        Fxe[n] = F1[n];
      }
    }
    if (mid_row(S)) return;
    if (k >= 2) {
      const int p1 = slot4(k - 1);
      R phi[2];
      cell_sensors(g, ring_cell(S, p1, c), ring_cell(S, p1, cl), ring_cell(S, p1, cr),
                   ring_cell(S, slot4(k - 2), c), ring_cell(S, slot4(k), c), phi);
      S.C[12][slot3(k - 1)][c] = phi[0];
      S.C[13][slot3(k - 1)][c] = phi[1];
      // gradients at the centres of row r-2
      const int p2 = slot4(k - 2), g2 = slot2(k - 2);
      const int z1 = slot3(k - 1), z2 = slot3(k - 2), z3s = slot3(k - 3);
#pragma unroll
      for (int q = 0; q < 2; ++q) {  // u, v
        const R (&ye_)[4][W] = S.P[YE][4 + q];
        const R (&xe_)[4][W] = S.P[XE][4 + q];
        const R (&zz)[3][W] = S.Z[4 + q];
        S.GO1[q][g2][c] = dc5(zz[z2][cl], xe_[p2][c], xe_[p2][cr], zz[z2][cr], ihx);
        S.GO1[2 + q][g2][c] = dc5(zz[z3s][c], ye_[p2][c], ye_[p1][c], zz[z1][c], ihy);
      }
    }
    STRIP_BARRIER();
  }
}

// ---- wave_yface --------------------------------------------------------------------
template <typename R, bool DEV>
__device__ __forceinline__ void wave_yface(Rings<R>& S, const Ctx<R>& X, bool& nonfinite, const afi::BatchInst* dinst,
                                           int rates, double& cfl_a, double& cfl_v) {
  const G2& g = X.g;
  const int c = X.lane, i = X.i0 - 2 + c;
  const bool own_col = c >= 2 && c < SX + 2 && i < g.n1;
  const int cr = c < W - 1 ? c + 1 : W - 1;
  FaceCell<R> low;  // the cell below the face
  R Flow[4];        // flux through the lower side of row r-3
#pragma unroll
  for (int n = 0; n < 4; ++n) {
    Flow[n] = R(0.0);
    low.U64[n] = 0.0;
    low.U[n] = low.F[n] = R(0.0);
  }
  low.rs = low.b = low.phi1 = low.phi2 = R(0.0);
  const double mxd = X.dt / g.dx, myd = X.dt / g.dy;
  const long nc = (long)g.n1 * g.n2;
  for (int k = 0; k < X.rows; ++k) {
    const int r = X.j0 - 2 + k;
    const int ju = r - 3;  // the row whose averages are updated
    const bool upd = ju >= X.j0 && ju < X.j1 && ju < g.n2;
    R F[4];
    double un[4], av[4];
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      F[n] = R(0.0);
      av[n] = low.U64[n];  // the average of row r-3
    }
    load_un(X, -1, i, ju, own_col && upd, un);
    if (k >= 3) {
      const int j = r - 2;
      const FaceCell<R> up = face_cell(S, 1, slot3(k - 2), slot4(k - 2), c);
      if (j >= X.j0 && j <= X.j1 && j <= g.n2) {
        R Fa[4], Fm[4], FH[4];
        point_flux<1>(X.ph, S.P[CO], slot4(k - 2), S.GE0, slot2(k - 2), c, Fa);
        point_flux<1>(X.ph, S.P[YE], slot4(k - 2), S.GO0, slot2(k - 2), c, Fm);
#pragma unroll
        for (int n = 0; n < 4; ++n)
          FH[n] = (Fa[n] + R(4.0) * Fm[n] + from_right(Fa[n])) * R(1.0 / 6.0);
        face_between(X, 1, i, j, low, up, FH, own_col, F);
      }
      low = up;
    }
    if (mid_row(S)) return;
    if (upd) {
      double o4[4];
      double* row = X.Uout + (long)ju * g.n1;
      const unsigned e = element(i);
#pragma unroll
      for (int n = 0; n < 4; ++n) {
        const double dfx = double(S.FX[n][cr]) - double(S.FX[n][c]);
        const double dfy = double(F[n]) - double(Flow[n]);
        const double fe = av[n] - mxd * dfx - myd * dfy;
        const double o = X.first ? fe : X.ca * un[n] + X.cb * fe;
        o4[n] = o;
        if (own_col) {
          if (!isfinite(o)) nonfinite = true;
          at(row + n * nc, e) = o;
        }
      }
      if constexpr (DEV) {
        // the last stage of a device-resident step: the CFL rates (eq. cfl)
        // of the new average, as the CFL kernel takes them, for the next step
        if (rates && own_col) {
          const double p = pressure2(o4[0], o4[1], o4[2], o4[3], X.phd.gm1);
          const double cs = root(X.phd.gam * p / o4[0]);
          cfl_a = mx(cfl_a, (fabs(o4[1] / o4[0]) + cs) * dinst->icx);
          cfl_a = mx(cfl_a, (fabs(o4[2] / o4[0]) + cs) * dinst->icy);
          cfl_v = mx(cfl_v, dinst->vcoef / o4[0]);
        }
      }
    }
#pragma unroll
    for (int n = 0; n < 4; ++n) Flow[n] = F[n];
    STRIP_BARRIER();
  }
}

// ---- wave_xres0 --------------------------------------------------------------------
template <typename R>
__device__ __forceinline__ void wave_xres0(Rings<R>& S, const Ctx<R>& X) {
  const G2& g = X.g;
  const int c = X.lane, cl = c > 0 ? c - 1 : 0, cr = c < W - 1 ? c + 1 : W - 1;
  for (int k = 0; k < X.rows; ++k) {
    const int j = X.j0 - 4 + k;
    const bool on = j >= X.j0 && j < X.j1;
    const int s2 = slot4(k - 2), gs = slot2(k - 2);
    Site<R> Ol, E, O, Er;
    R Rc[4], uo[2], vo[2], ue, ve;
    if (on) {
      const Site<R> El = site9(S.P[CO], s2, cl);
      Ol = site9(S.P[YE], s2, cl);
      E = site9(S.P[CO], s2, c);
      O = site9(S.P[YE], s2, c);
      Er = site9(S.P[CO], s2, cr);
      // derivatives along y of u and v: across the line
      uo[0] = S.GO0[3][gs][cl];
      vo[0] = S.GO0[4][gs][cl];
      uo[1] = S.GO0[3][gs][c];
      vo[1] = S.GO0[4][gs][c];
      ue = S.GE0[3][gs][cr];
      ve = S.GE0[4][gs][cr];
      const Site<R>* s[5] = {&El, &Ol, &E, &O, &Er};
      const R ga[5] = {S.GE0[3][gs][cl], uo[0], R(0.0), uo[1], ue};
      const R gb[5] = {S.GE0[4][gs][cl], vo[0], R(0.0), vo[1], ve};
      line_resid<0>(X.ph, g.dx, s, ga, gb, Rc);
    }
    if (mid_row(S)) return;
    if (on) {
      const Site<R> Or = site9(S.P[YE], s2, cr);
      const Site<R>* s[5] = {&Ol, &E, &O, &Er, &Or};
      const R ga[5] = {uo[0], S.GE0[3][gs][c], R(0.0), ue, S.GO0[3][gs][cr]};
      const R gb[5] = {vo[0], S.GE0[4][gs][c], R(0.0), ve, S.GO0[4][gs][cr]};
      R Ry[4];
      line_resid<0>(X.ph, g.dx, s, ga, gb, Ry);
#pragma unroll
      for (int n = 0; n < 4; ++n) {
        S.XC[n][c] = Rc[n];
        S.XY[n][c] = Ry[n];
      }
    }
    STRIP_BARRIER();
  }
}

// ---- wave_xlow0 --------------------------------------------------------------------
template <typename R>
__device__ __forceinline__ void wave_xlow0(Rings<R>& S, const Ctx<R>& X) {
  const G2& g = X.g;
  const int c = X.lane, cl = c > 0 ? c - 1 : 0, cr = c < W - 1 ? c + 1 : W - 1;
  const R ihx = R(1.0 / g.dx), ihy = R(1.0 / g.dy);
  const R cL = R(2.0 * X.dt / g.dx);
  // the lane's corners come in here, in the half that this wave has to spare
  const Columns col = columns_of(X);
  Raw nco;
  issue<CO>(X, col, X.j0 - 2, nco);
  for (int k = 0; k < X.rows; ++k) {
    const int j = X.j0 - 4 + k;
    const bool on = j >= X.j0 && j < X.j1 && (X.ph.lim & LIM_POINT);
    const int s2 = slot4(k - 2), s3 = slot4(k - 3);
    double V[4];
    signed_values(nco, V);
    if (k + 1 < X.rows) issue<CO>(X, col, X.j0 - 1 + k, nco);
    store_point(S, X, CO, slot4(k), V);
    if (mid_row(S)) return;
    if (on) {
      Site<R> E, O;
      LoFlux<R> fE, fO;
      E = site9(S.P[CO], s2, c);
      O = site9(S.P[YE], s2, c);
      fE = lo_flux<0>(X.ph, E, z3(S.P[YE], s2, cl), z3(O), z3(S.P[XE], s3, c), z3(S.P[XE], s2, c),
                      ihx, ihy);
      fO = lo_flux<0>(X.ph, O, z3(E), z3(S.P[CO], s2, cr), z3(S.AV, s3, c), z3(S.AV, s2, c), ihx,
                      ihy);
      LoFlux<R> fEr;
      Site<R> Er;
#pragma unroll
      for (int n = 0; n < 4; ++n) {
        fEr.F[n] = from_right(fE.F[n]);
        Er.U[n] = from_right(E.U[n]);
      }
      fEr.b = from_right(fE.b);
      Er.a[0] = from_right(E.a[0]);
      Er.a[4] = from_right(E.a[4]);
      R Feo[4], Foe[4];
      lo_face<0>(E, fE, O, fO, Feo);
      lo_face<0>(O, fO, Er, fEr, Foe);
#pragma unroll
      for (int n = 0; n < 4; ++n) {
        S.XC[4 + n][c] = cL * (Feo[n] - from_left(Foe[n]));
        S.XY[4 + n][c] = cL * (Foe[n] - Feo[n]);
      }
    }
    STRIP_BARRIER();
  }
}

// ---- wave_xe -----------------------------------------------------------------------
template <typename R>
__device__ __forceinline__ void wave_xe(Rings<R>& S, const Ctx<R>& X, bool& nonfinite) {
  const G2& g = X.g;
  const int c = X.lane, cl = c > 0 ? c - 1 : 0, cr = c < W - 1 ? c + 1 : W - 1;
  const int i = X.i0 - 2 + c;
  const bool own_col = c >= 2 && c < SX + 2 && i < g.n1x;
  for (int k = 0; k < X.rows; ++k) {
    const int j = X.j0 - 5 + k;
    const bool on = j >= X.j0 && j < X.j1 && j < g.n2;
    const int s3 = slot4(k - 3), z = slot3(k - 3);
    R Rx[4];
    double un[4], U0[4], Ls[4];
    if (on) {
      load_un(X, XE, i, j, own_col, un);
      const Site<R> E = site9(S.P[XE], s3, c);
      fp64_point(S, XE, s3, c, E.U, U0);
      const Site<R> El = site9(S.P[XE], s3, cl), Er = site9(S.P[XE], s3, cr);
      const Site<R> Zl = site9(S.Z, z, cl), Zr = site9(S.Z, z, c);
      const int e1 = slot3(k - 3), o1 = slot2(k - 3);
      const Site<R>* s[5] = {&El, &Zl, &E, &Zr, &Er};
      const R ga[5] = {S.GE1[3][e1][cl], S.GO1[2][o1][cl], R(0.0), S.GO1[2][o1][c],
                       S.GE1[3][e1][cr]};
      const R gb[5] = {S.GE1[4][e1][cl], S.GO1[3][o1][cl], R(0.0), S.GO1[3][o1][c],
                       S.GE1[4][e1][cr]};
      line_resid<0>(X.ph, g.dx, s, ga, gb, Rx);
#pragma unroll
      for (int n = 0; n < 4; ++n) Ls[n] = double(S.LX[n][c]) + double(S.LE[n][c]);
    }
    if (mid_row(S)) return;
    if (on) {
      R Rs[4];
#pragma unroll
      for (int n = 0; n < 4; ++n) Rs[n] = Rx[n] + S.RX[n][c];
      point_finish(X, XE, i, j, U0, Rs, Ls, un, own_col, nonfinite);
    }
    STRIP_BARRIER();
  }
}

// ---- wave_xlow1 --------------------------------------------------------------------
template <typename R>
__device__ __forceinline__ void wave_xlow1(Rings<R>& S, const Ctx<R>& X) {
  const G2& g = X.g;
  const int c = X.lane, cl = c > 0 ? c - 1 : 0, cr = c < W - 1 ? c + 1 : W - 1;
  const R ihx = R(1.0 / g.dx), ihy = R(1.0 / g.dy);
  const R cL = R(2.0 * X.dt / g.dx);
  // and the lane's lower edges, as in wave_xlow0
  const Columns col = columns_of(X);
  Raw nxe;
  issue<XE>(X, col, X.j0 - 2, nxe);
  for (int k = 0; k < X.rows; ++k) {
    const int j = X.j0 - 4 + k;
    const bool on = j >= X.j0 && j < X.j1 && j < g.n2 && (X.ph.lim & LIM_POINT);
    const int s1 = slot4(k - 1), s2 = slot4(k - 2);
    double V[4];
    signed_values(nxe, V);
    if (k + 1 < X.rows) issue<XE>(X, col, X.j0 - 1 + k, nxe);
    store_point(S, X, XE, slot4(k), V);
    if (mid_row(S)) return;
    if (on) {
      Site<R> E, A;
      LoFlux<R> fE, fA;
      // the line xe, average, xe
      E = site9(S.P[XE], s2, c);
      A = avg_site(S.AV, s2, c);
      fE = lo_flux<0>(X.ph, E, z3(S.AV, s2, cl), z3(A), z3(S.P[CO], s2, c), z3(S.P[CO], s1, c), ihx,
                      ihy);
      fA = lo_flux<0>(X.ph, A, z3(E), z3(S.P[XE], s2, cr), z3(S.P[YE], s2, c), z3(S.P[YE], s1, c),
                      ihx, ihy);
      Site<R> Al;
      LoFlux<R> fAl;
#pragma unroll
      for (int n = 0; n < 4; ++n) {
        Al.U[n] = from_left(A.U[n]);
        fAl.F[n] = from_left(fA.F[n]);
      }
      Al.a[0] = from_left(A.a[0]);
      Al.a[4] = from_left(A.a[4]);
      fAl.b = from_left(fA.b);
      R Fm[4], Fp[4];
      lo_face<0>(Al, fAl, E, fE, Fm);
      lo_face<0>(E, fE, A, fA, Fp);
#pragma unroll
      for (int n = 0; n < 4; ++n) S.LX[n][c] = cL * (Fp[n] - Fm[n]);
    }
    STRIP_BARRIER();
  }
}

// ---- wave_yres1 --------------------------------------------------------------------
template <typename R>
__device__ __forceinline__ void wave_yres1(Rings<R>& S, const Ctx<R>& X, bool& nonfinite) {
  const G2& g = X.g;
  const int c = X.lane, i = X.i0 - 2 + c;
  const bool own_col = c >= 2 && c < SX + 2 && i < g.n1x;
  Site<R> x4{};  // xe of row r-4, and its derivatives along x
  R gx4[2] = {};
  for (int k = 0; k < X.rows; ++k) {
    const int j = X.j0 - 5 + k;
    const bool on = j >= X.j0 && j < X.j1;
    const int s2 = slot4(k - 2), s3 = slot4(k - 3);
    R Rx[4];
    double un[4], Ls[4];
    if (k >= 3) {
      const Site<R> x3 = site9(S.P[XE], s3, c);
      const int e0 = slot2(k - 2), e1 = slot3(k - 2), e3 = slot3(k - 3);
      if (on) {
        const Site<R> c3 = site9(S.P[CO], s3, c), c2 = site9(S.P[CO], s2, c),
                      x2 = site9(S.P[XE], s2, c);
        const Site<R>* s[5] = {&x4, &c3, &x3, &c2, &x2};
        const R ga[5] = {gx4[1], S.GE0[1][slot2(k - 3)][c], R(0.0), S.GE0[1][e0][c], S.GE1[1][e1][c]};
        const R gb[5] = {gx4[0], S.GE0[0][slot2(k - 3)][c], R(0.0), S.GE0[0][e0][c], S.GE1[0][e1][c]};
        R Rd[4];
        line_resid<1>(X.ph, g.dy, s, ga, gb, Rd);
#pragma unroll
        for (int n = 0; n < 4; ++n) {
          S.RX[n][c] = Rd[n];
          Rx[n] = S.XC[n][c];
          Ls[n] = double(S.XC[4 + n][c]) + double(S.LC[n][c]);
        }
      }
      x4 = x3;
      gx4[0] = S.GE1[0][e3][c];
      gx4[1] = S.GE1[1][e3][c];
    }
    load_un(X, CO, i, j, own_col && on, un);
    if (mid_row(S)) return;
    if (on) {
      R U[4], Rs[4];
      double U0[4];
#pragma unroll
      for (int n = 0; n < 4; ++n) {
        U[n] = S.P[CO][n][s3][c];
        Rs[n] = Rx[n] + S.RC[n][c];
      }
      fp64_point(S, CO, s3, c, U, U0);
      point_finish(X, CO, i, j, U0, Rs, Ls, un, own_col, nonfinite);
    }
    STRIP_BARRIER();
  }
}

// ---- wave_yres0 --------------------------------------------------------------------
template <typename R>
__device__ __forceinline__ void wave_yres0(Rings<R>& S, const Ctx<R>& X) {
  const G2& g = X.g;
  const int c = X.lane, cl = c > 0 ? c - 1 : 0;
  const R ihx = R(1.0 / g.dx), ihy = R(1.0 / g.dy);
  const R cL = R(2.0 * X.dt / g.dy);
  // the line of the column: co and xe of row r-4 and their derivatives along x;
  // co of row r-2, its low-order data, and the LLF flux below it
  Site<R> c4{}, x4{}, c2{};
  R gc4[2] = {}, gx4[2] = {};
  LoFlux<R> fc2{};
  R Fprev[4] = {};
  for (int k = 0; k < X.rows; ++k) {
    const int j = X.j0 - 5 + k;
    const bool on = j >= X.j0 && j < X.j1;
    const int s1 = slot4(k - 1), s2 = slot4(k - 2), s3 = slot4(k - 3);
    if (k >= 3) {
      const Site<R> c3 = site9(S.P[CO], s3, c), x3 = site9(S.P[XE], s3, c);
      const int e0 = slot2(k - 2), e3 = slot3(k - 3);
      const R gx3[2] = {S.GE1[0][e3][c], S.GE1[1][e3][c]};
      if (on) {
        const Site<R>* s[5] = {&c4, &x4, &c3, &x3, &c2};
        const R ga[5] = {gc4[1], gx4[1], R(0.0), gx3[1], S.GE0[1][e0][c]};
        const R gb[5] = {gc4[0], gx4[0], R(0.0), gx3[0], S.GE0[0][e0][c]};
        R Rd[4];
        line_resid<1>(X.ph, g.dy, s, ga, gb, Rd);
#pragma unroll
        for (int n = 0; n < 4; ++n) S.RC[n][c] = Rd[n];
      }
      c4 = c3;
      x4 = x3;
#pragma unroll
      for (int n = 0; n < 2; ++n) {
        gc4[n] = S.GE0[n][slot2(k - 3)][c];
        gx4[n] = gx3[n];
      }
    }
    if (mid_row(S)) return;
    if (k >= 2) {
      const Site<R> c1 = site9(S.P[CO], s1, c);
      if (X.ph.lim & LIM_POINT) {
        const Site<R> x2 = site9(S.P[XE], s2, c);
        const LoFlux<R> fx2 = lo_flux<1>(X.ph, x2, z3(S.AV, s2, cl), z3(S.AV, s2, c), z3(c2), z3(c1),
                                         ihx, ihy);
        const LoFlux<R> fc1 = lo_flux<1>(X.ph, c1, z3(S.P[YE], s1, cl), z3(S.P[YE], s1, c), z3(x2),
                                         z3(S.P[XE], s1, c), ihx, ihy);
        R Fcx[4], Fxc[4];
        lo_face<1>(c2, fc2, x2, fx2, Fcx);
        lo_face<1>(x2, fx2, c1, fc1, Fxc);
#pragma unroll
        for (int n = 0; n < 4; ++n) {
          S.LC[n][c] = cL * (Fcx[n] - Fprev[n]);
          S.LE[n][c] = cL * (Fxc[n] - Fcx[n]);
          Fprev[n] = Fxc[n];
        }
        fc2 = fc1;
      }
      c2 = c1;
    }
    STRIP_BARRIER();
  }
}

// ---- wave_ye -----------------------------------------------------------------------
template <typename R>
__device__ __forceinline__ void wave_ye(Rings<R>& S, const Ctx<R>& X, bool& nonfinite) {
  const G2& g = X.g;
  const int c = X.lane, i = X.i0 - 2 + c;
  const bool own_col = c >= 2 && c < SX + 2 && i < g.n1;
  // the line of the column: ye and centre of row r-4, ye of row r-3
  Site<R> y4{}, z4{}, y3{};
  R gy4[2] = {}, gz4[2] = {}, gy3[2] = {};
  for (int k = 0; k < X.rows; ++k) {
    const int j = X.j0 - 5 + k;
    const bool on = j >= X.j0 && j < X.j1;
    Site<R> y2{}, z3_{};
    R gy2[2] = {}, gz3[2] = {}, Rs[4];
    double un[4], Ls[4];
    load_un(X, YE, i, j, own_col && on, un);
    if (k >= 3) {
      y2 = site9(S.P[YE], slot4(k - 2), c);
      z3_ = site9(S.Z, slot3(k - 3), c);
#pragma unroll
      for (int n = 0; n < 2; ++n) {
        gy2[n] = S.GO0[n][slot2(k - 2)][c];
        gz3[n] = S.GO1[n][slot2(k - 3)][c];
      }
    }
    if (on) {
      const Site<R>* s[5] = {&y4, &z4, &y3, &z3_, &y2};
      const R ga[5] = {gy4[1], gz4[1], R(0.0), gz3[1], gy2[1]};
      const R gb[5] = {gy4[0], gz4[0], R(0.0), gz3[0], gy2[0]};
      R Rd[4];
      line_resid<1>(X.ph, g.dy, s, ga, gb, Rd);
#pragma unroll
      for (int n = 0; n < 4; ++n) {
        Rs[n] = S.XY[n][c] + Rd[n];
        Ls[n] = double(S.XY[4 + n][c]) + double(S.LO[n][c]);
      }
    }
    if (mid_row(S)) return;
    if (on) {
      double U0[4];
      fp64_point(S, YE, slot4(k - 3), c, y3.U, U0);
      point_finish(X, YE, i, j, U0, Rs, Ls, un, own_col, nonfinite);
    }
    y4 = y3;
    z4 = z3_;
    y3 = y2;
#pragma unroll
    for (int n = 0; n < 2; ++n) {
      gy4[n] = gy3[n];
      gz4[n] = gz3[n];
      gy3[n] = gy2[n];
    }
    STRIP_BARRIER();
  }
}

// launch arguments
struct StripArgs {
  // one instance, its step driven by the host
  G2 g;
  Phys ph;
  const double* Uk;
  const double* Un;
  double* Uout;
  const double* dt_dev;
  double dt_host, dt_mul;  // the step is dt_mul * dt
  unsigned* flags;
  int nx, H;
  int shift;          // of the flags this stage raises
  unsigned stop_for;  // flags for which it stops
  const float* blend;  // see limit_face
  float* ts_out;
  // instances whose step machinery is on the device: their descriptors, the
  // instance of each workgroup (NULL: the first one), and where stage 2 leaves
  // the CFL maxima of the new state per workgroup (a, v), or NULL
  afi::BatchInst* inst;
  const int* wg_inst;
  double2* cfl_partial;
  int k;  // the stage
  double ca, cb;
  int first;
};

// p, known to point to memory that the kernel does not write, for scalar loads
template <typename T>
__device__ __forceinline__ const T* in_constant(const T* p) {
  return (const T*)(const __attribute__((address_space(4))) T*)(uintptr_t)p;
}

// BLEND: per-face blend input/output arrays; DEV: instances with descriptors
template <typename R, bool BLEND, bool DEV>
__global__ void __launch_bounds__(NT) k_strip(StripArgs) {
  __shared__ Rings<R> S;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // Each wave reads what it needs of the arguments for itself, through a pointer
  // the compiler does not see through: read once for all twelve, they are kept
  // in scalar registers across every wave's loop, and most of them spill
  auto args = [&]() {
    auto* q = __builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(q));
    return (const StripArgs*)q;
  };
  // the workgroup's instance
  afi::BatchInst* inst = nullptr;
  if constexpr (DEV) {
    const StripArgs* p = args();
    inst = p->inst + (p->wg_inst ? in_constant(p->wg_inst)[blockIdx.x] : 0);
    if (!in_constant(inst)->active) return;  // its step is done: nothing to do in this round
  }
  auto ctx = [&]() {
    const StripArgs* p = args();
    if constexpr (DEV) {
      auto q = (uintptr_t)inst;
      asm volatile("" : "+s"(q));
      const afi::BatchInst* I = in_constant((const afi::BatchInst*)q);
      // the three RK3 stages from buf[cur], through the other two buffers
      const int c = I->cur, a = (c + 1) % 3, b = (c + 2) % 3, k = p->k;
      const int wg = blockIdx.x - I->wg0;
      const int j0 = wg / I->snx * I->sH, n2y = I->g.n2y, j1 = min(j0 + I->sH, n2y);
      const Phys phd = I->ph;
      const double* Uk = k == 0 ? I->buf[c] : (k == 1 ? I->buf[a] : I->buf[b]);
      const double* Un = I->buf[c];
      return Ctx<R>{I->g,
                    phd,
                    phys_as<R>(phd),
                    in_global(Uk),
                    in_global(Un),
                    in_global(k == 1 ? I->buf[b] : I->buf[a]),
                    I->dt,
                    p->ca,
                    p->cb,
                    p->first,
                    in_global(&inst->flags),
                    kStageShift * k,
                    nullptr,
                    nullptr,
                    (int)(threadIdx.x & 63),
                    wg % I->snx * SX,
                    j0,
                    j1,
                    j1 - j0 + 5};  // a row is finished when the march is three rows past it
    } else {
      const int wg = blockIdx.x, nx = p->nx, H = p->H;
      const int j0 = wg / nx * H, n2y = p->g.n2y, j1 = min(j0 + H, n2y);
      const Phys phd = p->ph;
      const double* dt_dev = p->dt_dev;
      const double dt = p->dt_mul * (dt_dev ? *in_constant(dt_dev) : p->dt_host);
      return Ctx<R>{p->g,
                    phd,
                    phys_as<R>(phd),
                    in_global(p->Uk),
                    in_global(p->Un),
                    in_global(p->Uout),
                    dt,
                    p->ca,
                    p->cb,
                    p->first,
                    in_global(p->flags),
                    p->shift,
                    BLEND ? in_global(p->blend) : nullptr,
                    BLEND ? in_global(p->ts_out) : nullptr,
                    (int)(threadIdx.x & 63),
                    wg % nx * SX,
                    j0,
                    j1,
                    j1 - j0 + 5};
    }
  };
  auto stop_for = [&]() -> unsigned {
    if constexpr (DEV)
      return in_constant(inst)->halvings < in_constant(inst)->max_halvings
                 ? ~0u
                 : (1u << kStageShift * args()->k) - 1u;
    else
      return args()->stop_for;
  };
  bool nonfinite = false;
  double cfl_a = 0.0, cfl_v = 0.0;
  // waves go to the SIMDs round-robin: w, w + 4 and w + 8 share one, and the
  // parts are grouped so that the four carry equal work in either half
  switch (wave) {
    case 0: wave_xface(S, ctx()); break;
    case 4: wave_xlow0(S, ctx()); break;
    case 8: wave_xe(S, ctx(), nonfinite); break;
    case 1:
      wave_yface<R, DEV>(S, ctx(), nonfinite, inst, DEV && args()->k == 2, cfl_a, cfl_v);
      break;
    case 5: wave_xlow1(S, ctx()); break;
    case 9: wave_xres0(S, ctx()); break;
    case 2: wave_yres1(S, ctx(), nonfinite); break;
    case 6: wave_ye(S, ctx(), nonfinite); break;
    case 10: wave_edges(S, ctx()); break;
    case 3: wave_centre(S, ctx()); break;
    case 7: wave_yres0(S, ctx()); break;
    default: wave_cells(S, ctx(), stop_for()); break;
  }
  if (nonfinite)
    raise_flag(DEV ? &inst->flags : args()->flags,
               FLAG_NONFINITE << (DEV ? kStageShift * args()->k : args()->shift));
  if constexpr (DEV) {
    // the workgroup's CFL maxima of the new state (lanes that wrote no cell
    // hold 0, neutral for max)
    double2* part = args()->cfl_partial;
    if (wave == 1 && part && args()->k == 2) {
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) {
        cfl_a = mx(cfl_a, __shfl_xor(cfl_a, o, 64));
        cfl_v = mx(cfl_v, __shfl_xor(cfl_v, o, 64));
      }
      if ((threadIdx.x & 63) == 0) part[blockIdx.x] = make_double2(cfl_a, cfl_v);
    }
  }
}

int device_cus() {
  static int cache[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  if (cache[dev] == 0) {
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        cus <= 0)
      cus = 256;
    cache[dev] = cus;
  }
  return cache[dev];
}

afi::StripShape strips_of(const afi::Geo& g) {
  return afi::strip_shape(g.n1x, g.n2y, device_cus(), afi::kSingleCflBlocks);
}

// One object file holds the kernels of one arithmetic type, each with its own
// scheduling: with FP32 stencils there are registers to spare, and ordering the
// instructions for independence of neighbours is worth 5 % (82 -> 78 us at 1000
// x 500); the FP64 kernel spills over a hundred registers that way.
#ifndef AF_STRIP_REAL
#define AF_STRIP_REAL double
#define AF_STRIP_ENTRY(name) name##_fp64
#define AF_STRIP_SHAPES  // (once, in this object)
#else
#define AF_STRIP_ENTRY(name) name##_mixed
#endif
using Real = AF_STRIP_REAL;

hipError_t launch(const afi::Geo& geo, const Phys& ph, const afi::Work& w, const double* Un,
                  const double* Uk, double* Uout, const double* dt_dev, double dt_host,
                  afi::StageCoef sc, hipStream_t s, afi::Timer* tm) {
  const afi::StripShape b = strips_of(geo);
  StripArgs sa{};
  sa.g = afi::stage_geo(geo);
  sa.ph = ph;
  sa.nx = b.nx;
  sa.H = b.H;
  sa.Uk = Uk;
  sa.Un = Un;
  sa.Uout = Uout;
  sa.dt_dev = dt_dev;
  sa.dt_host = dt_host;
  sa.dt_mul = sc.dt_mul;
  sa.flags = w.flags;
  sa.ca = sc.a;
  sa.cb = sc.b;
  sa.first = sc.first;
  sa.shift = sc.skip_flagged ? kStageShift * sc.stage : 0;
  sa.stop_for = sc.skip_flagged == 0 ? 0u : (sc.skip_flagged == 1 ? ~0u : (1u << sa.shift) - 1u);
  sa.blend = sc.blend;
  sa.ts_out = sc.ts_out;
  const dim3 grid((unsigned)(b.nx * b.ny));
  if (sa.blend || sa.ts_out)
    AFI_TIMED(tm, 7, s, hipLaunchKernelGGL((k_strip<Real, true, false>), grid, dim3(NT), 0, s, sa));
  else
    AFI_TIMED(tm, 7, s, hipLaunchKernelGGL((k_strip<Real, false, false>), grid, dim3(NT), 0, s, sa));
  return hipGetLastError();
}

}  // namespace

namespace afi {

#ifdef AF_STRIP_SHAPES
StripShape strip_shape(const Geo& g) { return strips_of(g); }

// A single grid of few columns fills few of a strip's 60, and one of many rows
// too needs more row steps than tiles take.  Fitted to stages of 4 to 15 columns,
// in row steps of 2.23 us (FP64; mixed 1.73): tiles take 5.6 (10.4) a round and 1.8
// (1.7) to start, but no less than 13.3 (23).  Measured, us a stage on strips and
// tiles at 12 columns (FP64; mixed), the line lying between the first two rows and
// between the third and fourth:
//   12 x 1800    29.0, 30.0;  23.2, 37.1
//   12 x 2500    33.8, 29.3;  26.9, 39.7
//   12 x 4000    47.6, 41.5;  37.1, 40.5
//   12 x 5000    56.0, 42.1;  43.8, 39.7
//   12 x 30000   274, 212;    213, 160
// and at 16 columns, two of tiles: 273, 430; 213, 307 for 30000 rows.
bool single_on_tiles(const Geo& g) {
  if (g.n1 >= 16) return false;
  const int cus = device_cus();
  const StripShape b = strips_of(g);
  const long steps = ((long)b.nx * b.ny + cus - 1) / cus * (b.H + 5);
  const long rounds = (default_variant(g.mixed)->tiles(g) + cus - 1) / cus;
  return g.mixed ? 10 * steps > std::max(230L, 104 * rounds + 17)
                 : 10 * steps > std::max(133L, 56 * rounds + 18);
}

// One H for all instances of a batch: the strips of the instances run together,
// in any order, so a launch takes about the steps of all of them over the CUs,
// plus half a strip at its end, but no less than one strip.  (At 1024 rows the
// five steps a strip costs beyond its rows are half a percent: no need to look
// further.)
//
// Whether that beats the tiles is a question of how many of a strip's 60
// columns the grids fill.  A tile (16 x 7 cells FP64, 16 x 14 mixed) takes as
// long as 6.5 or 12 row steps, and the tile kernel's start some 3 or 1 more.
// Measured, us per RK3 step on strips and on the tiles (FP64; mixed):
//   8 grids up to 512 x 256     425, 586;   338, 465
//   2 of 1000 x 500             773, 1563;  647, 1159
//   512 of 64 x 32              1404, 2475; 1150, 2072
//   512 of 16 x 8               407, 646;   397, 518
//   256 of 8 x 8                214, 241;   219, 223
//   32 of 8 x 200               254, 226;   204, 179
bool strip_shapes(const Geo* g, int n, StripShape* out) {
  const int cus = device_cus();
  int tallest = 1;
  for (int i = 0; i < n; ++i) tallest = std::max(tallest, g[i].n2y);
  long best = 0;  // twice the steps
  int best_H = 0;
  for (int H = std::min(4, tallest); H <= std::min(1024, tallest); ++H) {
    long work = 0;
    for (int i = 0; i < n; ++i) {
      const StripShape t = strips_with(g[i].n1x, g[i].n2y, H);
      const int last = g[i].n2y - (t.ny - 1) * H;  // rows of the last range
      work += (long)t.nx * ((long)(t.ny - 1) * (H + 5) + last + 5);
    }
    const long steps =
        std::max(2L * (H + 5), 2 * work / cus + (work > (long)cus * (H + 5) ? H + 5 : 0));
    if (best_H == 0 || steps < best) {
      best = steps;
      best_H = H;
    }
  }
  long tiles = 0;
  for (int i = 0; i < n; ++i) {
    out[i] = strips_with(g[i].n1x, g[i].n2y, best_H);
    tiles += default_variant(g[i].mixed)->tiles(g[i]);
  }
  const long rounds = (tiles + cus - 1) / cus;
  return best <= (g[0].mixed ? 24 * rounds + 2 : 13 * rounds + 6);
}
#endif

hipError_t AF_STRIP_ENTRY(strips)(const Geo& geo, const Phys& ph, const Work& w, const double* Un,
                                  const double* Uk, double* Uout, const double* dt_dev,
                                  double dt_host, StageCoef sc, hipStream_t s, Timer* tm) {
  return launch(geo, ph, w, Un, Uk, Uout, dt_dev, dt_host, sc, s, tm);
}

hipError_t AF_STRIP_ENTRY(strips_dev)(BatchInst* inst, const int* wg_inst, int nwg,
                                      double2* cfl_partial, int k, hipStream_t s) {
  StripArgs sa{};
  sa.inst = inst;
  sa.wg_inst = wg_inst;
  sa.cfl_partial = cfl_partial;
  sa.k = k;
  sa.ca = k == 0 ? 0.0 : (k == 1 ? 0.75 : 1.0 / 3.0);
  sa.cb = k == 0 ? 1.0 : (k == 1 ? 0.25 : 2.0 / 3.0);
  sa.first = k == 0;
  hipLaunchKernelGGL((k_strip<Real, false, true>), dim3((unsigned)nwg), dim3(NT), 0, s, sa);
  return hipGetLastError();
}

}  // namespace afi
