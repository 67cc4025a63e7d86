// af_stage2d.hip -- one stage of a 2D instance, or of a batch of them, on gfx950
// as a single fused, LDS-tiled kernel: the tile variants of af_batch_set_variant
// and af_batch_tune, and the stage of grids too narrow for the strips of
// af_strip2d.hip (batches: strip_shapes, single instances: single_on_tiles),
// which give the same bits.
//
// A workgroup owns a tile of TX x TY cells, i.e. the half-lattice block
// [X0, X0+2TX) x [Y0, Y0+2TY): the cell averages, x-edge, y-edge and corner
// point values inside it.  It stages everything the stage needs for that
// block in LDS and writes only the stage output:
//   phase 0  lattice values on the block +- 4 half cells: ghosts as boundary
//            images, Simpson centres scaled toward the cell average (Sec. 2.2;
//            Remark after the pressure blend, Sec. 3.3), and (u, v, p, T, c)
//   phase 1  D_c gradients of (u, v, T) on the block +- 2 (Sec. 2.2 central
//            operator)
//   phase 2  low-order data of the cells of the tile +- 1: S, F_l, |u_l|+c,
//            b_l, the two smoothness sensors, (u, v, p, T, c) of the average
//            (Sec. 3.1, Sec. 3.2)
//   phase 3  limited face fluxes of the tile's cells: Simpson high-order
//            flux, LLF low-order flux, theta^s, theta^rho theta^p (Sec. 3.3)
//   phase 4  cell-average update and RK combination
//   phase 5a total flux and b of every lattice site the point LLF of Sec.
//            3.4 reads, once per site and direction (beside phase 4)
//   phase 5  point residual (biased inviscid operators with the downwind
//            point, compact D^2, mixed terms; Sec. 2.2), point LLF on the
//            lattice of point values and cell averages and the scaling limiter
//            (Sec. 3.4), wall projection, RK combination; two lanes per
//            point, one per direction
//
// The kernel is a template over the arithmetic type R of the stencils, fluxes
// and residuals (LDS included).  R = double is the FP64 stage.  R = float is
// the mixed-precision stage: stencils and fluxes in FP32, while the density
// and pressure blends (the Theta rule of Sec. 3.3 and 3.4), the cell-average
// update, the point-value update and the low-order point value stay FP64 on
// FP64 data read from the state, and the point sites' (u, v, p, T, c) are
// taken from their FP64 values; the state itself is FP64 in both.
#include "af_scheme2d.hpp"

using namespace afd;

namespace {

// One object file holds one instance: its arithmetic type and tile height
// are set when it is compiled (the FP64 stage with 16 x 7 tiles, the mixed
// stage with 16 x 14 tiles, which its FP32 LDS arrays leave room for), and
// its entry point is afi::AF_STAGE_ENTRY.
#ifndef AF_STAGE_REAL
#define AF_STAGE_REAL double
#endif
#ifndef AF_STAGE_TY
#define AF_STAGE_TY 7
#endif
#ifndef AF_STAGE_ENTRY
#define AF_STAGE_ENTRY stage2d_fp64
#endif
#define AF_CAT2(a, b) a##b
#define AF_CAT(a, b) AF_CAT2(a, b)
#define AF_STAGE_TILES AF_CAT(AF_STAGE_ENTRY, _tiles)
#define AF_STAGE_BATCH AF_CAT(AF_STAGE_ENTRY, _batch)

// tile shape: 16 x TY cells, 512 threads (eight wave64s, two per SIMD)
constexpr int TX = 16, TY = AF_STAGE_TY, NT = 512;
// lattice region [X0-4, X0+2TX+4] x [Y0-4, Y0+2TY+4]: both edges are face
// lines, so every centre inside has its eight neighbours inside
constexpr int WA = 2 * TX + 9, HA = 2 * TY + 9, NA = WA * HA;
constexpr int WG = 2 * TX + 4, HG = 2 * TY + 4, NG = WG * HG;  // block +- 2
constexpr int WC = TX + 2, HC = TY + 2, NC = WC * HC;          // tile cells +- 1
constexpr int NFX = TY * (TX + 1), NFY = (TY + 1) * TX;
constexpr int NCEN = (TX + 4) * (TY + 4);  // centre sites of the lattice region
constexpr int NPT = 3 * TX * TY;           // point DOF sites of a tile
// sites of the low-order point scheme: [X0-1, X0+2TX] x [Y0-1, Y0+2TY], the
// tile's point sites and their lattice neighbours; x-direction data on its
// rows Y0..Y0+2TY-1, y-direction data on its columns X0..X0+2TX-1
constexpr int SW = 2 * TX + 2, SH = 2 * TY + 2, NSR = SW * SH;
constexpr int NSX = SW * 2 * TY, NSY = 2 * TX * SH;

template <typename R>
constexpr bool kFP64 = std::is_same<R, double>::value;

// whether the centre site (X, Y) of the lattice is a ghost beyond a wall or
// outflow side (not a periodic one)
__device__ __forceinline__ bool ghost_centre(const G2& g, int X, int Y) {
  return ((X < 0 || X > 2 * g.n1) && g.bc0 != BC_PERIODIC) ||
         ((Y < 0 || Y > 2 * g.n2) && g.bc2 != BC_PERIODIC);
}

// LDS-resident tile data
template <typename R>
struct Tile {
  R U[4][NA];   // conservative values, block +- 4
  R A[5][NA];   // u, v, p, T, c
  R G[6][NG];   // du/dx dv/dx dT/dx du/dy dv/dy dT/dy, block +- 2
  union {
    R C[23][NC];  // cell low-order data, tile +- 1
    // phase 5: y-direction flux (components 1-3) and b_y of the low-order
    // point scheme's sites, over rows 0-13 of C, which only phase 3 reads
    R SY[4][NSY];
  };
  union {
    // FP32 stencils, phase 2: centre values and their (u, v, p, T, c),
    // staged while the cells read the averages in the centre slots
    R STG[kFP64<R> ? 1 : 9 * NCEN];
    R SX[4][NSX];  // phase 5: x-direction flux (components 1-3) and b_x
  };
  R FX[4][NFX];  // limited x-face fluxes of the tile's cells
  R FY[4][NFY];  // limited y-face fluxes
  // FP64 cell averages of the tile +- 1 for the mixed-precision stage (the
  // FP64 stage reads them from C)
  double AV[4][kFP64<R> ? 1 : NC];
  // mixed-precision stage: the low part V - float(V) of the FP64 value V of
  // each of the tile's point DOFs, so that phase 5 has V to 48 bits from
  // U (the high part) without reading the state again
  float PL[4][kFP64<R> ? 1 : NPT];
  // FP64 stage: the cell averages at the centre sites of the lattice region
  // (the centre slots of U take the Simpson centres in phase 2)
  R AVG[4][kFP64<R> ? NCEN : 1];
};
static_assert(4 * NSY <= 14 * NC, "the y-direction site data fit in rows 0-13 of C");

// auxiliaries (u, v, p, T, c) of LDS lattice site s from its FP64 value V:
// the pressure of a state whose internal energy is a small part of its
// total is a difference of nearly equal numbers, so it is taken in FP64
// before the FP32 stencils see it
template <typename R>
__device__ __forceinline__ void store_aux(Tile<R>& T, const PhysT<double>& pd, int s,
                                          const double* V) {
  R w[5];
  aux_of_fp64(pd, V, w);
#pragma unroll
  for (int k = 0; k < 5; ++k) T.A[k][s] = w[k];
}

// total flux F_d = F^c_d - F^v_d at an LDS site (a: block+-4 index, q: block+-2 index)
template <typename R>
__device__ __forceinline__ void site_flux(const Tile<R>& T, const PhysT<R>& ph, int a, int q,
                                          int d, R* F) {
  const R m1 = T.U[1][a], m2 = T.U[2][a], E = T.U[3][a];
  const R u = T.A[0][a], v = T.A[1][a], p = T.A[2][a];
  R Fv[4];
  visc_flux2(d, u, v, T.G[0][q], T.G[1][q], T.G[2][q], T.G[3][q], T.G[4][q], T.G[5][q], ph, Fv);
  const R ud = d == 0 ? u : v;
  F[0] = (d == 0 ? m1 : m2) - Fv[0];
  F[1] = m1 * ud + (d == 0 ? p : R(0.0)) - Fv[1];
  F[2] = m2 * ud + (d == 1 ? p : R(0.0)) - Fv[2];
  F[3] = (E + p) * ud - Fv[3];
}

// The low-order point scheme works on the half lattice whose point sites hold
// the point values and whose centre sites hold the cell averages (Sec. 3.4
// with the LLF flux of Sec. 3.1).  Sites are addressed by their coordinates
// (lx, ly) in the LDS lattice region; a centre site (both odd) reads the cell
// data of phase 2.
__device__ __forceinline__ int lo_cell(int lx, int ly) {
  return ((ly - 3) >> 1) * WC + ((lx - 3) >> 1);
}
template <typename R>
__device__ __forceinline__ void lo_z(const Tile<R>& T, int lx, int ly, R& u, R& v, R& t) {
  if (lx & ly & 1) {
    const int c = lo_cell(lx, ly);
    u = T.C[18][c];
    v = T.C[19][c];
    t = T.C[21][c];
  } else {
    const int a = ly * WA + lx;
    u = T.A[0][a];
    v = T.A[1][a];
    t = T.A[3][a];
  }
}
// state and (u, v, p, T, c) of a site
template <typename R>
__device__ __forceinline__ void lo_state(const Tile<R>& T, int lx, int ly, R* U, R* w) {
  if (lx & ly & 1) {
    const int c = lo_cell(lx, ly);
#pragma unroll
    for (int k = 0; k < 4; ++k) U[k] = T.C[14 + k][c];
#pragma unroll
    for (int k = 0; k < 5; ++k) w[k] = T.C[18 + k][c];
  } else {
    const int a = ly * WA + lx;
#pragma unroll
    for (int k = 0; k < 4; ++k) U[k] = T.U[k][a];
#pragma unroll
    for (int k = 0; k < 5; ++k) w[k] = T.A[k][a];
  }
}
// low-order gradient at a site: central differences of Z = (u, v, T) over the
// four neighbouring sites, half a cell away
template <typename R>
__device__ __forceinline__ void lo_grad(const Tile<R>& T, int lx, int ly, R ihx, R ihy, R* gr) {
  R um, vm, tm, up, vp, tp;
  lo_z(T, lx - 1, ly, um, vm, tm);
  lo_z(T, lx + 1, ly, up, vp, tp);
  gr[0] = (up - um) * ihx;
  gr[1] = (vp - vm) * ihx;
  gr[2] = (tp - tm) * ihx;
  lo_z(T, lx, ly - 1, um, vm, tm);
  lo_z(T, lx, ly + 1, up, vp, tp);
  gr[3] = (up - um) * ihy;
  gr[4] = (vp - vm) * ihy;
  gr[5] = (tp - tm) * ihy;
}

// x- or y-direction data of the low-order point scheme at a site: the total
// flux F_d (its density component is the momentum, not stored) and b_d, as
// SX/SY entry o
template <typename R>
__device__ __forceinline__ void lo_site(Tile<R>& T, const PhysT<R>& ph, int lx, int ly, R ihx,
                                        R ihy, bool need_x, bool need_y, int ox, int oy) {
  R U[4], w[5], gr[6];
  lo_state(T, lx, ly, U, w);
  lo_grad(T, lx, ly, ihx, ihy, gr);
#pragma unroll
  for (int d = 0; d < 2; ++d) {
    if (!(d == 0 ? need_x : need_y)) continue;
    R F[4];
    tot_flux(d, U, w[0], w[1], w[2], gr, ph, F);
    const R b = bvisc2_dir(d, w[2], w[3], gr[0], gr[1], gr[2], gr[3], gr[4], gr[5], ph);
    R* S = d == 0 ? &T.SX[0][0] : &T.SY[0][0];
    const int n = d == 0 ? NSX : NSY, o = d == 0 ? ox : oy;
    S[o] = F[1];
    S[n + o] = F[2];
    S[2 * n + o] = F[3];
    S[3 * n + o] = b;
  }
}

// direction-d part of the low-order point update of Sec. 3.4: the point at
// (lx, ly) moves by U^L - U = -sum_d L_d with
// L_d = (2 dt/h_d) (F^L(z, z+e_d) - F^L(z-e_d, z)) and the LLF flux
// F^L(a, b) = (F_a + F_b)/2 - (max(|u_d|+c) + max(b_d))/2 (U_b - U_a),
// from the site data of lo_site.  d is a lane value (lanes of one wave take
// either direction)
template <typename R>
__device__ __forceinline__ void lo_point_dir(const Tile<R>& T, int lx, int ly, int d, double h,
                                             double dt, R* L) {
  R U0[4], w0[5];
  lo_state(T, lx, ly, U0, w0);
  const int sx = lx - 3, sy = ly - 3;
  const R* S = d ? &T.SY[0][0] : &T.SX[0][0];
  const int n = d ? NSY : NSX;
  const int o0 = d ? sy * (2 * TX) + sx - 1 : (sy - 1) * SW + sx;
  const int st = d ? 2 * TX : 1;
  const R F0[4] = {d ? U0[2] : U0[1], S[o0], S[n + o0], S[2 * n + o0]};
  const R b0 = S[3 * n + o0];
  const R r0 = fabs(d ? w0[1] : w0[0]) + w0[4];
  R Fp[4];
#pragma unroll
  for (int sg = 1; sg >= -1; sg -= 2) {
    const int nx = lx + (d ? 0 : sg), ny = ly + (d ? sg : 0);
    const int on = o0 + sg * st;
    R Un[4], wn[5];
    lo_state(T, nx, ny, Un, wn);
    const R Fn[4] = {d ? Un[2] : Un[1], S[on], S[n + on], S[2 * n + on]};
    const R bn = S[3 * n + on];
    const R lam = mx(r0, fabs(d ? wn[1] : wn[0]) + wn[4]) + mx(b0, bn);
    if (sg == 1) {
#pragma unroll
      for (int k = 0; k < 4; ++k)
        Fp[k] = R(0.5) * (F0[k] + Fn[k]) - R(0.5) * lam * (Un[k] - U0[k]);
    } else {
      const R c = R(2.0 * dt / h);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const R Fm = R(0.5) * (Fn[k] + F0[k]) - R(0.5) * lam * (U0[k] - Un[k]);
        L[k] = c * (Fp[k] - Fm);
      }
    }
  }
}

// value of x in the other lane of this lane's pair (lanes 2m and 2m+1), by
// a quad permutation (1, 0, 3, 2)
__device__ __forceinline__ float pair_swap(float x) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0xB1, 0xF, 0xF, false));
}
__device__ __forceinline__ double pair_swap(double x) {
  const long long v = __double_as_longlong(x);
  const int lo = __builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_mov_dpp((int)(v >> 32), 0xB1, 0xF, 0xF, false);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// direction-d terms of the residual of the point at LDS site a (block +- 2
// index q), in components (rho, m_x, m_y, E): the biased inviscid operators
// with the downwind point, written as D+(F+) + D-(F-) = D_c(F) + alpha/(6h)
// times the fourth difference with alpha the max of |u_d| + c over the five
// sites of the line; the compact D^{(d),2}(K_dd, Z); the mixed term
// D_c^{(d)}(K_{d,o} D_c^{(o)} Z) with o the other direction (Sec. 2.2).  It
// is computed in components (rho, m_d, m_o, E), m_d the momentum along d and
// m_o the other, with a the velocity along d and b the other, so that both
// directions run the same instructions (d may differ between the lanes of a
// wave)
template <typename R>
__device__ __forceinline__ void point_resid_dir(const Tile<R>& T, const PhysT<R>& ph, int a, int q,
                                                int d, double h, R* Rd) {
  const int sa = d ? WA : 1, sq = d ? WG : 1;
  const R* Md = T.U[1 + d];
  const R* Mo = T.U[2 - d];
  const R* Va = T.A[d];
  const R* Vb = T.A[1 - d];
  // derivatives across d of the velocity along d and of the other one
  const R* Ga = T.G[d ? 1 : 3];
  const R* Gb = T.G[d ? 0 : 4];
  R sp[5], ga[5], gb[5], Rr[4];
#pragma unroll
  for (int o = 0; o < 5; ++o) {
    const int b = a + (o - 2) * sa, qq = q + (o - 2) * sq;
    sp[o] = fabs(Va[b]) + T.A[4][b];
    ga[o] = o == 2 ? R(0.0) : Ga[qq];
    gb[o] = o == 2 ? R(0.0) : Gb[qq];
  }
  line_terms(
      ph, h, mx5(sp[0], sp[1], sp[2], sp[3], sp[4]),
      [&](LineValue v, int o) {
        const int b = a + (o - 2) * sa;
        return v == kRho  ? T.U[0][b]
               : v == kMd ? Md[b]
               : v == kMo ? Mo[b]
               : v == kE  ? T.U[3][b]
               : v == kVa ? Va[b]
               : v == kVb ? Vb[b]
               : v == kP  ? T.A[2][b]
                          : T.A[3][b];
      },
      ga, gb, Rr);
  // back to (rho, m_x, m_y, E)
  Rd[0] = Rr[0];
  Rd[1] = d ? Rr[2] : Rr[1];
  Rd[2] = d ? Rr[1] : Rr[2];
  Rd[3] = Rr[3];
}

// raw values of the lattice region of the tile at (X0, Y0): point sites hold
// their DOF, centre sites the cell average, ghosts as boundary images.  Each
// thread gathers the sites tid, tid+NT, tid+2NT into registers, with the
// image's momentum sign flips as bits: the loads are only issued here, and
// nothing waits for them before the values are stored to LDS.
constexpr int kRawPerThread = (NA + NT - 1) / NT;

__device__ __forceinline__ void load_raw(const G2& g, const double* __restrict__ Uk, int X0, int Y0,
                                         int tid, double (&pre)[kRawPerThread][4],
                                         int (&flip)[kRawPerThread]) {
  const int Xlim = 2 * __builtin_amdgcn_readfirstlane(g.n1);
  const int Ylim = 2 * __builtin_amdgcn_readfirstlane(g.n2);
  // a region inside the grid on both axes (no ghost site, no periodic seam):
  // every site is read where it is, with no image map
  if (X0 >= 4 && X0 - 4 + WA <= Xlim && Y0 >= 4 && Y0 - 4 + HA <= Ylim) {
#pragma unroll
    for (int r = 0; r < kRawPerThread; ++r) {
      const int s = tid + r * NT;
      if (s >= NA) continue;
      flip[r] = 0;
      long o;
      int st;
      site_ofs(g, X0 - 4 + s % WA, Y0 - 4 + s / WA, o, st);
      const double* src = Uk + o;
#pragma unroll
      for (int k = 0; k < 4; ++k) pre[r][k] = src[(long)k * st];
    }
    return;
  }
#pragma unroll
  for (int r = 0; r < kRawPerThread; ++r) {
    const int s = tid + r * NT;
    const int X = X0 - 4 + s % WA, Y = Y0 - 4 + s / WA;
    if (s >= NA || X > Xlim + kMargin || Y > Ylim + kMargin) continue;
    int kx, ky;
    const int Xi = axis_image(X, Xlim, g.bc0, g.bc1, kx);
    const int Yi = axis_image(Y, Ylim, g.bc2, g.bc3, ky);
    flip[r] = image_flips(kx, ky);
    long o;
    int st;
    site_ofs(g, Xi, Yi, o, st);
    const double* src = Uk + o;
#pragma unroll
    for (int k = 0; k < 4; ++k) pre[r][k] = src[(long)k * st];
  }
}

// Tiles are visited by persistent workgroups.  Workgroups are dispatched to
// the eight XCDs round-robin by index, so the tiles are cut into eight
// contiguous bands, one per XCD: neighbouring tiles (whose lattice regions
// overlap) are then read through the same L2.
struct TileIter {
  int cur, end, step;
  __device__ TileIter(int ntiles, int wg, int nwg) {
    if (nwg >= 8 && nwg % 8 == 0) {
      const int xcd = wg % 8, local = wg / 8;
      cur = (int)((long)xcd * ntiles / 8) + local;
      end = (int)((long)(xcd + 1) * ntiles / 8);
      step = nwg / 8;
    } else {
      cur = wg;
      end = ntiles;
      step = nwg;
    }
  }
  __device__ int get() const { return cur < end ? cur : -1; }
  __device__ int advance() {
    cur += step;
    return get();
  }
};

// launch arguments of a stage: one instance, or a batch of 2D instances
constexpr int kMaxBatch = 512;
struct StageArgs {
  // one instance, its step driven by the host
  G2 g;
  Phys ph;
  const double* Uk;
  const double* Un;
  double* Uout;
  const double* dt_dev;
  double dt_host, dt_mul;  // the step is dt_mul * dt
  unsigned* flags;
  int ntx;
  const float* blend;  // see limit_face
  float* ts_out;
  // a batch: its instances (stage k reads and writes their rotating buffers)
  afi::BatchInst* inst;
  int ninst, k;
  const int* n_active;
  // both
  double ca, cb;
  int first, skip_flagged, ntiles;
};

// what one tile of a stage works on.  Geometry and physics are referenced,
// not copied: a copy would hold some thirty uniform values live across the
// whole tile (register pressure of a kernel that is at its VGPR limit), while
// a reference to the kernel arguments or to the batch descriptor in global
// memory is re-read where needed.
struct TileArgs {
  const G2* g;
  const Phys* phd;
  const double* Uk;
  const double* Un;
  double* Uout;
  double dt;
  unsigned* flags;
  int ntx, lt;  // tiles along x of its grid, the tile's index in its grid
};

// position of tile t in a batch's list of n active instances whose first
// tiles are t0[0] = 0 < t0[1] < ...
__device__ __forceinline__ int batch_slot_of(const int* t0, int n, int t) {
  int lo = 0, hi = n - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (t0[mid] <= t)
      lo = mid;
    else
      hi = mid - 1;
  }
  return lo;
}

// tile t of the active tiles of a batch: active instance j is instance
// id[j] and owns tiles [t0[j], t0[j + 1])
__device__ __forceinline__ TileArgs batch_tile(const StageArgs& sa, const int* t0, const int* id,
                                               int nact, int t) {
  // the instance is the same for the whole workgroup
  const int j = __builtin_amdgcn_readfirstlane(batch_slot_of(t0, nact, t));
  const int in = __builtin_amdgcn_readfirstlane(id[j]);
  const afi::BatchInst& I = sa.inst[in];
  TileArgs A;
  A.g = &I.g;
  A.phd = &I.ph;
  A.ntx = I.ntx;
  A.lt = t - t0[j];
  A.dt = I.dt;
  A.flags = &sa.inst[in].flags;
  // the three RK3 stages from buf[cur], through the other two buffers
  const int c = I.cur, a = (c + 1) % 3, b = (c + 2) % 3;
  A.Un = I.buf[c];
  A.Uk = sa.k == 0 ? I.buf[c] : (sa.k == 1 ? I.buf[a] : I.buf[b]);
  A.Uout = sa.k == 1 ? I.buf[b] : I.buf[a];
  return A;
}

// BLEND: one instance with per-face blend input/output arrays (a kernel of its
// own, so that the plain stage carries none of that code)
template <typename R, bool BATCH, bool BLEND = false>
__global__ void __launch_bounds__(NT) k_stage(StageArgs sa) {
  __shared__ Tile<R> T;
  __shared__ unsigned stop;  // workgroup-uniform copy of the flag word
  const int tid = threadIdx.x;
  const double ca = sa.ca, cb = sa.cb;
  const int first = sa.first, skip_flagged = sa.skip_flagged;
  bool nonfinite = false;
  // a batch: only the tiles of its active instances are numbered, so that
  // every XCD band holds an equal share of the work whichever instances are
  // active (instances finish their steps after different numbers of
  // attempts).  Active instance j is instance bid[j] and owns tiles
  // [bt0[j], bt0[j] + its ntiles); the numbering comes from two inclusive
  // scans over the instances (one per thread), done in place in bt0 / bid.
  __shared__ int bt0[BATCH ? kMaxBatch : 1], bid[BATCH ? kMaxBatch : 1];
  int ntiles = sa.ntiles, nact = 1;
  if constexpr (BATCH) {
    static_assert(kMaxBatch == NT, "one instance per thread in the scans");
    if (*sa.n_active == 0) return;  // every instance has finished its step
  }
  if (BATCH && sa.ninst == 1) {
    // one instance, active (n_active is not 0): its tiles are all the tiles
    if (tid == 0) {
      bid[0] = 0;
      bt0[0] = 0;
    }
    ntiles = sa.inst[0].ntiles;
    __syncthreads();
  } else if constexpr (BATCH) {
    const bool act = tid < sa.ninst && sa.inst[tid].active;
    const int own = act ? sa.inst[tid].ntiles : 0;
    bid[tid] = act ? 1 : 0;
    bt0[tid] = own;
    __syncthreads();
    for (int off = 1; off < NT; off <<= 1) {
      const int c = tid >= off ? bid[tid - off] : 0;
      const int t = tid >= off ? bt0[tid - off] : 0;
      __syncthreads();
      bid[tid] += c;
      bt0[tid] += t;
      __syncthreads();
    }
    const int pos = bid[tid] - 1, first_tile = bt0[tid] - own;
    nact = bid[NT - 1];
    ntiles = bt0[NT - 1];
    __syncthreads();
    if (act) {
      bid[pos] = tid;
      bt0[pos] = first_tile;
    }
    __syncthreads();
  }
  // the one instance's dt, read once (a read per tile costs 3 % of the stage)
  double dt1 = 0.0;
  if constexpr (!BATCH) dt1 = sa.dt_mul * (sa.dt_dev ? *sa.dt_dev : sa.dt_host);
  // what tile t works on (built where used, from the kernel arguments or the
  // batch descriptors, so that nothing of it stays live across tiles)
  auto args = [&](int t) {
    if constexpr (BATCH)
      return batch_tile(sa, bt0, bid, nact, t);
    else
      return TileArgs{&sa.g, &sa.ph, sa.Uk, sa.Un, sa.Uout, dt1, sa.flags, sa.ntx, t};
  };
  TileIter it(ntiles, blockIdx.x, gridDim.x);
  int tile = it.get();
  double pre[kRawPerThread][4];
  int flip[kRawPerThread] = {};
  // a batch: whether pre holds the current tile's raw values (tiles of an
  // instance whose attempt is rejected are passed over without loading them)
  bool have_pre = true;
  if (tile >= 0) {
    const TileArgs A = args(tile);
    load_raw(*A.g, A.Uk, 2 * TX * (A.lt % A.ntx), 2 * TY * (A.lt / A.ntx), tid, pre, flip);
  }
  while (tile >= 0) {
  const TileArgs A = args(tile);
  const G2& g = *A.g;
  const Phys& phd = *A.phd;
  const PhysT<R> ph = phys_as<R>(phd);
  const PhysT<double> phd64 = phys_as<double>(phd);
  const double* __restrict__ Uk = A.Uk;
  const double* __restrict__ Un = A.Un;
  double* __restrict__ Uout = A.Uout;
  const double dt = A.dt;
  unsigned* flags = A.flags;
  const int Xlim = 2 * g.n1, Ylim = 2 * g.n2;
  const int i0 = (A.lt % A.ntx) * TX, j0 = (A.lt / A.ntx) * TY;
  const int X0 = 2 * i0, Y0 = 2 * j0;
  // inside a step attempt, stop once any workgroup has flagged the attempt:
  // it is rejected and this output is never read (a batch skips the tiles of
  // that instance only)
  if (tid == 0) stop = skip_flagged ? peek_flags(flags) : 0u;
  __syncthreads();  // the previous tile is done with the LDS; stop is visible
  if (stop) {
    // with one active instance every later tile is that instance's too
    if (nact == 1) break;
    // every wave has read `stop` before thread 0 writes it for the next
    // tile, which is loaded only once it is known not to be skipped too
    __syncthreads();
    tile = it.advance();
    have_pre = false;
    continue;
  }
  if (!have_pre) {
    load_raw(g, Uk, X0, Y0, tid, pre, flip);
    have_pre = true;
  }

  // ---- phase 0a: raw values of the lattice region (prefetched) ----
#pragma unroll
  for (int r = 0; r < kRawPerThread; ++r) {
    const int s = tid + r * NT;
    const int X = X0 - 4 + s % WA, Y = Y0 - 4 + s / WA;
    if (s >= NA || X > Xlim + kMargin || Y > Ylim + kMargin) continue;
    double V[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const bool neg = (k == 1 && (flip[r] & 1)) || (k == 2 && (flip[r] & 2));
      V[k] = neg ? -pre[r][k] : pre[r][k];
    }
    if constexpr (kFP64<R>) {
      // FP64: averages to AVG, point values to U
      if ((X & 1) && (Y & 1)) {
        const int ci = ((s / WA - 1) >> 1) * (TX + 4) + ((s % WA - 1) >> 1);
#pragma unroll
        for (int k = 0; k < 4; ++k) T.AVG[k][ci] = V[k];
      } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) T.U[k][s] = V[k];
      }
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k) T.U[k][s] = R(V[k]);
    }
    // FP32 stencils: the point sites' (u, v, p, T, c) from the FP64 values
    // (centre sites get the Simpson centre's); the FP64 stage takes them in
    // phase 2, where they cost fewer live registers.  The FP64 averages of
    // the tile's cells +- 1 go to AV, and the low parts of the FP64 values
    // of the tile's own points to PL, for the FP64 updates
    if constexpr (!kFP64<R>) {
      const int lx = X - X0, ly = Y - Y0;
      if ((X & 1) && (Y & 1)) {
        const int ci = (lx + 1) >> 1, cj = (ly + 1) >> 1;  // cell offset + 1
        if (lx >= -1 && ly >= -1 && ci <= TX + 1 && cj <= TY + 1) {
#pragma unroll
          for (int k = 0; k < 4; ++k) T.AV[k][cj * WC + ci] = V[k];
        }
      } else {
        store_aux(T, phd64, s, V);
        if (lx >= 0 && ly >= 0 && lx < 2 * TX && ly < 2 * TY) {
          // point type 0 x-edge (X even, Y odd), 1 y-edge, 2 corner
          const int pt = (X & 1) ? 1 : ((Y & 1) ? 0 : 2);
          const int pi = pt * (TX * TY) + (ly >> 1) * TX + (lx >> 1);
#pragma unroll
          for (int k = 0; k < 4; ++k) T.PL[k][pi] = float(V[k] - double(float(V[k])));
        }
      }
    }
  }
  __syncthreads();

  // ---- phase 2: centre values (Simpson + scaling; waves 4-7, compact
  //      mapping, staged until the cells have read the averages in the centre
  //      slots), cell low-order data of the tile +- 1 (waves 0-2),
  //      auxiliaries of the point sites (all; FP64 stage only, the FP32
  //      stencils took theirs in phase 0a) ----
  // lattice slot of centre cidx of the region, or -1 beyond the grid's ghosts
  auto centre_slot = [&](int cidx) {
    const int X = X0 - 3 + 2 * (cidx % (TX + 4)), Y = Y0 - 3 + 2 * (cidx / (TX + 4));
    return (X <= Xlim + kMargin && Y <= Ylim + kMargin) ? (Y - Y0 + 4) * WA + (X - X0 + 4) : -1;
  };
  for (int cidx = tid - NT / 2; cidx >= 0 && cidx < NCEN; cidx += NT / 2) {
    const int cs = centre_slot(cidx);
    const int X = X0 - 3 + 2 * (cidx % (TX + 4)), Y = Y0 - 3 + 2 * (cidx / (TX + 4));
    // a centre beyond a wall or outflow side is taken from its image below;
    // periodic ghosts are computed here, from the wrapped values
    if (cs >= 0 && !ghost_centre(g, X, Y)) {
      R Ub[4], e[4], cc[4], cV[4], cw[5];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const R* z = T.U[k];
        Ub[k] = kFP64<R> ? T.AVG[k][cidx] : z[cs];
        e[k] = z[cs - 1] + z[cs + 1] + z[cs - WA] + z[cs + WA];
        cc[k] = z[cs - WA - 1] + z[cs - WA + 1] + z[cs + WA - 1] + z[cs + WA + 1];
      }
      centre_value(ph, phd, Ub, e, cc, cV, cw);
      if constexpr (kFP64<R>) {
        // the cells read the averages from AVG: the centre goes in place
#pragma unroll
        for (int k = 0; k < 4; ++k) T.U[k][cs] = cV[k];
#pragma unroll
        for (int k = 0; k < 5; ++k) T.A[k][cs] = cw[k];
      } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) T.STG[k * NCEN + cidx] = cV[k];
#pragma unroll
        for (int k = 0; k < 5; ++k) T.STG[(4 + k) * NCEN + cidx] = cw[k];
      }
    }
  }
  // cells: the first NT/2 on waves 0-3, the rest from the top thread down
  // (waves 7, 6, ...), away from the waves 4 and 5 that take the centres'
  // second round when there is one
  static_assert(NC <= NT, "one cell per thread");
  {
    const int s = tid < NT / 2 ? tid : NT / 2 + (NT - 1 - tid);
    const int i = i0 - 1 + s % WC, j = j0 - 1 + s / WC;
    if (s < NC && i <= g.n1 && j <= g.n2) {
    CellAvg<R> C0, Cxm, Cxp, Cym, Cyp;
    R o[23];
    if constexpr (kFP64<R>) {
      // the cell's index among the centres of the region
      const int c = (s / WC + 1) * (TX + 4) + s % WC + 1;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        C0.U[k] = T.AVG[k][c];
        Cxm.U[k] = T.AVG[k][c - 1];
        Cxp.U[k] = T.AVG[k][c + 1];
        Cym.U[k] = T.AVG[k][c - (TX + 4)];
        Cyp.U[k] = T.AVG[k][c + (TX + 4)];
      }
    } else {
      const int a = (2 * j + 1 - Y0 + 4) * WA + (2 * i + 1 - X0 + 4);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        C0.U[k] = T.U[k][a];
        Cxm.U[k] = T.U[k][a - 2];
        Cxp.U[k] = T.U[k][a + 2];
        Cym.U[k] = T.U[k][a - 2 * WA];
        Cyp.U[k] = T.U[k][a + 2 * WA];
      }
    }
    // one reciprocal density per cell
    for (CellAvg<R>* c : {&C0, &Cxm, &Cxp, &Cym, &Cyp}) {
      c->r = rcp(c->U[0]);
      c->p = pressure_r(ph, c->U, c->r);
    }
    const R u0 = C0.U[1] * C0.r, v0 = C0.U[2] * C0.r;
    const R c0 = root(ph.gam * C0.p * C0.r);
    // 0-11 see cell_low, 12 phi1, 13 phi2, 14-17 the average, 18-22 its
    // (u, v, p, T, c)
    cell_low(g, ph, C0, Cxm, Cxp, Cym, Cyp, c0, o);
    cell_sensors(g, C0, Cxm, Cxp, Cym, Cyp, o + 12);
#pragma unroll
    for (int k = 0; k < 4; ++k) o[14 + k] = C0.U[k];
    o[18] = u0;
    o[19] = v0;
    o[20] = C0.p;
    o[21] = C0.p * C0.r;
    o[22] = c0;
#pragma unroll
    for (int k = 0; k < 23; ++k) T.C[k][s] = o[k];
    }
  }
  if constexpr (kFP64<R>) {
    // the point sites of the lattice region, numbered p: each pair of rows
    // (an even one, all 41 sites points; an odd one, its 21 even sites)
    // holds 62 of them, so no lane falls on a centre
    constexpr int PPR = WA + (WA + 1) / 2;  // points per pair of rows
    constexpr int NPS = (HA + 1) / 2 * WA + HA / 2 * ((WA + 1) / 2);
    auto aux_point = [&](int p) {
      const int r2 = p / PPR, m = p % PPR;
      const int ly = m < WA ? 2 * r2 : 2 * r2 + 1, lx = m < WA ? m : 2 * (m - WA);
      const int s = ly * WA + lx;
      const int X = X0 - 4 + lx, Y = Y0 - 4 + ly;
      if (X > Xlim + kMargin || Y > Ylim + kMargin) return;
      const double V[4] = {T.U[0][s], T.U[1][s], T.U[2][s], T.U[3][s]};
      store_aux(T, phd64, s, V);
    };
    // one site per thread, then the rest on waves 3 and 7: the SIMD they
    // share (waves go to the SIMDs round-robin) updates no cells
    if (tid < NPS) aux_point(tid);
    const int wv = tid >> 6;
    if (wv == 3 || wv == 7) {
      for (int p = NT + (tid & 63) + (wv == 7 ? 64 : 0); p < NPS; p += 128) aux_point(p);
    }
  }
  __syncthreads();
  if constexpr (!kFP64<R>) {
    for (int cidx = tid - NT / 2; cidx >= 0 && cidx < NCEN; cidx += NT / 2) {
      const int cs = centre_slot(cidx);
      if (cs < 0) continue;
#pragma unroll
      for (int k = 0; k < 4; ++k) T.U[k][cs] = T.STG[k * NCEN + cidx];
#pragma unroll
      for (int k = 0; k < 5; ++k) T.A[k][cs] = T.STG[(4 + k) * NCEN + cidx];
    }
    __syncthreads();
  }
  // ghost centres: the value and (u, v, p, T, c) of the image centre, with
  // the image's momentum and velocity signs.  Ghosts reach at most four
  // lattice lines past a side, so the image (a mirror or the first interior
  // centre; along a periodic axis the unwrapped ghost itself) lies in this
  // tile's region, and phase 2 computed it from the same values in the same
  // order as the image's own Simpson value: the copy is that value exactly
  if (!(X0 >= 4 && X0 - 4 + WA <= Xlim && Y0 >= 4 && Y0 - 4 + HA <= Ylim)) {
    for (int cidx = tid; cidx < NCEN; cidx += NT) {
      const int cs = centre_slot(cidx);
      const int X = X0 - 3 + 2 * (cidx % (TX + 4)), Y = Y0 - 3 + 2 * (cidx / (TX + 4));
      if (cs < 0 || !ghost_centre(g, X, Y)) continue;
      int kx = -1, ky = -1;
      const int Xi = g.bc0 == BC_PERIODIC ? X : axis_image(X, Xlim, g.bc0, g.bc1, kx);
      const int Yi = g.bc2 == BC_PERIODIC ? Y : axis_image(Y, Ylim, g.bc2, g.bc3, ky);
      const int f = image_flips(kx, ky);
      const int si = (Yi - Y0 + 4) * WA + (Xi - X0 + 4);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const R v = T.U[k][si];
        T.U[k][cs] = ((k == 1 && (f & 1)) || (k == 2 && (f & 2))) ? -v : v;
      }
#pragma unroll
      for (int k = 0; k < 5; ++k) {
        const R v = T.A[k][si];
        T.A[k][cs] = ((k == 0 && (f & 1)) || (k == 1 && (f & 2))) ? -v : v;
      }
    }
    __syncthreads();
  }

  // prefetch the next tile's raw values; the loads complete while this tile
  // computes
  const int next = it.advance();
  if (next >= 0) {
    const TileArgs An = args(next);
    load_raw(*An.g, An.Uk, 2 * TX * (An.lt % An.ntx), 2 * TY * (An.lt / An.ntx), tid, pre, flip);
  }

  // ---- phase 1: gradients on the block +- 2 ----
  {
    const R ihx = R(1.0 / (6.0 * g.dx)), ihy = R(1.0 / (6.0 * g.dy));
    for (int s = tid; s < NG; s += NT) {
      const int lx = s % WG, ly = s / WG;
      const int X = X0 - 2 + lx, Y = Y0 - 2 + ly;
      if (X > Xlim + 2 || Y > Ylim + 2) continue;
      const int a = (ly + 2) * WA + (lx + 2);
      R gr[6];
      const int src[3] = {0, 1, 3};
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const R* z = T.A[src[c]];
        gr[c] = dc5(z[a - 2], z[a - 1], z[a + 1], z[a + 2], ihx);
        gr[3 + c] = dc5(z[a - 2 * WA], z[a - WA], z[a + WA], z[a + 2 * WA], ihy);
      }
#pragma unroll
      for (int c = 0; c < 6; ++c) T.G[c][s] = gr[c];
    }
  }
  __syncthreads();

  // ---- phase 3: limited face fluxes of the tile's cells ----
  const float* blend = BLEND ? sa.blend : nullptr;
  float* ts_out = BLEND ? sa.ts_out : nullptr;
  const int limc = (ph.lim & (LIM_SMOOTH | LIM_PP | LIM_LOWONLY)) | (blend ? 1 : 0);
  // FP64: the faces take waves 0-3 only; waves 4-7 compute the
  // x-direction site data of the low-order point scheme meanwhile (phase 5a
  // keeps the y-direction data, which overlay cell data the faces read)
  if constexpr (kFP64<R>) {
    static_assert(!kFP64<R> || NFX + NFY <= NT / 2, "the faces on waves 0-3");
    if ((ph.lim & LIM_POINT) && tid >= NT / 2) {
      const R ihx = R(1.0 / g.dx), ihy = R(1.0 / g.dy);
      for (int s = tid - NT / 2; s < NSX; s += NT / 2) {
        const int sx = s % SW, sy = 1 + s / SW;
        lo_site(T, ph, sx + 3, sy + 3, ihx, ihy, true, false, (sy - 1) * SW + sx, 0);
      }
    }
  }
  for (int s = tid; s < NFX + NFY; s += NT) {
    const int d = s < NFX ? 0 : 1;
    int ff, jj, i, j, X, Y;  // face (i,j) between cells a (minus) and b (plus)
    if (d == 0) {
      ff = s % (TX + 1);
      jj = s / (TX + 1);
      i = i0 + ff;
      j = j0 + jj;
      if (i > g.n1 || j >= g.n2) continue;
      X = 2 * i;
      Y = 2 * j + 1;
    } else {
      const int r = s - NFX;
      ff = r % TX;
      jj = r / TX;
      i = i0 + ff;
      j = j0 + jj;
      if (i >= g.n1 || j > g.n2) continue;
      X = 2 * i + 1;
      Y = 2 * j;
    }
    const int a = (Y - Y0 + 4) * WA + (X - X0 + 4);
    const int q = (Y - Y0 + 2) * WG + (X - X0 + 2);
    const int sa = d == 0 ? WA : 1, sq = d == 0 ? WG : 1;  // along the face
    R Fa[4], Fm[4], Fb[4], FH[4], F[4];
    site_flux(T, ph, a - sa, q - sq, d, Fa);
    site_flux(T, ph, a, q, d, Fm);
    site_flux(T, ph, a + sa, q + sq, d, Fb);
#pragma unroll
    for (int k = 0; k < 4; ++k) FH[k] = (Fa[k] + R(4.0) * Fm[k] + Fb[k]) * R(1.0 / 6.0);
    if (!limc) {
#pragma unroll
      for (int k = 0; k < 4; ++k) F[k] = FH[k];
    } else {
      const int cbx = (j - j0 + 1) * WC + (i - i0 + 1);
      const int cax = d == 0 ? cbx - 1 : cbx - WC;
      const R lam = mx(T.C[8 + d][cax], T.C[8 + d][cbx]) + mx(T.C[10 + d][cax], T.C[10 + d][cbx]);
      R FL[4], Fca[4], Fcb[4];
      double Ua[4], Ub[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if constexpr (kFP64<R>) {
          Ua[k] = T.C[14 + k][cax];
          Ub[k] = T.C[14 + k][cbx];
        } else {
          Ua[k] = T.AV[k][cax];
          Ub[k] = T.AV[k][cbx];
        }
        Fca[k] = T.C[4 * d + k][cax];
        Fcb[k] = T.C[4 * d + k][cbx];
        FL[k] = R(0.5) * (Fca[k] + Fcb[k]) - R(0.5) * lam * (T.C[14 + k][cbx] - T.C[14 + k][cax]);
      }
      FaceCells<R> fc;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        fc.Ua[k] = Ua[k];
        fc.Ub[k] = Ub[k];
        fc.Fa[k] = Fca[k];
        fc.Fb[k] = Fcb[k];
        fc.FL[k] = FL[k];
      }
      fc.phi1 = mx(T.C[12][cax], T.C[12][cbx]);
      fc.phi2 = mx(T.C[13][cax], T.C[13][cbx]);
      limit_face(g, ph, phd, d, i, j, dt, fc, FH, blend, ts_out, true, flags, FLAG_CELL_LOW, F);
    }
    if (d == 0) {
#pragma unroll
      for (int k = 0; k < 4; ++k) T.FX[k][jj * (TX + 1) + ff] = F[k];
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k) T.FY[k][jj * TX + ff] = F[k];
    }
  }
  __syncthreads();

  // ---- phase 4: cell averages (FP64 accumulation) ----
  {
    const double mxd = dt / g.dx, myd = dt / g.dy;
    const long nc = (long)g.n1 * g.n2;
    for (int s = tid; s < TX * TY; s += NT) {
      const int ii = s % TX, jj = s / TX;
      const int i = i0 + ii, j = j0 + jj;
      if (i >= g.n1 || j >= g.n2) continue;
      const int c = (jj + 1) * WC + ii + 1;
      const long gi = (long)j * g.n1 + i;
      // U^n of the cell, all four loads in flight together
      double un[4] = {0.0, 0.0, 0.0, 0.0};
      if (!first) {
#pragma unroll
        for (int k = 0; k < 4; ++k) un[k] = Un[k * nc + gi];
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const double dfx = double(T.FX[k][jj * (TX + 1) + ii + 1]) - double(T.FX[k][jj * (TX + 1) + ii]);
        const double dfy = double(T.FY[k][(jj + 1) * TX + ii]) - double(T.FY[k][jj * TX + ii]);
        double av;
        if constexpr (kFP64<R>)
          av = T.C[14 + k][c];
        else
          av = T.AV[k][c];
        const double fe = av - mxd * dfx - myd * dfy;
        const double o = first ? fe : ca * un[k] + cb * fe;
        if (!isfinite(o)) nonfinite = true;
        Uout[k * nc + gi] = o;
      }
    }
  }

  // ---- phase 5a: site data of the low-order point scheme (Sec. 3.4); it
  //      shares no LDS with phase 4, and starts on the threads phase 4 leaves
  //      idle ----
  if (ph.lim & LIM_POINT) {
    const R ihx = R(1.0 / g.dx), ihy = R(1.0 / g.dy);
    auto site = [&](int s) {
      const int sx = s % SW, sy = s / SW;
      const bool need_x = !kFP64<R> && sy >= 1 && sy <= 2 * TY, need_y = sx >= 1 && sx <= 2 * TX;
      if (need_x || need_y)
        lo_site(T, ph, sx + 3, sy + 3, ihx, ihy, need_x, need_y, (sy - 1) * SW + sx,
                sy * (2 * TX) + sx - 1);
    };
    if constexpr (kFP64<R>) {
      // the y-direction data (the x-direction data came during phase 3)
      const int s = (tid + NT - TX * TY) % NT;
      if (s < NSY) {
        const int sx = 1 + s % (2 * TX), sy = s / (2 * TX);
        lo_site(T, ph, sx + 3, sy + 3, ihx, ihy, false, true, 0, sy * (2 * TX) + sx - 1);
      }
      static_assert(!kFP64<R> || NSY <= NT, "one site per thread");
    } else {
      // the first NT sites from the first thread phase 4 leaves idle on; the
      // rest from wave 3 on, away from the waves that also update cells
      const int s1 = (tid + NT - TX * TY) % NT;
      if (s1 < NSR) site(s1);
      for (int s = NT + (tid + NT - 192) % NT; s < NSR; s += NT) site(s);
    }
    __syncthreads();
  }

  // ---- phase 5: point values (0 x-edge, 1 y-edge, 2 corner points).  The
  //      FP64 stage gives each point two lanes: lane d of a pair takes the
  //      direction-d terms of the residual and of the low-order point
  //      update, the pair swaps them, and each lane finishes the point and
  //      writes two of its four components (672 half-points spread over all
  //      eight waves, where 336 whole points left two SIMDs with two waves
  //      and two with one).  The FP32-stencil stage, whose tiles hold twice
  //      the points, keeps one lane per point ----
  constexpr int LPP = kFP64<R> ? 2 : 1;  // lanes per point
  constexpr int NW = 4 / LPP;            // components a lane writes
  for (int s2 = tid; s2 < LPP * NPT; s2 += NT) {
    const int s = s2 / LPP, d = LPP == 2 ? (s2 & 1) : 0;
    const int t = s / (TX * TY), r = s % (TX * TY);
    const int ni = t == 1 ? g.n1 : g.n1x;
    const int nj = t == 0 ? g.n2 : g.n2y;
    const long np = (long)ni * nj;
    const long off = t == 0 ? g.off_xe : (t == 1 ? g.off_ye : g.off_co);
    {
      const int i = i0 + r % TX, j = j0 + r / TX;
      // both lanes of a pair take this branch together
      if (i >= ni || j >= nj) continue;
      const int X = t == 1 ? 2 * i + 1 : 2 * i;
      const int Y = t == 0 ? 2 * j + 1 : 2 * j;
      const int a = (Y - Y0 + 4) * WA + (X - X0 + 4);
      const int q = (Y - Y0 + 2) * WG + (X - X0 + 2);
      const long gi = (long)j * ni + i;
      // U^n of the components this lane writes (NW * d onwards), loaded
      // while the residual is computed
      double un[NW];
#pragma unroll
      for (int c = 0; c < NW; ++c) un[c] = first ? 0.0 : Un[off + (NW * d + c) * np + gi];
      // the residual; the two directions' terms are added in the same order
      // in both lanes of a pair
      R Rs[4];
      if constexpr (LPP == 2) {
        R Rd[4];
        point_resid_dir(T, ph, a, q, d, d ? g.dy : g.dx, Rd);
#pragma unroll
        for (int k = 0; k < 4; ++k) Rs[k] = Rd[k] + pair_swap(Rd[k]);
      } else {
        R Rx[4], Ry[4];
        point_resid_dir(T, ph, a, q, 0, g.dx, Rx);
        point_resid_dir(T, ph, a, q, 1, g.dy, Ry);
#pragma unroll
        for (int k = 0; k < 4; ++k) Rs[k] = Rx[k] + Ry[k];
      }
      // the point update and its blend in FP64, from the FP64 point value
      double U0[4], UH[4], out[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if constexpr (kFP64<R>)
          U0[k] = T.U[k][a];
        else
          U0[k] = double(T.U[k][a]) + double(T.PL[k][s]);
        UH[k] = U0[k] + dt * double(Rs[k]);
      }
      if (ph.lim & LIM_POINT) {
        double Ls[4];
        if constexpr (LPP == 2) {
          R Ld[4];
          lo_point_dir(T, X - X0 + 4, Y - Y0 + 4, d, d ? g.dy : g.dx, dt, Ld);
#pragma unroll
          for (int k = 0; k < 4; ++k) Ls[k] = double(Ld[k]) + double(pair_swap(Ld[k]));
        } else {
          R Lx[4], Ly[4];
          lo_point_dir(T, X - X0 + 4, Y - Y0 + 4, 0, g.dx, dt, Lx);
          lo_point_dir(T, X - X0 + 4, Y - Y0 + 4, 1, g.dy, dt, Ly);
#pragma unroll
          for (int k = 0; k < 4; ++k) Ls[k] = double(Lx[k]) + double(Ly[k]);
        }
        double UL[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) UL[k] = U0[k] - Ls[k];
        bool lbad = false;
        double th = theta_pair2(UL, UH, phd.gm1, lbad, ph.lim & LIM_PEXACT);
        if (ph.lim & LIM_LOWONLY) th = 0.0;
        if (lbad && d == 0) raise_flag(flags, FLAG_POINT_LOW);
#pragma unroll
        for (int k = 0; k < 4; ++k) out[k] = (th == 1.0) ? UH[k] : UL[k] + th * (UH[k] - UL[k]);
      } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) out[k] = UH[k];
      }
      if (X == 0) project(wall_of(g.bc0), 0, out);
      if (X == Xlim) project(wall_of(g.bc1), 0, out);
      if (Y == 0) project(wall_of(g.bc2), 1, out);
      if (Y == Ylim) project(wall_of(g.bc3), 1, out);
      // this lane's components (selected by value: an index computed from d
      // would put out in scratch memory)
      double v[NW];
      if constexpr (LPP == 2) {
        v[0] = d ? out[2] : out[0];
        v[1] = d ? out[3] : out[1];
      } else {
#pragma unroll
        for (int c = 0; c < NW; ++c) v[c] = out[c];
      }
#pragma unroll
      for (int c = 0; c < NW; ++c) {
        const double o = first ? v[c] : ca * un[c] + cb * v[c];
        if (!isfinite(o)) nonfinite = true;
        Uout[off + (NW * d + c) * np + gi] = o;
      }
    }
  }
  if (nonfinite) raise_flag(flags, FLAG_NONFINITE);
  nonfinite = false;
  tile = next;
  }  // tiles
}

// persistent workgroups of a stage kernel instance: as many as fit on the
// device at once (the tile's LDS footprint decides), cached per device
template <typename R>
int resident_workgroups() {
  static int cache[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  if (cache[dev] == 0) {
    int cus = 0, per = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        cus <= 0)
      cus = 256;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, k_stage<R, true>, NT, 0) != hipSuccess ||
        per <= 0)
      per = 1;
    cache[dev] = cus * per;
  }
  return cache[dev];
}

// workgroups of a launch over ntiles tiles (see TileIter)
template <typename R>
int workgroups(int ntiles) {
  int nwg = resident_workgroups<R>();
  if (nwg > ntiles) nwg = ntiles;
  if (nwg >= 8) nwg -= nwg % 8;
  return nwg;
}

template <typename R>
hipError_t launch_batch(afi::BatchInst* inst, int ninst, int total_tiles, const int* n_active,
                        int k, hipStream_t s, afi::Timer* tm) {
  if (ninst > kMaxBatch) return hipErrorInvalidValue;
  StageArgs sa{};
  sa.inst = inst;
  sa.ninst = ninst;
  sa.k = k;
  sa.n_active = n_active;
  sa.ca = k == 0 ? 0.0 : (k == 1 ? 0.75 : 1.0 / 3.0);
  sa.cb = k == 0 ? 1.0 : (k == 1 ? 0.25 : 2.0 / 3.0);
  sa.first = k == 0;
  sa.skip_flagged = 1;
  sa.ntiles = total_tiles;
  const int nwg = workgroups<R>(total_tiles);
  AFI_TIMED(tm, 7, s,
            hipLaunchKernelGGL((k_stage<R, true>), dim3((unsigned)nwg), dim3(NT), 0, s, sa));
  return hipGetLastError();
}

}  // namespace

namespace afi {

// tiles of one 2D grid for this instance's tile shape
int AF_STAGE_TILES(const Geo& geo) { return (geo.n1 / TX + 1) * (geo.n2 / TY + 1); }

#ifdef AF_STAGE_ONE
// the stage of one instance (see single_on_tiles)
hipError_t AF_STAGE_ONE(const Geo& geo, const Phys& ph, const Work& w, const double* Un,
                        const double* Uk, double* Uout, const double* dt_dev, double dt_host,
                        StageCoef sc, hipStream_t s, Timer* tm) {
  using R = AF_STAGE_REAL;
  StageArgs sa{};
  sa.g = stage_geo(geo);
  sa.ph = ph;
  sa.Uk = Uk;
  sa.Un = Un;
  sa.Uout = Uout;
  sa.dt_dev = dt_dev;
  sa.dt_host = dt_host;
  sa.dt_mul = sc.dt_mul;
  sa.flags = w.flags;
  sa.ntx = geo.n1 / TX + 1;
  sa.ca = sc.a;
  sa.cb = sc.b;
  sa.first = sc.first;
  sa.skip_flagged = sc.skip_flagged;
  sa.blend = sc.blend;
  sa.ts_out = sc.ts_out;
  sa.ntiles = AF_STAGE_TILES(geo);
  const dim3 grid((unsigned)workgroups<R>(sa.ntiles));
  if (sa.blend || sa.ts_out)
    AFI_TIMED(tm, 7, s, hipLaunchKernelGGL((k_stage<R, false, true>), grid, dim3(NT), 0, s, sa));
  else
    AFI_TIMED(tm, 7, s, hipLaunchKernelGGL((k_stage<R, false>), grid, dim3(NT), 0, s, sa));
  return hipGetLastError();
}
#endif

// stage k of a step attempt of every active instance of a batch, one launch
hipError_t AF_STAGE_BATCH(BatchInst* inst, int ninst, int total_tiles, const int* n_active, int k,
                          hipStream_t s, Timer* tm) {
  return launch_batch<AF_STAGE_REAL>(inst, ninst, total_tiles, n_active, k, s, tm);
}

}  // namespace afi
