// k_lb.h -- the fused lattice-Boltzmann step (Sec. 3.1) for D2Q9.
//
// One kernel does, per node and time step: streaming of f, g, h, the moments
// of eq. MomentsDFs, the Laplacians and gradients of the concentrations, the
// chemical potentials and pressure tensor of Appendix A (with the coupling
// term of Sec. 3.1), the force of eqs. ForcingTermLBE / ForceFE plus the spread
// membrane force, the velocities of eqs. ActualFluidVel / VelCorrection and
// the BGK + exact-difference collision of eq. LBE.
//
// Dependency chain: the collision at row c needs the divergence of the
// pressure tensor there, i.e. the tensor on rows c-1..c+1, i.e. moments on
// rows c-2..c+2.  A wave owns a strip of 64 columns and marches up a segment
// of rows; per iteration it takes one row in and does
//   M  the moments of a row
//   U  potentials and tensor of the row below it
//   C  force and collision of the row below that.
// A lane keeps its own column of every stencil in registers (each 3 x 3
// stencil is a sum over the three rows of a row's own combination of its
// west, centre and east values) and takes its west and east neighbours' values
// by lane shifts, so a row needs no LDS and no barrier, and waves run
// independently of each other.  Columns at the strip's ends and rows beyond
// the segment's ends are formed by two waves.
//
// Two forms of the state.  Between calls the state is the populations after
// collision.  With tau = tau_phi = tau_psi = 1 (Sec. 3.1's choice, and the
// default) a collision replaces every population by its equilibrium, so
// the populations of a node are a function of nine of its numbers: density,
// u + delta u, v, Gamma mu and the order parameters (Macro2).  The steps
// inside a call of several then read and write those, 44 bytes per node
// instead of 116 in FP32, and every node's populations are evaluated (and
// rounded to the storage format) where they stream from: the call's first
// step reads populations, its last one writes them, and any division of the
// same steps into calls gives the same bits.
//
// Precision: populations and their equilibria use the storage's real type R
// (FP32 or FP64).  Moments, chemical potentials, their stencils and the force
// are FP64: the chemical potential is a sum of terms much larger than itself
// near interfaces, and its Laplacian/gradient chain would turn
// single-precision rounding of phi and psi into force noise.  Products and
// sums are written as the fused operations they are, with the compiler's own
// contraction off, so every kernel rounds alike.
#pragma once
#include <type_traits>

#include "common.h"
#include "store.h"

namespace lb {

struct LBParams {
  double inv_tau, inv_tau_phi, inv_tau_psi;  // 1/tau (eq. RelaxationTimes)
  double gphi, gpsi;                         // Gamma_phi, Gamma_psi (eq. EDF)
  double k1, k2, k3, a2, kc;                 // kappa_m, alpha^2, kappa_c
  double fext[3];                            // uniform external force density (eq. ForcingTermLBE)
  // component densities M_m (eq. MassDensity; all 1 in the paper): the
  // concentrations are C_m = sum_q cm[m][q] q with q = (rho, phi, psi), and
  // the lattice pressure is c_s^2 (rho + sp) with sp = -(psh[0] phi + psh[1] psi)
  double cm[3][3];
  double psh[2];
  double mb;                                 // (M_1 + M_2) / 2
  // reference density of the stored populations: a kernel holds f_i - w_i rho0
  // (rho0 = M_b, 1 for equal densities), so that the moving populations stay
  // small where the lattice pressure is c_s^2 M_b n with n ~ 1
  double rho0;
  int dens;                                  // 1 if some M_m differs from 1
  int nx, ny, nz, wall_y, wall_z;
  long long N;
  int ntx, nty, tile;                        // tile grid of the membrane maps (edge a power of two)
  int seg;                                   // rows (2D) or planes (3D) per workgroup
  int nstrip, nseg;                          // workgroup grid: strips x segments
  int nxcd;                                  // XCDs the dispatcher deals workgroups to
  int mode;                                  // 2D pass: 0 all, 1 regions without active tiles,
                                             // 2 regions with active tiles (in pieces)
  int seg2, npiece;                          // pass 2: rows per piece, pieces per segment
};

// Workgroup -> (strip, segment).  The dispatcher deals consecutive
// workgroups to the XCDs in turn, and each XCD has its own L2.  Give every
// XCD a contiguous run of the logical order (strips fastest), so the strips
// that share halo columns run side by side on one XCD and meet in its L2.
__device__ __forceinline__ int dealt_index(int b, int total, int nxcd) {
  const int c = b % nxcd, j = b / nxcd;
  // blocks dealt to XCDs before c: sum over c' < c of ceil((total - c') / nxcd)
  const int q = total / nxcd, rem = total % nxcd;
  return c * q + min(c, rem) + j;
}

__device__ __forceinline__ void strip_segment(int b, int nstrip, int nseg, int nxcd, int& s, int& g) {
  const int L = dealt_index(b, nstrip * nseg, nxcd);
  s = L % nstrip;
  g = L / nstrip;
}

// mu_rho (without the ideal-gas part), mu_phi, mu_psi' from local values and
// Laplacians, written through the concentrations C_m, a linear map of
// (rho, phi, psi) (eq. VariableTransform; with component densities, eq.
// MassDensity solved for C_1 + C_2).  The derivative of the Landau energy
// (eq. LandauFE) with respect to C_m is
// b_m = kappa_m C_m (1-C_m)(1-2C_m) - alpha^2 kappa_m lap C_m, and the chain
// rule gives mu_q = sum_m (dC_m/dq) b_m; for equal densities
// mu_rho = (b1+b2)/2, mu_phi = (b1-b2)/2, mu_psi = b3 - (b1+b2)/2.  The
// coupling energy (eq. CouplingE) adds kappa_c (psi - I) to mu_psi.  The
// map's coefficients for equal densities are 0, +-1/2 and 1, so the sums
// round as the closed forms do.
__device__ __forceinline__ void conc3(const LBParams& P, double a, double b, double c, double* C) {
#pragma unroll
  for (int m = 0; m < 3; m++) C[m] = P.cm[m][0] * a + P.cm[m][1] * b + P.cm[m][2] * c;
}

__device__ __forceinline__ void chem_pot(const LBParams& P, double drho, double phi, double psi,
                                         double lr, double lp, double ls, double I, double& mr,
                                         double& mp, double& ms) {
  const double rho = P.rho0 + drho;
  double C[3], Lc[3];
  conc3(P, rho, phi, psi, C);
  conc3(P, lr, lp, ls, Lc);
  const double km[3] = {P.k1, P.k2, P.k3};
  double b[3];
#pragma unroll
  for (int m = 0; m < 3; m++) b[m] = km[m] * (C[m] * (1.0 - C[m]) * (1.0 - 2.0 * C[m]) - P.a2 * Lc[m]);
  mr = (P.cm[0][0] * b[0] + P.cm[1][0] * b[1]) + P.cm[2][0] * b[2];
  mp = (P.cm[0][1] * b[0] + P.cm[1][1] * b[1]) + P.cm[2][1] * b[2];
  ms = (P.cm[0][2] * b[0] + P.cm[1][2] * b[1]) + P.cm[2][2] * b[2] + P.kc * (psi - I);
}

// BGK + exact-difference collision of one node, D2Q9, in place.  pf holds
// f_i - w_i rho0 (all i), pg/ph the moving g_i/h_i (i >= 1), g0/h0 the rest
// populations.  Moments and the total force (Fx, Fy) are FP64.
template <typename R>
__device__ __forceinline__ void collide9(const LBParams& P, R* pf, R* pg, R* ph, double& g0,
                                         double& h0, double drho, double jx, double jy, double phi,
                                         double psi, double mphi, double mpsi, double Fx, double Fy) {
  using L = Lattice<9>;
  const double rho = P.rho0 + drho;
  const double irho = 1.0 / rho;
  const double uxd = jx * irho, uyd = jy * irho;
  const double duxd = Fx * irho, duyd = Fy * irho;  // eq. VelCorrection
  const R ux = (R)uxd, uy = (R)uyd;
  const R vx = (R)(uxd + 0.5 * duxd), vy = (R)(uyd + 0.5 * duyd);  // eq. ActualFluidVel
  const R wx = (R)(uxd + duxd), wy = (R)(uyd + duyd);
  const R uu = ux * ux + uy * uy, ww = wx * wx + wy * wy, vv = vx * vx + vy * vy;
  const R rr = (R)rho, dr = (R)drho, ph_ = (R)phi, ps_ = (R)psi;
  const R gm = (R)(3.0 * P.gphi * mphi), hm = (R)(3.0 * P.gpsi * mpsi);
  const R itf = (R)P.inv_tau, itg = (R)P.inv_tau_phi, ith = (R)P.inv_tau_psi;
  // with component densities the equilibrium carries the lattice pressure
  // c_s^2 (rho + sp): w_i sp joins every moving population, -(1 - w_0) sp
  // the rest one (zero for equal densities)
  const double spd = -(P.psh[0] * phi + P.psh[1] * psi);
  const R sp = (R)spd, drs = dr + sp;
  double gsum = 0.0, hsum = 0.0;
#pragma unroll
  for (int i = 0; i < 9; i++) {
    const R w = R(L::w(i));
    const R cu = R(L::cx[i]) * ux + R(L::cy[i]) * uy;
    const R cw = R(L::cx[i]) * wx + R(L::cy[i]) * wy;
    const R pu = R(3) * cu + R(4.5) * cu * cu - R(1.5) * uu;
    const R pw = R(3) * cw + R(4.5) * cw * cw - R(1.5) * ww;
    // f^eq(rho, u) - w_i rho0 (drho = rho - rho0)
    const R feq = i == 0 ? w * (dr + rr * pu) - R(1.0 - L::w(0)) * sp : w * (drs + rr * pu);
    const R edm = w * rr * (pw - pu);  // f^eq(rho, u + du) - f^eq(rho, u)
    pf[i] = pf[i] - (pf[i] - feq) * itf + edm;
    if (i > 0) {
      const R cv = R(L::cx[i]) * vx + R(L::cy[i]) * vy;
      const R pv = R(3) * cv + R(4.5) * cv * cv - R(1.5) * vv;
      const R geq = w * (gm + ph_ * pv);
      const R heq = w * (hm + ps_ * pv);
      gsum += (double)geq;
      hsum += (double)heq;
      pg[i] = pg[i] - (pg[i] - geq) * itg;
      ph[i] = ph[i] - (ph[i] - heq) * ith;
    }
  }
  // rest populations close the zeroth moments (eq. EDF, i = 0)
  g0 = g0 - (g0 - (phi - gsum)) * P.inv_tau_phi;
  h0 = h0 - (h0 - (psi - hsum)) * P.inv_tau_psi;
}

// pull the populations of node (x, y), 0 <= x < nx, 0 <= y < ny, at the
// current time: population i arrives from x - c_i; across a wall it is the
// reversed population that left (x, y) (half-way bounce-back).
template <class St, typename R>
__device__ __forceinline__ void pull9(const St& src, const LBParams& P, int x, int y, R* pf, R* pg,
                                      R* ph, double& g0, double& h0) {
  using L = Lattice<9>;
  const long long here = (long long)y * P.nx + x;
  // the neighbour rows and columns, wrapped once per node
  const long long rlo = (long long)(y == 0 ? P.ny - 1 : y - 1) * P.nx;
  const long long rhi = (long long)(y == P.ny - 1 ? 0 : y + 1) * P.nx;
  const int xlo = x == 0 ? P.nx - 1 : x - 1;
  const int xhi = x == P.nx - 1 ? 0 : x + 1;
  const bool wlo = P.wall_y && y == 0;         // row y - 1 lies beyond a wall
  const bool whi = P.wall_y && y == P.ny - 1;  // row y + 1 lies beyond a wall
  pf[0] = src.template load<R>(0, 0, here);
  g0 = src.rest(1, here);
  h0 = src.rest(2, here);
#pragma unroll
  for (int i = 1; i < 9; i++) {
    const bool back = L::cy[i] > 0 ? wlo : (L::cy[i] < 0 ? whi : false);
    const long long row = L::cy[i] > 0 ? rlo : (L::cy[i] < 0 ? rhi : here - x);
    const int col = L::cx[i] > 0 ? xlo : (L::cx[i] < 0 ? xhi : x);
    const long long node = back ? here : row + col;
    const int dir = back ? L::opp[i] : i;
    pf[i] = src.template load<R>(0, dir, node);
    pg[i] = src.template load<R>(1, dir, node);
    ph[i] = src.template load<R>(2, dir, node);
  }
}

// moments of eq. MomentsDFs: the sums over the small values (f_i - w_i rho0 and
// the moving g_i, h_i) run in R, the rest populations g_0, h_0 join in FP64
template <typename R>
__device__ __forceinline__ void moments9(const R* pf, const R* pg, const R* ph, double g0, double h0,
                                         double& d, double& jx, double& jy, double& phi,
                                         double& psi) {
  using L = Lattice<9>;
  R sd = 0, sx = 0, sy = 0, sg = 0, sh = 0;
#pragma unroll
  for (int i = 0; i < 9; i++) {
    sd += pf[i];
    if (L::cx[i] != 0) sx += R(L::cx[i]) * pf[i];
    if (L::cy[i] != 0) sy += R(L::cy[i]) * pf[i];
    if (i > 0) {
      sg += pg[i];
      sh += ph[i];
    }
  }
  d = (double)sd;
  jx = (double)sx;
  jy = (double)sy;
  phi = g0 + (double)sg;
  psi = h0 + (double)sh;
}

// the same in the order in which the rows' shares of a march add up, which a
// mirror in y leaves alone bit for bit (ghost rows beyond a wall are the
// lattice mirrored)
template <typename R>
__device__ __forceinline__ void moments9m(const R* f, const R* g, const R* h, double g0, double h0, R& d, R& jx,
                                          R& jy, double& phi, double& psi) {
  const R n = f[3] + (f[5] + f[7]), s = f[4] + (f[6] + f[8]);
  d = (f[0] + (f[1] + f[2])) + (n + s);
  jx = (f[1] - f[2]) + ((f[5] - f[7]) + (f[8] - f[6]));
  jy = n - s;
  phi = g0 + (double)((g[1] + g[2]) + ((g[3] + (g[5] + g[7])) + (g[4] + (g[6] + g[8]))));
  psi = h0 + (double)((h[1] + h[2]) + ((h[3] + (h[5] + h[7])) + (h[4] + (h[6] + h[8]))));
}

// ---------------------------------------------------------------------------
// equilibria

__device__ __forceinline__ float fma_(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fma_(double a, double b, double c) { return __builtin_fma(a, b, c); }

// 1/x to the last bit or so: the hardware's estimate and two Newton steps
__device__ __forceinline__ double recip(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = fma_(fma_(-x, r, 1.0), r, r);
  return fma_(fma_(-x, r, 1.0), r, r);
}

// value of the lane to the west (lane - 1) or east (lane + 1) within the
// wave; the lanes at the ends get 0
template <int CTRL>
__device__ __forceinline__ int lane_mov(int v) {
  return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, true);
}
template <int CTRL>
__device__ __forceinline__ float lane_mov(float v) {
  return __builtin_bit_cast(float, lane_mov<CTRL>(__builtin_bit_cast(int, v)));
}
template <int CTRL>
__device__ __forceinline__ double lane_mov(double v) {
  const long long b = __builtin_bit_cast(long long, v);
  const unsigned lo = (unsigned)lane_mov<CTRL>((int)b), hi = (unsigned)lane_mov<CTRL>((int)(b >> 32));
  return __builtin_bit_cast(double, (long long)(((unsigned long long)hi << 32) | lo));
}
template <typename T>
__device__ __forceinline__ T west(T v) { return lane_mov<0x138>(v); }  // wave_shr:1
template <typename T>
__device__ __forceinline__ T east(T v) { return lane_mov<0x130>(v); }  // wave_shl:1

// What the populations of a node after a collision with tau = 1 depend on:
// dr = rho - rho0, w = u + delta u, v = u + delta u / 2, gm = 3 Gamma_phi
// mu_phi, hm = 3 Gamma_psi mu_psi, and the order parameters.  (For f the
// equilibrium at u and the exact-difference term add to the equilibrium at
// u + delta u.)
template <typename R>
struct Macro2 {
  R dr, wx, wy, vx, vy, gm, hm;
  double phi, psi;
};

// the pressure shift of component densities (zero for equal ones), eq.
// MassDensity: w_i sp joins every moving population of f, -(1 - w_0) sp the rest one
template <typename R>
__device__ __forceinline__ R eq_shift(double p0, double p1, double phi, double psi) {
#pragma clang fp contract(off)
  return (R)(-fma_(p0, phi, p1 * psi));
}

// The two populations along +-c of a set whose rest population closes the sum
// in FP64 (g, h): a (1 + 3 c.u + ..) + b with c.u = cu, q = -3/2 u^2, a3 = 3 a.
template <typename R>
__device__ __forceinline__ void eq_pair(R a, R a3, R b, R q, R cu, R& fp, R& fm) {
#pragma clang fp contract(off)
  const R base = fma_(a, fma_(R(4.5) * cu, cu, q), b);
  fp = fma_(a3, cu, base);
  fm = fma_(-a3, cu, base);
}

// The same for f, whose rounding is the node's mass and moves the fluid: the
// weight multiplies last, so no rounding is shared by the populations.
template <typename R>
__device__ __forceinline__ void eq_pair_f(R w, R rr, R drs, R q, R cu, R& fp, R& fm) {
#pragma clang fp contract(off)
  const R t = fma_(R(4.5) * cu, cu, q);
  fp = w * fma_(rr, fma_(R(3), cu, t), drs);
  fm = w * fma_(rr, fma_(R(-3), cu, t), drs);
}

// f_i^eq(rho, c) - w_i rho0 for all i
template <typename R>
__device__ __forceinline__ void eq9_f(R rho0, R dr, R sp, R cx, R cy, R* f) {
#pragma clang fp contract(off)
  using L = Lattice<9>;
  const R rr = rho0 + dr, drs = dr + sp;
  const R q = R(-1.5) * fma_(cx, cx, cy * cy);
  f[0] = fma_(R(L::w(0)), fma_(rr, q, dr), -(R(1.0 - L::w(0)) * sp));
  const R w1 = R(L::w(1)), w5 = R(L::w(5));
  eq_pair_f(w1, rr, drs, q, cx, f[1], f[2]);
  eq_pair_f(w1, rr, drs, q, cy, f[3], f[4]);
  eq_pair_f(w5, rr, drs, q, cx + cy, f[5], f[6]);
  eq_pair_f(w5, rr, drs, q, cx - cy, f[8], f[7]);
}

// the moving g_i^eq (order parameter ph, gm = 3 Gamma mu), i = 1..8, at v
template <typename R>
__device__ __forceinline__ void eq9_g(R ph, R gm, R cx, R cy, R* g) {
#pragma clang fp contract(off)
  using L = Lattice<9>;
  const R q = R(-1.5) * fma_(cx, cx, cy * cy);
  const R a1 = ph * R(L::w(1)), a13 = R(3) * a1, b1 = gm * R(L::w(1));
  const R a5 = ph * R(L::w(5)), a53 = R(3) * a5, b5 = gm * R(L::w(5));
  eq_pair(a1, a13, b1, q, cx, g[1], g[2]);
  eq_pair(a1, a13, b1, q, cy, g[3], g[4]);
  eq_pair(a5, a53, b5, q, cx + cy, g[5], g[6]);
  eq_pair(a5, a53, b5, q, cx - cy, g[8], g[7]);
}

// one population of f or (F false) of g or h in the direction of population i
// or (flip) its opposite: the same operations on the same values (a product
// by +-1 or 0 is exact)
template <bool F, typename R>
__device__ __forceinline__ R eq9_one(R a, R b, int i, bool flip, R cx, R cy) {
#pragma clang fp contract(off)
  using L = Lattice<9>;
  const R q = R(-1.5) * fma_(cx, cx, cy * cy), w = R(L::w(i));
  const R cu = L::cx[i] * cx + L::cy[i] * cy;
  const R t = fma_(R(4.5) * cu, cu, q);
  if (F) return w * fma_(a, fma_(flip ? R(-3) : R(3), cu, t), b);
  const R aw = a * w;
  return fma_(flip ? -(R(3) * aw) : R(3) * aw, cu, fma_(aw, t, b * w));
}

// rest populations close the zeroth moments (eq. EDF, i = 0); the eight
// moving ones are summed in FP64 in an order that a mirror in y leaves alone
template <typename R>
__device__ __forceinline__ double eq9_rest(double phi, const R* g) {
#pragma clang fp contract(off)
  return phi - ((((double)g[1] + (double)g[2]) + ((double)g[3] + (double)g[4])) +
                (((double)g[5] + (double)g[8]) + ((double)g[6] + (double)g[7])));
}

// a node's populations
template <typename R>
__device__ __forceinline__ void macro_pops(R rho0, double p0, double p1, const Macro2<R>& s, R* pf, R* pg, R* ph,
                                           double& g0, double& h0) {
  eq9_f(rho0, s.dr, eq_shift<R>(p0, p1, s.phi, s.psi), s.wx, s.wy, pf);
  eq9_g((R)s.phi, s.gm, s.vx, s.vy, pg);
  eq9_g((R)s.psi, s.hm, s.vx, s.vy, ph);
  g0 = eq9_rest(s.phi, pg);
  h0 = eq9_rest(s.psi, ph);
}

// The state between the steps of one call (tau = 1): planes dr, wx, wy, vx,
// vy, gm, hm in R and phi, psi in FP64.  Planes of one type stay below 4 GiB
// (checked on the host), so a node is a 32-bit byte offset; a store to node
// -1 is out of the buffer's range and dropped, so a store needs no branch.
template <typename R>
struct MacroStore2 {
  R* p;
  double* r;
  unsigned N;
  double rho0, p0, p1;
  static constexpr bool kMacro = true;
  static constexpr int kR = 7;
  __device__ __forceinline__ __amdgpu_buffer_rsrc_t rp() const {
    return __builtin_amdgcn_make_buffer_rsrc(p, 0, (int)(kR * N * (unsigned)sizeof(R)), 0x00020000);
  }
  __device__ __forceinline__ __amdgpu_buffer_rsrc_t rr() const {
    return __builtin_amdgcn_make_buffer_rsrc(r, 0, (int)(2 * N * 8u), 0x00020000);
  }
  __device__ __forceinline__ R get(int k, unsigned node) const {
    if constexpr (sizeof(R) == 4)
      return __builtin_bit_cast(R, __builtin_amdgcn_raw_buffer_load_b32(rp(), (int)(node * 4), (int)(k * N * 4), 0));
    else
      return __builtin_bit_cast(R, __builtin_amdgcn_raw_buffer_load_b64(rp(), (int)(node * 8), (int)(k * N * 8), 0));
  }
  __device__ __forceinline__ double getd(int k, unsigned node) const {
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rr(), (int)(node * 8), (int)(k * N * 8), 0));
  }
  __device__ __forceinline__ void put(int k, unsigned node, R v) const {
    if constexpr (sizeof(R) == 4)
      __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), rp(), (int)(node * 4), (int)(k * N * 4), 0);
    else
      __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), rp(), (int)(node * 8), (int)(k * N * 8), 0);
  }
  __device__ __forceinline__ void putd(int k, unsigned node, double v) const {
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), rr(), (int)(node * 8), (int)(k * N * 8), 0);
  }
  __device__ __forceinline__ Macro2<R> node(unsigned n) const {
    return Macro2<R>{get(0, n), get(1, n), get(2, n), get(3, n), get(4, n), get(5, n), get(6, n), getd(0, n), getd(1, n)};
  }
  __device__ __forceinline__ void set_node(unsigned n, const Macro2<R>& s) const {
    put(0, n, s.dr);
    put(1, n, s.wx);
    put(2, n, s.wy);
    put(3, n, s.vx);
    put(4, n, s.vy);
    put(5, n, s.gm);
    put(6, n, s.hm);
    putd(0, n, s.phi);
    putd(1, n, s.psi);
  }
  // single populations, for the kernels that read a few nodes near a membrane
  template <typename T>
  __device__ __forceinline__ T pull(int set, int i, bool flip, long long nd) const {
#pragma clang fp contract(off)
    const unsigned n = (unsigned)nd;
    if (i == 0) return (T)rest(set, nd);
    R v;
    if (set == 0) {
      const R dr = get(0, n);
      v = eq9_one<true, R>((R)rho0 + dr, dr + eq_shift<R>(p0, p1, getd(0, n), getd(1, n)), i, flip, get(1, n), get(2, n));
    } else {
      v = eq9_one<false, R>((R)getd(set - 1, n), get(4 + set, n), i, flip, get(3, n), get(4, n));
    }
    return (T)v;
  }
  __device__ __forceinline__ double rest(int set, long long nd) const {
    R pf[9], pg[9], ph[9];
    double g0, h0;
    macro_pops<R>((R)rho0, p0, p1, node((unsigned)nd), pf, pg, ph, g0, h0);
    return set == 0 ? (double)pf[0] : (set == 1 ? g0 : h0);
  }
};

// columns at each end of a wave's strip that the neighbouring strips form too:
// the pressure tensor needs moments one column out, the force the tensor one
// column out, and moments from Macro2 the populations one column out
template <class Src>
constexpr int strip_halo() {
  return Src::kMacro ? 3 : 2;
}
// waves per SIMD the register budget is sized for
template <typename R>
constexpr int step2d_waves() {
  return sizeof(R) == 8 ? 1 : 2;
}
// Waves of a workgroup that paces them (neighbouring strips, a barrier per row):
// as many as a CU holds.  From populations to populations on a lattice whose
// buffers exceed the last-level cache, waves on their own drift apart, and the
// lines that the strips of 60 columns share are fetched and written back for
// each of them.  Per step, on their own / paced, FP32 at tau = 1: 1000^2 49 / 50 us,
// 1400^2 124 / 112, 2048^2 272 / 229, 3000^2 579 / 472, 4500^2 1356 / 1083
// (four waves 110, 233, 482, 1155); FP64 700^2 43 / 43, 1000^2 113 / 102, 2048^2
// 460 / 389 (its eight waves would not fit a CU at these registers).  Inside the
// cache a barrier only costs: FP32 300^2 13.4 / 20 us; so it does on a single
// strip: 16 x 100000 185 / 213 us, but 120 x 20000 158 / 154.
template <typename R>
constexpr int step2d_paced() {
  return 4 * step2d_waves<R>();
}
constexpr size_t PACED_FROM = (size_t)256 << 20;  // bytes of both buffers

// One (strip, rows [y0, y1)) of the lattice: the whole march of a wave.
// FORM 0: the force of eq. ForceFE in its potential form, -sum q grad mu_q
// over q = rho, phi, psi (eq. GradPT).  FORM 1: its divergence form,
// -div P' - psi grad kappa_c (psi - I), with the non-ideal pressure tensor P'
// of Appendix A (the two forms agree up to the discretisation error).
// Src, Dst: St (populations) or MacroStore2.  RELAX: a collision needs the
// populations that came in (some tau differs from 1, or the storage rounds
// them to 16 bits); Src and Dst are St.  PACED: the waves of the workgroup keep
// to the same row.
template <class St, typename R, int FORM, class Src, class Dst, bool RELAX, bool PACED>
__device__ __forceinline__ void step2d_run(const Src& src, const Dst& dst, const LBParams& P,
                                           int strip, int y0, int y1, const int* __restrict__ tflag,
                                           const int* __restrict__ tstate, const double* __restrict__ Ifield,
                                           long long* __restrict__ fib, double* __restrict__ force) {
#pragma clang fp contract(off)
  constexpr bool SM = Src::kMacro, DM = Dst::kMacro;
  static_assert(!RELAX || (!SM && !DM), "relaxation needs the populations");
  constexpr int H = strip_halo<Src>();
  constexpr int LAG = SM ? 1 : 0;  // rows between the row taken in and the row of the moments
  const int j = threadIdx.x & 63;
  const int xc = strip * (64 - 2 * H) - H + j;
  const int x = wrap(xc, P.nx);
  const bool interior = j >= H && j < 64 - H && xc < P.nx;
  const int K = (y1 - y0) + 2 * H, rbase = y0 - H;
  const int stamp = tstate[1];  // tiles flagged with this step's stamp are active
  const int tsh = __builtin_ctz((unsigned)P.tile);  // log2 of the tile edge
  const int xt = x >> tsh;
  const R rho0 = (R)P.rho0;
  const double km[3] = {P.k1, P.k2, P.k3};

  // the row taken in: loaded one iteration ahead of its use (RELAX: at its use)
  Macro2<R> nxt = {};
  R npf[9], npg[9], nph[9];
  double ng0 = 0.0, nh0 = 0.0;
  int nfl = 0;
  // RELAX: populations of the last three rows
  R kf[RELAX ? 3 : 1][9], kg[RELAX ? 3 : 1][9], kh[RELAX ? 3 : 1][9];
  double kg0[RELAX ? 3 : 1], kh0[RELAX ? 3 : 1];
  // SM: shares of the moments: what the last row taken in sends north (and what
  // it would send back from a wall above it), what the row of the moments has
  // received from below and from its own row
  R sent[4] = {}, back[4] = {}, got[4] = {}, own[4] = {};
  double own_g0 = 0.0, own_h0 = 0.0;
  // moments of the last three rows: concentrations and their west-east sums
  // (hs = (west - c) + (east - c)) and differences (hd = east - west)
  double cq[3][3] = {}, hs[3][3] = {}, hd[3][3] = {}, mphi[3] = {};
  R md[3] = {}, mjx[3] = {}, mjy[3] = {};
  // stencils of the force, summed row by row (see the C stage)
  double ax[3] = {}, px[3] = {}, ay[3][2] = {};
  double fx0 = 0.0, fx1 = 0.0, fy0 = 0.0, fy1 = 0.0;
  double mpC = 0.0, msC = 0.0;  // potentials of the C row
  // active lanes of the rows taken in last, and the membrane fields fetched
  // for the next iteration: profile field of its U row, spread force of its C row
  unsigned long long act1 = 0, act2 = 0, act3 = 0;
  double Inx = 0.0;
  long long fb0n = 0, fb1n = 0;

  auto load_row = [&](int k) {
    const int ry = fd_row_near(rbase + k, P.ny, P.wall_y);
    nfl = tflag[(ry >> tsh) * P.ntx + xt];
    if constexpr (SM)
      nxt = src.node((unsigned)(ry * P.nx + x));
    else
      pull9(src, P, x, ry, npf, npg, nph, ng0, nh0);
  };

  // PH: iteration of the prologue (2 H of them, nothing to store yet), or 2 H
  // and more: steady, PH % 3 the ring slot
  auto body = [&](auto ph_c, int k) {
#pragma clang fp contract(off)
    constexpr int PH = decltype(ph_c)::value;
    constexpr int S = PH % 3, SB = (PH + 2) % 3, SA = (PH + 1) % 3;  // slots of rows m, m - 1 (U), m - 2 (C)
    constexpr bool doM = PH >= 2 * LAG, doU = PH >= 2 + 2 * LAG, doC = PH >= 4 + 2 * LAG;
    const int r = rbase + k;
    if constexpr (PACED) __builtin_amdgcn_s_barrier();
    if constexpr (RELAX) load_row(k);
    // ---- the row taken in
    R pf[9], pg[9], ph[9];
    double g0, h0;
    const unsigned long long act0 = __ballot(nfl == stamp);
    Macro2<R> s = nxt;
    if constexpr (!SM) {
#pragma unroll
      for (int i = 0; i < 9; i++) {
        pf[i] = npf[i];
        pg[i] = i ? npg[i] : R(0);
        ph[i] = i ? nph[i] : R(0);
      }
      g0 = ng0;
      h0 = nh0;
      if constexpr (RELAX) {
#pragma unroll
        for (int i = 0; i < 9; i++) {
          kf[S][i] = pf[i];
          kg[S][i] = pg[i];
          kh[S][i] = ph[i];
        }
        kg0[S] = g0;
        kh0[S] = h0;
      }
    }
    // ---- membrane fields of the next iteration's U and C rows
    const double Icur = Inx;
    const long long fb0 = fb0n, fb1 = fb1n;
    const unsigned long long actC = SM ? act3 : act2;  // the C row's, r - H
    {
      // next iteration: U row r - LAG (flags act1 when SM, act0 else), C row the one below it
      const unsigned long long au = SM ? act1 : act0, ac = SM ? act2 : act1;
      Inx = 0.0;
      fb0n = fb1n = 0;
      if (au | ac) {
        const int ur = r - LAG;
        if (PH + 1 >= 2 + 2 * LAG && (au >> j & 1))
          Inx = Ifield[(long long)fd_row_near(ur, P.ny, P.wall_y) * P.nx + x];
        if (PH + 1 >= 4 + 2 * LAG && (ac >> j & 1) && interior && k + 1 < K) {
          const long long* fp = fib + 2 * ((long long)(ur - 1) * P.nx + x);
          fb0n = fp[0];
          fb1n = fp[1];
        }
      }
    }
    if constexpr (!RELAX) load_row(min(k + 1, K - 1));

    // ---- M: moments of row m
    R d = 0, jx = 0, jy = 0;
    double phi = 0.0, psi = 0.0;
    if constexpr (SM) {
      if (P.wall_y && (r < 0 || r >= P.ny)) {  // a wall's ghost rows are mirrored
        s.wy = -s.wy;
        s.vy = -s.vy;
      }
      macro_pops<R>(rho0, P.psh[0], P.psh[1], s, pf, pg, ph, g0, h0);
      // Row m = r - 1 receives its own row's populations 0, 1, 2, what the row
      // below sent north (3, 5, 7) and what this row sends south (4, 6, 8):
      // its moments are the sums of three rows' shares, each four numbers
      // (f, the x momentum of f, g, h) formed as the row is taken in
      const bool crossing = P.wall_y && (r == 0 || r == P.ny);  // a wall between rows r - 1 and r
      R so[4], no[4];
      if (crossing) {  // half-way bounce-back on both sides of it
#pragma unroll
        for (int e = 0; e < 4; e++) so[e] = back[e];
        no[0] = pf[4] + (pf[6] + pf[8]);
        no[1] = pf[6] - pf[8];
        no[2] = pg[4] + (pg[6] + pg[8]);
        no[3] = ph[4] + (ph[6] + ph[8]);
      } else {
        const R f6 = east(pf[6]), f8 = west(pf[8]);
        so[0] = pf[4] + (f6 + f8);
        so[1] = f8 - f6;
        so[2] = pg[4] + (east(pg[6]) + west(pg[8]));
        so[3] = ph[4] + (east(ph[6]) + west(ph[8]));
#pragma unroll
        for (int e = 0; e < 4; e++) no[e] = sent[e];
      }
      if constexpr (doM) {
        d = own[0] + (got[0] + so[0]);
        jx = own[1] + (got[1] + so[1]);
        jy = got[0] - so[0];
        phi = own_g0 + (double)(own[2] + (got[2] + so[2]));
        psi = own_h0 + (double)(own[3] + (got[3] + so[3]));
      }
      const R f5 = west(pf[5]), f7 = east(pf[7]), f1 = west(pf[1]), f2 = east(pf[2]);
      own[0] = pf[0] + (f1 + f2);
      own[1] = f1 - f2;
      own[2] = west(pg[1]) + east(pg[2]);
      own[3] = west(ph[1]) + east(ph[2]);
      sent[0] = pf[3] + (f5 + f7);
      sent[1] = f5 - f7;
      sent[2] = pg[3] + (west(pg[5]) + east(pg[7]));
      sent[3] = ph[3] + (west(ph[5]) + east(ph[7]));
      back[0] = pf[3] + (pf[5] + pf[7]);
      back[1] = pf[7] - pf[5];
      back[2] = pg[3] + (pg[5] + pg[7]);
      back[3] = ph[3] + (ph[5] + ph[7]);
#pragma unroll
      for (int e = 0; e < 4; e++) got[e] = no[e];
      own_g0 = g0;
      own_h0 = h0;
    } else if constexpr (RELAX) {
      double dd, jxd, jyd;
      moments9(pf, pg, ph, g0, h0, dd, jxd, jyd, phi, psi);  // sums in R
      d = (R)dd;
      jx = (R)jxd;
      jy = (R)jyd;
    } else {
      moments9m(pf, pg, ph, g0, h0, d, jx, jy, phi, psi);
    }
    if constexpr (doM) {
      const double rho = P.rho0 + (double)d;
      const double C[3] = {fma_(P.cm[0][0], rho, fma_(P.cm[0][1], phi, P.cm[0][2] * psi)),
                           fma_(P.cm[1][0], rho, fma_(P.cm[1][1], phi, P.cm[1][2] * psi)), psi};
#pragma unroll
      for (int f = 0; f < 3; f++) {
        const double e = east(C[f]), w = west(C[f]);
        cq[S][f] = C[f];
        hs[S][f] = (w - C[f]) + (e - C[f]);
        hd[S][f] = e - w;
      }
      mphi[S] = phi;
      md[S] = d;
      mjx[S] = jx;
      mjy[S] = jy;
    }
    if constexpr (doU) {
      // ---- U: row m - 1, from the rows below (a), its own (b), above (c)
      double lap[3], b[3], t1[3];
#pragma unroll
      for (int f = 0; f < 3; f++) {
        const double q = cq[SB][f];
        // lap q = 6 sum_i w_i (q(x + c_i) - q(x)) with the D2Q9 weights
        lap[f] = fma_(1.0 / 6.0, fma_(4.0, hs[SB][f], hs[SA][f] + hs[S][f]), (cq[SA][f] - q) + (cq[S][f] - q));
        t1[f] = q * (1.0 - q);
        b[f] = km[f] * fma_(-P.a2, lap[f], t1[f] * fma_(-2.0, q, 1.0));
      }
      const double kp = P.kc * (cq[SB][2] - Icur);
      const double mp = fma_(P.cm[0][1], b[0], P.cm[1][1] * b[1]);
      const double ms = fma_(P.cm[0][2], b[0], P.cm[1][2] * b[1]) + (b[2] + kp);
      double Fx = 0.0, Fy = 0.0;
      if constexpr (FORM == 1) {
        // P' in the concentrations C_m (eq. VariableTransform, or its form
        // with component densities), where the energy of eq. LandauFE is a
        // sum of independent terms: for each m the bulk part
        // C f_m'(C) - f_m(C) = kappa_m/2 C^2 (1-C)(1-3C) and the gradient
        // part alpha^2 kappa_m (dC dC - (|grad C|^2/2 + C lap C) I)
        double iso = 0.0, dd = 0.0, xy = 0.0;
#pragma unroll
        for (int f = 0; f < 3; f++) {
          const double gx = (1.0 / 12.0) * fma_(4.0, hd[SB][f], hd[SA][f] + hd[S][f]);
          const double gy = fma_(0.5, cq[S][f] - cq[SA][f], (1.0 / 12.0) * (hs[S][f] - hs[SA][f]));
          const double C = cq[SB][f];
          iso = fma_(km[f] * C, fma_(0.5 * t1[f], fma_(-3.0, C, 1.0), -(P.a2 * lap[f])), iso);
          const double kx = km[f] * gx;
          xy = fma_(kx, gy, xy);
          dd = fma_(kx, gx, fma_(-(km[f] * gy), gy, dd));
        }
        const double ha = 0.5 * P.a2;
        const double Pxx = fma_(ha, dd, iso), Pyy = fma_(-ha, dd, iso), Pxy = P.a2 * xy;
        // ---- C: -div P' - psi grad kappa_c (psi - I) at row m - 2; 12 times
        // the stencil of a gradient, 3 sum_i w_i c_i q(x + c_i), summed over
        // the rows: east - west of the row below, 4 times that of the own
        // row, that of the row above; west + 4 centre + east above less below
        const double xe = east(Pxx), xw = west(Pxx), me = east(Pxy), mw = west(Pxy), ye = east(Pyy),
                     yw = west(Pyy), ke = east(kp), kw = west(kp);
        const double hxx = xe - xw, hxy = me - mw, sxy = fma_(4.0, Pxy, me + mw), syy = fma_(4.0, Pyy, ye + yw);
        const double hk = ke - kw, sk = fma_(4.0, kp, ke + kw);
        if constexpr (doC) {
          const double ps = cq[SA][2];
          const double tx = fx0 + (hxx + sxy), ty = fy0 + (hxy + syy);
          const double kx = ax[0] + hk, ky = sk - ay[0][0];
          Fx = (-1.0 / 12.0) * fma_(ps, kx, tx);
          Fy = (-1.0 / 12.0) * fma_(ps, ky, ty);
        }
        fx0 = fma_(4.0, hxx, fx1);
        fy0 = fma_(4.0, hxy, fy1);
        fx1 = hxx - sxy;
        fy1 = hxy - syy;
        ax[0] = fma_(4.0, hk, px[0]);
        px[0] = hk;
        ay[0][0] = ay[0][1];
        ay[0][1] = sk;
      } else {
        // ---- C: -(rho grad mu_rho + phi grad mu_phi + psi grad mu_psi) at
        // row m - 2 (eqs. ForceFE, GradPT), summed over the rows as above
        const double mr = fma_(P.cm[0][0], b[0], P.cm[1][0] * b[1]);
        const double mu[3] = {mr, mp, ms};
        double gx[3], gy[3];
#pragma unroll
        for (int f = 0; f < 3; f++) {
          const double e = east(mu[f]), w = west(mu[f]);
          const double h = e - w, sm = fma_(4.0, mu[f], e + w);
          gx[f] = ax[f] + h;
          gy[f] = sm - ay[f][0];
          ax[f] = fma_(4.0, h, px[f]);
          px[f] = h;
          ay[f][0] = ay[f][1];
          ay[f][1] = sm;
        }
        if constexpr (doC) {
          const double rho = P.rho0 + (double)md[SA], ph_ = mphi[SA], ps = cq[SA][2];
          Fx = (-1.0 / 12.0) * fma_(rho, gx[0], fma_(ph_, gx[1], ps * gx[2]));
          Fy = (-1.0 / 12.0) * fma_(rho, gy[0], fma_(ph_, gy[1], ps * gy[2]));
        }
      }
      if constexpr (doC) {
        Fx += P.fext[0];  // f_ext of eq. ForcingTermLBE
        Fy += P.fext[1];
        const int cy = r - H;  // the C row
        const unsigned node = interior ? (unsigned)(cy * P.nx + x) : 0xffffffffu;
        if (actC != 0) {
          Fx += from_fix(fb0);
          Fy += from_fix(fb1);
          if (interior && (actC >> j & 1)) {
            fib[2 * (long long)node] = 0;
            fib[2 * (long long)node + 1] = 0;
            force[2 * (long long)node] = Fx;
            force[2 * (long long)node + 1] = Fy;
          }
        }
        Macro2<R> o;
        R qf[9], qg[9], qh[9];
        double q0, r0;
        if constexpr (RELAX) {
#pragma unroll
          for (int i = 0; i < 9; i++) {
            qf[i] = kf[SA][i];
            qg[i] = kg[SA][i];
            qh[i] = kh[SA][i];
          }
          q0 = kg0[SA];
          r0 = kh0[SA];
          collide9(P, qf, qg, qh, q0, r0, (double)md[SA], (double)mjx[SA], (double)mjy[SA], mphi[SA], cq[SA][2], mpC,
                   msC, Fx, Fy);
        } else {
          const double ir = recip(P.rho0 + (double)md[SA]);
          const double jxd = (double)mjx[SA], jyd = (double)mjy[SA];
          o.dr = md[SA];
          o.wx = (R)((jxd + Fx) * ir);  // u + delta u, eq. VelCorrection
          o.wy = (R)((jyd + Fy) * ir);
          o.vx = (R)(fma_(0.5, Fx, jxd) * ir);  // eq. ActualFluidVel
          o.vy = (R)(fma_(0.5, Fy, jyd) * ir);
          o.gm = (R)(3.0 * P.gphi * mpC);
          o.hm = (R)(3.0 * P.gpsi * msC);
          o.phi = mphi[SA];
          o.psi = cq[SA][2];
          if constexpr (!DM) macro_pops<R>(rho0, P.psh[0], P.psh[1], o, qf, qg, qh, q0, r0);
        }
        if constexpr (DM) {
          dst.set_node(node, o);
        } else {
          if (St::kDropsOutOfRange || interior) {
            const long long nd = St::kDropsOutOfRange ? (long long)(int)node : (long long)node;
            dst.template store<R>(0, 0, nd, qf[0]);
            dst.store_rest(1, nd, q0);
            dst.store_rest(2, nd, r0);
#pragma unroll
            for (int i = 1; i < 9; i++) {
              dst.template store<R>(0, i, nd, qf[i]);
              dst.template store<R>(1, i, nd, qg[i]);
              dst.template store<R>(2, i, nd, qh[i]);
            }
          }
        }
      }
      mpC = mp;
      msC = ms;
    }
    act3 = act2;
    act2 = act1;
    act1 = act0;
  };

  if constexpr (!RELAX) load_row(0);
  constexpr int PRO = 2 * H;  // iterations before the first collision
  body(std::integral_constant<int, 0>{}, 0);
  body(std::integral_constant<int, 1>{}, 1);
  body(std::integral_constant<int, 2>{}, 2);
  body(std::integral_constant<int, 3>{}, 3);
  if constexpr (PRO == 6) {
    body(std::integral_constant<int, 4>{}, 4);
    body(std::integral_constant<int, 5>{}, 5);
  }
  for (int k = PRO; k < K; k += 3) {
    body(std::integral_constant<int, PRO>{}, k);
    if (k + 1 < K) body(std::integral_constant<int, PRO + 1>{}, k + 1);
    if (k + 2 < K) body(std::integral_constant<int, PRO + 2>{}, k + 2);
  }
}

// does the (strip, rows [y0, y1)) region of a wave read any membrane field,
// i.e. does an active tile cover a (row, lane) whose profile field or spread
// force it reads?  (rows y0-1 .. y1 of the interior lanes and one more each side)
template <int H>
__device__ __forceinline__ bool region_active(const LBParams& P, const int* __restrict__ tflag, int stamp,
                                              int strip, int y0, int y1) {
  const int j = threadIdx.x & 63;
  const int x = wrap(strip * (64 - 2 * H) - H + j, P.nx);
  bool a = false;
  if (j >= H - 1 && j < 65 - H)
    for (int r = y0 - 1; r <= y1; r++) a |= tflag[(fd_row(r, P.ny, P.wall_y) / P.tile) * P.ntx + x / P.tile] == stamp;
  return __ballot(a) != 0;
}

// The step over the whole lattice, one (strip, segment) per wave.
//
// What bounds it, at 2048^2 with 16 capsules in FP32, divergence form: 232 B
// per node from populations to populations took 246 us in a march of four
// waves through LDS rings (two barriers a row, two waves per SIMD), against
// 201 us for copying those bytes; it takes 240 us here, paced (step2d_paced).
// From Macro2 to Macro2 it moves 88 B per node (76 us at the rate of a copy) and
// takes 111 us; the vector units, some 450 instructions a row of which 200 are
// FP64, are then busy for 60 to 70 us of it.  227 registers leave two waves per
// SIMD.  A relaxing step keeps three rows of populations as well, 249 registers in
// the potential form and 256 with 11 spilled in the divergence form: without
// membranes 46 -> 42 us at 1000 x 777 and 246 -> 220 at 2048^2 in the former, 45 ->
// 43 and 233 -> 229 in the latter.
//
// P.mode: 0 every region; the same step in two passes: 1 the regions that read
// no membrane field, which may run beside the membrane kernels, 2 the others
// after them, each segment cut into npiece pieces of seg2 rows so that the few
// regions near the membranes still fill the GPU.
// NW: waves of a workgroup, 1 or (modes 0 and 1) step2d_paced().
template <class St, typename R, int FORM, class Src, class Dst, bool RELAX, int NW>
__global__ __launch_bounds__(64 * NW, step2d_waves<R>()) void k_lb2d(Src src, Dst dst, LBParams P,
                                                                     const int* __restrict__ tflag,
                                                                     const int* __restrict__ tstate,
                                                                     const double* __restrict__ Ifield,
                                                                     long long* __restrict__ fib,
                                                                     double* __restrict__ force) {
  int strip, sgm, piece = 0;
  if (P.mode == 2) {
    piece = (int)blockIdx.x % P.npiece;
    const int rg = (int)blockIdx.x / P.npiece;
    strip = rg % P.nstrip;
    sgm = rg / P.nstrip;
  } else {
    int q = dealt_index((int)blockIdx.x, (int)gridDim.x, P.nxcd) * NW;
    if constexpr (NW > 1) {
      q += __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
      if (q >= P.nstrip * P.nseg) return;  // (the others' barriers do not wait for a wave that has ended)
    }
    strip = q % P.nstrip;
    sgm = q / P.nstrip;
  }
  int y0 = sgm * P.seg, y1 = min(y0 + P.seg, P.ny);
  if (P.mode != 0) {
    if (region_active<strip_halo<Src>()>(P, tflag, tstate[1], strip, y0, y1) != (P.mode == 2)) return;
    if (P.mode == 2) {
      y0 += piece * P.seg2;
      if (y0 >= y1) return;
      y1 = min(y0 + P.seg2, y1);
    }
  }
  step2d_run<St, R, FORM, Src, Dst, RELAX, (NW > 1)>(src, dst, P, strip, y0, y1, tflag, tstate, Ifield, fib, force);
}

// the populations of the state that Macro2 holds (a call that fails between two
// steps leaves populations, as every call does)
template <class St, typename R>
__global__ __launch_bounds__(256) void k_expand2d(MacroStore2<R> src, St dst) {
  const unsigned n = blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= src.N) return;
  R f[9], g[9], h[9];
  double g0, h0;
  macro_pops<R>((R)src.rho0, src.p0, src.p1, src.node(n), f, g, h, g0, h0);
  dst.template store<R>(0, 0, n, f[0]);
  dst.store_rest(1, n, g0);
  dst.store_rest(2, n, h0);
#pragma unroll
  for (int i = 1; i < 9; i++) {
    dst.template store<R>(0, i, n, f[i]);
    dst.template store<R>(1, i, n, g[i]);
    dst.template store<R>(2, i, n, h[i]);
  }
}

}  // namespace lb
