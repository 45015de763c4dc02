// Device-side arithmetic of one node of the coupled D1Q3Q3 scheme
// (Dubois, Graille & Lallemand, arXiv 1802.02369, section 8, steps (ii)-(vii)).
//
// Formulation used on the GPU (algebraically equal to the paper's, fewer
// transcendental calls):
//   X = ln(T/T0) = (gamma-1) ln(rho/rho0) + gamma (s - s0)/cp, T = T0 e^X,
//   p = rho r T with r = cp (gamma-1)/gamma.  This is eq. gaz-parfait with
//   T0 = p0 / (rho0 r), p0 = rho0 c0^2 / gamma: one log and one exp per node,
//   both to base 2: Y = X / ln 2, T = T0 2^Y.
//   eps_eq = (2 cp lambda^2 / gamma) rho X + e_eq s, because the bracket of
//   eq. eq-energie-entropie-d1q3q3 equals e_eq of eq. energie-equilibre.
//   Step (vii): dt S_j = (sigma_e/4) (rho_j/T_j) [(u_{j+1}-u_{j-1})^2
//   + (cp/Pr) (T_{j+1}-T_{j-1})^2 / T_j], from S of eq. NS-rho-J-zeta with
//   centred differences, nu = sigma_e lambda dx (eq. nu-d1q3q3),
//   kappa = rho nu cp / Pr and dt = dx / lambda: dx cancels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lbm {

// Per-lattice constants derived on the host from lbm_params.
struct Consts {
  double rho0, irho0;
  double mJ, me;      // rho0 lambda, rho0 lambda^2
  double mz, mpsi, meps;  // rho0 cp, rho0 cp lambda, rho0 cp lambda^2
  double gm1, gcp, xs0;   // gamma - 1, gamma / cp, -gamma s0 / cp
  double gcp2, y0;        // Y = gm1 log2 rho + gcp2 s + y0: gcp / ln 2,
                          // (xs0 - gm1 ln rho0) / ln 2
  double T0, r;
  double two_l2;      // 2 lambda^2
  double eps_c;       // 2 cp lambda^2 / gamma
  double eps_y;       // eps_c ln 2
  double s_e, s_psi, s_eps;
  double src_c;       // sigma_e / 4, or 0 without the source
  double cPr;         // cp / Pr
  double fa, fb, fc;  // M^-1 for f: 1/(3 rho0), 1/(3 rho0 lambda^2), 1/(2 rho0 lambda)
  double ga, gb, gc;  // M^-1 for g: same with rho0 cp
  double gamma, cp;
  // linear equilibria (section 7, and the thermal scheme of section 4):
  // e = l[0] rho + l[1] J + l[2] zeta, psi = l[3..5] . W, eps = l[6..8] . W
  double lin[9];
  // The time step in scaled moments (see collide_local):
  double se_2;              // s_e / 2
  double ise2;              // 1 / s_e^2 (d sigma_e / d s_e = -1 / s_e^2)
  double sp_2, sx_2;        // s_psi / 2, s_eps / 2
  double hP;                // c0^2 / (gamma lambda^2) = p0 / (rho0 lambda^2)
  double hgam, hy0;         // gamma / ln 2, xs0 / ln 2
  double tg, tgy;           // 2 / (3 gamma), tg ln 2
  double hS, hC;            // source: src_c lambda^2 / (3 cp T0), cp T0 / (Pr lambda^2)
  double hSd;               // d hS / d s_e = -lambda^2 / (12 cp T0 s_e^2), or 0
  double hlin[9];           // linear equilibria in scaled moments
  int32_t eq_kind;  // 0 section 8, 1 linear, 2 isentropic fluid D1Q3
  int32_t flags;    // lbm_params.flags (LBM_CHECK_FINITE)
};

// One tile of a batched launch: tile t of lattice inst.
struct TileRef {
  int32_t inst;
  int32_t t;
};

// A lattice of a batch held in one workgroup's registers for a whole run
// (see k_batch_resident): wavefronts wave0 .. wave0 + nw - 1 of its
// workgroup.
struct ResidentItem {
  int32_t inst;
  int32_t wave0;
  int32_t nw;
  int32_t pad;
};

// rho = rho0 f0 + rho0 f+ + rho0 f-, summed in the order of the first row of
// eq. M-d1q3q3 without contraction.  X contains (gamma-1) ln rho, so a one-ulp
// change of rho moves eps_eq by ~1e-16 in absolute terms; a fixed order keeps
// rho reproducible across implementations.
__device__ __forceinline__ double density(const Consts& c, double f0, double fp,
                                          double fm) {
#pragma clang fp contract(off)
  const double a = c.rho0 * f0;
  const double b = c.rho0 * fp;
  const double d = c.rho0 * fm;
  return (a + b) + d;
}

// 1/x for the positive normal numbers of the step (rho, T): the hardware
// reciprocal estimate r (relative error e = 1 - x r below 2^-22) refined by
// one third-order step r (1 + e + e^2) = (1 - e^3)/x, within one ulp of 1/x
// (not always correctly rounded).
__device__ __forceinline__ double recip(double x) {
#pragma clang fp contract(off)
  const double r = __builtin_amdgcn_rcp(x);
  const double e = fma(-x, r, 1.0);
  return fma(r, fma(e, e, e), r);
}

// 1/x as recip, from the reciprocal square root: its estimate y is NaN for a
// negative x, so the logarithm below needs no test of its argument (two
// instructions), for one multiplication more.  y^2 x = 1 + O(2^-23), then the
// same third-order step.
__device__ __forceinline__ double recip_pos(double x) {
#pragma clang fp contract(off)
  const double y = __builtin_amdgcn_rsq(x);
  const double r = y * y;
  const double e = fma(-x, r, 1.0);
  return fma(r, fma(e, e, e), r);
}

// log2 x and 1/x of a positive finite x with one reciprocal.  Method: x = m 2^k
// with m in [sqrt(1/2), sqrt(2)) up to the 20 fraction bits of the high word,
// taken apart with 32-bit integer operations on that word (kk = k 2^20, which
// an FMA with 2^-20 adds); R = 1/(x (m+1)) gives 1/x = R (m+1)
// and 1/(m+1) = R x, each within about two ulp; log2 m = 2 atanh(z) / ln 2
// with z = (m-1)/(m+1), |z| < 0.1716, written z (c0 + w Q(w)), w = z^2, where
// Q is a degree-6 Chebyshev fit on [0, 0.02944] and c0 is 2/ln 2 rounded
// (relative error of the whole below 2e-17; coefficients from
// csrc/gen_poly.py).  Base 2 needs no product k ln 2 and gives the exponent
// of exp2_fin without a reduction by ln 2.  Non-positive, NaN or infinite x
// give NaN; subnormal x (whose inverse overflows) are not supported.
__device__ __forceinline__ double log2_inv(double x, double& inv) {
#pragma clang fp contract(off)
  const uint64_t b = __builtin_bit_cast(uint64_t, x);
  const uint32_t hi = (uint32_t)(b >> 32);
  const uint32_t kk = (hi - 0x3fe6a09eu) & 0xfff00000u;
  const double m = __builtin_bit_cast(
      double, ((uint64_t)(hi - kk) << 32) | (b & 0xffffffffu));
  const double d = m + 1.0;
  const double R = recip_pos(x * d);
  inv = R * d;
  const double z = (m - 1.0) * (R * x);
  const double w = z * z;
  double q = 0x1.afdd0afdc54ffp-3;
  q = fma(q, w, 0x1.c4ff413719d10p-3);
  q = fma(q, w, 0x1.0c9e91772d37ep-2);
  q = fma(q, w, 0x1.484b091bae181p-2);
  q = fma(q, w, 0x1.a61762b532fa8p-2);
  q = fma(q, w, 0x1.2776c50ef68fbp-1);
  q = fma(q, w, 0x1.ec709dc3a0401p-1);
  const double lm = z * fma(q, w, 0x1.71547652b82fep+1);
  return fma((double)(int32_t)kk, 0x1p-20, lm);
}

// 2^y for the moderate arguments of the equation of state: n = the nearest
// integer to y, f = y - n exactly, 2^f = 1 + f R(f) with R a degree-10
// Chebyshev fit on |f| <= 1/2 (relative error of 2^f below 2e-17; coefficients
// from csrc/gen_poly.py).  Error below one ulp.  Overflow gives +inf and
// underflow 0 (the hardware saturates n); NaN stays NaN, infinite y give NaN.
__device__ __forceinline__ double exp2_fin(double y) {
#pragma clang fp contract(off)
  const double n = __builtin_rint(y);
  const double f = y - n;
  double q = 0x1.e9d3fe4047b38p-32;
  q = fma(q, f, 0x1.e6063f7a40c36p-28);
  q = fma(q, f, 0x1.b524fae624087p-24);
  q = fma(q, f, 0x1.62bfd4776f20bp-20);
  q = fma(q, f, 0x1.ffcbfc670dce6p-17);
  q = fma(q, f, 0x1.430913096fdb5p-13);
  q = fma(q, f, 0x1.5d87fe78a5276p-10);
  q = fma(q, f, 0x1.3b2ab6fba1ddap-7);
  q = fma(q, f, 0x1.c6b08d704a0c2p-5);
  q = fma(q, f, 0x1.ebfbdff82c598p-3);
  q = fma(q, f, 0x1.62e42fefa39efp-1);
  q = fma(q, f, 1.0);
  return __builtin_amdgcn_ldexp(q, (int)n);
}

// Every function below fixes its own rounding sequence: contraction of a
// product and a sum into an FMA is off, and FMAs are written where wanted.
// A node-update therefore rounds identically in every kernel that inlines
// these functions (one-step, any tile shape, batched), and those kernels
// produce bitwise identical states.

// Thermodynamics from conserved moments: u, s, Y = log2(T/T0) and T; ir
// returns 1/rho.
__device__ __forceinline__ void thermo(const Consts& c, double rho, double J,
                                       double zeta, double& u, double& s,
                                       double& Y, double& T, double& ir) {
#pragma clang fp contract(off)
  const double lr = log2_inv(rho, ir);
  u = J * ir;
  s = zeta * ir;
  Y = fma(c.gm1, lr, fma(c.gcp2, s, c.y0));
  T = c.T0 * exp2_fin(Y);
}

__device__ __forceinline__ void thermo(const Consts& c, double rho, double J,
                                       double zeta, double& u, double& s,
                                       double& Y, double& T) {
  double ir;
  thermo(c, rho, J, zeta, u, s, Y, T, ir);
}

// Isentropic pressure p0 (rho/rho0)^gamma = rho r T0 (rho/rho0)^(gamma-1)
// of the fluid D1Q3 scheme (sections 2-3).
__device__ __forceinline__ double iso_pressure(const Consts& c, double rho) {
#pragma clang fp contract(off)
  double unused;
  return ((rho * c.r) * c.T0) *
         exp2_fin(c.gm1 * log2_inv(rho * c.irho0, unused));
}

// Step (iv): equilibria of the non-conserved moments from rho, J, zeta and
// the thermodynamic state (physical units; the initialisation uses them).
template <int EQ>
__device__ __forceinline__ void equilibria(const Consts& c, double rho,
                                           double J, double zeta, double u,
                                           double s, double Y, double T,
                                           double& e_eq, double& psi_eq,
                                           double& eps_eq) {
#pragma clang fp contract(off)
  if (EQ == 0 || c.eq_kind == 0) {
    e_eq = fma(3.0, fma(J, u, (rho * c.r) * T), -(c.two_l2 * rho));
    psi_eq = zeta * u;
    eps_eq = fma(e_eq, s, (c.eps_y * rho) * Y);
  } else if (c.eq_kind == 2) {
    e_eq = fma(3.0, fma(J, u, iso_pressure(c, rho)), -(c.two_l2 * rho));
    psi_eq = 0.0;
    eps_eq = 0.0;
  } else {
    e_eq = fma(c.lin[2], zeta, fma(c.lin[1], J, c.lin[0] * rho));
    psi_eq = fma(c.lin[5], zeta, fma(c.lin[4], J, c.lin[3] * rho));
    eps_eq = fma(c.lin[8], zeta, fma(c.lin[7], J, c.lin[6] * rho));
  }
}

// The time step works in scaled moments, which removes the scale factors
// rho0, lambda, cp, T0 from the per-node arithmetic:
//   rh = rho/rho0 = f0 + f+ + f-,  Jh = J/(rho0 lambda) = f+ - f-,
//   zh = zeta/(rho0 cp) = g0 + g+ + g-,  uh = u/lambda,  sh = s/cp,
//   Th = T/T0 = 2^Y,  Y = [(gamma-1) ln rh + gamma sh - gamma s0/cp] / ln 2,
// and the equilibria divided by the scale of their moment (rho0 lambda^2 for
// e, rho0 cp lambda for psi, rho0 cp lambda^2 for eps):
//   eh = 3 rh y - 2 rh with y = uh^2 + hP Th, hP = c0^2/(gamma lambda^2),
//   psih = zh uh,  epsh = (2/gamma) ln 2 rh Y + eh sh.
// (With rho0 = 1, rh is the density summed in the order of eq. M-d1q3q3.)
// lr returns log2 rh, ir 1/rh.
__device__ __forceinline__ void thermo_scaled(const Consts& c, double rh,
                                              double Jh, double zh, double& uh,
                                              double& sh, double& Y,
                                              double& Th, double& lr,
                                              double& ir) {
#pragma clang fp contract(off)
  lr = log2_inv(rh, ir);
  uh = Jh * ir;
  sh = zh * ir;
  Y = fma(c.gm1, lr, fma(c.hgam, sh, c.hy0));
  Th = exp2_fin(Y);
}

__device__ __forceinline__ void thermo_scaled(const Consts& c, double rh,
                                              double Jh, double zh, double& uh,
                                              double& sh, double& Y,
                                              double& Th, double& lr) {
  double ir;
  thermo_scaled(c, rh, Jh, zh, uh, sh, Y, Th, lr, ir);
}

// The thermodynamic state of a node's incoming populations, as the time
// step computes it (kept by the reverse sweep for a state it recomputes).
struct NodeThermo {
  double uh, sh, Y, Th, lr, ir, w;
  double du, dT;  // uh and Th of the right neighbour less the left one's
};

// Steps (ii)-(vi) at one node, in place on the six populations: moments,
// equilibria, relaxation, back to populations.  Returns uh, Th and the two
// factors the source needs: rw = rh / Th and w = 1 / Th.  EQ = 0, 1 or 2
// compiles those equilibria only (every lattice of the launch has that
// eq_kind); EQ = -1 selects them per lattice from c.eq_kind, whose branches
// at every node keep a lane's nodes from sharing registers.  SAVE: also
// writes the node's thermodynamic state into *save.
//
// (v) relaxation (eq. relaxation-d1q3q3) and (vi) f* = M^-1 m*, combined: only
// e, psi, eps change, so f* = f + M^-1 (m* - m).  With the entries of M^-1
// the changes are f0 -= s_e d, f+- += s_e d / 2 and g0 -= s_eps dx,
// g+- += s_eps dx / 2 +- s_psi dp / 2, where
//   d = (eh - (f+ + f- - 2 f0)) / 3,  dp = psih - (g+ - g-),
//   dx = (epsh - (g+ + g- - 2 g0)) / 3.
// For the equilibria of section 8 the sums of populations in eh and epsh
// cancel (rh = f0 + f+ + f-, rh sh = zh = g0 + g+ + g-):
//   d = rh y - (f+ + f-),  dx = rh (y sh + tgy Y) - (g+ + g-),
// with tgy = (2/(3 gamma)) ln 2: three FMAs instead of eh, epsh and their
// differences.  The kernels are bound by the issue of these instructions; with
// the base-2 logarithm and exponential a node of a P = 8 tile takes 86 VALU
// instructions (78 of them FP64, two of those reciprocal estimates at a
// quarter of the rate) where ln, exp and separate equilibria took 98 (91):
// 200 steps of 2^24 nodes 11.5 -> 10.1 ms, 4096 ragged lattices 12.5 -> 11.0
// ms for 160 steps.
template <int EQ, bool SAVE = false>
__device__ __forceinline__ void collide_local(const Consts& c, double& f0,
                                              double& fp, double& fm,
                                              double& g0, double& gp,
                                              double& gm, double& u, double& T,
                                              double& rw, double& w,
                                              NodeThermo* save = nullptr) {
#pragma clang fp contract(off)
  // (ii) the conserved moments, eq. M-d1q3q3, scaled
  const double rh = (f0 + fp) + fm;
  const double Jh = fp - fm;
  const double sf = fp + fm;
  const double sg = gp + gm;
  const double zh = g0 + sg;
  // (iv) equilibria
  double sh, Y, lr, ir;
  thermo_scaled(c, rh, Jh, zh, u, sh, Y, T, lr, ir);
  double d, dp, dx;
  if (EQ == 0 || (EQ < 0 && c.eq_kind == 0)) {
    const double y = fma(u, u, c.hP * T);
    d = fma(rh, y, -sf);
    dp = fma(zh, u, gm - gp);
    dx = fma(rh, fma(y, sh, c.tgy * Y), -sg);
  } else if (EQ == 2 || (EQ < 0 && c.eq_kind == 2)) {
    d = fma(rh, fma(u, u, c.hP * exp2_fin(c.gm1 * lr)), -sf);
    dp = gm - gp;
    dx = fma(2.0, g0, -sg) * (1.0 / 3.0);
  } else {
    const double eh = fma(c.hlin[2], zh, fma(c.hlin[1], Jh, c.hlin[0] * rh));
    const double psih = fma(c.hlin[5], zh, fma(c.hlin[4], Jh, c.hlin[3] * rh));
    const double epsh = fma(c.hlin[8], zh, fma(c.hlin[7], Jh, c.hlin[6] * rh));
    d = (eh - fma(-2.0, f0, sf)) * (1.0 / 3.0);
    dp = psih - (gp - gm);
    dx = (epsh - fma(-2.0, g0, sg)) * (1.0 / 3.0);
  }
  f0 = fma(-c.s_e, d, f0);
  fp = fma(c.se_2, d, fp);
  fm = fma(c.se_2, d, fm);
  g0 = fma(-c.s_eps, dx, g0);
  gp = fma(c.sp_2, dp, fma(c.sx_2, dx, gp));
  gm = fma(-c.sp_2, dp, fma(c.sx_2, dx, gm));
  w = recip(T);
  rw = rh * w;
  if constexpr (SAVE) *save = NodeThermo{u, sh, Y, T, lr, ir, w, 0.0, 0.0};
}

// uh and Th of a node (the halo nodes of the one-step kernel), rounded as in
// collide_local.
__device__ __forceinline__ void node_uT(const Consts& c, double f0, double fp,
                                        double fm, double g0, double gp,
                                        double gm, double& u, double& T) {
#pragma clang fp contract(off)
  const double rh = (f0 + fp) + fm;
  const double Jh = fp - fm;
  const double zh = g0 + (gp + gm);
  double sh, Y, lr;
  thermo_scaled(c, rh, Jh, zh, u, sh, Y, T, lr);
}

// Step (vii): adds the increment of zeta at node j, already divided into the
// M^-1 column of zeta (each of g0, g+, g- receives ga dt S_j), from scaled
// quantities: ga dt S_j = hS rh wh [(uh_{j+1} - uh_{j-1})^2
// + hC (Th_{j+1} - Th_{j-1})^2 wh] with wh = 1/Th_j, as an FMA each.
__device__ __forceinline__ void add_source(const Consts& c, double rw, double w,
                                           double uL, double uR, double TL,
                                           double TR, double& g0, double& gp,
                                           double& gm) {
#pragma clang fp contract(off)
  const double du = uR - uL;
  const double dT = TR - TL;
  const double a = c.hS * rw;
  const double q = fma(du, du, (c.hC * (dT * dT)) * w);
  g0 = fma(a, q, g0);
  gp = fma(a, q, gp);
  gm = fma(a, q, gm);
}

// Equilibrium populations from (rho, J, zeta).
__device__ __forceinline__ void equilibrium(const Consts& c, double rho,
                                            double J, double zeta, double f[6]) {
#pragma clang fp contract(off)
  double u, s, Y, T;
  thermo(c, rho, J, zeta, u, s, Y, T);
  double e_eq, psi_eq, eps_eq;
  equilibria<-1>(c, rho, J, zeta, u, s, Y, T, e_eq, psi_eq, eps_eq);
  const double fr = c.fa * rho, fe = c.fb * e_eq, fj = c.fc * J;
  f[0] = fr - fe;
  f[1] = fma(0.5, fe, fr) + fj;
  f[2] = fma(0.5, fe, fr) - fj;
  const double gz = c.ga * zeta, ge = c.gb * eps_eq, gj = c.gc * psi_eq;
  f[3] = gz - ge;
  f[4] = fma(0.5, ge, gz) + gj;
  f[5] = fma(0.5, ge, gz) - gj;
}

// Cross-lane moves of a double over the whole 64-lane wavefront (DPP
// wave_shr:1 / wave_shl:1 on both 32-bit halves).  from_left: lane l receives
// lane l-1's value; from_right: lane l receives lane l+1's value.  The edge
// lane (0, resp. 63) has no source and receives 0 (bound_ctrl); callers use
// it only for nodes whose values are discarded or replaced.
__device__ __forceinline__ double from_left(double v) {
  const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), 0x138, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), 0x138, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double from_right(double v) {
  const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), 0x130, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), 0x130, 0xf, 0xf, true);
  return __hiloint2double(hi, lo);
}

// Node-wise kernels of a batch: workgroup b of 256 threads takes the nodes
// [1024 b, 1024 b + 1024) of the state, whatever lattices they belong to, so
// the accesses are aligned and a long lattice is spread over the chip (one
// workgroup per lattice took 3.1 ms for the initial-field adjoint of 2^20
// nodes, 20 us this way).  The lattices of its first and last node come from
// the offsets by bisection (scalar loads); where they are the same, the
// constants are the whole workgroup's, else each thread finds its own node's.
constexpr int kNodeBlock = 1024;

__device__ __forceinline__ int64_t find_lattice(const int64_t* __restrict__ offs,
                                                int64_t lo, int64_t hi,
                                                int64_t j) {
  while (lo < hi) {  // the last i with offs[i] <= j
    const int64_t mid = (lo + hi + 1) >> 1;
    if (offs[mid] <= j)
      lo = mid;
    else
      hi = mid - 1;
  }
  return lo;
}

template <class Body>
__device__ __forceinline__ void batch_nodes(const Consts* __restrict__ cs,
                                            const int64_t* __restrict__ offs,
                                            int64_t n_inst, Body body) {
  const int64_t n = offs[n_inst];
  const int64_t b = (int64_t)blockIdx.x * kNodeBlock;
  if (b >= n) return;
  const int64_t e = b + kNodeBlock < n ? b + kNodeBlock : n;
  const int64_t first = find_lattice(offs, 0, n_inst - 1, b);
  if (first + 1 == n_inst || e <= offs[first + 1]) {
    const Consts c = cs[first];
#pragma unroll
    for (int k = 0; k < kNodeBlock / 256; ++k) {
      const int64_t j = b + k * 256 + threadIdx.x;
      if (j < e) body(c, j);
    }
  } else {
    const int64_t last = find_lattice(offs, first + 1, n_inst - 1, e - 1);
    for (int64_t j = b + threadIdx.x; j < e; j += 256)
      body(cs[find_lattice(offs, first, last, j)], j);
  }
}

__device__ __forceinline__ int64_t wrap_mod(int64_t x, int64_t n) {
  int64_t r = x % n;
  return r < 0 ? r + n : r;
}

}  // namespace lbm
