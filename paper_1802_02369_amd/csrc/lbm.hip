// HIP kernels and C ABI of the coupled D1Q3Q3 lattice Boltzmann scheme
// (Dubois, Graille & Lallemand, arXiv 1802.02369) for gfx950.
//
// Forward kernels:
//   k_step_plain   one time step per launch, one node per thread; the
//                  neighbours' u and T for the source term and the streamed
//                  populations go through LDS, so every store is aligned.
//   k_step_tile    K time steps per launch.  Each 64-lane wavefront holds
//                  64*P consecutive nodes (P per lane, contiguous) in VGPRs
//                  for all K steps; neighbour values move between lanes with
//                  DPP wave shifts, and neighbouring wavefronts of a
//                  workgroup share 2M lanes that are refreshed through LDS
//                  every MP/2 steps.  A step has radius 2 (the source reads u, T at
//                  j+-1 of the node whose populations stream to j+-1), so a
//                  tile loads 2K halo nodes on each side and stores its
//                  interior.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <algorithm>
#include <cstring>
#include <string>

#include "../../include/lbm.h"
#include "lbm_device.hpp"
#include "lbm_internal.hpp"
#include "lbm_tile.hpp"

using lbm::Consts;

// ------------------------------------------------------------ errors ----

namespace lbm {
thread_local std::string g_err;

int set_err(int code, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_err = buf;
  return code;
}

int hip_check(hipError_t e, const char* what) {
  if (e == hipSuccess) return LBM_OK;
  return set_err(LBM_EHIP, "%s: %s", what, hipGetErrorString(e));
}

constexpr double kLn2 = 0x1.62e42fefa39efp-1;  // ln 2

static bool finite_pos(double x) { return std::isfinite(x) && x > 0.0; }
static bool valid_rate(double s) { return std::isfinite(s) && s > 0.0 && s < 2.0; }

int make_consts(const lbm_params* p, Consts* c) {
  if (!p) return set_err(LBM_EINVAL, "params is NULL");
  if (!finite_pos(p->lambda) || !finite_pos(p->rho0) || !finite_pos(p->cp) ||
      !finite_pos(p->prandtl) || !finite_pos(p->c0))
    return set_err(LBM_EINVAL,
                   "lambda, rho0, cp, prandtl and c0 must be finite and > 0");
  if (!(std::isfinite(p->gamma) && p->gamma > 1.0))
    return set_err(LBM_EINVAL, "gamma must be finite and > 1");
  if (!std::isfinite(p->s0) || !std::isfinite(p->u0_lin) ||
      !std::isfinite(p->s0_lin) || !std::isfinite(p->alpha))
    return set_err(LBM_EINVAL, "s0, u0_lin, s0_lin, alpha must be finite");
  if (!valid_rate(p->s_e) || !valid_rate(p->s_psi) || !valid_rate(p->s_eps))
    return set_err(LBM_EINVAL, "relaxation rates must lie in (0, 2)");
  if (p->source_on != 0 && p->source_on != 1)
    return set_err(LBM_EINVAL, "source_on must be 0 or 1");
  if (p->eq_kind < 0 || p->eq_kind > 3)
    return set_err(LBM_EINVAL, "eq_kind must be 0, 1, 2 or 3");
  if (p->eq_kind >= 2 && p->source_on)
    return set_err(LBM_EINVAL, "the single-distribution schemes need source_on = 0");
  if (p->eq_kind == 3 && !(p->alpha > -2.0 && p->alpha < 1.0))
    return set_err(LBM_EINVAL, "alpha must lie in (-2, 1)");
  if (p->eq_kind == 1 && (p->lambda != 1.0 || p->cp != 1.0 || p->rho0 != 1.0))
    return set_err(LBM_EINVAL,
                   "linear equilibria are defined for lambda = cp = rho0 = 1");
  if ((p->flags & ~LBM_CHECK_FINITE) != 0 || p->reserved != 0)
    return set_err(LBM_EINVAL, "flags may hold LBM_CHECK_FINITE only; reserved must be 0");
  const double l = p->lambda, cp = p->cp, r0 = p->rho0, g = p->gamma;
  std::memset(c, 0, sizeof *c);
  c->rho0 = r0;
  c->irho0 = 1.0 / r0;
  c->mJ = r0 * l;
  c->me = r0 * l * l;
  c->mz = r0 * cp;
  c->mpsi = r0 * cp * l;
  c->meps = r0 * cp * l * l;
  c->gm1 = g - 1.0;
  c->gcp = g / cp;
  c->xs0 = -g * p->s0 / cp;
  c->r = cp * (g - 1.0) / g;
  const double p0 = r0 * p->c0 * p->c0 / g;
  c->T0 = p0 / (r0 * c->r);
  c->two_l2 = 2.0 * l * l;
  c->eps_c = 2.0 * cp * l * l / g;
  c->s_e = p->s_e;
  c->s_psi = p->s_psi;
  c->s_eps = p->s_eps;
  c->src_c = p->source_on ? 0.25 * (1.0 / p->s_e - 0.5) : 0.0;
  c->cPr = cp / p->prandtl;
  c->fa = 1.0 / (3.0 * r0);
  c->fb = 1.0 / (3.0 * r0 * l * l);
  c->fc = 1.0 / (2.0 * r0 * l);
  c->ga = 1.0 / (3.0 * r0 * cp);
  c->gb = 1.0 / (3.0 * r0 * cp * l * l);
  c->gc = 1.0 / (2.0 * r0 * cp * l);
  c->gamma = g;
  c->cp = cp;
  c->se_2 = p->s_e / 2.0;
  c->ise2 = 1.0 / (p->s_e * p->s_e);
  c->sp_2 = p->s_psi / 2.0;
  c->sx_2 = p->s_eps / 2.0;
  c->hP = p->c0 * p->c0 / (g * l * l);
  c->hgam = g / kLn2;
  c->hy0 = c->xs0 / kLn2;
  c->tg = 2.0 / (3.0 * g);
  c->tgy = c->tg * kLn2;
  c->hS = c->src_c * l * l / (3.0 * cp * c->T0);
  c->hC = cp * c->T0 / (p->prandtl * l * l);
  c->hSd = p->source_on ? -0.25 * c->ise2 * l * l / (3.0 * cp * c->T0) : 0.0;
  c->gcp2 = c->gcp / kLn2;
  c->y0 = (c->xs0 - c->gm1 * std::log(r0)) / kLn2;
  c->eps_y = c->eps_c * kLn2;
  c->eq_kind = p->eq_kind;
  c->flags = p->flags;
  if (p->eq_kind == 1) {
    // Eq. equilibres-NS-linearise (lambda = cp = rho0 = 1).  The zeta
    // coefficient of e_eq is 3 c0^2 (printed 3 u0^2): the flux of J in
    // eq. NS-rho-J-zeta-linearise has the term c0^2 d_x zeta, and the
    // printed psi_eq, eps_eq are compatible with that system's entropy
    // equation at second order only with it.
    const double u0 = p->u0_lin, s0 = p->s0_lin, c0 = p->c0;
    c->lin[0] = 3.0 * (1.0 - s0) * c0 * c0 - 3.0 * u0 * u0 - 2.0;
    c->lin[1] = 6.0 * u0;
    c->lin[2] = 3.0 * c0 * c0;
    c->lin[3] = -u0 * s0;
    c->lin[4] = s0;
    c->lin[5] = u0;
    c->lin[6] = -3.0 * (s0 * c0) * (s0 * c0) - 6.0 * s0 * u0 * u0 +
                3.0 * s0 * c0 * c0 + 2.0 - 2.0 * s0 - 2.0 / g;
    c->lin[7] = 6.0 * u0 * s0;
    c->lin[8] = 3.0 * (u0 * u0 + s0 * c0 * c0);
  } else if (p->eq_kind == 3) {
    // Thermal scheme of section 4: its equilibria are linear in (rho, J,
    // zeta), so it runs on the linear path.
    c->eq_kind = 1;
    c->lin[0] = 3.0 * p->c0 * p->c0 - 2.0 * l * l;
    c->lin[5] = p->u0_lin;
    c->lin[8] = p->alpha * l * l;
  }
  // the same linear equilibria in scaled moments: e / (rho0 lambda^2),
  // psi / (rho0 cp lambda), eps / (rho0 cp lambda^2) in terms of
  // rho / rho0, J / (rho0 lambda), zeta / (rho0 cp)
  c->hlin[0] = c->lin[0] / (l * l);
  c->hlin[1] = c->lin[1] / l;
  c->hlin[2] = c->lin[2] * cp / (l * l);
  c->hlin[3] = c->lin[3] / (cp * l);
  c->hlin[4] = c->lin[4] / cp;
  c->hlin[5] = c->lin[5] / l;
  c->hlin[6] = c->lin[6] / (cp * l * l);
  c->hlin[7] = c->lin[7] / (cp * l);
  c->hlin[8] = c->lin[8] / (l * l);
  return LBM_OK;
}

}  // namespace lbm

// ----------------------------------------------------------- kernels ----

namespace {

// nodes per block of the one-step kernel: 15 wavefronts and one more for the
// halo (960 against 256 nodes per block: 60.7 -> 61.4 GLUPS at N = 2^24), or 3
// and one while blocks of 960 would not give every compute unit one
constexpr int kPlainBlock = 960, kPlainSmall = 192;
constexpr int kDiagBlock = 256;
constexpr int kDiagMaxBlocks = 1024;

__global__ __launch_bounds__(256) void k_equilibrium(
    Consts c, const double* __restrict__ rho, const double* __restrict__ J,
    const double* __restrict__ zeta, double* __restrict__ f, int64_t n) {
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= n) return;
  double v[6];
  lbm::equilibrium(c, rho[j], J[j], zeta[j], v);
#pragma unroll
  for (int k = 0; k < 6; ++k) f[k * n + j] = v[k];
}

__global__ __launch_bounds__(256) void k_moments(Consts c,
                                                 const double* __restrict__ f,
                                                 double* __restrict__ m,
                                                 int64_t n) {
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= n) return;
  const double f0 = f[j], fp = f[n + j], fm = f[2 * n + j];
  const double g0 = f[3 * n + j], gp = f[4 * n + j], gm = f[5 * n + j];
  const double sf = fp + fm, sg = gp + gm;
  m[j] = lbm::density(c, f0, fp, fm);
  m[n + j] = c.mJ * (fp - fm);
  m[2 * n + j] = c.mz * (g0 + sg);
  m[3 * n + j] = c.me * (sf - 2.0 * f0);
  m[4 * n + j] = c.mpsi * (gp - gm);
  m[5 * n + j] = c.meps * (sg - 2.0 * g0);
}

// One time step, one node per thread.  Block b stores nodes
// [b*B, b*B + B), each thread its own node with aligned
// stores: the streamed values f+(j) = f+*(j-1) and f-(j) = f-*(j+1) come
// through LDS.  One more wavefront handles the four halo nodes: b*B - 1 and
// b*B + B are collided too (their f+* and f-* stream into the block), and
// b*B - 2, b*B + B + 1 give u, T for those two nodes' sources.  LDS slot s
// holds node b*B - 2 + s.  NT: non-temporal loads and stores, for states far
// larger than the caches (measured on a 6-array copy: 6.1 against 5.6 TB/s;
// with stores shifted by one node, as push streaming writes them, 5.5).
// HALO: the step is in place (fin = fout = f): the four halo nodes of every
// block, which other blocks overwrite, come from `halo`, where k_save_halo put
// them before; a block's own nodes are read and written by one thread each.
// One step by itself thus costs its 96 bytes per node and a small launch
// instead of a step into the second state and a copy of it back (n = 4194301:
// 72 us instead of 82 + 85).
template <int B, int EQ, bool NT, bool HALO>
__global__ __launch_bounds__(B + 64) void k_step_plain(
    Consts c, const double* fin, double* fout, const double* halo, int64_t n) {
  constexpr int NS = B + 4;
  __shared__ double su[NS], sT[NS], sfp[NS], sgp[NS], sfm[NS], sgm[NS];
  const int tid = threadIdx.x;
  const int64_t b0 = (int64_t)blockIdx.x * B;
  const int64_t rem = n - b0;
  const int nloc = rem < B ? (int)rem : B;
  // this thread's node and LDS slot; -1: no node
  int slot = -1;
  int64_t j = 0;
  if (tid < B) {
    if (tid < nloc) {
      slot = tid + 2;
      j = b0 + tid;
    }
  } else if (tid < B + 4) {
    const int h = tid - B;  // b0-2, b0-1, b0+nloc, b0+nloc+1
    slot = h < 2 ? h : nloc + h;
    j = lbm::wrap_mod(b0 - 2 + slot, n);
  }
  const bool own = tid < nloc;
  const bool collide = slot >= 1 && slot <= nloc + 2;
  double f0 = 0, fp = 0, fm = 0, g0 = 0, gp = 0, gm = 0, u = 0, T = 0, rw = 0,
         w = 0;
  if (slot >= 0) {
    if (HALO && tid >= B) {
      const double* h = halo + ((int64_t)blockIdx.x * 4 + (tid - B)) * 6;
      f0 = h[0];
      fp = h[1];
      fm = h[2];
      g0 = h[3];
      gp = h[4];
      gm = h[5];
    } else if (NT) {
      f0 = __builtin_nontemporal_load(&fin[j]);
      fp = __builtin_nontemporal_load(&fin[n + j]);
      fm = __builtin_nontemporal_load(&fin[2 * n + j]);
      g0 = __builtin_nontemporal_load(&fin[3 * n + j]);
      gp = __builtin_nontemporal_load(&fin[4 * n + j]);
      gm = __builtin_nontemporal_load(&fin[5 * n + j]);
    } else {
      f0 = fin[j];
      fp = fin[n + j];
      fm = fin[2 * n + j];
      g0 = fin[3 * n + j];
      gp = fin[4 * n + j];
      gm = fin[5 * n + j];
    }
    if (collide)
      lbm::collide_local<EQ>(c, f0, fp, fm, g0, gp, gm, u, T, rw, w);
    else
      lbm::node_uT(c, f0, fp, fm, g0, gp, gm, u, T);
    su[slot] = u;
    sT[slot] = T;
  }
  __syncthreads();
  if (collide) {
    lbm::add_source(c, rw, w, su[slot - 1], su[slot + 1], sT[slot - 1],
                    sT[slot + 1], g0, gp, gm);
    sfp[slot] = fp;
    sgp[slot] = gp;
    sfm[slot] = fm;
    sgm[slot] = gm;
  }
  __syncthreads();
  if (!own) return;
  // (viii) streaming, pulled from the neighbours' post-collision values
  fp = sfp[slot - 1];
  gp = sgp[slot - 1];
  fm = sfm[slot + 1];
  gm = sgm[slot + 1];
  if (NT) {
    __builtin_nontemporal_store(f0, &fout[j]);
    __builtin_nontemporal_store(fp, &fout[n + j]);
    __builtin_nontemporal_store(fm, &fout[2 * n + j]);
    __builtin_nontemporal_store(g0, &fout[3 * n + j]);
    __builtin_nontemporal_store(gp, &fout[4 * n + j]);
    __builtin_nontemporal_store(gm, &fout[5 * n + j]);
  } else {
    fout[j] = f0;
    fout[n + j] = fp;
    fout[2 * n + j] = fm;
    fout[3 * n + j] = g0;
    fout[4 * n + j] = gp;
    fout[5 * n + j] = gm;
  }
}

// The halo nodes of every block of k_step_plain, [block][4][6].
__global__ __launch_bounds__(256) void k_save_halo(const double* __restrict__ f,
                                                   double* __restrict__ halo,
                                                   int64_t n, int64_t blocks,
                                                   int B) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= 4 * blocks) return;
  const int64_t b0 = (i >> 2) * B;
  const int h = (int)(i & 3);
  const int64_t rem = n - b0;
  const int nloc = rem < B ? (int)rem : B;
  const int64_t j = lbm::wrap_mod(b0 - 2 + (h < 2 ? h : nloc + h), n);
#pragma unroll
  for (int q = 0; q < 6; ++q) halo[i * 6 + q] = f[q * n + j];
}

// Wavefronts per SIMD the tile kernels are compiled for (the register
// budget: 512 / n VGPRs each).  Kernels of one kind of equilibria are held to
// three at P = 8 (they hold 150 VGPRs and spill nothing; three measured 297 ->
// 312 GLUPS at N = 2^24 against two); with 8 wavefronts per workgroup a CU
// gains no third one, so those stay at two.  The kernels that select the
// equilibria per lattice (226 VGPRs at P = 8, 127 at P = 4), or store the
// states of a reverse sweep, are not held to a budget at P >= 4: a launch whose
// lattices share linear or fluid equilibria has its own (150 and 151 VGPRs at
// P = 8; n = 500 in one workgroup 0.45 -> 0.35 us per step, 3e5 1.56 -> 1.37,
// 8e6 33.8 -> 31.1).  P <= 2 needs few registers: four.
constexpr int tile_waves_per_simd(int P, int WG, bool one_eq_plain) {
  return P <= 2 ? 4 : WG > 8 ? 3 : !one_eq_plain ? 1 : P == 8 && WG <= 4 ? 3 : 2;
}

template <int P, int WG, int M, int EQ>
__global__ __launch_bounds__(64 * WG, tile_waves_per_simd(P, WG, EQ >= 0)) void k_step_tile(
    Consts c, const double* __restrict__ fin, double* __restrict__ fout,
    int64_t n, int K, int64_t ntiles) {
  const int64_t tile = blockIdx.x;
  if (tile >= ntiles) return;  // uniform over the workgroup
  const int OUT = lbm::tile_nodes(P, WG, M) - 4 * K;
  tile_run<P, WG, M, EQ>(c, fin, fout, n, n, tile * OUT - 2 * K, 2 * K, K);
}

// Batched form: workgroup b advances tile tiles[b].t of lattice tiles[b].inst,
// which occupies [offs[inst], offs[inst+1]) of every array of a state of
// array stride S, with that lattice's own constants.  The tiling (halo H,
// OUT = W - 2H) is fixed by the tile table; a launch runs K <= H/2 steps.
// EVERY: store the states of a checkpoint segment that the reverse sweep
// loads (see tile_run: first, every).
template <int P, int WG, int M, int EQ, bool EVERY>
__global__ __launch_bounds__(64 * WG, tile_waves_per_simd(P, WG, EQ >= 0 && !EVERY)) void k_batch_tile(
    const Consts* __restrict__ cs, const int64_t* __restrict__ offs,
    const lbm::TileRef* __restrict__ tiles, const double* __restrict__ fin,
    double* __restrict__ fout, int64_t S, int H, int K, int64_t ntiles,
    int64_t state_stride, int first, int every) {
  const int64_t b = blockIdx.x;
  if (b >= ntiles) return;  // uniform over the workgroup
  const lbm::TileRef tr = tiles[b];
  const int64_t off = offs[tr.inst];
  const int64_t n = offs[tr.inst + 1] - off;
  const Consts c = cs[tr.inst];
  const int OUT = lbm::tile_nodes(P, WG, M) - 2 * H;
  tile_run<P, WG, M, EQ>(c, fin + off, fout + off, S, n, (int64_t)tr.t * OUT - H, H,
                  K, EVERY, state_stride, first, every);
}

// Resident lattices of a batch: a periodic lattice of L nodes short enough
// for the registers of one workgroup runs every time step of the call in one
// launch, with no halo and no global memory traffic between the first load
// and the last store.  The lattice is laid out as a tile that starts at
// position -P: lane l of its wavefront w (w = 0 .. nw-1, nw = ceil(L / 62P))
// holds positions 62 P w + P (l - 1) + k, neighbouring wavefronts sharing
// two lanes as in the tile kernels.  Positions outside [0, L) stand for the
// nodes their periodic image names: lane 0 of wavefront 0 holds nodes
// L-P .. L-1 and positions L .. L+P-1 hold nodes 0 .. P-1; every P/2 steps
// those copies and the mirror lanes are refreshed from the lanes that own
// the nodes, through LDS with one workgroup barrier (every lattice of a
// workgroup runs the same steps, so all its wavefronts meet at each).  A
// step has radius 2, so the wrong values that come in from beyond a copy
// (or from the unused positions past L+P) move two nodes per step and stay
// inside the copy until the refresh, as for the mirror lanes.  Several
// lattices share a workgroup of kResWaves wavefronts (items[wg_first[b] ..
// wg_first[b+1]), each on its own wavefronts); wavefronts without a
// lattice end at once.
// Every node-update rounds as in the other kernels: results are bitwise
// those of the tiled path.
constexpr int kResWaves = lbm::kResidentWaves;

// The copies of the periodic wrap, in P-node blocks: every lane holds the
// P positions p0 .. p0+P-1 with p0 a multiple of P, so with o = L mod P
// the nodes L-P .. L-1 are the last P - o nodes of the owner lane at
// L-P-o followed by the first o of the owner lane at L-o, and the
// positions L .. L+P-1 are the last P - o of the lane at L-o (every lane
// holding that block: a mirror lane as well) followed by the first o of
// the lane at L-o+P.  Those owners write their whole P nodes into a 2P-node
// buffer read at offset o, which keeps the exchange free of per-node
// conditions.
template <int P>
__device__ __forceinline__ void resident_refresh(
    double (&f)[6][P], double (*edge)[2][6 * P], double (*head)[6 * P],
    double (*tail)[12 * P], int lane, int wave, int lw, int nw, int w0,
    int L) {
  const int p0 = 62 * P * lw + P * (lane - 1);  // position of node 0 of the lane
  const int o = L % P;                          // uniform over the lattice
  if (lane == 1 || lane == 62) {
    double* d = edge[wave][lane == 62];
#pragma unroll
    for (int q = 0; q < 6; ++q)
#pragma unroll
      for (int k = 0; k < P; ++k) d[q * P + k] = f[q][k];
  }
  if (lw == 0 && lane == 1) {  // nodes 0 .. P-1
#pragma unroll
    for (int q = 0; q < 6; ++q)
#pragma unroll
      for (int k = 0; k < P; ++k) head[w0][q * P + k] = f[q][k];
  }
  const bool owner = lane >= 1 && lane <= 62;
  if (owner && (p0 == L - P - o || (o != 0 && p0 == L - o))) {  // nodes L-P .. L-1
    double* d = tail[w0] + (p0 == L - o ? P : 0);
#pragma unroll
    for (int q = 0; q < 6; ++q)
#pragma unroll
      for (int k = 0; k < P; ++k) d[q * 2 * P + k] = f[q][k];
  }
  __syncthreads();
  if (lane == 0 && lw > 0) {
#pragma unroll
    for (int q = 0; q < 6; ++q)
#pragma unroll
      for (int k = 0; k < P; ++k) f[q][k] = edge[wave - 1][1][q * P + k];
  } else if (lane == 63 && lw < nw - 1) {
#pragma unroll
    for (int q = 0; q < 6; ++q)
#pragma unroll
      for (int k = 0; k < P; ++k) f[q][k] = edge[wave + 1][0][q * P + k];
  } else if (lane == 0) {  // lw == 0: nodes L-P .. L-1
#pragma unroll
    for (int q = 0; q < 6; ++q)
#pragma unroll
      for (int k = 0; k < P; ++k) f[q][k] = tail[w0][q * 2 * P + o + k];
  }
  // positions L .. L+P-1 (nodes 0 .. P-1 again), after the mirror reads
  if (p0 == L - o) {
#pragma unroll
    for (int q = 0; q < 6; ++q)
#pragma unroll
      for (int k = 0; k < P; ++k)
        if (k >= o) f[q][k] = head[w0][q * P + k - o];
  } else if (o != 0 && p0 == L - o + P) {
#pragma unroll
    for (int q = 0; q < 6; ++q)
#pragma unroll
      for (int k = 0; k < P; ++k)
        if (k < o) f[q][k] = head[w0][q * P + P - o + k];
  }
}

template <int P, int EQ>
__global__ __launch_bounds__(64 * kResWaves, 3) void k_batch_resident(
    const Consts* __restrict__ cs, const int64_t* __restrict__ offs,
    const lbm::ResidentItem* __restrict__ items,
    const int32_t* __restrict__ wg_first, const double* fin, double* fout,
    int64_t S, int64_t T) {
  // fin and fout may be the same state (the run is in place): no restrict
  constexpr int WG = kResWaves;
  constexpr int WW = 64 * P;
  constexpr int WS = 62 * P;
  __shared__ double stage[WG * (WW + 64)];
  __shared__ double edge[2][WG][2][6 * P];
  __shared__ double head[2][WG][6 * P];
  __shared__ double tail[2][WG][12 * P];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // this wavefront's lattice (uniform over the wavefront)
  int item = -1;
  for (int i = wg_first[blockIdx.x]; i < wg_first[blockIdx.x + 1]; ++i) {
    const int w0 = items[i].wave0;
    if (wave >= w0 && wave < w0 + items[i].nw) item = i;
  }
  if (item < 0) return;
  const lbm::ResidentItem it = items[item];
  const int lw = wave - it.wave0;
  const int64_t off = offs[it.inst];
  const int L = (int)(offs[it.inst + 1] - off);
  const Consts c = cs[it.inst];
  double* lds = stage + wave * (WW + 64);
  const int64_t wstart = -P + (int64_t)lw * WS;
  double f[6][P];
  tile_load<P>(fin + off, S, L, wstart, false, true, lane, lds, f);
  // every wavefront has loaded before any stores (fout may be fin)
  __syncthreads();
  int since = 0, buf = 0;
  for (int64_t step = 0; step < T; ++step) {
    tile_step<P, EQ>(c, f);
    if (++since == P / 2 && step + 1 < T) {
      resident_refresh<P>(f, edge[buf], head[buf], tail[buf], lane, wave, lw,
                          it.nw, it.wave0, L);
      buf ^= 1;
      since = 0;
    }
  }
  // owned positions 0 .. L-1: lanes 1 .. 62, and 63 in the last wavefront
  tile_store<P>(fout + off, S, L, wstart, P, lw < it.nw - 1 ? WW - P : WW, lane,
                lds, f);
}

// The same for 1, 2 or 4 nodes per lane (short lattices, or a chip that has
// room: a step of P nodes per lane takes about 0.1 + 0.15 P us on a SIMD of its
// own), with M = 8/P mirror lanes on each side of a wavefront, so that at every
// P the copies hold 8 nodes and are refreshed every four steps.  Lane l of
// wavefront lw holds positions WS lw + P (l - M) + k, WS = (64 - 2M) P; lanes
// M .. 63-M own the positions below L.  Published before a refresh: the 8
// nodes next to the mirror lanes at both ends of every wavefront, and the
// lattice's last 8 nodes; what a position that is not owned takes from them
// (its mirror, or its periodic image) is worked out once.  Positions from
// L + 8 on are never refreshed: what they hold reaches 8 nodes in, to L.
// `copies`: two buffers of 3 x 48 doubles per wavefront of the workgroup
// (left edge, right edge, tail of a lattice by its first wavefront).
constexpr int kCopyDoubles = 3 * 48;

template <int P, int EQ>
__device__ __forceinline__ void resident_run(
    const Consts& c, const double* fin, double* fout, int64_t S, int L,
    int lane, int wave, int lw, int nw, int W, int64_t T, double* stage,
    double* copies) {
  constexpr int M = 8 / P;
  constexpr int WW = 64 * P;
  constexpr int WS = (64 - 2 * M) * P;
  const int w0 = wave - lw;
  const int p0 = WS * lw + P * (lane - M);
  // offsets into a buffer: left and right edge of wavefront w, tail
  auto edge = [](int w, int side) { return (2 * w + side) * 48; };
  const int tail = (2 * W + w0) * 48;
  const bool hi = lane >= 32;
  const int pl = hi ? lane - (64 - 2 * M) : lane - M;
  const int pub = pl >= 0 && pl < M ? edge(wave, hi) + pl * P : -1;
  const bool mid = lane >= M && lane < 64 - M;
  int put[P], src[P];
#pragma unroll
  for (int k = 0; k < P; ++k) {
    const int p = p0 + k;
    put[k] = mid && p < L && p >= L - 8 ? tail + p - (L - 8) : -1;
    if (mid && p < L)
      src[k] = -1;  // owned
    else if (p < 0)
      src[k] = tail + p + 8;
    else if (p >= L)
      src[k] = p - L < 8 ? edge(w0, 0) + p - L : -1;
    else if (lane < M)
      src[k] = edge(wave - 1, 1) + lane * P + k;
    else
      src[k] = edge(wave + 1, 0) + (lane - (64 - M)) * P + k;
  }
  double f[6][P];
  tile_load<P>(fin, S, L, WS * lw - 8, false, true, lane, stage, f);
  // every wavefront has loaded before any stores (fout may be fin)
  __syncthreads();
  int since = 0;
  double* buf = copies;
  for (int64_t step = 0; step < T; ++step) {
    tile_step<P, EQ>(c, f);
    if (++since == 4 && step + 1 < T) {
      if (pub >= 0) {
#pragma unroll
        for (int q = 0; q < 6; ++q)
#pragma unroll
          for (int k = 0; k < P; ++k) buf[pub + q * 8 + k] = f[q][k];
      }
#pragma unroll
      for (int k = 0; k < P; ++k)
        if (put[k] >= 0) {
#pragma unroll
          for (int q = 0; q < 6; ++q) buf[put[k] + q * 8] = f[q][k];
        }
      __syncthreads();
#pragma unroll
      for (int k = 0; k < P; ++k)
        if (src[k] >= 0) {
#pragma unroll
          for (int q = 0; q < 6; ++q) f[q][k] = buf[src[k] + q * 8];
        }
      buf = buf == copies ? copies + W * kCopyDoubles : copies;
      since = 0;
    }
  }
  tile_store<P>(fout, S, L, WS * lw - 8, 8, WW - 8, lane, stage, f);
}

// Dynamic LDS of a workgroup of W wavefronts: the copies and, for more than
// two nodes per lane, the load and store staging.
constexpr size_t resident_lds(int P, int W) {
  return sizeof(double) * W * (2 * kCopyDoubles + (staged(P) ? 64 * P + 64 : 0));
}

template <int P>
__device__ __forceinline__ double* resident_stage(double* sm, int W, int wave) {
  return staged(P) ? sm + W * 2 * kCopyDoubles + wave * (64 * P + 64) : sm;
}

// Lattices of a batch (items), W wavefronts per workgroup.
template <int P, int EQ>
__global__ __launch_bounds__(1024) void k_batch_resident_small(
    const Consts* __restrict__ cs, const int64_t* __restrict__ offs,
    const lbm::ResidentItem* __restrict__ items,
    const int32_t* __restrict__ wg_first, const double* fin, double* fout,
    int64_t S, int64_t T) {
  extern __shared__ double sm[];
  const int W = blockDim.x >> 6;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int item = -1;  // this wavefront's lattice (uniform over the wavefront)
  for (int i = wg_first[blockIdx.x]; i < wg_first[blockIdx.x + 1]; ++i) {
    const int w0 = items[i].wave0;
    if (wave >= w0 && wave < w0 + items[i].nw) item = i;
  }
  if (item < 0) return;
  const lbm::ResidentItem it = items[item];
  const int64_t off = offs[it.inst];
  const Consts c = cs[it.inst];
  resident_run<P, EQ>(c, fin + off, fout + off, S,
                      (int)(offs[it.inst + 1] - off), lane, wave,
                      wave - it.wave0, it.nw, W, T,
                      resident_stage<P>(sm, W, wave), sm);
}

// One lattice of n nodes in one workgroup.
template <int P, int EQ>
__global__ __launch_bounds__(1024) void k_step_resident(Consts c, double* f,
                                                        int n, int64_t T) {
  extern __shared__ double sm[];
  const int W = blockDim.x >> 6;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  resident_run<P, EQ>(c, f, f, n, n, lane, wave, wave, W, W, T,
                      resident_stage<P>(sm, W, wave), sm);
}

// Moments m = M f (eq. M-d1q3q3) of a batch.
__global__ __launch_bounds__(256) void k_batch_moments(
    const Consts* __restrict__ cs, const int64_t* __restrict__ offs,
    int64_t n_inst, const double* __restrict__ f, double* __restrict__ m,
    int64_t S) {
  lbm::batch_nodes(cs, offs, n_inst, [&](const Consts& c, int64_t j) {
    const double f0 = f[j], fp = f[S + j], fm = f[2 * S + j];
    const double g0 = f[3 * S + j], gp = f[4 * S + j], gm = f[5 * S + j];
    const double sf = fp + fm, sg = gp + gm;
    m[j] = lbm::density(c, f0, fp, fm);
    m[S + j] = c.mJ * (fp - fm);
    m[2 * S + j] = c.mz * (g0 + sg);
    m[3 * S + j] = c.me * (sf - 2.0 * f0);
    m[4 * S + j] = c.mpsi * (gp - gm);
    m[5 * S + j] = c.meps * (sg - 2.0 * g0);
  });
}

// Equilibrium populations of a batch.
__global__ __launch_bounds__(256) void k_batch_equilibrium(
    const Consts* __restrict__ cs, const int64_t* __restrict__ offs,
    int64_t n_inst, const double* __restrict__ rho,
    const double* __restrict__ J, const double* __restrict__ zeta,
    double* __restrict__ f, int64_t S) {
  lbm::batch_nodes(cs, offs, n_inst, [&](const Consts& c, int64_t j) {
    double v[6];
    lbm::equilibrium(c, rho[j], J[j], zeta[j], v);
#pragma unroll
    for (int k = 0; k < 6; ++k) f[k * S + j] = v[k];
  });
}

struct DiagAcc {
  double v[8];
};

__host__ __device__ inline void diag_combine(double* a, const double* b) {
  a[0] += b[0];
  a[1] += b[1];
  a[2] += b[2];
  a[3] += b[3];
  a[4] = fmin(a[4], b[4]);
  a[5] = fmin(a[5], b[5]);
  a[6] += b[6];
  a[7] += b[7];
}

// Block partials of the diagnostics, fixed tree order (deterministic).  They
// go straight to pinned host memory, at most 64 KB, and the host combines
// them once the launch has ended: a second launch for that and a copy of its
// eight values took 19 us of the 42 us that 25 steps of n = 30011 and their
// diagnostics took.
__global__ __launch_bounds__(kDiagBlock) void k_diag_partial(
    Consts c, const double* __restrict__ f, int64_t n,
    double* __restrict__ partial) {
  __shared__ double s[kDiagBlock][8];
  double a[8] = {0, 0, 0, 0, INFINITY, INFINITY, 0, 0};
  for (int64_t j = (int64_t)blockIdx.x * kDiagBlock + threadIdx.x; j < n;
       j += (int64_t)gridDim.x * kDiagBlock) {
    const double f0 = f[j], fp = f[n + j], fm = f[2 * n + j];
    const double g0 = f[3 * n + j], gp = f[4 * n + j], gm = f[5 * n + j];
    const double v[6] = {f0, fp, fm, g0, gp, gm};
    double nf = 0;
    for (int k = 0; k < 6; ++k) nf += isfinite(v[k]) ? 0.0 : 1.0;
    const double rho = lbm::density(c, f0, fp, fm);
    const double J = c.mJ * (fp - fm);
    const double zeta = c.mz * (g0 + (gp + gm));
    double u, s_, Y, T;
    lbm::thermo(c, rho, J, zeta, u, s_, Y, T);
    const double p = rho * c.r * T;
    const double b[8] = {rho, J, zeta, p / c.gm1 + 0.5 * J * u,
                         rho, T, nf, (rho > 0.0 && T > 0.0) ? 0.0 : 1.0};
    diag_combine(a, b);
  }
  for (int k = 0; k < 8; ++k) s[threadIdx.x][k] = a[k];
  __syncthreads();
  for (int w = kDiagBlock / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) diag_combine(s[threadIdx.x], s[threadIdx.x + w]);
    __syncthreads();
  }
  if (threadIdx.x < 8) partial[blockIdx.x * 8 + threadIdx.x] = s[0][threadIdx.x];
}

// The combination of the block partials, as combine_diagnostics on the host.
__global__ __launch_bounds__(kDiagBlock) void k_diag_final(
    const double* __restrict__ partial, int nblocks, double* __restrict__ out) {
  __shared__ double s[kDiagBlock][8];
  const int t = threadIdx.x;
  const int rows = nblocks < kDiagBlock ? nblocks : kDiagBlock;
  if (t < rows) {
    for (int k = 0; k < 8; ++k) s[t][k] = partial[8 * t + k];
    for (int b = t + kDiagBlock; b < nblocks; b += kDiagBlock)
      diag_combine(s[t], partial + 8 * b);
  }
  __syncthreads();
  for (int w = kDiagBlock / 2; w > 0; w >>= 1) {
    if (t < w && t + w < rows) diag_combine(s[t], s[t + w]);
    __syncthreads();
  }
  if (t < 8) out[t] = s[0][t];
}

// Per-lattice diagnostics of a batch, one workgroup per lattice, fixed tree
// order; out[8*inst + k] as in lbm_diagnostics.
__global__ __launch_bounds__(kDiagBlock) void k_batch_diag(
    const Consts* __restrict__ cs, const int64_t* __restrict__ offs,
    const double* __restrict__ f, int64_t S, double* __restrict__ out) {
  __shared__ double s[kDiagBlock][8];
  const int inst = blockIdx.x;
  const Consts c = cs[inst];
  double a[8] = {0, 0, 0, 0, INFINITY, INFINITY, 0, 0};
  for (int64_t j = offs[inst] + threadIdx.x; j < offs[inst + 1];
       j += kDiagBlock) {
    const double f0 = f[j], fp = f[S + j], fm = f[2 * S + j];
    const double g0 = f[3 * S + j], gp = f[4 * S + j], gm = f[5 * S + j];
    const double v[6] = {f0, fp, fm, g0, gp, gm};
    double nf = 0;
    for (int k = 0; k < 6; ++k) nf += isfinite(v[k]) ? 0.0 : 1.0;
    const double rho = lbm::density(c, f0, fp, fm);
    const double J = c.mJ * (fp - fm);
    const double zeta = c.mz * (g0 + (gp + gm));
    double u, s_, Y, T;
    lbm::thermo(c, rho, J, zeta, u, s_, Y, T);
    const double p = rho * c.r * T;
    const double b[8] = {rho, J, zeta, p / c.gm1 + 0.5 * J * u,
                         rho, T, nf, (rho > 0.0 && T > 0.0) ? 0.0 : 1.0};
    diag_combine(a, b);
  }
  for (int k = 0; k < 8; ++k) s[threadIdx.x][k] = a[k];
  __syncthreads();
  for (int w = kDiagBlock / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) diag_combine(s[threadIdx.x], s[threadIdx.x + w]);
    __syncthreads();
  }
  if (threadIdx.x < 8) out[8 * inst + threadIdx.x] = s[0][threadIdx.x];
}

// ------------------------------------------------- failure detection ---
//
// LBM_CHECK_FINITE: after a launch, every node the launch wrote is checked
// as lbm_diagnostics counts it: its six populations finite, rho > 0 and
// T > 0 (T from the equation of state).  A failing node gives the key
// (steps << shift) | index, with steps the time steps done when the launch
// ended and index its node (single lattice) or lattice (batch); the record
// keeps the smallest key: each lane's minimum over its nodes, the wavefront's
// minimum by a butterfly, then one 64-bit vector atomic min per wavefront.

__device__ __forceinline__ bool node_fails(const Consts& c,
                                           const double* __restrict__ f,
                                           int64_t S, int64_t j) {
  const double f0 = f[j], fp = f[S + j], fm = f[2 * S + j];
  const double g0 = f[3 * S + j], gp = f[4 * S + j], gm = f[5 * S + j];
  const bool finite = isfinite(f0) && isfinite(fp) && isfinite(fm) &&
                      isfinite(g0) && isfinite(gp) && isfinite(gm);
  const double rho = lbm::density(c, f0, fp, fm);
  const double J = c.mJ * (fp - fm);
  const double zeta = c.mz * (g0 + (gp + gm));
  double u, s_, Y, T;
  lbm::thermo(c, rho, J, zeta, u, s_, Y, T);
  return !(finite && rho > 0.0 && T > 0.0);
}

// Every lane of the wavefront takes part (lanes without a failing node
// bring ~0).
__device__ __forceinline__ void record_min(unsigned long long* rec,
                                           unsigned long long key) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) {
    const unsigned long long o = __shfl_xor(key, m, 64);
    key = o < key ? o : key;
  }
  if ((threadIdx.x & 63) == 0 && key != ~0ull) atomicMin(rec, key);
}

__global__ __launch_bounds__(64) void k_check_reset(unsigned long long* rec) {
  if (threadIdx.x == 0) *rec = ~0ull;
}

// Single lattice: nodes [0, n), key steps_key | j.
__global__ __launch_bounds__(256) void k_check_state(
    Consts c, const double* __restrict__ f, int64_t n,
    unsigned long long steps_key, unsigned long long* rec) {
  unsigned long long key = ~0ull;
  for (int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x; j < n;
       j += (int64_t)gridDim.x * 256)
    if (node_fails(c, f, n, j) && (steps_key | (unsigned long long)j) < key)
      key = steps_key | (unsigned long long)j;
  record_min(rec, key);
}

// Batch: workgroup b checks the nodes tile tiles[b] stored, [t OUT,
// t OUT + OUT) of its lattice, if that lattice asks for it; key
// steps_key | inst.
__global__ __launch_bounds__(256) void k_batch_check(
    const Consts* __restrict__ cs, const int64_t* __restrict__ offs,
    const lbm::TileRef* __restrict__ tiles, const double* __restrict__ f,
    int64_t S, int OUT, unsigned long long steps_key,
    unsigned long long* rec) {
  const lbm::TileRef tr = tiles[blockIdx.x];
  if (!(cs[tr.inst].flags & LBM_CHECK_FINITE)) return;  // uniform
  const Consts c = cs[tr.inst];
  const int64_t off = offs[tr.inst];
  const int64_t n = offs[tr.inst + 1] - off;
  const int64_t lo = (int64_t)tr.t * OUT;
  const int64_t hi = lo + OUT < n ? lo + OUT : n;
  bool bad = false;
  for (int64_t j = lo + threadIdx.x; j < hi; j += 256)
    bad = bad || node_fails(c, f + off, S, j);
  record_min(rec, bad ? steps_key | (unsigned long long)tr.inst : ~0ull);
}

// Checks (LBM_CHECK_FINITE) of the resident lattices, one workgroup per
// item, those whose flags ask for it; key steps_key | inst.
__global__ __launch_bounds__(256) void k_batch_check_lattices(
    const Consts* __restrict__ cs, const int64_t* __restrict__ offs,
    const lbm::ResidentItem* __restrict__ items, const double* __restrict__ f,
    int64_t S, unsigned long long steps_key, unsigned long long* rec) {
  const int inst = items[blockIdx.x].inst;
  if (!(cs[inst].flags & LBM_CHECK_FINITE)) return;  // uniform
  const Consts c = cs[inst];
  const int64_t off = offs[inst];
  const int64_t n = offs[inst + 1] - off;
  bool bad = false;
  for (int64_t j = threadIdx.x; j < n; j += 256) bad = bad || node_fails(c, f + off, S, j);
  record_min(rec, bad ? steps_key | (unsigned long long)inst : ~0ull);
}

// Copy of the nodes [t OUT, t OUT + OUT) of tile b's lattice from src to
// dst, one workgroup per tile: brings back into the caller's state the
// lattices of a launch sequence that ended in the workspace state.
__global__ __launch_bounds__(256) void k_batch_copy_tiles(
    const int64_t* __restrict__ offs, const lbm::TileRef* __restrict__ tiles,
    int OUT, const double* __restrict__ src, double* __restrict__ dst,
    int64_t S) {
  const lbm::TileRef tr = tiles[blockIdx.x];
  const int64_t off = offs[tr.inst];
  const int64_t n = offs[tr.inst + 1] - off;
  const int64_t lo = off + (int64_t)tr.t * OUT;
  const int64_t hi = off + ((int64_t)tr.t * OUT + OUT < n ? (int64_t)tr.t * OUT + OUT : n);
  for (int64_t j = lo + threadIdx.x; j < hi; j += 256)
#pragma unroll
    for (int q = 0; q < 6; ++q) dst[q * S + j] = src[q * S + j];
}

}  // namespace

// ----------------------------------------------------- launch helpers ---

namespace lbm {

static int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

int launch_equilibrium(const Consts& c, const double* rho, const double* J,
                       const double* zeta, double* f, int64_t n,
                       hipStream_t s) {
  hipLaunchKernelGGL(k_equilibrium, dim3((unsigned)cdiv(n, 256)), dim3(256), 0,
                     s, c, rho, J, zeta, f, n);
  return hip_check(hipGetLastError(), "k_equilibrium");
}

template <int B, int EQ>
static void launch_plain_t(const Consts& c, const double* fin, double* fout,
                           double* halo, int64_t n, hipStream_t s) {
  const int64_t blocks = cdiv(n, B);
  const dim3 grid((unsigned)blocks), block(B + 64);
  // non-temporal accesses once the two states (96 B per node) outgrow the
  // 256 MB of on-die cache
  const bool nt = 96 * n > (int64_t(256) << 20);
  if (fin == fout)
    hipLaunchKernelGGL(k_save_halo, dim3((unsigned)cdiv(4 * blocks, 256)),
                       dim3(256), 0, s, fin, halo, n, blocks, B);
  if (fin == fout && nt)
    hipLaunchKernelGGL((k_step_plain<B, EQ, true, true>), grid, block, 0, s, c,
                       fin, fout, halo, n);
  else if (fin == fout)
    hipLaunchKernelGGL((k_step_plain<B, EQ, false, true>), grid, block, 0, s, c,
                       fin, fout, halo, n);
  else if (nt)
    hipLaunchKernelGGL((k_step_plain<B, EQ, true, false>), grid, block, 0, s, c,
                       fin, fout, halo, n);
  else
    hipLaunchKernelGGL((k_step_plain<B, EQ, false, false>), grid, block, 0, s, c,
                       fin, fout, halo, n);
}

// One step from fin to fout, or in place (fin = fout) with `halo` for 24
// doubles per block.
int launch_step_plain(const Consts& c, const double* fin, double* fout,
                      double* halo, int64_t n, hipStream_t s) {
  if (n >= kComputeUnits * kPlainBlock) {
    if (c.eq_kind == 0)
      launch_plain_t<kPlainBlock, 0>(c, fin, fout, halo, n, s);
    else
      launch_plain_t<kPlainBlock, -1>(c, fin, fout, halo, n, s);
  } else {
    if (c.eq_kind == 0)
      launch_plain_t<kPlainSmall, 0>(c, fin, fout, halo, n, s);
    else
      launch_plain_t<kPlainSmall, -1>(c, fin, fout, halo, n, s);
  }
  return hip_check(hipGetLastError(), "k_step_plain");
}

template <int P, int WG, int M>
static void launch_tile_t(const Consts& c, const double* fin, double* fout,
                          int64_t n, int K, hipStream_t s) {
  const int64_t ntiles = cdiv(n, tile_nodes(P, WG, M) - 4 * K);
  const dim3 grid((unsigned)ntiles), block(64 * WG);
  if (c.eq_kind == 0)
    hipLaunchKernelGGL((k_step_tile<P, WG, M, 0>), grid, block, 0, s, c, fin, fout,
                       n, K, ntiles);
  else if (c.eq_kind == 2)
    hipLaunchKernelGGL((k_step_tile<P, WG, M, 2>), grid, block, 0, s, c, fin, fout,
                       n, K, ntiles);
  else
    hipLaunchKernelGGL((k_step_tile<P, WG, M, 1>), grid, block, 0, s, c, fin, fout,
                       n, K, ntiles);
}

// The tile shapes (P, wavefronts, mirror lanes) of tuning records, and the
// wide ones that plan_steps chooses from besides them.
#define LBM_TILE_SHAPES(X)                                                    \
  X(1, 1, 1) X(2, 1, 1) X(2, 2, 1) X(2, 4, 1) X(2, 8, 1) X(4, 1, 1)           \
  X(4, 2, 1) X(4, 4, 1) X(4, 8, 1) X(8, 1, 1) X(8, 2, 1) X(8, 4, 1)           \
  X(8, 8, 1)
#define LBM_WIDE_SHAPES(X)                                                    \
  X(1, 4, 8) X(1, 8, 8) X(1, 12, 8) X(2, 8, 4) X(2, 12, 4) X(4, 4, 2)         \
  X(4, 8, 2) X(4, 12, 2)

int launch_step_tile(const Consts& c, const double* fin, double* fout,
                     int64_t n, const TileShape& t, int K, hipStream_t s) {
  if (K < 1 || 4 * K >= tile_nodes(t.P, t.W, t.M))
    return set_err(LBM_EINVAL, "bad tile geometry K=%d", K);
#define LBM_STEP_CASE(PP, WW, MM)                                             \
  if (t.P == PP && t.W == WW && t.M == MM) {                                  \
    launch_tile_t<PP, WW, MM>(c, fin, fout, n, K, s);                         \
    return hip_check(hipGetLastError(), "k_step_tile");                       \
  }
  LBM_TILE_SHAPES(LBM_STEP_CASE)
  LBM_WIDE_SHAPES(LBM_STEP_CASE)
#undef LBM_STEP_CASE
  return set_err(LBM_EINVAL, "unsupported tile shape P=%d waves=%d mirror=%d",
                 t.P, t.W, t.M);
}

// The workspace behind the states: of diagnostics without pinned memory (8
// final values, 8 per block), then the failure record of LBM_CHECK_FINITE (4
// doubles).
size_t diag_ws_doubles() { return (size_t)kDiagMaxBlocks * 8 + 8 + 4; }
size_t check_record_double() { return (size_t)kDiagMaxBlocks * 8 + 8; }

int launch_check_reset(unsigned long long* rec, hipStream_t s) {
  hipLaunchKernelGGL(k_check_reset, dim3(1), dim3(64), 0, s, rec);
  return hip_check(hipGetLastError(), "k_check_reset");
}

int launch_check_state(const Consts& c, const double* f, int64_t n,
                       int64_t steps, unsigned long long* rec, hipStream_t s) {
  const unsigned long long sk =
      (unsigned long long)std::min<int64_t>(steps, kCheckMaxSteps1) << 36;
  const int nb = (int)std::min<int64_t>(2048, cdiv(n, 256));
  hipLaunchKernelGGL(k_check_state, dim3(nb), dim3(256), 0, s, c, f, n, sk, rec);
  return hip_check(hipGetLastError(), "k_check_state");
}

int launch_batch_check(const Consts* cs, const int64_t* offs,
                       const TileRef* tiles, int64_t ntiles, const double* f,
                       int64_t S, int OUT, int64_t steps,
                       unsigned long long* rec, hipStream_t s) {
  if (ntiles <= 0) return LBM_OK;
  const unsigned long long sk =
      (unsigned long long)std::min<int64_t>(steps, kCheckMaxStepsB) << 31;
  hipLaunchKernelGGL(k_batch_check, dim3((unsigned)ntiles), dim3(256), 0, s, cs,
                     offs, tiles, f, S, OUT, sk, rec);
  return hip_check(hipGetLastError(), "k_batch_check");
}

int launch_batch_copy_tiles(const int64_t* offs, const TileRef* tiles,
                            int64_t ntiles, int OUT, const double* src,
                            double* dst, int64_t S, hipStream_t s) {
  if (ntiles <= 0) return LBM_OK;
  hipLaunchKernelGGL(k_batch_copy_tiles, dim3((unsigned)ntiles), dim3(256), 0, s,
                     offs, tiles, OUT, src, dst, S);
  return hip_check(hipGetLastError(), "k_batch_copy_tiles");
}

int launch_batch_resident(const Consts* cs, const int64_t* offs,
                          const ResidentItem* items, const int32_t* wg_first,
                          int64_t nwg, const double* fin, double* fout,
                          int64_t S, int64_t T, int P, int W, int eq,
                          hipStream_t s) {
  if (nwg <= 0 || T <= 0) return LBM_OK;
  if (eq != 0)
    return set_err(LBM_EINVAL, "resident lattices need the section-8 equilibria");
  if (W < 1 || W > resident_max_waves(P) || (P == kResP && W != kResWaves))
    return set_err(LBM_EINVAL, "bad resident workgroup of %d wavefronts", W);
  const dim3 grid((unsigned)nwg), block(64 * W);
  if (P == 1)
    hipLaunchKernelGGL((k_batch_resident_small<1, 0>), grid, block,
                       resident_lds(1, W), s, cs, offs, items, wg_first, fin,
                       fout, S, T);
  else if (P == 2)
    hipLaunchKernelGGL((k_batch_resident_small<2, 0>), grid, block,
                       resident_lds(2, W), s, cs, offs, items, wg_first, fin,
                       fout, S, T);
  else if (P == 4)
    hipLaunchKernelGGL((k_batch_resident_small<4, 0>), grid, block,
                       resident_lds(4, W), s, cs, offs, items, wg_first, fin,
                       fout, S, T);
  else if (P == kResP)
    hipLaunchKernelGGL((k_batch_resident<kResP, 0>), grid, block, 0, s, cs, offs,
                       items, wg_first, fin, fout, S, T);
  else
    return set_err(LBM_EINVAL, "unsupported resident shape P=%d", P);
  return hip_check(hipGetLastError(), "k_batch_resident");
}

int launch_step_resident(const Consts& c, double* f, int64_t n, int64_t T,
                         int P, hipStream_t s) {
  const int64_t W = cdiv(n, resident_span(P));
  if ((P != 1 && P != 2 && P != 4) || n < kResidentMin || W > resident_max_waves(P))
    return set_err(LBM_EINVAL, "bad resident lattice of %lld nodes at P=%d",
                   (long long)n, P);
  const dim3 grid(1), block((unsigned)(64 * W));
#define LBM_RES_CASE(PP)                                                      \
  if (P == PP && c.eq_kind == 0)                                              \
    hipLaunchKernelGGL((k_step_resident<PP, 0>), grid, block,                 \
                       resident_lds(PP, (int)W), s, c, f, (int)n, T);         \
  else if (P == PP && c.eq_kind == 2)                                         \
    hipLaunchKernelGGL((k_step_resident<PP, 2>), grid, block,                 \
                       resident_lds(PP, (int)W), s, c, f, (int)n, T);         \
  else if (P == PP)                                                           \
    hipLaunchKernelGGL((k_step_resident<PP, 1>), grid, block,                 \
                       resident_lds(PP, (int)W), s, c, f, (int)n, T);
  LBM_RES_CASE(1)
  LBM_RES_CASE(2)
  LBM_RES_CASE(4)
#undef LBM_RES_CASE
  return hip_check(hipGetLastError(), "k_step_resident");
}

int launch_batch_check_lattices(const Consts* cs, const int64_t* offs,
                                const ResidentItem* items, int64_t nitems,
                                const double* f, int64_t S, int64_t steps,
                                unsigned long long* rec, hipStream_t s) {
  if (nitems <= 0) return LBM_OK;
  const unsigned long long sk =
      (unsigned long long)std::min<int64_t>(steps, kCheckMaxStepsB) << 31;
  hipLaunchKernelGGL(k_batch_check_lattices, dim3((unsigned)nitems), dim3(256), 0,
                     s, cs, offs, items, f, S, sk, rec);
  return hip_check(hipGetLastError(), "k_batch_check_lattices");
}

int read_check_record(const unsigned long long* rec, hipStream_t s,
                      unsigned long long* out) {
  int rc = hip_check(hipMemcpyAsync(out, rec, sizeof *out, hipMemcpyDeviceToHost, s),
                     "hipMemcpyAsync");
  if (!rc) rc = hip_check(hipStreamSynchronize(s), "hipStreamSynchronize");
  return rc;
}

static int diag_blocks(int64_t n) {
  return (int)std::min<int64_t>(kDiagMaxBlocks, cdiv(n, kDiagBlock));
}

size_t diag_sums_bytes() { return sizeof(double) * 8 * kDiagMaxBlocks; }

int launch_diagnostics(const Consts& c, const double* f, int64_t n,
                       double* sums, hipStream_t s) {
  hipLaunchKernelGGL(k_diag_partial, dim3(diag_blocks(n)), dim3(kDiagBlock), 0,
                     s, c, f, n, sums);
  return hip_check(hipGetLastError(), "k_diag_partial");
}

int launch_combine(const double* sums, int64_t n, double* out, hipStream_t s) {
  hipLaunchKernelGGL(k_diag_final, dim3(1), dim3(kDiagBlock), 0, s, sums,
                     diag_blocks(n), out);
  return hip_check(hipGetLastError(), "k_diag_final");
}

// In the order of k_diag_final, so that the result depends on n alone.
void combine_diagnostics(const double* sums, int64_t n, double out[8]) {
  const int nb = diag_blocks(n), rows = std::min(nb, kDiagBlock);
  double s[kDiagBlock][8];
  for (int t = 0; t < rows; ++t) {
    for (int k = 0; k < 8; ++k) s[t][k] = sums[8 * t + k];
    for (int b = t + kDiagBlock; b < nb; b += kDiagBlock)
      diag_combine(s[t], sums + 8 * b);
  }
  for (int w = kDiagBlock / 2; w > 0; w >>= 1)
    for (int t = 0; t < w && t + w < rows; ++t) diag_combine(s[t], s[t + w]);
  for (int k = 0; k < 8; ++k) out[k] = s[0][k];
}

int launch_moments(const Consts& c, const double* f, double* m, int64_t n,
                   hipStream_t s) {
  hipLaunchKernelGGL(k_moments, dim3((unsigned)cdiv(n, 256)), dim3(256), 0, s,
                     c, f, m, n);
  return hip_check(hipGetLastError(), "k_moments");
}

// SEGMENTS: the shape also stores checkpoint segments (state_stride > 0)
template <int P, int WG, int M, bool SEGMENTS>
static void launch_batch_t(const Consts* cs, const int64_t* offs,
                           const TileRef* tiles, int64_t ntiles,
                           const double* fin, double* fout, int64_t S, int H,
                           int K, int64_t state_stride, int first, int every,
                           int eq, hipStream_t s) {
  const dim3 grid((unsigned)ntiles), block(64 * WG);
  if constexpr (SEGMENTS) {
    if (state_stride != 0) {
      if (eq == 0)
        hipLaunchKernelGGL((k_batch_tile<P, WG, M, 0, true>), grid, block, 0, s,
                           cs, offs, tiles, fin, fout, S, H, K, ntiles,
                           state_stride, first, every);
      else
        hipLaunchKernelGGL((k_batch_tile<P, WG, M, -1, true>), grid, block, 0, s,
                           cs, offs, tiles, fin, fout, S, H, K, ntiles,
                           state_stride, first, every);
      return;
    }
  }
#define LBM_EQ_LAUNCH(EE)                                                     \
  hipLaunchKernelGGL((k_batch_tile<P, WG, M, EE, false>), grid, block, 0, s,  \
                     cs, offs, tiles, fin, fout, S, H, K, ntiles,             \
                     state_stride, first, every)
  if (eq == 0)
    LBM_EQ_LAUNCH(0);
  else if (eq == 1)
    LBM_EQ_LAUNCH(1);
  else if (eq == 2)
    LBM_EQ_LAUNCH(2);
  else
    LBM_EQ_LAUNCH(-1);
#undef LBM_EQ_LAUNCH
}

int launch_batch_tile(const Consts* cs, const int64_t* offs,
                      const TileRef* tiles, int64_t ntiles, const double* fin,
                      double* fout, int64_t S, const TileShape& t, int H, int K,
                      int eq, hipStream_t s, int64_t state_stride, int first,
                      int every) {
  if (ntiles <= 0) return LBM_OK;
  if (K < 1 || 2 * K > H || 2 * H >= tile_nodes(t.P, t.W, t.M))
    return set_err(LBM_EINVAL, "bad batched tile geometry H=%d K=%d", H, K);
  if (first < 0 || every < 1)
    return set_err(LBM_EINVAL, "bad segment state numbering");
#define LBM_BATCH_CASE(PP, WW, MM)                                            \
  if (t.P == PP && t.W == WW && t.M == MM) {                                  \
    launch_batch_t<PP, WW, MM, true>(cs, offs, tiles, ntiles, fin, fout, S, H, \
                                     K, state_stride, first, every, eq, s);   \
    return hip_check(hipGetLastError(), "k_batch_tile");                      \
  }
  LBM_TILE_SHAPES(LBM_BATCH_CASE)
#undef LBM_BATCH_CASE
  // of the wide shapes, only those of the recompute store segments
#define LBM_BATCH_CASE(PP, WW, MM)                                            \
  if (t.P == PP && t.W == WW && t.M == MM &&                                  \
      (state_stride == 0 || (PP <= 2 && WW <= 8))) {                          \
    launch_batch_t<PP, WW, MM, (PP <= 2 && WW <= 8)>(                         \
        cs, offs, tiles, ntiles, fin, fout, S, H, K, state_stride, first,     \
        every, eq, s);                                                        \
    return hip_check(hipGetLastError(), "k_batch_tile");                      \
  }
  LBM_WIDE_SHAPES(LBM_BATCH_CASE)
#undef LBM_BATCH_CASE
  // the recompute of k_sweep_tile's shape of two nodes per lane
  if (t.P == 2 && t.W == 4 && t.M == 4 && state_stride != 0) {
    const dim3 grid((unsigned)ntiles), block(256);
    if (eq == 0)
      hipLaunchKernelGGL((k_batch_tile<2, 4, 4, 0, true>), grid, block, 0, s, cs,
                         offs, tiles, fin, fout, S, H, K, ntiles, state_stride,
                         first, every);
    else
      hipLaunchKernelGGL((k_batch_tile<2, 4, 4, -1, true>), grid, block, 0, s, cs,
                         offs, tiles, fin, fout, S, H, K, ntiles, state_stride,
                         first, every);
    return hip_check(hipGetLastError(), "k_batch_tile");
  }
  return set_err(LBM_EINVAL, "unsupported tile shape P=%d waves=%d mirror=%d",
                 t.P, t.W, t.M);
}

int launch_batch_equilibrium(const Consts* cs, const int64_t* offs,
                             int64_t n_inst, const double* rho, const double* J,
                             const double* zeta, double* f, int64_t S,
                             hipStream_t s) {
  hipLaunchKernelGGL(k_batch_equilibrium, dim3((unsigned)cdiv(S, kNodeBlock)),
                     dim3(256), 0, s, cs, offs, n_inst, rho, J, zeta, f, S);
  return hip_check(hipGetLastError(), "k_batch_equilibrium");
}

int launch_batch_moments(const Consts* cs, const int64_t* offs, int64_t n_inst,
                         const double* f, double* m, int64_t S, hipStream_t s) {
  hipLaunchKernelGGL(k_batch_moments, dim3((unsigned)cdiv(S, kNodeBlock)),
                     dim3(256), 0, s, cs, offs, n_inst, f, m, S);
  return hip_check(hipGetLastError(), "k_batch_moments");
}

int launch_batch_diag(const Consts* cs, const int64_t* offs, int64_t n_inst,
                      const double* f, int64_t S, double* out, hipStream_t s) {
  hipLaunchKernelGGL(k_batch_diag, dim3((unsigned)n_inst), dim3(kDiagBlock), 0,
                     s, cs, offs, f, S, out);
  return hip_check(hipGetLastError(), "k_batch_diag");
}

}  // namespace lbm
