// Register tiles, shared by the forward and reverse tile kernels: coalesced
// loads and stores of a wavefront's segment, the time step of its nodes, the
// wavefronts a tile needs, and a whole tile's steps (tile_run).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "lbm_device.hpp"

namespace {

// Global memory is always touched coalesced.  With one or two nodes per lane a
// lane loads and stores its own nodes (two as one 16-byte access: a state's
// arrays are 8-byte aligned, which such accesses allow).  With more, node i of
// a wavefront's segment travels through that wavefront's LDS buffer between
// the coalesced order (lane l handles i = k*64 + l) and the register order
// (lane l owns i = l*P + k); the LDS index i + i/P pads one double per lane
// row so that both orders are free of bank conflicts.  Staging is private to
// a wavefront (wave_barrier only).
constexpr bool staged(int P) { return P > 2; }

typedef double pair_t __attribute__((ext_vector_type(2), aligned(8)));

template <int P>
__device__ __forceinline__ int lds_idx(int i) {
  return i + i / P;
}

// Node of the segment that access k of a lane touches.
template <int P>
__device__ __forceinline__ int seg_idx(int lane, int k) {
  return staged(P) ? k * 64 + lane : lane * P + k;
}

// Node x of a tile in a lattice of n nodes.  small (the lattice is shorter
// than the tile): x and n fit 32 bits.
__device__ __forceinline__ int64_t wrap_near(int64_t x, int64_t n, bool small) {
  if (small) {
    const int r = (int)x % (int)n;
    return r < 0 ? r + (int)n : r;
  }
  return x < 0 ? x + n : (x >= n ? x - n : x);
}

// Where a wavefront's segment lies in its lattice: from node `start` on where
// the whole tile is inside (uniform), else the wrapped index of each access.
template <int P>
struct Segment {
  bool inside;
  int64_t start;
  int64_t gi[P];
};

template <int P>
__device__ __forceinline__ Segment<P> make_segment(int64_t n, int64_t start,
                                                   bool inside, bool small,
                                                   int lane) {
  Segment<P> sg{inside, start, {}};
  if (!inside) {
#pragma unroll
    for (int k = 0; k < P; ++k)
      sg.gi[k] = wrap_near(start + seg_idx<P>(lane, k), n, small);
  }
  return sg;
}

// The segment's loads (arrays of a lattice at fin + q*S, S the array stride of
// the state) into registers in the order of the accesses, to be followed by
// tile_transpose; they may be issued a step ahead of it.
template <int P>
__device__ __forceinline__ void tile_fetch(const double* __restrict__ fin,
                                           int64_t S, const Segment<P>& sg,
                                           int lane, double (&raw)[6][P]) {
  if (sg.inside) {  // one scalar base per array
#pragma unroll
    for (int q = 0; q < 6; ++q) {
      const double* src = fin + ((int64_t)q * S + sg.start);
      if constexpr (P == 2) {
        const pair_t v = *reinterpret_cast<const pair_t*>(src + 2 * lane);
        raw[q][0] = v.x;
        raw[q][1] = v.y;
      } else {
#pragma unroll
        for (int k = 0; k < P; ++k) raw[q][k] = src[seg_idx<P>(lane, k)];
      }
    }
  } else {
#pragma unroll
    for (int q = 0; q < 6; ++q)
#pragma unroll
      for (int k = 0; k < P; ++k) raw[q][k] = fin[(int64_t)q * S + sg.gi[k]];
  }
}

// The pass through LDS into the register order (raw and f may be one array).
template <int P>
__device__ __forceinline__ void tile_transpose(int lane, double* lds,
                                               const double (&raw)[6][P],
                                               double (&f)[6][P]) {
#pragma unroll
  for (int q = 0; q < 6; ++q) {
    if constexpr (!staged(P)) {
#pragma unroll
      for (int k = 0; k < P; ++k) f[q][k] = raw[q][k];
      continue;
    }
#pragma unroll
    for (int k = 0; k < P; ++k) lds[lds_idx<P>(k * 64 + lane)] = raw[q][k];
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int k = 0; k < P; ++k) f[q][k] = lds[lds_idx<P>(lane * P + k)];
    __builtin_amdgcn_wave_barrier();
  }
}

// A segment's load.  All global loads are issued
// before the first pass through LDS, so a wavefront waits for memory once:
// array by array it waited six times in a row, which was most of a launch's
// fixed cost (at n = 8192, one-wavefront tiles: 4.1 -> 2.4 us per launch at
// P = 1, 14 -> 5 us at P = 8; 2000 steps of it 1146 -> 918 us).
template <int P>
__device__ __forceinline__ void tile_load(const double* __restrict__ fin,
                                          int64_t S, int64_t n, int64_t start,
                                          bool inside, bool small, int lane,
                                          double* lds, double (&f)[6][P]) {
  const Segment<P> sg = make_segment<P>(n, start, inside, small, lane);
  tile_fetch<P>(fin, S, sg, lane, f);
  tile_transpose<P>(lane, lds, f, f);
}

// Stores the nodes of this wavefront's segment whose tile index lies in
// [lo, hi) and whose global index is below n.
template <int P>
__device__ __forceinline__ void tile_store(double* __restrict__ fout,
                                           int64_t S, int64_t n, int64_t start,
                                           int lo, int hi, int lane, double* lds,
                                           const double (&f)[6][P]) {
  // one 64-bit lane base and a wavefront-uniform upper bound keep few
  // values live around a kernel's step loop
  const int64_t g0 = start + (staged(P) ? lane : lane * P);
  const int64_t lim = n - start;  // i < lim  <=>  start + i < n
  const int top = lim < hi ? (int)lim : hi;
#pragma unroll
  for (int q = 0; q < 6; ++q) {
    double* dst = fout + (int64_t)q * S + g0;
    if constexpr (P == 1) {
      if (lane >= lo && lane < top) dst[0] = f[q][0];
      continue;
    }
    if constexpr (P == 2) {
      const int i = 2 * lane;
      if (i >= lo && i + 1 < top) {
        pair_t v;
        v.x = f[q][0];
        v.y = f[q][1];
        *reinterpret_cast<pair_t*>(dst) = v;
      } else {
        if (i >= lo && i < top) dst[0] = f[q][0];
        if (i + 1 >= lo && i + 1 < top) dst[1] = f[q][1];
      }
      continue;
    }
    if constexpr (staged(P)) {
#pragma unroll
      for (int k = 0; k < P; ++k) lds[lds_idx<P>(lane * P + k)] = f[q][k];
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int k = 0; k < P; ++k) {
        const int i = k * 64 + lane;
        if (i >= lo && i < top) dst[k * 64] = lds[lds_idx<P>(i)];
      }
      __builtin_amdgcn_wave_barrier();
    }
  }
}

// One time step of a wavefront's nodes.  The source of node k needs u, T of
// k-1 and k+1, so the collisions run in the order P-1, 0, 1, ..., P-2 and
// each source is applied as soon as its right neighbour exists; only a window
// of three nodes' (u, T) stays live besides the populations.
// SAVE: also keeps each node's thermodynamic state of the incoming state in
// th[k] (the reverse sweep reuses it for that state's own reverse step).
template <int P, int EQ, bool SAVE = false>
__device__ __forceinline__ void tile_step(const lbm::Consts& c, double (&f)[6][P],
                                          lbm::NodeThermo* th = nullptr) {
  if constexpr (P == 1) {
    // one node per lane: both neighbours are the adjacent lanes
    double u, T, rw, w;
    lbm::collide_local<EQ, SAVE>(c, f[0][0], f[1][0], f[2][0], f[3][0], f[4][0],
                                 f[5][0], u, T, rw, w, th);
    const double ul = lbm::from_left(u), ur = lbm::from_right(u);
    const double Tl = lbm::from_left(T), Tr = lbm::from_right(T);
    lbm::add_source(c, rw, w, ul, ur, Tl, Tr, f[3][0], f[4][0], f[5][0]);
    if constexpr (SAVE) {
      th->du = ur - ul;
      th->dT = Tr - Tl;
    }
    f[1][0] = lbm::from_left(f[1][0]);
    f[4][0] = lbm::from_left(f[4][0]);
    f[2][0] = lbm::from_right(f[2][0]);
    f[5][0] = lbm::from_right(f[5][0]);
    return;
  }
  double uA, TA, rwA, wA;  // node P-1, collided first
  lbm::collide_local<EQ, SAVE>(c, f[0][P - 1], f[1][P - 1], f[2][P - 1],
                               f[3][P - 1], f[4][P - 1], f[5][P - 1], uA, TA,
                               rwA, wA, SAVE ? th + (P - 1) : nullptr);
  double um, Tm, rwm, wm;  // node k (the one whose source is next)
  __builtin_amdgcn_sched_barrier(0);
  lbm::collide_local<EQ, SAVE>(c, f[0][0], f[1][0], f[2][0], f[3][0], f[4][0],
                               f[5][0], um, Tm, rwm, wm, th);
  double ul = lbm::from_left(uA), Tl = lbm::from_left(TA);
  const double uR = lbm::from_right(um), TR = lbm::from_right(Tm);
#pragma unroll
  for (int k = 0; k < P; ++k) {
    double ur, Tr, rwr = 0.0, wr = 0.0;
    // Keep the scheduler from interleaving the collisions of different
    // nodes: that would hold several nodes' temporaries live at once.
    __builtin_amdgcn_sched_barrier(0);
    if (k + 1 < P - 1) {
      lbm::collide_local<EQ, SAVE>(c, f[0][k + 1], f[1][k + 1], f[2][k + 1],
                                   f[3][k + 1], f[4][k + 1], f[5][k + 1], ur, Tr,
                                   rwr, wr, SAVE ? th + (k + 1) : nullptr);
    } else if (k + 1 == P - 1) {
      ur = uA;
      Tr = TA;
      rwr = rwA;
      wr = wA;
    } else {
      ur = uR;
      Tr = TR;
    }
    lbm::add_source(c, rwm, wm, ul, ur, Tl, Tr, f[3][k], f[4][k], f[5][k]);
    if constexpr (SAVE) {
      th[k].du = ur - ul;
      th[k].dT = Tr - Tl;
    }
    ul = um;
    Tl = Tm;
    um = ur;
    Tm = Tr;
    rwm = rwr;
    wm = wr;
  }
  // (viii) streaming: + populations move one node right, - one node left.
  const double fpL = lbm::from_left(f[1][P - 1]);
  const double gpL = lbm::from_left(f[4][P - 1]);
  const double fmR = lbm::from_right(f[2][0]);
  const double gmR = lbm::from_right(f[5][0]);
#pragma unroll
  for (int k = P - 1; k > 0; --k) {
    f[1][k] = f[1][k - 1];
    f[4][k] = f[4][k - 1];
  }
  f[1][0] = fpL;
  f[4][0] = gpL;
#pragma unroll
  for (int k = 0; k < P - 1; ++k) {
    f[2][k] = f[2][k + 1];
    f[5][k] = f[5][k + 1];
  }
  f[2][P - 1] = fmR;
  f[5][P - 1] = gmR;
}

// Active wavefronts of a tile that starts at lattice index `start` (halo H)
// in a lattice of n nodes: the fewest of the WG whose span
// P((64 - 2M) nw + 2M) still covers the nodes the tile stores plus both halos.
// Only a lattice's last tile, or a lattice shorter than one tile, needs fewer
// than WG.
template <int P, int WG, int M>
__device__ __forceinline__ int active_waves(int64_t n, int64_t start, int H) {
  constexpr int WS = (64 - 2 * M) * P;
  const int64_t store = n - (start + H);  // nodes from the tile's first output
  const int64_t need = store + 2 * H - 2 * M * P;  // beyond the mirror lanes
  if (need >= (int64_t)WS * WG) return WG;
  const int nw = ((int)need + WS - 1) / WS;
  return nw < 1 ? 1 : nw;
}

// K time steps of one register-resident tile per workgroup.  The workgroup has
// WG wavefronts of 64 lanes, lane l of wavefront
// w holding the P consecutive nodes starting at tile index
// P ((64 - 2M) w + l).  Neighbouring wavefronts overlap by 2M lanes: the first
// M lanes of wavefront w > 0 mirror lanes 64-2M .. 63-M of w-1, the last M
// lanes of w < WG-1 mirror lanes M .. 2M-1 of w+1.  A tile thus spans
// tile_nodes = P((64 - 2M) WG + 2M) nodes; tile t stores nodes
// [t*OUT, t*OUT + OUT) with OUT = tile_nodes - 4K and loads
// [t*OUT - 2K, t*OUT + OUT + 2K) (periodic).
//
// Every step runs within the wavefront (lane neighbours through DPP).  The
// outermost lanes have no neighbour there; as one step has radius 2, the
// error this leaves at the mirror lanes' outer end moves two nodes inwards per
// step and reaches the wavefront's own lanes after MP/2 steps.  So every MP/2
// steps the wavefronts copy their edge lanes into the neighbours' mirror
// lanes through LDS (one workgroup barrier per copy, double-buffered); each
// wavefront stores only its own lanes.  The error at the tile's two outer
// ends is what the halo of 2K nodes absorbs.  A copy costs about 0.3 us of
// latency.  With M = 1 a P = 2 tile pays it at every step (n = 8192, 4
// wavefronts, K = 40: 0.80 us per step, 0.54 with M = 4), so the wide shapes
// of plan_steps take 8/P mirror lanes: a copy every four steps at every P.
// One node per lane needs them to have several wavefronts at all.
//
// Refresh of the mirror lanes: the M lanes next to them on each side publish
// their populations in `edge` (one buffer of the double-buffered pair: a
// buffer is written again only after the next refresh's barrier, which every
// reader of its previous contents has passed), then the mirror lanes take
// those of the neighbouring wavefronts.
template <int P, int WG, int M>
__device__ __forceinline__ void mirror_refresh(double (&f)[6][P],
                                               double (*edge)[2][6 * P * M],
                                               int lane, int wave, int nw) {
  const bool hi = lane >= 32;  // the right half of the wavefront
  const int pub = hi ? lane - (64 - 2 * M) : lane - M;
  if (pub >= 0 && pub < M) {
    double* d = edge[wave][hi] + pub;
#pragma unroll
    for (int q = 0; q < 6; ++q)
#pragma unroll
      for (int k = 0; k < P; ++k) d[(q * P + k) * M] = f[q][k];
  }
  __syncthreads();
  const bool left = lane < M && wave > 0, right = lane >= 64 - M && wave < nw - 1;
  if (left || right) {
    const double* e = left ? edge[wave - 1][1] + lane
                           : edge[wave + 1][0] + (lane - (64 - M));
#pragma unroll
    for (int q = 0; q < 6; ++q)
#pragma unroll
      for (int k = 0; k < P; ++k) f[q][k] = e[(q * P + k) * M];
  }
}

// Tile t of a lattice of n nodes (array stride S) starting at lattice index
// `start` = t*OUT - H, OUT = tile_nodes - 2H: load, K <= H/2 steps, store of
// the interior [H, span - H) (one step has radius 2, so K steps need
// H >= 2K).  Only the first nw wavefronts work (active_waves); the
// others end at once, which a workgroup barrier allows (it waits for the
// wavefronts that have not ended), and leave their SIMDs to other
// workgroups.  With every_step (the recompute of a checkpoint segment for a
// reverse sweep), the state after step s = 1..K is state i = first + s of
// the segment, and the interior of those states whose i is a multiple of
// `every` is stored, state i into fout + ((i-1)/every)*state_stride.
template <int P, int WG, int M, int EQ>
__device__ __forceinline__ void tile_run(const lbm::Consts& c,
                                         const double* __restrict__ fin,
                                         double* __restrict__ fout, int64_t S,
                                         int64_t n, int64_t start, int H,
                                         int K, bool every_step = false,
                                         int64_t state_stride = 0,
                                         int first = 0, int every = 1) {
  // mirror lanes must hold at least one step's two wrong nodes
  static_assert(WG == 1 || (M * P >= 2 && 2 * M <= 32), "mirror lanes");
  constexpr int WW = 64 * P;              // nodes of one wavefront
  constexpr int WS = (64 - 2 * M) * P;    // wavefront stride in the tile
  __shared__ double stage[staged(P) ? WG * (WW + 64) : 1];
  __shared__ double edge[2][WG][2][6 * P * M];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nw = active_waves<P, WG, M>(n, start, H);
  if (wave >= nw) return;  // uniform over the wavefront
  const int W = lbm::tile_nodes(P, nw, M);
  double* lds = stage + (staged(P) ? wave * (WW + 64) : 0);
  const int64_t wstart = start + wave * WS;
  const bool inside = start >= 0 && start + W <= n;
  const bool small = n < W;
  double f[6][P];
  tile_load<P>(fin, S, n, wstart, inside, small, lane, lds, f);
  // the tile's valid indices [H, W - H), in this wavefront's numbering and
  // restricted to its own lanes (the mirror lanes belong to the neighbours)
  const int lo = max(H - wave * WS, wave > 0 ? M * P : 0);
  const int hi = min(W - H - wave * WS, wave < nw - 1 ? WW - M * P : WW);
  int since = 0, buf = 0;
  // the next state to store and the steps up to it: counted, since dividing
  // by `every` in each step took longer (n = 8192, P = 1, 34 steps:
  // 18.1 -> 16.5 us)
  int wait = every_step ? every - first % every : 0;
  double* dst = every_step ? fout + (int64_t)(first / every) * state_stride : fout;
  for (int step = 0; step < K; ++step) {
    tile_step<P, EQ>(c, f);
    if (every_step && --wait == 0) {
      tile_store<P>(dst, S, n, wstart, lo, hi, lane, lds, f);
      dst += state_stride;
      wait = every;
    }
    if (WG > 1 && ++since == M * P / 2 && step + 1 < K) {
      mirror_refresh<P, WG, M>(f, edge[buf], lane, wave, nw);
      buf ^= 1;
      since = 0;
    }
  }
  if (!every_step) tile_store<P>(fout, S, n, wstart, lo, hi, lane, lds, f);
}

}  // namespace
