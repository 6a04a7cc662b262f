// Damage update (Sec. 2.2, eq. damage_pde_at2 / eq. damage_pde_at1; Sec. 2.4):
// minimise 1/2 d'Ad - b'd over d_prev <= d <= 1 by a projected CG over the
// assembled rows of A, preconditioned by a Chebyshev-Jacobi polynomial.
//
// The system is scaled by l0/Gc (the minimiser is unchanged), so that its
// entries are of the order of the element areas in either precision; every
// dot product and scalar of the CG is accumulated in FP64.
//
// Method.  CG runs on the free nodes with the held nodes frozen at a bound
// (d_prev or 1), and the held set is updated between CG runs, the bound
// treatment of Sec. 2.4 organised as primal-dual active-set steps.  The held
// set starts from the caller's
// guess (normally the previous step's flags).  After each converged CG run
// a check pass recomputes the true residual r = b - Ax, moves free nodes that
// left [d_prev, 1] onto the bound they crossed, and releases held nodes whose
// scaled residual r_i/A_ii points into the interior by more than tol/4; the
// solve ends when a check changes nothing and the free residual passes.
// (With a release threshold near tol, where the solution's tail varies on the
// scale of tol, each release pushes the next ring of held nodes just over the
// threshold and the held set shrinks one ring per check; well below tol the
// whole tail is released at once.)  A restart pass sees the state a check
// would see and counts the changes that check would make: a restart whose
// free residual passes with none to make ends the solve (a damage field that
// does not move, e.g. AT1 below its threshold, takes one round).
// Each check is one primal-dual active-set update; if eight updates have not
// settled the set, the solve switches to a monotone projected CG: steps are
// cut at the first bound and followed by a projected Jacobi-gradient step of
// length 0.25 (below 2/lambda_max(D^-1 A) for row sums of |A_ij|/A_ii up to
// 8), and held nodes are released only when CG on the current face has
// converged.  Nodes with d_prev = 1 are fixed.  A CG run is also cut short
// for a check when a quarter of its free nodes have left [d_prev, 1] (a far
// wrong held set, e.g. the first AT1 step, would otherwise cost a solve of a
// nearly singular free system).
//
// Iteration.  The CG recurrences are arranged so that one iteration needs a
// single reduction (the Chronopoulos-Gear form): with z = M r (M = D^-1 on
// free nodes, 0 on held ones), w = A z and s = A p,
//     p = z + beta p,  s = w + beta s,  x += alpha p,  r -= alpha s,
//     z = M r,  w = A z,  gamma = r'z,  delta = z'w,
//     beta' = gamma'/gamma,  alpha' = gamma'/(delta' - beta' gamma'/alpha).
// The preconditioner is the Chebyshev-Jacobi polynomial of D^-1 A (degree 1 is
// Jacobi), applied inside the pass: a tile keeps `degree` rings of neighbours,
// applies A once per degree on shrinking sets of rings, and needs nothing from
// other tiles in between.  A round of degree 8 crosses the chip once, as one of
// degree 1 does, and a solve takes about a fifth of the rounds (256x128 plate at
// 1e-12: 60 Jacobi, 22 degree 3, 12 degree 8).
//
// One round of the solve is one or two launches:
//   k_cg_setup the solve's first restart: b, the diagonal and the rows of A that
//              a tile multiplies by (owned nodes and rings; large AT1 plates
//              leave the rings of held tiles out) from the element operator,
//              the start and its true residual;
//   k_cg       one pass of the current phase for every row tile of every
//              instance that is not done:
//                restart / check: x-matvec in FP64, true residual, held-set
//                  update;
//                first: z = M r and w = A z of a new CG run;
//                iterate: the vector updates above, z = M r and w = A z, where
//                  each tile recomputes r on its rings from the previous
//                  vectors;
//              both with per-tile partial sums;
//   k_dmg_red  one workgroup per instance combines its tiles' partials in a
//              fixed order (bitwise reproducible results) and advances the
//              instance's state.
// For instances of few tiles (rows.cpp: combine_in_pass) the combination
// instead runs at the end of the pass, in the instance's last workgroup to
// finish (arrivals counted by integer atomics; same order, same bits), so a
// round is a single launch.
// (r, s), (w, z) and x are ping-pong pairs: a pass reads one half and writes
// the other, so ring reads never race with the owners' writes.  No
// floating-point atomics and no device-wide fences are used.  Linear mode
// (CG_LINEAR) solves A_FF x_F = b_F for a fixed held set and is used by the
// adjoint step.
#include <cstring>

#include "device_common.hpp"

namespace pf {

constexpr int kSwitchAfter = 8;        // active-set updates before the monotone fallback
constexpr double kExpandStep = 0.25;   // projected-gradient step of the fallback
constexpr double kRelease = 0.25;      // held nodes are released when their scaled residual
                                       // points inward by more than kRelease * tol

// held-set states; HELD_FIXED: d_prev = 1, the node cannot move
enum { HELD_NONE = 0, HELD_LOWER = 1, HELD_UPPER = 2, HELD_FIXED = 3 };

// partial sums of one tile, and how each combines (2 bits each: 0 sum, 1 min, 2 max)
enum { PT_DELTA = 0, PT_AMIN = 1, PT_GAMMA = 2, PT_CF = 3, PT_CA = 4, PT_NA = 5, PT_RB = 6, PT_CH = 7 };
constexpr uint32_t kPartOps = (0u << 0) | (1u << 2) | (0u << 4) | (2u << 6) | (2u << 8) | (0u << 10) | (2u << 12) |
                              (0u << 14);

template <typename T>
struct alignas(2 * sizeof(T)) Two {
  T x, y;
};

template <typename T>
struct DmgArgs {
  DevMesh dm;
  DevRows dr;
  const InstP<T>* __restrict__ ip;
  Ctl* ctl;
  const InstFix* __restrict__ fix;
  double* part;
  const T* __restrict__ H;
  const T* __restrict__ lb;      // the caller's lower bound (internal order)
  const uint8_t* __restrict__ guess;
  T* dout;                       // damage solve: output array (read at set-up when start = 1); linear: x
  const T* __restrict__ bin;     // linear: right-hand side (internal order)
  const uint8_t* __restrict__ win;   // linear: held set (internal order)
  // vectors in row order
  double* x0; double* x1;        // iterate pair: FP64 in either mode, so that its rounding does not bound the
                                 // true residual (in FP32 a linear solve's would sit at its tolerance); a
                                 // damage solve's restarts and checks round it to T, the result's type
  Two<T>* rs0; Two<T>* rs1;      // (r, s = A p) pair
  Two<T>* wz0; Two<T>* wz1;      // (w = A z, z) pair
  T* p;                          // search direction (read and written by the owner only)
  T* dim;                        // D^-1, negative on held nodes
  T* rsum;                       // row sums of A
  T* b;
  T* lbr;                        // lower bound
  uint8_t* W0; uint8_t* W1;      // held-set pair (flipped by restart and check passes)
  double tol;
  int32_t max_iter;
  int32_t kind;        // CG_QP or CG_LINEAR
  int32_t start;       // 1: extrapolated start for the damage solve
  int32_t deg;         // polynomial degree asked for (see cg_degree)
  // combination of the round in the pass's last workgroup: 0 none (a
  // k_dmg_red launch follows), 1 combine and advance the solver, 2 combine and
  // run the state machine without storing it (timing aid)
  int32_t fuse;
  uint32_t* arrive;    // arrival counters (see kArriveGroup)
  int32_t nch;         // set-up: the elements' values in LDS together (1) or one after the other (2)
};

// Chebyshev-Jacobi preconditioner z = p(D^-1 A) D^-1 r: `deg` steps of the
// Chebyshev iteration for A y = r from y = 0 with Jacobi scaling on the
// interval [lmax/kChebRatio, lmax] (Saad, Iterative Methods for Sparse Linear
// Systems, Sec. 12.3): with theta, delta the centre and half-width of the
// interval, sigma = theta/delta, rho_0 = 1/sigma,
//   y_1 = D^-1 r / theta,  d_0 = y_1,
//   rho_j = 1/(2 sigma - rho_{j-1}),
//   d_j = rho_j rho_{j-1} d_{j-1} + (2 rho_j/delta) D^-1 (r - A y_j),  y_{j+1} = y_j + d_j.
// Every eigenvalue of D^-1 A lies in (0, lmax] (lmax from pf_mesh_create), where
// the polynomial is positive, so M is symmetric positive definite and CG
// applies unchanged.  The ratio suits the operator's condition number of
// about 30 at l0 = 2h: rounds at 1e-12 for degree 3 with ratios 10, 20, 30 are
// 23, 22, 21 on the 256x128 plate (CPU), for degree 8 with ratios 15, 20, 30, 40
// and 60 14, 13, 12, 12 and 15.
constexpr double kChebRatio = 30.0;

__global__ void k_dmg_init(Ctl* ctl, const InstFix* fix, int n_inst, int kind, int monotone, int ask) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n_inst) return;
  Ctl& c = ctl[k];
  c.mode = MODE_RESTART;
  c.setup = 1;
  c.release = 0;
  c.hit = 0;
  c.iters = 0;
  c.restarts = 0;
  c.flags = 0;
  c.nact = 0;
  c.pbuf = 0;
  c.wbuf = 0;
  c.flavor = (kind == CG_QP && monotone) ? 1 : 0;
  c.outer = 0;
  c.deg = cg_degree(fix[k], ask);
  c.inner = 0;
  c.rz = 0.0;
  c.alpha = 0.0;
  c.beta = 0.0;
  c.amax = 0.0;
  c.resid = 0.0;
  c.pq = 0.0;
  c.ref = (kind == CG_QP) ? 1.0 : 0.0;
}

void chebyshev_steps(InstFix& f, double lmax) {
  const double la = lmax / kChebRatio;
  const double theta = 0.5 * (lmax + la), delta = 0.5 * (lmax - la), sigma = theta / delta;
  f.ith = 1.0 / theta;
  double rp = 1.0 / sigma;
  for (int j = 0; j < kMaxRing - 1; ++j) {
    const double rj = 1.0 / (2.0 * sigma - rp);
    f.ch1[j] = rj * rp;
    f.ch2[j] = 2.0 * rj / delta;
    rp = rj;
  }
}

template <typename T>
__device__ __forceinline__ T clamp01(T v, T lo) {
  return v < lo ? lo : (v > T(1) ? T(1) : v);
}

// Held set, bounds and stopping values of one node at a restart or check: the
// node's new held state, its iterate moved onto a bound it crossed, and the
// pass's counts.
struct NodeCheck {
  double cf = 0.0, ca = -INFINITY, na = 0.0, ch = 0.0;
  __device__ __forceinline__ void stop(uint8_t w, double sr) {
    if (w) {
      if (w != HELD_FIXED) ca = fmax(ca, w == HELD_UPPER ? -sr : sr);
      na += 1.0;
    } else {
      cf = fmax(cf, fabs(sr));
    }
  }
  // what a check pass of this state would change: it would see the same x, held
  // set and residual, so a restart whose free residual passes and which counts
  // nothing here ends the solve itself
  __device__ __forceinline__ void restart_would_change(uint8_t w, double lbv, double xv, double sr, double tol) {
    const bool viol = w == HELD_NONE && (lbv - xv > tol || xv - 1.0 > tol);
    const bool rel = (w == HELD_LOWER && sr > kRelease * tol) || (w == HELD_UPPER && sr < -kRelease * tol);
    ch += (viol || rel) ? 1.0 : 0.0;
  }
};

template <typename T>
__device__ __forceinline__ void arrive_and_advance(const DmgArgs<T>& a, int inst, int tile, int bnd, double* red);

// The value of v in lane j (the same j in every lane of the wave).
__device__ __forceinline__ float lane_value(float v, int j) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), j));
}
__device__ __forceinline__ double lane_value(double v, int j) {
  const long long u = __double_as_longlong(v);
  const uint32_t lo = uint32_t(__builtin_amdgcn_readlane(int(uint32_t(u)), j));
  const uint32_t hi = uint32_t(__builtin_amdgcn_readlane(int(uint32_t(static_cast<unsigned long long>(u) >> 32)), j));
  return __longlong_as_double(static_cast<long long>((static_cast<unsigned long long>(hi) << 32) | lo));
}

template <int N>
struct Int {
  static constexpr int value = N;
};

// Partials of a pass, in PT_* order, stored value-major [8][n_tiles] so the
// reduction reads them coalesced; thread k holds value k.  FUSE: stored
// through to the device-coherent level for the combination in this launch's
// last workgroup.
template <typename T, bool FUSE>
__device__ __forceinline__ void finish_pass(const DmgArgs<T>& a, int inst, double (&v)[8], int tile, int bnd,
                                            double* red, bool cg_only = false) {
  const int n_tiles = a.dr.n_tiles;
  double tot = 0.0;
  uint32_t at = threadIdx.x;   // the value that thread k < 8 stores
  if (cg_only) {
    // the values of an iteration: the others are their operations' identities
    constexpr uint32_t ops = ((kPartOps >> (2 * PT_CF)) & 3u) << 4;   // delta, gamma, cf, ch
    double u[4] = {v[PT_DELTA], v[PT_GAMMA], v[PT_CF], v[PT_CH]};
    tot = block_reduce_waves<4, ops>(u, red);
    const int k = threadIdx.x;
    if (k == 4) tot = INFINITY;
    if (k == 5) tot = -INFINITY;
    constexpr uint32_t slot = PT_DELTA | PT_GAMMA << 4 | PT_CF << 8 | PT_CH << 12 | PT_AMIN << 16 | PT_CA << 20 |
                              PT_NA << 24 | uint32_t(PT_RB) << 28;
    at = (slot >> (4 * (k & 7))) & 15u;
  } else {
    tot = block_reduce_waves<8, kPartOps>(v, red);
  }
  if constexpr (FUSE) {
    if (threadIdx.x < 8)
      __hip_atomic_store(&a.part[size_t(at) * n_tiles + tile], tot, __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
    arrive_and_advance(a, inst, tile, bnd, red);
  } else {
    if (threadIdx.x < 8) a.part[size_t(at) * n_tiles + tile] = tot;
  }
}

// Stiffness part of the rows, sum phi_e K^e_ij over an entry's elements: once
// per handle with phi_e = 1, and in a copy of its own whenever a toughness field
// is set, so that a graph captured with or without one keeps its rows.  The
// element operator's entries are kap phi_e K^e + mA (1 + delta_kl) with K^e given
// by its off-diagonals K01, K02, K12 (its rows sum to zero).
template <typename T>
__global__ __launch_bounds__(kBlock) void k_rows_stiffness(DevMesh dm, DevRows dr) {
  const RowTile* const tp = dr.tiles + blockIdx.x;
  const T* __restrict__ kw = static_cast<const T*>(dm.kw);
  const T* __restrict__ gcs = static_cast<const T*>(dm.gcs);
  auto part = [&](uint32_t cd) {
    if (cd == kNoCode) return 0.0;
    const size_t te = dr.ete[tp->el0 + int(cd & kCodeElem) - 1];
    return (gcs ? double(gcs[te]) : 1.0) * double(kw[size_t(cd >> kCodeEdge) * size_t(dm.n_te) + te]);
  };
  auto entry = [&](uint2 cd) {
    return Two<T>{T(part(cd.x & 0xffffu) + part(cd.x >> 16)), T(part(cd.y & 0xffffu) + part(cd.y >> 16))};
  };
  const size_t base = size_t(tp->slice0) * (kRowPairs * 64);
  for (int i = threadIdx.x; i < tp->nslice * kRowPairs * 64; i += kBlock)
    static_cast<Two<T>*>(dr.sv)[base + i] = entry(dr.code[base + i]);
  const int2 x0 = dr.xs[tp->slice0], x1 = dr.xs[tp->slice0 + tp->nslice - 1];   // the tile's extra pairs are one run
  for (int i = threadIdx.x; i < (x1.x + x1.y - x0.x) * 64; i += kBlock)
    static_cast<Two<T>*>(dr.xsv)[size_t(x0.x) * 64 + i] = entry(dr.xcode[size_t(x0.x) * 64 + i]);
  const T* __restrict__ area = static_cast<const T*>(dm.geo) + 6 * size_t(dm.n_te);
  for (int i = threadIdx.x; i < tp->nel[kMaxRing - 1]; i += kBlock)
    static_cast<T*>(dr.earea)[tp->el0 + i] = area[dr.ete[tp->el0 + i]];
}

void rows_stiffness(pf_dtype_t dtype, const DevMesh& dm, const DevRows& dr, hipStream_t s) {
  if (dtype == PF_F64)
    hipLaunchKernelGGL(k_rows_stiffness<double>, dim3(dr.n_tiles), dim3(kBlock), 0, s, dm, dr);
  else
    hipLaunchKernelGGL(k_rows_stiffness<float>, dim3(dr.n_tiles), dim3(kBlock), 0, s, dm, dr);
}

// The mass coefficient of an element, and a row's entry from its stiffness part
// and the coefficients of the pair's elements.
template <typename T>
__device__ __forceinline__ T elem_mass(const InstP<T>& P, T area, T ph, T He) {
  return (P.c0 * ph + P.cH * He) * area * T(1.0 / 12.0);
}
template <typename T>
__device__ __forceinline__ T row_entry(double kap, T sv, double m0, double m1) {
  return T(kap * double(sv) + (m0 + m1));
}

// DevRows::idle of a tile
enum { TILE_IDLE = 1, TILE_NO_RINGS = 2 };

// The ring rows that the set-up left out, up to row nrow: taken by a tile that
// turns out to own free nodes after all.  A rare path and slow, one row per
// thread and every value from memory; the entries have the set-up's bits.
template <typename T>
__device__ __forceinline__ void late_rings(const DmgArgs<T>& a, const RowTile* tp, const InstP<T>* P, int nrow) {
  const T* const gcs = static_cast<const T*>(a.dm.gcs);
  const T* const area = static_cast<const T*>(a.dr.earea) + tp->el0;
  const double kap = double(P->kap);
  auto mass = [&](uint32_t cd) {
    const int e = int(cd & kCodeElem) - 1;
    if (e < 0) return 0.0;
    return double(elem_mass<T>(*P, area[e], gcs ? gcs[a.dr.ete[tp->el0 + e]] : T(1), a.H[a.dr.egid[tp->el0 + e]]));
  };
  auto entry = [&](Two<T> sv, uint2 cd) {
    return Two<T>{row_entry<T>(kap, sv.x, mass(cd.x), mass(cd.x >> 16)), row_entry<T>(kap, sv.y, mass(cd.y), mass(cd.y >> 16))};
  };
#pragma unroll 1
  for (int i = tp->nl[0] + threadIdx.x; i < nrow; i += kBlock) {
    const int sl = tp->slice0 + i / 64;
    const int2 x = a.dr.xs[sl];
#pragma unroll 1
    for (int q = 0; q < kRowPairs + x.y; ++q) {
      const bool base = q < kRowPairs;
      const size_t at = (base ? size_t(sl) * kRowPairs + q : size_t(x.x) + (q - kRowPairs)) * 64 + i % 64;
      const Two<T>* const sv = static_cast<const Two<T>*>(base ? a.dr.sv : a.dr.xsv);
      Two<T>* const av = static_cast<Two<T>*>(base ? a.dr.av : a.dr.xav);
      av[at] = entry(sv[at], (base ? a.dr.code : a.dr.xcode)[at]);
    }
  }
  __syncthreads();
}

// The first restart of a solve: the rows of this solve, A_ij = kap S_ij + the
// mass coefficients of the pair's elements, the load and the diagonal, and the
// true residual of the start,
//   (A x)_i = sum_j A_ij (x_j - x_i) + x_i sum_e 4 mA_e.
// The mass coefficients and loads of the tile's elements stand in LDS, together
// or (nch = 2) one after the other in half the space; no value depends on that.
// Sums in FP64, rounded once.  Bound by the bytes of the rows (S and the codes
// read, A written: 331 MB in 62 us on the 1024x512 FP64 plate), so on large
// handles (not FUSE) a tile of an AT1 plate whose owned nodes all start held
// leaves its rings out: it will sit out the CG runs (see late_rings).  Standing
// perforated plate, us per windowed step: FP64 331 -> 267, FP32 polled 194 -> 187.
template <typename T, int RPT, int OWN, bool FUSE>
__global__ __launch_bounds__(kBlock) void k_cg_setup(DmgArgs<T> a) {
  __shared__ double red[8 * kWaves];
  const int tile = tile_of_block(a.dr.n_tiles);
  const RowTile* const tp = a.dr.tiles + tile;
  const int n_own = tp->nl[0], nall = tp->nl[1], node0 = tp->node0, halo0 = tp->halo0, slice0 = tp->slice0;
  const int64_t el0 = tp->el0;
  const int inst = tp->inst;
  const Ctl* const c = a.ctl + inst;
  const InstP<T>* const P = a.ip + inst;
  const int bnd = P->bounds;
  const bool qp = (a.kind == CG_QP);
  const bool projected = qp && (bnd == PF_BOUNDS_PROJECTED);
  const bool monotone = projected && (c->flavor != 0);
  const double tol = a.tol;
  const int deg = cg_degree(a.fix[inst], a.deg);
  int nrow = tp->nl[deg - 1], nel = tp->nel[deg - 1];
  const int tid = threadIdx.x;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  extern __shared__ __align__(16) unsigned char smem[];
  T* const ya = reinterpret_cast<T*>(smem);   // [nall] the start
  // the start: d_prev (or its extrapolation in time), or 1 where the guess
  // holds the node at the upper bound; linear solves at the caller's x
  auto held_at = [&](int g, T xv) -> uint8_t {   // the held state that a node starts with
    if (!qp) return a.win[g];
    if (!projected) return HELD_NONE;
    const T lbv = a.lb[g];
    if (lbv >= T(1)) return HELD_FIXED;   // d_prev = 1: the node is fixed
    const uint8_t gs = a.guess ? a.guess[g] : uint8_t(0);
    return ((gs & PF_ACTIVE_LOWER) && xv <= lbv) ? HELD_LOWER
                                                 : (((gs & PF_ACTIVE_UPPER) && xv >= T(1)) ? HELD_UPPER : HELD_NONE);
  };
  // AT1 alone: its threshold holds most nodes of a plate, AT2 holds hardly any,
  // and asking first puts the elements' loads behind the nodes'
  const bool ask = !FUSE && !monotone && P->model == PF_AT1;
  bool rings = false;
  for (int i = tid; i < nall; i += kBlock) {
    const int g = i < n_own ? a.dr.node[node0 + i] : a.dr.hnode[halo0 + i - n_own];
    T v;
    if (!qp) {
      v = a.dout[g];
    } else {
      const T lbv = a.lb[g];
      v = lbv;
      if (a.start) {
        const T e = clamp01<T>(T(2) * lbv - a.dout[g], lbv);
        // FP32: no movement within tol is carried on, as a start that creeps upward
        // by it step after step leaves the tolerance again and again, and d cannot
        // come back down (perforated plate, steps 21-80, windowed: 1 round each in
        // place of 1 to 5, 217 -> 138 us per step).  FP64, the type of gradients,
        // carries every movement on (267 us there, 215 without): where the terms of
        // dL/dGc cancel, the sum is the residual of this start, and another start
        // changes all its digits.
        if (sizeof(T) == 8 || !(double(e) - double(lbv) <= tol)) v = e;   // a NaN goes on to be reported
      }
      if (projected && a.guess && (a.guess[g] & PF_ACTIVE_UPPER)) v = T(1);
    }
    ya[i] = v;
    if (ask && i < n_own) rings = rings || held_at(g, v) == HELD_NONE;
  }
  if constexpr (!FUSE) {
    if (ask) rings = __syncthreads_or(rings);
    const bool left_out = ask && !rings;
    if (tid == 0) a.dr.idle[tile] = left_out ? TILE_NO_RINGS : 0;
    if (left_out) nrow = n_own, nel = tp->nel[0];
  }
  // [1 + nel] mass coefficients (nch = 2: then the loads) of the elements, 0
  // first for entries of fewer than two elements
  T* const sm = ya + nall;
  T* const sb = a.nch == 2 ? sm : sm + 1 + nel;   // [1 + nel] loads
  // per-element toughness factor phi_e (Gc_e = Gc phi_e) scales every Gc
  // term of the element's operator and load; absent, phi_e = 1 exactly
  const T* __restrict__ gcs = static_cast<const T*>(a.dm.gcs);
  const T* __restrict__ area = static_cast<const T*>(a.dr.earea) + el0;
  const int32_t* __restrict__ egid = a.dr.egid + el0;
  const uint32_t* __restrict__ ete = a.dr.ete + el0;
  // f(l, area, phi, H) for the tile's elements l: the loads of kBatch elements
  // per thread go out together, twice (ids and areas, then what the ids index)
  constexpr int kBatch = 6;
  auto elements = [&](auto f) {
    for (int l0 = tid; l0 < nel; l0 += kBatch * kBlock) {
      int32_t ge[kBatch];
      T A[kBatch], He[kBatch], ph[kBatch];
#pragma unroll
      for (int j = 0; j < kBatch; ++j) {
        const int l = min(l0 + j * kBlock, nel - 1);
        ge[j] = egid[l], A[j] = area[l];
        ph[j] = gcs ? gcs[ete[l]] : T(1);
      }
#pragma unroll
      for (int j = 0; j < kBatch; ++j) He[j] = a.H[ge[j]];
#pragma unroll
      for (int j = 0; j < kBatch; ++j)
        if (l0 + j * kBlock < nel) f(l0 + j * kBlock, A[j], ph[j], He[j]);
    }
  };

  const T b0 = P->b0, bH = P->bH;
  elements([&](int l, T A, T ph, T He) {
    sm[1 + l] = elem_mass<T>(*P, A, ph, He);
    if (a.nch != 2) sb[1 + l] = (b0 * ph + bH * He) * A * T(1.0 / 3.0);
  });
  if (tid == 0) sm[0] = sb[0] = T(0);
  __syncthreads();

  const Two<T>* const SV = static_cast<const Two<T>*>(a.dr.sv);
  const Two<T>* const XSV = static_cast<const Two<T>*>(a.dr.xsv);
  Two<T>* const AV = static_cast<Two<T>*>(a.dr.av);
  Two<T>* const XAV = static_cast<Two<T>*>(a.dr.xav);
  const double kap = double(P->kap);
  double qi[RPT], bs[RPT], rs[RPT], off[RPT];
#pragma unroll
  for (int k = 0; k < RPT; ++k) {
    qi[k] = bs[k] = rs[k] = off[k] = 0.0;
    if ((wv + k * kWaves) * 64 >= nrow) continue;
    const int i = tid + k * kBlock;
    const bool own = k < OWN && i < n_own;
    const double xi = own ? double(ya[i]) : 0.0;
    const int sl = slice0 + wv + k * kWaves;
    const int2 x = a.dr.xs[sl];
    // one pair of entries; its first elements are those it stands for
    auto pair = [&](Two<T> sv, uint2 cd, uint32_t cc, Two<T>& out) {
      auto mass = [&](uint32_t e) { return double(sm[e & kCodeElem]); };
      const double m0 = mass(cd.x), m1 = mass(cd.y);
      out.x = row_entry<T>(kap, sv.x, m0, mass(cd.x >> 16));
      out.y = row_entry<T>(kap, sv.y, m1, mass(cd.y >> 16));
      if (!own) return;
      rs[k] += m0;
      rs[k] += m1;
      if (a.nch != 2) {
        bs[k] += double(sb[cd.x & kCodeElem]);
        bs[k] += double(sb[cd.y & kCodeElem]);
      }
      // from here on the entries as the passes read them
      qi[k] += double(out.x) * (double(ya[cc & 0xffffu]) - xi);
      qi[k] += double(out.y) * (double(ya[cc >> 16]) - xi);
      off[k] += double(out.x) + double(out.y);
    };
    const size_t at = size_t(sl) * (kRowPairs * 64) + lane;
    Two<T> sv[kRowPairs];
    uint2 cd[kRowPairs];
    uint32_t cc[kRowPairs];
#pragma unroll
    for (int q = 0; q < kRowPairs; ++q) sv[q] = SV[at + q * 64], cd[q] = i < nrow ? a.dr.code[at + q * 64] : uint2{0, 0}, cc[q] = a.dr.ac[at + q * 64];
#pragma unroll
    for (int q = 0; q < kRowPairs; ++q) {
      Two<T> v;
      pair(sv[q], cd[q], own ? cc[q] : 0u, v);
      AV[at + q * 64] = v;
    }
    for (int e = 0; e < x.y; ++e) {
      const size_t xo = (size_t(x.x) + e) * 64 + lane;
      Two<T> v;
      pair(XSV[xo], i < nrow ? a.dr.xcode[xo] : uint2{0, 0}, own ? a.dr.xac[xo] : 0u, v);
      XAV[xo] = v;
    }
  }
  if (a.nch == 2) {
    __syncthreads();
    elements([&](int l, T A, T ph, T He) { sb[1 + l] = (b0 * ph + bH * He) * A * T(1.0 / 3.0); });
    __syncthreads();
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
      if (k >= OWN || tid + k * kBlock >= n_own) continue;
      const int sl = slice0 + wv + k * kWaves;
      const int2 x = a.dr.xs[sl];
      auto add = [&](uint2 cd) {
        bs[k] += double(sb[cd.x & kCodeElem]);
        bs[k] += double(sb[cd.y & kCodeElem]);
      };
#pragma unroll
      for (int q = 0; q < kRowPairs; ++q) add(a.dr.code[size_t(sl) * (kRowPairs * 64) + q * 64 + lane]);
      for (int e = 0; e < x.y; ++e) add(a.dr.xcode[(size_t(x.x) + e) * 64 + lane]);
    }
  }

  NodeCheck nc;
  double rb = 0.0;   // max |b|/A_ii (linear solves)
#pragma unroll
  for (int k = 0; k < RPT; ++k) {
    const int i = tid + k * kBlock;
    if (k >= OWN || i >= n_own) continue;
    const int q0 = node0 + i;
    const int g = a.dr.node[q0];
    const T xv = ya[i];
    const T rsv = T(4.0 * rs[k]);   // the rows of an element's mass matrix sum to 4 mA
    const T bi = qp ? T(bs[k]) : a.bin[g];   // linear solves read the caller's right-hand side
    const T ri = T(double(bi) - (double(rsv) * double(xv) + qi[k]));
    const T di = T(1.0 / (double(rsv) - off[k]));   // the diagonal from the rows' sums
    const double sr = double(ri) * double(di);
    const uint8_t w = held_at(g, xv);
    if (!qp) {
      if (w == HELD_NONE) rb = fmax(rb, fabs(double(bi) * double(di)));
    } else {
      const T lbv = a.lb[g];
      a.lbr[q0] = lbv;
      if (projected && !monotone && w != HELD_FIXED)
        nc.restart_would_change(w, double(lbv), double(xv), sr, tol);
    }
    a.b[q0] = bi;
    a.rsum[q0] = rsv;
    a.x1[q0] = double(xv);   // the halves that the state machine makes current
    a.rs1[q0].x = ri;
    a.W1[q0] = w;
    a.dim[q0] = w ? -di : di;
    nc.stop(w, sr);
  }
  double v[8] = {0.0, INFINITY, 0.0, nc.cf, nc.ca, nc.na, rb, nc.ch};   // in PT_* order
  finish_pass<T, FUSE>(a, inst, v, tile, bnd, red);
}

// One pass of a solve over the row tiles, after the set-up.  RPT: rows (owned and
// ring nodes) per thread, OWN: of which owned nodes (256 owned nodes per tile:
// 1, which frees the registers and loads of the other rows' iterate, direction
// and bound).  The rows' entries and column ids sit in registers for the whole
// pass (a row is multiplied deg times), the vector being multiplied in LDS;
// PAIRS = 4: the first extra pair of a longer row as well (with random
// diagonals nearly every slice has one, and each product would load it again).
// On large plates the rows' bytes bound it, ring rows included: 158 MB per pass of
// the 1024x512 FP64 plate in 32 us, 0.95 of a copy's rate (FP32 94 MB in 22 us,
// 0.83).  On small ones a workgroup's time is latency: on the 256x128 plate (one
// workgroup per CU) it was 22 thousand clocks, of which the control block and the
// vectors 5.5, nine products 10.6 and the reduction with the arrival 5.4.  So
// whatever the start needs is asked for at once, a thread's rows are summed side
// by side (row_sums), the two halves of the vector in LDS share their addresses,
// and the reduction ends in DPP (block_reduce_waves) on four values where only
// four are new: 18.5 thousand clocks.  Measured, us per step: FP64 64x32 227 ->
// 191, 256x128 246 -> 219, 1024x512 775 -> 733; FP32 397x211 238 -> 209, 16
// plates 584 -> 512.  OWN = 1: FP64 1024x512 764 -> 742; PAIRS = 4: FP32 397x211
// with random diagonals 258 -> 238.
template <typename T, int RPT, int OWN, int PAIRS, bool FUSE>
__global__ __launch_bounds__(kBlock, RPT <= 4 ? (RPT <= 2 ? 4 : 3) : 1) void k_cg(DmgArgs<T> a) {
  __shared__ double red[8 * kWaves];
  const int tile = tile_of_block(a.dr.n_tiles);
  const RowTile* const tp = a.dr.tiles + tile;
  const int n_own = tp->nl[0];
  const int node0 = tp->node0, halo0 = tp->halo0, slice0 = tp->slice0, nslice = tp->nslice, inst = tp->inst;
  const Ctl* const c = a.ctl + inst;
  const InstP<T>* const P = a.ip + inst;
  const int mode = c->mode, flavor = c->flavor, pbuf = c->pbuf, bnd = P->bounds;
  const int ask = cg_degree(a.fix[inst], a.deg), dset = c->deg, idle_tile = a.dr.idle[tile];
  const double beta = c->beta, alpha = c->alpha;
  const int tid = threadIdx.x;
  // where this thread's rows stand: loaded beside the control block
  int pos[RPT];
  const int nring = tp->nl[kMaxRing] - n_own;
#pragma unroll
  for (int k = 0; k < RPT; ++k) {
    const int i = tid + k * kBlock;
    pos[k] = node0 + min(i, n_own - 1);
    if (i >= n_own && nring > 0) pos[k] = a.dr.halo[halo0 + min(i - n_own, nring - 1)];
  }
  // all of these in one round trip with the mode, not one after the other behind its branch
  asm volatile("" ::"s"(flavor), "s"(pbuf), "s"(bnd), "s"(ask), "s"(dset), "s"(idle_tile), "s"(beta), "s"(alpha));
  if (mode == MODE_DONE) return;
  const bool qp = (a.kind == CG_QP);
  const bool projected = qp && (bnd == PF_BOUNDS_PROJECTED);
  const bool monotone = projected && (flavor != 0);
  const bool xpass = (mode == MODE_RESTART || mode == MODE_CHECK);
  const bool iter = (mode == MODE_ITER);
  if (iter && !monotone && (idle_tile & TILE_IDLE)) {
    // no free node here: z, p and the update of x are 0 (see the first pass)
    double v[8] = {0.0, INFINITY, 0.0, 0.0, -INFINITY, 0.0, 0.0, 0.0};
    finish_pass<T, FUSE>(a, inst, v, tile, bnd, red);
    return;
  }
  const bool cur1 = pbuf != 0;
  const T al = T(alpha), be = T(beta);
  const double tol = a.tol;
  // a resumed call may ask for more rings than the set-up assembled rows for
  const int deg = min(ask, dset);
  // current halves (read) and next halves (written) of the pairs
  const double* __restrict__ xc = cur1 ? a.x1 : a.x0;
  double* xn_ = cur1 ? a.x0 : a.x1;
  const Two<T>* rsc = cur1 ? a.rs1 : a.rs0;
  Two<T>* rsn = cur1 ? a.rs0 : a.rs1;
  const Two<T>* wzc = cur1 ? a.wz1 : a.wz0;
  Two<T>* wzn = iter ? (cur1 ? a.wz0 : a.wz1) : (cur1 ? a.wz1 : a.wz0);

  extern __shared__ __align__(16) unsigned char smem[];
  const int nall = tp->nl[xpass ? 1 : deg];   // nodes whose values the pass needs
  T* const ya = reinterpret_cast<T*>(smem);   // the vector the pass multiplies by A, two halves
  // the other half stands at a fixed distance, so that a column's address serves
  // both (degree 1 has one vector, of any length)
  T* const yb = ya + (RPT + 1) * kBlock;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  // the steps of the Chebyshev iteration and the rings' sizes, one per lane:
  // read back lane by lane, so no step waits for memory
  const int sl_ = min(lane, kMaxRing - 2);
  const T steps_c1 = T(a.fix[inst].ch1[sl_]), steps_c2 = T(a.fix[inst].ch2[sl_]);
  const int steps_nl = tp->nl[min(lane, kMaxRing)];

  // ---- the rows of this thread --------------------------------------------------
  Two<T> av[RPT][PAIRS];
  uint32_t ac[RPT][PAIRS];
  int xb[RPT], xk[RPT], longest = 0;   // extra pairs, and the most of this wave's rows
  T rsu[RPT];
  Two<T>* const AV = static_cast<Two<T>*>(a.dr.av);
  Two<T>* const XAV = static_cast<Two<T>*>(a.dr.xav);
  auto load_rows = [&]() {
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
      const int sl = min(wv + k * kWaves, nslice - 1);
      const size_t at = size_t(slice0 + sl) * (kRowPairs * 64) + lane;
      const int2 x = a.dr.xs[slice0 + sl];
      xb[k] = x.x, xk[k] = x.y;
      longest = max(longest, x.y);
#pragma unroll
      for (int q = 0; q < kRowPairs; ++q) {
        ac[k][q] = a.dr.ac[at + q * 64];
        av[k][q] = AV[at + q * 64];
      }
      if constexpr (PAIRS > kRowPairs) {
        // a slice without extra pairs gets entries of 0
        const size_t xo = size_t(xk[k] > 0 ? xb[k] : 0) * 64 + lane;
        const Two<T> v = XAV[xo];
        ac[k][kRowPairs] = xk[k] > 0 ? a.dr.xac[xo] : 0u;
        av[k][kRowPairs] = Two<T>{xk[k] > 0 ? v.x : T(0), xk[k] > 0 ? v.y : T(0)};
      }
      if (k < OWN) rsu[k] = a.rsum[node0 + min(tid + k * kBlock, n_own - 1)];
    }
  };
  // s[k] = sum over row k < N of f(k, entry, value at the column), the rows side
  // by side: their LDS reads go out together and their sums do not wait for
  // each other
  auto row_sums = [&](auto n, const auto* y, auto& s, auto f) {
    constexpr int N = decltype(n)::value;
#pragma unroll
    for (int k = 0; k < N; ++k) s[k] = 0;
    constexpr int G = RPT >= 4 ? 2 : N;   // rows at a time: the registers of four are not there
#pragma unroll
    for (int g = 0; g < N; g += G)
#pragma unroll
      for (int q = 0; q < PAIRS; ++q)
#pragma unroll
        for (int k = g; k < (g + G < N ? g + G : N); ++k) {
          s[k] += f(k, av[k][q].x, y[ac[k][q] & 0xffffu]);
          s[k] += f(k, av[k][q].y, y[ac[k][q] >> 16]);
        }
    if (longest <= PAIRS - kRowPairs) return;
#pragma unroll
    for (int k = 0; k < N; ++k)
      for (int e = PAIRS - kRowPairs; e < xk[k]; ++e) {
        const size_t xo = (size_t(xb[k]) + e) * 64 + lane;
        const Two<T> v = XAV[xo];
        const uint32_t cc = a.dr.xac[xo];
        s[k] += f(k, v.x, y[cc & 0xffffu]);
        s[k] += f(k, v.y, y[cc >> 16]);
      }
  };
  constexpr bool kEarlyRows = RPT <= 2 || (RPT <= 3 && OWN == 1);

  // ---- loads of the node vectors --------------------------------------------------
  T dmv[RPT];
#pragma unroll
  for (int k = 0; k < RPT; ++k) dmv[k] = a.dim[pos[k]];

  double amin = INFINITY, gam = 0.0, del = 0.0;
  NodeCheck nc;
  if (xpass) {
    // ---- restart / check: true residual b - A x in FP64 -------------------------
    double xv_[RPT];
    T rv_[RPT];
#pragma unroll
    for (int k = 0; k < RPT; ++k) xv_[k] = xc[pos[k]], rv_[k] = rsc[pos[k]].x;
    load_rows();
    const bool cut = c->hit != 0, release = c->release != 0;
    const uint8_t* Wc = c->wbuf ? a.W1 : a.W0;
    uint8_t* Wn = c->wbuf ? a.W0 : a.W1;
    double* const xs = reinterpret_cast<double*>(smem);
    auto value = [&](int q, double v, T r, T dm) {
      if (cut && Wc[q] == HELD_NONE) {
        // monotone flavour: the last step cut at the first bound (step amax
        // along p, whose A p is in the other half of its pair), then a
        // projected Jacobi-gradient step
        const double xh = v + c->amax * double(a.p[q]);
        const T rh = r - T(c->amax) * rsn[q].y;
        v = clamp01<double>(xh + double(T(kExpandStep) * fabs(dm) * rh), double(a.lbr[q]));
      }
      // what the damage solve may end on is what it delivers: d is a T
      return qp ? double(T(v)) : v;
    };
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
      const int i = tid + k * kBlock;
      if (i < nall) xs[i] = value(pos[k], xv_[k], rv_[k], dmv[k]);
    }
    for (int i = RPT * kBlock + tid; i < nall; i += kBlock) {
      const int q = a.dr.halo[halo0 + i - n_own];
      xs[i] = value(q, xc[q], rsc[q].x, a.dim[q]);
    }
    __syncthreads();
    double q_[OWN], xo_[OWN];
#pragma unroll
    for (int k = 0; k < OWN; ++k) xo_[k] = xs[min(tid + k * kBlock, n_own - 1)];
    row_sums(Int<OWN>{}, xs, q_, [&](int k, T e, double y) { return double(e) * (y - xo_[k]); });
#pragma unroll
    for (int k = 0; k < OWN; ++k) {
      const int i = tid + k * kBlock;
      if (i >= n_own) continue;
      const int g = node0 + i;
      const double xi = xo_[k];
      double xv = xi;
      const double qi = double(rsu[k]) * xi + q_[k];
      const T ri = T(double(a.b[g]) - qi);
      const T di = fabs(dmv[k]);
      const double sr = double(ri) * double(di);
      const uint8_t wold = Wc[g];
      uint8_t w = wold;   // linear solves keep their held set; without bounds no node is held
      if (projected) {
        const double lbv = double(a.lbr[g]);
        if (w == HELD_FIXED) {
          // d_prev = 1: the node is fixed
        } else if (mode == MODE_CHECK) {
          const bool viol_lo = wold == HELD_NONE && lbv - xv > tol;
          const bool viol_up = wold == HELD_NONE && xv - 1.0 > tol;
          const bool rel = (wold == HELD_LOWER && sr > kRelease * tol) || (wold == HELD_UPPER && sr < -kRelease * tol);
          w = viol_lo ? HELD_LOWER : (viol_up ? HELD_UPPER : (rel ? HELD_NONE : wold));
          if (viol_lo) xv = lbv;
          if (viol_up) xv = 1.0;
          nc.ch += (viol_lo || viol_up || rel) ? 1.0 : 0.0;
        } else if (!monotone) {
          nc.restart_would_change(w, lbv, xv, sr, tol);
        } else {
          const bool want_lo = ri < T(0) || (wold == HELD_LOWER && !(release && sr > kRelease * tol));
          const bool want_up = ri > T(0) || (wold == HELD_UPPER && !(release && sr < -kRelease * tol));
          w = (xv <= lbv && want_lo) ? HELD_LOWER : ((xv >= 1.0 && want_up) ? HELD_UPPER : HELD_NONE);
        }
      }
      xn_[g] = xv;
      rsn[g].x = ri;   // s of this half may still be read by a neighbouring tile's cut
      Wn[g] = w;
      a.dim[g] = w ? -di : di;
      nc.stop(w, sr);
    }
  } else {
    // ---- first / iterate ---------------------------------------------------------
    if (!iter) {
      // A tile whose owned nodes are all held does nothing in this CG run: z
      // and p vanish there, x stays (in both halves of its pair), and r and A p
      // of held nodes are read nowhere (the monotone flavour reads them).  Most
      // tiles of an AT1 plate are such tiles.
      bool free_node = monotone;
#pragma unroll
      for (int k = 0; k < RPT; ++k) free_node = free_node || (k < OWN && tid + k * kBlock < n_own && !(dmv[k] < T(0)));
      const bool idle = !__syncthreads_or(free_node);
      const bool late = !FUSE && (idle_tile & TILE_NO_RINGS) != 0;
      if (tid == 0) a.dr.idle[tile] = idle ? TILE_IDLE | (late ? TILE_NO_RINGS : 0) : 0;
      if constexpr (!FUSE)
        if (late && !idle) late_rings(a, tp, P, tp->nl[dset - 1]);
      if (idle) {
        for (int i = tid; i < n_own; i += kBlock) xn_[node0 + i] = xc[node0 + i];
        double v[8] = {0.0, INFINITY, 0.0, 0.0, -INFINITY, 0.0, 0.0, 0.0};
        finish_pass<T, FUSE>(a, inst, v, tile, bnd, red);
        return;
      }
    }
    const T ith = deg > 1 ? T(a.fix[inst].ith) : T(1);
    T r_[RPT], y_[RPT], d_[RPT];   // residual, Chebyshev iterate and its update of this thread's rows
    Two<T> rsv[RPT], wzv[RPT];
    T pv_[RPT], lbv_[RPT];
    double xv_[RPT];
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
      rsv[k] = rsc[pos[k]];
      if (iter) {
        wzv[k] = wzc[pos[k]];
        if (k >= OWN) continue;
        const int po = node0 + min(tid + k * kBlock, n_own - 1);
        pv_[k] = a.p[po];
        xv_[k] = xc[po];
        lbv_[k] = projected ? a.lbr[po] : T(0);
      }
    }
    if constexpr (kEarlyRows) load_rows();
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
      const int i = tid + k * kBlock;
      const bool held = dmv[k] < T(0);
      T rn = rsv[k].x;
      if (iter) {
        const T sn = (beta == 0.0) ? wzv[k].x : wzv[k].x + be * rsv[k].y;   // s = A p of this iteration
        rn = rn - al * sn;
        if (k < OWN && i < n_own) {
          const int g = node0 + i;
          const T pv = (beta == 0.0) ? wzv[k].y : wzv[k].y + be * pv_[k];
          const double xv = xv_[k], lbd = double(lbv_[k]);
          double xn = xv + double(al) * double(pv);
          if (monotone && !held) {
            // largest step that keeps this node inside [d_prev, 1]
            if (pv < T(0)) amin = fmin(amin, (lbd - xv) / double(pv));
            if (pv > T(0)) amin = fmin(amin, (1.0 - xv) / double(pv));
            xn = clamp01<double>(xn, lbd);
          } else if (projected && !held) {
            if (lbd - xn > tol || xn - 1.0 > tol) nc.ch += 1.0;   // free node outside the bounds
          }
          a.p[g] = pv;
          xn_[g] = xn;
          rsn[g] = Two<T>{rn, sn};
        }
      }
      if (held && monotone && k < OWN && i < n_own) {
        const double sr = double(rn) * double(-dmv[k]);
        const uint8_t w = (c->wbuf ? a.W1 : a.W0)[node0 + i];
        if (w != HELD_FIXED) nc.ca = fmax(nc.ca, w == HELD_UPPER ? -sr : sr);
      }
      // on held nodes z and every Chebyshev iterate are 0
      if (held) dmv[k] = T(0), rn = T(0);
      r_[k] = rn;
      y_[k] = d_[k] = dmv[k] * rn * ith;
      if (i < nall) ya[i] = y_[k];
    }
    for (int i = RPT * kBlock + tid; i < nall; i += kBlock) {   // nodes of the outermost ring without a row here
      const int q = a.dr.halo[halo0 + i - n_own];
      const Two<T> rs = rsc[q];
      const T dm = a.dim[q];
      T rn = rs.x;
      if (iter) {
        const Two<T> wz = wzc[q];
        const T sn = (beta == 0.0) ? wz.x : wz.x + be * rs.y;
        rn = rn - al * sn;
      }
      ya[i] = dm < T(0) ? T(0) : dm * rn * ith;
    }
    if constexpr (!kEarlyRows) load_rows();
    __syncthreads();
    // One step of the Chebyshev iteration from the values in ys to yd, over the
    // rows that the steps still to come read.  A wave takes those of its rows
    // whose slice holds any; what it computes past the last of them is not
    // read (its columns lie in the pass's LDS, see cg_shape).
    auto step = [&](int j, const T* ys, T* yd) {
      const int lim = __builtin_amdgcn_readlane(steps_nl, deg - j);
      const T c1 = lane_value(steps_c1, j - 1), c2 = lane_value(steps_c2, j - 1);
      auto rows = [&](auto n) {
        constexpr int N = decltype(n)::value;
        T s_[N];
        row_sums(n, ys, s_, [](int, T e, T y) { return e * y; });
#pragma unroll
        for (int k = 0; k < N; ++k) {
          // D^-1 (r - A y): the diagonal's part of D^-1 A y is y itself
          d_[k] = c1 * d_[k] + c2 * (dmv[k] * (r_[k] - s_[k]) - y_[k]);
          y_[k] += d_[k];
          yd[tid + k * kBlock] = y_[k];
        }
      };
      const int nk = (lim - wv * 64 + kBlock - 1) / kBlock;   // rows of this wave with a node below lim
      if constexpr (RPT > 4) {
        if (nk > 4) rows(Int<RPT>{});
        else if (nk > 0) rows(Int<4>{});
      } else {
        if (nk >= RPT) rows(Int<RPT>{});
        if constexpr (RPT > 3) { if (nk == 3) rows(Int<3>{}); }
        if constexpr (RPT > 2) { if (nk == 2) rows(Int<2>{}); }
        if constexpr (RPT > 1) { if (nk == 1) rows(Int<1>{}); }
      }
      __syncthreads();
    };
#pragma unroll 1
    for (int j = 1; j < deg; j += 2) {
      step(j, ya, yb);
      if (j + 1 < deg) step(j + 1, yb, ya);
    }
    const T* const ys = (deg & 1) ? ya : yb;
    // w = A z on the owned nodes
    T w_[OWN];
    row_sums(Int<OWN>{}, ys, w_, [&](int k, T e, T y) { return e * (y - y_[k]); });
#pragma unroll
    for (int k = 0; k < OWN; ++k) {
      const int i = tid + k * kBlock;
      if (i >= n_own) continue;
      const T zv = y_[k];
      const T s = rsu[k] * zv + w_[k];
      wzn[node0 + i] = Two<T>{s, zv};
      gam += double(r_[k]) * double(zv);
      del += double(zv) * double(s);
      // a CG run ends when max |r_i|/A_ii and max |z_i| are at most tol: the
      // polynomial leaves smooth residuals, whose error is up to
      // 1/lambda_min(D^-1 A) (about 15) times |r|/A_ii, and z = M r has nearly
      // the error's size (with Jacobi the two are the same)
      nc.cf = fmax(nc.cf, fmax(fabs(double(r_[k]) * double(dmv[k])), fabs(double(zv))));
    }
  }
  double v[8] = {del, amin, gam, nc.cf, nc.ca, nc.na, 0.0, nc.ch};   // in PT_* order
  finish_pass<T, FUSE>(a, inst, v, tile, bnd, red, !xpass && !monotone);
}

// Combination of an instance's per-tile partials, in a fixed order: thread t
// adds the partials of tiles tile0 + t, tile0 + t + block, ... in that order,
// then the block's values are reduced (by wave, then a fixed-order combine);
// thread k < 8 returns value k.  k_dmg_red runs the same order with the loads
// of kRedBatch tiles per thread in flight (it is latency-bound: one
// workgroup, a few kilobytes; tiles past the end combine as the identity of
// each operation through selects, not a branch, so the loads stay ahead of
// every use).  This flavour, for the last workgroup of a pass, reads one
// tile's partials per thread at a time past this die's L2 (the partials of the
// running kernel) and keeps the pass's register count.
constexpr int kRedBatch = 8;
__device__ __forceinline__ double combine_partials(double* part, size_t nt, int tile0, int ntiles, double* red) {
  const int tile_end = tile0 + ntiles;
  double v[8] = {0.0, INFINITY, 0.0, 0.0, -INFINITY, 0.0, 0.0, 0.0};
#pragma unroll 1
  for (int k = tile0 + int(threadIdx.x); k < tile_end; k += kBlock) {
    double q[8];
#pragma unroll
    for (int f = 0; f < 8; ++f) q[f] = __hip_atomic_load(part + size_t(f) * nt + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    v[PT_DELTA] += q[PT_DELTA];
    v[PT_AMIN] = fmin(v[PT_AMIN], q[PT_AMIN]);
    v[PT_GAMMA] += q[PT_GAMMA];
    v[PT_CF] = fmax(v[PT_CF], q[PT_CF]);
    v[PT_CA] = fmax(v[PT_CA], q[PT_CA]);
    v[PT_NA] += q[PT_NA];
    v[PT_RB] = fmax(v[PT_RB], q[PT_RB]);
    v[PT_CH] += q[PT_CH];
  }
  return block_reduce_waves<8, kPartOps>(v, red);
}

// The solver's state machine: one round's combined partials advance the
// instance's control block c (a register copy; the caller stores it).
__device__ __forceinline__ void advance_solver(Ctl* c, int nnodes, const double (&v)[8], int bnd, int kind, double tol,
                                               int max_iter) {
  const int mode = c->mode;
  const double sdel = v[PT_DELTA], samin = v[PT_AMIN], sgam = v[PT_GAMMA], scf = v[PT_CF], sca = v[PT_CA];
  const double sna = v[PT_NA], srb = v[PT_RB], sch = v[PT_CH];
  const bool qp = (kind == CG_QP);
  const bool projected = qp && (bnd == PF_BOUNDS_PROJECTED);
  const bool monotone = projected && (c->flavor != 0);
  const bool setup = c->setup != 0;
  c->iters += 1;
  c->inner = (mode == MODE_ITER) ? c->inner + 1 : 0;
  if (setup && !qp) c->ref = srb;   // linear solves stop relative to max |b_i|/A_ii
  const double tl = tol * c->ref;
  const double rs = c->ref > 0.0 ? c->ref : 1.0;
  if (mode == MODE_RESTART || mode == MODE_CHECK) {
    // the pass wrote x, r and the held set into the other halves of their pairs
    c->pbuf ^= 1;
    c->wbuf ^= 1;
    c->setup = 0;
    c->hit = 0;
    c->nact = int32_t(sna);
    c->resid = (monotone ? fmax(scf, sca) : scf) / rs;
    if (!isfinite(scf)) {
      c->flags |= PF_FLAG_NONFINITE;
      c->mode = MODE_DONE;
    } else if (!qp && c->ref == 0.0) {
      c->mode = MODE_DONE;   // zero right-hand side: the solution is 0 (set by the final kernel)
    } else if (mode == MODE_CHECK) {
      if (sch > 0.0) {
        c->outer += 1;
        c->restarts += 1;
        if (c->outer >= kSwitchAfter) c->flavor = 1;
        c->release = 0;
        c->mode = MODE_RESTART;
      } else if (scf <= tl) {
        c->mode = MODE_DONE;
      } else {
        c->mode = MODE_FIRST;
      }
    } else if (monotone) {
      if (scf <= tl && sca <= kRelease * tl) {
        c->mode = MODE_DONE;
      } else if (scf <= tl) {
        c->mode = MODE_RESTART;   // face converged, held nodes want to leave: release them
        c->release = 1;
        c->restarts += 1;
      } else {
        c->mode = MODE_FIRST;
      }
    } else if (scf <= tl) {
      // a restart counts the changes a check of its state would make
      c->mode = (projected && sch > 0.0) ? MODE_CHECK : MODE_DONE;
    } else {
      c->mode = MODE_FIRST;
    }
  } else if (mode == MODE_FIRST) {
    if (!isfinite(sgam) || !isfinite(sdel)) {
      c->flags |= PF_FLAG_NONFINITE;
      c->mode = MODE_DONE;
    } else if (!(sdel > 0.0)) {
      // z = 0 on every free node: the free residual vanishes
      c->mode = projected && !monotone ? MODE_CHECK : MODE_RESTART;
      c->release = monotone ? 1 : 0;
    } else {
      c->alpha = sgam / sdel;
      c->beta = 0.0;
      c->rz = sgam;
      c->mode = MODE_ITER;
    }
  } else if (monotone && samin < c->alpha) {
    // the step crosses a bound: cut it there and restart (x, r stay in the
    // current halves; p and s = A p of this step are kept for the cut)
    c->amax = fmax(samin, 0.0);
    c->hit = 1;
    c->release = 0;
    c->restarts += 1;
    c->mode = MODE_RESTART;
  } else {
    c->pbuf ^= 1;
    c->resid = scf / rs;
    const double beta = sgam / c->rz;
    const double den = sdel - beta * sgam / c->alpha;
    const bool early = projected && !monotone && c->inner >= 2 && sch > 0.25 * double(nnodes - c->nact);
    if (!isfinite(sgam) || !isfinite(sdel)) {
      c->flags |= PF_FLAG_NONFINITE;
      c->mode = MODE_DONE;
    } else if (scf <= tl || sgam == 0.0 || early || !(den > 0.0)) {
      // this CG run converged on its recurrence residual, a quarter of the
      // free nodes already left their bounds, or the recurrence lost
      // definiteness: recompute the true residual (and update the held set)
      if (projected && !monotone) {
        c->mode = MODE_CHECK;
      } else {
        c->mode = MODE_RESTART;
        c->release = (monotone && sca > kRelease * tl) ? 1 : 0;
        c->restarts += monotone ? 1 : 0;
      }
    } else {
      c->beta = beta;
      c->alpha = sgam / den;
      c->rz = sgam;
    }
  }
  if (c->mode != MODE_DONE && c->iters >= max_iter) {
    c->flags |= PF_FLAG_NOT_CONVERGED;
    c->mode = MODE_DONE;
  }
}

// One workgroup per instance: combine the tiles' partials and advance the
// state (passes run without the combination in their last workgroup).  Bound by
// what one CU can load: the mode is read first, so that an iteration loads four
// values per tile instead of eight, in one batch up to 4096 tiles, and a finished
// solve none (1024x512 FP64 step 743 -> 716 us, FP32 350 -> 338).
constexpr int kRedBlock = kBlock;
__global__ __launch_bounds__(kRedBlock) void k_dmg_red(Ctl* ctl, const InstFix* fix, const double* part, int n_tiles, const int* bounds,
                                                       int kind, double tol, int max_iter) {
  __shared__ double red[8 * (kRedBlock / 64)];
  __shared__ double tot[8];
  Ctl* const cp = ctl + blockIdx.x;
  Ctl cc;
  int bnd = 0, nnodes = 0;
  if (threadIdx.x == 0) {
    cc = *cp;
    bnd = bounds[blockIdx.x];
    nnodes = fix[blockIdx.x].nnodes;
  }
  const int mode = cp->mode, flavor = cp->flavor;
  const int tile0 = fix[blockIdx.x].rt0, tile_end = tile0 + fix[blockIdx.x].nrt;
  if (mode == MODE_DONE) return;
  double v[8] = {0.0, INFINITY, 0.0, 0.0, -INFINITY, 0.0, 0.0, 0.0};
  const size_t nt = size_t(n_tiles);
  // B tiles per thread at a time, of them the values in `set`
  auto add = [&](auto batch, auto set) {
    constexpr int B = decltype(batch)::value;
    constexpr uint32_t S = decltype(set)::value;
#pragma unroll 1
    for (int k0 = tile0 + threadIdx.x; k0 < tile_end; k0 += B * kRedBlock) {
      double q[B][8];
#pragma unroll
      for (int j = 0; j < B; ++j) {
        const int k = min(k0 + j * kRedBlock, tile_end - 1);   // clamped: loaded, not added
#pragma unroll
        for (int f = 0; f < 8; ++f)
          if (S >> f & 1u) q[j][f] = part[size_t(f) * nt + k];
      }
#pragma unroll
      for (int j = 0; j < B; ++j) {
        const bool in = k0 + j * kRedBlock < tile_end;
#pragma unroll
        for (int f = 0; f < 8; ++f) {
          if (!(S >> f & 1u)) continue;
          const uint32_t op = (kPartOps >> (2 * f)) & 3u;
          const double x = in ? q[j][f] : (op == 0 ? 0.0 : (op == 1 ? INFINITY : -INFINITY));
          v[f] = combine_op(op, v[f], x);
        }
      }
    }
  };
  // an iteration's pass stores constants in the other four: half the bytes
  if ((mode == MODE_ITER || mode == MODE_FIRST) && flavor == 0)
    add(Int<2 * kRedBatch>{}, Int<(1 << PT_DELTA | 1 << PT_GAMMA | 1 << PT_CF | 1 << PT_CH)>{});
  else
    add(Int<kRedBatch>{}, Int<255>{});
  const double vk = block_reduce_waves<8, kPartOps, kRedBlock / 64>(v, red);
  if (threadIdx.x < 8) tot[threadIdx.x] = vk;
  __syncthreads();
  if (threadIdx.x != 0) return;
#pragma unroll
  for (int k = 0; k < 8; ++k) v[k] = tot[k];
  advance_solver(&cc, nnodes, v, bnd, kind, tol, max_iter);
  *cp = cc;
}

// The end of a pass that combines in place: each workgroup counts its arrival once its
// partial sums are stored, and the instance's last workgroup to arrive
// combines every tile's partials and advances the solver, so a round is one
// launch.  Nothing waits for anything: a workgroup that is not last exits.
// The partials are stored through to the device-coherent level (the L2s of
// the chip's dies are not coherent with each other) and counted only after
// the stores have completed; the last workgroup reads them past its L2.  The
// fixed combination order is that of k_dmg_red, so the bits are the same.
template <typename T>
__device__ __forceinline__ void arrive_and_advance(const DmgArgs<T>& a, int inst, int tile, int bnd, double* red) {
  const InstFix* const c = a.fix + inst;
  const int tile0 = c->rt0, ntiles = c->nrt, nnodes = c->nnodes;
  const unsigned ngroup = unsigned((ntiles + kArriveGroup - 1) / kArriveGroup);
  __shared__ int s_last;
  __shared__ double s_tot[8];
  const int tid = threadIdx.x;
  uint32_t* const top = a.arrive + size_t(c->ctop) * kArriveStride;
  if (tid < 64) {
    // threads 0-7 of this wave stored the partials: wait for the stores
    __builtin_amdgcn_s_waitcnt(0);
    if (tid == 0) {
      const int g = (tile - tile0) / kArriveGroup;
      const unsigned gsize = unsigned(min(kArriveGroup, ntiles - g * kArriveGroup));
      uint32_t* const gc = a.arrive + size_t(c->cbase + g) * kArriveStride;
      bool last = false;
      if (__hip_atomic_fetch_add(gc, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gsize - 1) {
        __hip_atomic_store(gc, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        last = ngroup == 1 || __hip_atomic_fetch_add(top, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == ngroup - 1;
      }
      s_last = last;
    }
  }
  __syncthreads();
  if (!s_last) return;
  Ctl* const cp = a.ctl + inst;
  Ctl cc;
  if (tid == 0) cc = *cp;   // loaded beside the partials
  const double vk = combine_partials(a.part, size_t(a.dr.n_tiles), tile0, ntiles, red);
  if (tid < 8) s_tot[tid] = vk;
  __syncthreads();
  if (tid != 0) return;
  double v[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) v[k] = s_tot[k];
  advance_solver(&cc, nnodes, v, bnd, a.kind, a.tol, a.max_iter);
  if (a.fuse == 1) *cp = cc;
  __hip_atomic_store(top, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Final pass: bounds, active flags and statistics.
template <typename T>
__global__ __launch_bounds__(kBlock) void k_dmg_final(DmgArgs<T> a, uint8_t* active_out, pf_cg_stats_t* stats) {
  const int tile = tile_of_block(a.dm.n_tiles);
  const TileRec t = a.dm.tiles[tile];
  const Ctl* c = a.ctl + t.inst;
  const InstP<T> P = a.ip[t.inst];
  const bool projected = (P.bounds == PF_BOUNDS_PROJECTED);
  const double* xc = c->pbuf ? a.x1 : a.x0;
  const uint8_t* Wc = c->wbuf ? a.W1 : a.W0;
  if (a.kind != CG_QP) {
    for (int i = threadIdx.x; i < t.n_own; i += kBlock) {
      const int g = t.node_begin + i;
      a.dout[g] = (c->ref == 0.0) ? T(0) : T(xc[a.dr.pos[g]]);
    }
  } else {
    for (int i = threadIdx.x; i < t.n_own; i += kBlock) {
      const int g = t.node_begin + i;
      const int q = a.dr.pos[g];
      T xv = T(xc[q]);
      const T lbv = a.lb[g];
      uint8_t act = 0;
      if (projected) {
        const uint8_t w = Wc[q];
        act = (w == HELD_LOWER || w == HELD_FIXED) ? PF_ACTIVE_LOWER : ((w == HELD_UPPER) ? PF_ACTIVE_UPPER : 0);
        xv = clamp01<T>(xv, lbv);   // free nodes within tol outside the bounds
      } else {
        if (xv < lbv) {
          xv = lbv;
          act = PF_ACTIVE_LOWER;
        }
        if (xv > T(1)) {
          xv = T(1);
          act |= PF_ACTIVE_UPPER;
        }
      }
      a.dout[g] = xv;
      if (active_out) active_out[g] = act;
    }
  }
  if (stats && threadIdx.x == 0 && tile == a.fix[t.inst].tile0) {
    pf_cg_stats_t s;
    s.iters = c->iters;
    s.restarts = c->restarts;
    s.n_active = c->nact;
    s.flags = c->flags | (c->mode == MODE_DONE ? 0 : PF_FLAG_NOT_CONVERGED);
    s.resid = c->resid;
    stats[t.inst] = s;
  }
}

template <typename T>
static DmgArgs<T> dmg_args(pf_mesh_s* m, int kind, const void* H, const void* d_prev, void* d,
                           const uint8_t* guess, const pf_cg_opts_t* o) {
  DmgArgs<T> a;
  a.kind = kind;
  a.start = (kind == CG_QP) ? o->start : 0;
  a.dm = m->dm;
  a.dr = m->dr;
  a.ip = static_cast<const InstP<T>*>(m->dw.instp);
  a.ctl = m->dw.ctl;
  a.fix = m->dw.fix;
  a.part = m->dw.part;
  a.H = static_cast<const T*>(H);
  a.lb = static_cast<const T*>(d_prev);
  a.guess = guess;
  // linear solves start from, and end in, the caller's array
  a.dout = static_cast<T*>(d);
  a.bin = static_cast<const T*>(m->dw.b);
  a.win = m->dw.wset;
  a.x0 = static_cast<double*>(m->dw.x0);
  a.x1 = static_cast<double*>(m->dw.x1);
  a.rs0 = static_cast<Two<T>*>(m->dw.rs0);
  a.rs1 = static_cast<Two<T>*>(m->dw.rs1);
  a.wz0 = static_cast<Two<T>*>(m->dw.wz0);
  a.wz1 = static_cast<Two<T>*>(m->dw.wz1);
  a.p = static_cast<T*>(m->dw.p);
  a.dim = static_cast<T*>(m->dw.dim);
  a.rsum = static_cast<T*>(m->dw.rsum);
  a.b = static_cast<T*>(m->dw.br);
  a.lbr = static_cast<T*>(m->dw.lbr);
  a.W0 = m->dw.wr;
  a.W1 = m->dw.wr + m->n_nodes;
  a.tol = o->tol;
  a.max_iter = o->max_iter;
  a.deg = o->precond;
  a.fuse = m->fuse ? 1 : 0;
  a.arrive = m->dw.arrive;
  a.nch = 1;
  return a;
}

// The CG pass for row tiles of up to 256 rpt rows, of which the first 256 own
// hold the owned nodes.
template <typename T>
using CgKernel = void (*)(DmgArgs<T>);
template <typename T, int RPT, int OWN>
static CgKernel<T> cg_kernel_of(const pf_mesh_s* m, bool fuse, bool setup) {
  if (setup) return fuse ? k_cg_setup<T, RPT, OWN, true> : k_cg_setup<T, RPT, OWN, false>;
  // the first extra pair in registers too, where there are any and the registers suffice
  if constexpr (RPT <= (sizeof(T) == 4 ? 4 : 3)) {
    constexpr int X = kRowPairs + 1;
    if (m->cg.extra_pairs) return fuse ? k_cg<T, RPT, OWN, X, true> : k_cg<T, RPT, OWN, X, false>;
  }
  return fuse ? k_cg<T, RPT, OWN, kRowPairs, true> : k_cg<T, RPT, OWN, kRowPairs, false>;
}
template <typename T>
static CgKernel<T> cg_kernel(const pf_mesh_s* m, int deg, bool setup) {
  const bool fuse = m->fuse;
  const bool one = cg_own_rows(m->cg, deg) == 1;
  switch (cg_rows(m->cg, deg)) {
    case 1: return cg_kernel_of<T, 1, 1>(m, fuse, setup);
    case 2: return cg_kernel_of<T, 2, 1>(m, fuse, setup);
    case 3: return one ? cg_kernel_of<T, 3, 1>(m, fuse, setup) : cg_kernel_of<T, 3, 3>(m, fuse, setup);
    case 4: return cg_kernel_of<T, 4, 4>(m, fuse, setup);
    default: return cg_kernel_of<T, 8, 8>(m, fuse, setup);
  }
}

template <typename T>
static void launch_cg(const pf_mesh_s* m, DmgArgs<T> a, int nch, hipStream_t s) {
  a.nch = nch;
  hipLaunchKernelGGL(cg_kernel<T>(m, a.deg, nch > 0), dim3(m->dr.n_tiles), dim3(kBlock), cg_lds(m->cg, a.deg, nch, sizeof(T)), s, a);
}

// Element chunks of the set-up pass: two (the elements' mass coefficients and
// their loads one after the other in LDS) when the halved space lets more
// workgroups share a CU; the row plan takes care that one fits.
template <typename T>
static int damage_chunks(pf_mesh_s* m) {
  if (m->dmg_nch > 0) return m->dmg_nch;
  int nch = m->damage_chunks;
  auto occ = [&](int n) {
    int o = 0;
    const void* k = reinterpret_cast<const void*>(cg_kernel<T>(m, 0, true));
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&o, k, kBlock, cg_lds(m->cg, 0, n, sizeof(T))) != hipSuccess) o = 0;
    return o;
  };
  if (nch <= 0) nch = occ(2) > occ(1) ? 2 : 1;
  m->dmg_nch = nch;
  return nch;
}

void damage_plan(pf_mesh_s* m) {
  if (m->dtype == PF_F64)
    (void)damage_chunks<double>(m);
  else
    (void)damage_chunks<float>(m);
}

template <typename T>
static pf_status_t run_solve(pf_mesh_s* m, int kind, const void* H, const void* d_prev, void* d,
                             const uint8_t* guess, uint8_t* active_out, const pf_cg_opts_t* o,
                             pf_cg_stats_t* stats, hipStream_t s) {
  DmgArgs<T> a = dmg_args<T>(m, kind, H, d_prev, d, guess, o);
  const dim3 grid(m->n_tiles), block(kBlock), igrid(m->n_inst);
  const int nch = damage_chunks<T>(m);
  bool setup = !o->resume;   // the first round of a solve is its set-up restart
  if (setup) {
    timer_begin(m, 2, s);
    hipLaunchKernelGGL(k_dmg_init, dim3((m->n_inst + 63) / 64), dim3(64), 0, s, m->dw.ctl, m->dw.fix, m->n_inst,
                       kind, o->monotone, o->precond);
    timer_end(m, 2, s);
  }
  if (kind == CG_QP) {
    const unsigned char* ab = reinterpret_cast<const unsigned char*>(&a);
    m->last_qp_args.assign(ab, ab + sizeof(a));
    m->last_qp_precond = o->precond;
  }
  auto round = [&]() {
    timer_begin(m, 1, s);
    launch_cg<T>(m, a, setup ? nch : 0, s);
    timer_end(m, 1, s);
    if (!a.fuse) {
      timer_begin(m, 4, s);
      hipLaunchKernelGGL(k_dmg_red, igrid, dim3(kRedBlock), 0, s, m->dw.ctl, m->dw.fix, m->dw.part,
                         m->dr.n_tiles, m->dw.bounds, kind, o->tol, o->max_iter);
      timer_end(m, 4, s);
    }
    setup = false;
  };
  const int max_rounds = (o->check_every <= 0 && o->rounds > 0) ? std::min(o->rounds, o->max_iter) : o->max_iter;
  int launched = 0;
  if (o->check_every <= 0) {
    for (; launched < max_rounds; ++launched) round();
  } else {
    // first poll after two rounds more than the last solve of this kind
    // needed (solves of consecutive steps take similar counts, and a round of
    // a finished solve costs only two near-empty launches), then every
    // check_every rounds
    const int last = m->last_rounds[kind == CG_QP ? 0 : 1];
    int chunk = last > 0 ? last + 2 : std::min(o->check_every, 8);
    if (o->check_every == 1) chunk = 1;   // poll after every round: no round runs after the solve ends
    while (launched < max_rounds) {
      const int n = std::min(chunk, max_rounds - launched);
      for (int k = 0; k < n; ++k) round();
      launched += n;
      PF_HIP(hipGetLastError());
      PF_HIP(hipMemcpyAsync(m->ctl_pinned, m->dw.ctl, sizeof(Ctl) * m->n_inst, hipMemcpyDeviceToHost, s));
      PF_HIP(hipEventRecord(m->poll_ev, s));
      // spin rather than block: the wait is short and a sleeping host thread
      // wakes up tens of microseconds late
      hipError_t q;
      while ((q = hipEventQuery(m->poll_ev)) == hipErrorNotReady) {
      }
      if (q != hipSuccess) return hip_fail(q, "hipEventQuery");
      bool all_done = true;
      for (int k = 0; k < m->n_inst; ++k) all_done = all_done && (m->ctl_pinned[k].mode == MODE_DONE);
      if (all_done) break;
      chunk = o->check_every;
    }
  }
  timer_begin(m, 2, s);
  hipLaunchKernelGGL(k_dmg_final<T>, grid, block, 0, s, a, active_out, stats);
  timer_end(m, 2, s);
  PF_HIP(hipGetLastError());
  if (o->check_every > 0) {
    // the last poll saw every instance done, or the round budget is spent:
    // either way the control blocks it copied are final
    int flags = 0, rounds = 0;
    for (int k = 0; k < m->n_inst; ++k) {
      flags |= m->ctl_pinned[k].flags;
      if (m->ctl_pinned[k].mode != MODE_DONE) flags |= PF_FLAG_NOT_CONVERGED;
      rounds = std::max(rounds, int(m->ctl_pinned[k].iters));
    }
    m->last_rounds[kind == CG_QP ? 0 : 1] = rounds;
    if (flags & PF_FLAG_NONFINITE) return fail(PF_ERR_NONFINITE, "non-finite value in the damage CG");
    if (flags & PF_FLAG_NOT_CONVERGED) return fail(PF_ERR_NOT_CONVERGED, "damage CG reached max_iter");
  }
  return PF_OK;
}

// n launches of the main pass of the last damage solve's current round, with
// no reduction in between (a throughput measurement; see pf.h).
template <typename T>
static pf_status_t repeat_pass(pf_mesh_s* m, const void* H, const void* d_prev, void* d, int n, hipStream_t s) {
  DmgArgs<T> a;
  if (m->last_qp_args.size() != sizeof(a)) return fail(PF_ERR_ARG, "no damage solve on this handle");
  if (m->last_qp_precond >= 2)
    return fail(PF_ERR_ARG, "repeated passes need the default or the Jacobi preconditioner");
  std::memcpy(&a, m->last_qp_args.data(), sizeof(a));
  // the caller's arrays as given now; the workspaces are the handle's
  a.H = static_cast<const T*>(H);
  a.lb = static_cast<const T*>(d_prev);
  a.dout = static_cast<T*>(d);
  a.guess = nullptr;
  // where the solver's rounds combine the partials in the pass's last
  // workgroup, each launch does so too but leaves the control block as it is
  a.fuse = a.fuse ? 2 : 0;
  PF_HIP(hipMemcpyAsync(m->ctl_pinned, m->dw.ctl, sizeof(Ctl) * m->n_inst, hipMemcpyDeviceToHost, s));
  PF_HIP(hipStreamSynchronize(s));
  for (int k = 0; k < m->n_inst; ++k)
    if (m->ctl_pinned[k].mode != MODE_ITER)
      return fail(PF_ERR_ARG, "the last damage solve did not stop in a CG iteration");
  for (int i = 0; i < n; ++i) launch_cg<T>(m, a, 0, s);
  PF_HIP(hipGetLastError());
  return PF_OK;
}

pf_status_t damage_cg(pf_mesh_s* m, int kind, const void* H, const void* lb, void* x, const uint8_t* guess,
                      uint8_t* active_out, const pf_cg_opts_t* o, pf_cg_stats_t* stats, hipStream_t s) {
  return (m->dtype == PF_F64) ? run_solve<double>(m, kind, H, lb, x, guess, active_out, o, stats, s)
                              : run_solve<float>(m, kind, H, lb, x, guess, active_out, o, stats, s);
}

}  // namespace pf

using namespace pf;

extern "C" pf_status_t pf_damage_solve(pf_mesh_t m, const pf_params_t* p, const void* H, const void* d_prev, void* d,
                                       const uint8_t* active_guess, uint8_t* active_out, const pf_cg_opts_t* opts,
                                       pf_cg_stats_t* stats, pf_stream_t stream) {
  if (!m) return fail(PF_ERR_ARG, "mesh is NULL");
  pf_status_t st;
  if ((st = check_params(m, p, nullptr, false)) != PF_OK) return st;
  if (!H || !d_prev || !d || !opts) return fail(PF_ERR_ARG, "NULL argument");
  if (d == d_prev) return fail(PF_ERR_ARG, "d must not alias d_prev");
  if (!(opts->tol > 0) || opts->max_iter < 1) return fail(PF_ERR_ARG, "need tol > 0 and max_iter >= 1");
  if (opts->rounds < 0) return fail(PF_ERR_ARG, "rounds must be >= 0");
  if (opts->precond < 0 || opts->precond > 4) return fail(PF_ERR_ARG, "precond must be in [0, 4]");
  if (opts->resume && !m->qp_started) return fail(PF_ERR_ARG, "resume without a previous damage solve on this handle");
  hipStream_t s = static_cast<hipStream_t>(stream);
  if ((st = upload_params(m, p, nullptr, s)) != PF_OK) return st;
  m->qp_started = true;
  return damage_cg(m, CG_QP, H, d_prev, d, active_guess, active_out, opts, stats, s);
}

extern "C" pf_status_t pf_damage_pass_repeat(pf_mesh_t m, const void* H, const void* d_prev, void* d,
                                             int32_t n_passes, pf_stream_t stream) {
  if (!m) return fail(PF_ERR_ARG, "mesh is NULL");
  if (!H || !d_prev || !d) return fail(PF_ERR_ARG, "NULL argument");
  if (n_passes < 1) return fail(PF_ERR_ARG, "n_passes must be >= 1");
  hipStream_t s = static_cast<hipStream_t>(stream);
  return (m->dtype == PF_F64) ? repeat_pass<double>(m, H, d_prev, d, n_passes, s)
                              : repeat_pass<float>(m, H, d_prev, d, n_passes, s);
}
