// gfx950 kernels of the two-species D2Q9 MRT chemotaxis step, its exact
// discrete adjoint (AMRT) and the cost / gradient / update reductions.
//
// Method: arXiv:1908.03876, Section 3.1 (eq:LBE, S, PhiS, MF, MC, phieq,
// BC11, the relaxation matrix Pi and D = d Cs^2 tau (K^-1 - I/2)) and
// Section 3.2.1 (LIBEG, CAE, AEDs, RFS1, CAEL, gradientLattice).
//
// Design (a stencil of about 240 vector instructions a node and step, no
// contraction, so no MFMA):
//  * One thread per lattice node; populations live in SoA planes, so each
//    wavefront reads and writes whole rows of a plane.
//  * The state between launches is post-collision, and the kernels pull:
//    node x gathers phi*_i(x - e_i) (or its own phi*_opp(i) at a wall,
//    halfway bounce-back).  Collision runs in registers in moment space;
//    M0^-1 is applied as M0^T with the row norms folded into the rates.
//  * The adjoint is a gather too: nu_i(x) = lambda_i(x + e_i), or
//    lambda_opp(i)(x) when x + e_i is a wall (exact transpose of the pull).
//  * One step per launch is bound by HBM (the AMRT step's 172 B a node at 68%
//    of 8 TB/s: 125 us at 2048^2); so a launch takes several steps in a region
//    of the lattice held in registers, streaming through LDS, and reads and
//    writes the state once for all of them (see "time-step kernels").
//  * Regions are dealt so that each of the 8 XCDs walks a contiguous band of
//    rows: its L2 serves the rows that neighbouring regions share.
//  * Walls cost no test in the pull: see the wall slots in mrt_device.h.
//  * Reductions: wave shuffles (64 lanes), LDS across waves, one partial per
//    block, then a single-block pass in fixed order (deterministic).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <mutex>
#include <type_traits>

#include "mrt_device.h"
#include "mrt_internal.h"
#include "mrt_region.h"

namespace mrt {
namespace {

using namespace dev;

// -------------------------------------------------------------- link mask

// bit 0: node solid; bit i (1..8): x - e_i is solid (wrapped when periodic)
// or outside a non-periodic lattice.
__global__ void build_link_kernel(Geometry g, int periodic,
                                  const uint8_t* __restrict__ mask,
                                  uint16_t* __restrict__ link,
                                  uint32_t* __restrict__ wflag) {
  const int x = blockIdx.x * blockDim.x + threadIdx.x;
  const int y = blockIdx.y;
  if (x >= g.nx) return;
  const int ex[9] = {0, 1, 0, -1, 0, 1, -1, -1, 1};
  const int ey[9] = {0, 0, 1, 0, -1, 1, 1, -1, -1};
  uint16_t bits = 0;
  for (int i = 0; i < 9; ++i) {
    int xs = x - ex[i], ys = y - ey[i];
    const bool out = xs < 0 || ys < 0 || xs >= g.nx || ys >= g.ny;
    if (out && !periodic) {
      bits |= uint16_t(1u << i);
      continue;
    }
    xs = (xs + g.nx) % g.nx;
    ys = (ys + g.ny) % g.ny;
    if (mask[size_t(ys) * g.pitch + xs]) bits |= uint16_t(1u << i);
  }
  link[size_t(y) * g.pitch + x] = bits;
  // blocks are 256 wide along x, so each wavefront is one 64-node segment
  const unsigned long long any = __ballot(bits != 0);
  const unsigned long long fluid = __ballot((bits & 1u) == 0);
  if ((threadIdx.x & 63) == 0)
    wflag[size_t(y) * g.nsx + (x >> 6)] = fluid == 0ull ? 2u : (any != 0ull);
}

// ------------------------------------------------------- time-step kernels

// One thread's node of a region.  Regions that reach past a lattice edge
// wrap around it, periodic or not: across a wall nothing is taken from the
// nodes beyond.
struct RegionNode {
  int x, y;
  bool owner;  // its results are stored by this thread
};

template <int RX, int RY>
__device__ __forceinline__ RegionNode region_node(const Geometry& g, const TileGrid& tg,
                                                  int tid) {
  const int halo = kRows<RY> ? 0 : tg.steps - 1;
  const int t = xcd_tile(blockIdx.x, tg.ntiles);
  int ty = int((unsigned long long)unsigned(t) * tg.inv_ntx >> 32), tx = t - ty * tg.ntx;
  if (tx >= tg.ntx) {  // the reciprocal is rounded down
    ++ty;
    tx -= tg.ntx;
  }
  int dx = unsigned(tid) % RX, dy = unsigned(tid) / RX;
  if (RX % 64 == 0) dy = __builtin_amdgcn_readfirstlane(dy);  // a wavefront is one row
  RegionNode r;
  r.x = tx * (RX - 2 * halo) - halo + dx;
  r.y = ty * (RY - 2 * halo) - halo + dy;
  r.owner = dx >= halo && dx < RX - halo && r.x < g.nx && dy >= halo && dy < RY - halo &&
            r.y < g.ny;
  if (kRows<RY>) return r;  // the others leave at once
  // at most RX (RY) nodes past an edge: once around, unless the lattice is
  // smaller than that
  if (g.nx < RX) {
    r.x %= g.nx;
  } else {
    r.x = r.x >= g.nx ? r.x - g.nx : r.x;
  }
  if (g.ny < RY) {
    r.y %= g.ny;
  } else {
    r.y = r.y >= g.ny ? r.y - g.ny : r.y;
  }
  r.x = r.x < 0 ? r.x + g.nx : r.x;
  r.y = r.y < 0 ? r.y + g.ny : r.y;
  if (RX % 64 == 0) r.y = __builtin_amdgcn_readfirstlane(r.y);
  return r;
}

__device__ __forceinline__ Steps steps_of(const TileGrid& tg) {
  return {tg.steps, tg.steps - 1};
}

// The node again, at the end of a launch, with the plane size it is
// addressed by: computed afresh, so that nothing derived from it stays in
// registers over the steps (the stores' row bases alone would not fit beside
// the coefficients).  False: another thread stores its results.
template <int RX, int RY>
__device__ __forceinline__ bool node_again(Geometry& g, const TileGrid& tg, NodeIdx& n) {
  if (kRows<RY>) return true;
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid), "+s"(g.plane), "+s"(g.nx), "+s"(g.ny));
  const RegionNode r = region_node<RX, RY>(g, tg, tid);
  make_node(g, r.x, r.y, n);
  return r.owner;
}

// Link word of a node; of a non-periodic lattice without a mask, from the
// coordinates.
template <Lanes A>
__device__ __forceinline__ unsigned link_word(const Geometry& g, const NodeIdx& n) {
  if (g.link) return *own_at<A>(g.link, n);
  unsigned w = 0;
#pragma unroll
  for (int i = 1; i < 9; ++i) w |= pull_outside(n, i) ? 1u << i : 0u;
  return w;
}

// Link word in a kernel of rows (a wavefront is one of the 64-node segments
// that the flags describe): read only where the segment touches a solid node.
// False: the wavefront lies inside a solid region.
template <bool ROWS, Lanes A>
__device__ __forceinline__ bool links(const Geometry& g, const NodeIdx& n, unsigned& lm) {
  if (ROWS && g.masked) {
    const unsigned flag = wave_flag(g, n);
    if (flag == 2u) return false;
    lm = flag ? unsigned(*own_at<A>(g.link, n)) : 0u;
    return true;
  }
  lm = link_word<A>(g, n);
  return true;
}

// Are all nodes of this work-group's region solid, by the flags of the 64-node
// segments that it touches?  Every wavefront reads all of them (a lane per row
// and side) and comes to the same answer without a barrier.  A region that wraps
// around an end of its rows is not asked.
//
// The look stands before a region's loads and costs 5% where it finds nothing
// (2048^2, AMRT step 53.2 -> 56.3 us), so only lattices of which a share of the
// segments is all solid (kSolidAreas) have kernels that look (kAreas).  Forward
// step in us without and with it, by the share of fluid in one square block:
//            2%           10%           25%           50%           75%
//   2048^2  45.3 12.9    48.5 24.1     48.6 31.3     55.4 46.2     58.6 56.0
//   1024^2  11.8  5.7    12.1  7.9     12.6  9.5     13.1 11.7     13.9 13.9
template <int RX, int RY>
__device__ __forceinline__ bool solid_region(const Geometry& g, const TileGrid& tg) {
  static_assert(RX <= 64 && 2 * RY <= 64, "two flags a row");
  const int lane = threadIdx.x & 63;
  const int t = xcd_tile(blockIdx.x, tg.ntiles), halo = tg.steps - 1;
  const int x0 = t % tg.ntx * (RX - 2 * halo) - halo;
  int y = t / tg.ntx * (RY - 2 * halo) - halo + lane % RY;
  if (x0 < 0 || x0 + RX > g.nx) return false;
  y = (y < 0 ? y + g.ny * RY : y) % g.ny;
  const int x = x0 + (lane / RY & 1) * (RX - 1);
  return __builtin_amdgcn_ballot_w64(g.wflag[size_t(y) * g.nsx + (x >> 6)] != 2u) == 0ull;
}

// What a kernel meets: no walls, walls, walls with solid areas.
constexpr int kOpen = 0, kWalls = 1, kAreas = 2;

// Regions of 16 x 16 and of 32 x 32 nodes are taken only where a plane's offsets
// fit 32 bits (plan_steps).
template <int RX, int RY>
constexpr Lanes lanes_of = short_offsets(RX, RY) ? kSmall : RX % 64 == 0 ? kRow : kAny;

// A node's populations take more than the 72 bytes of two species in FP32.
template <typename T, int VAR>
constexpr bool kWide = sizeof(T) == 8 || VAR == kVarThree;

// Wavefronts per SIMD that a region kernel is compiled for.
template <typename T, int VAR>
constexpr int kRegionWaves = (sizeof(T) == 4 ? 8 : 4) / (VAR == kVarThree ? 2 : 1);

#define MRT_REGION_BOUNDS(T, VAR, RX, RY)                            \
  __attribute__((amdgpu_flat_work_group_size(RX * RY, RX * RY),      \
                 amdgpu_waves_per_eu(kRegionWaves<T, VAR>)))

// Forward steps n .. n + K - 1 (FIRST: n = 0, from the initial fields).
template <typename T, int KIND, int VAR, int RX, int RY, bool FIRST>
__global__ MRT_REGION_BOUNDS(T, VAR, RX, RY) void forward_kernel(Geometry g, ModelCoef<T> m,
                                                                 FwdLaunch<T> a, TileGrid tg) {
  constexpr bool W3 = VAR == kVarThree, LAG = VAR == kVarExplicit;
  constexpr bool WALLS = KIND != kOpen;
  constexpr Lanes A = lanes_of<RX, RY>;
  __shared__ Exchange<T, RX, RY, W3> lds;
  const RegionNode r = region_node<RX, RY>(g, tg, threadIdx.x);
  if (kRows<RY> && !r.owner) return;
  NodeIdx n;
  make_node(g, r.x, r.y, n);
  if constexpr (KIND == kAreas)
    if (solid_region<RX, RY>(g, tg)) return;
  unsigned lm = 0;
  T fu[9], fv[9], fw[9], lag[2] = {T(0), T(0)}, c = T(0);
  if (WALLS && !links<kRows<RY>, A>(g, n, lm)) return;
  if (kRows<RY> && WALLS && (lm & 1u)) {
    // a solid node loads nothing and collides zeros: it takes part in the
    // record stores, so that these fill whole 64-byte chunks
#pragma unroll
    for (int i = 0; i < 9; ++i) fu[i] = fv[i] = fw[i] = T(0);
  } else {
    pull_species<A, FIRST>(g, n, m.u, a.src, a.u0, fu);
    pull_species<A, FIRST>(g, n, m.v, a.src + 9 * g.plane, a.v0, fv);
    if (W3) pull_species<A, FIRST>(g, n, m.w, a.src + 18 * g.plane, a.w0, fw);
    c = *own_at<A>(a.ctrl, n);
    if (LAG && !FIRST) {
      lag[0] = *own_at<A>(a.lag, n);
      lag[1] = *own_at<A>(a.lag + g.plane, n);
    }
  }
  if (!forward_steps<WALLS, VAR, A, FIRST>(lds, g, n, lm, m, c, r.owner, fu, fv, fw, lag, a.rec,
                                           a.rec_stride, steps_of(tg)))
    return;
  if (!node_again<RX, RY>(g, tg, n)) return;
  if (LAG) {
    *own_at<A>(a.lag_out, n) = lag[0];
    *own_at<A>(a.lag_out + g.plane, n) = lag[1];
  }
  if (WALLS && (lm & 1u)) return;  // its slots hold the neighbours' wall stores
  store_species<A, WALLS, false, kRows<RY>>(g, n, fu, a.dst, lm);
  store_species<A, WALLS, false, kRows<RY>>(g, n, fv, a.dst + 9 * g.plane, lm);
  if (W3) store_species<A, WALLS, false, kRows<RY>>(g, n, fw, a.dst + 18 * g.plane, lm);
}

template <typename T, bool IMPL, bool W3>
__global__ __launch_bounds__(kBlock) void finalize_kernel(
    Geometry g, ModelCoef<T> m, const T* __restrict__ src, const T* __restrict__ ctrl,
    T* __restrict__ state, T* __restrict__ uN, T* __restrict__ vN) {
  NodeIdx n;
  if (!node_of_block(g, n)) return;
  finalize_node<T, IMPL, W3>(g, n, src, state, uN, vN, &m, ctrl);
}

// Pull of the populations streamed into node n after the last step (zeros
// on solid nodes) and their sums G.
template <typename T>
__device__ __forceinline__ bool pull_sums(const Geometry& g, const NodeIdx& n,
                                          const T* __restrict__ src, T& Gu, T& Gv) {
  const size_t idx = n.r0 + n.x;
  if (g.masked && (link_of(g, wave_flag(g, n), idx) & 1u)) return false;
  Gu = T(0);
  Gv = T(0);
#pragma unroll
  for (int i = 0; i < 9; ++i) {
    Gu += *pull_at<kAny>(src + size_t(i) * g.plane, n, i);
    Gv += *pull_at<kAny>(src + size_t(9 + i) * g.plane, n, i);
  }
  return true;
}

// Implicit characteristic difference, terminal condition of the adjoint:
// the cost sees Theta^N, a function of the sums G^N of the last state, so
// the seeds (dJ/du^N, dJ/dv^N) = (a, b) become the adjoint of G^N:
// beta b and alpha (a + (tau/2) a_uv beta b), with alpha and beta of the
// node equation at u^N.  v^N also depends on the control (weight tau/2 in
// the node equation): the gradient accumulator starts at (tau/2) beta b.
// Zero on solid nodes.
template <typename T>
__global__ __launch_bounds__(kBlock) void implicit_terminal_kernel(
    Geometry g, ModelCoef<T> m, const T* __restrict__ src, const T* __restrict__ ctrl,
    const T* __restrict__ seed_u, const T* __restrict__ seed_v, T* __restrict__ out_u,
    T* __restrict__ out_v, double* __restrict__ gacc) {
  NodeIdx n;
  if (!node_of_block(g, n)) return;
  const size_t idx = n.r0 + n.x;
  T Gu, Gv;
  if (!pull_sums<T>(g, n, src, Gu, Gv)) {
    out_u[idx] = T(0);
    out_v[idx] = T(0);
    gacc[idx] = 0.0;
    return;
  }
  T u, v;
  implicit_solve(m, Gu, Gv, ctrl[idx], u, v);
  const T alpha = T(1) / (T(1) - T(0.5) * m.r_u * (T(1) - T(2) * u));
  const T beta = T(1) / (T(1) + T(0.5) * m.b_v);
  const T b = seed_v ? seed_v[idx] : T(0);
  out_v[idx] = beta * b;
  out_u[idx] = alpha * (seed_u[idx] + T(0.5) * m.a_uv * beta * b);
  gacc[idx] = double(T(0.5) * beta * b);
}

// Implicit characteristic difference, end of the tangent sweep: the
// perturbation of Theta^N from that of G^N (node equation linearised at the
// forward's u^N, with the control perturbation).
template <typename T>
__global__ __launch_bounds__(kBlock) void implicit_tlm_final_kernel(
    Geometry g, ModelCoef<T> m, const T* __restrict__ fsrc, const T* __restrict__ dsrc,
    const T* __restrict__ ctrl, const T* __restrict__ dc, T* __restrict__ duN,
    T* __restrict__ dvN) {
  NodeIdx n;
  if (!node_of_block(g, n)) return;
  const size_t idx = n.r0 + n.x;
  T Gu, Gv, dGu, dGv;
  if (!pull_sums<T>(g, n, fsrc, Gu, Gv)) {
    if (duN) duN[idx] = T(0);
    if (dvN) dvN[idx] = T(0);
    return;
  }
  pull_sums<T>(g, n, dsrc, dGu, dGv);
  T u, v;
  implicit_solve(m, Gu, Gv, ctrl[idx], u, v);
  const T du = dGu / (T(1) - T(0.5) * m.r_u * (T(1) - T(2) * u));
  const T dcc = dc ? dc[idx] : T(0);
  if (duN) duN[idx] = du;
  if (dvN) dvN[idx] = (dGv + T(0.5) * (m.a_uv * du + dcc)) / (T(1) + T(0.5) * m.b_v);
}

// Adjoint steps n, n - 1, ..., n - K + 1.
template <typename T, int KIND, int VAR, int RX, int RY, bool FIRST>
__global__ MRT_REGION_BOUNDS(T, VAR, RX, RY) void adjoint_kernel(Geometry g, ModelCoef<T> m,
                                                            AdjLaunch<T> a, TileGrid tg) {
  constexpr bool W3 = VAR == kVarThree, LAG = VAR == kVarExplicit, IMPL = VAR == kVarImplicit;
  constexpr bool WALLS = KIND != kOpen;
  __shared__ Exchange<T, RX, RY, W3> lds;
  constexpr Lanes A = lanes_of<RX, RY>;
  const RegionNode r = region_node<RX, RY>(g, tg, threadIdx.x);
  if (kRows<RY> && !r.owner) return;
  NodeIdx n;
  make_node(g, r.x, r.y, n);
  unsigned lm = 0;
  T nu[9], nv[9], nw[9], mu[2] = {T(0), T(0)};
  double sum = 0.0;
  constexpr bool fresh = FIRST && !IMPL;  // the sweep's first step: g starts at zero
  // a sweep's outputs are zero on solid nodes: what it starts, it clears there
  // in its first launch, what it ends in its last
  auto clear = [&] {
    if (fresh) *own_at<A>(a.g, n) = 0.0;
    if (a.adj_u0) *own_at<A>(a.adj_u0, n) = T(0);
    if (a.adj_v0) *own_at<A>(a.adj_v0, n) = T(0);
  };
  if (WALLS && !links<kRows<RY> && !FIRST, A>(g, n, lm)) lm = 1u;
  if (kRows<RY> && WALLS && !FIRST && (lm & 1u)) return clear();
  if constexpr (KIND == kAreas)
    if (solid_region<RX, RY>(g, tg)) {
      if (r.owner) clear();
      return;
    }
  if (kRows<RY> && !a.dst && !a.adj_u0 && !a.adj_v0) {
    // step 0 of a sweep that asks for the gradient alone: its share needs no
    // record and no adjoint of u
    if (WALLS && (lm & 1u)) return clear();
    adjoint_gather<A, WALLS, VAR, FIRST, T>(g, n, a.src, a.seed_u, a.seed_v, lm, nu, nv, nw);
    const T share = weighted(nv);
    *own_at<A>(a.g, n) = (fresh ? 0.0 : *own_at<A>(a.g, n)) + double(IMPL ? T(0.5) * share : share);
    return;
  }
  adjoint_gather<A, WALLS, VAR, FIRST, T>(g, n, a.src, a.seed_u, a.seed_v, lm, nu, nv, nw);
  if (LAG && !FIRST) {
    mu[0] = *own_at<A>(a.mu, n);
    mu[1] = *own_at<A>(a.mu + g.plane, n);
  }
  if (r.owner && !fresh) sum = *own_at<A>(a.g, n);
  if (!adjoint_steps<WALLS, VAR, A, FIRST>(lds, g, n, lm, m, a.step, nu, nv, nw, mu, sum, a.rec,
                                           a.rec_stride, steps_of(tg)))
    return;
  if (!node_again<RX, RY>(g, tg, n)) return;
  if (WALLS && (lm & 1u)) return clear();
  *own_at<A>(a.g, n) = sum;
  if (LAG) {
    *own_at<A>(a.mu_out, n) = mu[0];
    *own_at<A>(a.mu_out + g.plane, n) = mu[1];
  }
  if (a.adj_u0) *own_at<A>(a.adj_u0, n) = adjoint_initial(m.u, nu);
  if (a.adj_v0) *own_at<A>(a.adj_v0, n) = adjoint_initial(m.v, nv);
  if (a.dst == nullptr) return;
  store_species<A, WALLS, true, kRows<RY>>(g, n, nu, a.dst, lm);
  store_species<A, WALLS, true, kRows<RY>>(g, n, nv, a.dst + 9 * g.plane, lm);
  if (W3) store_species<A, WALLS, true, kRows<RY>>(g, n, nw, a.dst + 18 * g.plane, lm);
}

// Tangent-linear steps n .. n + K - 1: pull the perturbation (FIRST, step 0:
// the equilibrium of (du0, dv0); the third species starts at zero),
// linearised collision at the recorded (u, j_v), streaming as the forward.
template <typename T, int KIND, int VAR, int RX, int RY, bool FIRST>
__global__ MRT_REGION_BOUNDS(T, VAR, RX, RY) void tlm_kernel(Geometry g, ModelCoef<T> m,
                                                             TlmLaunch<T> a, TileGrid tg) {
  constexpr bool W3 = VAR == kVarThree, LAG = VAR == kVarExplicit;
  constexpr bool WALLS = KIND != kOpen;
  constexpr Lanes A = lanes_of<RX, RY>;
  __shared__ Exchange<T, RX, RY, W3> lds;
  const RegionNode r = region_node<RX, RY>(g, tg, threadIdx.x);
  if (kRows<RY> && !r.owner) return;
  NodeIdx n;
  make_node(g, r.x, r.y, n);
  if constexpr (KIND == kAreas)
    if (solid_region<RX, RY>(g, tg)) return;
  unsigned lm = 0;
  T fu[9], fv[9], fw[9], rec[5], lag[2] = {T(0), T(0)}, c = T(0);
  const T* in = a.rec;
  if (WALLS && !links<kRows<RY>, A>(g, n, lm)) return;
  if (kRows<RY> && WALLS && (lm & 1u)) return;
  pull_species<A, FIRST>(g, n, m.u, a.src, a.du0, fu);
  pull_species<A, FIRST>(g, n, m.v, a.src + 9 * g.plane, a.dv0, fv);
  if (W3)
    pull_species<A, FIRST>(g, n, m.w, a.src + 18 * g.plane, static_cast<const T*>(nullptr), fw);
  load_record<A, VAR, kRows<RY>>(g, n, in, rec);
  if (a.dc) c = *own_at<A>(a.dc, n);
  if (LAG && !FIRST) {
    lag[0] = *own_at<A>(a.dlag, n);
    lag[1] = *own_at<A>(a.dlag + g.plane, n);
  }
  const Steps st = steps_of(tg);
  const int row = first_row<RX, RY>();
  if (WALLS && !kRows<RY> && st.count > 1) lm = links_inside<RX, RY>(lm);
  int s = 0;
  if (FIRST) {
    tlm_collide<T, VAR>(m, fu, fv, fw, c, rec, lag, true);
    if (!kRows<RY> && tg.steps > 1) {
      in = scalar(in + a.rec_stride);
      load_record<A, VAR, kRows<RY>>(g, n, in, rec);
      give<WALLS, false>(lds, fu, fv, fw, lm);
      if (!live_rows<RX, RY>(st, 1, row)) return void(retire(st, 0));
      take<false>(lds, fu, fv, fw);
    }
    s = 1;
  }
  for (; s < tg.steps; ++s) {
    tlm_collide<T, VAR>(m, fu, fv, fw, c, rec, lag, false);
    if (kRows<RY> || s + 1 == tg.steps) break;
    in = scalar(in + a.rec_stride);
    load_record<A, VAR, kRows<RY>>(g, n, in, rec);
    give<WALLS, false>(lds, fu, fv, fw, lm);
    if (!live_rows<RX, RY>(st, s + 1, row)) return void(retire(st, s));
    take<false>(lds, fu, fv, fw);
  }
  if (!node_again<RX, RY>(g, tg, n) || (WALLS && (lm & 1u))) return;
  if (LAG) {
    *own_at<A>(a.dlag_out, n) = lag[0];
    *own_at<A>(a.dlag_out + g.plane, n) = lag[1];
  }
  store_species<A, WALLS, false, kRows<RY>>(g, n, fu, a.dst, lm);
  store_species<A, WALLS, false, kRows<RY>>(g, n, fv, a.dst + 9 * g.plane, lm);
  if (W3) store_species<A, WALLS, false, kRows<RY>>(g, n, fw, a.dst + 18 * g.plane, lm);
}

// Continuous-adjoint steps: pull the adjoint populations (or, at the first
// reversed step, p = seed_u at equilibrium and q = 0) and collide with the
// records of the forward steps n, n - 1, ... at those times.
template <typename T, int KIND, int RX, int RY, bool FIRST>
__global__ MRT_REGION_BOUNDS(T, kVarFirst, RX, RY) void cadj_kernel(Geometry g, ModelCoef<T> m,
                                                         CadjCoef<T> cc, CadjLaunch<T> a,
                                                         TileGrid tg) {
  constexpr bool WALLS = KIND != kOpen;
  constexpr Lanes A = lanes_of<RX, RY>;
  __shared__ Exchange<T, RX, RY, false> lds;
  const RegionNode r = region_node<RX, RY>(g, tg, threadIdx.x);
  if (kRows<RY> && !r.owner) return;
  NodeIdx n;
  make_node(g, r.x, r.y, n);
  unsigned lm = 0;
  T fp[9], fq[9], rec[5];
  double sum = 0.0;
  const T* in = a.rec;
  if constexpr (KIND == kAreas)
    if (solid_region<RX, RY>(g, tg)) {
      if (FIRST && r.owner) *own_at<A>(a.g, n) = 0.0;
      return;
    }
  if (WALLS && !links<kRows<RY> && !FIRST, A>(g, n, lm)) return;
  if (kRows<RY> && WALLS && !FIRST && (lm & 1u)) return;
  pull_species<A, FIRST>(g, n, m.u, a.src, a.seed_u, fp);
  pull_species<A, FIRST>(g, n, m.v, a.src + 9 * g.plane, static_cast<const T*>(nullptr), fq);
  load_record<A, kVarFirst, kRows<RY>>(g, n, in, rec);
  if (r.owner && !FIRST) sum = *own_at<A>(a.g, n);
  // as the loop of several steps, which carries its populations, sees them
  if (FIRST && kRows<RY>) keep_rounded<false>(fp, fq, static_cast<T*>(nullptr));
  const Steps st = steps_of(tg);
  const int row = first_row<RX, RY>();
  if (WALLS && !kRows<RY> && st.count > 1) lm = links_inside<RX, RY>(lm);
  for (int s = 0;; ++s) {
    sum += double(cadj_collide<T>(m, cc, fp, fq, rec));
    if (kRows<RY> || s + 1 == tg.steps) break;
    in = scalar(in - a.rec_stride);
    load_record<A, kVarFirst, kRows<RY>>(g, n, in, rec);
    give<WALLS, false>(lds, fp, fq, static_cast<T*>(nullptr), lm);
    if (!live_rows<RX, RY>(st, s + 1, row)) return void(retire(st, s));
    take<false>(lds, fp, fq, static_cast<T*>(nullptr));
  }
  if (!node_again<RX, RY>(g, tg, n)) return;
  if (WALLS && (lm & 1u)) {
    if (FIRST) *own_at<A>(a.g, n) = 0.0;
    return;
  }
  *own_at<A>(a.g, n) = sum;
  store_species<A, WALLS, false, kRows<RY>>(g, n, fp, a.dst, lm);
  store_species<A, WALLS, false, kRows<RY>>(g, n, fq, a.dst + 9 * g.plane, lm);
}

// Fluid test on the tape's link word (bit 0 = solid) or, for the calls that
// take no tape, on the caller's byte mask (non-zero = solid).  Null: all fluid.
__device__ __forceinline__ bool is_fluid(const uint16_t* link, size_t idx) {
  return link == nullptr || !(link[idx] & 1u);
}
__device__ __forceinline__ bool is_fluid(const uint8_t* mask, size_t idx) {
  return mask == nullptr || mask[idx] == 0;
}

template <typename T, typename M>
__global__ __launch_bounds__(kBlock) void cost_grad_kernel(
    Geometry g, const M* __restrict__ link, const T* __restrict__ uN, const T* __restrict__ ut,
    const T* __restrict__ ctrl, const double* __restrict__ gacc, T* __restrict__ seed,
    T* __restrict__ grad, double alpha, double* __restrict__ partials) {
  double acc[kRedSlots] = {0.0, 0.0, 0.0, 0.0, 0.0};
  const size_t total = size_t(g.nx) * g.ny;
  for (size_t k = size_t(blockIdx.x) * kBlock + threadIdx.x; k < total;
       k += size_t(gridDim.x) * kBlock) {
    const size_t y = k / g.nx, x = k % g.nx;
    const size_t idx = y * g.pitch + x;
    const bool fl = is_fluid(link, idx);
    double d = 0.0, cc = 0.0, e = 0.0;
    if (fl) {
      d = double(uN[idx]) - double(ut[idx]);
      cc = double(ctrl[idx]);
      acc[0] += 0.5 * d * d;
      acc[1] += 0.5 * alpha * cc * cc;
      if (!isfinite(d) || !isfinite(cc)) acc[4] += 1.0;
    }
    if (seed) seed[idx] = fl ? T(d) : T(0);
    if (gacc) {
      if (fl) {
        e = gacc[idx] + alpha * cc;
        acc[2] += e * e;
        acc[3] = fmax(acc[3], fabs(e));
        if (!isfinite(e)) acc[4] += 1.0;
      }
      grad[idx] = fl ? T(e) : T(0);
    }
  }
  block_reduce_store(acc, partials + size_t(blockIdx.x) * kRedSlots);
}

__global__ __launch_bounds__(kBlock) void finish_reduce_kernel(
    const double* __restrict__ partials, int nblocks,
    double* __restrict__ result) {
  double acc[kRedSlots] = {0.0, 0.0, 0.0, 0.0, 0.0};
  for (int b = threadIdx.x; b < nblocks; b += kBlock) {
#pragma unroll
    for (int k = 0; k < kRedSlots; ++k) {
      double v = partials[size_t(b) * kRedSlots + k];
      acc[k] = (k == 3) ? fmax(acc[k], v) : acc[k] + v;
    }
  }
  block_reduce_store(acc, result);
}

template <typename T>
__global__ __launch_bounds__(kBlock) void grad_max_kernel(
    Geometry g, const T* __restrict__ grad, double* __restrict__ partials) {
  const uint16_t* link = g.link;
  double acc[kRedSlots] = {0.0, 0.0, 0.0, 0.0, 0.0};
  const size_t total = size_t(g.nx) * g.ny;
  for (size_t k = size_t(blockIdx.x) * kBlock + threadIdx.x; k < total;
       k += size_t(gridDim.x) * kBlock) {
    const size_t y = k / g.nx, x = k % g.nx;
    const size_t idx = y * g.pitch + x;
    if (is_fluid(link, idx)) {
      const double e = double(grad[idx]);
      acc[3] = fmax(acc[3], fabs(e));
      if (!isfinite(e)) acc[4] += 1.0;
    }
  }
  block_reduce_store(acc, partials + size_t(blockIdx.x) * kRedSlots);
}

// zeta > 0: fixed step; zeta <= 0: heuristic min(1, 1/||E||_inf) from the
// reduced maximum in result[3] (written by grad_max_kernel on the device).
template <typename T>
__global__ __launch_bounds__(kBlock) void gd_update_kernel(
    Geometry g, T* __restrict__ ctrl, const T* __restrict__ grad, double zeta,
    double lo, double hi, double* __restrict__ result) {
  const uint16_t* link = g.link;
  double z = zeta;
  if (z <= 0.0) {
    const double emax = result[3];
    z = emax > 0.0 ? fmin(1.0, 1.0 / emax) : 1.0;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) result[kRedSlots] = z;
  const size_t total = size_t(g.nx) * g.ny;
  for (size_t k = size_t(blockIdx.x) * kBlock + threadIdx.x; k < total;
       k += size_t(gridDim.x) * kBlock) {
    const size_t y = k / g.nx, x = k % g.nx;
    const size_t idx = y * g.pitch + x;
    if (!is_fluid(link, idx)) continue;
    double c = double(ctrl[idx]) - z * double(grad[idx]);
    c = fmin(fmax(c, lo), hi);
    ctrl[idx] = T(c);
  }
}

// Partial sums of x . y over the fluid nodes (slot 0), non-finite count
// (slot 4).
template <typename T>
__global__ __launch_bounds__(kBlock) void dot_kernel(Geometry g, const T* __restrict__ x,
                                                     const T* __restrict__ y,
                                                     double* __restrict__ partials) {
  const uint16_t* link = g.link;
  double acc[kRedSlots] = {0.0, 0.0, 0.0, 0.0, 0.0};
  const size_t total = size_t(g.nx) * g.ny;
  for (size_t k = size_t(blockIdx.x) * kBlock + threadIdx.x; k < total;
       k += size_t(gridDim.x) * kBlock) {
    const size_t yy = k / g.nx, xx = k % g.nx;
    const size_t idx = yy * g.pitch + xx;
    if (is_fluid(link, idx)) {
      const double v = double(x[idx]) * double(y[idx]);
      acc[0] += v;
      if (!isfinite(v)) acc[4] += 1.0;
    }
  }
  block_reduce_store(acc, partials + size_t(blockIdx.x) * kRedSlots);
}

// Up to four inner products over the fluid nodes in one pass, each summed
// in the order of dot_kernel (so each equals that kernel's result bit for
// bit): products k = 0, 1, 2, 3 go to slots 0, 1, 2, 4; slot 3 (a maximum)
// flags a non-finite product.
template <typename T>
__global__ __launch_bounds__(kBlock) void dots_kernel(Geometry g, DotPairs<T> d,
                                                      double* __restrict__ partials) {
  const uint16_t* link = g.link;
  double acc[kRedSlots] = {0.0, 0.0, 0.0, 0.0, 0.0};
  const size_t total = size_t(g.nx) * g.ny;
  for (size_t k = size_t(blockIdx.x) * kBlock + threadIdx.x; k < total;
       k += size_t(gridDim.x) * kBlock) {
    const size_t yy = k / g.nx, xx = k % g.nx;
    const size_t idx = yy * g.pitch + xx;
    if (is_fluid(link, idx)) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (j < d.n) {
          const double v = double(d.a[j][idx]) * double(d.b[j][idx]);
          acc[j < 3 ? j : 4] += v;
          if (!isfinite(v)) acc[3] = 1.0;
        }
      }
    }
  }
  block_reduce_store(acc, partials + size_t(blockIdx.x) * kRedSlots);
}

// y <- a x + b y on the fluid nodes, 0 on the solid ones.
template <typename T>
__global__ __launch_bounds__(kBlock) void axpby_kernel(Geometry g, const T* __restrict__ x,
                                                       T* __restrict__ y, double a,
                                                       double b) {
  const uint16_t* link = g.link;
  const size_t total = size_t(g.nx) * g.ny;
  for (size_t k = size_t(blockIdx.x) * kBlock + threadIdx.x; k < total;
       k += size_t(gridDim.x) * kBlock) {
    const size_t yy = k / g.nx, xx = k % g.nx;
    const size_t idx = yy * g.pitch + xx;
    y[idx] = is_fluid(link, idx) ? T(a * double(x[idx]) + b * double(y[idx])) : T(0);
  }
}

template <typename M>
__global__ __launch_bounds__(kBlock) void count_fluid_kernel(
    Geometry g, const M* __restrict__ link, double* __restrict__ partials) {
  double acc[kRedSlots] = {0.0, 0.0, 0.0, 0.0, 0.0};
  const size_t total = size_t(g.nx) * g.ny;
  for (size_t k = size_t(blockIdx.x) * kBlock + threadIdx.x; k < total;
       k += size_t(gridDim.x) * kBlock) {
    const size_t y = k / g.nx, x = k % g.nx;
    if (is_fluid(link, y * g.pitch + x)) acc[0] += 1.0;
  }
  if (g.wflag)
    for (size_t k = size_t(blockIdx.x) * kBlock + threadIdx.x; k < size_t(g.nsx) * g.ny;
         k += size_t(gridDim.x) * kBlock)
      if (g.wflag[k] == 2u) acc[1] += 1.0;
  block_reduce_store(acc, partials + size_t(blockIdx.x) * kRedSlots);
}

int stencil_blocks(const Geometry& g) {
  return ((g.nx + kBlock - 1) / kBlock) * g.ny;
}

}  // namespace

// ----------------------------------------------------------- launchers

void launch_build_link(const Geometry& g, int periodic, const uint8_t* mask,
                       uint16_t* link_out, uint32_t* wflag_out, hipStream_t s) {
  dim3 grid((g.nx + kBlock - 1) / kBlock, g.ny);
  hipLaunchKernelGGL(build_link_kernel, grid, dim3(kBlock), 0, s, g, periodic,
                     mask, link_out, wflag_out);
}

namespace {

TileGrid region_grid(const Geometry& g, const StepPlan& p) {
  TileGrid t;
  t.steps = p.steps;
  const int wx = p.rx - 2 * (p.steps - 1), wy = p.ry - 2 * (p.steps - 1);
  t.ntx = (g.nx + wx - 1) / wx;
  t.inv_ntx = 0xFFFFFFFFu / unsigned(t.ntx);
  t.ntiles = t.ntx * ((g.ny + wy - 1) / wy);
  return t;
}

// Calls f(integral constants kind of walls, region width, region height) for a
// lattice and a plan.
template <typename T, int VAR, typename F>
void dispatch_region(const Geometry& g, const StepPlan& p, F f) {
  using std::integral_constant;
  auto shape = [&](auto K) {
    if (p.rx == 16) return f(K, integral_constant<int, 16>(), integral_constant<int, 16>());
    if constexpr (kWide<T, VAR>) {
      f(K, integral_constant<int, 32>(), integral_constant<int, 16>());
    } else {
      if (p.ry == 32) return f(K, integral_constant<int, 32>(), integral_constant<int, 32>());
      f(K, integral_constant<int, 64>(), integral_constant<int, 16>());
    }
  };
  auto rows = [&](auto K) {
    f(K, integral_constant<int, 256>(), integral_constant<int, 1>());
  };
  const integral_constant<int, kOpen> open;
  const integral_constant<int, kWalls> walls;
  if (!g.masked && g.periodic)
    p.ry == 1 ? rows(open) : shape(open);
  else if (p.ry == 1)
    rows(walls);
  else if (g.solid_areas)
    shape(integral_constant<int, kAreas>());
  else
    shape(walls);
}

// Calls f(integral constant variant).
template <typename F>
void dispatch_variant(int variant, F f) {
  using std::integral_constant;
  if (variant == kVarExplicit)
    f(integral_constant<int, kVarExplicit>());
  else if (variant == kVarImplicit)
    f(integral_constant<int, kVarImplicit>());
  else if (variant == kVarThree)
    f(integral_constant<int, kVarThree>());
  else
    f(integral_constant<int, kVarFirst>());
}

}  // namespace

// A launch costs about 5 us beside its steps (the gather, the stores and the
// gap before it), every further step costs a ring of each region, and the time
// of a small lattice goes up in whole rounds of regions: with up to 256 of them
// each has a compute unit to itself, with up to 512 two share one.  (The counts
// are of a whole device; in a partition of fewer compute units the plan is as
// right, its rounds only more.)  So: the most steps whose regions fit one round
// of 256, or else of 512, as long as the rings leave enough of a region; and 5
// for the large lattices, between memory (fewer) and the rings (more).
// Of the shapes, 16 x 16 spreads the smallest lattices over the chip; 64 x 16,
// whose rows are scalar addresses, has the shortest steps; 32 x 32 owns more of
// its nodes (with 5 steps 56% instead of 44%).  Measured in us per forward step,
// FP32, steps per launch in brackets:
//            64 x 16                                      32 x 32
//   2048^2   64.2 (3)  57.0 (4)  51.2 (5)  57.2 (6)       61.4 (4)  50.9 (5)  53.2 (6)
//            54.7 (5) the AMRT step                       52.7 (5)
//   1024^2   12.8 (3)  13.9 (4)  12.2 (5)  13.8 (6)       12.8 (4)  11.8 (5)  12.3 (6)
//    512^2    4.7 (3)   4.2 (4)   4.7 (5)   4.9 (6)        4.4 (4)   3.8 (5)   4.6 (6)
//    400^2    3.5 (3)   3.8 (4)   3.3 (5)   3.7 (6)        3.2 (4)   3.3 (6)   3.1 (7)
//    300^2    2.9 (3)   2.6 (4)   2.4 (5)   2.8 (6)        2.4 (6)   2.3 (7)   2.7 (9)
//    256^2    2.7 (4)   2.4 (5)   2.2 (6)   2.5 (7)        2.3 (8)   2.1 (9)   2.6 (10)
//    200^2    2.2 (5)   1.9 (6)   1.75 (7)                 1.9 (9)   1.8 (10)
//  301x157    2.1 (5)   1.9 (6)   1.8 (7)                  2.0 (9)   2.4 (10)
//            16 x 16
//    128^2    1.8 (4)   1.6 (5)   1.7 (6)  (64 x 16: 2.0 (6), 1.9 (7))
//     64^2    1.9 (4)   1.6 (5)   1.4 (7)  (64 x 16: 1.8 (7))
// The regions of wide nodes are 32 x 16: 1024^2, FP64, 30.4 (4) and 28.7 (5);
// 32 x 32, which leaves one of them to a compute unit, 34.7 (5).
//
// Low lattices of many columns: a region has nodes of a row several times over.
// 64 x 16 regions are taken where they are fewer than 32 x 32, and one step a
// launch in rows of 256 nodes where the regions take more than one round (wide
// nodes: two) and compute over eight times the nodes that the rows do (4.5 times
// with three species in FP64, of which a compute unit holds one region).  A
// forward step in us, 32 x 32 (FP64: 32 x 16), 64 x 16 and rows:
//   32768 x 1   7.8   -    3.7      FP64   7.1  4.5     three species, FP64   -    6.1
//   32768 x 2   7.8   -    4.9             7.3  7.0                           -    9.4
//   32768 x 4   8.1  4.7   6.4             7.8  9.8                         15.8  11.9
//   32768 x 8   8.9  5.0   9.6             8.2 17.1                         31.4  30.3 (x 9)
//
// A step by itself (an interval of one step, a sweep of one) exchanges nothing,
// and rows of 256 nodes take it faster: whole chunks of non-temporal stores, and
// small work-groups, which leave solid segments at once.  In us a forward step
// checkpointed at every step, regions and rows: 2048^2 134 and 114, FP64 259 and
// 233; 1024^2 FP64 65 and 60; 256^2 5.6 and 4.2.  Only where rows need more than
// one round of eight work-groups a compute unit and compute more than four times
// (wide nodes: eight times) the nodes of the regions do they lose: 16 x 32768 30
// and 34, FP64 41 and 54; not 24 x 32768 in FP64, the AMRT step 143 and 129.
StepPlan plan_steps(const Geometry& g, size_t elem, int variant, int left, bool one) {
  constexpr StepPlan kRowPlan = {256, 1, 1};
  if (one) return kRowPlan;
  StepPlan p;
  // the most steps, from `most` down to `least`, whose regions are at most n
  auto fits = [&](int rx, int ry, int most, int least, int n) {
    for (p = {rx, ry, most}; p.steps >= least; --p.steps)
      if (region_grid(g, p).ntiles <= n) return true;
    return false;
  };
  // 2^29 elements (of which a lattice of few nodes may have as many, its rows
  // lying far apart): the FP64 accumulator is addressed with the FP32 fields
  const bool small = g.plane * kWidestElement < (size_t(1) << 32);
  const bool wide = elem == 8 || variant == kVarThree;
  bool large = false;  // more than a round or two of regions
  if (!small || !fits(16, 16, 7, 4, 256)) {
    if (wide) {
      large = !fits(32, 16, 7, 6, 256) && !fits(32, 16, 5, 4, 512);
      if (large) p = {32, 16, 5};
    } else if (!fits(64, 16, 7, 7, 256)) {
      large = !small || (!fits(32, 32, 10, 5, 256) && !fits(32, 32, 10, 4, 512));
      if (large) {
        const StepPlan low = {64, 16, 5};
        p = {32, 32, 5};
        if (!small || region_grid(g, low).ntiles < region_grid(g, p).ntiles) p = low;
      }
    }
  }
  if (large) {
    const bool widest = elem == 8 && variant == kVarThree;
    const size_t n = region_grid(g, p).ntiles, nodes = n * p.rx * p.ry;
    if (n > (wide ? 1024 : 512) &&
        nodes > (widest ? 9 : 16) * size_t(region_grid(g, kRowPlan).ntiles) * 128)
      return kRowPlan;
  }
  // as many launches as that takes, their steps spread evenly
  const int launches = (left + p.steps - 1) / p.steps;
  p.steps = (left + launches - 1) / launches;
  if (p.steps == 1) {
    const int n = region_grid(g, kRowPlan).ntiles;
    const size_t most = (wide ? 8 : 4) * size_t(region_grid(g, p).ntiles) * p.rx * p.ry;
    if (n <= 8 * 256 || size_t(n) * 256 <= most) return kRowPlan;
  }
  return p;
}

template <typename T>
void launch_forward(const Geometry& g, const ModelCoef<T>& m, const FwdLaunch<T>& a,
                    const StepPlan& p, hipStream_t s) {
  const TileGrid t = region_grid(g, p);
  dispatch_variant(a.variant, [&](auto V) {
    dispatch_region<T, V()>(g, p, [&](auto W, auto RX, auto RY) {
      if (a.src)
        hipLaunchKernelGGL((forward_kernel<T, W(), V(), RX(), RY(), false>), dim3(t.ntiles),
                           dim3(RX() * RY()), 0, s, g, m, a, t);
      else
        hipLaunchKernelGGL((forward_kernel<T, W(), V(), RX(), RY(), true>), dim3(t.ntiles),
                           dim3(RX() * RY()), 0, s, g, m, a, t);
    });
  });
}

template <typename T>
void launch_finalize(const Geometry& g, const T* src, T* state, T* uN, T* vN,
                     hipStream_t s, const ModelCoef<T>* m, const T* ctrl, bool three) {
  const int nb = stencil_blocks(g);
  const bool impl = m != nullptr;
  const ModelCoef<T> mc = impl ? *m : ModelCoef<T>{};
  auto fin = [&](auto I, auto W) {
    hipLaunchKernelGGL((finalize_kernel<T, I(), W()>), dim3(nb), dim3(kBlock), 0, s, g, mc, src,
                       ctrl, state, uN, vN);
  };
  if (impl)
    fin(std::true_type(), std::false_type());
  else if (three)
    fin(std::false_type(), std::true_type());
  else
    fin(std::false_type(), std::false_type());
}

template <typename T>
void launch_implicit_terminal(const Geometry& g, const ModelCoef<T>& m, const T* src,
                              const T* ctrl, const T* seed_u, const T* seed_v, T* out_u,
                              T* out_v, double* gacc, hipStream_t s) {
  const int nb = stencil_blocks(g);
  hipLaunchKernelGGL((implicit_terminal_kernel<T>), dim3(nb), dim3(kBlock), 0, s, g, m, src, ctrl,
                     seed_u, seed_v, out_u, out_v, gacc);
}

template <typename T>
void launch_implicit_tlm_final(const Geometry& g, const ModelCoef<T>& m, const T* fsrc,
                               const T* dsrc, const T* ctrl, const T* dc, T* duN, T* dvN,
                               hipStream_t s) {
  const int nb = stencil_blocks(g);
  hipLaunchKernelGGL((implicit_tlm_final_kernel<T>), dim3(nb), dim3(kBlock), 0, s, g, m, fsrc,
                     dsrc, ctrl, dc, duN, dvN);
}

template <typename T>
void launch_adjoint(const Geometry& g, const ModelCoef<T>& m, const AdjLaunch<T>& a,
                    const StepPlan& p, hipStream_t s) {
  const TileGrid t = region_grid(g, p);
  dispatch_variant(a.variant, [&](auto V) {
    dispatch_region<T, V()>(g, p, [&](auto W, auto RX, auto RY) {
      if (a.src)
        hipLaunchKernelGGL((adjoint_kernel<T, W(), V(), RX(), RY(), false>), dim3(t.ntiles),
                           dim3(RX() * RY()), 0, s, g, m, a, t);
      else
        hipLaunchKernelGGL((adjoint_kernel<T, W(), V(), RX(), RY(), true>), dim3(t.ntiles),
                           dim3(RX() * RY()), 0, s, g, m, a, t);
    });
  });
}

template <typename T>
void launch_cost_grad(const Geometry& g, const T* uN, const T* ut,
                      const T* ctrl, const double* gacc, T* seed, T* grad,
                      double alpha, double* partials, double* result,
                      hipStream_t s) {
  hipLaunchKernelGGL((cost_grad_kernel<T, uint16_t>), dim3(kRedBlocks), dim3(kBlock), 0,
                     s, g, g.link, uN, ut, ctrl, gacc, seed, grad, alpha,
                     partials);
  hipLaunchKernelGGL(finish_reduce_kernel, dim3(1), dim3(kBlock), 0, s,
                     partials, kRedBlocks, result);
}

// ---- cost and gradient reduction without a tape or any allocation
//
// The block partials and the two reduced rows live in this file-scope array,
// one copy per device for the life of the process.  Host code never passes
// the array's name to a kernel (on the host it is only a stand-in symbol):
// the device address is looked up once per device with hipGetSymbolAddress
// and that pointer is what the kernels receive.  Every block overwrites its
// partial row and the finishing kernel its result row, so nothing needs
// clearing between calls; two calls that overlap on one device share the
// array and race.
static __device__ __align__(256) double scratch[kNoallocScratchDoubles];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
double* g_scratch_ptr[kMaxDevices] = {};

hipError_t scratch_address(double** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch_ptr[dev] = static_cast<double*>(ptr);
  }
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}
}  // namespace

template <typename T>
hipError_t launch_cost_grad_noalloc(const Geometry& g, const uint8_t* mask, const T* uN,
                                    const T* ut, const T* ctrl, const double* gacc, T* seed,
                                    T* grad, double alpha, double* host_out, hipStream_t s) {
  double* base = nullptr;
  hipError_t e = scratch_address(&base);
  if (e != hipSuccess) return e;
  double* partials = base;
  double* result = base + size_t(kRedBlocks) * kRedSlots;  // [2][kRedSlots]
  hipLaunchKernelGGL((cost_grad_kernel<T, uint8_t>), dim3(kRedBlocks), dim3(kBlock), 0,
                     s, g, mask, uN, ut, ctrl, gacc, seed, grad, alpha, partials);
  hipLaunchKernelGGL(finish_reduce_kernel, dim3(1), dim3(kBlock), 0, s,
                     partials, kRedBlocks, result);
  hipLaunchKernelGGL((count_fluid_kernel<uint8_t>), dim3(kRedBlocks), dim3(kBlock), 0, s,
                     g, mask, partials);
  hipLaunchKernelGGL(finish_reduce_kernel, dim3(1), dim3(kBlock), 0, s,
                     partials, kRedBlocks, result + kRedSlots);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  e = hipMemcpyAsync(host_out, result, sizeof(double) * 2 * kRedSlots,
                     hipMemcpyDeviceToHost, s);
  if (e != hipSuccess) return e;
  return hipStreamSynchronize(s);
}

template <typename T>
void launch_gd_step(const Geometry& g, T* ctrl, const T* grad, double zeta,
                    double lo, double hi, double* partials, double* result,
                    hipStream_t s) {
  if (zeta <= 0.0) {
    hipLaunchKernelGGL((grad_max_kernel<T>), dim3(kRedBlocks), dim3(kBlock), 0,
                       s, g, grad, partials);
    hipLaunchKernelGGL(finish_reduce_kernel, dim3(1), dim3(kBlock), 0, s,
                       partials, kRedBlocks, result);
  }
  hipLaunchKernelGGL((gd_update_kernel<T>), dim3(kRedBlocks), dim3(kBlock), 0,
                     s, g, ctrl, grad, zeta, lo, hi, result);
}

template <typename T>
void launch_tlm(const Geometry& g, const ModelCoef<T>& m, const TlmLaunch<T>& a,
                const StepPlan& p, hipStream_t s) {
  const TileGrid t = region_grid(g, p);
  dispatch_variant(a.variant, [&](auto V) {
    dispatch_region<T, V()>(g, p, [&](auto W, auto RX, auto RY) {
      if (a.src)
        hipLaunchKernelGGL((tlm_kernel<T, W(), V(), RX(), RY(), false>), dim3(t.ntiles),
                           dim3(RX() * RY()), 0, s, g, m, a, t);
      else
        hipLaunchKernelGGL((tlm_kernel<T, W(), V(), RX(), RY(), true>), dim3(t.ntiles),
                           dim3(RX() * RY()), 0, s, g, m, a, t);
    });
  });
}

template <typename T>
void launch_cadj(const Geometry& g, const ModelCoef<T>& m, const CadjCoef<T>& cc,
                 const CadjLaunch<T>& a, const StepPlan& p, hipStream_t s) {
  const TileGrid t = region_grid(g, p);
  dispatch_region<T, kVarFirst>(g, p, [&](auto W, auto RX, auto RY) {
    if (a.src)
      hipLaunchKernelGGL((cadj_kernel<T, W(), RX(), RY(), false>), dim3(t.ntiles),
                         dim3(RX() * RY()), 0, s, g, m, cc, a, t);
    else
      hipLaunchKernelGGL((cadj_kernel<T, W(), RX(), RY(), true>), dim3(t.ntiles),
                         dim3(RX() * RY()), 0, s, g, m, cc, a, t);
  });
}

template <typename T>
void launch_dot(const Geometry& g, const T* x, const T* y, double* partials, double* result,
                hipStream_t s) {
  hipLaunchKernelGGL((dot_kernel<T>), dim3(kRedBlocks), dim3(kBlock), 0, s, g, x, y,
                     partials);
  hipLaunchKernelGGL(finish_reduce_kernel, dim3(1), dim3(kBlock), 0, s, partials, kRedBlocks,
                     result);
}

template <typename T>
void launch_dots(const Geometry& g, const DotPairs<T>& d, double* partials, double* result,
                 hipStream_t s) {
  hipLaunchKernelGGL((dots_kernel<T>), dim3(kRedBlocks), dim3(kBlock), 0, s, g, d, partials);
  hipLaunchKernelGGL(finish_reduce_kernel, dim3(1), dim3(kBlock), 0, s, partials, kRedBlocks,
                     result);
}

template <typename T>
void launch_axpby(const Geometry& g, const T* x, T* y, double a, double b, hipStream_t s) {
  hipLaunchKernelGGL((axpby_kernel<T>), dim3(kRedBlocks), dim3(kBlock), 0, s, g, x, y, a, b);
}

void launch_count_fluid(const Geometry& g, double* partials, double* result,
                        hipStream_t s) {
  hipLaunchKernelGGL((count_fluid_kernel<uint16_t>), dim3(kRedBlocks), dim3(kBlock), 0, s,
                     g, g.link, partials);
  hipLaunchKernelGGL(finish_reduce_kernel, dim3(1), dim3(kBlock), 0, s,
                     partials, kRedBlocks, result);
}

#define MRT_INSTANTIATE(T)                                                   \
  template void launch_dots<T>(const Geometry&, const DotPairs<T>&, double*, double*,  \
                               hipStream_t);                                          \
  template void launch_forward<T>(const Geometry&, const ModelCoef<T>&,      \
                                  const FwdLaunch<T>&, const StepPlan&,      \
                                  hipStream_t);                              \
  template void launch_finalize<T>(const Geometry&, const T*, T*, T*, T*,    \
                                   hipStream_t, const ModelCoef<T>*,         \
                                   const T*, bool);                          \
  template void launch_implicit_terminal<T>(const Geometry&,                 \
                                            const ModelCoef<T>&, const T*,   \
                                            const T*, const T*, const T*,    \
                                            T*, T*, double*, hipStream_t);   \
  template void launch_implicit_tlm_final<T>(const Geometry&,                \
                                             const ModelCoef<T>&, const T*,  \
                                             const T*, const T*, const T*,   \
                                             T*, T*, hipStream_t);           \
  template void launch_adjoint<T>(const Geometry&, const ModelCoef<T>&,      \
                                  const AdjLaunch<T>&, const StepPlan&,      \
                                  hipStream_t);                              \
  template void launch_cost_grad<T>(const Geometry&, const T*, const T*,    \
                                    const T*, const double*, T*, T*, double, \
                                    double*, double*, hipStream_t);          \
  template hipError_t launch_cost_grad_noalloc<T>(                           \
      const Geometry&, const uint8_t*, const T*, const T*, const T*,         \
      const double*, T*, T*, double, double*, hipStream_t);                  \
  template void launch_gd_step<T>(const Geometry&, T*, const T*, double,     \
                                  double, double, double*, double*,          \
                                  hipStream_t);                              \
  template void launch_cadj<T>(const Geometry&, const ModelCoef<T>&,         \
                               const CadjCoef<T>&, const CadjLaunch<T>&,      \
                               const StepPlan&, hipStream_t);                \
  template void launch_tlm<T>(const Geometry&, const ModelCoef<T>&,          \
                              const TlmLaunch<T>&, const StepPlan&,          \
                              hipStream_t);                                  \
  template void launch_dot<T>(const Geometry&, const T*, const T*, double*,  \
                              double*, hipStream_t);                         \
  template void launch_axpby<T>(const Geometry&, const T*, T*, double,       \
                                double, hipStream_t);
MRT_INSTANTIATE(float)
MRT_INSTANTIATE(double)
#undef MRT_INSTANTIATE

}  // namespace mrt
