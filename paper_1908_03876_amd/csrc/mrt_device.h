// Per-node device code of the two- and three-species D2Q9 MRT step and of
// its exact discrete adjoint (AMRT), shared by the single-lattice kernels
// and the batched persistent kernels.
//
// Method: arXiv:1908.03876, Section 3.1 (eq:LBE, S, PhiS, MF, MC, phieq,
// BC11, the relaxation matrix Pi and D = d Cs^2 tau (K^-1 - I/2)) and
// Section 3.2.1 (LIBEG, CAE, AEDs, RFS1, CAEL, gradientLattice).
#pragma once

#include <hip/hip_runtime.h>

#include "mrt_internal.h"

namespace mrt {
namespace dev {

constexpr int kBlock = 256;
constexpr int kXcds = 8;

// D2Q9 opposite directions: e3 = -e1, e4 = -e2, e7 = -e5, e8 = -e6.
__device__ __forceinline__ constexpr int opp(int i) {
  return i == 0 ? 0 : (i <= 4 ? ((i + 1) & 3) + 1 : ((i - 3) & 3) + 5);
}

// Linear work-group id -> tile id such that XCD k (ids = k mod 8) owns the
// contiguous tile range [k*n/8, (k+1)*n/8).
__device__ __forceinline__ int xcd_tile(int id, int n) {
  const int per = n / kXcds, rem = n % kXcds;
  const int xcd = id % kXcds, k = id / kXcds;
  // the first `rem` XCDs own per+1 tiles
  const int base = xcd * per + (xcd < rem ? xcd : rem);
  return base + k;
}

struct NodeIdx {
  int x, y;
  int xm, xp;        // x - 1, x + 1 with periodic wrap
  size_t r0, rm, rp; // row offsets of y, y - 1, y + 1 with wrap
  bool ex0, ex1;     // x == 0, x == nx - 1
  bool ey0, ey1;     // y == 0, y == ny - 1
};

// Neighbour bookkeeping of node (x, y) of a lattice.
__device__ __forceinline__ void make_node(const Geometry& g, int x, int y,
                                          NodeIdx& n) {
  n.x = x;
  n.y = y;
  n.ex0 = n.x == 0;
  n.ex1 = n.x + 1 == g.nx;
  n.ey0 = n.y == 0;
  n.ey1 = n.y + 1 == g.ny;
  n.xm = n.ex0 ? g.nx - 1 : n.x - 1;
  n.xp = n.ex1 ? 0 : n.x + 1;
  const int ym = n.ey0 ? g.ny - 1 : n.y - 1;
  const int yp = n.ey1 ? 0 : n.y + 1;
  n.r0 = size_t(n.y) * g.pitch;
  n.rm = size_t(ym) * g.pitch;
  n.rp = size_t(yp) * g.pitch;
}

// Node of this thread in the single-lattice kernels: 256-node row tiles,
// XCD-banded (each of the 8 XCDs owns a contiguous range of tiles).
__device__ __forceinline__ bool node_of_block(const Geometry& g, NodeIdx& n) {
  const int nbx = (g.nx + kBlock - 1) / kBlock;
  const int ntiles = nbx * g.ny;
  const int id = blockIdx.x;
  if (id >= ntiles) return false;
  // the id -> tile map is a bijection on [0, ntiles) because ids are dealt
  // round-robin to XCDs
  const int t = xcd_tile(id, ntiles);
  const int x = (t % nbx) * kBlock + threadIdx.x;
  if (x >= g.nx) return false;
  make_node(g, x, t / nbx, n);
  return true;
}

// Per-wavefront wall flag (64 consecutive nodes of a row, one scalar load):
// 0 = the nodes and their neighbours are all fluid, 1 = mixed, 2 = all
// nodes solid.  Flag-0 wavefronts never read the link mask; in mixed ones
// the link load is independent of the population loads, so it adds no
// latency to them.
__device__ __forceinline__ unsigned wave_flag(const Geometry& g,
                                              const NodeIdx& n) {
  const int seg = __builtin_amdgcn_readfirstlane(n.y * g.nsx + (n.x >> 6));
  return g.wflag[seg];
}

__device__ __forceinline__ unsigned link_of(const Geometry& g, unsigned flag,
                                            size_t idx) {
  return flag ? unsigned(g.link[idx]) : 0u;
}

// How the lanes of a wavefront lie, and so how an element is addressed:
// kRow, one row (a scalar row base and a 32-bit lane offset); kSmall, several
// rows of a plane below 4 GiB, whatever its element (a scalar plane base and a
// 32-bit lane offset); kAny, several rows of any plane (a 64-bit address per
// lane).
enum Lanes { kRow, kSmall, kAny };

template <Lanes A, typename T>
__device__ __forceinline__ T* element(T* plane, size_t row, int col) {
  if (A == kRow)
    return (T*)((char*)(plane + row) + unsigned(col) * unsigned(sizeof(T)));
  if (A == kSmall)
    return (T*)((char*)plane + (unsigned(row) + unsigned(col)) * unsigned(sizeof(T)));
  return plane + row + col;
}

// Element of a plane at node x - e_i for i = 0..8 (periodic wrap).
template <Lanes A, typename T>
__device__ __forceinline__ T* pull_at(T* plane, const NodeIdx& n, int i) {
  switch (i) {
    case 0: return element<A>(plane, n.r0, n.x);
    case 1: return element<A>(plane, n.r0, n.xm);  // e1 = (1,0)
    case 2: return element<A>(plane, n.rm, n.x);   // e2 = (0,1)
    case 3: return element<A>(plane, n.r0, n.xp);  // e3 = (-1,0)
    case 4: return element<A>(plane, n.rp, n.x);   // e4 = (0,-1)
    case 5: return element<A>(plane, n.rm, n.xm);  // e5 = (1,1)
    case 6: return element<A>(plane, n.rm, n.xp);  // e6 = (-1,1)
    case 7: return element<A>(plane, n.rp, n.xp);  // e7 = (-1,-1)
    default: return element<A>(plane, n.rp, n.xm); // e8 = (1,-1)
  }
}

// At node x + e_i = x - e_opp(i).
template <Lanes A, typename T>
__device__ __forceinline__ T* push_at(T* plane, const NodeIdx& n, int i) {
  return pull_at<A>(plane, n, opp(i));
}

// At the node itself.
template <Lanes A, typename T>
__device__ __forceinline__ T* own_at(T* plane, const NodeIdx& n) {
  return element<A>(plane, n.r0, n.x);
}

// Walls.  The pull reads plane i at x - e_i without a test: where that
// neighbour is solid, its (otherwise unused) slot holds the node's own
// reflected population, parked there by the step before; where it lies
// outside a non-periodic lattice, the address wraps to the opposite edge,
// whose population of that direction leaves the lattice and is read by
// nobody, so its slot takes the reflected one.  The adjoint gathers plane i
// at x + e_i in the same way.  A node's link word has bit 0 set if it is
// solid and bit i if x - e_i is solid or outside a non-periodic lattice.

// Is x - e_i outside the lattice (meaningful for non-periodic lattices)?
__device__ __forceinline__ bool pull_outside(const NodeIdx& n, int i) {
  switch (i) {
    case 0: return false;
    case 1: return n.ex0;
    case 2: return n.ey0;
    case 3: return n.ex1;
    case 4: return n.ey1;
    case 5: return n.ex0 || n.ey0;
    case 6: return n.ex1 || n.ey0;
    case 7: return n.ex1 || n.ey1;
    default: return n.ex0 || n.ey1;
  }
}

// Is x + e_i outside the lattice?
__device__ __forceinline__ bool push_outside(const NodeIdx& n, int i) {
  return pull_outside(n, opp(i));
}

// a b + c d with one rounding for a b and the sum and one for c d.  Written
// out where a sum of two products may be contracted either way, so that every
// kernel that contains the expression computes the same bits.
__device__ __forceinline__ float dot2(float a, float b, float c, float d) {
  return __builtin_fmaf(a, b, c * d);
}
__device__ __forceinline__ double dot2(double a, double b, double c, double d) {
  return __builtin_fma(a, b, c * d);
}

// w . f with the lattice weights.
template <typename T>
__device__ __forceinline__ T weighted(const T f[9]) {
  return dot2(T(4.0 / 9.0), f[0], T(1.0 / 9.0), f[1] + f[2] + f[3] + f[4]) +
         T(1.0 / 36.0) * (f[5] + f[6] + f[7] + f[8]);
}

// Relaxation in moment space: f <- f - M0^-1 Pi (M0 f - m_eq(theta)).
// Without the equilibrium (EQ false) and with the K block transposed this is
// f <- f - C^T f (C^T = M0^-1 Pi^T M0 since Pi only couples moments of equal
// row norm), without the conserved zeroth-moment part.  Returns the scaled amounts
// (a1, a2) of the e and epsilon moments for the adjoint equilibrium term.
template <bool EQ, typename T>
__device__ __forceinline__ void relax(T f[9], T theta,
                                      const SpeciesCoef<T>& c, T& a1o,
                                      T& a2o) {
  const T sa = f[1] + f[2] + f[3] + f[4];
  const T sd = f[5] + f[6] + f[7] + f[8];
  const T m1 = T(-4) * f[0] - sa + T(2) * sd;       // e
  const T m2 = T(4) * f[0] - T(2) * sa + sd;        // epsilon
  const T dx = f[5] - f[6] - f[7] + f[8];
  const T dy = f[5] + f[6] - f[7] - f[8];
  const T m3 = f[1] - f[3] + dx;                    // j_x
  const T m4 = T(-2) * (f[1] - f[3]) + dx;          // q_x
  const T m5 = f[2] - f[4] + dy;                    // j_y
  const T m6 = T(-2) * (f[2] - f[4]) + dy;          // q_y
  const T m7 = f[1] - f[2] + f[3] - f[4];           // p_xx
  const T m8 = f[5] - f[6] + f[7] - f[8];           // p_xy
  const T a1 = c.s1 * (EQ ? m1 - c.e_eq * theta : m1);
  const T a2 = c.s2 * (EQ ? m2 - c.eps_eq * theta : m2);
  const T a3 = dot2(c.k00, m3, c.k01, m5);
  const T a5 = dot2(c.k10, m3, c.k11, m5);
  const T a4 = c.s3 * m4;
  const T a6 = c.s4 * m6;
  const T a7 = c.s5 * m7;
  const T a8 = c.s6 * m8;
  const T b = T(2) * a1 + a2;
  const T h = -a1 - T(2) * a2;
  f[0] -= T(4) * (a2 - a1);
  f[1] -= h + a3 - T(2) * a4 + a7;
  f[2] -= h + a5 - T(2) * a6 - a7;
  f[3] -= h - a3 + T(2) * a4 + a7;
  f[4] -= h - a5 + T(2) * a6 - a7;
  f[5] -= b + a3 + a4 + a5 + a6 + a8;
  f[6] -= b - a3 - a4 + a5 + a6 - a8;
  f[7] -= b - a3 - a4 - a5 - a6 + a8;
  f[8] -= b + a3 + a4 - a5 - a6 - a8;
  a1o = a1;
  a2o = a2;
}

// --------------------------------------------------------------- forward

// Pre-collision populations of one species at node n: the pull from its
// planes in src, or (FIRST) the equilibrium initialisation phi_i = w_i
// Theta_0 (phieq, zero flux; a null theta0 is zero).
template <Lanes A, bool FIRST, typename T>
__device__ __forceinline__ void pull_species(const Geometry& g, const NodeIdx& n,
                                             const SpeciesCoef<T>& c, const T* __restrict__ src,
                                             const T* __restrict__ theta0, T f[9]) {
  if (FIRST) {
    const T a = theta0 ? *own_at<A>(theta0, n) : T(0);
    f[0] = c.w_rest * a;
#pragma unroll
    for (int i = 1; i < 5; ++i) f[i] = c.w_axis * a;
#pragma unroll
    for (int i = 5; i < 9; ++i) f[i] = c.w_diag * a;
  } else {
#pragma unroll
    for (int i = 0; i < 9; ++i) f[i] = *pull_at<A>(src + size_t(i) * g.plane, n, i);
  }
}

// Sources tau S_i + tau w_i Phi (S, PhiS) with tau = 1, 1/Cs^2 = 3: the
// chemotactic flux (ax, ay) and the kinetics phu on the u populations, phv
// on the v populations.
template <typename T>
__device__ __forceinline__ void add_sources(T fu[9], T fv[9], T phu, T ax, T ay, T phv) {
  const T p9 = phu * T(1.0 / 9.0), p36 = phu * T(1.0 / 36.0);
  const T x3 = ax * T(1.0 / 3.0), y3 = ay * T(1.0 / 3.0);
  const T x12 = ax * T(1.0 / 12.0), y12 = ay * T(1.0 / 12.0);
  fu[0] += phu * T(4.0 / 9.0);
  fu[1] += p9 + x3;
  fu[2] += p9 + y3;
  fu[3] += p9 - x3;
  fu[4] += p9 - y3;
  fu[5] += p36 + x12 + y12;
  fu[6] += p36 - x12 + y12;
  fu[7] += p36 - x12 - y12;
  fu[8] += p36 + x12 - y12;
  const T q9 = phv * T(1.0 / 9.0), q36 = phv * T(1.0 / 36.0);
  fv[0] += phv * T(4.0 / 9.0);
#pragma unroll
  for (int i = 1; i < 5; ++i) fv[i] += q9;
#pragma unroll
  for (int i = 5; i < 9; ++i) fv[i] += q36;
}

// Non-temporal (NT) or ordinary store.  Non-temporal ones suit values of whole
// 64-byte chunks that are next read a sweep later; a part of a chunk goes to
// memory by itself, at the cost of a read-modify-write there.
template <bool NT, typename T>
__device__ __forceinline__ void put(T* p, T v) {
  if (NT)
    __builtin_nontemporal_store(v, p);
  else
    *p = v;
}

// Stores of one species' populations at a fluid node (its 9 planes at dst),
// with the wall slots.  Forward: a population phi*_i streaming into a wall
// at x + e_i is reflected; it is parked in that node's slot of plane
// opp(i), where the next step's pull in direction opp(i) at x reads it.
// Adjoint (ADJ): the next gather in direction i at x reads plane i at the
// wall x + e_i and must find lambda_opp(i)(x).  A population whose slot a
// node across a non-periodic lattice uses (it leaves the lattice there; in
// the adjoint, plane i at x is gathered by x - e_i) is not stored itself.
template <Lanes A, bool WALLS, bool ADJ, bool NT = false, typename T>
__device__ __forceinline__ void store_species(const Geometry& g, const NodeIdx& n, const T f[9],
                                              T* __restrict__ dst, unsigned lm) {
  bool edge = WALLS && !g.periodic && (n.ex0 || n.ex1 || n.ey0 || n.ey1);
  // a wavefront of which some lanes store less than the others makes ordinary
  // stores, so that the parts of a chunk merge
  if (WALLS && NT) edge = __builtin_amdgcn_ballot_w64(edge) != 0ull;
  if (edge) {
#pragma unroll
    for (int i = 0; i < 9; ++i)
      if (!(ADJ ? pull_outside(n, i) : push_outside(n, i)))
        *own_at<A>(dst + size_t(i) * g.plane, n) = f[i];
  } else {
#pragma unroll
    for (int i = 0; i < 9; ++i) put<NT>(own_at<A>(dst + size_t(i) * g.plane, n), f[i]);
  }
  if (WALLS && (lm & 0x1FEu)) {
#pragma unroll
    for (int i = 1; i < 9; ++i)
      if ((lm >> opp(i)) & 1u)
        *push_at<A>(dst + size_t(ADJ ? i : opp(i)) * g.plane, n, i) = f[ADJ ? opp(i) : i];
  }
}

__device__ __forceinline__ float dsqrt(float x) { return __builtin_sqrtf(x); }
__device__ __forceinline__ double dsqrt(double x) { return __builtin_sqrt(x); }

// Implicit characteristic difference of the second-order source (eq:LBEG
// with kappa_t = kappa_x = 1): the scheme carries g = phi - (tau/2) w Phi,
// and Theta solves Theta - (tau/2) Phi(Theta) = G = sum_i g_i at each node:
// u from (tau r_u / 2) u^2 + (1 - tau r_u / 2) u - G_u = 0 (the root that
// tends to G_u as r_u -> 0, written without cancellation; tau r_u < 2),
// then v from the linear equation (a_uv u - b_v v + c enters at weight 1/2).
template <typename T>
__device__ __forceinline__ void implicit_solve(const ModelCoef<T>& m, T Gu, T Gv, T c, T& u,
                                               T& v) {
  const T hr = T(0.5) * m.r_u;
  const T bq = T(1) - hr;
  u = T(2) * Gu / (bq + dsqrt(dot2(T(4) * hr, Gu, bq, bq)));
  v = (Gv + T(0.5) * (m.a_uv * u + c)) / (T(1) + T(0.5) * m.b_v);
}

// Scheme variants: the source term of (eq:LBEG) for two species, 1 first
// order (tau F_i), 2 explicit characteristic difference (kappa_t = 1,
// kappa_x = 0), 3 implicit characteristic difference (kappa_t = kappa_x =
// 1); 4 three species (u, v and a repulsive signal w, first-order source).
constexpr int kVarFirst = 1, kVarExplicit = 2, kVarImplicit = 3, kVarThree = 4;

// Kinetics source tau w_i Phi on one species' populations.
template <typename T>
__device__ __forceinline__ void add_kinetics(T f[9], T ph) {
  f[0] += ph * T(4.0 / 9.0);
#pragma unroll
  for (int i = 1; i < 5; ++i) f[i] += ph * T(1.0 / 9.0);
#pragma unroll
  for (int i = 5; i < 9; ++i) f[i] += ph * T(1.0 / 36.0);
}

// Collision of a node's gathered populations, one forward step.
//
// LAG: second-order source term of (eq:LBEG) with kappa_t = 1, kappa_x = 0
// by the explicit characteristic difference: tau F + (tau/2)(F - F_prev)
// = tau (3/2 F - 1/2 F_prev) per population.  lag [2][plane] holds the
// kinetics r_u u (1-u), a_uv u - b_v v of the previous step at this node
// (the static control cancels in the difference) and is overwritten with
// this step's; at the first step there is no previous value and the
// difference is zero.
//
// kVarImplicit: the gathered values are g (phi at the first step, which
// starts from phi^0 = w~ Theta_0); Theta comes from implicit_solve, phi =
// g + (tau/2) w Phi, and the stored post-collision value is
// g* = relax(phi) + tau S + (tau/2) w Phi: the departure half of the
// difference, -(tau/2) F_i(x, t), plus the arrival half, which the next
// step's node solve takes at x + e_i.  The first moment of g equals that of
// phi (sum_i w_i e_i = 0).
//
// kVarThree: fw holds the third species; the record gains j_w (planes 3
// and 4), the chemotactic flux of u gains u Bw j_w (the repulsion
// A_u2 grad w with grad w = -K_w j_w / (tau d_w Cs^2)), and w relaxes with
// its own rates and receives Phi_w = a_w u - b_w w + s_w.
//
// forward_collide does the arithmetic in registers: f in place, the record
// (u, j_v, and j_w of three species) to r[0..4], lag (LAG) from the previous
// step's kinetics to this step's.  `first` marks step 0.
template <typename T, int VAR>
__device__ __forceinline__ void forward_collide(const ModelCoef<T>& m, T fu[9], T fv[9], T fw[9],
                                                T c, T r[5], T lag[2], bool first) {
  constexpr bool W3 = VAR == kVarThree;
  constexpr bool LAG = VAR == kVarExplicit;
  // macroscopic values (UGS) and the first moment of v
  T u = fu[0], v = fv[0];
#pragma unroll
  for (int i = 1; i < 9; ++i) {
    u += fu[i];
    v += fv[i];
  }
  const T jx = fv[1] - fv[3] + fv[5] - fv[6] - fv[7] + fv[8];
  const T jy = fv[2] - fv[4] + fv[5] + fv[6] - fv[7] - fv[8];
  if (VAR == kVarImplicit && !first) {
    const T Gu = u, Gv = v;
    implicit_solve(m, Gu, Gv, c, u, v);
    const T hu = T(0.5) * m.r_u * u * (T(1) - u);
    const T hv = T(0.5) * (m.a_uv * u - m.b_v * v + c);
    add_sources(fu, fv, hu, T(0), T(0), hv);  // phi = g + (tau/2) w Phi
  }
  T wv = T(0), kx = T(0), ky = T(0);
  if (W3) {
    wv = fw[0];
#pragma unroll
    for (int i = 1; i < 9; ++i) wv += fw[i];
    kx = fw[1] - fw[3] + fw[5] - fw[6] - fw[7] + fw[8];
    ky = fw[2] - fw[4] + fw[5] + fw[6] - fw[7] - fw[8];
    r[3] = kx;
    r[4] = ky;
  }
  r[0] = u;
  r[1] = jx;
  r[2] = jy;
  // chemotactic source: A_u1 grad v = u * B * j_v with the local gradient
  // grad v = -K_v j_v / (tau d_v Cs^2)
  T ax = u * dot2(m.b00, jx, m.b01, jy);
  T ay = u * dot2(m.b10, jx, m.b11, jy);
  if (W3) {
    ax += u * dot2(m.bw00, kx, m.bw01, ky);
    ay += u * dot2(m.bw10, kx, m.bw11, ky);
  }
  const T ru = m.r_u * u * (T(1) - u);
  const T rv = m.a_uv * u - m.b_v * v;
  T phu, phv;
  if (LAG) {
    const T lu = first ? ru : lag[0];
    const T lv = first ? rv : lag[1];
    phu = T(1.5) * ru - T(0.5) * lu;
    phv = T(1.5) * rv - T(0.5) * lv + c;
    lag[0] = ru;
    lag[1] = rv;
  } else if (VAR == kVarImplicit) {
    phu = T(0.5) * ru;
    phv = T(0.5) * (rv + c);
  } else {
    phu = ru;
    phv = rv + c;
  }
  T t1, t2;
  relax<true>(fu, u, m.u, t1, t2);
  relax<true>(fv, v, m.v, t1, t2);
  add_sources(fu, fv, phu, ax, ay, phv);
  if (W3) {
    relax<true>(fw, wv, m.w, t1, t2);
    add_kinetics(fw, m.a_w * u - m.b_w * wv + m.s_w);
  }
}

// Record of one step at a node.
template <Lanes A, int VAR, bool NT = false, typename T>
__device__ __forceinline__ void store_record(const Geometry& g, const NodeIdx& n,
                                             T* __restrict__ rec, const T r[5]) {
#pragma unroll
  for (int k = 0; k < (VAR == kVarThree ? 5 : 3); ++k)
    put<NT>(own_at<A>(rec + size_t(k) * g.plane, n), r[k]);
}

// Non-temporal (NT) for a record that one thread reads; regions share the
// records of their rings.
template <Lanes A, int VAR, bool NT = false, typename T>
__device__ __forceinline__ void load_record(const Geometry& g, const NodeIdx& n,
                                            const T* __restrict__ rec, T r[5]) {
#pragma unroll
  for (int k = 0; k < (VAR == kVarThree ? 5 : 3); ++k) {
    const T* p = own_at<A>(rec + size_t(k) * g.plane, n);
    r[k] = NT ? __builtin_nontemporal_load(p) : *p;
  }
}

// Tangent-linear step (sensitivity LBE, LIBEG-V) at a node: the derivative
// of the collision of forward step n applied to the gathered perturbation
// (fu, fv), with the recorded pre-collision u and j_v of that step and the
// control perturbation dc.  The relaxation is linear (relax with theta =
// the perturbed density); the sources give
//   d(u B j_v) = du B j_v + u B dj_v,   dPhi_u = r_u (1 - 2u) du,
//   dPhi_v = a_uv du - b_v dv + dc.
// LAG: the second-order source as in the forward, on the perturbed
// kinetics; dlag [2][plane] carries their previous-step values.
// kVarImplicit: the perturbation of g; the node equation linearised at the
// recorded u gives du = dG_u / (1 - (tau/2) r_u (1 - 2u)) and
// dv = (dG_v + (tau/2)(a_uv du + dc)) / (1 + (tau/2) b_v) (none at the first
// step, whose input is dphi^0).
// kVarThree: fw holds the perturbation of the third species;
// d(u Bw j_w) = du Bw j_w + u Bw dj_w with j_w recorded, and
// dPhi_w = a_w du - b_w dw.
// r: the recorded u, j_v (and j_w) of the step.
template <typename T, int VAR>
__device__ __forceinline__ void tlm_collide(const ModelCoef<T>& m, T fu[9], T fv[9], T fw[9], T dc,
                                            const T r[5], T dlag[2], bool first) {
  constexpr bool LAG = VAR == kVarExplicit;
  constexpr bool W3 = VAR == kVarThree;
  const T u = r[0], jx = r[1], jy = r[2];
  T du = fu[0], dv = fv[0];
#pragma unroll
  for (int i = 1; i < 9; ++i) {
    du += fu[i];
    dv += fv[i];
  }
  if (VAR == kVarImplicit && !first) {
    du = du / (T(1) - T(0.5) * m.r_u * (T(1) - T(2) * u));
    dv = (dv + T(0.5) * (m.a_uv * du + dc)) / (T(1) + T(0.5) * m.b_v);
    const T hu = T(0.5) * m.r_u * (T(1) - T(2) * u) * du;
    const T hv = T(0.5) * (m.a_uv * du - m.b_v * dv + dc);
    add_sources(fu, fv, hu, T(0), T(0), hv);  // dphi = dg + (tau/2) w dPhi
  }
  const T djx = fv[1] - fv[3] + fv[5] - fv[6] - fv[7] + fv[8];
  const T djy = fv[2] - fv[4] + fv[5] + fv[6] - fv[7] - fv[8];
  const T fx = dot2(m.b00, jx, m.b01, jy), dfx = dot2(m.b00, djx, m.b01, djy);
  const T fy = dot2(m.b10, jx, m.b11, jy), dfy = dot2(m.b10, djx, m.b11, djy);
  constexpr bool IMPL = VAR == kVarImplicit;
  T dax = IMPL ? dot2(du, fx, u, dfx) : dot2(u, dfx, du, fx);
  T day = IMPL ? dot2(du, fy, u, dfy) : dot2(u, dfy, du, fy);
  T dw = T(0);
  if (W3) {
    const T kx = r[3], ky = r[4];
    dw = fw[0];
#pragma unroll
    for (int i = 1; i < 9; ++i) dw += fw[i];
    const T dkx = fw[1] - fw[3] + fw[5] - fw[6] - fw[7] + fw[8];
    const T dky = fw[2] - fw[4] + fw[5] + fw[6] - fw[7] - fw[8];
    dax += du * dot2(m.bw00, kx, m.bw01, ky) + u * dot2(m.bw00, dkx, m.bw01, dky);
    day += du * dot2(m.bw10, kx, m.bw11, ky) + u * dot2(m.bw10, dkx, m.bw11, dky);
  }
  const T dru = m.r_u * (T(1) - T(2) * u) * du;
  const T drv = m.a_uv * du - m.b_v * dv;
  T dphu, dphv;
  if (LAG) {
    const T lu = first ? dru : dlag[0];
    const T lv = first ? drv : dlag[1];
    dphu = T(1.5) * dru - T(0.5) * lu;
    dphv = T(1.5) * drv - T(0.5) * lv + dc;
    dlag[0] = dru;
    dlag[1] = drv;
  } else if (VAR == kVarImplicit) {
    dphu = T(0.5) * dru;
    dphv = T(0.5) * (drv + dc);
  } else {
    dphu = dru;
    dphv = drv + dc;
  }
  T t1, t2;
  relax<true>(fu, du, m.u, t1, t2);
  relax<true>(fv, dv, m.v, t1, t2);
  add_sources(fu, fv, dphu, dax, day, dphv);
  if (W3) {
    relax<true>(fw, dw, m.w, t1, t2);
    add_kinetics(fw, m.a_w * du - m.b_w * dw);
  }
}

// Continuous-adjoint step (Section 3.2.2: the continuous adjoint system of
// the two-species instance solved by the MRT scheme in reversed time) at a
// node, from the gathered adjoint populations (fp of p, fq of q) and the
// recorded forward u, j_v at this time:
//   p_s = div(D_u grad p) + chi (C grad v).grad p + r_u (1 - 2u) p + a_uv q
//   q_s = div(D_v grad q) - b_v q - div(chi u C^T grad p)
// p relaxes like u and q like v; the advection and the couplings are
// scalar sources, the cross-diffusion of q a flux source, as the
// chemotaxis of u in the forward.  Returns tau q (pre-collision), the step's
// share of the time integral.
template <typename T>
__device__ __forceinline__ T cadj_collide(const ModelCoef<T>& m, const CadjCoef<T>& cc, T fp[9],
                                          T fq[9], const T r[5]) {
  const T u = r[0], jvx = r[1], jvy = r[2];
  T P = fp[0], Qv = fq[0];
#pragma unroll
  for (int i = 1; i < 9; ++i) {
    P += fp[i];
    Qv += fq[i];
  }
  const T jpx = fp[1] - fp[3] + fp[5] - fp[6] - fp[7] + fp[8];
  const T jpy = fp[2] - fp[4] + fp[5] + fp[6] - fp[7] - fp[8];
  const T adv = dot2(jpx, dot2(cc.m00, jvx, cc.m01, jvy), jpy, dot2(cc.m10, jvx, cc.m11, jvy));
  const T php = dot2(m.a_uv, Qv, m.r_u * (T(1) - T(2) * u), P) + adv;
  const T phq = -m.b_v * Qv;
  const T aqx = u * dot2(cc.q00, jpx, cc.q01, jpy);
  const T aqy = u * dot2(cc.q10, jpx, cc.q11, jpy);
  T t1, t2;
  relax<true>(fp, P, m.u, t1, t2);
  relax<true>(fq, Qv, m.v, t1, t2);
  add_sources(fp, fq, php, T(0), T(0), phq);
  // flux source of q: 3 w_i e_i . a_q
  const T x3 = aqx * T(1.0 / 3.0), y3 = aqy * T(1.0 / 3.0);
  const T x12 = aqx * T(1.0 / 12.0), y12 = aqy * T(1.0 / 12.0);
  fq[1] += x3;
  fq[2] += y3;
  fq[3] -= x3;
  fq[4] -= y3;
  fq[5] += x12 + y12;
  fq[6] += y12 - x12;
  fq[7] -= x12 + y12;
  fq[8] += x12 - y12;
  return Qv;
}

// Terminal streaming: the state after the last step and its sums.  IMPL
// (implicit characteristic difference): the streamed values are g; Theta^N
// comes from the node solve and the state is phi^N = g + (tau/2) w Phi.
// W3: the third species' populations are also streamed into the state.
template <typename T, bool IMPL = false, bool W3 = false>
__device__ __forceinline__ void finalize_node(
    const Geometry& g, const NodeIdx& n, const T* __restrict__ src, T* __restrict__ state,
    T* __restrict__ uN, T* __restrict__ vN, const ModelCoef<T>* m = nullptr,
    const T* __restrict__ ctrl = nullptr) {
  const size_t idx = n.r0 + n.x;
  const bool solid = g.masked && (link_of(g, wave_flag(g, n), idx) & 1u);
  T fu[9], fv[9];
  if (solid) {
#pragma unroll
    for (int i = 0; i < 9; ++i) fu[i] = fv[i] = T(0);
  } else {
#pragma unroll
    for (int i = 0; i < 9; ++i) {
      fu[i] = *pull_at<kAny>(src + size_t(i) * g.plane, n, i);
      fv[i] = *pull_at<kAny>(src + size_t(9 + i) * g.plane, n, i);
    }
  }
  T u = T(0), v = T(0);
#pragma unroll
  for (int i = 0; i < 9; ++i) {
    u += fu[i];
    v += fv[i];
  }
  if (IMPL && !solid) {
    const T c = ctrl[idx];
    const T Gu = u, Gv = v;
    implicit_solve(*m, Gu, Gv, c, u, v);
    add_sources(fu, fv, T(0.5) * m->r_u * u * (T(1) - u), T(0), T(0),
                T(0.5) * (m->a_uv * u - m->b_v * v + c));
  }
  if (uN) uN[idx] = u;
  if (vN) vN[idx] = v;
  if (state) {
#pragma unroll
    for (int i = 0; i < 9; ++i) {
      state[size_t(i) * g.plane + idx] = fu[i];
      state[size_t(9 + i) * g.plane + idx] = fv[i];
    }
    if (W3) {
#pragma unroll
      for (int i = 0; i < 9; ++i)
        state[size_t(18 + i) * g.plane + idx] =
            solid ? T(0) : *pull_at<kAny>(src + size_t(18 + i) * g.plane, n, i);
    }
  }
}

// --------------------------------------------------------------- adjoint

// LAG: adjoint of the second-order source.  The scheme's state then also
// holds the previous step's kinetics F_prev; mu [2][plane] is the adjoint
// of the kinetics this step stores for the next one.  With sigma = w . nu
// per species, the adjoint of this step's kinetics is rho = 3/2 sigma + mu
// (sigma + mu at step 0, where F_prev = F), and the new mu = -1/2 sigma.
// Step N-1 reads no mu: nothing reads the last stored kinetics.
//
// kVarImplicit: the adjoint of g.  With A the relaxation (phi -> phi -
// C (phi - w~ Theta)), a step maps g to g* = A g + (tau/2)(A w + w) Phi +
// tau S with Theta from the node equation, so the sensitivity to Phi_s is
// kappa_s = (tau/2)(w . A^T nu_s + sigma_s); through the linearised node
// solve (alpha = 1 / (1 - (tau/2) r_u (1 - 2u)), beta = 1 / (1 +
// (tau/2) b_v)) the sums G_s receive Gbar_v = beta vbar and Gbar_u =
// alpha (ubar + (tau/2) a_uv beta vbar), and the control kappa_v beta.  At
// step 0 the input is phi^0 itself: kappa_s = (tau/2) sigma_s, no solve.
//
// kVarThree: the adjoint of w as well (planes 18..26; zero at the terminal
// step, the cost not depending on w): sigma_w enters u's source through
// a_w, w's own through -b_w; the repulsive flux u Bw j_w adds
// p . (Bw j_w) to u's and e_i . (u Bw^T p) to w's.
//
// adjoint_gather loads, adjoint_collide does the arithmetic.
//
// Adjoint gather of node n from the state of the step after (src), or
// (FIRST) the terminal seeds.
template <Lanes A, bool WALLS, int VAR, bool FIRST, typename T>
__device__ __forceinline__ void adjoint_gather(const Geometry& g, const NodeIdx& n,
                                               const T* __restrict__ src,
                                               const T* __restrict__ seed_u,
                                               const T* __restrict__ seed_v, unsigned lm,
                                               T nu[9], T nv[9], T nw[9]) {
  constexpr bool W3 = VAR == kVarThree;
  // reverse streaming: nu_i(x) = lambda_i(x + e_i), or lambda_opp(i)(x)
  // when x + e_i is a wall (exact transpose of the pull with bounce-back)
  if (FIRST) {
    // terminal condition lambda_i^N = seed for every i (psi(T) = dI0/dphi);
    // the seed fields carry no wall slots, so walls are tested here
    const T own_u = *own_at<A>(seed_u, n), own_v = seed_v ? *own_at<A>(seed_v, n) : T(0);
#pragma unroll
    for (int i = 0; i < 9; ++i) {
      const bool wall = WALLS && i > 0 && ((lm >> opp(i)) & 1u);
      const T su = *push_at<A>(seed_u, n, i), sv = seed_v ? *push_at<A>(seed_v, n, i) : T(0);
      nu[i] = wall ? own_u : su;
      nv[i] = wall ? own_v : sv;
      if (W3) nw[i] = T(0);
    }
  } else {
#pragma unroll
    for (int i = 0; i < 9; ++i) {
      nu[i] = *push_at<A>(src + size_t(i) * g.plane, n, i);
      nv[i] = *push_at<A>(src + size_t(9 + i) * g.plane, n, i);
      if (W3) nw[i] = *push_at<A>(src + size_t(18 + i) * g.plane, n, i);
    }
  }
}

// Transposed flux source: f_i += e_i . (u q).  Of the two products in u q_x +-
// u q_y the one along x is fused where there are walls, the other without
// (either is as near the exact value; each kind of lattice keeps its bits).
template <bool WALLS, typename T>
__device__ __forceinline__ void add_flux_adjoint(T f[9], T u, T qx, T qy) {
  f[1] += u * qx;
  f[2] += u * qy;
  f[3] -= u * qx;
  f[4] -= u * qy;
  const T sum = WALLS ? dot2(u, qx, u, qy) : dot2(u, qy, u, qx);
  const T dif = WALLS ? dot2(u, qx, -u, qy) : dot2(-u, qy, u, qx);
  f[5] += sum;
  f[6] -= dif;
  f[7] -= sum;
  f[8] += dif;
}

// The adjoint collision in registers: nu, nv (nw) in place; r is the
// recorded u, j_v (j_w) of the step; mu (LAG) the adjoint of the stored
// kinetics, from the step after to this one; `first` marks step N-1, `step0`
// step 0.  Returns the step's share of the gradient, dF_v,i/dc = tau w_i
// (the implicit form: see above).
template <typename T, bool WALLS, int VAR>
__device__ __forceinline__ T adjoint_collide(const ModelCoef<T>& m, T nu[9], T nv[9], T nw[9],
                                             const T r[5], T mu[2], bool first, bool step0) {
  constexpr bool W3 = VAR == kVarThree;
  constexpr bool LAG = VAR == kVarExplicit;
  constexpr bool IMPL = VAR == kVarImplicit;
  // weighted sums: sigma = w . nu, p = (tau/Cs^2) sum_i w_i nu_u,i e_i
  const T su_ = weighted(nu), sv_ = weighted(nv);
  const T px = dot2(T(1.0 / 3.0), nu[1] - nu[3],
                    T(1.0 / 12.0), nu[5] - nu[6] - nu[7] + nu[8]);
  const T py = dot2(T(1.0 / 3.0), nu[2] - nu[4],
                    T(1.0 / 12.0), nu[5] + nu[6] - nu[7] - nu[8]);
  const T u = r[0], jx = r[1], jy = r[2];
  const T bjx = dot2(m.b00, jx, m.b01, jy);
  const T bjy = dot2(m.b10, jx, m.b11, jy);
  // transposed sources: d(tau S_u + tau Phi_u)/dphi_u is rank one along 1,
  // d(tau S_u)/dphi_v = (tau/Cs^2) diag(w) E u B E^T, dPhi_v/dphi = (a, -b).
  T rho_u = su_, rho_v = sv_;
  if (LAG) {
    const T mu_u = first ? T(0) : mu[0];
    const T mu_v = first ? T(0) : mu[1];
    if (step0) {
      rho_u = su_ + mu_u;
      rho_v = sv_ + mu_v;
    } else {
      rho_u = T(1.5) * su_ + mu_u;
      rho_v = T(1.5) * sv_ + mu_v;
      mu[0] = T(-0.5) * su_;
      mu[1] = T(-0.5) * sv_;
    }
  }
  const T qx = dot2(m.b00, px, m.b10, py);
  const T qy = dot2(m.b01, px, m.b11, py);
  T wu, wv, share = sv_;
  if (!IMPL) {
    T cu = dot2(rho_u * m.r_u, T(1) - T(2) * u, px, bjx) + py * bjy + rho_v * m.a_uv;
    const T cv = -rho_v * m.b_v;
    if (W3) {
      const T kx = r[3], ky = r[4];
      const T sw_ = weighted(nw);
      cu += px * dot2(m.bw00, kx, m.bw01, ky) + py * dot2(m.bw10, kx, m.bw11, ky) +
            sw_ * m.a_w;
      T a1, a2;
      relax<false>(nw, T(0), m.wt, a1, a2);
      const T ww = dot2(m.w.eps_eq, a2, m.w.e_eq, a1) - sw_ * m.b_w;
#pragma unroll
      for (int i = 0; i < 9; ++i) nw[i] += ww;
      add_flux_adjoint<WALLS>(nw, u, dot2(m.bw00, px, m.bw10, py), dot2(m.bw01, px, m.bw11, py));
    }
    // adjoint collision: nu - C^T nu + 1 * weq^T C^T nu  (AEDs with O = 1 weq^T)
    T a1, a2;
    relax<false>(nu, T(0), m.ut, a1, a2);
    wu = dot2(m.u.eps_eq, a2, m.u.e_eq, a1) + cu;
    relax<false>(nv, T(0), m.vt, a1, a2);
    wv = dot2(m.v.eps_eq, a2, m.v.e_eq, a1) + cv;
  } else {
    T a1, a2;
    relax<false>(nu, T(0), m.ut, a1, a2);
    const T eu = dot2(m.u.eps_eq, a2, m.u.e_eq, a1);
    relax<false>(nv, T(0), m.vt, a1, a2);
    const T ev = dot2(m.v.eps_eq, a2, m.v.e_eq, a1);
    T ku = T(0.5) * su_, kv = T(0.5) * sv_;
    if (!step0) {
      // w . A^T nu = w . (relaxed nu) + e (sum_i w_i = 1)
      const T tu = weighted(nu) + eu;
      const T tv = weighted(nv) + ev;
      ku = T(0.5) * (tu + su_);
      kv = T(0.5) * (tv + sv_);
    }
    const T ubar = dot2(m.a_uv, kv, ku * m.r_u, T(1) - T(2) * u) + px * bjx + py * bjy;
    const T vbar = -kv * m.b_v;
    T gu = ubar, gv = vbar;
    share = kv;
    if (!step0) {
      const T beta = T(1) / (T(1) + T(0.5) * m.b_v);
      const T alpha = T(1) / (T(1) - T(0.5) * m.r_u * (T(1) - T(2) * u));
      gv = beta * vbar;
      gu = alpha * (ubar + T(0.5) * m.a_uv * gv);
      share = kv * beta;
    }
    wu = eu + gu;
    wv = ev + gv;
  }
#pragma unroll
  for (int i = 0; i < 9; ++i) {
    nu[i] += wu;
    nv[i] += wv;
  }
  add_flux_adjoint<WALLS>(nv, u, qx, qy);
  return share;
}

// Transpose of phi_i^0 = w_i Theta_0: the sensitivity to an initial field.
template <typename T>
__device__ __forceinline__ T adjoint_initial(const SpeciesCoef<T>& c, const T f[9]) {
  return dot2(c.w_rest, f[0], c.w_axis, f[1] + f[2] + f[3] + f[4]) +
         c.w_diag * (f[5] + f[6] + f[7] + f[8]);
}

// ------------------------------------------------------------ reductions

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
  return v;
}

__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_down(v, off, 64));
  return v;
}

// Block reduction of kRedSlots values (slot 3 is a max, the others sums);
// lane 0 of the block writes the block partial.
__device__ void block_reduce_store(double vals[kRedSlots], double* out) {
  __shared__ double lds[kRedSlots][kBlock / 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < kRedSlots; ++k) {
    double r = (k == 3) ? wave_max(vals[k]) : wave_sum(vals[k]);
    if (lane == 0) lds[k][wave] = r;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int k = 0; k < kRedSlots; ++k) {
      double r = lds[k][0];
      for (int w = 1; w < kBlock / 64; ++w)
        r = (k == 3) ? fmax(r, lds[k][w]) : r + lds[k][w];
      out[k] = r;
    }
  }
}

}  // namespace dev
}  // namespace mrt
