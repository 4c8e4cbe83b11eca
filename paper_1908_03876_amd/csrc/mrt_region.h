// Several time steps in one launch: what the kernels of a single lattice and
// of a batch share.
//
// Method: arXiv:1908.03876, Sections 3.1 and 3.2.1, as in mrt_device.h.
#pragma once

#include "mrt_device.h"

namespace mrt {
namespace dev {

// A launch advances several time steps.  A work-group owns a region of
// RX x RY nodes, one per thread; the first step gathers from memory, the
// steps in between exchange their populations through LDS (u and v of a
// direction side by side, one 8- or 16-byte access each), and the last one
// stores.  With K steps the K - 1 outer rings of the region go stale one
// after the other: they recompute what the neighbouring regions own, so a
// region stores the RX - 2(K-1) by RY - 2(K-1) nodes inside them, and a
// wavefront whose rows are stale leaves the work to the others.
//
// The regions are 32 x 32, or 64 x 16 (a wavefront is one row, so rows are
// scalar addresses), for the 72 bytes a node of two species in FP32: 1024
// threads and two work-groups a compute unit, 64 registers a thread, 67 KB of
// LDS.  Twice as wide nodes take 32 x 16.  Lattices of a few thousand nodes take
// 16 x 16 regions, which spread them over the chip.  The explicit second-order
// source also reads the previous step's kinetics of its nodes, which a
// neighbouring region may not find overwritten: where the tape holds only one
// buffer for them it takes one step at a time.  A launch of one step goes over
// rows of 256 nodes (kRows).
//
// What bounds it: the vector units.  With 5 steps a launch the state's traffic
// falls from 144 to 29 B a node and step, and at 2048^2 in FP32 vector
// instructions take 88% (forward) and 90% (AMRT step) of the issue slots at 2.4
// GHz, a third of them for the rings, beside 4.1 to 4.4 TB/s.  Stores are
// ordinary ones: a region's rows begin anywhere in a 64-byte chunk, and two
// regions' parts of a chunk merge in L2 (with non-temporal stores each part went
// to memory by itself: 65 us a step at 2048^2 instead of 55).  Measured at 2048^2, masked, FP32, in us a step:
// forward with record 122 -> 50.9, AMRT step 125 -> 52.7 (periodic: 49.6 and
// 49.4); at 1024^2, periodic, 27 -> 11.8 and 36 -> 13.2; at 512^2, masked,
// 9.7 -> 3.8 and 10.4 -> 4.0; at 128^2 4.4 -> 1.6.

// The steps of a launch, and how many nodes on each side of a region it does
// not own (at least count - 1).
struct Steps {
  int count, halo;
};

// Regions of one row and one step.
template <int RY>
constexpr bool kRows = RY == 1;

template <typename T>
struct alignas(2 * sizeof(T)) Pair {
  T u, v;
};

template <typename T, int RX, int RY, bool W3>
struct Exchange {
  static constexpr int kNodes = RX * RY;
  static constexpr int kPad = RX + 1;  // the outer ring reads past the region
  Pair<T> uv[8 * kNodes + 2 * kPad];
  T w[W3 ? 8 * kNodes + 2 * kPad : 1];
};

// Streaming between two steps of a launch: the populations of every node go
// to LDS (give), and each node takes back those its neighbours send it (ADJ:
// the transposed stream, from x + e_i).
//
// Walls cost no test in take, as in memory: a population that meets a wall or
// a non-periodic edge goes to the slot of that neighbour from which its node
// takes the opposite one, and solid nodes give nothing.  A node writes each
// population once, here or there, so a wavefront that touches no wall (all
// link words zero) pays one scalar branch.  (With the test in take, which kept
// the reflected populations over the reads, it paid 36 register moves of 270
// vector instructions a step: AMRT step 65.4 us at 2048^2 instead of 57.1.)
template <bool WALLS, bool ADJ, typename T, int RX, int RY, bool W3>
__device__ __forceinline__ void give(Exchange<T, RX, RY, W3>& lds, const T fu[9], const T fv[9],
                                     const T fw[9], unsigned lm) {
  constexpr int N = RX * RY, P = RX + 1;
  constexpr int ex[9] = {0, 1, 0, -1, 0, 1, -1, -1, 1};
  constexpr int ey[9] = {0, 0, 1, 0, -1, 1, 1, -1, -1};
  __syncthreads();  // the reads of the exchange before are done
  if (WALLS && __builtin_amdgcn_ballot_w64(lm != 0u) != 0ull) {
    if (!(lm & 1u)) {
#pragma unroll
      for (int i = 1; i < 9; ++i) {
        const int wall = ADJ ? i : opp(i);
        const int there = (opp(i) - i) * N + (ADJ ? -1 : 1) * (ex[i] + ey[i] * RX);
        const int o = P + (i - 1) * N + int(threadIdx.x) + ((lm >> wall) & 1u ? there : 0);
        lds.uv[o] = Pair<T>{fu[i], fv[i]};
        if (W3) lds.w[o] = fw[i];
      }
    }
  } else {
#pragma unroll
    for (int i = 1; i < 9; ++i) {
      lds.uv[P + (i - 1) * N + int(threadIdx.x)] = Pair<T>{fu[i], fv[i]};
      if (W3) lds.w[P + (i - 1) * N + int(threadIdx.x)] = fw[i];
    }
  }
  __syncthreads();
}

template <bool ADJ, typename T, int RX, int RY, bool W3>
__device__ __forceinline__ void take(const Exchange<T, RX, RY, W3>& lds, T fu[9], T fv[9],
                                     T fw[9]) {
  constexpr int N = RX * RY, P = RX + 1;
  constexpr int ex[9] = {0, 1, 0, -1, 0, 1, -1, -1, 1};
  constexpr int ey[9] = {0, 0, 1, 0, -1, 1, 1, -1, -1};
#pragma unroll
  for (int i = 1; i < 9; ++i) {
    const int o = P + (i - 1) * N + (ADJ ? 1 : -1) * (ex[i] + ey[i] * RX) + int(threadIdx.x);
    const Pair<T> p = lds.uv[o];
    fu[i] = p.u;
    fv[i] = p.v;
    if (W3) fw[i] = lds.w[o];
  }
}

// The links of a node across which it may write to the slot of a neighbour:
// not those out of the region.  (A node at the region's edge goes stale with
// the first exchange; no launch of several steps stores its results.)
template <int RX, int RY>
__device__ __forceinline__ unsigned links_inside(unsigned lm) {
  const int dx = unsigned(threadIdx.x) % RX, dy = unsigned(threadIdx.x) / RX;
  unsigned out = dx == 0 ? 0x122u : 0u;        // x - e_i for i = 1, 5, 8
  out |= dx == RX - 1 ? 0x0C8u : 0u;           // 3, 6, 7
  out |= dy == 0 ? 0x064u : 0u;                // 2, 5, 6
  out |= dy == RY - 1 ? 0x190u : 0u;           // 4, 7, 8
  return lm & ~out;
}

// Does this wavefront still hold rows that step s of a launch needs?  The
// outer rows go stale with their rings: step s needs those that the region
// owns (all but `halo` on each side) and as many more as steps follow it.
template <int RX, int RY>
__device__ __forceinline__ int first_row() {
  return __builtin_amdgcn_readfirstlane(threadIdx.x / 64) * 64 / RX;
}
template <int RX, int RY>
__device__ __forceinline__ bool live_rows(const Steps& st, int s, int lo) {
  const int hi = lo + (RX < 64 ? 64 / RX : 1) - 1;
  const int stale = st.halo - (st.count - 1 - s);
  return hi >= stale && lo < RY - stale;
}

// A uniform pointer that the next step moves on: kept in scalar registers, so
// that its accesses take a lane offset and no 64-bit vector arithmetic.
template <typename T>
__device__ __forceinline__ T* scalar(T* p) {
  auto q = (__attribute__((address_space(1))) T*)p;
  asm("" : "+s"(q));
  return (T*)q;
}

// A wavefront of stale rows after step s: it only meets the others at the
// barriers of the exchanges to come.
__device__ __forceinline__ bool retire(const Steps& st, int s) {
  for (; s < st.count - 2; ++s) {
    __syncthreads();
    __syncthreads();
  }
  return false;
}

// The initial populations of a lattice with walls enter the collision as
// rounded products: the compiler may not contract them into its sums.  (On
// the others it may.  Either way is as near the exact value; each kind of
// lattice keeps its bits.)
template <bool W3, typename T>
__device__ __forceinline__ void keep_rounded(T fu[9], T fv[9], T fw[9]) {
#pragma unroll
  for (int i = 0; i < 9; ++i) {
    asm volatile("" : "+v"(fu[i]), "+v"(fv[i]));
    if (W3) asm volatile("" : "+v"(fw[i]));
  }
}

// The steps themselves, after the gather; each returns false to a wavefront
// whose rows are stale before the last one.
//
// Forward: from the pulled populations (FIRST: of step 0) to the last step's
// post-collision ones, recording each step where rec is not null.
template <bool WALLS, int VAR, Lanes A, bool FIRST, typename T, int RX, int RY, bool W3>
__device__ __forceinline__ bool forward_steps(Exchange<T, RX, RY, W3>& lds, const Geometry& g,
                                              const NodeIdx& n, unsigned& lm,
                                              const ModelCoef<T>& m, T c, bool owner, T fu[9],
                                              T fv[9], T fw[9], T lag[2], T* __restrict__ rec,
                                              size_t rec_stride, const Steps& st) {
  T r[5];
  const int row = first_row<RX, RY>();
  auto record = [&] {
    if (rec == nullptr) return;
    if (owner) store_record<A, VAR, kRows<RY>>(g, n, rec, r);
    rec = scalar(rec + rec_stride);
  };
  if (WALLS && !kRows<RY> && st.count > 1) lm = links_inside<RX, RY>(lm);
  int s = 0;
  if (FIRST) {  // step 0 on its own: it differs for the second-order sources
    if (WALLS) keep_rounded<W3>(fu, fv, fw);
    forward_collide<T, VAR>(m, fu, fv, fw, c, r, lag, true);
    record();
    if (kRows<RY>) return true;
    if (st.count > 1) {
      give<WALLS, false>(lds, fu, fv, fw, lm);
      if (!live_rows<RX, RY>(st, 1, row)) return retire(st, 0);
      take<false>(lds, fu, fv, fw);
    }
    s = 1;
  }
  for (; s < st.count; ++s) {
    forward_collide<T, VAR>(m, fu, fv, fw, c, r, lag, false);
    record();
    if (kRows<RY> || s + 1 == st.count) break;
    give<WALLS, false>(lds, fu, fv, fw, lm);
    if (!live_rows<RX, RY>(st, s + 1, row)) return retire(st, s);
    take<false>(lds, fu, fv, fw);
  }
  return true;
}

// Adjoint steps step, step - 1, ...: rec is the record slot of the first.
template <bool WALLS, int VAR, Lanes A, bool FIRST, typename T, int RX, int RY, bool W3>
__device__ __forceinline__ bool adjoint_steps(Exchange<T, RX, RY, W3>& lds, const Geometry& g,
                                              const NodeIdx& n, unsigned& lm,
                                              const ModelCoef<T>& m, int step, T nu[9], T nv[9],
                                              T nw[9], T mu[2], double& sum,
                                              const T* __restrict__ rec, size_t rec_stride,
                                              const Steps& st) {
  T r[5];
  const int row = first_row<RX, RY>();
  load_record<A, VAR, kRows<RY>>(g, n, rec, r);
  if (WALLS && !kRows<RY> && st.count > 1) lm = links_inside<RX, RY>(lm);
  for (int s = 0;; ++s) {
    sum += double(
        adjoint_collide<T, WALLS, VAR>(m, nu, nv, nw, r, mu, FIRST && s == 0, step - s == 0));
    if (kRows<RY> || s + 1 == st.count) break;
    rec = scalar(rec - rec_stride);
    load_record<A, VAR, kRows<RY>>(g, n, rec, r);
    give<WALLS, true>(lds, nu, nv, nw, lm);
    if (!live_rows<RX, RY>(st, s + 1, row)) return retire(st, s);
    take<true>(lds, nu, nv, nw);
  }
  return true;
}

}  // namespace dev
}  // namespace mrt
