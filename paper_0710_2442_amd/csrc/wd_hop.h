// Per-site Wilson hop (Eq. 3 on one checkerboard), shared by the
// single-lattice, multi-RHS and batched multi-lattice kernels.
#pragma once

#include <utility>

#include "wd_device.h"

namespace wd {

template <int P>
using RealOf = typename Spinor<P>::real;

struct KDslash {
  Geom g;
  const char *in;
  char *out;
  const char *X;
  const char *Y;
  const char *links;  // hop-link arrays of this output parity
  double a;
  int parity;
  const int *skip;
  double *partials;
  // block -> tile mapping (see tile_of)
  int groups;           // 0: linear; G > 0: G contiguous regions per time slice
  int tiles_per_slice;  // tiles (blocks) per time slice of one parity
  int occ;              // register-budget variant (0 or 4), host side only
  int nt_store;         // 1: streaming output stores; 0: cached stores
  int preload;          // 1: load all 8 links before the first hop (FP32 arithmetic only), host side
  int stage;            // 1: stage the tile's input spinors in LDS (FP64, FP32), host side
  int split;            // 1: one wave per hop direction, host side
  int spl;              // sites per lane along x4 (1, 2, 4): lane covers tiles t, t + T, ... of consecutive slices
};

// Workgroups are dispatched round-robin over the XCDs (8 on MI355X), each
// with its own L2.  groups = G > 0: block b goes to region b % G and the
// blocks of one region walk its tiles slice by slice in time order, so a
// region's neighbour spinors (x1..x3 inside the slice, x4 one slice away)
// are fetched into one L2 and re-read from there.  Requires
// tiles_per_slice % G == 0.  groups = -X: the time slices are cut into X
// contiguous ranges and block b walks range b % X in time order; with X = 8
// each XCD sweeps its own block of slices, so the spatial neighbours (same
// slice) and the time neighbours (the slices before and after) of a site are
// all re-read from that XCD's L2.  Requires L4 % X == 0.  Both need
// gridDim.x == tiles_per_slice * L4.
__device__ __forceinline__ int tile_of(const KDslash &k, int b) {
  if (k.groups == 0) return b;
  const int T = k.tiles_per_slice;
  if (k.groups <= -100) {
    // box order: dispatch lane x = b % 8 (one per XCD) owns the box of x3
    // planes [bx * P, bx * P + P) and time slices [bt * S, bt * S + S),
    // nx3 = -groups - 100 boxes along x3 and 8 / nx3 along x4, and walks it
    // slice by slice, plane by plane, so that every neighbour of a site but
    // those across a box face is fetched into that XCD's L2, and the next
    // slice's sites (the time neighbours) are at most one box slice away.
    const int nx3 = -k.groups - 100;
    const int P = k.g.L[2] / nx3, S = k.g.L[3] / (8 / nx3);
    const int tpp = T / k.g.L[2];  // tiles per x3 plane
    const int x = b & 7, q = b >> 3;
    const int bx = x % nx3, bt = x / nx3;
    const int s = q / (P * tpp), pl = (q / tpp) % P, tp = q % tpp;
    return ((bt * S + s) * k.g.L[2] + bx * P + pl) * tpp + tp;
  }
  if (k.groups < 0) {
    const int X = -k.groups;
    const int x = b % X, q = b / X;
    const int per = k.g.L[3] / X;  // slices per range
    return (x * per + q / T) * T + (q % T);
  }
  const int G = k.groups;
  const int per = T / G;
  const int x = b % G, q = b / G;
  return (q / per) * T + x * per + (q % per);
}
__device__ __forceinline__ int tile_of(const KDslash &k) { return tile_of(k, (int)blockIdx.x); }


// Site coordinates of checkerboard index i on parity p.
struct Coords {
  int x1, x2, x3, x4, rest;
};
__device__ __forceinline__ Coords coords_of(const Geom &g, int i, int parity) {
  Coords c;
  c.rest = fdiv(i, g.dl1h);
  const int x1h = i - c.rest * g.L1h;
  const int r2 = fdiv(c.rest, g.dl2);
  c.x2 = c.rest - r2 * g.L[1];
  c.x4 = fdiv(r2, g.dl3);
  c.x3 = r2 - c.x4 * g.L[2];
  c.x1 = 2 * x1h + ((parity + c.x2 + c.x3 + c.x4) & 1);
  return c;
}

// Checkerboard indices of the 8 neighbours, in hop order
// (x1+, x2+, x3+, x4+, x1-, x2-, x3-, x4-).
__device__ __forceinline__ void neighbours(const Geom &g, const Coords &c, int i, int (&nb)[8]) {
  const int xp1 = (c.x1 + 1 == g.L[0]) ? 0 : c.x1 + 1;
  const int xm1 = (c.x1 == 0) ? g.L[0] - 1 : c.x1 - 1;
  nb[0] = (xp1 >> 1) + g.L1h * c.rest;
  nb[4] = (xm1 >> 1) + g.L1h * c.rest;
  nb[1] = i + ((c.x2 == g.L[1] - 1) ? -(g.L[1] - 1) * g.s2 : g.s2);
  nb[5] = i + ((c.x2 == 0) ? (g.L[1] - 1) * g.s2 : -g.s2);
  nb[2] = i + ((c.x3 == g.L[2] - 1) ? -(g.L[2] - 1) * g.s3 : g.s3);
  nb[6] = i + ((c.x3 == 0) ? (g.L[2] - 1) * g.s3 : -g.s3);
  nb[3] = i + ((c.x4 == g.L[3] - 1) ? -(g.L[3] - 1) * g.s4 : g.s4);
  nb[7] = i + ((c.x4 == 0) ? (g.L[3] - 1) * g.s4 : -g.s4);
}

// One hop: acc += M (1 + S gamma_MU) psi_nb, M = the hop link u (rows 0, 1;
// row 2 rebuilt).  Time hops (MU = 3) read only the half of the neighbour
// spinor that their projector keeps (see the spin basis in wd_device.h).
// LDAG: multiply by u^dag instead of u (u holds the rows of the link that
// the neighbour stores as its forward link).
template <int P, int MU, int S, bool LDAG = false>
__device__ __forceinline__ void hop_term_h(cplx<RealOf<P>> (&acc)[12], const cplx<RealOf<P>> (&h)[6],
                                           const cplx<RealOf<P>> (&u)[6]);

template <int P, int MU, int S, bool LDAG = false>
__device__ __forceinline__ void hop_term_u(cplx<RealOf<P>> (&acc)[12], const char *in, int nb,
                                           const cplx<RealOf<P>> (&u)[6], RealOf<P> sign) {
  using T = RealOf<P>;
  cplx<T> h[6];
  if constexpr (MU == 3) {
    Spinor<P>::template load_half<(S < 0)>(in, nb, h);
    const T f = (T)2 * sign;
#pragma unroll
    for (int c = 0; c < 6; ++c) h[c] = f * h[c];
  } else {
    cplx<T> psi[12];
    Spinor<P>::load(in, nb, psi);
    project<MU, S>(psi, h);
  }
  hop_term_h<P, MU, S, LDAG>(acc, h, u);
}

// The same for a spatial hop (MU < 3) whose neighbour spinor is already in
// registers (read from LDS by the staged kernel).
template <int P, int MU, int S>
__device__ __forceinline__ void hop_term_psi(cplx<RealOf<P>> (&acc)[12], const cplx<RealOf<P>> (&psi)[12],
                                             const cplx<RealOf<P>> (&u)[6]) {
  static_assert(MU < 3, "time hops read half spinors");
  cplx<RealOf<P>> h[6];
  project<MU, S>(psi, h);
  hop_term_h<P, MU, S>(acc, h, u);
}

// acc += reconstruct(M h): the projected half spinor h times the link.
template <int P, int MU, int S, bool LDAG>
__device__ __forceinline__ void hop_term_h(cplx<RealOf<P>> (&acc)[12], const cplx<RealOf<P>> (&h)[6],
                                           const cplx<RealOf<P>> (&u)[6]) {
  using T = RealOf<P>;
  cplx<T> r2[3];
  rebuild_row2(u, r2);
  cplx<T> g[6];
  {
    cplx<T> v[3] = {h[0], h[1], h[2]};
    cplx<T> y[3];
    if constexpr (LDAG) su3_mul_dag(u, r2, v, y);
    else su3_mul(u, r2, v, y);
    g[0] = y[0]; g[1] = y[1]; g[2] = y[2];
  }
  {
    cplx<T> v[3] = {h[3], h[4], h[5]};
    cplx<T> y[3];
    if constexpr (LDAG) su3_mul_dag(u, r2, v, y);
    else su3_mul(u, r2, v, y);
    g[3] = y[0]; g[4] = y[1]; g[5] = y[2];
  }
  reconstruct_add<MU, S>(acc, g);
}

// The same hop with the link loaded from the hop-link array (direction d).
template <int P, int MU, int S>
__device__ __forceinline__ void hop_term(cplx<RealOf<P>> (&acc)[12], const char *in, int nb,
                                         const char *links, int d, size_t i, RealOf<P> sign) {
  cplx<RealOf<P>> u[6];
  Link<RealOf<P>>::load(links, d, i, u);
  hop_term_u<P, MU, S>(acc, in, nb, u, sign);
}

// The 8 hops of site i with its links already in registers: u[d] for hop
// direction d (x1+, x2+, x3+, x4+, x1-, x2-, x3-, x4-).
template <int P, bool DAG>
__device__ __forceinline__ void hop_all_u(const char *in, const int (&nb)[8], const cplx<RealOf<P>> (&u)[8][6],
                                          RealOf<P> sf, RealOf<P> sb, cplx<RealOf<P>> (&acc)[12]) {
  using T = RealOf<P>;
  const T one = (T)1;
  constexpr int F = DAG ? -1 : 1;
  constexpr int B = -F;
#pragma unroll
  for (int c2 = 0; c2 < 12; ++c2) acc[c2] = {(T)0, (T)0};
  hop_term_u<P, 0, F>(acc, in, nb[0], u[0], one);
  hop_term_u<P, 1, F>(acc, in, nb[1], u[1], one);
  hop_term_u<P, 2, F>(acc, in, nb[2], u[2], one);
  hop_term_u<P, 3, F>(acc, in, nb[3], u[3], sf);
  hop_term_u<P, 0, B>(acc, in, nb[4], u[4], one);
  hop_term_u<P, 1, B>(acc, in, nb[5], u[5], one);
  hop_term_u<P, 2, B>(acc, in, nb[6], u[6], one);
  hop_term_u<P, 3, B>(acc, in, nb[7], u[7], sb);
}

template <int P, bool DAG>
__device__ __forceinline__ void hop_all(const KDslash &k, int i, cplx<RealOf<P>> (&acc)[12]) {
  using T = RealOf<P>;
  const Coords c = coords_of(k.g, i, k.parity);
  int nb[8];
  neighbours(k.g, c, i, nb);
  const T one = (T)1;
  const T sf = (c.x4 == k.g.L[3] - 1) ? (T)k.g.tbc : one;
  const T sb = (c.x4 == 0) ? (T)k.g.tbc : one;
  constexpr int F = DAG ? -1 : 1;  // forward hop projector (1 + F gamma)
  constexpr int B = -F;            // backward hop projector (1 + B gamma)
  const char *L = k.links;
#pragma unroll
  for (int c2 = 0; c2 < 12; ++c2) acc[c2] = {(T)0, (T)0};
  hop_term<P, 0, F>(acc, k.in, nb[0], L, 0, i, one);
  hop_term<P, 1, F>(acc, k.in, nb[1], L, 1, i, one);
  hop_term<P, 2, F>(acc, k.in, nb[2], L, 2, i, one);
  hop_term<P, 3, F>(acc, k.in, nb[3], L, 3, i, sf);
  hop_term<P, 0, B>(acc, k.in, nb[4], L, 4, i, one);
  hop_term<P, 1, B>(acc, k.in, nb[5], L, 5, i, one);
  hop_term<P, 2, B>(acc, k.in, nb[6], L, 6, i, one);
  hop_term<P, 3, B>(acc, k.in, nb[7], L, 7, i, sb);
}

// The 8 hops of site i with all 8 links loaded first: 48 (FP64) or 24
// (FP32) independent 16-byte loads in flight per lane before any arithmetic,
// at the cost of holding the links in registers.
template <int P, bool DAG>
__device__ __forceinline__ void hop_all_preload(const KDslash &k, int i, cplx<RealOf<P>> (&acc)[12]) {
  using T = RealOf<P>;
  const Coords c = coords_of(k.g, i, k.parity);
  int nb[8];
  neighbours(k.g, c, i, nb);
  const T sf = (c.x4 == k.g.L[3] - 1) ? (T)k.g.tbc : (T)1;
  const T sb = (c.x4 == 0) ? (T)k.g.tbc : (T)1;
  cplx<T> u[8][6];
#pragma unroll
  for (int d = 0; d < 8; ++d) Link<T>::load(k.links, d, i, u[d]);
  hop_all_u<P, DAG>(k.in, nb, u, sf, sb, acc);
}

// Neighbour spinors staged in LDS by a block whose tile is k whole x1 rows
// of one x3 plane (k | L2, k >= 2) or whole planes.  Slots 0 .. n-1 are the
// tile's own input sites t0 .. t0+n-1, slots n .. n+L1h-1 the x1 row before
// the tile's first row (its x2 - 1 neighbour row, wrapping in the plane)
// starting at site lo, and slots n+L1h .. n+2 L1h-1 the row after its last
// row starting at site hi: every x1 and x2 neighbour of the tile's output
// sites is one of these.  A slot holds the whole input spinor (the four x1
// and x2 hops project it four different ways) as 16-byte packets, packet-
// major: packet q (complex numbers qK .. qK+K-1, K = 16 / sizeof(cplx<T>))
// of slot s is packet q * ns + s, ns = n + 2 L1h.  Lanes that read one packet
// of consecutive slots touch consecutive 16-byte words, so the layout needs
// no padding against bank conflicts: 192 B per slot in FP64, 96 B in FP32.
template <class T>
struct __align__(16) StagePacket {
  cplx<T> v[16 / sizeof(cplx<T>)];
};
template <class T>
struct Stage {
  const cplx<T> *lds;
  int t0, n, lo, hi, l1h, ns;
};

// (every candidate computed, then selected: no branches, which would cut the
// hop into basic blocks the scheduler cannot interleave)
template <class T>
__device__ __forceinline__ int stage_slot(const Stage<T> &sv, int nb) {
  const int s = nb - sv.t0;
  const int l = nb - sv.lo;
  const int in_lo = sv.n + l;
  const int in_hi = sv.n + sv.l1h + (nb - sv.hi);
  int r = ((unsigned)l < (unsigned)sv.l1h) ? in_lo : in_hi;
  r = ((unsigned)s < (unsigned)sv.n) ? s : r;
  return r;
}

// psi into slot s of a stage of ns slots.
template <class T>
__device__ __forceinline__ void stage_store(cplx<T> *lds, int s, int ns, const cplx<T> (&psi)[12]) {
  constexpr int K = 16 / sizeof(cplx<T>);
  StagePacket<T> *p = (StagePacket<T> *)lds + s;
#pragma unroll
  for (int q = 0; q < 12 / K; ++q) {
    StagePacket<T> w;
#pragma unroll
    for (int j = 0; j < K; ++j) w.v[j] = psi[q * K + j];
    p[(size_t)q * ns] = w;
  }
}

// The spinor of slot `slot`.
template <class T>
__device__ __forceinline__ void stage_load(const Stage<T> &sv, int slot, cplx<T> (&psi)[12]) {
  constexpr int K = 16 / sizeof(cplx<T>);
  const StagePacket<T> *p = (const StagePacket<T> *)sv.lds + slot;
#pragma unroll
  for (int q = 0; q < 12 / K; ++q) {
    const StagePacket<T> w = p[(size_t)q * sv.ns];
#pragma unroll
    for (int j = 0; j < K; ++j) psi[q * K + j] = w.v[j];
  }
}

// A spatial hop (x1 or x2) with the neighbour's projection from the staged
// tile: the same values as projected from memory, so the result is bitwise
// that of hop_term.
template <int P, int MU, int S>
__device__ __forceinline__ void staged_term(cplx<RealOf<P>> (&acc)[12], const KDslash &k, const Stage<RealOf<P>> &sv,
                                            int nb, int d, size_t i) {
  using T = RealOf<P>;
  static_assert(MU < 2, "x1 and x2 hops only");
  cplx<T> u[6];
  Link<T>::load(k.links, d, i, u);
  cplx<T> psi[12];
  stage_load(sv, stage_slot(sv, nb), psi);
  hop_term_psi<P, MU, S>(acc, psi, u);
  // FP64: one hop at a time (started all at once, the hops' operands exceed
  // the registers); FP32 keeps the early loads, which hide more latency
  if constexpr (P == WD_F64) __builtin_amdgcn_sched_barrier(0);
}

// The same with the link already in registers.
template <int P, int MU, int S>
__device__ __forceinline__ void staged_term_u(cplx<RealOf<P>> (&acc)[12], const Stage<RealOf<P>> &sv, int nb,
                                              const cplx<RealOf<P>> (&u)[6]) {
  using T = RealOf<P>;
  cplx<T> psi[12];
  stage_load(sv, stage_slot(sv, nb), psi);
  hop_term_psi<P, MU, S>(acc, psi, u);
}

// A time hop on a half spinor h already loaded (load_half of the hop's
// projector), the same arithmetic as hop_term_u's time path.
template <int P, int S>
__device__ __forceinline__ void hop_term_x4(cplx<RealOf<P>> (&acc)[12], const cplx<RealOf<P>> (&hraw)[6],
                                            const cplx<RealOf<P>> (&u)[6], RealOf<P> sign) {
  using T = RealOf<P>;
  const T f = (T)2 * sign;
  cplx<T> h[6];
#pragma unroll
  for (int c = 0; c < 6; ++c) h[c] = f * hraw[c];
  hop_term_h<P, 3, S>(acc, h, u);
}

// The 8 hops with the x1 and x2 neighbours read from the staged tile, the x3
// and x4 neighbours from memory.  Same hop order and arithmetic as hop_all.
// FP32: every link and every neighbour in memory is loaded before the first
// hop (the loads in flight hide more latency); FP64 takes one hop at a time
// (its operands would not fit the registers all at once).
template <int P, bool DAG>
__device__ __forceinline__ void hop_all_staged(const KDslash &k, int i, const Stage<RealOf<P>> &sv,
                                               cplx<RealOf<P>> (&acc)[12]) {
  using T = RealOf<P>;
  const Coords c = coords_of(k.g, i, k.parity);
  int nb[8];
  neighbours(k.g, c, i, nb);
  const T one = (T)1;
  const T sf = (c.x4 == k.g.L[3] - 1) ? (T)k.g.tbc : one;
  const T sb = (c.x4 == 0) ? (T)k.g.tbc : one;
  constexpr int F = DAG ? -1 : 1;
  constexpr int B = -F;
  const char *L = k.links;
  if constexpr (P == WD_F32) {
    cplx<T> u[8][6];
#pragma unroll
    for (int d = 0; d < 8; ++d) Link<T>::load(L, d, i, u[d]);
    cplx<T> p2f[12], p2b[12], h3f[6], h3b[6];
    Spinor<P>::load(k.in, nb[2], p2f);
    Spinor<P>::load(k.in, nb[6], p2b);
    Spinor<P>::template load_half<(F < 0)>(k.in, nb[3], h3f);
    Spinor<P>::template load_half<(B < 0)>(k.in, nb[7], h3b);
#pragma unroll
    for (int c2 = 0; c2 < 12; ++c2) acc[c2] = {(T)0, (T)0};
    staged_term_u<P, 0, F>(acc, sv, nb[0], u[0]);
    staged_term_u<P, 1, F>(acc, sv, nb[1], u[1]);
    hop_term_psi<P, 2, F>(acc, p2f, u[2]);
    hop_term_x4<P, F>(acc, h3f, u[3], sf);
    staged_term_u<P, 0, B>(acc, sv, nb[4], u[4]);
    staged_term_u<P, 1, B>(acc, sv, nb[5], u[5]);
    hop_term_psi<P, 2, B>(acc, p2b, u[6]);
    hop_term_x4<P, B>(acc, h3b, u[7], sb);
    return;
  }
#pragma unroll
  for (int c2 = 0; c2 < 12; ++c2) acc[c2] = {(T)0, (T)0};
  constexpr bool one_at_a_time = (P == WD_F64);
  staged_term<P, 0, F>(acc, k, sv, nb[0], 0, i);
  staged_term<P, 1, F>(acc, k, sv, nb[1], 1, i);
  hop_term<P, 2, F>(acc, k.in, nb[2], L, 2, i, one);
  if constexpr (one_at_a_time) __builtin_amdgcn_sched_barrier(0);
  hop_term<P, 3, F>(acc, k.in, nb[3], L, 3, i, sf);
  if constexpr (one_at_a_time) __builtin_amdgcn_sched_barrier(0);
  staged_term<P, 0, B>(acc, k, sv, nb[4], 4, i);
  staged_term<P, 1, B>(acc, k, sv, nb[5], 5, i);
  hop_term<P, 2, B>(acc, k.in, nb[6], L, 6, i, one);
  if constexpr (one_at_a_time) __builtin_amdgcn_sched_barrier(0);
  hop_term<P, 3, B>(acc, k.in, nb[7], L, 7, i, sb);
}

// One output site i of the hop with the fused epilogue
//   EPI 0: out = a H in;  1: out = X + a H in;  2: out = X - Y + a H in.
// Padding slots (vh <= i < vpad) get zeros.  Returns |stored out|^2 (FP64)
// when NORM, else 0.  PRE: links loaded up front (same arithmetic).  STG:
// x1, x2 neighbours from the block's staged input tile sv.
template <int P, bool DAG, int EPI, bool NORM, bool PRE = false, bool STG = false>
__device__ __forceinline__ double dslash_site(const KDslash &k, int i, Stage<RealOf<P>> sv = {}) {
  using T = RealOf<P>;
  double nrm = 0.0;
  if (i < k.g.vh) {
    cplx<T> acc[12];
    if constexpr (PRE) hop_all_preload<P, DAG>(k, i, acc);
    else if constexpr (STG) hop_all_staged<P, DAG>(k, i, sv, acc);
    else hop_all<P, DAG>(k, i, acc);
    const T a = (T)k.a;
#pragma unroll
    for (int c = 0; c < 12; ++c) acc[c] = a * acc[c];
    if constexpr (EPI >= 1) {
      cplx<T> x[12];
      Spinor<P>::load(k.X, i, x);
#pragma unroll
      for (int c = 0; c < 12; ++c) acc[c] = acc[c] + x[c];
    }
    if constexpr (EPI == 2) {
      cplx<T> y[12];
      Spinor<P>::load(k.Y, i, y);
#pragma unroll
      for (int c = 0; c < 12; ++c) acc[c] = acc[c] - y[c];
    }
    if (k.nt_store) Spinor<P>::template store<true>(k.out, i, acc);
    else Spinor<P>::template store<false>(k.out, i, acc);
    if constexpr (NORM) {
      // norm of what was stored (after rounding to the storage format)
      cplx<T> st[12];
      if constexpr (P == WD_F64 || P == WD_F32) {
#pragma unroll
        for (int c = 0; c < 12; ++c) st[c] = acc[c];
      } else {
        Spinor<P>::load(k.out, i, st);
      }
#pragma unroll
      for (int c = 0; c < 12; ++c) nrm += (double)st[c].re * st[c].re + (double)st[c].im * st[c].im;
    }
  } else if (i < k.g.vpad) {
    cplx<T> z[12];
#pragma unroll
    for (int c = 0; c < 12; ++c) z[c] = {(T)0, (T)0};
    Spinor<P>::store(k.out, i, z);
  }
  return nrm;
}

// ---------------------------------------------- one wave per hop direction
// A block of 8 waves serves 64 output sites: wave d takes hop d of every
// site (link and neighbour spinor loaded, projected, multiplied) and leaves
// the transported half spinor in LDS; after one barrier a few waves add the
// eight contributions of each output component in hop order, with the same
// arithmetic as hop_all, so the result is the same bit for bit.
//
// A lane's chain is one load latency and one link multiply instead of eight,
// and a CU holds 24 (FP64) or 32 waves (one hop's operands fit 80 or 54
// registers) instead of 8 to 12.
//
// LDS: component c of hop d at site s is element (6 d + c) 64 + s, so the
// lanes of a wave touch consecutive words: 48 KiB in FP64, 24 KiB else (FP16 768
// bytes more).
constexpr int SPLIT_SITES = 64;
constexpr int SPLIT_BS = 512;
template <int P>
struct SplitMax {};
template <>
struct SplitMax<WD_F16> {
  float mx[3][SPLIT_SITES];  // a site's largest number among each summing wave's components
};
template <int P>
struct SplitLds : SplitMax<P> {
  cplx<RealOf<P>> g[8 * 6 * SPLIT_SITES];
  // |component C|^2 of an output (norm epilogue): in the time-hop element that
  // only component C adds up, free once it has
  template <bool DAG, int C>
  __device__ __forceinline__ double &n2(int lane) {
    constexpr int d = ((C < 6) != DAG) ? 3 : 7;
    return *(double *)&g[(6 * d + C % 6) * SPLIT_SITES + lane];
  }
};
// waves per SIMD the register budget is held to (a block adds 2 to each SIMD)
constexpr int split_occ(int prec) {
  return prec == WD_F64 ? 6 : 8;
}

// Checkerboard index of the neighbour of site i (parity p) in direction MU,
// forward or backward; edge: the hop crosses the time boundary.
template <int MU, bool FWD>
__device__ __forceinline__ int neighbour_of(const Geom &g, int i, int p, bool &edge) {
  edge = false;
  const int rest = fdiv(i, g.dl1h);
  const int r2 = fdiv(rest, g.dl2);
  const int x4 = fdiv(r2, g.dl3);
  if constexpr (MU == 0) {
    const int x1h = i - rest * g.L1h;
    // the extents are even: x2 and x3 have the parities of rest and r2
    const int odd = (p + rest + r2 + x4) & 1;
    int y = x1h;
    if (FWD && odd) y = (x1h + 1 == g.L1h) ? 0 : x1h + 1;
    if (!FWD && !odd) y = (x1h == 0) ? g.L1h - 1 : x1h - 1;
    return y + g.L1h * rest;
  } else {
    const int x = (MU == 1) ? rest - r2 * g.L[1] : (MU == 2) ? r2 - x4 * g.L[2] : x4;
    const int s = (MU == 1) ? g.s2 : (MU == 2) ? g.s3 : g.s4;
    const int last = g.L[MU] - 1;
    if (FWD) {
      edge = MU == 3 && x == last;
      return i + ((x == last) ? -last * s : s);
    }
    edge = MU == 3 && x == 0;
    return i + ((x == 0) ? last * s : -s);
  }
}

// Hop D of site i: the transported half spinor into LDS.
template <int P, bool DAG, int D>
__device__ __forceinline__ void split_hop(const KDslash &k, int i, int lane, SplitLds<P> &lds) {
  using T = RealOf<P>;
  constexpr int MU = D & 3;
  constexpr bool FWD = D < 4;
  constexpr int S = (FWD != DAG) ? 1 : -1;
  bool edge;
  const int nb = neighbour_of<MU, FWD>(k.g, i, k.parity, edge);
  cplx<T> u[6], h[6], r2[3];
  Link<T>::load(k.links, D, i, u);
  if constexpr (MU == 3) {
    Spinor<P>::template load_half<(S < 0)>(k.in, nb, h);
    const T f = (T)2 * (edge ? (T)k.g.tbc : (T)1);
#pragma unroll
    for (int c = 0; c < 6; ++c) h[c] = f * h[c];
  } else {
    cplx<T> psi[12];
    Spinor<P>::load(k.in, nb, psi);
    project<MU, S>(psi, h);
  }
  cplx<T> *q = lds.g + D * 6 * SPLIT_SITES + lane;
  // rows 0 and 1 first, the rebuilt row last: the spinor is dead before the
  // products start and the stored rows before the last two are (FP64: 72
  // registers of operands of the 80 that three blocks a CU leave each lane)
  if constexpr (P == WD_F64) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      cplx<T> y = u[3 * a] * h[3 * s];
      cfma(y, u[3 * a + 1], h[3 * s + 1]);
      cfma(y, u[3 * a + 2], h[3 * s + 2]);
      q[(3 * s + a) * SPLIT_SITES] = y;
    }
  if constexpr (P == WD_F64) __builtin_amdgcn_sched_barrier(0);
  rebuild_row2(u, r2);
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    cplx<T> y = r2[0] * h[3 * s];
    cfma(y, r2[1], h[3 * s + 1]);
    cfma(y, r2[2], h[3 * s + 2]);
    q[(3 * s + 2) * SPLIT_SITES] = y;
  }
}

template <int P, bool DAG>
__device__ __forceinline__ void split_hops(const KDslash &k, int i, int w, int lane, SplitLds<P> &lds) {
  switch (w) {
    case 0: split_hop<P, DAG, 0>(k, i, lane, lds); break;
    case 1: split_hop<P, DAG, 1>(k, i, lane, lds); break;
    case 2: split_hop<P, DAG, 2>(k, i, lane, lds); break;
    case 3: split_hop<P, DAG, 3>(k, i, lane, lds); break;
    case 4: split_hop<P, DAG, 4>(k, i, lane, lds); break;
    case 5: split_hop<P, DAG, 5>(k, i, lane, lds); break;
    case 6: split_hop<P, DAG, 6>(k, i, lane, lds); break;
    default: split_hop<P, DAG, 7>(k, i, lane, lds); break;
  }
}

// Output component C of the lane's site: the sum over the hops, in hop order,
// of what reconstruct_add adds to it.
template <int P, bool DAG, int C>
__device__ __forceinline__ cplx<RealOf<P>> split_sum(const SplitLds<P> &lds, int lane) {
  using T = RealOf<P>;
  constexpr int sp = C / 3, a = C % 3;
  const cplx<T> *g = lds.g + lane;
  cplx<T> acc = {(T)0, (T)0};
#pragma unroll
  for (int d = 0; d < 8; ++d) {
    const int mu = d & 3, S = ((d < 4) != DAG) ? 1 : -1;
    const T s = (T)S;
    if (mu == 3 && (sp < 2) != (S > 0)) continue;
    const int h = (sp < 2 || mu == 3) ? (sp & 1) : (mu == 2 ? sp - 2 : 3 - sp);  // which spin row of g
    const cplx<T> v = g[(6 * d + 3 * h + a) * SPLIT_SITES];
    if (sp < 2 || mu == 3) acc = acc + v;
    else if (mu == 0) acc = acc + s * mul_i(v);
    else if (mu == 1) acc = (sp == 2) ? acc - s * v : acc + s * v;
    else acc = (sp == 2) ? acc + s * mul_i(v) : acc - s * mul_i(v);
  }
  if constexpr (P == WD_F16) __builtin_amdgcn_sched_barrier(0);  // one component's operands at a time
  return acc;
}

// Components [0, 12) are summed by NW waves, CW components each: whole
// 16-byte packets of the storage format.  (FP16's scale is the site's largest
// number: the waves exchange theirs in LDS before they store.)
template <int P>
struct SplitOut {
  static constexpr int CW = (P == WD_F64 || P == WD_F32) ? 2 : 4;
  static constexpr int NW = 12 / CW;
};

// Components W CW .. of a stored spinor (w = W may be a run-time value).
template <int P>
__device__ __forceinline__ void split_load(const char *base, int i, int w, cplx<RealOf<P>> (&x)[SplitOut<P>::CW]) {
  if constexpr (P == WD_F64) {
    const v2d *p = (const v2d *)base + chunk_base<Spinor<P>::CHUNK>((size_t)i) + 64 * 2 * w;
    const v2d a = p[0], b = p[64];
    x[0] = {a.x, a.y};
    x[1] = {b.x, b.y};
  } else if constexpr (P == WD_F32) {
    const v4f v = *((const v4f *)base + chunk_base<Spinor<P>::CHUNK>((size_t)i) + 64 * w);
    x[0] = {v.x, v.y};
    x[1] = {v.z, v.w};
  } else if constexpr (P == WD_BF16) {
    Packet<WD_BF16>::unpack(*((const v4u *)base + chunk_base<Spinor<P>::CHUNK>((size_t)i) + 64 * w), x);
  } else {
    const v4u v = *((const v4u *)base + chunk_base<Spinor<P>::CHUNK>((size_t)i) + 64 * w);
    const float n = Spinor<P>::scale(base, (size_t)i);
    const uint32_t q[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int j = 0; j < 4; ++j)
      x[j] = {n * f16_to_f32((uint16_t)(q[j] & 0xffffu)), n * f16_to_f32((uint16_t)(q[j] >> 16))};
  }
}

// Stores them (FP16: with the site's scale m); on return x holds the stored
// (rounded) values when NORM.
template <int P, int W, bool NT, bool NORM>
__device__ __forceinline__ void split_store(char *base, int i, cplx<RealOf<P>> (&x)[SplitOut<P>::CW], float m) {
  if constexpr (P == WD_F64) {
    v2d *p = (v2d *)base + chunk_base<Spinor<P>::CHUNK>((size_t)i) + 64 * 2 * W;
    st_policy<NT>(v2d{x[0].re, x[0].im}, p);
    st_policy<NT>(v2d{x[1].re, x[1].im}, p + 64);
  } else if constexpr (P == WD_F32) {
    st_policy<NT>(v4f{x[0].re, x[0].im, x[1].re, x[1].im},
                  (v4f *)base + chunk_base<Spinor<P>::CHUNK>((size_t)i) + 64 * W);
  } else if constexpr (P == WD_BF16) {
    uint32_t w[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) w[j] = pack_bf16(x[j].re, x[j].im);
    st_policy<NT>(v4u{w[0], w[1], w[2], w[3]}, (v4u *)base + chunk_base<Spinor<P>::CHUNK>((size_t)i) + 64 * W);
    if constexpr (NORM) {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        x[j] = {bf16_to_f32((uint16_t)(w[j] & 0xffffu)), bf16_to_f32((uint16_t)(w[j] >> 16))};
    }
  } else {
    const float inv = m > 0.f ? 1.0f / m : 0.f;
    v4u *p = (v4u *)base + chunk_base<Spinor<P>::CHUNK>((size_t)i);
    uint32_t w[4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
      w[j] = (uint32_t)f32_to_f16(x[j].re * inv) | ((uint32_t)f32_to_f16(x[j].im * inv) << 16);
    st_policy<NT>(v4u{w[0], w[1], w[2], w[3]}, p + 64 * W);
    if constexpr (W == 0)
      st_policy<NT>(m, (float *)((v4u *)base + ((size_t)i >> 6) * Spinor<P>::CHUNK + 3 * 64) + (i & 63));
    if constexpr (NORM) {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        x[j] = {m * f16_to_f32((uint16_t)(w[j] & 0xffffu)), m * f16_to_f32((uint16_t)(w[j] >> 16))};
    }
  }
}

// FP16: the site's largest number, from the components of the NW summing waves
// (a barrier of the block, which the other waves join with split_max_rest).
template <int W>
__device__ __forceinline__ float split_max(const cplx<float> (&x)[4], SplitLds<WD_F16> &lds, int lane) {
  float m = 0.f;
#pragma unroll
  for (int j = 0; j < 4; ++j) m = fmaxf(m, fmaxf(fabsf(x[j].re), fabsf(x[j].im)));
  lds.mx[W][lane] = m;
  __syncthreads();
  return fmaxf(fmaxf(lds.mx[0][lane], lds.mx[1][lane]), lds.mx[2][lane]);
}
template <int P>
__device__ __forceinline__ void split_max_rest() {
  if constexpr (P == WD_F16) __syncthreads();
}

// The epilogue of wave W's components of site i (EPI 0 and 1 of dslash_site).
template <int P, bool DAG, int EPI, bool NORM, int W, int... J>
__device__ __forceinline__ void split_finish_w(const KDslash &k, int i, int lane, SplitLds<P> &lds,
                                               const cplx<RealOf<P>> (&x)[SplitOut<P>::CW],
                                               std::integer_sequence<int, J...>) {
  using T = RealOf<P>;
  constexpr int CW = SplitOut<P>::CW;
  cplx<T> o[CW];
  if (i < k.g.vh) {
    const T a = (T)k.a;
    ((o[J] = split_sum<P, DAG, W * CW + J>(lds, lane)), ...);
#pragma unroll
    for (int j = 0; j < CW; ++j) {
      o[j] = a * o[j];
      if constexpr (EPI >= 1) o[j] = o[j] + x[j];
    }
  } else {
#pragma unroll
    for (int j = 0; j < CW; ++j) o[j] = {(T)0, (T)0};
  }
  float m = 0.f;
  if constexpr (P == WD_F16) m = split_max<W>(o, lds, lane);
  if (k.nt_store) split_store<P, W, true, NORM>(k.out, i, o, m);
  else split_store<P, W, false, NORM>(k.out, i, o, m);
  if constexpr (NORM)
    ((lds.template n2<DAG, W * CW + J>(lane) = (double)o[J].re * o[J].re + (double)o[J].im * o[J].im), ...);
}

template <int P, bool DAG, int EPI, bool NORM, int W>
__device__ __forceinline__ void split_wave(const KDslash &k, int i, int lane, SplitLds<P> &lds) {
  using T = RealOf<P>;
  constexpr int CW = SplitOut<P>::CW;
  // the epilogue operand is loaded before the barrier
  cplx<T> x[CW];
  if constexpr (EPI >= 1)
    if (i < k.g.vh) split_load<P>(k.X, i, W, x);
  __syncthreads();
  split_finish_w<P, DAG, EPI, NORM, W>(k, i, lane, lds, x, std::make_integer_sequence<int, CW>{});
}

template <int P, bool DAG, int... C>
__device__ __forceinline__ double split_norm(SplitLds<P> &lds, int lane, std::integer_sequence<int, C...>) {
  double nrm = 0.0;
  ((nrm += lds.template n2<DAG, C>(lane)), ...);
  return nrm;
}

// Tile of block b in the order SPLIT_RANGES: dispatch lane b % 8 (one per
// XCD) takes the b % 8-th of eight contiguous ranges of tiles, on any
// lattice, so a tile's x1..x3 neighbours and most x4 ones are fetched into
// one L2.  The grid is 8 ceil(ntiles / 8); a tile >= ntiles is empty.
constexpr int SPLIT_RANGES = WD_ORDER_RANGES;
__device__ __forceinline__ int split_tile_of(const KDslash &k, int b) {
  if (k.groups == SPLIT_RANGES) return (b & 7) * k.tiles_per_slice + (b >> 3);
  return tile_of(k, b);
}

// 64 output sites of the hop by a block of SPLIT_BS threads: sites 64 tile ..
// Returns the tile's |out|^2 in thread 0 when NORM (the same sum as a 64-site
// block of dslash_site), else 0.
template <int P, bool DAG, int EPI, bool NORM>
__device__ __forceinline__ double dslash_split_tile(const KDslash &k, int tile, SplitLds<P> &lds) {
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = (int)threadIdx.x & 63;
  const int i = tile * SPLIT_SITES + lane;
  if (i < k.g.vh) split_hops<P, DAG>(k, i, w, lane, lds);
  constexpr int NW = SplitOut<P>::NW;
  switch (w) {
    case 0: split_wave<P, DAG, EPI, NORM, 0>(k, i, lane, lds); break;
    case 1: if constexpr (NW > 1) { split_wave<P, DAG, EPI, NORM, 1>(k, i, lane, lds); break; }
    case 2: if constexpr (NW > 1) { split_wave<P, DAG, EPI, NORM, 2>(k, i, lane, lds); break; }
    case 3: if constexpr (NW > 3) { split_wave<P, DAG, EPI, NORM, 3>(k, i, lane, lds); break; }
    case 4: if constexpr (NW > 3) { split_wave<P, DAG, EPI, NORM, 4>(k, i, lane, lds); break; }
    case 5: if constexpr (NW > 3) { split_wave<P, DAG, EPI, NORM, 5>(k, i, lane, lds); break; }
    default:
      __syncthreads();
      split_max_rest<P>();
      break;
  }
  double nrm = 0.0;
  if constexpr (NORM) {
    __syncthreads();
    if (w == 0) {
      if (i < k.g.vh) nrm = split_norm<P, DAG>(lds, lane, std::make_integer_sequence<int, 12>{});
      nrm = wave_sum(nrm);
    }
  }
  return nrm;
}

}  // namespace wd
