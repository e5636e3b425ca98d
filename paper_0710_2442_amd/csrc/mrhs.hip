// Multi right-hand-side Wilson hop (Eq. 3 on one checkerboard), gfx950:
// nrhs half fields share every link load.
#include <algorithm>

#include "wd_hop.h"

namespace wd {

// ---------------------------------------------------------------- mrhs
// Lanes of a wave cover 16 sites x 4 right-hand sides (lane = site + 16*rhs),
// so the four lanes of one site issue the same link addresses and the
// hardware merges them into one fetch; the waves of a block stack RHS groups
// of the same 16 sites so the links stay in L1/L2 for the whole block.
// Per-RHS epilogue as in k_dslash, per-RHS skip flags and FP64 norms.
struct KMrhs {
  KDslash k;
  int nrhs;
  size_t rhs_stride;   // bytes between right-hand sides (all operands)
  int skip_stride;     // ints between consecutive RHS skip flags
  int rpl;             // right-hand sides per lane (FP32-arithmetic kernel)
  int nx3;             // > 0: box order with tile-major RHS chunks (mrhs_box)
  int nchunks;         // RHS chunks of rpl right-hand sides
  int ntiles;          // tiles of one parity
};

// Box order for the multi-RHS hop.  Dispatch lane x = b % 8 (one per XCD)
// owns one box: a contiguous 1/nx3 of the tiles of every time slice in a
// range of 8/nx3 of the slices (boxes nx3 along the slice, 8/nx3 along x4).
// The lane walks its box slice by slice, and the nchunks blocks of one tile
// (its RHS chunks) follow each other, so they run side by side on one XCD:
// the tile's links are fetched into that L2 once, and the sites in flight
// on an XCD, whose neighbours of all right-hand sides the L2 must hold, are
// fewer by the number of chunks; the next slice of the box (the time
// neighbours) is one box-slice away.  Sets the tile and the RHS chunk of
// block b.
__device__ __forceinline__ void mrhs_box(const KMrhs &m, int b, int &tile, int &chunk) {
  const int x = b & 7, q = b >> 3;
  const int T = m.k.tiles_per_slice, Tb = T / m.nx3, S = m.k.g.L[3] / (8 / m.nx3);
  const int tq = q / m.nchunks;
  chunk = q % m.nchunks;
  const int bx = x % m.nx3, bt = x / m.nx3;
  tile = (bt * S + tq / Tb) * T + bx * Tb + tq % Tb;
}

template <int P, bool DAG, int EPI, bool NORM>
__global__ __launch_bounds__(256) void k_dslash_mrhs(KMrhs m) {
  using T = RealOf<P>;
  const int lane = threadIdx.x & 15;
  const int rl = threadIdx.x >> 4;             // rhs within the block
  const int rg = blockIdx.y * 16 + rl;         // global rhs
  const int i = tile_of(m.k) * 16 + lane;
  const bool live = rg < m.nrhs && !(m.k.skip && m.k.skip[(size_t)rg * m.skip_stride]);
  double nrm = 0.0;
  if (live) {
    KDslash k = m.k;
    const size_t off = (size_t)rg * m.rhs_stride;
    k.in = m.k.in + off;
    char *out = m.k.out + off;
    if (i < k.g.vh) {
      cplx<T> acc[12];
      hop_all<P, DAG>(k, i, acc);
      const T a = (T)k.a;
#pragma unroll
      for (int c = 0; c < 12; ++c) acc[c] = a * acc[c];
      if constexpr (EPI >= 1) {
        cplx<T> x[12];
        Spinor<P>::load(m.k.X + off, i, x);
#pragma unroll
        for (int c = 0; c < 12; ++c) acc[c] = acc[c] + x[c];
      }
      if constexpr (EPI == 2) {
        cplx<T> y[12];
        Spinor<P>::load(m.k.Y + off, i, y);
#pragma unroll
        for (int c = 0; c < 12; ++c) acc[c] = acc[c] - y[c];
      }
      Spinor<P>::store(out, i, acc);
      if constexpr (NORM) {
        cplx<T> st[12];
        if constexpr (P == WD_F64 || P == WD_F32) {
#pragma unroll
          for (int c = 0; c < 12; ++c) st[c] = acc[c];
        } else {
          Spinor<P>::load(out, i, st);
        }
#pragma unroll
        for (int c = 0; c < 12; ++c) nrm += (double)st[c].re * st[c].re + (double)st[c].im * st[c].im;
      }
    } else if (i < k.g.vpad) {
      cplx<T> z[12];
#pragma unroll
      for (int c = 0; c < 12; ++c) z[c] = {(T)0, (T)0};
      Spinor<P>::store(out, i, z);
    }
  }
  if constexpr (NORM) {
    // the 16 lanes of one RHS are contiguous in a wave: reduce within them;
    // the per-RHS block partials are summed by the finishing kernel
#pragma unroll
    for (int off = 8; off > 0; off >>= 1) nrm += __shfl_xor(nrm, off, 64);
    if (lane == 0 && rg < m.nrhs) m.k.partials[(size_t)rg * gridDim.x + blockIdx.x] = nrm;
  }
}

// Multi-RHS hop for FP32 arithmetic (FP32, FP16 and BF16 spinors): one lane
// per output site loads its 8 hop links once into registers and then walks
// the m.rpl right-hand sides of its block's chunk (grid.y = chunk), so a link
// is read once per chunk and every spinor load of a wave is one contiguous
// run.  Chunks are dispatched one after the other (grid.x fastest), so the
// blocks resident at one time share a chunk and their neighbour spinors stay
// in L2; rpl trades that locality against link reuse and is tuned.  Per-RHS
// skip flags, epilogue and FP64 norms as in the kernel above.
constexpr int MR_CHUNK = 16;  // largest rpl

template <int P, bool DAG, int EPI, bool NORM>
__global__ __launch_bounds__(256) void k_dslash_mrhs_reg(KMrhs m) {
  using T = RealOf<P>;
  const KDslash &k = m.k;
  int tile, chunk;
  if (m.nx3 > 0) {
    mrhs_box(m, (int)blockIdx.x, tile, chunk);
  } else {
    tile = tile_of(k);
    chunk = (int)blockIdx.y;
  }
  const int i = tile * (int)blockDim.x + (int)threadIdx.x;
  const int r0 = chunk * m.rpl;
  const int r1 = min(m.nrhs, r0 + m.rpl);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  __shared__ double sred[MR_CHUNK][4];
  const bool site = i < k.g.vh;
  int nb[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  cplx<T> u[8][6];
  T sf = (T)1, sb = (T)1;
  if (site) {
    const Coords c = coords_of(k.g, i, k.parity);
    neighbours(k.g, c, i, nb);
    if (c.x4 == k.g.L[3] - 1) sf = (T)k.g.tbc;
    if (c.x4 == 0) sb = (T)k.g.tbc;
#pragma unroll
    for (int d = 0; d < 8; ++d) Link<T>::load(k.links, d, i, u[d]);
  }
  const T a = (T)k.a;
  for (int r = r0; r < r1; ++r) {
    const bool live = !(k.skip && k.skip[(size_t)r * m.skip_stride]);
    double nrm = 0.0;
    if (live) {
      const size_t off = (size_t)r * m.rhs_stride;
      char *out = k.out + off;
      if (site) {
        cplx<T> acc[12];
        hop_all_u<P, DAG>(k.in + off, nb, u, sf, sb, acc);
#pragma unroll
        for (int c = 0; c < 12; ++c) acc[c] = a * acc[c];
        if constexpr (EPI >= 1) {
          cplx<T> x[12];
          Spinor<P>::load(k.X + off, i, x);
#pragma unroll
          for (int c = 0; c < 12; ++c) acc[c] = acc[c] + x[c];
        }
        if constexpr (EPI == 2) {
          cplx<T> y[12];
          Spinor<P>::load(k.Y + off, i, y);
#pragma unroll
          for (int c = 0; c < 12; ++c) acc[c] = acc[c] - y[c];
        }
        Spinor<P>::store(out, i, acc);
        if constexpr (NORM) {
          cplx<T> st[12];
          if constexpr (P == WD_F32) {
#pragma unroll
            for (int c = 0; c < 12; ++c) st[c] = acc[c];
          } else {
            Spinor<P>::load(out, i, st);
          }
#pragma unroll
          for (int c = 0; c < 12; ++c) nrm += (double)st[c].re * st[c].re + (double)st[c].im * st[c].im;
        }
      } else if (i < k.g.vpad) {
        cplx<T> z[12];
#pragma unroll
        for (int c = 0; c < 12; ++c) z[c] = {(T)0, (T)0};
        Spinor<P>::store(out, i, z);
      }
    }
    if constexpr (NORM) {
      const double t = wave_sum(nrm);
      if (lane == 0) sred[r - r0][w] = t;
    }
  }
  if constexpr (NORM) {
    // per-RHS partials at partials[r * ntiles + tile], summed in tile order
    // by the finishing kernel (the same sum for every schedule)
    __syncthreads();
    if (threadIdx.x == 0) {
      const int nw = (int)blockDim.x >> 6;
      for (int r = r0; r < r1; ++r) {
        double s = 0.0;
        for (int q = 0; q < nw; ++q) s += sred[r - r0][q];
        k.partials[(size_t)r * m.ntiles + tile] = s;
      }
    }
  }
}


// ---------------------------------------------- one wave per hop direction
// The packets of one neighbour spinor (or of the half that a time hop keeps),
// loaded one right-hand side ahead and unpacked when used: in 16-bit storage
// they take half the registers of the numbers.
template <int P>
struct NbRaw;
template <>
struct NbRaw<WD_F64> {
  cplx<double> s[12];
  // time: the half of the spinor (lower: spins 2, 3) that the hop keeps
  __device__ __forceinline__ void load(const char *in, int nb, bool time, bool lower) {
    const v2d *p = (const v2d *)in + chunk_base<Spinor<WD_F64>::CHUNK>((size_t)nb) + (lower ? 6 * 64 : 0);
#pragma unroll
    for (int c = 0; c < 6; ++c) {
      const v2d v = p[64 * c];
      s[c] = {v.x, v.y};
    }
    if (time) return;
#pragma unroll
    for (int c = 6; c < 12; ++c) {
      const v2d v = p[64 * c];
      s[c] = {v.x, v.y};
    }
  }
  // the spinor, or the half (components 0 .. 5 of what was loaded) of a time hop
  __device__ __forceinline__ void whole(cplx<double> (&psi)[12]) const {
#pragma unroll
    for (int c = 0; c < 12; ++c) psi[c] = s[c];
  }
  template <bool LOWER>
  __device__ __forceinline__ void half(cplx<double> (&h)[6]) const {
#pragma unroll
    for (int c = 0; c < 6; ++c) h[c] = s[c];
  }
};
template <>
struct NbRaw<WD_F32> {
  v4f a, b, c, d, e, f;
  __device__ __forceinline__ void load(const char *in, int nb, bool time, bool lower) {
    const v4f *p = (const v4f *)in + chunk_base<Spinor<WD_F32>::CHUNK>((size_t)nb) + (lower ? 192 : 0);
    a = p[0]; b = p[64]; c = p[128];
    if (!time) { d = p[192]; e = p[256]; f = p[320]; }
  }
  template <bool LOWER>
  __device__ __forceinline__ void half(cplx<float> (&h)[6]) const {
    h[0] = {a.x, a.y}; h[1] = {a.z, a.w}; h[2] = {b.x, b.y}; h[3] = {b.z, b.w}; h[4] = {c.x, c.y}; h[5] = {c.z, c.w};
  }
  __device__ __forceinline__ void whole(cplx<float> (&s)[12]) const {
    s[0] = {a.x, a.y}; s[1] = {a.z, a.w}; s[2] = {b.x, b.y}; s[3] = {b.z, b.w};
    s[4] = {c.x, c.y}; s[5] = {c.z, c.w}; s[6] = {d.x, d.y}; s[7] = {d.z, d.w};
    s[8] = {e.x, e.y}; s[9] = {e.z, e.w}; s[10] = {f.x, f.y}; s[11] = {f.z, f.w};
  }
};
template <int P>
struct NbRaw16 {
  v4u a, b, c;
  float n;  // FP16: the site's scale
  // components 6h .. 6h+5 live in packets (0, 1) or (1, 2)
  __device__ __forceinline__ void load(const char *in, int nb, bool time, bool lower) {
    const v4u *p = (const v4u *)in + chunk_base<Spinor<P>::CHUNK>((size_t)nb) + (lower ? 64 : 0);
    a = p[0]; b = p[64];
    if (!time) c = p[128];
    if constexpr (P == WD_F16) n = Spinor<P>::scale(in, (size_t)nb);
  }
  __device__ __forceinline__ cplx<float> num(uint32_t w) const {
    if constexpr (P == WD_F16) return {n * f16_to_f32((uint16_t)(w & 0xffffu)), n * f16_to_f32((uint16_t)(w >> 16))};
    else return {bf16_to_f32((uint16_t)(w & 0xffffu)), bf16_to_f32((uint16_t)(w >> 16))};
  }
  __device__ __forceinline__ void whole(cplx<float> (&s)[12]) const {
    s[0] = num(a.x); s[1] = num(a.y); s[2] = num(a.z); s[3] = num(a.w);
    s[4] = num(b.x); s[5] = num(b.y); s[6] = num(b.z); s[7] = num(b.w);
    s[8] = num(c.x); s[9] = num(c.y); s[10] = num(c.z); s[11] = num(c.w);
  }
  template <bool LOWER>
  __device__ __forceinline__ void half(cplx<float> (&h)[6]) const {
    if constexpr (LOWER) {
      h[0] = num(a.z); h[1] = num(a.w); h[2] = num(b.x); h[3] = num(b.y); h[4] = num(b.z); h[5] = num(b.w);
    } else {
      h[0] = num(a.x); h[1] = num(a.y); h[2] = num(a.z); h[3] = num(a.w); h[4] = num(b.x); h[5] = num(b.y);
    }
  }
};
template <>
struct NbRaw<WD_F16> : NbRaw16<WD_F16> {};
template <>
struct NbRaw<WD_BF16> : NbRaw16<WD_BF16> {};

// h = the half spinor that hop D projects from the loaded neighbour.
template <int P, bool DAG, int D>
__device__ __forceinline__ void mrhs_split_project(const NbRaw<P> &raw, RealOf<P> f, cplx<RealOf<P>> (&h)[6]) {
  constexpr int S = ((D < 4) != DAG) ? 1 : -1;
  if constexpr ((D & 3) == 3) {
    raw.template half<(S < 0)>(h);
#pragma unroll
    for (int c = 0; c < 6; ++c) h[c] = f * h[c];
  } else {
    cplx<RealOf<P>> psi[12];
    raw.whole(psi);
    project<D & 3, S>(psi, h);
  }
}

// The wave's hop of one right-hand side into LDS (q: the lane's first
// element): the products of split_hop.
template <int P>
__device__ __forceinline__ void mrhs_split_mul(const cplx<RealOf<P>> (&u)[6], const cplx<RealOf<P>> (&r2)[3],
                                               const cplx<RealOf<P>> (&h)[6], cplx<RealOf<P>> *q) {
  using T = RealOf<P>;
  if constexpr (P == WD_F64) {
    // One number at a time: 128 registers then hold the links, this half spinor and
    // the next neighbour.  Three at a time spilled packets of the neighbour as they
    // came (24^3x48 with 12: 554 us, 478 now).
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        cplx<T> y = (a < 2 ? u[3 * (a & 1)] : r2[0]) * h[3 * s];
        cfma(y, a < 2 ? u[3 * (a & 1) + 1] : r2[1], h[3 * s + 1]);
        cfma(y, a < 2 ? u[3 * (a & 1) + 2] : r2[2], h[3 * s + 2]);
        q[(3 * s + a) * SPLIT_SITES] = y;
      }
    return;
  }
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const cplx<T> v[3] = {h[3 * s], h[3 * s + 1], h[3 * s + 2]};
    cplx<T> y[3];
    su3_mul(u, r2, v, y);
#pragma unroll
    for (int a = 0; a < 3; ++a) q[(3 * s + a) * SPLIT_SITES] = y[a];
  }
}

// The sums and the epilogue of wave slot W for one right-hand side (out at
// byte offset off, epilogue operands x, y); returns the lane's |components|^2
// when NORM.
template <int P, bool DAG, int EPI, bool NORM, int W, int... J>
__device__ __forceinline__ double mrhs_split_finish(const KDslash &k, size_t off, int i, int lane,
                                                    SplitLds<P> &lds, cplx<RealOf<P>> (&x)[SplitOut<P>::CW],
                                                    cplx<RealOf<P>> (&y)[SplitOut<P>::CW],
                                                    std::integer_sequence<int, J...>) {
  using T = RealOf<P>;
  constexpr int CW = SplitOut<P>::CW;
  cplx<T> o[CW];
  if (i < k.g.vh) {
    const T a = (T)k.a;
    // one component's LDS reads at a time: the links and the next neighbour
    // stay in registers meanwhile
    ((o[J] = split_sum<P, DAG, W * CW + J>(lds, lane), __builtin_amdgcn_sched_barrier(0)), ...);
    if constexpr (P == WD_F64) {
      if constexpr (EPI >= 1) split_load<P>(k.X + off, i, W, x);
      if constexpr (EPI == 2) split_load<P>(k.Y + off, i, W, y);
    }
#pragma unroll
    for (int j = 0; j < CW; ++j) {
      o[j] = a * o[j];
      if constexpr (EPI >= 1) o[j] = o[j] + x[j];
      if constexpr (EPI == 2) o[j] = o[j] - y[j];
    }
  } else {
#pragma unroll
    for (int j = 0; j < CW; ++j) o[j] = {(T)0, (T)0};
  }
  float m = 0.f;
  if constexpr (P == WD_F16) m = split_max<W>(o, lds, lane);  // (the second barrier)
  split_store<P, W, true, NORM>(k.out + off, i, o, m);
  double n = 0.0;
  if constexpr (NORM) {
    if (i < k.g.vh) {
#pragma unroll
      for (int j = 0; j < CW; ++j) n += (double)o[j].re * o[j].re + (double)o[j].im * o[j].im;
    }
  }
  return n;
}

// Multi-RHS hop with one wave per direction (see wd_hop.h): a block of eight
// waves keeps the links of 64 sites, one direction per wave, in registers and
// walks the rpl right-hand sides of its chunk.  Per right-hand side each wave
// transports one neighbour into LDS (the next neighbour is already on its
// way), and after a barrier NW of the waves, another set for each right-hand
// side, add up and store.  Two LDS buffers, so one barrier a right-hand side
// (FP64: one buffer and two barriers, two blocks a CU instead of one; FP16 has
// the second barrier for the scale, and so one buffer).  80 registers a lane and
// 24 waves a CU (FP64 128 and 16); all eight links in one lane took 232
// registers, 8 waves a CU.  FP16 24^3x48 with 12: 187 us; 218 with a site's sums
// in one wave, another one for each right-hand side.  Bound by VALU issue in BF16
// (about 1400 instructions per 64 sites and right-hand side, 158 us of the 161
// at 24^3x48 with 12) and by fetches in FP64 (tuned order there: 1.59 times the
// algorithmic bytes, 5.9 TB/s).
template <int P, bool DAG, int EPI, bool NORM>
__global__ __launch_bounds__(SPLIT_BS, P == WD_F64 ? 4 : 6) void k_dslash_mrhs_split(KMrhs m) {
  using T = RealOf<P>;
  constexpr int NB = (P == WD_F64 || P == WD_F16) ? 1 : 2, NW = SplitOut<P>::NW, CW = SplitOut<P>::CW;
  __shared__ SplitLds<P> lds[NB];
  __shared__ double sred[NORM ? MR_CHUNK : 1][NW];
  const KDslash &k = m.k;
  int tile, chunk;
  if (m.nx3 > 0) {
    mrhs_box(m, (int)blockIdx.x, tile, chunk);
  } else if (k.groups == SPLIT_RANGES) {
    // a contiguous range of tiles per XCD, a tile's chunks side by side
    const int q = (int)blockIdx.x >> 3;
    chunk = q % m.nchunks;
    tile = ((int)blockIdx.x & 7) * k.tiles_per_slice + q / m.nchunks;
    if (tile >= m.ntiles) return;
  } else {
    tile = tile_of(k);
    chunk = (int)blockIdx.y;
  }
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = (int)threadIdx.x & 63;
  const int i = tile * SPLIT_SITES + lane;
  const bool site = i < k.g.vh;
  const int r0 = chunk * m.rpl, r1 = min(m.nrhs, r0 + m.rpl);
  // the chunk's systems that are not masked, one bit each: a finished system
  // costs neither loads nor a barrier, a finished chunk not even its links
  // (12 systems of 16^4 in BF16, none live: 13 us a launch -> 2)
  bool mine = r0 + lane < r1;
  if (k.skip && mine) mine = k.skip[(size_t)(r0 + lane) * m.skip_stride] == 0;
  const unsigned chosen = (unsigned)__ballot(mine);  // (MR_CHUNK bits at most)
  if (!chosen) {
    if constexpr (NORM)
      for (int r = r0 + (int)threadIdx.x; r < r1; r += SPLIT_BS) k.partials[(size_t)r * m.ntiles + tile] = 0.0;
    return;
  }
  int nb = 0;
  bool edge = false;
  cplx<T> u[6], r2[3];
  if (site) {
    switch (w) {
      case 0: nb = neighbour_of<0, true>(k.g, i, k.parity, edge); break;
      case 1: nb = neighbour_of<1, true>(k.g, i, k.parity, edge); break;
      case 2: nb = neighbour_of<2, true>(k.g, i, k.parity, edge); break;
      case 3: nb = neighbour_of<3, true>(k.g, i, k.parity, edge); break;
      case 4: nb = neighbour_of<0, false>(k.g, i, k.parity, edge); break;
      case 5: nb = neighbour_of<1, false>(k.g, i, k.parity, edge); break;
      case 6: nb = neighbour_of<2, false>(k.g, i, k.parity, edge); break;
      default: nb = neighbour_of<3, false>(k.g, i, k.parity, edge); break;
    }
  }
  Link<T>::load(k.links, w, i, u);  // (padding slots hold zero links)
  rebuild_row2(u, r2);
  const T f = (T)2 * (edge ? (T)k.g.tbc : (T)1);
  NbRaw<P> nx;  // (padding lanes read site 0)
  const bool time = (w & 3) == 3, lower = time && (w == 3) == DAG;
  unsigned todo = chosen;
  nx.load(k.in + (size_t)(r0 + __builtin_ctz(todo)) * m.rhs_stride, nb, time, lower);
#pragma unroll 1
  for (int n = 0; todo; ++n) {  // n-th live system of the chunk: r
    const int r = r0 + __builtin_ctz(todo);
    todo &= todo - 1;
    // opaque copies: the addresses of the six sums are formed where they are
    // used, not kept in registers across the loop
    int li = lane, ii = i;
    asm volatile("" : "+v"(li), "+v"(ii));
    const int slot = w * 6 * SPLIT_SITES + li;
    SplitLds<P> &L = lds[NB == 2 ? n & 1 : 0];
    // the next right-hand side's neighbour is loaded, by one load for all
    // directions, before this one's products
    cplx<T> *q = L.g + slot;
    cplx<T> h[6];
#define WD_HOP(D) mrhs_split_project<P, DAG, D>(nx, f, h)
    switch (w) {
      case 0: WD_HOP(0); break;
      case 1: WD_HOP(1); break;
      case 2: WD_HOP(2); break;
      case 3: WD_HOP(3); break;
      case 4: WD_HOP(4); break;
      case 5: WD_HOP(5); break;
      case 6: WD_HOP(6); break;
      default: WD_HOP(7); break;
    }
#undef WD_HOP
    if (todo) nx.load(k.in + (size_t)(r0 + __builtin_ctz(todo)) * m.rhs_stride, nb, time, lower);
    mrhs_split_mul<P>(u, r2, h, q);
    const int ws = NB == 2 ? (w + NW * n) & 7 : w;  // the waves take turns
    const size_t off = (size_t)r * m.rhs_stride;
    cplx<T> x[CW], y[CW];  // loaded before the barrier (FP64, short of registers: after the sums)
    if (P != WD_F64 && ws < NW && ii < k.g.vh) {
      if constexpr (EPI >= 1) split_load<P>(k.X + off, ii, ws, x);
      if constexpr (EPI == 2) split_load<P>(k.Y + off, ii, ws, y);
    }
    __syncthreads();
    double nrm = 0.0;
    constexpr auto J = std::make_integer_sequence<int, CW>{};
    if (ws == 0) nrm = mrhs_split_finish<P, DAG, EPI, NORM, 0>(k, off, ii, li, L, x, y, J);
    if constexpr (NW > 1) {
      if (ws == 1) nrm = mrhs_split_finish<P, DAG, EPI, NORM, 1>(k, off, ii, li, L, x, y, J);
      if (ws == 2) nrm = mrhs_split_finish<P, DAG, EPI, NORM, 2>(k, off, ii, li, L, x, y, J);
    }
    if constexpr (NW > 3) {
      if (ws == 3) nrm = mrhs_split_finish<P, DAG, EPI, NORM, 3>(k, off, ii, li, L, x, y, J);
      if (ws == 4) nrm = mrhs_split_finish<P, DAG, EPI, NORM, 4>(k, off, ii, li, L, x, y, J);
      if (ws == 5) nrm = mrhs_split_finish<P, DAG, EPI, NORM, 5>(k, off, ii, li, L, x, y, J);
    }
    if (ws >= NW) split_max_rest<P>();
    if constexpr (NORM) {
      if (ws < NW) {
        nrm = wave_sum(nrm);
        if (lane == 0) sred[r - r0][ws] = nrm;
      }
    }
    // before the next right-hand side overwrites the buffer (FP16: the barrier of its scale)
    if constexpr (P == WD_F64) __syncthreads();
  }
  if constexpr (NORM) {
    __syncthreads();
    for (int q = (int)threadIdx.x; q < r1 - r0; q += SPLIT_BS) {
      double s = 0.0;
      if (chosen >> q & 1) {
#pragma unroll
        for (int v = 0; v < NW; ++v) s += sred[q][v];
      }
      k.partials[(size_t)(r0 + q) * m.ntiles + tile] = s;
    }
  }
}

// ------------------------------------------------------------ launchers
static KDslash make_k_mrhs(const wd_gauge *g, wd_prec prec, int parity) {
  KDslash k{};
  k.nt_store = 1;
  k.g = g->geom;
  const bool dbl = (prec == WD_F64);
  const char *base = (const char *)(dbl ? g->links64 : g->links32);
  k.links = base + (size_t)parity * link_parity_bytes(g->geom, dbl);
  k.parity = parity;
  return k;
}

// `lds` bytes of dynamic LDS (unused by the kernel) cap the resident blocks
// per CU (160 KiB of LDS per CU): fewer sites in flight per XCD means a
// smaller set of neighbour spinors the L2 must hold for reuse.

// FP64 multi-RHS hop in box order, one right-hand side per block: block b
// is (tile, RHS) by mrhs_box with RHS chunks of one, so the nrhs blocks of a
// tile follow each other on one XCD; each runs the single-RHS hop on its RHS
// (same arithmetic, same bits), its links coming from that XCD's L2 after
// the first of them.  Norm partials per (RHS, tile) as above.
template <int P, bool DAG, int EPI, bool NORM>
__global__ __launch_bounds__(256) void k_dslash_mrhs_l2(KMrhs m) {
  int tile, r;
  mrhs_box(m, (int)blockIdx.x, tile, r);
  const bool live = !(m.k.skip && m.k.skip[(size_t)r * m.skip_stride]);
  double nrm = 0.0;
  if (live) {
    KDslash k = m.k;
    const size_t off = (size_t)r * m.rhs_stride;
    k.in = m.k.in + off;
    k.out = m.k.out + off;
    if (k.X) k.X += off;
    if (k.Y) k.Y += off;
    nrm = dslash_site<P, DAG, EPI, NORM, false>(k, tile * (int)blockDim.x + (int)threadIdx.x);
  }
  if constexpr (NORM) {
    double v[1] = {nrm};
    block_sum_n<1>(v);
    if (threadIdx.x == 0 && live) m.k.partials[(size_t)r * m.ntiles + tile] = v[0];
  }
}

template <int P, bool DAG, int EPI, bool NORM>
static void launch_mrhs_t(const KMrhs &m, dim3 grid, dim3 block, hipStream_t st) {
  if (m.k.split) {
    hipLaunchKernelGGL((k_dslash_mrhs_split<P, DAG, EPI, NORM>), grid, block, 0, st, m);
    return;
  }
  if constexpr (P == WD_F64) {
    if (m.nx3 > 0) hipLaunchKernelGGL((k_dslash_mrhs_l2<P, DAG, EPI, NORM>), grid, block, 0, st, m);
    else hipLaunchKernelGGL((k_dslash_mrhs<P, DAG, EPI, NORM>), grid, block, 0, st, m);
  } else {
    hipLaunchKernelGGL((k_dslash_mrhs_reg<P, DAG, EPI, NORM>), grid, block, 0, st, m);
  }
}

template <int P>
static void launch_mrhs_p(const KMrhs &m, bool dag, int epi, bool norm, dim3 grid, dim3 block, hipStream_t st) {
#define WD_M(D, E, N) if (dag == D && epi == E && norm == N) launch_mrhs_t<P, D, E, N>(m, grid, block, st);
  WD_M(false, 0, false) WD_M(false, 1, false) WD_M(false, 2, false)
  WD_M(false, 0, true) WD_M(false, 1, true) WD_M(false, 2, true)
  WD_M(true, 0, false) WD_M(true, 1, false) WD_M(true, 2, false)
  WD_M(true, 0, true) WD_M(true, 1, true) WD_M(true, 2, true)
#undef WD_M
}

// Box order of the FP32-arithmetic multi-RHS hop (groups = -(100 + nx3)):
// whole tiles per time slice, and the slices and each slice's tiles split
// evenly over the 8 boxes.
bool mrhs_box_ok(const Geom &G, int bs, int groups) {
  if (groups > -100) return false;
  const int nx3 = -groups - 100;
  if (nx3 != 1 && nx3 != 2 && nx3 != 4 && nx3 != 8) return false;
  const long slice = (long)G.vh / G.L[3];
  if (G.vpad != G.vh || slice % bs != 0) return false;
  return (slice / bs) % nx3 == 0 && G.L[3] % (8 / nx3) == 0;
}

// Orders of the one-wave-per-direction form (block SPLIT_BS, 64-site tiles).
bool mrhs_split_order_ok(const Geom &G, int groups) {
  if (groups == SPLIT_RANGES) return true;
  return groups <= -100 ? mrhs_box_ok(G, SPLIT_SITES, groups) : dslash_variant_ok(G, SPLIT_SITES, groups, 1);
}

// Block size of the multi-RHS hop: FP64 keeps 16 sites x RHS lanes, the
// others one lane per site (tunable, 64..256).
static int mrhs_block_of(const wd_gauge *g, wd_prec prec, int &groups) {
  const int pi = (int)prec;
  int bs = g->mrhs_block[pi];
  groups = g->mrhs_groups[pi];
  if (bs == SPLIT_BS) {
    if (!mrhs_split_order_ok(g->geom, groups)) groups = SPLIT_RANGES;
    return bs;
  }
  const bool box = mrhs_box_ok(g->geom, bs, groups);
  if (prec == WD_F64) {
    // FP64: 16-site x RHS tiles, or one RHS per block in box order
    if (box && (bs == 64 || bs == 128 || bs == 256)) return bs;
    bs = 16;
    if (groups <= -100 || !dslash_variant_ok(g->geom, bs, groups, 1)) groups = 0;
    return bs;
  }
  if (bs != 64 && bs != 128 && bs != 256) bs = 128;
  if (!box && !dslash_variant_ok(g->geom, bs, groups, 1)) groups = 0;
  return bs;
}

// The variant of a new handle: one wave per direction, up to 12 right-hand
// sides per block (fewer on small lattices, see mrhs_split_rpl).  us per
// launch against the defaults of the other forms (128 sites, 4 right-hand
// sides per lane; FP64 16-site tiles), 12 right-hand sides: BF16 8^4 6.7 / 16,
// 20^3x40 85 / 108, 24^3x48 161 / 208; FP32 20^3x40 120 / 153, 24^3x48 246 /
// 309; FP64 16^4 42 / 67, 24^3x48 480 / 700, 32^3x64 1460 / 2250; FP16 8^4 4.7 /
// 14, 16^4 23.7 / 26.2 (with 24 43.8 / 45.1), 24^3x48 187 / 218, 32^4 296 / 334
// (with 3 93 / 92).  Alone on 24^3x48, one lane per site in box order with all 12
// (tuned) is faster in BF16, 139 us, but slower in a solve of 12, where systems
// finish and epilogues add operands: 99.8 ms against 89.5; FP32 235 / 235 us and
// 158 / 155 ms.
// Order as for the single-RHS hop: contiguous ranges per XCD (BF16 24^3x48 161
// against 166 with regions); from 2^18 sites eight regions of each slice where
// they divide it (32^4: FP64 721 / 809, FP32 366 / 397, FP16 306 / 310, BF16 250 /
// 254), else in FP64 and FP32 four (FP64 24^3x48 480 / 507).
constexpr int MRHS_SPLIT_RPL = 12;
void mrhs_default_variant(wd_gauge *g, int p) {
  const Geom &G = g->geom;
  g->mrhs_rpl[p] = MRHS_SPLIT_RPL;
  g->mrhs_block[p] = SPLIT_BS;
  g->mrhs_groups[p] = SPLIT_RANGES;
  if (G.vh >= (1 << 18)) {
    if (dslash_variant_ok(G, SPLIT_SITES, 8)) g->mrhs_groups[p] = 8;
    else if (p <= WD_F32 && dslash_variant_ok(G, SPLIT_SITES, 4)) g->mrhs_groups[p] = 4;
  }
  g->mrhs_groups0[p] = g->mrhs_groups[p];
}

// Right-hand sides per block.  The default variant (its block, order and rpl,
// whether set or never touched) adds chunks until the blocks are two a CU, for fewer would leave the chain of right-hand sides as
// the run time: 8^4 (32 tiles), 12 right-hand sides BF16: 3 per block 6.7 us,
// 12 per block 15.2; 16^4 (512 tiles) FP64: 12 per block 42, 4 per block 55.
static int mrhs_split_rpl(const wd_gauge *g, int prec, int nrhs, int ntiles) {
  const int most = g->mrhs_rpl[prec];
  if (most != MRHS_SPLIT_RPL || g->mrhs_groups[prec] != g->mrhs_groups0[prec]) return most;
  const int chunks = std::max((nrhs + most - 1) / most, std::min(nrhs, (512 + ntiles - 1) / ntiles));
  return (nrhs + chunks - 1) / chunks;
}

wd_status launch_dslash_mrhs_ex(const wd_gauge *g, wd_prec prec, const MrhsArgs &a, hipStream_t st) {
  if (a.nrhs < 1) return set_error(WD_ERR_ARG, "dslash_mrhs: nrhs = %d", a.nrhs);
  if (a.Y && !a.X) return set_error(WD_ERR_ARG, "dslash_mrhs epilogue: Y given without X");
  KMrhs m{};
  m.k = make_k_mrhs(g, prec, a.parity);
  m.k.in = (const char *)a.in;
  m.k.out = (char *)a.out;
  m.k.X = (const char *)a.X;
  m.k.Y = (const char *)a.Y;
  m.k.a = a.a;
  m.k.skip = a.skip;
  m.k.partials = a.red.partials;
  m.nrhs = a.nrhs;
  m.rhs_stride = a.rhs_stride ? a.rhs_stride : half_bytes(g->geom, prec);
  m.skip_stride = a.skip_stride;
  const bool norm = a.norm_out != nullptr;
  if (norm && !m.k.partials) return set_error(WD_ERR_ARG, "dslash_mrhs norm: no reduction buffer");
  const int epi = a.Y ? 2 : (a.X ? 1 : 0);
  int groups;
  int bs = mrhs_block_of(g, prec, groups);
  m.k.split = bs == SPLIT_BS;
  if (m.k.split) bs = SPLIT_SITES;
  m.k.groups = groups;
  m.k.tiles_per_slice = groups ? (int)((long)g->geom.vh / g->geom.L[3] / bs) : 0;
  dim3 grid, block;
  if (m.k.split) {
    m.ntiles = g->geom.vpad / SPLIT_SITES;
    m.rpl = std::max(1, std::min(MR_CHUNK, mrhs_split_rpl(g, (int)prec, a.nrhs, m.ntiles)));
    m.nchunks = (a.nrhs + m.rpl - 1) / m.rpl;
    m.rpl = (a.nrhs + m.nchunks - 1) / m.nchunks;  // even chunks
    block = dim3(SPLIT_BS);
    if (groups == SPLIT_RANGES) {
      m.k.tiles_per_slice = (m.ntiles + 7) / 8;  // tiles per range
      grid = dim3((unsigned)(8 * m.k.tiles_per_slice * m.nchunks));
    } else if (groups <= -100) {
      m.nx3 = -groups - 100;
      grid = dim3((unsigned)(m.ntiles * m.nchunks));
    } else {
      grid = dim3((unsigned)m.ntiles, (unsigned)m.nchunks);
    }
  } else if (prec == WD_F64 && groups <= -100) {
    m.rpl = 1;
    m.nchunks = a.nrhs;
    m.ntiles = (int)((g->geom.vpad + bs - 1) / bs);
    m.nx3 = -groups - 100;
    grid = dim3((unsigned)(m.ntiles * m.nchunks), 1);
    block = dim3((unsigned)bs);
  } else if (prec == WD_F64) {
    const int per_block = std::min(16, (a.nrhs + 3) / 4 * 4);
    grid = dim3((unsigned)mrhs_grid_blocks(g), (unsigned)((a.nrhs + 15) / 16));
    block = dim3((unsigned)(16 * per_block));
  } else {
    m.rpl = std::max(1, std::min(MR_CHUNK, g->mrhs_rpl[(int)prec]));
    m.nchunks = (a.nrhs + m.rpl - 1) / m.rpl;
    m.ntiles = (int)((g->geom.vpad + bs - 1) / bs);
    if (groups <= -100) {
      m.nx3 = -groups - 100;
      grid = dim3((unsigned)(m.ntiles * m.nchunks), 1);
    } else {
      grid = dim3((unsigned)m.ntiles, (unsigned)m.nchunks);
    }
    block = dim3((unsigned)bs);
  }
  switch (prec) {
    case WD_F64: launch_mrhs_p<WD_F64>(m, a.dagger, epi, norm, grid, block, st); break;
    case WD_F32: launch_mrhs_p<WD_F32>(m, a.dagger, epi, norm, grid, block, st); break;
    case WD_F16: launch_mrhs_p<WD_F16>(m, a.dagger, epi, norm, grid, block, st); break;
    case WD_BF16: launch_mrhs_p<WD_BF16>(m, a.dagger, epi, norm, grid, block, st); break;
    default: return set_error(WD_ERR_PREC, "dslash_mrhs: unknown precision %d", (int)prec);
  }
  WD_TRY(hip_check(hipGetLastError(), "dslash_mrhs launch"));
  const unsigned nparts = m.ntiles > 0 ? (unsigned)m.ntiles : grid.x;
  if (norm && !leave_partials(a.red, nparts))
    return launch_finish_sums(m.k.partials, nparts, a.nrhs, a.norm_out,
                              a.norm_stride, a.norm_accumulate, m.k.skip, m.skip_stride, st);
  return WD_OK;
}

wd_status launch_dslash_mrhs(const wd_gauge *g, wd_prec prec, const void *in, void *out, double a, int parity,
                             int dagger, int nrhs, hipStream_t st) {
  MrhsArgs m;
  m.in = in; m.out = out; m.a = a; m.parity = parity; m.dagger = dagger; m.nrhs = nrhs;
  return launch_dslash_mrhs_ex(g, prec, m, st);
}

}  // namespace wd
