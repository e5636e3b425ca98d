// Level-1 kernels on spin-colour fields: caxpy (Sec. 4), inner products and
// norms with FP64 accumulation in a fixed order, precision conversion, and
// the fused CG recurrences whose scalars never leave the device.
//
// Every kernel works on `nsys` independent systems at once (grid.y): system
// y's vectors start at y * sys_stride bytes and it owns its own scalar block
// and reduction slots, so a batch of right-hand sides shares each launch.
// A vector is `nhalf` half fields of vh valid sites (half_stride bytes apart).
#include <algorithm>

#include "wd_blas.h"
#include "wd_device.h"

namespace wd {

template <int P>
using RealOf = typename Spinor<P>::real;

constexpr int BLAS_BS = 256;

struct VecGeom {
  int vh;
  int vpad;
  int nhalf;
  size_t half_stride;  // bytes between half fields of one vector (per precision)
};

struct KBlas {
  VecGeom v;
  unsigned nblk;  // blocks per system (grid.x)
  // operands (system 0); per-system offsets below
  const char *x;
  const char *y;
  char *out;
  char *out2;
  size_t sx, sy, so, so2;  // per-system byte strides of x, y, out, out2
  size_t hx, hy, ho, ho2;  // per-half byte strides
  double c_re, c_im;
  CgScalars *sc;
  int j;  // ping-pong slot of the CG iteration
  double *partials;
  double *result;  // reductions: per-system result (N doubles each)
  // CG recurrences: the hop's norm partials, nparts per system (0: the sum is
  // already in the scalars), and the |s|^2 partials of the update, nss per system
  const double *parts;
  unsigned nparts;
  const double *ss_parts;
  unsigned nss;
  size_t npk;  // packets of a vector (all halves)
};

__device__ __forceinline__ bool site_of(const VecGeom &v, long f, int &h, int &i) {
  h = (int)(f / v.vh);
  i = (int)(f - (long)h * v.vh);
  return h < v.nhalf;
}

// ------------------------------------------------------------ reductions
// A spinor read with streaming (non-temporal) loads, for operands read once
// per kernel (caxpy and the reductions |x|^2, <x, y>): full fields of the
// solvers are larger than the caches, so keeping them buys nothing and
// streaming them frees the caches for the hop's gathers.  FP16 and BF16 as
// Spinor<P>::load.
template <int P>
__device__ __forceinline__ void load_stream(const char *base, int i, cplx<RealOf<P>> (&s)[12]) {
  if constexpr (P == WD_F64) {
    const v2d *p = (const v2d *)base + chunk_base<Spinor<WD_F64>::CHUNK>((size_t)i);
#pragma unroll
    for (int c = 0; c < 12; ++c) {
      const v2d v = ld_stream(p + 64 * c);
      s[c] = {v.x, v.y};
    }
  } else if constexpr (P == WD_F32) {
    const v4f *p = (const v4f *)base + chunk_base<Spinor<WD_F32>::CHUNK>((size_t)i);
#pragma unroll
    for (int q = 0; q < 6; ++q) {
      const v4f v = ld_stream(p + 64 * q);
      s[2 * q] = {v.x, v.y};
      s[2 * q + 1] = {v.z, v.w};
    }
  } else {
    Spinor<P>::load(base, (size_t)i, s);
  }
}

template <int P>
__global__ __launch_bounds__(BLAS_BS) void k_norm2(KBlas k) {
  using T = RealOf<P>;
  const int sys = blockIdx.y;
  const char *x = k.x + sys * k.sx;
  const long n = (long)k.v.vh * k.v.nhalf;
  double acc = 0.0;
  for (long f = (long)blockIdx.x * BLAS_BS + threadIdx.x; f < n; f += (long)k.nblk * BLAS_BS) {
    int h, i;
    site_of(k.v, f, h, i);
    cplx<T> a[12];
    load_stream<P>(x + h * k.hx, i, a);
#pragma unroll
    for (int c = 0; c < 12; ++c) acc += (double)a[c].re * a[c].re + (double)a[c].im * a[c].im;
  }
  double v[1] = {acc};
  block_sum_store<1>(v, k.partials + (size_t)sys * k.nblk, k.nblk, blockIdx.x);
}

template <int P>
__global__ __launch_bounds__(BLAS_BS) void k_cdot(KBlas k) {
  using T = RealOf<P>;
  const int sys = blockIdx.y;
  const char *x = k.x + sys * k.sx;
  const char *y = k.y + sys * k.sy;
  const long n = (long)k.v.vh * k.v.nhalf;
  double re = 0.0, im = 0.0;
  for (long f = (long)blockIdx.x * BLAS_BS + threadIdx.x; f < n; f += (long)k.nblk * BLAS_BS) {
    int h, i;
    site_of(k.v, f, h, i);
    cplx<T> a[12], b[12];
    load_stream<P>(x + h * k.hx, i, a);
    load_stream<P>(y + h * k.hy, i, b);
#pragma unroll
    for (int c = 0; c < 12; ++c) {
      re += (double)a[c].re * b[c].re + (double)a[c].im * b[c].im;
      im += (double)a[c].re * b[c].im - (double)a[c].im * b[c].re;
    }
  }
  double v[2] = {re, im};
  block_sum_store<2>(v, k.partials + (size_t)sys * 2 * k.nblk, k.nblk, blockIdx.x);
}

// ------------------------------------------------------------ finishing sums
constexpr int FIN_BS = 1024;

__global__ __launch_bounds__(FIN_BS) void k_finish_sums(const double *partials, unsigned nblocks, double *out,
                                                        int ostride, int accumulate, const int *skip, int sstride) {
  const int j = blockIdx.x;
  double v[1] = {0.0};
  for (unsigned b = threadIdx.x; b < nblocks; b += FIN_BS) v[0] += partials[(size_t)j * nblocks + b];
  block_sum_n<1>(v);
  if (threadIdx.x == 0 && !(skip && skip[(size_t)j * sstride])) {
    double *d = out + (size_t)j * ostride;
    *d = accumulate ? (*d + v[0]) : v[0];
  }
}

// ------------------------------------------------------------ elementwise
// out = c * x + y  (out may alias y)
template <int P>
__global__ __launch_bounds__(BLAS_BS) void k_caxpy(KBlas k) {
  using T = RealOf<P>;
  const int sys = blockIdx.y;
  const long n = (long)k.v.vh * k.v.nhalf;
  const cplx<T> c = {(T)k.c_re, (T)k.c_im};
  for (long f = (long)blockIdx.x * BLAS_BS + threadIdx.x; f < n; f += (long)k.nblk * BLAS_BS) {
    int h, i;
    site_of(k.v, f, h, i);
    cplx<T> a[12], b[12];
    // both operands are read once: streaming loads
    load_stream<P>(k.x + sys * k.sx + h * k.hx, i, a);
    load_stream<P>(k.y + sys * k.sy + h * k.hy, i, b);
#pragma unroll
    for (int q = 0; q < 12; ++q) cfma(b[q], c, a[q]);
    Spinor<P>::store(k.out + sys * k.so + h * k.ho, i, b);
  }
}

// out(PO) = s * x(PI); s = c_re, or c_re / sqrt(sc[sys].rnorm2) when sc != 0.
// Also zero-fills padding slots so every output slot is defined.
template <int PI, int PO>
__global__ __launch_bounds__(BLAS_BS) void k_convert(KBlas k) {
  using TI = RealOf<PI>;
  using TO = RealOf<PO>;
  const int sys = blockIdx.y;
  double s = k.c_re;
  if (k.sc) s = k.c_re / sqrt(k.sc[sys].rnorm2);
  const long n = (long)k.v.vpad * k.v.nhalf;
  for (long f = (long)blockIdx.x * BLAS_BS + threadIdx.x; f < n; f += (long)k.nblk * BLAS_BS) {
    const int h = (int)(f / k.v.vpad);
    const int i = (int)(f - (long)h * k.v.vpad);
    cplx<TO> b[12];
    if (i < k.v.vh) {
      cplx<TI> a[12];
      Spinor<PI>::load(k.x + sys * k.sx + h * k.hx, i, a);
      if constexpr (PO == WD_F64) {
#pragma unroll
        for (int q = 0; q < 12; ++q) b[q] = {(TO)(s * (double)a[q].re), (TO)(s * (double)a[q].im)};
      } else {
        const TO sf = (TO)s;
#pragma unroll
        for (int q = 0; q < 12; ++q) b[q] = {sf * (TO)a[q].re, sf * (TO)a[q].im};
      }
    } else {
#pragma unroll
      for (int q = 0; q < 12; ++q) b[q] = {(TO)0, (TO)0};
    }
    Spinor<PO>::store(k.out + sys * k.so + h * k.ho, i, b);
  }
}

// out(F64) += sqrt(sc[sys].rnorm2) * c_re * e(PE)   (defect-correction update)
template <int PE>
__global__ __launch_bounds__(BLAS_BS) void k_accum(KBlas k) {
  using TE = RealOf<PE>;
  const int sys = blockIdx.y;
  const double s = k.c_re * sqrt(k.sc[sys].rnorm2);
  const long n = (long)k.v.vh * k.v.nhalf;
  for (long f = (long)blockIdx.x * BLAS_BS + threadIdx.x; f < n; f += (long)k.nblk * BLAS_BS) {
    int h, i;
    site_of(k.v, f, h, i);
    cplx<TE> e[12];
    cplx<double> x[12];
    Spinor<PE>::load(k.x + sys * k.sx + h * k.hx, i, e);
    char *o = k.out + sys * k.so + h * k.ho;
    Spinor<WD_F64>::load(o, i, x);
#pragma unroll
    for (int q = 0; q < 12; ++q) {
      x[q].re = fma(s, (double)e[q].re, x[q].re);
      x[q].im = fma(s, (double)e[q].im, x[q].im);
    }
    Spinor<WD_F64>::store(o, i, x);
  }
}

// ------------------------------------------------------------ CG recurrences
// The scalars of a step are sums of the norm partials that the hop before it
// left behind.  Where these are few, every block of the step adds them up
// itself (sum_partials); else a finishing launch came first.  The vectors are
// walked packet by packet (FP64, FP32, BF16), padding zeros included: small
// fields spread over more threads than sites, and every access is contiguous.

// Packets a thread has in flight at a time (the fields may alias for the
// compiler, so the loads are grouped by hand): 2, a grid apart, where that
// spreads a small field over more threads; 4 runs of the block side by side
// where the field has them for every thread (cg_side), so that what is in
// flight from each field is contiguous.  2 apart / 4 side by side, ms: FP64 CG
// on full fields 32^3x64 236.3 / 232.2, 24^3x48 78.3 / 77.7, FP64 CG 32^3x64
// 82.0 / 80.9; on 16^3x32, where 4 would leave threads idle, 6.03 / 6.08.
constexpr int CG_APART = 2, CG_SIDE = 4;

// |M p|^2 of system sys: done = breakdown on a value that is no norm.
__device__ __forceinline__ bool cg_alpha(const KBlas &k, int sys, double &alpha) {
  CgScalars *sc = k.sc + sys;
  double qq;
  if (k.nparts) {
    qq = sum_partials(k.parts + (size_t)sys * k.nparts, k.nparts);
    if (blockIdx.x == 0 && threadIdx.x == 0) sc->qq = qq;
  } else {
    qq = sc->qq;
  }
  const double rr = sc->rr[k.j];
  if (!(qq > 0.0) || !(qq < 1e300) || !(rr < 1e300)) return false;  // breakdown: the p update ends the CG
  alpha = rr / qq;
  return true;
}

// alpha = rr[j] / qq;  X += alpha P;  S -= alpha Q;  ss = |S|^2.
// x = X (precision PX), y = P, out = S, out2 = Q (precision PV) -- Q is read only.
// FP16 storage (a scale per site): one site per thread.
template <int PX, int PV, int U>
__global__ __launch_bounds__(BLAS_BS) void k_cg_update(KBlas k) {
  using TV = RealOf<PV>;
  using TX = RealOf<PX>;
  const int sys = blockIdx.y;
  if (blockIdx.x == 0 && threadIdx.x == 0) k.sc[sys].live = k.sc[sys].done == 0;
  if (k.sc[sys].done) return;
  double alpha;
  if (!cg_alpha(k, sys, alpha)) return;
  const TV a = (TV)alpha;
  const TX ax = (TX)alpha;
  char *X = (char *)k.x + sys * k.sx;
  const char *Pv = k.y + sys * k.sy;
  char *S = k.out + sys * k.so;
  const char *Q = k.out2 + sys * k.so2;
  double acc = 0.0;
  if constexpr (PV == WD_F16) {
    const long n = (long)k.v.vh * k.v.nhalf;
    for (long f = (long)blockIdx.x * BLAS_BS + threadIdx.x; f < n; f += (long)k.nblk * BLAS_BS) {
      int h, i;
      site_of(k.v, f, h, i);
      cplx<TV> p[12], s[12], q[12];
      cplx<TX> x[12];
      Spinor<PV>::load(Pv + h * k.hy, i, p);
      Spinor<PV>::load(Q + h * k.ho2, i, q);
      Spinor<PV>::load(S + h * k.ho, i, s);
      Spinor<PX>::load(X + h * k.hx, i, x);
#pragma unroll
      for (int c = 0; c < 12; ++c) {
        x[c].re = fma(ax, (TX)p[c].re, x[c].re);
        x[c].im = fma(ax, (TX)p[c].im, x[c].im);
        s[c].re = fma(-a, q[c].re, s[c].re);
        s[c].im = fma(-a, q[c].im, s[c].im);
      }
      Spinor<PX>::store(X + h * k.hx, i, x);
      Spinor<PV>::store(S + h * k.ho, i, s);
      Spinor<PV>::load(S + h * k.ho, i, s);  // norm of the stored (rounded) residual
#pragma unroll
      for (int c = 0; c < 12; ++c) acc += (double)s[c].re * s[c].re + (double)s[c].im * s[c].im;
    }
  } else {
    using KV = Packet<PV>;
    using KX = Packet<PX>;
    constexpr int R = KV::CW / KX::CW;  // X packets per V packet
    const size_t grid = (size_t)k.nblk * BLAS_BS, step = U == CG_SIDE ? BLAS_BS : grid;
    const size_t b = (size_t)blockIdx.x * BLAS_BS * (U == CG_SIDE ? U : 1);
    for (size_t f0 = b + threadIdx.x; f0 < k.npk; f0 += U * grid) {
      cplx<TV> p[U][KV::CW], s[U][KV::CW], q[U][KV::CW];
      cplx<TX> x[U][KV::CW];
      size_t fx[U];
#pragma unroll
      for (int e = 0; e < U; ++e) {
        const size_t f = min(f0 + e * step, k.npk - 1);  // (past the end: loaded, not stored)
        KV::load(Pv, f, p[e]);
        KV::load(Q, f, q[e]);
        KV::load(S, f, s[e]);
        // packet k of a site is X packets R k .. R k + R - 1 of the same site
        const size_t chunk = f / (64 * KV::NP), r = f - chunk * (64 * KV::NP);
        fx[e] = chunk * (64 * KX::NP) + (r >> 6) * (64 * R) + (r & 63);
#pragma unroll
        for (int w = 0; w < R; ++w) {
          cplx<TX> t[KX::CW];
          KX::load(X, fx[e] + 64 * w, t);
#pragma unroll
          for (int c = 0; c < KX::CW; ++c) x[e][w * KX::CW + c] = t[c];
        }
      }
#pragma unroll
      for (int e = 0; e < U; ++e) {
        const size_t f = f0 + e * step;
        if (f >= k.npk) break;
#pragma unroll
        for (int w = 0; w < R; ++w) {
          cplx<TX> t[KX::CW];
#pragma unroll
          for (int c = 0; c < KX::CW; ++c) {
            const int b = w * KX::CW + c;
            t[c] = {fma(ax, (TX)p[e][b].re, x[e][b].re), fma(ax, (TX)p[e][b].im, x[e][b].im)};
          }
          KX::store(X, fx[e] + 64 * w, t);
        }
#pragma unroll
        for (int c = 0; c < KV::CW; ++c) {
          s[e][c].re = fma(-a, q[e][c].re, s[e][c].re);
          s[e][c].im = fma(-a, q[e][c].im, s[e][c].im);
        }
        KV::store(S, f, s[e]);
#pragma unroll
        for (int c = 0; c < KV::CW; ++c)
          acc += (double)s[e][c].re * s[e][c].re + (double)s[e][c].im * s[e][c].im;
      }
    }
  }
  double v[1] = {acc};
  block_sum_store<1>(v, k.partials + (size_t)sys * k.nblk, k.nblk, blockIdx.x);
}

// What ends an iteration of system *sc: |s|^2, iteration count, convergence.
__device__ __forceinline__ void cg_end(CgScalars *sc, int j, double ss) {
  const double qq = sc->qq, rr = sc->rr[j];
  sc->ss = ss;
  if (!(qq > 0.0) || !(qq < 1e300) || !(rr < 1e300)) {
    sc->done = 2;  // breakdown / non-finite
  } else {
    sc->iters += 1;
    if (ss <= sc->stop2) sc->done = 1;
    else if (sc->iters >= sc->max_iters) sc->done = 3;
  }
}

// The end of the iteration right after the update (early_end): one block per
// system.  A system that converged is masked from here on.
__global__ __launch_bounds__(BLAS_BS) void k_cg_end(KBlas k) {
  CgScalars *sc = k.sc + blockIdx.x;
  if (!sc->live) return;
  const double ss = sum_partials(k.ss_parts + (size_t)blockIdx.x * k.nss, k.nss);
  if (threadIdx.x != 0) return;
  cg_end(sc, k.j, ss);
  sc->live = sc->done == 0;
}

// beta = rr[1-j] / rr[j];  P = R + beta P.   x = R, out = P.  Unless k_cg_end
// did (nss = 0), one more block per system (blockIdx.x = 0) ends the iteration:
// rr[1-j], ss = sum of the update's partials, iteration count and convergence
// flag.  A system that converged in this iteration then still gets its P here,
// which nothing reads.
template <int PV, int U>
__global__ __launch_bounds__(BLAS_BS) void k_cg_pupdate(KBlas k) {
  using TV = RealOf<PV>;
  const int sys = blockIdx.y;
  CgScalars *sc = k.sc + sys;
  // (not `done`, which block 0 changes: waves of one block that saw different
  // values would add up different lists below)
  if (!sc->live) return;
  double rrn;
  if (k.nparts) rrn = sum_partials(k.parts + (size_t)sys * k.nparts, k.nparts);
  else rrn = sc->rr[1 - k.j];
  const unsigned first = k.nss ? 1 : 0;
  if (blockIdx.x < first) {
    const double ss = sum_partials(k.ss_parts + (size_t)sys * k.nss, k.nss);
    if (threadIdx.x == 0) {
      if (k.nparts) sc->rr[1 - k.j] = rrn;
      cg_end(sc, k.j, ss);
    }
    return;
  }
  const TV b = (TV)(rrn / sc->rr[k.j]);
  const char *R = k.x + sys * k.sx;
  char *Pp = k.out + sys * k.so;
  if constexpr (PV == WD_F16) {
    const long n = (long)k.v.vh * k.v.nhalf;
    for (long f = (long)(blockIdx.x - first) * BLAS_BS + threadIdx.x; f < n; f += (long)k.nblk * BLAS_BS) {
      int h, i;
      site_of(k.v, f, h, i);
      cplx<TV> r[12], p[12];
      Spinor<PV>::load(R + h * k.hx, i, r);
      Spinor<PV>::load(Pp + h * k.ho, i, p);
#pragma unroll
      for (int c = 0; c < 12; ++c) {
        p[c].re = fma(b, p[c].re, r[c].re);
        p[c].im = fma(b, p[c].im, r[c].im);
      }
      Spinor<PV>::store(Pp + h * k.ho, i, p);
    }
  } else {
    using KV = Packet<PV>;
    const size_t grid = (size_t)k.nblk * BLAS_BS, step = U == CG_SIDE ? BLAS_BS : grid;
    const size_t b0 = (size_t)(blockIdx.x - first) * BLAS_BS * (U == CG_SIDE ? U : 1);
    for (size_t f0 = b0 + threadIdx.x; f0 < k.npk; f0 += U * grid) {
      cplx<TV> r[U][KV::CW], p[U][KV::CW];
#pragma unroll
      for (int e = 0; e < U; ++e) {
        const size_t f = min(f0 + e * step, k.npk - 1);  // (past the end: loaded, not stored)
        KV::load(R, f, r[e]);
        KV::load(Pp, f, p[e]);
      }
#pragma unroll
      for (int e = 0; e < U; ++e) {
        if (f0 + e * step >= k.npk) break;
#pragma unroll
        for (int c = 0; c < KV::CW; ++c) {
          p[e][c].re = fma(b, p[e][c].re, r[e][c].re);
          p[e][c].im = fma(b, p[e][c].im, r[e][c].im);
        }
        KV::store(Pp, f0 + e * step, p[e]);
      }
    }
  }
}

// ------------------------------------------------------------ launchers
static unsigned blocks_for(long n) {
  long b = (n + BLAS_BS - 1) / BLAS_BS;
  if (b > BLAS_MAX_BLOCKS) b = BLAS_MAX_BLOCKS;
  if (b < 1) b = 1;
  return (unsigned)b;
}

static VecGeom vgeom(const Geom &g, int nhalf, wd_prec p) {
  return VecGeom{g.vh, g.vpad, nhalf, half_bytes(g, p)};
}

#define WD_DISPATCH_P(prec, KERNEL, grid, k, st)                                               \
  switch (prec) {                                                                             \
    case WD_F64: hipLaunchKernelGGL(KERNEL<WD_F64>, grid, dim3(BLAS_BS), 0, st, k); break;    \
    case WD_F32: hipLaunchKernelGGL(KERNEL<WD_F32>, grid, dim3(BLAS_BS), 0, st, k); break;    \
    case WD_F16: hipLaunchKernelGGL(KERNEL<WD_F16>, grid, dim3(BLAS_BS), 0, st, k); break;    \
    case WD_BF16: hipLaunchKernelGGL(KERNEL<WD_BF16>, grid, dim3(BLAS_BS), 0, st, k); break;  \
    default: return set_error(WD_ERR_PREC, "blas: unknown precision %d", (int)prec);          \
  }

wd_status blas_norm2(const Geom &g, wd_prec prec, const VecRef &x, int nsys, RedBuf red, double *result,
                     hipStream_t st) {
  KBlas k{};
  k.v = vgeom(g, x.nhalf, prec);
  k.nblk = blocks_for((long)g.vh * x.nhalf);
  k.x = (const char *)x.p; k.sx = x.sys_stride; k.hx = k.v.half_stride;
  k.partials = red.partials; k.result = result;
  dim3 grid(k.nblk, (unsigned)nsys);
  WD_DISPATCH_P(prec, k_norm2, grid, k, st);
  WD_TRY(hip_check(hipGetLastError(), "norm2 launch"));
  return launch_finish_sums(red.partials, k.nblk, nsys, result, 1, 0, nullptr, 1, st);
}

wd_status blas_cdot(const Geom &g, wd_prec prec, const VecRef &x, const VecRef &y, int nsys, RedBuf red,
                    double *result, hipStream_t st) {
  KBlas k{};
  k.v = vgeom(g, x.nhalf, prec);
  k.nblk = blocks_for((long)g.vh * x.nhalf);
  k.x = (const char *)x.p; k.sx = x.sys_stride; k.hx = k.v.half_stride;
  k.y = (const char *)y.p; k.sy = y.sys_stride; k.hy = k.v.half_stride;
  k.partials = red.partials; k.result = result;
  dim3 grid(k.nblk, (unsigned)nsys);
  WD_DISPATCH_P(prec, k_cdot, grid, k, st);
  WD_TRY(hip_check(hipGetLastError(), "cdot launch"));
  return launch_finish_sums(red.partials, k.nblk, 2 * nsys, result, 1, 0, nullptr, 1, st);
}

wd_status blas_caxpy(const Geom &g, wd_prec prec, double cre, double cim, const VecRef &x, const VecRef &y,
                     int nsys, hipStream_t st) {
  KBlas k{};
  k.v = vgeom(g, x.nhalf, prec);
  k.nblk = blocks_for((long)g.vh * x.nhalf);
  k.x = (const char *)x.p; k.sx = x.sys_stride; k.hx = k.v.half_stride;
  k.y = (const char *)y.p; k.sy = y.sys_stride; k.hy = k.v.half_stride;
  k.out = (char *)y.p; k.so = y.sys_stride; k.ho = k.v.half_stride;
  k.c_re = cre; k.c_im = cim;
  dim3 grid(k.nblk, (unsigned)nsys);
  WD_DISPATCH_P(prec, k_caxpy, grid, k, st);
  return hip_check(hipGetLastError(), "caxpy launch");
}

template <int PI>
static void launch_convert_out(wd_prec po, dim3 grid, const KBlas &k, hipStream_t st) {
  switch (po) {
    case WD_F64: hipLaunchKernelGGL((k_convert<PI, WD_F64>), grid, dim3(BLAS_BS), 0, st, k); break;
    case WD_F32: hipLaunchKernelGGL((k_convert<PI, WD_F32>), grid, dim3(BLAS_BS), 0, st, k); break;
    case WD_F16: hipLaunchKernelGGL((k_convert<PI, WD_F16>), grid, dim3(BLAS_BS), 0, st, k); break;
    case WD_BF16: hipLaunchKernelGGL((k_convert<PI, WD_BF16>), grid, dim3(BLAS_BS), 0, st, k); break;
  }
}

wd_status blas_convert(const Geom &g, wd_prec pi, const VecRef &x, wd_prec po, const VecRef &out, double scale,
                       CgScalars *sc_inv_sqrt_rnorm, int nsys, hipStream_t st) {
  if ((unsigned)pi > 3u || (unsigned)po > 3u) return set_error(WD_ERR_PREC, "convert: bad precision");
  KBlas k{};
  k.v = vgeom(g, x.nhalf, pi);
  k.nblk = blocks_for((long)g.vpad * x.nhalf);
  k.x = (const char *)x.p; k.sx = x.sys_stride; k.hx = half_bytes(g, pi);
  k.out = (char *)out.p; k.so = out.sys_stride; k.ho = half_bytes(g, po);
  k.c_re = scale;
  k.sc = sc_inv_sqrt_rnorm;
  dim3 grid(k.nblk, (unsigned)nsys);
  switch (pi) {
    case WD_F64: launch_convert_out<WD_F64>(po, grid, k, st); break;
    case WD_F32: launch_convert_out<WD_F32>(po, grid, k, st); break;
    case WD_F16: launch_convert_out<WD_F16>(po, grid, k, st); break;
    case WD_BF16: launch_convert_out<WD_BF16>(po, grid, k, st); break;
  }
  return hip_check(hipGetLastError(), "convert launch");
}

wd_status blas_accum(const Geom &g, wd_prec pe, const VecRef &e, const VecRef &x64, double scale, CgScalars *sc,
                     int nsys, hipStream_t st) {
  KBlas k{};
  k.v = vgeom(g, e.nhalf, pe);
  k.nblk = blocks_for((long)g.vh * e.nhalf);
  k.x = (const char *)e.p; k.sx = e.sys_stride; k.hx = half_bytes(g, pe);
  k.out = (char *)x64.p; k.so = x64.sys_stride; k.ho = half_bytes(g, WD_F64);
  k.c_re = scale;
  k.sc = sc;
  dim3 grid(k.nblk, (unsigned)nsys);
  WD_DISPATCH_P(pe, k_accum, grid, k, st);
  return hip_check(hipGetLastError(), "accum launch");
}

// Blocks per system of a CG recurrence over npk packets (FP16: sites): up to
// CG_APART items per thread.  Where every block first adds up the system's
// nparts partials, 2048 blocks of all systems together, with the one that ends
// the iteration, are enough: 12 systems of 12^3x24 in FP32 take 11.8 ms, 12.2
// with twice as many.  Without that list 2047 of each system: 12 systems of
// 24^3x48 in BF16 102.3 ms, 105.1 with the cap of all together.  (2048 and the
// one that ends the iteration are one more than is resident at once: FP64 CG on
// 32^3x64 83.1 ms, 82.0 with 2047.)
static unsigned cg_blocks(const Geom &g, wd_prec pv, int nhalf, int nsys, unsigned nparts, size_t &npk) {
  const int np = pv == WD_F64 ? 12 : pv == WD_F32 ? 6 : 3;
  npk = (size_t)g.vpad * np * nhalf;
  const unsigned b = blocks_for((long)(pv == WD_F16 ? (size_t)g.vh * nhalf : npk));
  return std::min(b, nparts ? std::max(2u, BLAS_MAX_BLOCKS / (unsigned)nsys) - 1 : BLAS_MAX_BLOCKS - 1);
}

// Whether every thread of the grid has CG_SIDE packets.
static bool cg_side(wd_prec pv, const KBlas &k) {
  return pv != WD_F16 && k.npk >= (size_t)CG_SIDE * BLAS_BS * k.nblk;
}

// Whether a launch of its own ends the iteration right after the update: where
// the sums take finishing launches anyway, and half an iteration of a system
// that has just converged (two hops and the p update, once an inner solve) costs
// more than that launch in each iteration.  BF16 defect correction, end in the
// p update against after the update: 20^3x40 7.9 / 8.1 ms, 24^3x48 13.6 / 13.6,
// 32^3x64 37.8 / 37.2; 12 systems of 20^3x40 44.9 / 44.2, of 24^3x48 90.5 / 88.9.
static bool early_end(const Geom &g, wd_prec px, int nhalf, int nsys, unsigned nparts) {
  return px == WD_F32 && !nparts && (size_t)g.vh * nhalf * nsys >= ((size_t)1 << 19);
}

wd_status blas_cg_update(const Geom &g, wd_prec px, const VecRef &x, wd_prec pv, const VecRef &p, const VecRef &s,
                         const VecRef &q, CgScalars *sc, int j, int nsys, CgParts &cp, hipStream_t st) {
  if (!((px == WD_F64 && pv == WD_F64) || (px == WD_F32 && pv != WD_F64)))
    return set_error(WD_ERR_PREC, "cg_update: unsupported precision pair");
  KBlas k{};
  k.v = vgeom(g, p.nhalf, pv);
  k.nblk = cg_blocks(g, pv, p.nhalf, nsys, cp.nnorm, k.npk);
  k.x = (const char *)x.p; k.sx = x.sys_stride; k.hx = half_bytes(g, px);
  k.y = (const char *)p.p; k.sy = p.sys_stride; k.hy = half_bytes(g, pv);
  k.out = (char *)s.p; k.so = s.sys_stride; k.ho = half_bytes(g, pv);
  k.out2 = (char *)q.p; k.so2 = q.sys_stride; k.ho2 = half_bytes(g, pv);
  k.sc = sc; k.j = j;
  k.parts = cp.norm;
  k.nparts = cp.nnorm;
  k.partials = cp.ss;
  cp.nss = k.nblk;
  dim3 grid(k.nblk, (unsigned)nsys);
  const bool side = cg_side(pv, k);
#define WD_CGU(PX, PV)                                                                                       \
  if (side) hipLaunchKernelGGL((k_cg_update<PX, PV, CG_SIDE>), grid, dim3(BLAS_BS), 0, st, k);             \
  else hipLaunchKernelGGL((k_cg_update<PX, PV, CG_APART>), grid, dim3(BLAS_BS), 0, st, k)
  switch (pv) {
    case WD_F64: WD_CGU(WD_F64, WD_F64); break;
    case WD_F32: WD_CGU(WD_F32, WD_F32); break;
    case WD_F16: hipLaunchKernelGGL((k_cg_update<WD_F32, WD_F16, CG_APART>), grid, dim3(BLAS_BS), 0, st, k); break;
    case WD_BF16: WD_CGU(WD_F32, WD_BF16); break;
  }
#undef WD_CGU
  WD_TRY(hip_check(hipGetLastError(), "cg_update launch"));
  if (!early_end(g, px, p.nhalf, nsys, cp.nnorm)) return WD_OK;
  k.ss_parts = cp.ss;
  k.nss = cp.nss;
  cp.nss = 0;
  hipLaunchKernelGGL(k_cg_end, dim3((unsigned)nsys), dim3(BLAS_BS), 0, st, k);
  return hip_check(hipGetLastError(), "cg end launch");
}

wd_status blas_cg_pupdate(const Geom &g, wd_prec pv, const VecRef &r, const VecRef &p, CgScalars *sc, int j,
                          int nsys, const CgParts &cp, hipStream_t st) {
  KBlas k{};
  k.v = vgeom(g, p.nhalf, pv);
  k.nblk = cg_blocks(g, pv, p.nhalf, nsys, cp.nnorm, k.npk);
  k.x = (const char *)r.p; k.sx = r.sys_stride; k.hx = half_bytes(g, pv);
  k.out = (char *)p.p; k.so = p.sys_stride; k.ho = half_bytes(g, pv);
  k.sc = sc; k.j = j;
  k.parts = cp.norm;
  k.nparts = cp.nnorm;
  k.ss_parts = cp.ss;
  k.nss = cp.nss;
  dim3 grid(k.nblk + (cp.nss ? 1 : 0), (unsigned)nsys);
  const bool side = cg_side(pv, k);
#define WD_CGP(PV)                                                                                 \
  if (side) hipLaunchKernelGGL((k_cg_pupdate<PV, CG_SIDE>), grid, dim3(BLAS_BS), 0, st, k);      \
  else hipLaunchKernelGGL((k_cg_pupdate<PV, CG_APART>), grid, dim3(BLAS_BS), 0, st, k)
  switch (pv) {
    case WD_F64: WD_CGP(WD_F64); break;
    case WD_F32: WD_CGP(WD_F32); break;
    case WD_F16: hipLaunchKernelGGL((k_cg_pupdate<WD_F16, CG_APART>), grid, dim3(BLAS_BS), 0, st, k); break;
    case WD_BF16: WD_CGP(WD_BF16); break;
  }
#undef WD_CGP
  return hip_check(hipGetLastError(), "cg_pupdate launch");
}

wd_status launch_finish_sums(const double *partials, unsigned nblocks, int n, double *out, int ostride,
                             int accumulate, const int *skip, int sstride, hipStream_t st) {
  if (n < 1) return WD_OK;
  hipLaunchKernelGGL(k_finish_sums, dim3((unsigned)n), dim3(FIN_BS), 0, st, partials, nblocks, out, ostride,
                     accumulate, skip, sstride);
  return hip_check(hipGetLastError(), "finishing sums launch");
}

}  // namespace wd
