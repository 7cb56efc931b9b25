// FFT and stencil kernels of the pressure projection for gfx950 (wave64, LDS-staged).
//
// Phases of one projection (the FFT pressure solver of the paper's Sec. 4:
// forward FFT, vertical ODE per wavenumber in Fourier space, backward FFT):
//   xfwd     divergence D(u*) (or the FP64 residual D(u*) - D(G p1) of the
//            mixed path) computed straight into the first radix pass of the
//            x-direction real FFT; two real rows ride in one complex
//            transform and are separated afterwards
//   ffty     y-direction complex FFT of every (level, m) column
//   tridiag  FP64 tridiagonal solve in z of every (m, n) column, partitioned
//            over lanes, (0,0) column with the gauge
//   xinv     x-direction complex-to-real FFT, writes p (or p1 + delta)
//   grad     pressure-gradient correction u -= G p, w lid = 0
//
// The FFT phases exist twice: with the transform length fixed at compile
// time (CtFft, for the lengths listed in kernels.h: 16 to 4096) and with a
// runtime length (fft_lds) for every other 2^a 3^b length.
//
// Every kernel serves a group of members: blockIdx.x is mapped to a member
// through LaunchArgs::block_start, and each member's sizes and tables come
// from its MemberDesc.
#pragma once
#include <hip/hip_runtime.h>

#include "device_common.h"
#include "kernels.h"

namespace monc {

// ---------------------------------------------------------------------------
// per-row context of the stencils: offsets of the neighbouring rows and the
// vertical metrics of the row's level
// ---------------------------------------------------------------------------
struct RowCtx {
  long long off;    // row (k, j)
  long long soff;   // row (k, j-1)
  long long noff;   // row (k, j+1)
  long long plane;  // ny * nx
  int k;
  bool top;         // k < nz-1: a w face above
  bool bot;         // k > 0: a w face below
  double rho0, rhow, rhowm, rdz, rdzc, rdzcm;
  float rho0f, rhowf, rhowmf, rdzf;
};

// (rows, ny nz of them, and their level and row index fit 31 bits)
__device__ __forceinline__ int row_level(const MemberDesc& d, int r) { return (int)fast_div(r, d.ny_mul, d.ny_shift); }

__device__ __forceinline__ RowCtx make_row(const MemberDesc& d, long long row, bool valid) {
  RowCtx c;
  const int ny = d.ny, nz = d.nz;
  const long long r = valid ? row : 0;
  const int k = row_level(d, (int)r);
  const int j = (int)r - k * ny;
  c.k = k;
  c.off = r * d.nx;
  c.soff = ((long long)k * ny + (j == 0 ? ny - 1 : j - 1)) * d.nx;
  c.noff = ((long long)k * ny + (j == ny - 1 ? 0 : j + 1)) * d.nx;
  c.plane = (long long)ny * d.nx;
  c.top = k < nz - 1;
  c.bot = k > 0;
  // the level's metrics sit together (kLev64, kLev32 values a level): rhow and
  // 1/dzc are 0 on the lid row, those of the level below 0 on the bottom row
  typedef double d2 __attribute__((ext_vector_type(2)));
  typedef float f4 __attribute__((ext_vector_type(4)));
  const d2* l64 = reinterpret_cast<const d2*>(d.lev + (long long)k * kLev64);
  const d2 a = ldg(l64), b = ldg(l64 + 1), e = ldg(l64 + 2);
  c.rho0 = a.x;
  c.rdz = a.y;
  c.rhow = b.x;
  c.rhowm = b.y;
  c.rdzc = e.x;
  c.rdzcm = e.y;
  const f4 l32 = ldg(reinterpret_cast<const f4*>(d.levf + (long long)k * kLev32));
  c.rho0f = l32.x;
  c.rdzf = l32.y;
  c.rhowf = l32.z;
  c.rhowmf = l32.w;
  return c;
}

__device__ __forceinline__ RowCtx wuni(const RowCtx& c) {
  RowCtx r;
  r.off = wuni(c.off);
  r.soff = wuni(c.soff);
  r.noff = wuni(c.noff);
  r.plane = wuni(c.plane);
  r.k = wuni(c.k);
  r.top = wuni((int)c.top) != 0;
  r.bot = wuni((int)c.bot) != 0;
  r.rho0 = wuni(c.rho0);
  r.rhow = wuni(c.rhow);
  r.rhowm = wuni(c.rhowm);
  r.rdz = wuni(c.rdz);
  r.rdzc = wuni(c.rdzc);
  r.rdzcm = wuni(c.rdzcm);
  r.rho0f = wuni(c.rho0f);
  r.rhowf = wuni(c.rhowf);
  r.rhowmf = wuni(c.rhowmf);
  r.rdzf = wuni(c.rdzf);
  return r;
}

template <typename T>
__device__ __forceinline__ T div_at(const MemberDesc& d, const RowCtx& c, const T* __restrict__ u,
                                    const T* __restrict__ v, const T* __restrict__ w, int i);

template <>
__device__ __forceinline__ double div_at<double>(const MemberDesc& d, const RowCtx& c, const double* __restrict__ u,
                                                 const double* __restrict__ v, const double* __restrict__ w, int i) {
  const int im = (i == 0) ? d.nx - 1 : i - 1;
  const double hor = (u[c.off + i] - u[c.off + im]) * d.rdx + (v[c.off + i] - v[c.soff + i]) * d.rdy;
  const double ft = c.top ? c.rhow * w[c.off + i] : 0.0;
  const double fb = c.bot ? c.rhowm * w[c.off - c.plane + i] : 0.0;
  return c.rho0 * hor + (ft - fb) * c.rdz;
}

template <>
__device__ __forceinline__ float div_at<float>(const MemberDesc& d, const RowCtx& c, const float* __restrict__ u,
                                               const float* __restrict__ v, const float* __restrict__ w, int i) {
  const int im = (i == 0) ? d.nx - 1 : i - 1;
  const float hor = (u[c.off + i] - u[c.off + im]) * d.rdxf + (v[c.off + i] - v[c.soff + i]) * d.rdyf;
  const float ft = c.top ? c.rhowf * w[c.off + i] : 0.0f;
  const float fb = c.bot ? c.rhowmf * w[c.off - c.plane + i] : 0.0f;
  return c.rho0f * hor + (ft - fb) * c.rdzf;
}

// FP64 operator L p1 = D(G p1) at one point from the float first-pass
// pressure p1 and its six neighbours (pE, pW along x, pN, pS along y, pU, pD
// along z; pU, pD ignored on the lid and bottom rows).
__device__ __forceinline__ double lap_at(const MemberDesc& d, const RowCtx& c, double p0, double pE, double pW,
                                         double pN, double pS, double pU, double pD) {
  const double gxe = (pE - p0) * d.rdx, gxw = (p0 - pW) * d.rdx;
  const double gyn = (pN - p0) * d.rdy, gys = (p0 - pS) * d.rdy;
  const double ft = c.top ? c.rhow * ((pU - p0) * c.rdzc) : 0.0;
  const double fb = c.bot ? c.rhowm * ((p0 - pD) * c.rdzcm) : 0.0;
  return c.rho0 * ((gxe - gxw) * d.rdx + (gyn - gys) * d.rdy) + (ft - fb) * c.rdz;
}

// FP64 divergence D(u*) of float fields at one point
__device__ __forceinline__ double div64_at(const MemberDesc& d, const RowCtx& c, const float* __restrict__ u,
                                           const float* __restrict__ v, const float* __restrict__ w, int i) {
  const int im = (i == 0) ? d.nx - 1 : i - 1;
  const double hor = ((double)u[c.off + i] - (double)u[c.off + im]) * d.rdx +
                     ((double)v[c.off + i] - (double)v[c.soff + i]) * d.rdy;
  const double ft = c.top ? c.rhow * (double)w[c.off + i] : 0.0;
  const double fb = c.bot ? c.rhowm * (double)w[c.off - c.plane + i] : 0.0;
  return c.rho0 * hor + (ft - fb) * c.rdz;
}

// FP64 residual r = D(u*) - L p1 of the mixed path at one point, from the
// float inputs u*, v*, w* and the first-pass pressure p1 (io.s2).
__device__ __forceinline__ double resid_at(const MemberDesc& d, const RowCtx& c, const IoPtrs& io, int i) {
  const float* __restrict__ p = io.s2;
  const int nx = d.nx;
  const int im = (i == 0) ? nx - 1 : i - 1;
  const int ip = (i == nx - 1) ? 0 : i + 1;
  const double pc = p[c.off + i];
  const double pu = c.top ? (double)p[c.off + c.plane + i] : pc;
  const double pd = c.bot ? (double)p[c.off - c.plane + i] : pc;
  const double b = div64_at(d, c, reinterpret_cast<const float*>(io.u), reinterpret_cast<const float*>(io.v),
                            reinterpret_cast<const float*>(io.w), i);
  return b - lap_at(d, c, pc, p[c.off + ip], p[c.off + im], p[c.noff + i], p[c.soff + i], pu, pd);
}

// Sources of the x-forward transform: MODE 0 the divergence D(u*), MODE 1
// the mixed path's FP64 residual D(u*) - L p1, MODE 2 a given FP64 field
// (io.u) rounded to T, i.e. the spectral solve applied to an arbitrary
// right-hand side (the preconditioner of the variable-density Krylov
// solver), MODE 3 the Krylov solver's residual, updated on the way: r (io.u)
// -= alpha q (io.v), alpha = rz / dq from the iteration's scalars (io.w:
// <r, z> and <d, q>), and the workgroup's sum of dz r^2 into io.stats. The
// update as a kernel of its own read and wrote r once more.
template <typename T, int MODE>
__device__ __forceinline__ T source_at(const MemberDesc& d, const RowCtx& c, const IoPtrs& io, int i) {
  if constexpr (MODE == 0) {
    return div_at<T>(d, c, reinterpret_cast<const T*>(io.u), reinterpret_cast<const T*>(io.v),
                     reinterpret_cast<const T*>(io.w), i);
  } else if constexpr (MODE == 2) {
    return (T)reinterpret_cast<const double*>(io.u)[c.off + i];
  } else {
    return (T)resid_at(d, c, io, i);
  }
}

// MODE 3 at points i0 .. i0+V-1 of a row
template <typename T, int V>
__device__ __forceinline__ void update_vec(const RowCtx& c, const IoPtrs& io, int i0, double alpha, double dz,
                                           double& acc, T* out);

// alpha of a Krylov iteration from its scalars (kVarRZ, kVarDQ)
__device__ __forceinline__ double krylov_alpha(const void* row) {
  const double rz = ldc(static_cast<const double*>(row)), dq = ldc(static_cast<const double*>(row) + 1);
  return dq != 0.0 ? rz / dq : 0.0;
}

// Sum of x over the workgroup (any size) in a fixed order, in thread 0. buf:
// LDS of a double per thread, free for use; every thread calls it.
__device__ __forceinline__ double group_sum(double x, double* buf) {
  __syncthreads();
  buf[threadIdx.x] = x;
  __syncthreads();
  double s = 0.0;
  if (threadIdx.x < 16)
    for (int i = threadIdx.x; i < (int)blockDim.x; i += 16) s += buf[i];
  __syncthreads();
  if (threadIdx.x < 16) buf[threadIdx.x] = s;
  __syncthreads();
  s = 0.0;
  if (threadIdx.x == 0)
    for (int i = 0; i < min(16, (int)blockDim.x); ++i) s += buf[i];
  return s;
}

// ---------------------------------------------------------------------------
// Vector forms of the stencils: V consecutive points of one row (x_chunk: 16
// bytes' worth where the row length divides by it and the rows so start
// aligned, else 2 or 1). The x-neighbours outside the vector come from scalar
// loads (cache hits).
// ---------------------------------------------------------------------------
template <typename T, int V> struct Vec {
  typedef T type __attribute__((ext_vector_type(V)));
};

template <int V, typename T>
__device__ __forceinline__ typename Vec<T, V>::type ldv(const T* p) {
  return *reinterpret_cast<const typename Vec<T, V>::type*>(p);
}

// divergence D(u) at points i0 .. i0+V-1 of a row, arithmetic in T
template <typename T, int V>
__device__ __forceinline__ void div_vec(const MemberDesc& d, const RowCtx& c, const IoPtrs& io, int i0, T* out) {
  using vt = typename Vec<T, V>::type;
  const T* __restrict__ u = reinterpret_cast<const T*>(io.u);
  const T* __restrict__ v = reinterpret_cast<const T*>(io.v);
  const T* __restrict__ w = reinterpret_cast<const T*>(io.w);
  const bool f64 = sizeof(T) == 8;
  const T rdx = f64 ? (T)d.rdx : (T)d.rdxf, rdy = f64 ? (T)d.rdy : (T)d.rdyf;
  const T rho0 = f64 ? (T)c.rho0 : (T)c.rho0f, rdz = f64 ? (T)c.rdz : (T)c.rdzf;
  const T rhow = f64 ? (T)c.rhow : (T)c.rhowf, rhowm = f64 ? (T)c.rhowm : (T)c.rhowmf;
  const vt uc = ldv<V>(u + c.off + i0);
  const T um = u[c.off + (i0 == 0 ? d.nx - 1 : i0 - 1)];
  const vt vc = ldv<V>(v + c.off + i0), vs = ldv<V>(v + c.soff + i0);
  vt wc = (vt)(T)0, wb = (vt)(T)0;
  if constexpr (sizeof(T) == 8) {
    // FP64: both w loads unconditional (level k clamped on the bottom row) so
    // they issue with the others; the lid and bottom faces are selected away
    const vt wcl = ldv<V>(w + c.off + i0), wbl = ldv<V>(w + c.off - (c.bot ? c.plane : 0) + i0);
#pragma unroll
    for (int e = 0; e < V; ++e) {
      wc[e] = c.top ? wcl[e] : (T)0;
      wb[e] = c.bot ? wbl[e] : (T)0;
    }
  } else {
    // FP32: the branches keep fewer loads in flight and fewer registers live,
    // which measures faster here
    if (c.top) wc = ldv<V>(w + c.off + i0);
    if (c.bot) wb = ldv<V>(w + c.off - c.plane + i0);
  }
#pragma unroll
  for (int e = 0; e < V; ++e) {
    const T uw = e ? uc[e - 1] : um;
    out[e] = rho0 * ((uc[e] - uw) * rdx + (vc[e] - vs[e]) * rdy) + (rhow * wc[e] - rhowm * wb[e]) * rdz;
  }
}

// Both rows of a pair (k, j) and (k, j+1) of one level: row j's v is row j+1's
// southern neighbour, so 11 loads serve the two rows instead of 12. The
// arithmetic is div_vec's, term for term.
template <typename T, int V>
__device__ __forceinline__ void div_pair_vec(const MemberDesc& d, const RowCtx& c0, const RowCtx& c1,
                                             const IoPtrs& io, int i0, T* out0, T* out1) {
  using vt = typename Vec<T, V>::type;
  const T* __restrict__ u = reinterpret_cast<const T*>(io.u);
  const T* __restrict__ v = reinterpret_cast<const T*>(io.v);
  const T* __restrict__ w = reinterpret_cast<const T*>(io.w);
  const bool f64 = sizeof(T) == 8;
  const T rdx = f64 ? (T)d.rdx : (T)d.rdxf, rdy = f64 ? (T)d.rdy : (T)d.rdyf;
  // one level: both rows share the vertical coefficients and lid flags
  const T rho0 = f64 ? (T)c0.rho0 : (T)c0.rho0f, rdz = f64 ? (T)c0.rdz : (T)c0.rdzf;
  const T rhow = f64 ? (T)c0.rhow : (T)c0.rhowf, rhowm = f64 ? (T)c0.rhowm : (T)c0.rhowmf;
  const int iw = (i0 == 0) ? d.nx - 1 : i0 - 1;
  const vt u0 = ldv<V>(u + c0.off + i0), u1 = ldv<V>(u + c1.off + i0);
  const T um0 = u[c0.off + iw], um1 = u[c1.off + iw];
  const vt vs = ldv<V>(v + c0.soff + i0), v0 = ldv<V>(v + c0.off + i0), v1 = ldv<V>(v + c1.off + i0);
  vt wc0 = (vt)(T)0, wb0 = (vt)(T)0, wc1 = (vt)(T)0, wb1 = (vt)(T)0;
  if constexpr (sizeof(T) == 8) {
    const long long bo = c0.bot ? c0.plane : 0;
    const vt a0 = ldv<V>(w + c0.off + i0), a1 = ldv<V>(w + c1.off + i0);
    const vt b0 = ldv<V>(w + c0.off - bo + i0), b1 = ldv<V>(w + c1.off - bo + i0);
#pragma unroll
    for (int e = 0; e < V; ++e) {
      wc0[e] = c0.top ? a0[e] : (T)0;
      wc1[e] = c0.top ? a1[e] : (T)0;
      wb0[e] = c0.bot ? b0[e] : (T)0;
      wb1[e] = c0.bot ? b1[e] : (T)0;
    }
  } else {
    if (c0.top) {
      wc0 = ldv<V>(w + c0.off + i0);
      wc1 = ldv<V>(w + c1.off + i0);
    }
    if (c0.bot) {
      wb0 = ldv<V>(w + c0.off - c0.plane + i0);
      wb1 = ldv<V>(w + c1.off - c0.plane + i0);
    }
  }
#pragma unroll
  for (int e = 0; e < V; ++e) {
    const T uw0 = e ? u0[e - 1] : um0, uw1 = e ? u1[e - 1] : um1;
    out0[e] = rho0 * ((u0[e] - uw0) * rdx + (v0[e] - vs[e]) * rdy) + (rhow * wc0[e] - rhowm * wb0[e]) * rdz;
    out1[e] = rho0 * ((u1[e] - uw1) * rdx + (v1[e] - v0[e]) * rdy) + (rhow * wc1[e] - rhowm * wb1[e]) * rdz;
  }
}

typedef float f4v __attribute__((ext_vector_type(4)));
template <int W> using fwv = float __attribute__((ext_vector_type(W)));

template <int W>
__device__ __forceinline__ fwv<W> ldw(const float* p) {
  return *reinterpret_cast<const fwv<W>*>(p);
}

// FP64 residual D(u*) - L p1 at points i0 .. i0+W-1 of a row from the loaded
// neighbourhood (float data; pc: p1 of the row, pn/ps: rows j +- 1, pu/pd:
// levels k +- 1, pe/pw: x-neighbours outside the vector, um: u west of the
// vector; pu/pd, wc/wb ignored on the lid and bottom rows).
// The same terms as div64_at - lap_at with the row's coefficients multiplied
// out once (rho0/dx, rho0/dx^2, ...) and every pressure difference taken
// before it is scaled: one FP64 fused multiply-add per term. The callers pass
// wc = 0 and pu = pc on the lid row, wb = 0 and pd = pc on the bottom row,
// where the row's rhow (lid) and rhowm (bottom) are 0 as well. A point's
// value does not depend on W.
template <int W>
__device__ __forceinline__ void resid_core(const MemberDesc& d, const RowCtx& c, fwv<W> pc, fwv<W> pn, fwv<W> ps,
                                           fwv<W> pu, fwv<W> pd, float pw, float pe, fwv<W> uc, float um,
                                           fwv<W> vc, fwv<W> vs, fwv<W> wc, fwv<W> wb, float* out) {
  const double bx = c.rho0 * d.rdx, by = c.rho0 * d.rdy;      // D(u*) horizontal
  const double wt = c.rdz * c.rhow, wm = c.rdz * c.rhowm;     // D(u*) vertical
  const double ax = bx * d.rdx, ay = by * d.rdy;              // L p1 horizontal
  const double cu = wt * c.rdzc, cd = wm * c.rdzcm;           // L p1 vertical
#pragma unroll
  for (int e = 0; e < W; ++e) {
    const double uW = (e > 0) ? (double)uc[e > 0 ? e - 1 : 0] : (double)um;
    const double p0 = pc[e];
    const double pE = (e < W - 1) ? (double)pc[e < W - 1 ? e + 1 : 0] : (double)pe;
    const double pW = (e > 0) ? (double)pc[e > 0 ? e - 1 : 0] : (double)pw;
    const double dxx = (pE - p0) - (p0 - pW), dyy = ((double)pn[e] - p0) - (p0 - (double)ps[e]);
    double r = bx * ((double)uc[e] - uW);
    r = fma(by, (double)vc[e] - (double)vs[e], r);
    r = fma(wt, (double)wc[e], r);
    r = fma(-wm, (double)wb[e], r);
    r = fma(-ax, dxx, r);
    r = fma(-ay, dyy, r);
    r = fma(-cu, (double)pu[e] - p0, r);
    r = fma(cd, p0 - (double)pd[e], r);
    out[e] = (float)r;
  }
}

template <int W>
__device__ __forceinline__ void resid_vec(const MemberDesc& d, const RowCtx& c, const IoPtrs& io, int i0,
                                          float* out) {
  const float* __restrict__ u = reinterpret_cast<const float*>(io.u);
  const float* __restrict__ v = reinterpret_cast<const float*>(io.v);
  const float* __restrict__ w = reinterpret_cast<const float*>(io.w);
  const float* __restrict__ p = io.s2;
  const int nx = d.nx;
  const int iw = (i0 == 0) ? nx - 1 : i0 - 1, ie = (i0 + W == nx) ? 0 : i0 + W;
  const fwv<W> pc = ldw<W>(p + c.off + i0);
  const float pw = p[c.off + iw], pe = p[c.off + ie];
  const fwv<W> pn = ldw<W>(p + c.noff + i0), ps = ldw<W>(p + c.soff + i0);
  const fwv<W> uc = ldw<W>(u + c.off + i0);
  const float um = u[c.off + iw];
  const fwv<W> vc = ldw<W>(v + c.off + i0), vs = ldw<W>(v + c.soff + i0);
  fwv<W> pu = pc, pd = pc, wc = (fwv<W>)0.0f, wb = (fwv<W>)0.0f;
  if (c.top) {
    pu = ldw<W>(p + c.off + c.plane + i0);
    wc = ldw<W>(w + c.off + i0);
  }
  if (c.bot) {
    pd = ldw<W>(p + c.off - c.plane + i0);
    wb = ldw<W>(w + c.off - c.plane + i0);
  }
  resid_core<W>(d, c, pc, pn, ps, pu, pd, pw, pe, uc, um, vc, vs, wc, wb, out);
}

// Both rows of a pair (k, j) and (k, j+1) of one level: they share p1 rows j
// and j+1 and v row j, so 17 vector loads serve the two rows instead of 20.
template <int W>
__device__ __forceinline__ void resid_pair_vec(const MemberDesc& d, const RowCtx& c0, const RowCtx& c1,
                                               const IoPtrs& io, int i0, float* out0, float* out1) {
  const float* __restrict__ u = reinterpret_cast<const float*>(io.u);
  const float* __restrict__ v = reinterpret_cast<const float*>(io.v);
  const float* __restrict__ w = reinterpret_cast<const float*>(io.w);
  const float* __restrict__ p = io.s2;
  const int nx = d.nx;
  const int iw = (i0 == 0) ? nx - 1 : i0 - 1, ie = (i0 + W == nx) ? 0 : i0 + W;
  const fwv<W> ps = ldw<W>(p + c0.soff + i0), p0 = ldw<W>(p + c0.off + i0), p1 = ldw<W>(p + c1.off + i0);
  const fwv<W> p2 = ldw<W>(p + c1.noff + i0);
  const float pw0 = p[c0.off + iw], pe0 = p[c0.off + ie], pw1 = p[c1.off + iw], pe1 = p[c1.off + ie];
  const fwv<W> u0 = ldw<W>(u + c0.off + i0), u1 = ldw<W>(u + c1.off + i0);
  const float um0 = u[c0.off + iw], um1 = u[c1.off + iw];
  const fwv<W> vs = ldw<W>(v + c0.soff + i0), v0 = ldw<W>(v + c0.off + i0), v1 = ldw<W>(v + c1.off + i0);
  fwv<W> pu0 = p0, pd0 = p0, pu1 = p1, pd1 = p1;
  fwv<W> wc0 = (fwv<W>)0.0f, wb0 = (fwv<W>)0.0f, wc1 = (fwv<W>)0.0f, wb1 = (fwv<W>)0.0f;
  if (c0.top) {  // one level: c0.top == c1.top, c0.bot == c1.bot
    pu0 = ldw<W>(p + c0.off + c0.plane + i0);
    pu1 = ldw<W>(p + c1.off + c1.plane + i0);
    wc0 = ldw<W>(w + c0.off + i0);
    wc1 = ldw<W>(w + c1.off + i0);
  }
  if (c0.bot) {
    pd0 = ldw<W>(p + c0.off - c0.plane + i0);
    pd1 = ldw<W>(p + c1.off - c1.plane + i0);
    wb0 = ldw<W>(w + c0.off - c0.plane + i0);
    wb1 = ldw<W>(w + c1.off - c1.plane + i0);
  }
  resid_core<W>(d, c0, p0, p1, ps, pu0, pd0, pw0, pe0, u0, um0, v0, vs, wc0, wb0, out0);
  resid_core<W>(d, c1, p1, p2, p0, pu1, pd1, pw1, pe1, u1, um1, v1, v0, wc1, wb1, out1);
}

template <typename T, int V>
__device__ __forceinline__ void update_vec(const RowCtx& c, const IoPtrs& io, int i0, double alpha, double dz,
                                           double& acc, T* out) {
  constexpr int W = V % 2 == 0 ? 2 : 1;
  using dv = typename Vec<double, W>::type;
  double* r = reinterpret_cast<double*>(io.u) + c.off + i0;
  const double* q = reinterpret_cast<const double*>(io.v) + c.off + i0;
#pragma unroll
  for (int e = 0; e < V; e += W) {
    dv x = ldv<W>(r + e);
    const dv y = ldv<W>(q + e);
#pragma unroll
    for (int h = 0; h < W; ++h) {
      x[h] -= alpha * y[h];
      acc += dz * x[h] * x[h];
      out[e + h] = (T)x[h];
    }
    *reinterpret_cast<dv*>(r + e) = x;
  }
}

template <typename T, int MODE, int V>
__device__ __forceinline__ void source_vec(const MemberDesc& d, const RowCtx& c, const IoPtrs& io, int i0, T* out) {
  if constexpr (MODE == 0) {
    div_vec<T, V>(d, c, io, i0, out);
  } else if constexpr (MODE == 2) {
    constexpr int W = V % 2 == 0 ? 2 : 1;
    const double* __restrict__ r = reinterpret_cast<const double*>(io.u) + c.off + i0;
#pragma unroll
    for (int e = 0; e < V; e += W) {
      const typename Vec<double, W>::type x = ldv<W>(r + e);
#pragma unroll
      for (int h = 0; h < W; ++h) out[e + h] = (T)x[h];
    }
  } else {
    resid_vec<V>(d, c, io, i0, reinterpret_cast<float*>(out));
  }
}

// Separate two real rows packed as z = a + i b:
// A[m] = (Z[m] + conj Z[N-m])/2, B[m] = (Z[m] - conj Z[N-m])/(2i).
// (row 0 gives A[m], row 1 gives B[m]; zr = Z[N-m])
template <typename T>
__device__ __forceinline__ cx<T> split_bin(cx<T> z, cx<T> zr, int row) {
  const T h = (T)0.5;
  return row ? cx<T>{h * (z.y + zr.y), h * (zr.x - z.x)} : cx<T>{h * (z.x + zr.x), h * (z.y - zr.y)};
}

// Spectral layout (column blocks of sbw bins, see MemberDesc): the value of
// row r = k*ny + j at bin m sits at spec_row(r) + spec_col(m). Levels are
// `plane` apart (padded so that the plane stride is an odd multiple of 256
// bytes); inside a block the rows are sbw apart, so a y-FFT tile of sbw
// columns is one contiguous run and a row pair writes 2 sbw adjacent values.
__device__ __forceinline__ long long spec_row(const MemberDesc& d, long long r) {
  const int k = row_level(d, (int)r);
  return (long long)k * d.plane + (long long)((int)r - k * d.ny) * d.sbw;
}
__device__ __forceinline__ long long spec_col(const MemberDesc& d, int m) {
  return (long long)(m >> d.lbw) * d.bst + (m & (d.sbw - 1));
}
// A row pair's spectral values in slot order: slots walk the column blocks,
// and inside a block first row 0's sbw bins, then row 1's. When the two rows
// are adjacent (same level) that is their memory order, so consecutive lanes
// touch consecutive addresses and a store or load covers 2 sbw values at a
// time. Slot s holds bin m of row `row` at offset `off` from the row start.
struct PairSlot {
  int row, m;
  long long off;
};
__device__ __forceinline__ PairSlot pair_slot(const MemberDesc& d, int s) {
  const int blk = s >> (d.lbw + 1), w = s & (2 * d.sbw - 1);
  return PairSlot{w >> d.lbw, (blk << d.lbw) | (w & (d.sbw - 1)), (long long)blk * d.bst + (w & (d.sbw - 1))};
}
// slots covering bins 0 .. nxh-1 (whole blocks)
__device__ __forceinline__ int pair_slots(const MemberDesc& d) { return ((d.nxh + d.sbw - 1) >> d.lbw) << (d.lbw + 1); }

// Row pairs of the stencil kernels in (level, pair) tiles: consecutive
// pair slots walk d.ptj pairs of d.ptk consecutive levels before moving on, so
// the rows a stencil re-reads (levels k +- 1, rows j +- 1) are read by
// workgroups that run at about the same time on the same XCD and meet in its
// L2. ptk = 1 or odd ny (pairs straddle levels) keeps the linear order.
// Bijection of [0, nz * per) that walks tiles of TJ consecutive items of TK
// consecutive levels (per items per level), ragged tiles at the edges;
// identity for TK <= 1 and beyond the grid.
// (32-bit arithmetic: nz * per, a count of rows or row pairs, fits 32 bits)
__device__ __forceinline__ long long tiled_index(long long p, long long per, int nz, int TK, int TJ) {
  if (TK <= 1 || p >= (long long)nz * per) return p;
  const int pi = (int)p, pe = (int)per;
  const int blk = TK * pe;
  const int kb = pi / blk;
  const int rem = pi - kb * blk;
  const int tk = min(TK, nz - kb * TK);          // levels in this block
  const int jt = rem / (tk * TJ);
  const int tj = min(TJ, pe - jt * TJ);
  const int in = rem - jt * tk * TJ;
  const int k = kb * TK + in / tj;
  const int jp = jt * TJ + in % tj;
  return (long long)k * pe + jp;
}

__device__ __forceinline__ long long tiled_pair(const MemberDesc& d, long long p) {
  if (d.ny & 1) return p;
  return tiled_index(p, d.ny / 2, d.nz, d.ptk, d.ptj);
}

// ---------------------------------------------------------------------------
// x-direction forward real FFT, compile-time length N (NT = ct_threads(N)
// threads per transform; blockDim =
// transforms per workgroup * NT)
// ---------------------------------------------------------------------------
// The transform of the row pair `pair` by the NT threads q of instance inst
// (ipw in the workgroup lb): stencil, FFT, half spectrum into the spectral
// buffer. Returns the thread's part of MODE 3's sum. LEVEL: a pair of the
// workgroup's level (k_level_fwd); in = false only takes part in the barriers.
// (The descriptor by value, here and below: by reference the compiler orders the
// loads otherwise and the FP64 kernels measure 3-6 % slower.)
template <typename T, int MODE, int N, bool LEVEL>
__device__ __forceinline__ double xfwd_pair(MemberDesc d, IoPtrs io, int lb, int ipw, int inst, int q,
                                            long long pair, bool in) {
  extern __shared__ unsigned char smem_raw[];
  constexpr int NT = ct_threads(N, sizeof(T));
  using F = CtFft<T, N, NT, false>;
  // scalar row contexts for the residual only, and only where a transform
  // spans whole waves (NT a multiple of 64: then no wave holds lanes of two
  // transforms): its registers fall from 174 to 126 and its occupancy rises
  // from 2 to 4 waves per SIMD, and it gains; the divergence variants measure
  // slower with scalar contexts
  constexpr bool UNI = NT % 64 == 0 && MODE == 1;
  cx<T>* lds = reinterpret_cast<cx<T>*>(smem_raw) + inst * xlds_len(N, 2 * sizeof(T));
  const long long r0 = 2 * pair, r1 = 2 * pair + 1;
  const bool v0 = in && r0 < d.nrow, v1 = in && r1 < d.nrow;
  RowCtx c0 = make_row(d, r0, v0), c1 = make_row(d, r1, v1);
  if constexpr (UNI) {
    c0 = wuni(c0);
    c1 = wuni(c1);
  }
  // 1. vector phase: the stencil on chunks of V points of both rows, packed as
  //    z = row0 + i row1 into LDS in natural order: chunk i0 of the rows with
  //    contexts (c0, c1) and validity (v0, v1) into transform slot L
  constexpr int V = x_chunk(N, sizeof(T)), NCH = N / V;  // chunks of a row
  double alpha = 0.0, dz0 = 0.0, dz1 = 0.0, rr = 0.0;     // MODE 3
  if constexpr (MODE == 3) {
    alpha = krylov_alpha(io.w);
    dz0 = ldg(d.dz + c0.k);
    dz1 = ldg(d.dz + c1.k);
  }
  auto stencil = [&](const RowCtx& c0, const RowCtx& c1, bool v0, bool v1, int i0, cx<T>* L) {
    T s0[V], s1[V];
    // a full pair within one level (even ny): the two rows share loads
    const bool pair = !(d.ny & 1) && v1;
    if constexpr (MODE == 3) {
#pragma unroll
      for (int e = 0; e < V; ++e) s0[e] = s1[e] = (T)0;
      if (v0) update_vec<T, V>(c0, io, i0, alpha, dz0, rr, s0);
      if (v1) update_vec<T, V>(c1, io, i0, alpha, dz1, rr, s1);
    } else if constexpr (sizeof(T) == 8) {
      if (MODE == 0 && pair) {
        div_pair_vec<T, V>(d, c0, c1, io, i0, s0, s1);
      } else {
        // both rows unconditionally (an invalid row's context points at row
        // 0), so all loads of the chunk issue together; invalid rows zeroed
        source_vec<T, MODE, V>(d, c0, io, i0, s0);
        source_vec<T, MODE, V>(d, c1, io, i0, s1);
#pragma unroll
        for (int e = 0; e < V; ++e) {
          s0[e] = v0 ? s0[e] : (T)0;
          s1[e] = v1 ? s1[e] : (T)0;
        }
      }
    } else {
      if (pair && MODE == 0) {
        div_pair_vec<T, V>(d, c0, c1, io, i0, s0, s1);
      } else if (pair && MODE == 1) {
        resid_pair_vec<V>(d, c0, c1, io, i0, s0, s1);
      } else {
        if (v0) source_vec<T, MODE, V>(d, c0, io, i0, s0);
        else
          for (int e = 0; e < V; ++e) s0[e] = (T)0;
        if (v1) source_vec<T, MODE, V>(d, c1, io, i0, s1);
        else
          for (int e = 0; e < V; ++e) s1[e] = (T)0;
      }
    }
#pragma unroll
    for (int e = 0; e < V; ++e) L[xpad<T, N>(i0 + e)] = cx<T>{s0[e], s1[e]};
  };
  if constexpr (MODE == 1 && !LEVEL && xres_wave_rows(N)) {
    // residual with transforms narrower than a wave: each wave takes one
    // transform's run of 64 chunks of W points at a time (the host launches
    // whole waves), so the row contexts are wave-uniform, in scalar
    // registers, as in the case above; this halves the registers and doubles
    // the waves. Every point's value is the per-thread mapping's.
    constexpr int W = xres_chunk(N);
    constexpr int C = N / (64 * W);  // wave runs per transform
    const int nw = blockDim.x / 64, wv = wuni((int)(threadIdx.x / 64)), ln = threadIdx.x & 63;
    cx<T>* lds0 = reinterpret_cast<cx<T>*>(smem_raw);
    for (int it = wv; it < ipw * C; it += nw) {
      const int ins = it / C, ch = it - ins * C;
      const long long pr = tiled_pair(d, (long long)lb * ipw + ins);
      const bool w0 = 2 * pr < d.nrow, w1 = 2 * pr + 1 < d.nrow;
      const RowCtx e0 = wuni(make_row(d, 2 * pr, w0)), e1 = wuni(make_row(d, 2 * pr + 1, w1));
      const int i0 = (ch * 64 + ln) * W;
      float s0[W], s1[W];
      if (!(d.ny & 1) && w1) {
        resid_pair_vec<W>(d, e0, e1, io, i0, s0, s1);
      } else {
        if (w0) resid_vec<W>(d, e0, io, i0, s0);
        else
          for (int e = 0; e < W; ++e) s0[e] = 0.0f;
        if (w1) resid_vec<W>(d, e1, io, i0, s1);
        else
          for (int e = 0; e < W; ++e) s1[e] = 0.0f;
      }
      cx<T>* L = lds0 + ins * xlds_len(N, 2 * sizeof(T));
#pragma unroll
      for (int e = 0; e < W; ++e) L[xpad<T, N>(i0 + e)] = cx<T>{s0[e], s1[e]};
    }
  } else {
#pragma unroll
    for (int t = 0; t < (NCH + NT - 1) / NT; ++t)
      if (NCH % NT == 0 || q + t * NT < NCH) stencil(c0, c1, v0, v1, (q + t * NT) * V, lds);
  }
  __syncthreads();
  cx<T> v[F::VMAX];
#pragma unroll
  for (int t = 0; t < F::BT0; ++t) {
    const int b = q + t * NT;
    if (F::valid_first(b)) {
#pragma unroll
      for (int r = 0; r < F::R0; ++r) v[t * F::R0 + r] = lds[xpad<T, N>(b + r * F::NB0)];
    }
  }
  __syncthreads();
  auto li = [](int i) { return xpad<T, N>(i); };
  F::run(v, lds, li, q, reinterpret_cast<const cx<T>*>(d.twx));
#pragma unroll
  for (int t = 0; t < F::BTL; ++t) {
    const int b = q + t * NT;
    if (F::valid_last(b)) {
#pragma unroll
      for (int r = 0; r < F::RL; ++r) lds[xpad<T, N>(F::out_index(q, t, r))] = v[t * F::RL + r];
    }
  }
  __syncthreads();
  cx<T>* S = reinterpret_cast<cx<T>*>(io.spec);
  const long long so0 = spec_row(d, v0 ? r0 : 0), so1 = spec_row(d, v1 ? r1 : 0);
  const int ns = pair_slots(d);
  if (sizeof(T) == 4 && d.sbw >= 2) {
    // FP32 with column blocks at least 2 wide: a lane takes two adjacent
    // slots (bins m, m+1 of one row, adjacent in memory, 16-byte aligned:
    // m, the block and row offsets and the plane are even) and stores them
    // with one 16-byte access; a block's last valid bin may be alone. Half
    // the store instructions of one slot per lane, which measured as the
    // costliest phase of these kernels.
    for (int s2 = q; s2 < ns / 2; s2 += NT) {
      const PairSlot ps = pair_slot(d, 2 * s2);
      if (ps.m < d.nxh && (ps.row ? v1 : v0)) {
        const cx<T> b0 = split_bin<T>(lds[xpad<T, N>(ps.m)], lds[xpad<T, N>(ps.m == 0 ? 0 : N - ps.m)], ps.row);
        cx<T>* dst = S + (ps.row ? so1 : so0) + ps.off;
        if (ps.m + 1 < d.nxh) {
          const cx<T> b1 = split_bin<T>(lds[xpad<T, N>(ps.m + 1)], lds[xpad<T, N>(N - ps.m - 1)], ps.row);
          typedef T t4 __attribute__((ext_vector_type(4)));
          t4 v;
          v[0] = b0.x;
          v[1] = b0.y;
          v[2] = b1.x;
          v[3] = b1.y;
          *reinterpret_cast<t4*>(dst) = v;
        } else {
          *dst = b0;
        }
      }
    }
  } else {
    for (int s = q; s < ns; s += NT) {
      const PairSlot ps = pair_slot(d, s);
      if (ps.m < d.nxh && (ps.row ? v1 : v0)) {
        const cx<T> z = lds[xpad<T, N>(ps.m)];
        const cx<T> zr = lds[xpad<T, N>(ps.m == 0 ? 0 : N - ps.m)];
        S[(ps.row ? so1 : so0) + ps.off] = split_bin<T>(z, zr, ps.row);
      }
    }
  }
  return rr;
}

// The residual variant at lengths whose transforms share a wave and whose
// stencil does not walk whole rows per wave (lengths that are not a multiple
// of 64, such as 16-48, 96, 144, 288, or whose whole-wave workgroups would
// pass 512 threads: 1152, 1728, 2304, 3456) keeps its row contexts in vector
// registers: about 172 registers, 2 waves per SIMD. A budget for 3 spills 2-6
// registers and measured about 1 % faster where it applied before the
// whole-row stencil; a budget for 5 waves at the longer lengths spills 16 and
// loses 6 %.
template <typename T, int MODE, int N>
__global__ void __launch_bounds__(512)
    __attribute__((amdgpu_waves_per_eu(MODE == 1 && ct_threads(N, sizeof(T)) % 64 != 0 && !xres_wave_rows(N) ? 3 : 1, 8)))
    k_xfwd_ct(LaunchArgs a) {
  constexpr int NT = ct_threads(N, sizeof(T));
  extern __shared__ unsigned char smem_raw[];
  const Member mb = launch_member(a, blockIdx.x);
  const MemberDesc d = load_desc(mb.desc);
  keep_x(d);
  if (skipped(d)) return;
  const IoPtrs& io = mb.io;
  // workgroups in launch order for the residual (1-7 % faster than grouped
  // by XCD: 2048^2 x 160, 1024^2 x 256, 4096^2 x 64 and the ensemble), by XCD
  // for the divergence (FP32 2 % faster that way at 2048^2 x 160; FP64 4 %
  // slower there but 7 % faster at 4096^2 x 64) and the given-field mode
  constexpr bool PLAIN = MODE == 1;
  const int lb = PLAIN ? (int)blockIdx.x - mb.start : xcd_local_block(mb);
  const int ipw = blockDim.x / NT;
  constexpr bool UNI = NT % 64 == 0 && MODE == 1;
  const int inst = UNI ? wuni((int)(threadIdx.x / NT)) : (int)(threadIdx.x / NT);
  const int q = threadIdx.x - inst * NT;
  const long long pair = tiled_pair(d, (long long)lb * ipw + inst);
  const double rr = xfwd_pair<T, MODE, N, false>(d, io, lb, ipw, inst, q, pair, true);
  if constexpr (MODE == 3) {
    const double s = group_sum(rr, reinterpret_cast<double*>(smem_raw));
    if (threadIdx.x == 0) io.stats[blockIdx.x] = s;
  }
}

// runtime length (fallback)
template <typename T, int MODE>
__global__ void __launch_bounds__(1024) k_xfwd_gen(LaunchArgs a) {
  extern __shared__ unsigned char smem_raw[];
  cx<T>* smem = reinterpret_cast<cx<T>*>(smem_raw);
  const Member mb = launch_member(a, blockIdx.x);
  const MemberDesc d = load_desc(mb.desc);
  keep_x(d);
  if (skipped(d)) return;
  const IoPtrs& io = mb.io;
  const int lb = xcd_local_block(mb);
  const int N = d.nx, nt = d.fx.nt;
  const int ipw = blockDim.x / nt;
  const int inst = threadIdx.x / nt;
  const bool active = inst < ipw;
  const int q = active ? (int)(threadIdx.x - inst * nt) : kBig;
  cx<T>* buf = smem + (active ? inst : 0) * N;
  const long long pair = tiled_pair(d, (long long)lb * ipw + inst);
  const long long r0 = 2 * pair, r1 = 2 * pair + 1;
  const bool v0 = active && r0 < d.nrow, v1 = active && r1 < d.nrow;
  const RowCtx c0 = make_row(d, r0, v0), c1 = make_row(d, r1, v1);
  double alpha = 0.0, dz0 = 0.0, dz1 = 0.0, rr = 0.0;  // MODE 3
  if constexpr (MODE == 3) {
    alpha = krylov_alpha(io.w);
    dz0 = ldg(d.dz + c0.k);
    dz1 = ldg(d.dz + c1.k);
  }
  if (active) {
    for (int i = q; i < N; i += nt) {
      T s0 = 0, s1 = 0;
      if constexpr (MODE == 3) {
        if (v0) update_vec<T, 1>(c0, io, i, alpha, dz0, rr, &s0);
        if (v1) update_vec<T, 1>(c1, io, i, alpha, dz1, rr, &s1);
      } else {
        if (v0) s0 = source_at<T, MODE>(d, c0, io, i);
        if (v1) s1 = source_at<T, MODE>(d, c1, io, i);
      }
      buf[i] = cx<T>{s0, s1};
    }
  }
  __syncthreads();
  fft_lds<T, false>(buf, 1, d.fx, reinterpret_cast<const cx<T>*>(d.twx), q);
  if (active) {
    cx<T>* S = reinterpret_cast<cx<T>*>(io.spec);
    const long long so0 = spec_row(d, v0 ? r0 : 0), so1 = spec_row(d, v1 ? r1 : 0);
    for (int m = q; m < d.nxh; m += nt) {
      const cx<T> z = buf[m], zr = buf[m == 0 ? 0 : N - m];
      const long long cm = spec_col(d, m);
      if (v0) S[so0 + cm] = split_bin<T>(z, zr, 0);
      if (v1) S[so1 + cm] = split_bin<T>(z, zr, 1);
    }
  }
  if constexpr (MODE == 3) {
    const double s = group_sum(rr, reinterpret_cast<double*>(smem_raw));
    if (threadIdx.x == 0) io.stats[blockIdx.x] = s;
  }
}

// ---------------------------------------------------------------------------
// y-direction complex FFT, in place on the spectral buffer. A workgroup takes
// one level and MT = blockDim / NT consecutive m columns; LDS holds them as
// [j][c] so that consecutive lanes touch consecutive columns (128-byte rows).
// ---------------------------------------------------------------------------
template <typename T, bool INV, int N, int EPT>
__global__ void __launch_bounds__(1024) k_ffty_ct(LaunchArgs a) {
  constexpr int NT = ct_threads_y(N, EPT);
  using F = CtFft<T, N, NT, INV>;
  extern __shared__ unsigned char smem_raw[];
  cx<T>* lds = reinterpret_cast<cx<T>*>(smem_raw);
  const Member mb = launch_member(a, blockIdx.x);
  const MemberDesc d = load_desc(mb.desc);
  keep_y(d);
  if (skipped(d)) return;
  const IoPtrs& io = mb.io;
  const int lb = xcd_local_block(mb);
  const int mt = blockDim.x / NT;
  const int tiles = (d.nxh + mt - 1) / mt;
  const int k = lb / tiles;
  const int c = threadIdx.x % mt;
  const int q = threadIdx.x / mt;
  const int m = (lb - k * tiles) * mt + c;
  constexpr bool part = true;
#include "ffty_column.h"
}

// y-direction complex FFT, persistent form (FP32, 32 elements per thread, so
// that the 8 columns of a 2048-point tile take 512 threads and the prefetch
// below fits the register budget of two waves per SIMD). The grid covers the
// CUs once; workgroup w walks the launch's tiles w, w + gridDim.x, ... and
// issues the loads of its next tile before transforming the current one, so
// that the transform, its LDS exchanges and its stores overlap the next
// tile's loads (a workgroup holds a CU's LDS alone, so nothing else would
// cover them). Twiddles come from an LDS copy of the table: a global load
// issued during the transform would wait behind the prefetched tile.
template <bool INV, int N>
__global__ void __launch_bounds__(512) k_ffty_pp(LaunchArgs a) {
  using T = float;
  constexpr int NT = ct_threads_y(N, 32);
  constexpr int MT = pp_columns(N);  // columns per tile
  using F = CtFft<T, N, NT, INV>;
  extern __shared__ unsigned char smem_raw[];
  cx<T>* lds = reinterpret_cast<cx<T>*>(smem_raw);
  cx<T>* twl = lds + N * MT;
  const int total = a.block_start[a.nmem];
  if ((int)blockIdx.x >= total) return;
  // every member of a launch has the same length N, hence the same table
  {
    const cx<T>* tw = reinterpret_cast<const cx<T>*>(a.mem[0]->twy);
    for (int i = threadIdx.x; i < N; i += blockDim.x) twl[i] = load_tw(tw + i);
  }
  // Tile tb of the launch: a workgroup-uniform base (the tile's first column
  // in its level) and this lane's 32-bit element offset from it, so that every
  // access is a scalar base plus one vector offset. A column past nxh takes
  // the level's last column (transformed, never stored).
  struct Tile {
    cx<T>* base;
    unsigned off;
    int rs;
    bool valid, live;
  };
  auto tile = [&](int tb, int c) {
    const int mi = find_member(a, tb);
    const MemberDesc& d = *a.mem[mi];
    const int lb = tb - a.block_start[mi];
    const int tiles = (d.nxh + MT - 1) / MT;
    const int k = lb / tiles;
    const int m0 = (lb - k * tiles) * MT;
    const int m = m0 + c;
    Tile t;
    t.valid = m < d.nxh;
    t.live = !skipped(d);
    t.rs = wuni(d.sbw);
    const long long b0 = (long long)k * d.plane + spec_col(d, m0);
    t.base = reinterpret_cast<cx<T>*>(a.io[mi].spec) + b0;
    t.off = (unsigned)(spec_col(d, t.valid ? m : d.nxh - 1) - spec_col(d, m0));
    return t;
  };
  // element i of the lane's column (global-address-space accesses through
  // the two-float vector type)
  typedef T pair __attribute__((ext_vector_type(2)));
  auto ld = [](const Tile& t, int i) -> cx<T> {
    const pair x = ((const __attribute__((address_space(1))) pair*)t.base)[t.off + (unsigned)(i * t.rs)];
    return cx<T>{x.x, x.y};
  };
  auto st = [](const Tile& t, int i, cx<T> x) {
    ((__attribute__((address_space(1))) pair*)t.base)[t.off + (unsigned)(i * t.rs)] = pair{x.x, x.y};
  };
  cx<T> v[F::VMAX], nx[F::VMAX];
  // The lane's column and row index are re-read through an empty asm at every
  // tile: the LDS and twiddle addresses derived from them are then computed
  // where they are used instead of being hoisted out of the loop, where they
  // would hold registers the prefetched tile needs.
  auto lane = [](int& c, int& q) {
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    c = t % MT;
    q = t / MT;
  };
  int cur = blockIdx.x, c, q;
  lane(c, q);
  Tile tc = tile(cur, c);
  auto load = [&](const Tile& t, int q, cx<T>* dst) {
#pragma unroll
    for (int u = 0; u < F::BT0; ++u) {
      const int b = q + u * NT;
      if (F::valid_first(b)) {
#pragma unroll
        for (int r = 0; r < F::R0; ++r) dst[u * F::R0 + r] = ld(t, b + r * F::NB0);
      }
    }
  };
  if (tc.live) load(tc, q, v);
  __syncthreads();  // the twiddle table
  while (true) {
    const int nxt = cur + gridDim.x;
    Tile tn;
    tn.live = false;
    lane(c, q);
    if (nxt < total) {
      tn = tile(nxt, c);
      if (tn.live) load(tn, q, nx);
    }
    if (tc.live) {  // uniform over the workgroup (one member per tile)
      lane(c, q);
      F::run_tw(v, lds, [c](int i) { return i * MT + c; }, q, [twl](int i) { return twl[i]; });
      if (tc.valid) {
#pragma unroll
        for (int u = 0; u < F::BTL; ++u) {
          const int b = q + u * NT;
          if (F::valid_last(b)) {
#pragma unroll
            for (int r = 0; r < F::RL; ++r) st(tc, F::out_index(q, u, r), v[u * F::RL + r]);
          }
        }
      }
    }
    if (nxt >= total) break;
    cur = nxt;
    tc = tn;
#pragma unroll
    for (int i = 0; i < F::VMAX; ++i) v[i] = nx[i];
  }
}

template <typename T, bool INV>
__global__ void __launch_bounds__(1024) k_ffty_gen(LaunchArgs a) {
  extern __shared__ unsigned char smem_raw[];
  cx<T>* buf = reinterpret_cast<cx<T>*>(smem_raw);
  const Member mb = launch_member(a, blockIdx.x);
  const MemberDesc d = load_desc(mb.desc);
  keep_y(d);
  if (skipped(d)) return;
  const IoPtrs& io = mb.io;
  const int lb = xcd_local_block(mb);
  const int mt = d.ymt, ny = d.ny, nt = d.fy.nt;
  const int tiles = (d.nxh + mt - 1) / mt;
  const int k = lb / tiles;
  const int m0 = (lb - k * tiles) * mt;
  const int c = threadIdx.x % mt;
  int q = threadIdx.x / mt;
  if (q >= nt) q = kBig;
  cx<T>* S = reinterpret_cast<cx<T>*>(io.spec) + (long long)k * d.plane;
  const int tot = ny * mt;
  for (int idx = threadIdx.x; idx < tot; idx += blockDim.x) {
    const int j = idx / mt, cc = idx - j * mt, m = m0 + cc;
    buf[idx] = (m < d.nxh) ? S[(long long)j * d.sbw + spec_col(d, m)] : cx<T>{0, 0};
  }
  __syncthreads();
  fft_lds<T, INV>(buf + c, mt, d.fy, reinterpret_cast<const cx<T>*>(d.twy), q);
  for (int idx = threadIdx.x; idx < tot; idx += blockDim.x) {
    const int j = idx / mt, cc = idx - j * mt, m = m0 + cc;
    if (m < d.nxh) S[(long long)j * d.sbw + spec_col(d, m)] = buf[idx];
  }
}

// ---------------------------------------------------------------------------
// x-direction inverse (complex-to-real) FFT of row pairs, written to
// MODE 0: io.p (storage type T), the pressure;
// MODE 1 (mixed, T = float): io.s1, the refinement's correction delta;
// MODE 2 (mixed, T = float): io.s2, the first-pass pressure p1;
// MODE 3: io.p, the Krylov solver's z = M^-1 r, with the workgroup's sums of
// dz r z (r: io.u) into io.stats and, for the flexible update (T = float, q
// given in io.v), of dz z q into io.w: the inner products as a kernel of their
// own read z again.
// Z[m] = X_a[m] + i X_b[m], Z[N-m] = conj X_a[m] + i conj X_b[m]; the
// imaginary parts of the self-conjugate bins (m = 0, m = N/2) are dropped.
// ---------------------------------------------------------------------------
template <typename T, class Idx>
__device__ __forceinline__ void pack_bins(cx<T>* buf, const Idx& idx, cx<T> xa, cx<T> xb, int N, int m) {
  const bool selfconj = (m == 0) || (2 * m == N);
  if (selfconj) {
    xa.y = 0;
    xb.y = 0;
  }
  buf[idx(m)] = cx<T>{xa.x - xb.y, xa.y + xb.x};
  if (!selfconj) buf[idx(N - m)] = cx<T>{xa.x + xb.y, xb.x - xa.y};
}

template <typename T, class Idx>
__device__ __forceinline__ void pack_rows(cx<T>* buf, const Idx& idx, const cx<T>* __restrict__ S, long long o0,
                                          long long o1, bool v0, bool v1, int N, int m, long long cm) {
  cx<T> xa = v0 ? S[o0 + cm] : cx<T>{0, 0};
  cx<T> xb = v1 ? S[o1 + cm] : cx<T>{0, 0};
  const bool selfconj = (m == 0) || (2 * m == N);
  if (selfconj) {
    xa.y = 0;
    xb.y = 0;
  }
  buf[idx(m)] = cx<T>{xa.x - xb.y, xa.y + xb.x};
  if (!selfconj) buf[idx(N - m)] = cx<T>{xa.x + xb.y, xb.x - xa.y};
}

template <typename T, int MODE>
__device__ __forceinline__ __attribute__((address_space(1))) T* xinv_dest(const IoPtrs& io) {
  if constexpr (MODE == 0 || MODE == 3) return gptr(reinterpret_cast<T*>(io.p));
  else if constexpr (MODE == 1) return gptr(reinterpret_cast<T*>(io.s1));
  else return gptr(reinterpret_cast<T*>(io.s2));
}

// MODE 3's inner products over values z of a row from point o on
template <typename T, int V>
__device__ __forceinline__ void dots_vec(const IoPtrs& io, long long o, const T* z, double dz, double& rz, double& zq) {
  constexpr int W = V % 2 == 0 ? 2 : 1;
  using dv = typename Vec<double, W>::type;
  const double* r = reinterpret_cast<const double*>(io.u) + o;
  const double* q = reinterpret_cast<const double*>(io.v) + o;
#pragma unroll
  for (int e = 0; e < V; e += W) {
    const dv x = ldv<W>(r + e);
#pragma unroll
    for (int h = 0; h < W; ++h) rz += dz * x[h] * (double)z[e + h];
    if (sizeof(T) == 4 && io.v) {
      const dv y = ldv<W>(q + e);
#pragma unroll
      for (int h = 0; h < W; ++h) zq += dz * (double)z[e + h] * y[h];
    }
  }
}
template <typename T>
__device__ __forceinline__ void dots_commit(const IoPtrs& io, double rz, double zq, unsigned char* smem) {
  const double s = group_sum(rz, reinterpret_cast<double*>(smem));
  if (threadIdx.x == 0) io.stats[blockIdx.x] = s;
  if (sizeof(T) == 4 && io.v) {
    const double t = group_sum(zq, reinterpret_cast<double*>(smem));
    if (threadIdx.x == 0) reinterpret_cast<double*>(io.w)[blockIdx.x] = t;
  }
}

template <typename T, int MODE>
__device__ __forceinline__ void store_rows(const MemberDesc& d, const IoPtrs& io, long long r0, long long r1, bool v0,
                                           bool v1, int i, cx<T> z) {
  const int N = d.nx;
  auto p = xinv_dest<T, MODE>(io);
  if (v0) p[r0 * N + i] = z.x;
  if (v1) p[r1 * N + i] = z.y;
}

template <typename T, int MODE, int N>
__global__ void __launch_bounds__(512) k_xinv_ct(LaunchArgs a) {
  constexpr int NT = ct_threads(N, sizeof(T));
  using F = CtFft<T, N, NT, true>;
  extern __shared__ unsigned char smem_raw[];
  const Member mb = launch_member(a, blockIdx.x);
  const MemberDesc d = load_desc(mb.desc);
  keep_x(d);
  if (skipped(d)) return;
  const IoPtrs& io = mb.io;
  const int lb = blockIdx.x - mb.start;
  const int ipw = blockDim.x / NT;
  const int inst = threadIdx.x / NT;
  const int q = threadIdx.x - inst * NT;
  cx<T>* lds = reinterpret_cast<cx<T>*>(smem_raw) + inst * xlds_len(N, 2 * sizeof(T));
  const long long pair = (long long)lb * ipw + inst;
  constexpr bool part = true;
#include "xinv_pair.h"
  if constexpr (MODE == 3) dots_commit<T>(io, rz, zq, smem_raw);
}

template <typename T, int MODE>
__global__ void __launch_bounds__(1024) k_xinv_gen(LaunchArgs a) {
  extern __shared__ unsigned char smem_raw[];
  cx<T>* smem = reinterpret_cast<cx<T>*>(smem_raw);
  const Member mb = launch_member(a, blockIdx.x);
  const MemberDesc d = load_desc(mb.desc);
  keep_x(d);
  if (skipped(d)) return;
  const IoPtrs& io = mb.io;
  const int lb = blockIdx.x - mb.start;
  const int N = d.nx, nt = d.fx.nt;
  const int ipw = blockDim.x / nt;
  const int inst = threadIdx.x / nt;
  const bool active = inst < ipw;
  const int q = active ? (int)(threadIdx.x - inst * nt) : kBig;
  cx<T>* buf = smem + (active ? inst : 0) * N;
  const long long pair = (long long)lb * ipw + inst;
  const long long r0 = 2 * pair, r1 = 2 * pair + 1;
  const bool v0 = active && r0 < d.nrow, v1 = active && r1 < d.nrow;
  const cx<T>* S = reinterpret_cast<const cx<T>*>(io.spec);
  auto ident = [](int i) { return i; };
  const long long so0 = spec_row(d, v0 ? r0 : 0), so1 = spec_row(d, v1 ? r1 : 0);
  if (active)
    for (int m = q; m < d.nxh; m += nt) pack_rows<T>(buf, ident, S, so0, so1, v0, v1, N, m, spec_col(d, m));
  __syncthreads();
  fft_lds<T, true>(buf, 1, d.fx, reinterpret_cast<const cx<T>*>(d.twx), q);
  if (active)
    for (int i = q; i < N; i += nt) store_rows<T, MODE>(d, io, r0, r1, v0, v1, i, buf[i]);
  if constexpr (MODE == 3) {
    const double dz0 = ldg(d.dz + row_level(d, v0 ? (int)r0 : 0)), dz1 = ldg(d.dz + row_level(d, v1 ? (int)r1 : 0));
    double rz = 0.0, zq = 0.0;
    if (active)
      for (int i = q; i < N; i += nt) {
        const cx<T> z = buf[i];
        if (v0) dots_vec<T, 1>(io, r0 * N + i, &z.x, dz0, rz, zq);
        if (v1) dots_vec<T, 1>(io, r1 * N + i, &z.y, dz1, rz, zq);
      }
    dots_commit<T>(io, rz, zq, smem_raw);
  }
}

}  // namespace monc
