// Kernels of the variable-density projection: preconditioned conjugate
// gradients for D_rho(G p) = D_rho(u*) with a density rho(x, y, z), the
// non-separable problem on which the FFT solve is only an approximate
// inverse (the paper's Sec. 4 sets the FFT solver beside a Krylov solver;
// Sec. 5 proposes a preconditioner built from the problem's structure and a
// mixed-precision solver with a double-precision restart).
//
// Preconditioner: M^-1 = Lbar^-1, Lbar the separable operator with the
// plan's rho0(z), solved spectrally. Both D_rho G and Lbar are
// -D (face density) G, so their energies p^T A p differ only in the face
// density that weighs each face's |G p|^2: the preconditioned operator's
// condition is at most max(rho_face / rho0) / min(rho_face / rho0) on every
// grid (12 iterations at +-30 % density to a relative residual of 1e-10,
// from 16 x 32 to 256^2 points a level). A symmetric density scaling
// S Lbar^-1 S, S = diag(sqrt(rho0 / rho)), saved a few iterations on square
// domains but loses that bound: G(S p) carries p G(S), which dominates for
// the lowest modes of a long domain (16 x 1024 x 6, dy = 57 m: no
// convergence in 200 iterations), so it is not used.
//
// All vectors are FP64 (nz, ny, nx) fields; the preconditioned residual z is
// in the plan's storage type (ZT). Face densities come from rho on the fly:
//   rx = (rho_i + rho_{i+1})/2, ry = (rho_j + rho_{j+1})/2 (periodic),
//   rz_k = za_k rho_k + zb_k rho_{k+1}, za_k = dz_{k+1}/(dz_k + dz_{k+1}),
//   zb_k = dz_k/(dz_k + dz_{k+1}) (0 on the lid).
// A workgroup of kVarBlock threads takes a 2-D tile of a level, min(nx, 256)
// wide, a few points per thread at stride kVarBlock in the tile, coalesced
// along rows. The stencil kernels (divergence, operator; kVarStPts points a
// thread) walk them up a group of kVarLevels levels (the divergence's is
// blockIdx.y, the operator's follows var_operator_block), keeping the column's values of the levels below and above in
// registers, so only the x and y neighbours come through the caches; the
// pointwise kernels (kVarPts points a thread) take one level per workgroup (more, shorter
// workgroups stream faster). Two points and two levels a stencil thread leave
// enough workgroups to even out the last wave of them: the operator 68 us with
// four and four, 60 us with two and two at 256^2 x 128, 39.5 and 29.5 us at 288 x 216
// x 48. For even nx the operator works on pairs of adjacent x
// points with 16-byte loads (k_var_apply2).
// Inner products are weighted by dz_k (the weight that makes D_rho G
// self-adjoint); each workgroup writes its partial sum and a one-workgroup
// kernel adds the partials in a fixed order, so results are deterministic.
// Loads are unconditional (a point past the level reads point 0, a missing
// level reads its own) and the results selected, so that all loads of a
// thread's points issue together.
#include <hip/hip_runtime.h>

#include "krylov.h"

namespace monc {

namespace {

__device__ __forceinline__ double wave_sum(double x) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
  return x;
}

// sum over a workgroup of NT threads, valid in thread 0
template <int NT>
__device__ __forceinline__ double block_sum(double x) {
  __shared__ double part[NT / 64];
  x = wave_sum(x);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = x;
  __syncthreads();
  double s = 0.0;
  if (threadIdx.x == 0)
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) s += part[w];
  return s;
}

// One thread's points: NPTS points of a level at stride kVarBlock (horizontal
// offsets inside a level and their x and y neighbours, periodic), revisited on
// each level of the workgroup's group of kVarLevels levels.
template <int NPTS>
struct Col {
  int h[NPTS], hw[NPTS], he[NPTS], hs[NPTS], hn[NPTS];
  bool live[NPTS];
};

// The workgroup's (point chunk, level group)
struct Blk {
  int x, y;
};
__device__ __forceinline__ Blk var_block() { return Blk{(int)blockIdx.x, (int)blockIdx.y}; }

// The operator's blocks (a 1-D grid) in an order that lets the rows and levels a
// stencil reads again meet in the L2 that holds them: of every 64 blocks an XCD
// (block mod 8) takes 8 neighbouring ones, and the blocks walk the level groups
// of a band of kVarBand tiles (about 32 K points a level) before the next band.
// Against launch order: 535 -> 475 us at 1024^2 x 64, 29 -> 26 at 288 x 216 x 48,
// equal at 256^2 x 128 (64; an eighth of the grid per XCD 75). The divergence,
// run once, is 0-10 % slower that way and keeps launch order.
__device__ __forceinline__ Blk var_operator_block(const VarGrid& g) {
  const int tiles = (int)var_blocks_per_level(g.nx, g.ny, kVarStPts), groups = var_level_groups(g.nz);
  const int b = blockIdx.x;
  const int id = b < (tiles * groups & ~63) ? (b & ~63) | (b & 7) << 3 | (b >> 3 & 7) : b;
  const int band = id / (kVarBand * groups), rem = id - band * kVarBand * groups;
  const int nb = min(kVarBand, tiles - band * kVarBand);
  const int grp = rem / nb;
  return Blk{band * kVarBand + rem - grp * nb, grp};
}

template <int NPTS>
__device__ __forceinline__ Col<NPTS> columns(const VarGrid& g, const Blk& bk) {
  Col<NPTS> c;
  const int tw = var_tile_w(g.nx), th = var_tile_h(g.nx, NPTS), ntx = var_tiles_x(g.nx);
  const int tile_y = bk.x / ntx, tile_x = bk.x - tile_y * ntx;
#pragma unroll
  for (int t = 0; t < NPTS; ++t) {
    const int sl = t * kVarBlock + threadIdx.x;          // slot in the tile
    const int rr = sl / tw, ic = tile_x * tw + (sl - rr * tw), jr = tile_y * th + rr;
    c.live[t] = rr < th && ic < g.nx && jr < g.ny;
    // outside the grid: point 0, nothing stored
    const int j = c.live[t] ? jr : 0, i = c.live[t] ? ic : 0;
    const int row = j * g.nx;
    c.h[t] = row + i;
    c.hw[t] = row + (i == 0 ? g.nx - 1 : i - 1);
    c.he[t] = row + (i == g.nx - 1 ? 0 : i + 1);
    c.hs[t] = (j == 0 ? g.ny - 1 : j - 1) * g.nx + i;
    c.hn[t] = (j == g.ny - 1 ? 0 : j + 1) * g.nx + i;
  }
  return c;
}

// levels [level_begin, level_end) of a workgroup whose group holds LV levels
template <int LV>
__device__ __forceinline__ int level_begin(const Blk& bk) { return bk.y * LV; }
template <int LV>
__device__ __forceinline__ int level_end(const VarGrid& g, const Blk& bk) { return min(g.nz, (bk.y + 1) * LV); }

__device__ __forceinline__ long long part_index() { return (long long)blockIdx.y * gridDim.x + blockIdx.x; }

__device__ __forceinline__ bool var_done(const double* scal) { return scal[kVarDone] != 0.0; }

// vertical metrics of level k
struct Lev {
  bool top, bot;      // a face above / below inside the domain
  double dz, rdz, ct, cb, za, zb, zam, zbm;
};

__device__ __forceinline__ Lev level(const VarGrid& g, int k) {
  Lev L;
  L.top = k < g.nz - 1;
  L.bot = k > 0;
  L.dz = g.dz[k];
  L.rdz = g.rdz[k];
  L.ct = L.top ? g.rdzc[k] * L.rdz : 0.0;
  L.cb = L.bot ? g.rdzc[k - 1] * L.rdz : 0.0;
  L.za = g.za[k];       // 0 on the lid
  L.zb = g.zb[k];
  L.zam = L.bot ? g.za[k - 1] : 0.0;
  L.zbm = L.bot ? g.zb[k - 1] : 0.0;
  return L;
}

}  // namespace

// r = D_rho(u*) and p = 0; partial sums of dz r^2. Each thread walks up its group of
// levels keeping rho and w of the level below in registers.
__global__ void __launch_bounds__(kVarBlock) k_var_div(VarGrid g, const double* __restrict__ u,
                                                     const double* __restrict__ v, const double* __restrict__ w,
                                                     double* __restrict__ r, double* __restrict__ p,
                                                     double* __restrict__ part) {
  const Blk bk = var_block();
  const Col<kVarStPts> c = columns<kVarStPts>(g, bk);
  const long long nh = (long long)g.nx * g.ny;
  const int k0 = level_begin<kVarLevels>(bk), k1 = level_end<kVarLevels>(g, bk);
  double rdn[kVarStPts], wdn[kVarStPts], rc[kVarStPts];
  {
    const long long b0 = (long long)k0 * nh, bd = k0 > 0 ? b0 - nh : b0;
#pragma unroll
    for (int t = 0; t < kVarStPts; ++t) {
      rdn[t] = g.rho[bd + c.h[t]];
      wdn[t] = w[bd + c.h[t]];
      rc[t] = g.rho[b0 + c.h[t]];
    }
  }
  double acc = 0.0;
  for (int k = k0; k < k1; ++k) {
    const Lev L = level(g, k);
    const long long b = (long long)k * nh, bu = L.top ? b + nh : b;
#pragma unroll
    for (int t = 0; t < kVarStPts; ++t) {
      const double ru = g.rho[bu + c.h[t]], wc = w[b + c.h[t]];
      const double rxe = 0.5 * (rc[t] + g.rho[b + c.he[t]]), rxw = 0.5 * (g.rho[b + c.hw[t]] + rc[t]);
      const double ryn = 0.5 * (rc[t] + g.rho[b + c.hn[t]]), rys = 0.5 * (g.rho[b + c.hs[t]] + rc[t]);
      // top and bottom face fluxes, selected away on the lids (whatever w holds there)
      const double ft = L.top ? (L.za * rc[t] + L.zb * ru) * wc : 0.0;
      const double fb = L.bot ? (L.zam * rdn[t] + L.zbm * rc[t]) * wdn[t] : 0.0;
      const double div = (rxe * u[b + c.h[t]] - rxw * u[b + c.hw[t]]) * g.rdx +
                         (ryn * v[b + c.h[t]] - rys * v[b + c.hs[t]]) * g.rdy + (ft - fb) * L.rdz;
      if (c.live[t]) {
        r[b + c.h[t]] = div;
        p[b + c.h[t]] = 0.0;
        acc += L.dz * div * div;
      }
      rdn[t] = rc[t];
      rc[t] = ru;
      wdn[t] = wc;
    }
  }
  const double s = block_sum<kVarBlock>(acc);
  if (threadIdx.x == 0) part[part_index()] = s;
}

// q = D_rho(G d), partial sums of dz d q; d and rho of the levels below and
// above stay in registers as the thread walks up
__global__ void __launch_bounds__(kVarBlock) k_var_apply(VarGrid g, const double* __restrict__ scal,
                                                       const double* __restrict__ d, double* __restrict__ q,
                                                       double* __restrict__ part) {
  if (var_done(scal)) return;
  const Blk bk = var_operator_block(g);
  const Col<kVarStPts> c = columns<kVarStPts>(g, bk);
  const long long nh = (long long)g.nx * g.ny;
  const int k0 = level_begin<kVarLevels>(bk), k1 = level_end<kVarLevels>(g, bk);
  double ddn[kVarStPts], rdn[kVarStPts], dc[kVarStPts], rc[kVarStPts];
  {
    const long long b0 = (long long)k0 * nh, bd = k0 > 0 ? b0 - nh : b0;
#pragma unroll
    for (int t = 0; t < kVarStPts; ++t) {
      ddn[t] = d[bd + c.h[t]];
      rdn[t] = g.rho[bd + c.h[t]];
      dc[t] = d[b0 + c.h[t]];
      rc[t] = g.rho[b0 + c.h[t]];
    }
  }
  double acc = 0.0;
  for (int k = k0; k < k1; ++k) {
    const Lev L = level(g, k);
    const long long b = (long long)k * nh, bu = L.top ? b + nh : b;
#pragma unroll
    for (int t = 0; t < kVarStPts; ++t) {
      const double du = d[bu + c.h[t]], ru = g.rho[bu + c.h[t]];
      const double rxe = 0.5 * (rc[t] + g.rho[b + c.he[t]]), rxw = 0.5 * (g.rho[b + c.hw[t]] + rc[t]);
      const double ryn = 0.5 * (rc[t] + g.rho[b + c.hn[t]]), rys = 0.5 * (g.rho[b + c.hs[t]] + rc[t]);
      const double rzt = L.za * rc[t] + L.zb * ru;          // 0 on the lid
      const double rzb = L.zam * rdn[t] + L.zbm * rc[t];    // 0 at k = 0
      const double a = (rxe * (d[b + c.he[t]] - dc[t]) - rxw * (dc[t] - d[b + c.hw[t]])) * g.rdx2 +
                       (ryn * (d[b + c.hn[t]] - dc[t]) - rys * (dc[t] - d[b + c.hs[t]])) * g.rdy2 +
                       rzt * (du - dc[t]) * L.ct - rzb * (dc[t] - ddn[t]) * L.cb;
      if (c.live[t]) {
        q[b + c.h[t]] = a;
        acc += L.dz * dc[t] * a;
      }
      ddn[t] = dc[t];
      dc[t] = du;
      rdn[t] = rc[t];
      rc[t] = ru;
    }
  }
  const double s = block_sum<kVarBlock>(acc);
  if (threadIdx.x == 0) part[part_index()] = s;
}

// The operator for even nx on pairs of adjacent x points with 16-byte
// loads: a workgroup's tile (var_tile_h rows of var_tile_w / 2 pairs) holds
// half as many pairs as points, at stride kVarBlock per thread; six 16-byte
// loads a pair and level instead of 16 8-byte ones for two points.
// The x neighbours come from the neighbouring lanes (a DPP shift by one lane of
// the wave) wherever those hold the pair beside, else (the ends of a wave and of
// a row of the tile) from memory: 64.7 -> 61.9 us at 256^2 x 128, 26.2 -> 24.7 at
// 288 x 216 x 48, where the 8-byte loads for them were two in eight.
template <int CTRL>
__device__ __forceinline__ double wave_shift(double v) {  // 0x138: from the lane below, 0x130: above
  const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xF, 0xF, true);
  return __hiloint2double(hi, lo);
}
typedef double d2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ d2v ld2(const double* p) { return *reinterpret_cast<const d2v*>(p); }

__global__ void __launch_bounds__(kVarBlock) k_var_apply2(VarGrid g, const double* __restrict__ scal,
                                                        const double* __restrict__ d, double* __restrict__ q,
                                                        double* __restrict__ part) {
  if (var_done(scal)) return;
  constexpr int NP = kVarStPts / 2;   // pairs per thread
  const Blk bk = var_operator_block(g);
  const int hx = g.nx / 2;
  const int txp = var_tile_w(g.nx) / 2, tyr = var_tile_h(g.nx, kVarStPts), ntx = var_tiles_x(g.nx);
  const int tile_y = bk.x / ntx, tile_x = bk.x - tile_y * ntx;
  int h[NP], hw[NP], he[NP], hs[NP], hn[NP];
  bool live[NP], loadw[NP], loade[NP];
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int t = 0; t < NP; ++t) {
    const int sl = t * kVarBlock + threadIdx.x;          // slot in the tile
    const int rr = sl / txp, pt = sl - rr * txp, pc = tile_x * txp + pt, jr = tile_y * tyr + rr;
    loadw[t] = lane == 0 || pt == 0;
    loade[t] = lane == 63 || pt == txp - 1 || pc == hx - 1;
    live[t] = rr < tyr && pc < hx && jr < g.ny;
    const int j = live[t] ? jr : 0, i0 = live[t] ? 2 * pc : 0;   // outside the grid: pair 0, nothing stored
    const int row = j * g.nx;
    h[t] = row + i0;
    hw[t] = row + (i0 == 0 ? g.nx - 1 : i0 - 1);
    he[t] = row + (i0 + 2 == g.nx ? 0 : i0 + 2);
    hs[t] = (j == 0 ? g.ny - 1 : j - 1) * g.nx + i0;
    hn[t] = (j == g.ny - 1 ? 0 : j + 1) * g.nx + i0;
  }
  const long long nh = (long long)g.nx * g.ny;
  const int k0 = level_begin<kVarLevels>(bk), k1 = level_end<kVarLevels>(g, bk);
  d2v ddn[NP], rdn[NP], dc[NP], rc[NP];
  {
    const long long b0 = (long long)k0 * nh, bd = k0 > 0 ? b0 - nh : b0;
#pragma unroll
    for (int t = 0; t < NP; ++t) {
      ddn[t] = ld2(d + bd + h[t]);
      rdn[t] = ld2(g.rho + bd + h[t]);
      dc[t] = ld2(d + b0 + h[t]);
      rc[t] = ld2(g.rho + b0 + h[t]);
    }
  }
  double acc = 0.0;
  for (int k = k0; k < k1; ++k) {
    const Lev L = level(g, k);
    const long long b = (long long)k * nh, bu = L.top ? b + nh : b;
#pragma unroll
    for (int t = 0; t < NP; ++t) {
      const d2v du = ld2(d + bu + h[t]), ru = ld2(g.rho + bu + h[t]);
      const d2v dn = ld2(d + b + hn[t]), ds = ld2(d + b + hs[t]);
      const d2v rn = ld2(g.rho + b + hn[t]), rs = ld2(g.rho + b + hs[t]);
      double dw = wave_shift<0x138>(dc[t][1]), rw = wave_shift<0x138>(rc[t][1]);
      double de = wave_shift<0x130>(dc[t][0]), re = wave_shift<0x130>(rc[t][0]);
      if (loadw[t]) {
        dw = d[b + hw[t]];
        rw = g.rho[b + hw[t]];
      }
      if (loade[t]) {
        de = d[b + he[t]];
        re = g.rho[b + he[t]];
      }
      d2v a;
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const double dce = dc[t][e], rce = rc[t][e];
        const double dE = e ? de : dc[t][1], dW = e ? dc[t][0] : dw;
        const double rE = e ? re : rc[t][1], rW = e ? rc[t][0] : rw;
        const double rxe = 0.5 * (rce + rE), rxw = 0.5 * (rW + rce);
        const double ryn = 0.5 * (rce + rn[e]), rys = 0.5 * (rs[e] + rce);
        const double rzt = L.za * rce + L.zb * ru[e];          // 0 on the lid
        const double rzb = L.zam * rdn[t][e] + L.zbm * rce;    // 0 at k = 0
        a[e] = (rxe * (dE - dce) - rxw * (dce - dW)) * g.rdx2 + (ryn * (dn[e] - dce) - rys * (dce - ds[e])) * g.rdy2 +
               rzt * (du[e] - dce) * L.ct - rzb * (dce - ddn[t][e]) * L.cb;
      }
      if (live[t]) {
        *reinterpret_cast<d2v*>(q + b + h[t]) = a;
        acc += L.dz * (dc[t][0] * a[0] + dc[t][1] * a[1]);
      }
      ddn[t] = dc[t];
      dc[t] = du;
      rdn[t] = rc[t];
      rc[t] = ru;
    }
  }
  const double sm = block_sum<kVarBlock>(acc);
  if (threadIdx.x == 0) part[part_index()] = sm;
}

// alpha of iteration it
__device__ __forceinline__ double var_alpha(const double* scal, int it) {
  const double rz = scal[var_slot(it, kVarRZ)], dq = scal[var_slot(it, kVarDQ)];
  return dq != 0.0 ? rz / dq : 0.0;
}

// The solution takes the step the residual took (p += alpha_{it-1} d_{it-1}),
// then d = z + beta d (d = z at it = 0, and p unchanged), in one pass over d;
// flexible (Polak-Ribiere):
// beta = <z_it, r_it - r_{it-1}> / rz_{it-1} = -alpha_{it-1} <z_it, q_{it-1}> / rz_{it-1};
// otherwise (Fletcher-Reeves) beta = rz_it / rz_{it-1}
template <typename ZT, bool FLEX>
__global__ void __launch_bounds__(kVarBlock) k_var_dir(VarGrid g, const double* __restrict__ scal, int it,
                                                     const ZT* __restrict__ z, double* __restrict__ d,
                                                     double* __restrict__ p) {
  if (var_done(scal)) return;
  double beta = 0.0, alpha = 0.0;
  if (it > 0) {
    const double rzp = scal[var_slot(it - 1, kVarRZ)];
    alpha = var_alpha(scal, it - 1);
    if constexpr (FLEX) beta = rzp != 0.0 ? -alpha * scal[var_slot(it, kVarZQ)] / rzp : 0.0;
    else beta = rzp != 0.0 ? scal[var_slot(it, kVarRZ)] / rzp : 0.0;
  }
  const Blk bk = var_block();
  const Col<kVarPts> c = columns<kVarPts>(g, bk);
  const long long nh = (long long)g.nx * g.ny;
  for (int k = level_begin<1>(bk), k1 = level_end<1>(g, bk); k < k1; ++k) {
    const long long b = (long long)k * nh;
#pragma unroll
    for (int t = 0; t < kVarPts; ++t) {
      const long long o = b + c.h[t];
      const double zc = (double)z[o];
      if (it > 0) {  // d is not yet defined at it = 0
        const double dc = d[o], pn = p[o] + alpha * dc;
        if (c.live[t]) {
          p[o] = pn;
          d[o] = zc + beta * dc;
        }
      } else if (c.live[t]) {
        d[o] = zc;
      }
    }
  }
}

// The last iteration's step of the solution (p += alpha_{it-1} d_{it-1}: the
// direction update that would take it is not run once the solve is done), and
// partial sums of dz p (the gauge)
__global__ void __launch_bounds__(kVarBlock) k_var_wsum(VarGrid g, const double* __restrict__ scal, int it,
                                                      const double* __restrict__ d, double* __restrict__ p,
                                                      double* __restrict__ part) {
  const double alpha = var_alpha(scal, it - 1);
  const Blk bk = var_block();
  const Col<kVarPts> c = columns<kVarPts>(g, bk);
  const long long nh = (long long)g.nx * g.ny;
  double acc = 0.0;
  for (int k = level_begin<1>(bk), k1 = level_end<1>(g, bk); k < k1; ++k) {
    const long long b = (long long)k * nh;
    const double dz = g.dz[k];
#pragma unroll
    for (int t = 0; t < kVarPts; ++t) {
      const long long o = b + c.h[t];
      const double pn = p[o] + alpha * d[o];
      if (c.live[t]) {
        p[o] = pn;
        acc += dz * pn;
      }
    }
  }
  const double s = block_sum<kVarBlock>(acc);
  if (threadIdx.x == 0) part[part_index()] = s;
}

// p -= scal[slot] * rw: with rw = 1 / (nx ny sum dz) the dz-weighted mean
__global__ void __launch_bounds__(kVarBlock) k_var_shift(VarGrid g, const double* __restrict__ scal, int slot,
                                                       double rw, double* __restrict__ p) {
  const double m = scal[slot] * rw;
  const Blk bk = var_block();
  const Col<kVarPts> c = columns<kVarPts>(g, bk);
  const long long nh = (long long)g.nx * g.ny;
  for (int k = level_begin<1>(bk), k1 = level_end<1>(g, bk); k < k1; ++k) {
    const long long b = (long long)k * nh;
#pragma unroll
    for (int t = 0; t < kVarPts; ++t) {
      const double pn = p[b + c.h[t]] - m;
      if (c.live[t]) p[b + c.h[t]] = pn;
    }
  }
}

// sum of part[0 .. n) in a fixed order (one workgroup of kVarFinishBlock threads)
__device__ __forceinline__ double finish_sum(const double* __restrict__ part, long long n) {
  double acc = 0.0;
  for (long long i = threadIdx.x; i < n; i += 4 * kVarFinishBlock) {
    double a[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const long long ie = i + (long long)e * kVarFinishBlock;
      a[e] = ie < n ? part[ie] : 0.0;
    }
    acc += (a[0] + a[1]) + (a[2] + a[3]);
  }
  return block_sum<kVarFinishBlock>(acc);
}

__global__ void __launch_bounds__(kVarFinishBlock) k_var_finish(const double* __restrict__ part0,
                                                              const double* __restrict__ part1, long long n,
                                                              double* __restrict__ scal, int slot0, int slot1,
                                                              int gated) {
  if (gated && var_done(scal)) return;
  const double s0 = finish_sum(part0, n);
  if (threadIdx.x == 0) scal[slot0] = s0;
  if (part1) {
    __syncthreads();  // block_sum's LDS is reused
    const double s1 = finish_sum(part1, n);
    if (threadIdx.x == 0) scal[slot1] = s1;
  }
}

__global__ void __launch_bounds__(kVarFinishBlock) k_var_finish_rr(const double* __restrict__ part, long long n,
                                                                 double* __restrict__ scal, int it, double tol2) {
  if (var_done(scal)) return;
  const double rr = finish_sum(part, n);
  if (threadIdx.x == 0) {
    scal[var_slot(it, kVarRR)] = rr;
    scal[kVarLast] = (double)it;
    scal[kVarLastRR] = rr;
    if (!isfinite(rr)) scal[kVarDone] = 2.0;
    else if (rr <= tol2 * scal[var_slot(0, kVarRR)]) scal[kVarDone] = 1.0;
  }
}

__global__ void k_var_zero(double* __restrict__ x, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) x[i] = 0.0;
}

// ---------------------------------------------------------------------------
// host-side launchers
// ---------------------------------------------------------------------------
// the stencil kernels' grid (level groups of kVarLevels) and the pointwise
// kernels' grid (one level per workgroup)
static dim3 var_grid_stencil(const VarGrid& g) {
  return dim3((unsigned)var_blocks_per_level(g.nx, g.ny, kVarStPts), (unsigned)var_level_groups(g.nz));
}
static dim3 var_grid_operator(const VarGrid& g) { return dim3((unsigned)var_stencil_parts(g.nx, g.ny, g.nz)); }
static dim3 var_grid(const VarGrid& g) { return dim3((unsigned)var_blocks_per_level(g.nx, g.ny, kVarPts), (unsigned)g.nz); }

void launch_var_div(const VarGrid& g, const double* u, const double* v, const double* w, double* r, double* p,
                    double* part, void* stream) {
  hipLaunchKernelGGL(k_var_div, var_grid_stencil(g), dim3(kVarBlock), 0, (hipStream_t)stream, g, u, v, w, r, p, part);
}

void launch_var_apply(const VarGrid& g, const double* scal, const double* d, double* q, double* part, void* stream) {
  if (g.nx % 2 == 0)
    hipLaunchKernelGGL(k_var_apply2, var_grid_operator(g), dim3(kVarBlock), 0, (hipStream_t)stream, g, scal, d, q,
                       part);
  else
    hipLaunchKernelGGL(k_var_apply, var_grid_operator(g), dim3(kVarBlock), 0, (hipStream_t)stream, g, scal, d, q, part);
}

// the FP64 preconditioner takes the Fletcher-Reeves update, the FP32 one the
// flexible update
void launch_var_dir(const VarGrid& g, const double* scal, int it, const void* z, bool z64, double* d, double* p,
                    void* stream) {
  if (z64)
    hipLaunchKernelGGL((k_var_dir<double, false>), var_grid(g), dim3(kVarBlock), 0, (hipStream_t)stream, g, scal,
                       it, static_cast<const double*>(z), d, p);
  else
    hipLaunchKernelGGL((k_var_dir<float, true>), var_grid(g), dim3(kVarBlock), 0, (hipStream_t)stream, g, scal, it,
                       static_cast<const float*>(z), d, p);
}

void launch_var_wsum(const VarGrid& g, const double* scal, int it, const double* d, double* p, double* part,
                     void* stream) {
  hipLaunchKernelGGL(k_var_wsum, var_grid(g), dim3(kVarBlock), 0, (hipStream_t)stream, g, scal, it, d, p, part);
}

void launch_var_shift(const VarGrid& g, const double* scal, int slot, double rw, double* p, void* stream) {
  hipLaunchKernelGGL(k_var_shift, var_grid(g), dim3(kVarBlock), 0, (hipStream_t)stream, g, scal, slot, rw, p);
}

void launch_var_finish(const double* part0, const double* part1, long long n, double* scal, int slot0, int slot1,
                       bool gated, void* stream) {
  hipLaunchKernelGGL(k_var_finish, dim3(1), dim3(kVarFinishBlock), 0, (hipStream_t)stream, part0, part1, n, scal,
                     slot0, slot1, gated ? 1 : 0);
}

void launch_var_finish_rr(const double* part, long long n, double* scal, int it, double tol2, void* stream) {
  hipLaunchKernelGGL(k_var_finish_rr, dim3(1), dim3(kVarFinishBlock), 0, (hipStream_t)stream, part, n, scal, it,
                     tol2);
}

void launch_var_zero(double* x, int n, void* stream) {
  if (n > 0) hipLaunchKernelGGL(k_var_zero, dim3((n + 255) / 256), dim3(256), 0, (hipStream_t)stream, x, n);
}

}  // namespace monc
