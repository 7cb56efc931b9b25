// Tridiagonal kernels of the pressure projection for gfx950: the vertical
// solve of every horizontal wavenumber (m, n), in FP64 whatever the storage
// type.
#include <hip/hip_runtime.h>

#include "device_common.h"
#include "kernels.h"
#include "launch.h"

namespace monc {

// ---------------------------------------------------------------------------
// FP64 tridiagonal solve per wavenumber column (partitioned elimination).
//
// Column (m, n): rows a_k P_{k-1} + (-a_k - c_k - rho0_k lam) P_k + c_k P_{k+1}
// = B_k, lam = lamx[m] + lamy[n], solved in FP64 whatever the storage type.
// P lanes of one wave share a column; lane q owns rows q*S .. q*S+S-1 (rows
// >= nz read P_k - P_{k-1} = 0: decoupled from the system by the lid).
//  1. each lane eliminates inside its chunk so that every row depends only on
//     the chunk's first unknown F_q and last unknown L_q;
//  2. the interface rows of L_q are substituted into those of F_q, leaving a
//     tridiagonal system in F_0..F_{P-1}, one row per lane;
//  3. that system is solved by parallel cyclic reduction over the P lanes
//     (wave shuffles, log2 P steps);
//  4. L_q follows from F_q, F_{q+1}; every lane substitutes back.
// The result is scaled by 1/(nx ny) (the inverse-FFT factor). The singular
// (0,0) column: its right-hand side loses its dz-weighted mean, the top
// unknown is pinned to 0, and the solution is shifted to the gauge
// sum_k dz_k P_k = 0.
// ---------------------------------------------------------------------------
struct Row5 {
  double a, b, c, x, y;  // sub, diag, sup, rhs (re, im)
};

__device__ __forceinline__ double shfl_d(double v, int src) { return __shfl(v, src); }

// 1/x in FP64: the hardware reciprocal refined by one Newton step (error
// about one ulp; the solve does not need the correctly rounded quotient)
__device__ __forceinline__ double rcp64(double x) {
  double r = __builtin_amdgcn_rcp(x);
  const double e = fma(-x, r, 1.0);
  r = fma(r, e, r);
  return r;
}

// Value of lane q - H (FROM_BELOW) or q + H of the same 16-lane row, moved
// with DPP (row_shr / row_shl) on the vector ALU instead of the LDS
// crossbar; a lane whose source lies outside its row reads 0. With P = 16
// lanes per column, a row is a column; every use multiplies such a value by
// a coupling that is already zero at the column's ends.
template <int H, bool FROM_BELOW>
__device__ __forceinline__ double dpp_shift(double v) {
  constexpr int ctrl = FROM_BELOW ? 0x110 + H : 0x100 + H;
  const int lo = __double2loint(v), hi = __double2hiint(v);
  const int l2 = __builtin_amdgcn_mov_dpp(lo, ctrl, 0xF, 0xF, true);
  const int h2 = __builtin_amdgcn_mov_dpp(hi, ctrl, 0xF, 0xF, true);
  return __hiloint2double(h2, l2);
}

// One cyclic-reduction step at distance H on unit-diagonal rows (a, c, x, y).
template <int H>
__device__ __forceinline__ void pcr_step16(double& a, double& c, double& x, double& y) {
  const double la = dpp_shift<H, true>(a), lc = dpp_shift<H, true>(c);
  const double lx = dpp_shift<H, true>(x), ly = dpp_shift<H, true>(y);
  const double ha = dpp_shift<H, false>(a), hc = dpp_shift<H, false>(c);
  const double hx = dpp_shift<H, false>(x), hy = dpp_shift<H, false>(y);
  const double ib = rcp64(1.0 - lc * a - ha * c);
  const double na = -la * a, nc = -hc * c;
  const double nx = x - lx * a - hx * c, ny = y - ly * a - hy * c;
  a = na * ib;
  c = nc * ib;
  x = nx * ib;
  y = ny * ib;
}

// sum over the P lanes of a column (aligned power-of-two lane group)
__device__ __forceinline__ double2 column_sum(double2 v, int P) {
  for (int o = P / 2; o > 0; o /= 2) {
    v.x += __shfl_xor(v.x, o);
    v.y += __shfl_xor(v.y, o);
  }
  return v;
}

// One tile of columns; SING: the tile holds the (0,0) column (tile 0), so
// the mean removal, the pinned top row and the gauge are compiled in.
template <typename TS, int S, bool SING, bool PAIRS>
__device__ __forceinline__ void tri_tile(const MemberDesc& d, const IoPtrs& io, int lb, double2* stage) {
  const int P = d.triP, CW = d.tricw, nz = d.nz, nxh = d.nxh, nxp = d.nxp;
  const int lp = __builtin_ctz(P), lcw = __builtin_ctz(CW);  // both powers of two
  constexpr bool F32 = sizeof(TS) == 4;      // FP32 storage: rows staged as FP32
  constexpr int SP = tri_lane_slots(S, F32); // padded chunk length in LDS (16-byte slots)
  // slot of the parked right-hand side of row r (1 <= r <= S-2)
  constexpr int PK0 = F32 ? 1 : 0;
  const int lrow = P * SP + 1;               // odd stride: columns start in different banks
  // columns run linearly over the padded level plane in memory order (offset
  // x inside a level holds column (n, m) = spec_nm(x)), so a tile is one
  // aligned contiguous run of each level; padding columns (m >= nxh) ride
  // along as dummy systems with a zero right-hand side and are neither read
  // nor written
  const int ncolp = d.ny * nxp;
  const int col0 = lb * CW;
  using CS = cx<TS>;
  CS* Sg = reinterpret_cast<CS*>(io.spec);
  const long long plane = d.plane;

  // 1. coalesced load of CW columns x nz levels into LDS. blockDim = CW P:
  //    thread (cc, kq) = (tid mod CW, tid / CW) stages rows kq S .. kq S + S-1
  //    of column cc, i.e. exactly the rows that lane kq of that column will
  //    eliminate; a wave's load touches CW consecutive columns of each of its
  //    levels. The loads are unconditional (clamped address, zero selected
  //    afterwards) so that all of them are in flight before the first wait.
  //    The PAIRS instance (FP32 storage, even S, tiles of at least 8
  //    columns): thread (cp, kr) = (tid mod CW/2, tid / (CW/2)) stages levels
  //    kr S/2 .. kr S/2 + S/2-1 of the column pair 2cp, 2cp+1 instead, with
  //    16-byte accesses: the same runs in half the memory instructions. A pair
  //    never straddles the end of the plane (col0, ncolp and the plane are
  //    even), so its address is in bounds whenever either column is valid.
  const int tid = threadIdx.x;
  const int cc = tid & (CW - 1), kq = tid >> lcw;
  const int ks = kq * S;
  double2* sst = stage + cc * lrow + kq * SP;
  const int scol_g = col0 + cc;
  int sn, sm;
  spec_nm(d, scol_g, sn, sm);
  const bool sok = scol_g < ncolp && sm < nxh;
  static_assert(!PAIRS || (F32 && S % 2 == 0), "column pairs need FP32 storage and an even row count");
  constexpr int S2 = PAIRS ? S / 2 : 1;
  constexpr bool pairs = PAIRS;
  const int cp = pairs ? tid & ((CW >> 1) - 1) : 0, kr = pairs ? tid >> (lcw - 1) : 0;
  const int gA = col0 + 2 * cp, ks2 = kr * S2;
  int nA, mA, nB, mB;
  spec_nm(d, gA, nA, mA);
  spec_nm(d, gA + 1, nB, mB);
  const bool okA = pairs && gA < ncolp && mA < nxh, okB = pairs && gA + 1 < ncolp && mB < nxh;
  const long long plane4 = plane / 2;  // a level in 16-byte units (FP32 pairs)
  // the pair's chunk slots: column 2cp + h, lane chunk kr / 2, rows (kr mod 2) S/2 ..
  auto pslot = [&](int h) {
    return reinterpret_cast<float2*>(stage + (2 * cp + h) * lrow + (kr >> 1) * SP) + (kr & 1) * S2;
  };
  CS ld[S];
  float4 ld4[S2];
  if constexpr (pairs) {
    // levels ks2 .. ks2+S2-1, clamped to nz-1 (those rows are zeroed below)
    const float4* src = reinterpret_cast<const float4*>(Sg + ((okA || okB) ? gA : 0) + (long long)min(ks2, nz - 1) * plane);
#pragma unroll
    for (int j = 0; j < S2; ++j) {
      ld4[j] = src[0];
      if (j + 1 < S2) src += (ks2 + j + 1 < nz) ? plane4 : 0;
    }
  } else {
    // levels ks .. ks+S-1, clamped to nz-1 (those rows are zeroed below)
    const CS* src = Sg + (sok ? scol_g : 0) + (long long)min(ks, nz - 1) * plane;
#pragma unroll
    for (int j = 0; j < S; ++j) {
      ld[j] = src[0];
      if (j + 1 < S) src += (ks + j + 1 < nz) ? plane : 0;
    }
  }

  const int c = tid >> lp, q = tid & (P - 1);
  const int col = col0 + c;
  int ncol, mcol;
  spec_nm(d, col, ncol, mcol);
  const bool valid = col < ncolp && mcol < nxh;
  const bool singular = SING && valid && (col == 0);
  double2* scol = stage + c * lrow;
  const int k0 = q * S;

  // coefficients of the lane's rows (the tables run past nz with rows that
  // are decoupled from the system): loads issued while the column data is
  // still arriving
  const double lamv = ldg(d.lamy + min(ncol, d.ny - 1)) + ldg(d.lamx + min(mcol, nxh - 1));
  double A[S], B[S], C[S], R0[S];
#pragma unroll
  for (int r = 0; r < S; ++r) {
    A[r] = ldg(d.tra + k0 + r);
    C[r] = ldg(d.trc + k0 + r);
    R0[r] = ldg(d.trr + k0 + r);
  }
  // column data into LDS (zero outside the grid)
  if constexpr (pairs) {
    float2* la = pslot(0);
    float2* lb = pslot(1);
#pragma unroll
    for (int j = 0; j < S2; ++j) {
      const bool in = ks2 + j < nz;  // every slot exists; rows >= nz are never read
      la[j] = okA && in ? make_float2(ld4[j].x, ld4[j].y) : make_float2(0.0f, 0.0f);
      lb[j] = okB && in ? make_float2(ld4[j].z, ld4[j].w) : make_float2(0.0f, 0.0f);
    }
  } else {
#pragma unroll
    for (int j = 0; j < S; ++j) {
      const bool in = sok && ks + j < nz;  // every slot exists; rows >= nz are never read
      if constexpr (F32)
        reinterpret_cast<float2*>(sst)[j] = in ? make_float2(ld[j].x, ld[j].y) : make_float2(0.0f, 0.0f);
      else
        sst[j] = make_double2(in ? (double)ld[j].x : 0.0, in ? (double)ld[j].y : 0.0);
    }
  }
  // padding columns (m >= nxh) solve a well-conditioned dummy system with a
  // zero right-hand side and are never stored
  const double lam = valid ? lamv : 1.0;
#pragma unroll
  for (int r = 0; r < S; ++r) B[r] = -(A[r] + C[r]) - R0[r] * lam;
  if (singular) {  // (0,0) column: its top row is pinned (identity)
#pragma unroll
    for (int r = 0; r < S; ++r)
      if (k0 + r == nz - 1) {
        A[r] = 0.0;
        B[r] = 1.0;
        C[r] = 0.0;
      }
  }
  __syncthreads();

  // staged data: zero for rows >= nz and for padding columns
  double2 D[S];
#pragma unroll
  for (int r = 0; r < S; ++r) {
    if constexpr (F32) {
      const float2 t = reinterpret_cast<const float2*>(scol + q * SP)[r];
      D[r] = make_double2(t.x, t.y);
    } else {
      D[r] = scol[q * SP + r];
    }
  }
  asm volatile("" ::: "memory");  // the slots are reused as FP64 below
  // (0,0) column (one per member, lanes of one wave): remove the dz-weighted
  // mean of the right-hand side, then pin the top row (identity, rhs 0)
  if (singular) {
    double2 sum = make_double2(0.0, 0.0);
#pragma unroll
    for (int r = 0; r < S; ++r) {
      const double dzr = (k0 + r < nz) ? ldg(d.dz + (k0 + r)) : 0.0;
      sum.x += dzr * D[r].x;
      sum.y += dzr * D[r].y;
    }
    sum = column_sum(sum, P);
#pragma unroll
    for (int r = 0; r < S; ++r) {
      const int k = k0 + r;
      if (k < nz - 1) {
        D[r].x -= sum.x * d.rH;
        D[r].y -= sum.y * d.rH;
      } else {
        D[r] = make_double2(0.0, 0.0);
      }
    }
  }

  // Deflation of the near-null direction (FP64 storage). The dz-weighted sum
  // of a column's rows cancels its vertical fluxes, which leaves
  // sum_k dz_k B_k = -lam sum_k dz_k rho0_k P_k: the component of P along
  // the constants, c = -sum dz B / (lam sum dz rho0), is known in closed
  // form. With P = c + Q the elimination solves T Q = B - rho0 sum dz B /
  // sum dz rho0 for the part orthogonal to it, so round-off amplified by the
  // near-singularity of the low-wavenumber columns (lam -> 0) acts on Q, not
  // on the large c ~ 1/lam. The (0,0) column (lam = 0) keeps its own gauge
  // treatment; padding columns have B = 0, so c = 0.
  // Only waves holding a column with lam < lamdef (condition number above
  // ~1e4: the lowest wavenumbers, a few columns in a million) do it; the
  // branch is uniform over the wave, so the lane reduction sees every lane.
  double2 cdef = make_double2(0.0, 0.0);
  if constexpr (!F32) {
    if (__any(lam < d.lamdef)) {
    double2 sb = make_double2(0.0, 0.0);
#pragma unroll
    for (int r = 0; r < S; ++r) {
      const double dzr = (k0 + r < nz) ? ldg(d.dz + (k0 + r)) : 0.0;
      sb.x += dzr * D[r].x;
      sb.y += dzr * D[r].y;
    }
    sb = column_sum(sb, P);  // every lane of the column takes part
    if (!singular) {
      const double gx = sb.x * d.rSr, gy = sb.y * d.rSr;
#pragma unroll
      for (int r = 0; r < S; ++r) {  // R0 = rho0 on real rows, 0 past nz
        D[r].x -= R0[r] * gx;
        D[r].y -= R0[r] * gy;
      }
      const double il = 1.0 / lam;
      cdef = make_double2(-gx * il, -gy * il);
    }
    }
  }

  // 1. chunk elimination: x_r + al_r x_0 + ga_r x_{r+1} = de_r (r >= 1), then
  //    backward to x_r = e_r - f_r x_0 - g_r x_{S-1}, kept in (de, al, ga)
  double al[S], ga[S];
  double2 de[S];
#pragma unroll
  for (int r = 1; r < S; ++r) {
    if (r == 1) {
      const double inv = rcp64(B[1]);
      al[1] = A[1] * inv;
      ga[1] = C[1] * inv;
      de[1] = make_double2(D[1].x * inv, D[1].y * inv);
    } else {
      const double inv = rcp64(B[r] - A[r] * ga[r - 1]);
      al[r] = -A[r] * al[r - 1] * inv;
      ga[r] = C[r] * inv;
      de[r] = make_double2((D[r].x - A[r] * de[r - 1].x) * inv, (D[r].y - A[r] * de[r - 1].y) * inv);
    }
  }
  // interface row of L_q:  al L_q... written as  aL F_q + L_q + cL F_{q+1} = dL
  const double aL = al[S - 1], cL = ga[S - 1];
  const double2 dL = de[S - 1];
  de[S - 1] = make_double2(0.0, 0.0);
  al[S - 1] = 0.0;
  ga[S - 1] = -1.0;
#pragma unroll
  for (int r = S - 2; r >= 1; --r) {
    const double g = ga[r];
    de[r] = make_double2(de[r].x - g * de[r + 1].x, de[r].y - g * de[r + 1].y);
    al[r] = al[r] - g * al[r + 1];
    ga[r] = -g * ga[r + 1];
  }
  // interface row of F_q:  A0 L_{q-1} + (B0 - C0 f1) F_q - C0 g1 L_q = D0 - C0 e1
  const double aF = A[0], bF = B[0] - C[0] * al[1], cF = -C[0] * ga[1];
  const double2 dF = make_double2(D[0].x - C[0] * de[1].x, D[0].y - C[0] * de[1].y);
  // park e_r in the lane's own LDS slots (their right-hand sides are
  // consumed) while the interface system is solved: fewer live registers
#pragma unroll
  for (int r = 1; r < S - 1; ++r) scol[q * SP + r - PK0] = de[r];
  asm volatile("" ::: "memory");

  // 2. substitute L_{q-1} (from lane q-1) and L_q into the F_q row
  const int lane = __lane_id();
  const int up = (q > 0) ? lane - 1 : lane, dn = (q < P - 1) ? lane + 1 : lane;
  const bool row16 = P == 16;  // a column is one DPP row: shifts on the vector ALU
  const double aLm = row16 ? dpp_shift<1, true>(aL) : shfl_d(aL, up);
  const double cLm = row16 ? dpp_shift<1, true>(cL) : shfl_d(cL, up);
  const double dLmx = row16 ? dpp_shift<1, true>(dL.x) : shfl_d(dL.x, up);
  const double dLmy = row16 ? dpp_shift<1, true>(dL.y) : shfl_d(dL.y, up);
  Row5 row;
  {
    const double am = (q > 0) ? aF : 0.0;  // coupling to L_{q-1}
    row.a = -am * aLm;
    row.b = bF - am * cLm - cF * aL;
    row.c = -cF * cL;
    row.x = dF.x - am * dLmx - cF * dL.x;
    row.y = dF.y - am * dLmy - cF * dL.y;
  }

  // 3. parallel cyclic reduction over the P lanes of the column, on rows
  //    scaled to a unit diagonal (four values travel per neighbour, one
  //    reciprocal per step). A lane without a partner at distance h already
  //    has a zero coupling on that side (the first lane's a and the last
  //    lane's c are zero, and each step keeps them zero out to distance 2h),
  //    so whatever it reads there (its own row through an LDS permute, 0
  //    through DPP) is multiplied by zero.
  {
    const double ib = rcp64(row.b);
    row.a *= ib;
    row.c *= ib;
    row.x *= ib;
    row.y *= ib;
  }
  if (row16) {
    pcr_step16<1>(row.a, row.c, row.x, row.y);
    pcr_step16<2>(row.a, row.c, row.x, row.y);
    pcr_step16<4>(row.a, row.c, row.x, row.y);
    pcr_step16<8>(row.a, row.c, row.x, row.y);
  } else
  for (int h = 1; h < P; h *= 2) {
    const int sl = (q >= h) ? lane - h : lane, sr = (q + h < P) ? lane + h : lane;
    const double la = shfl_d(row.a, sl), lc = shfl_d(row.c, sl), lx = shfl_d(row.x, sl), ly = shfl_d(row.y, sl);
    const double ha = shfl_d(row.a, sr), hc = shfl_d(row.c, sr), hx = shfl_d(row.x, sr), hy = shfl_d(row.y, sr);
    const double nb = 1.0 - lc * row.a - ha * row.c;
    const double ib = rcp64(nb);
    const double na = -la * row.a, nc = -hc * row.c;
    const double nx = row.x - lx * row.a - hx * row.c;
    const double ny = row.y - ly * row.a - hy * row.c;
    row.a = na * ib;
    row.c = nc * ib;
    row.x = nx * ib;
    row.y = ny * ib;
  }
  const double2 F = make_double2(row.x, row.y);

  // 4. L_q = dL - aL F_q - cL F_{q+1}, then the chunk's interior rows
  const double Fnx = row16 ? dpp_shift<1, false>(F.x) : shfl_d(F.x, dn);
  const double Fny = row16 ? dpp_shift<1, false>(F.y) : shfl_d(F.y, dn);
  const double2 Fn = (q < P - 1) ? make_double2(Fnx, Fny) : make_double2(0.0, 0.0);
  const double2 L = make_double2(dL.x - aL * F.x - cL * Fn.x, dL.y - aL * F.y - cL * Fn.y);
  double2 X[S];
#pragma unroll
  for (int r = 0; r < S; ++r) {
    if (r == 0) X[r] = F;
    else if (r == S - 1) X[r] = L;
    else {
      const double2 e = scol[q * SP + r - PK0];
      X[r] = make_double2(e.x - al[r] * F.x - ga[r] * L.x, e.y - al[r] * F.y - ga[r] * L.y);
    }
  }
  // the deflated constant back (0 for the (0,0) and padding columns)
  if constexpr (!F32) {
#pragma unroll
    for (int r = 0; r < S; ++r) {
      X[r].x += cdef.x;
      X[r].y += cdef.y;
    }
  }
  // (0,0) column: gauge sum_k dz_k P_k = 0
  if (singular) {
    double2 sum = make_double2(0.0, 0.0);
#pragma unroll
    for (int r = 0; r < S; ++r) {
      const double dzr = (k0 + r < nz) ? ldg(d.dz + (k0 + r)) : 0.0;
      sum.x += dzr * X[r].x;
      sum.y += dzr * X[r].y;
    }
    sum = column_sum(sum, P);
#pragma unroll
    for (int r = 0; r < S; ++r) {
      X[r].x -= sum.x * d.rH;
      X[r].y -= sum.y * d.rH;
    }
  }
  // the solution back into the chunk (rows >= nz are never stored); FP32
  // storage writes it scaled by 1/(nx ny) and rounded, over the parked values
  asm volatile("" ::: "memory");
  if constexpr (F32) {
    const double sc = d.inv_nxny;
    float2* out = reinterpret_cast<float2*>(scol + q * SP);
#pragma unroll
    for (int r = 0; r < S; ++r) out[r] = make_float2((float)(X[r].x * sc), (float)(X[r].y * sc));
  } else {
#pragma unroll
    for (int r = 0; r < S; ++r) scol[q * SP + r] = X[r];
  }
  __syncthreads();

  // coalesced store (the staging thread's rows), scaled by 1/(nx ny)
  if constexpr (pairs) {
    const float2* la = pslot(0);
    const float2* lb = pslot(1);
    float2 xa[S2], xb[S2];
#pragma unroll
    for (int j = 0; j < S2; ++j) {
      xa[j] = la[j];
      xb[j] = lb[j];
    }
    CS* dA = Sg + gA + (long long)ks2 * plane;
    float4* d4 = reinterpret_cast<float4*>(dA);
#pragma unroll
    for (int j = 0; j < S2; ++j) {
      if (ks2 + j < nz) {
        if (okA && okB) d4[j * plane4] = make_float4(xa[j].x, xa[j].y, xb[j].x, xb[j].y);
        else if (okA) dA[j * plane] = CS{xa[j].x, xa[j].y};
        else if (okB) dA[j * plane + 1] = CS{xb[j].x, xb[j].y};
      }
    }
  } else if (sok) {
    CS* dst = Sg + scol_g + (long long)ks * plane;
    if constexpr (F32) {
      float2 x[S];
#pragma unroll
      for (int j = 0; j < S; ++j) x[j] = reinterpret_cast<const float2*>(sst)[j];
#pragma unroll
      for (int j = 0; j < S; ++j)
        if (ks + j < nz) dst[j * plane] = CS{x[j].x, x[j].y};
    } else {
      const double sc = d.inv_nxny;
      double2 x[S];
#pragma unroll
      for (int j = 0; j < S; ++j) x[j] = sst[j];
#pragma unroll
      for (int j = 0; j < S; ++j)
        if (ks + j < nz) dst[j * plane] = CS{(TS)(x[j].x * sc), (TS)(x[j].y * sc)};
    }
  }
}

// FP32 storage up to 10 rows per lane: a register budget for 4 waves per
// SIMD (the LDS chunks then fit 4 such workgroups per CU); the solve is
// latency-bound and gains more from the extra wave than it loses to a
// 16-byte spill at 10 rows
template <typename TS, int S, int MAXT, bool PAIRS>
__global__ void __launch_bounds__(MAXT) __attribute__((amdgpu_waves_per_eu(S <= 10 && sizeof(TS) == 4 ? 4 : 1, 8)))
k_tridiag(LaunchArgs a) {
  extern __shared__ unsigned char smem_raw[];
  double2* stage = reinterpret_cast<double2*>(smem_raw);
  const Member mb = launch_member(a, blockIdx.x);
  const MemberDesc d = load_desc(mb.desc);
  keep_tri(d);
  if (skipped(d)) return;
  const IoPtrs& io = mb.io;
  // a spectrum larger than the 256 MB Infinity Cache: tiles in launch order,
  // not grouped by XCD. A column is read once, so there is no L2 reuse to
  // group for, and the workgroups in flight then cover one contiguous run of
  // columns of every level instead of eight runs an eighth of a plane apart
  // (2048^2 x 160, 1024^2 x 256, 4096^2 x 64: 2-7 % faster). Smaller members
  // keep the XCD grouping, which measured 3 % faster on an ensemble of them.
  const bool big = (double)d.plane * d.nz * sizeof(cx<TS>) > 256.0 * (1 << 20);
  const int lb = big ? (int)blockIdx.x - mb.start : xcd_local_block(mb);
  if (lb == 0)
    tri_tile<TS, S, true, PAIRS>(d, io, lb, stage);
  else
    tri_tile<TS, S, false, PAIRS>(d, io, lb, stage);
}

// ---------------------------------------------------------------------------
// FP64 tridiagonal solve over FP32 storage, a wave per row chunk (the grids
// tricol_shape picks, at most kTriColMax levels). The same partition method as
// above, mapped the other way round: a workgroup takes 64 consecutive entries of
// the level plane, lane c of every wave holds column c, and wave q eliminates rows
// q S .. q S + S-1. Every load and store is then a run of 64 columns of one level
// (512 bytes) straight between memory and registers, the rows' coefficients are
// wave-uniform (scalar loads and operands), and only the interface system
// crosses waves, through LDS. Registers: a row keeps 1/pivot and its
// right-hand side (6 registers) between the elimination and the back
// substitution; the couplings to the chunk's first row are regenerated from
// them.
//
// Bound by the access pattern: with the elimination left out (a copy of the
// kernel that loads and stores its tiles) it takes 1.15 of 1.32 ms at 2048^2 x
// 160, 4.7 TB/s over nz runs a level apart against 6.5 TB/s of one contiguous
// copy. Against the lanes-per-column kernel, us: 1024^2 x 256 1161 -> 461 (32
// lanes 686), 1024^2 x 100 211 -> 160, 512^2 x 256 189 -> 126. FP64 storage, whose
// runs are twice as long in either kernel, was no faster this way (2048^2 x 160
// 2166 against 2274 us, 1024^2 x 256 907 / 924, 512^2 x 128 108 / 118).
// The interface rows are eliminated by two waves from both ends: parallel cyclic
// reduction on all waves took as long as the chunk elimination itself (1.42 ms
// at 2048^2 x 160), and loading the next tile during the solve (a persistent
// workgroup) gained 1 % there and lost up to 25 % at 384 x 256 x 96.
// ---------------------------------------------------------------------------
// The (0,0) column, one wave: with no horizontal part the rows telescope.
// c_k dz_k (P_{k+1} - P_k) = sum_{j <= k} dz_j (B_j - mean) is the flux through
// the top of level k (a_{k+1} dz_{k+1} = c_k dz_k), so P is a running sum of
// running sums; mean is the right-hand side's dz-weighted mean, and the gauge
// sum_k dz_k P_k = 0 closes it. Lane l holds levels 4l .. 4l+3 (kTriColMax is
// 256).
__device__ __forceinline__ double2 wave_scan(double2 v) {  // inclusive
  const int l = threadIdx.x & 63;
#pragma unroll
  for (int o = 1; o < 64; o *= 2) {
    const double x = __shfl_up(v.x, o), y = __shfl_up(v.y, o);
    if (l >= o) {
      v.x += x;
      v.y += y;
    }
  }
  return v;
}

__device__ __forceinline__ void tri_mean_column(cx<float>* S, int nz, long long plane, const double* dz, const double* trc,
                                                double rH, double sc) {
  using CS = cx<float>;
  const int k0 = 4 * (threadIdx.x & 63);
  double2 v[4];
  double w[4];
  double2 s = make_double2(0.0, 0.0);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int k = min(k0 + r, nz - 1);
    const CS b = S[(long long)k * plane];
    w[r] = k0 + r < nz ? ldg(dz + k) : 0.0;
    v[r] = make_double2(b.x, b.y);
    s.x += w[r] * v[r].x;
    s.y += w[r] * v[r].y;
  }
  s = wave_scan(s);
  const double mx = __shfl(s.x, 63) * rH, my = __shfl(s.y, 63) * rH;
  // fluxes (running sums inside the lane, then over the lanes), as jumps of P
  double2 f = make_double2(0.0, 0.0);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    f.x += w[r] * (v[r].x - mx);
    f.y += w[r] * (v[r].y - my);
    v[r] = f;
  }
  double2 t = wave_scan(f);
  const double2 below = make_double2(t.x - f.x, t.y - f.y);
  double2 jump = make_double2(0.0, 0.0);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const bool in = k0 + r < nz - 1;
    const double g = in ? 1.0 / (ldg(trc + k0 + r) * w[r]) : 0.0;
    const double2 j = make_double2((v[r].x + below.x) * g, (v[r].y + below.y) * g);
    v[r] = jump;  // P at this level, from the lane's first
    jump.x += j.x;
    jump.y += j.y;
  }
  t = wave_scan(jump);
  s = make_double2(0.0, 0.0);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    v[r].x += t.x - jump.x;
    v[r].y += t.y - jump.y;
    s.x += w[r] * v[r].x;
    s.y += w[r] * v[r].y;
  }
  s = wave_scan(s);
  const double gx = __shfl(s.x, 63) * rH, gy = __shfl(s.y, 63) * rH;
#pragma unroll
  for (int r = 0; r < 4; ++r)
    if (k0 + r < nz) S[(long long)(k0 + r) * plane] = CS{(float)((v[r].x - gx) * sc), (float)((v[r].y - gy) * sc)};
}

// A wave-uniform index whose value the compiler cannot trace: coefficients
// read through it are read again instead of being kept in scalar registers
// (three doubles a row) since an earlier read.
__device__ __forceinline__ int fresh(int i) {
  int zero;
  asm volatile("s_mov_b32 %0, 0" : "=s"(zero));
  return wuni(i) + zero;
}

// Interface system of 64 columns (lane = column), P >= 2 rows a x_{q-1} + b x_q
// + c x_{q+1} = (x, y) in Ib [5][P][64], eliminated from both ends at once:
// wave 0 takes rows 0 .. P/2-1 upwards, wave 1 (up) rows P-1 .. P/2 downwards;
// the two meet in a 2 x 2 system. The eliminated rows x_q + u x_next = s go
// back into slots 0, 3, 4 of their row. One wave works while the others wait,
// so it is the latency that counts: a row is read from LDS while the row
// before it is eliminated.
__device__ __forceinline__ void tri_interface_eliminate(double* Ib, int P, int c, bool up) {
  const int VS = P * 64, step = up ? -64 : 64;
  const int o0 = up ? 2 * VS : 0, o2 = up ? 0 : 2 * VS;  // coupling to the row before, to the next
  double* r = Ib + (up ? P - 1 : 0) * 64 + c;
  double prev = r[o0], b = r[VS], next = r[o2], x = r[3 * VS], y = r[4 * VS];
  double u = 0.0, sx = 0.0, sy = 0.0;
#pragma unroll 1
  for (int i = P / 2 - 1;; --i) {
    const double* n = r + (i ? step : 0);
    const double nprev = n[o0], nb = n[VS], nnext = n[o2], nx = n[3 * VS], ny = n[4 * VS];
    const double ib = rcp64(b - prev * u);
    u = next * ib;
    sx = (x - prev * sx) * ib;
    sy = (y - prev * sy) * ib;
    r[0] = u;
    r[3 * VS] = sx;
    r[4 * VS] = sy;
    if (i == 0) break;
    r += step;
    prev = nprev;
    b = nb;
    next = nnext;
    x = nx;
    y = ny;
  }
}

// The solution of the wave's half into Fb [2][P][64] (after a barrier), two
// rows read at a time.
__device__ __forceinline__ void tri_interface_back(const double* Ib, double* Fb, int P, int c, bool up) {
  const int VS = P * 64, h = P / 2, step = up ? 64 : -64;
  const int q = up ? h : h - 1;
  const double* r = Ib + q * 64 + c;
  const double* o = up ? r - 64 : r + 64;        // the other half's last row
  const double u = r[0];
  const double ib = rcp64(1.0 - u * o[0]);
  double x = (r[3 * VS] - u * o[3 * VS]) * ib, y = (r[4 * VS] - u * o[4 * VS]) * ib;
  double* f = Fb + q * 64 + c;
  f[0] = x;
  f[VS] = y;
#pragma unroll 1
  for (int i = 1; i < h; i += 2) {
    const double *s = r + i * step, *t = r + min(i + 1, h - 1) * step;
    const double su = s[0], sx = s[3 * VS], sy = s[4 * VS], tu = t[0], tx = t[3 * VS], ty = t[4 * VS];
    x = sx - su * x;
    y = sy - su * y;
    f[i * step] = x;
    f[i * step + VS] = y;
    if (i + 1 < h) {
      x = tx - tu * x;
      y = ty - tu * y;
      f[(i + 1) * step] = x;
      f[(i + 1) * step + VS] = y;
    }
  }
}

template <int S>
__global__ void __launch_bounds__(1024) k_tricol(LaunchArgs a) {
  extern __shared__ double smem[];
  using CS = cx<float>;
  typedef float cv __attribute__((ext_vector_type(2)));
  const int P = blockDim.x >> 6;                 // waves = row chunks
  const int q = wuni((int)(threadIdx.x >> 6)), c = threadIdx.x & 63;
  const Member mb = launch_member(a, blockIdx.x);
  const MemberDesc d = load_desc(mb.desc);
  keep_tri(d);
  if (skipped(d)) return;
  // tiles in launch order or by XCD, as in k_tridiag
  const bool big = (double)d.plane * d.nz * sizeof(CS) > 256.0 * (1 << 20);
  const int lb = wuni(big ? (int)blockIdx.x - mb.start : xcd_local_block(mb));
  const int nz = d.nz, ncolp = d.ny * d.nxp;
  const long long plane = d.plane;
  CS* const S0 = reinterpret_cast<CS*>(mb.io.spec) + (long long)lb * 64;  // the tile in level 0
  const int col = lb * 64 + c;
  const int x = min(col, ncolp - 1), blk = (int)fast_div(x, d.bst_mul, d.bst_shift), rem = x - blk * d.bst;
  const int n = rem >> d.lbw, m = (blk << d.lbw) | (rem & (d.sbw - 1));  // as spec_nm
  // column 0 is the (0,0) one (tri_mean_column); it and the padding columns
  // (m >= nxh) solve a dummy system with a zero right-hand side here and are
  // not stored
  const bool valid = col > 0 && col < ncolp && m < d.nxh;
  if (lb == 0 && q == 0) tri_mean_column(S0, nz, plane, d.dz, d.trc, d.rH, d.inv_nxny);  // no barrier inside

  // rows q S .. q S + S-1 of the lane's column: entries past the plane read
  // the tile's first, rows past nz the last level
  int k0 = fresh(q * S);
  double2 D[S];
  {
    cv ld[S];
    const unsigned off = (unsigned)(col < ncolp ? c : 0);
#pragma unroll
    for (int r = 0; r < S; ++r)
      ld[r] = ((const __attribute__((address_space(1))) cv*)(S0 + (long long)min(k0 + r, nz - 1) * plane))[off];
#pragma unroll
    for (int r = 0; r < S; ++r) {
      const bool in = valid && k0 + r < nz;
      D[r] = make_double2(in ? (double)ld[r].x : 0.0, in ? (double)ld[r].y : 0.0);
    }
  }
  const double lamv = ldg(d.lamy + n) + ldg(d.lamx + min(m, d.nxh - 1));
  const double lam = valid ? lamv : 1.0;           // dummy: well conditioned
  const double *ta = d.tra, *tc = d.trc, *tr = d.trr;
  const int VS = P * 64;
  double* Ib = smem;                               // [5][P][64] interface rows
  double* Lb = smem + 5 * VS;                      // [4][P][64] last rows of the chunks
  double* Fb = smem + 9 * VS;                      // [2][P][64] interface solution

  // 1. chunk elimination, x_r + al_r x_0 + ga_r x_{r+1} = de_r (de in D), and
  //    the same sums run forward for x_1 = e1 - f1 x_0 + g1 x_{S-1}
  double inv[S], al = 0.0, ga = 0.0, e1x = 0.0, e1y = 0.0, f1 = 0.0, g1 = 1.0;
  const double2 D0 = D[0];
#pragma unroll
  for (int r = 1; r < S; ++r) {
    if (r % 4 == 0) k0 = fresh(q * S);
    const double A = ldc(ta + k0 + r), C = ldc(tc + k0 + r), B = -(A + C) - ldc(tr + k0 + r) * lam;
    if (r == 1) {
      inv[r] = rcp64(B);
      al = A * inv[r];
      D[r] = make_double2(D[r].x * inv[r], D[r].y * inv[r]);
    } else {
      inv[r] = rcp64(B - A * ga);
      al = -A * al * inv[r];
      D[r] = make_double2((D[r].x - A * D[r - 1].x) * inv[r], (D[r].y - A * D[r - 1].y) * inv[r]);
    }
    ga = C * inv[r];
    if (r < S - 1) {
      e1x += g1 * D[r].x;
      e1y += g1 * D[r].y;
      f1 += g1 * al;
      g1 *= -ga;
    }
  }
  const double aL = al, cL = ga;
  const double2 dL = D[S - 1];
  // 2. L_{q-1} and L_q substituted into the F_q row; the interface system by
  //    two waves
  {
    double* w = Lb + threadIdx.x;
    w[0] = aL;
    w[VS] = cL;
    w[2 * VS] = dL.x;
    w[3 * VS] = dL.y;
  }
  __syncthreads();
  {
    const double A0 = ldc(ta + k0), C0 = ldc(tc + k0);
    const double am = q ? A0 : 0.0, cF = C0 * g1;
    const double* l = Lb + threadIdx.x - (q ? 64 : 0);
    double* w = Ib + threadIdx.x;
    w[0] = -am * l[0];
    w[VS] = -(A0 + C0) - ldc(tr + k0) * lam - C0 * f1 - am * l[VS] - cF * aL;
    w[2 * VS] = -cF * cL;
    w[3 * VS] = D0.x - C0 * e1x - am * l[2 * VS] - cF * dL.x;
    w[4 * VS] = D0.y - C0 * e1y - am * l[3 * VS] - cF * dL.y;
  }
  __syncthreads();
  if (q < 2) tri_interface_eliminate(Ib, P, c, q == 1);
  __syncthreads();
  if (q < 2) tri_interface_back(Ib, Fb, P, c, q == 1);
  __syncthreads();

  // 3. back substitution of the chunk's interior rows; the coefficients are
  //    read again (see fresh)
  k0 = fresh(q * S);
  const double* f = Fb + threadIdx.x;
  const double2 F = make_double2(f[0], f[VS]);
  const int up = q < P - 1 ? 64 : 0;               // the last chunk's cL is 0 (the lid)
  const double2 Fn = make_double2(f[up], f[VS + up]);
  D[0] = F;
  D[S - 1] = make_double2(dL.x - aL * F.x - cL * Fn.x, dL.y - aL * F.y - cL * Fn.y);
  if constexpr (S > 2) {
#pragma unroll
    for (int r = 1; r < S - 1; ++r) {
      al = (r == 1 ? inv[r] : -al * inv[r]) * ldc(ta + k0 + r);
      D[r].x -= al * F.x;
      D[r].y -= al * F.y;
    }
#pragma unroll
    for (int r = S - 2; r >= 1; --r) {
      const double g = ldc(tc + k0 + r) * inv[r];
      D[r].x -= g * D[r + 1].x;
      D[r].y -= g * D[r + 1].y;
    }
  }
  if (valid) {
    const double sc = d.inv_nxny;
#pragma unroll
    for (int r = 0; r < S; ++r)
      if (k0 + r < nz) {
        cv v;
        v.x = (float)(D[r].x * sc);
        v.y = (float)(D[r].y * sc);
        ((__attribute__((address_space(1))) cv*)(S0 + (long long)(k0 + r) * plane))[c] = v;
      }
  }
}

// ---------------------------------------------------------------------------
// host-side launchers
// ---------------------------------------------------------------------------
#define MONC_TRI_ROWS(X) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(10) X(12) X(16)
// rows per wave of the wave-per-chunk tridiagonal kernel
#define MONC_TRICOL_ROWS(X) \
  X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14) X(15) X(16)

void init_tridiag_attributes() {
#define MONC_TRI_ATTR(S)                   \
  set_lds_limit(k_tridiag<double, S, 256, false>); \
  set_lds_limit(k_tridiag<float, S, 256, false>);  \
  set_lds_limit(k_tridiag<double, S, 512, false>); \
  set_lds_limit(k_tridiag<float, S, 512, false>);  \
  if constexpr (S % 2 == 0) {                      \
    set_lds_limit(k_tridiag<float, S, 256, S % 2 == 0>); \
    set_lds_limit(k_tridiag<float, S, 512, S % 2 == 0>); \
  }
  MONC_TRI_ROWS(MONC_TRI_ATTR)
#undef MONC_TRI_ATTR
#define MONC_TRICOL_ATTR(S) set_lds_limit(k_tricol<S>);
  MONC_TRICOL_ROWS(MONC_TRICOL_ATTR)
#undef MONC_TRICOL_ATTR
}

// FP32 tridiagonal instance: column pairs (even S only) or single columns
template <int S, int MAXT>
static void launch_tri_f32(const LaunchArgs& a, int grid, int block, size_t lds, bool pairs, void* stream) {
  if constexpr (S % 2 == 0) {
    if (pairs) {
      MONC_GO((k_tridiag<float, S, MAXT, S % 2 == 0>));
      return;
    }
  }
  MONC_GO((k_tridiag<float, S, MAXT, false>));
}

void launch_tridiag(const LaunchArgs& a, int grid, int block, size_t lds, bool fp64, int rows, bool pairs,
                    void* stream) {
  switch (rows) {
#define MONC_CASE(S)                                         \
  case S:                                                    \
    if (block <= 256) {                                      \
      if (fp64) MONC_GO((k_tridiag<double, S, 256, false>)); \
      else launch_tri_f32<S, 256>(a, grid, block, lds, pairs, stream); \
    } else {                                                 \
      if (fp64) MONC_GO((k_tridiag<double, S, 512, false>)); \
      else launch_tri_f32<S, 512>(a, grid, block, lds, pairs, stream); \
    }                                                        \
    return;
    MONC_TRI_ROWS(MONC_CASE)
#undef MONC_CASE
  }
}

void launch_tricol(const LaunchArgs& a, int grid, int block, size_t lds, int rows, void* stream) {
  switch (rows) {
#define MONC_CASE(S)         \
  case S:                    \
    MONC_GO((k_tricol<S>));  \
    return;
    MONC_TRICOL_ROWS(MONC_CASE)
#undef MONC_CASE
  }
}

}  // namespace monc
