// Launchers of the variable-density Krylov kernels (krylov.hip): plain
// device pointers to FP64 (nz, ny, nx) fields.
#pragma once

namespace monc {

constexpr int kVarBlock = 256;                  // threads per workgroup
constexpr int kVarPts = 4;                      // points per thread of the pointwise kernels
constexpr int kVarStPts = 2;                    // points per thread of the stencil kernels (even)
constexpr int kVarLevels = 2;                   // levels per stencil workgroup (walked upwards)
constexpr int kVarBand = 64;                    // tiles a level of the stencil kernels' block order
constexpr int kVarFinishBlock = 1024;           // threads of the partial-sum reduction

// Scalars in scal[]: a status row, then per iteration it the dz-weighted
// <r_it, z_it>, <d_it, q_it>, <r_it, r_it> and <z_it, q_{it-1}>.
// Status: the gauge sum of p; the done flag (0 running, 1 converged,
// 2 non-finite residual); the last iteration whose <r, r> was formed, and
// that <r, r>. Once the flag is set every later kernel of the solve returns
// at once, so the host can queue several iterations between reads.
enum { kVarRZ = 0, kVarDQ = 1, kVarRR = 2, kVarZQ = 3, kVarSlots = 4 };
enum { kVarGauge = 0, kVarDone = 1, kVarLast = 2, kVarLastRR = 3 };
inline __host__ __device__ int var_slot(int it, int s) { return kVarSlots * (it + 1) + s; }

// A workgroup of kVarBlock threads with pts points each covers a 2-D tile of a
// level: var_tile_w(nx) = min(nx, 256) points wide and kVarBlock pts /
// var_tile_w rows high, so that the rows a stencil reads above and below its
// own are few against the rows it computes.
inline __host__ __device__ int var_tile_w(int nx) { return nx < 256 ? nx : 256; }
inline __host__ __device__ int var_tile_h(int nx, int pts) { return kVarBlock * pts / var_tile_w(nx); }
inline __host__ __device__ int var_tiles_x(int nx) { return (nx + var_tile_w(nx) - 1) / var_tile_w(nx); }
inline __host__ __device__ int var_tiles_y(int nx, int ny, int pts) {
  return (ny + var_tile_h(nx, pts) - 1) / var_tile_h(nx, pts);
}
inline __host__ __device__ long long var_blocks_per_level(int nx, int ny, int pts) {
  return (long long)var_tiles_x(nx) * var_tiles_y(nx, ny, pts);
}
inline __host__ __device__ int var_level_groups(int nz) { return (nz + kVarLevels - 1) / kVarLevels; }
inline long long var_stencil_parts(int nx, int ny, int nz) {
  return var_blocks_per_level(nx, ny, kVarStPts) * var_level_groups(nz);
}
inline long long var_point_parts(int nx, int ny, int nz) { return var_blocks_per_level(nx, ny, kVarPts) * nz; }

struct VarGrid {
  int nx, ny, nz;
  double rdx, rdy;          // 1/dx, 1/dy
  double rdx2, rdy2;        // 1/dx^2, 1/dy^2
  const double* rho;        // density at the cell centres, (nz, ny, nx)
  const double* dz;         // [nz] layer thicknesses (inner-product weights)
  const double* rdz;        // [nz] 1/dz_k
  const double* rdzc;       // [nz] 1/dzc_k (0 at nz-1)
  const double* za;         // [nz] dz_{k+1}/(dz_k + dz_{k+1}) (0 at nz-1)
  const double* zb;         // [nz] dz_k/(dz_k + dz_{k+1}) (0 at nz-1)
};

// part: one partial sum per workgroup: var_stencil_parts entries after the
// divergence and the operator, var_point_parts after the gauge sum.
// Kernels taking scal (except the divergence) do nothing once the done
// flag is set.
void launch_var_div(const VarGrid& g, const double* u, const double* v, const double* w, double* r, double* p,
                    double* part, void* stream);
void launch_var_apply(const VarGrid& g, const double* scal, const double* d, double* q, double* part, void* stream);
// p += alpha_{it-1} d (it > 0), then d = z + beta d; z: FP64 (z64) or FP32
void launch_var_dir(const VarGrid& g, const double* scal, int it, const void* z, bool z64, double* d, double* p,
                    void* stream);
// p += alpha_{it-1} d (it >= 1 iterations taken) and the dz-weighted sum of p;
// p -= scal[slot] * rw
void launch_var_wsum(const VarGrid& g, const double* scal, int it, const double* d, double* p, double* part,
                     void* stream);
void launch_var_shift(const VarGrid& g, const double* scal, int slot, double rw, double* p, void* stream);
// scal[slot0] = sum part0 (and scal[slot1] = sum part1 when part1 is given);
// gated: skip once done
void launch_var_finish(const double* part0, const double* part1, long long n, double* scal, int slot0, int slot1,
                       bool gated, void* stream);
// <r, r> of iteration it into its slot and the status row; sets the done
// flag when it is <= tol2 <r_0, r_0> or not finite
void launch_var_finish_rr(const double* part, long long n, double* scal, int it, double tol2, void* stream);
void launch_var_zero(double* x, int n, void* stream);

}  // namespace monc
