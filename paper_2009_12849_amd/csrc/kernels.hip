// Gradient kernels of the pressure projection for gfx950, and the dispatch of
// the FFT kernels' launches to the instances of fft_inst.hip.
#include <hip/hip_runtime.h>

#include <mutex>

#include "fft_kernels.h"
#include "launch.h"

namespace monc {

// ---------------------------------------------------------------------------
// Pressure-gradient correction u -= G p, evaluated in FP64 from an FP64
// pressure (p itself on the FP64 path; on the mixed path p1 + delta, summed
// in FP64 from the two float scratch fields, and written rounded to float as
// the output p); the fields are T. A thread owns VEC consecutive points of one row of one
// level (vector loads and stores need nx % VEC == 0); w[nz-1] = 0.
// ---------------------------------------------------------------------------
// Per-level horizontal reductions of the projection's outputs (the
// diagnostics an I/O server takes of a prognostic field, Sec. 3): stats[(2 f
// + s) nz + k] for field f = u, v, w, p and statistic s = mean, max over the
// nx ny points of level k. p is the pressure the velocities were corrected
// with (p1 + delta in FP64 on the mixed path). The gradient kernel folds them
// in: each workgroup reduces its points and adds one partial per statistic
// with a device-wide atomic, so the accumulation order (and the last bits of
// the means) can vary from run to run.
__global__ void __launch_bounds__(256) k_stats_init(double* stats, int nz) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t < 8 * nz) stats[t] = ((t / nz) & 1) ? -__builtin_inf() : 0.0;
}

// st[0..3]: sums of u, v, w, p over the caller's points, st[4..7]: maxima;
// added into level k's statistics (sums scaled by rh = 1/(nx ny)) with the
// hardware FP64 atomic add and max (the buffer is device memory)
__device__ __forceinline__ void stats_commit(double* stats, int nz, int k, const double* st, double rh) {
#pragma unroll
  for (int f = 0; f < 4; ++f) {
    __hip_atomic_fetch_add(stats + (2 * f) * nz + k, st[f] * rh, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_fetch_max(stats + (2 * f + 1) * nz + k, st[4 + f], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// Workgroup reduction of the statistics (`whole`: every point of the
// workgroup is in level k), else one partial per thread.
__device__ __forceinline__ void stats_reduce(double* stats, int nz, int k, double* st, double rh, bool whole,
                                             bool live) {
  if (!whole) {
    if (live) stats_commit(stats, nz, k, st, rh);
    return;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
#pragma unroll
    for (int f = 0; f < 4; ++f) {
      st[f] += __shfl_xor(st[f], o);
      st[4 + f] = fmax(st[4 + f], __shfl_xor(st[4 + f], o));
    }
  }
  __shared__ double part[16][8];  // one row per wave (blockDim <= 1024)
  const int wv = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
  if ((threadIdx.x & 63) == 0) {
#pragma unroll
    for (int f = 0; f < 8; ++f) part[wv][f] = st[f];
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int i = 1; i < nw; ++i) {
#pragma unroll
      for (int f = 0; f < 4; ++f) {
        st[f] += part[i][f];
        st[4 + f] = fmax(st[4 + f], part[i][4 + f]);
      }
    }
    stats_commit(stats, nz, k, st, rh);
  }
}

template <typename T, int VEC, bool RED>
__global__ void __launch_bounds__(256) k_grad(LaunchArgs a) {
  typedef T tv __attribute__((ext_vector_type(VEC)));
  typedef double dv __attribute__((ext_vector_type(VEC)));
  const Member mb = launch_member(a, blockIdx.x);
  const MemberDesc d = load_desc(mb.desc);
  keep_grad(d);
  const IoPtrs& io = mb.io;
  const int lb = xcd_local_block(mb);
  const int nx = d.nx, ny = d.ny, nz = d.nz;
  const long long nh = (long long)nx * ny;
  // blocks walk (level, row) tiles like the stencil kernels when a row is a
  // whole number of blocks: p one level up is then read by a block of the
  // same tile, close in time, and hits the XCD's L2
  long long blk = lb;
  const int bpr = d.nx / (int)(blockDim.x * VEC);  // blocks per row
  const bool rowblk = bpr >= 1 && bpr * (int)blockDim.x * VEC == d.nx;  // a block lies in one row
  if (d.ptk > 1 && rowblk) {
    const long long row = tiled_index(lb / bpr, d.ny, d.nz, d.ptk, 8);
    blk = row * bpr + lb % bpr;
  }
  const long long g0 = (blk * blockDim.x + threadIdx.x) * VEC;  // first point
  // a block inside one row: its row (level k, row j) and liveness follow from
  // the block index, workgroup-uniform, so the divisions and the level's
  // coefficient load run on the scalar unit
  const int row = rowblk ? (int)(blk / bpr) : 0;
  const bool live = rowblk ? row < ny * nz : g0 < nh * nz;
  if (!RED && !live) return;
  // with the reductions every thread reaches the workgroup reduction: one
  // past the grid reads point 0, stores nothing and contributes nothing
  const long long g = live ? g0 : 0;
  int k, j, i;
  if (rowblk) {
    const int rw = live ? row : 0;
    k = row_level(d, rw);
    j = rw - k * ny;
    i = live ? (int)(blk - (long long)row * bpr) * (int)blockDim.x * VEC + (int)threadIdx.x * VEC : 0;
  } else {
    // (a grid of 2^31 points or more: 64-bit division)
    k = nh * nz < (1LL << 31) ? (int)fast_div((int)g, d.nh_mul, d.nh_shift) : (int)(g / nh);
    const int h = (int)(g - (long long)k * nh);  // nx ny fits 31 bits
    j = (int)fast_div(h, d.nx_mul, d.nx_shift);
    i = h - j * nx;
  }
  const long long base = (long long)k * nh;
  const long long he = base + (long long)j * nx + ((i + VEC == nx) ? 0 : i + VEC);  // east of the last point
  const long long hn = base + (long long)((j == ny - 1) ? 0 : j + 1) * nx + i;
  T* __restrict__ u = reinterpret_cast<T*>(io.u);
  T* __restrict__ v = reinterpret_cast<T*>(io.v);
  T* __restrict__ w = reinterpret_cast<T*>(io.w);
  const bool top = k == nz - 1;
  // p in FP64: the FP64 path's p, or on the mixed path p1 + delta from the
  // first-pass pressure (io.s2) and the correction (io.s1), summed in FP64.
  // Loads go through global-address-space pointers (the pointers come from a
  // by-value argument struct).
  auto ldp = [&](long long o) -> dv {
    if constexpr (sizeof(T) == 8) {
      return ldg(reinterpret_cast<const dv*>(reinterpret_cast<const double*>(io.p) + o));
    } else {
      const tv hi = ldg(reinterpret_cast<const tv*>(io.s2 + o));
      const tv lo = ldg(reinterpret_cast<const tv*>(io.s1 + o));
      dv r;
#pragma unroll
      for (int e = 0; e < VEC; ++e) r[e] = (double)hi[e] + (double)lo[e];
      return r;
    }
  };
  auto ldp1 = [&](long long o) -> double {
    if constexpr (sizeof(T) == 8) return ldg(reinterpret_cast<const double*>(io.p) + o);
    else return (double)ldg(io.s2 + o) + (double)ldg(io.s1 + o);
  };
  const dv pc = ldp(g);
  const dv pn = ldp(hn);
  const double pel = ldp1(he);
  // p one level up is read unconditionally (clamped on the lid row, where w
  // is set to 0 below) so that all loads issue together
  const dv pu = ldp(top ? g : g + nh);
  // u, v, w are read and written once per point: nontemporal accesses (the
  // pressure fields, re-read as neighbours by other workgroups, keep the
  // normal cache policy)
  tv uu = __builtin_nontemporal_load(reinterpret_cast<const tv*>(u + g));
  tv vv = __builtin_nontemporal_load(reinterpret_cast<const tv*>(v + g));
  tv ww = __builtin_nontemporal_load(reinterpret_cast<const tv*>(w + g));
  const double rz = ldg(d.rdzc + k);  // 0 on the lid row
  const double rdx = d.rdx, rdy = d.rdy;
#pragma unroll
  for (int e = 0; e < VEC; ++e) {
    const double pe = (e + 1 < VEC) ? pc[(e + 1) % VEC] : pel;
    uu[e] = (T)((double)uu[e] - (pe - pc[e]) * rdx);
    vv[e] = (T)((double)vv[e] - (pn[e] - pc[e]) * rdy);
    ww[e] = top ? (T)0 : (T)((double)ww[e] - (pu[e] - pc[e]) * rz);
  }
  if (live) {
    __builtin_nontemporal_store(uu, reinterpret_cast<tv*>(u + g));
    __builtin_nontemporal_store(vv, reinterpret_cast<tv*>(v + g));
    __builtin_nontemporal_store(ww, reinterpret_cast<tv*>(w + g));
    if constexpr (sizeof(T) == 4) {
      // the mixed path's pressure output: p1 + delta rounded to float
      tv po;
#pragma unroll
      for (int e = 0; e < VEC; ++e) po[e] = (T)pc[e];
      __builtin_nontemporal_store(po, reinterpret_cast<tv*>(reinterpret_cast<T*>(io.p) + g));
    }
  }
  if constexpr (RED) {
    double st[8];
#pragma unroll
    for (int f = 0; f < 4; ++f) {
      st[f] = 0.0;
      st[4 + f] = -__builtin_inf();
    }
    if (live) {
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        const double x[4] = {(double)uu[e], (double)vv[e], (double)ww[e], pc[e]};
#pragma unroll
        for (int f = 0; f < 4; ++f) {
          st[f] += x[f];
          st[4 + f] = fmax(st[4 + f], x[f]);
        }
      }
    }
    // a workgroup whose points lie in one level reduces them first
    const long long gb = blk * blockDim.x * VEC;
    const long long gl = min(gb + (long long)blockDim.x * VEC, nh * nz) - 1;
    stats_reduce(io.stats, nz, k, st, 1.0 / (double)nh, gb / nh == gl / nh, live);
  }
}

// ---------------------------------------------------------------------------
// host-side launchers
// ---------------------------------------------------------------------------
// A group's limits are set, and its code is loaded, when the first plan with one
// of its lengths is made: setting all of them took 33 of the 85 ms of a process's
// first plan.
void init_fft_attributes(int n) {
#define MONC_CASE(N) case N:
#define MONC_GROUP_INIT(K)                      \
  switch (n) {                                  \
    MONC_CT_GROUP_##K(MONC_CASE) {              \
      static std::once_flag once;               \
      std::call_once(once, init_fft_group_##K); \
    }                                           \
  }
  MONC_FFT_GROUPS(MONC_GROUP_INIT)
#undef MONC_GROUP_INIT
#undef MONC_CASE
}

void init_kernel_attributes() {
  init_tridiag_attributes();
  init_level_attributes();
  set_lds_limit(k_xfwd_gen<double, 0>);
  set_lds_limit(k_xfwd_gen<float, 0>);
  set_lds_limit(k_xfwd_gen<float, 1>);
  set_lds_limit(k_xfwd_gen<double, 2>);
  set_lds_limit(k_xfwd_gen<float, 2>);
  set_lds_limit(k_xfwd_gen<double, 3>);
  set_lds_limit(k_xfwd_gen<float, 3>);
  set_lds_limit(k_ffty_gen<double, false>);
  set_lds_limit(k_ffty_gen<double, true>);
  set_lds_limit(k_ffty_gen<float, false>);
  set_lds_limit(k_ffty_gen<float, true>);
  set_lds_limit(k_xinv_gen<double, 0>);
  set_lds_limit(k_xinv_gen<float, 0>);
  set_lds_limit(k_xinv_gen<float, 1>);
  set_lds_limit(k_xinv_gen<float, 2>);
  set_lds_limit(k_xinv_gen<double, 3>);
  set_lds_limit(k_xinv_gen<float, 3>);
}

void launch_xfwd(const LaunchArgs& a, int grid, int block, size_t lds, bool fp64, int mode, int ct_n, void* stream) {
  if (ct_n) {
#define MONC_GROUP_TRY(K) \
  if (launch_xfwd_group_##K(a, grid, block, lds, fp64, mode, ct_n, stream)) return;
    MONC_FFT_GROUPS(MONC_GROUP_TRY)
#undef MONC_GROUP_TRY
    return;
  }
  if (fp64 && mode == 2) MONC_GO((k_xfwd_gen<double, 2>));
  else if (fp64 && mode == 3) MONC_GO((k_xfwd_gen<double, 3>));
  else if (fp64) MONC_GO((k_xfwd_gen<double, 0>));
  else if (mode == 0) MONC_GO((k_xfwd_gen<float, 0>));
  else if (mode == 1) MONC_GO((k_xfwd_gen<float, 1>));
  else if (mode == 2) MONC_GO((k_xfwd_gen<float, 2>));
  else MONC_GO((k_xfwd_gen<float, 3>));
}

void launch_ffty(const LaunchArgs& a, int grid, int block, size_t lds, bool fp64, bool inverse, int ct_n, int ept,
                 void* stream) {
  if (ct_n) {
#define MONC_GROUP_TRY(K) \
  if (launch_ffty_group_##K(a, grid, block, lds, fp64, inverse, ct_n, ept, stream)) return;
    MONC_FFT_GROUPS(MONC_GROUP_TRY)
#undef MONC_GROUP_TRY
    return;
  }
  if (fp64) {
    if (inverse) MONC_GO((k_ffty_gen<double, true>));
    else MONC_GO((k_ffty_gen<double, false>));
  } else {
    if (inverse) MONC_GO((k_ffty_gen<float, true>));
    else MONC_GO((k_ffty_gen<float, false>));
  }
}

void launch_xinv(const LaunchArgs& a, int grid, int block, size_t lds, bool fp64, int mode, int ct_n, void* stream) {
  if (ct_n) {
#define MONC_GROUP_TRY(K) \
  if (launch_xinv_group_##K(a, grid, block, lds, fp64, mode, ct_n, stream)) return;
    MONC_FFT_GROUPS(MONC_GROUP_TRY)
#undef MONC_GROUP_TRY
    return;
  }
  if (fp64 && mode == 3) MONC_GO((k_xinv_gen<double, 3>));
  else if (fp64) MONC_GO((k_xinv_gen<double, 0>));
  else if (mode == 0) MONC_GO((k_xinv_gen<float, 0>));
  else if (mode == 1) MONC_GO((k_xinv_gen<float, 1>));
  else if (mode == 2) MONC_GO((k_xinv_gen<float, 2>));
  else MONC_GO((k_xinv_gen<float, 3>));
}

void launch_grad(const LaunchArgs& a, int grid, bool fp64, int vec, bool red, void* stream) {
  const dim3 g(grid), b(256);
  hipStream_t st = (hipStream_t)stream;
#define MONC_GRAD(V)                                                                       \
  if (red) {                                                                               \
    if (fp64) hipLaunchKernelGGL((k_grad<double, V, true>), g, b, 0, st, a);               \
    else hipLaunchKernelGGL((k_grad<float, V, true>), g, b, 0, st, a);                     \
  } else {                                                                                 \
    if (fp64) hipLaunchKernelGGL((k_grad<double, V, false>), g, b, 0, st, a);              \
    else hipLaunchKernelGGL((k_grad<float, V, false>), g, b, 0, st, a);                    \
  }
  if (vec == 4) {
    MONC_GRAD(4)
  } else if (vec == 2) {
    MONC_GRAD(2)
  } else {
    MONC_GRAD(1)
  }
#undef MONC_GRAD
}

void launch_stats_init(double* stats, int nz, void* stream) {
  hipLaunchKernelGGL(k_stats_init, dim3((8 * nz + 255) / 256), dim3(256), 0, (hipStream_t)stream, stats, nz);
}

}  // namespace monc
