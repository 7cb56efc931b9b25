// Launchers of the projection kernels (kernels.hip, fft_inst.hip, tridiag.hip,
// level.hip).
#pragma once
#include <stddef.h>

#include "monc_types.h"

namespace monc {

// Raise the dynamic-LDS limit of the kernels to the CU's 160 KB: of all but the
// compile-time FFT ones, and of those of length n (once per group of lengths).
void init_kernel_attributes();
void init_fft_attributes(int n);
void init_tridiag_attributes();  // the tridiagonal kernels' part of it
void init_level_attributes();    // the level kernels'

// Transform lengths with compile-time FFT kernels: every 2^a 3^b from 16 to
// 4096 (others take the runtime-length kernels). The kernels need blockDim =
// (transforms or columns per workgroup) * threads per transform (ct_threads_x_n,
// ct_threads_y_n). Their instances are compiled in groups, one object each
// (fft_inst.hip with MONC_FFT_GROUP = 0..7).
#define MONC_FFT_GROUPS(Y) Y(0) Y(1) Y(2) Y(3) Y(4) Y(5) Y(6) Y(7)
#define MONC_CT_GROUP_0(X) X(16) X(64) X(192) X(486) X(1024) X(2187)
#define MONC_CT_GROUP_1(X) X(18) X(72) X(216) X(512) X(1152) X(2304)
#define MONC_CT_GROUP_2(X) X(24) X(81) X(243) X(576) X(1296) X(2592)
#define MONC_CT_GROUP_3(X) X(27) X(96) X(256) X(648) X(1458) X(2916)
#define MONC_CT_GROUP_4(X) X(32) X(108) X(288) X(729) X(1536) X(3072)
#define MONC_CT_GROUP_5(X) X(36) X(128) X(324) X(768) X(1728) X(3456)
#define MONC_CT_GROUP_6(X) X(48) X(144) X(384) X(864) X(1944) X(3888)
#define MONC_CT_GROUP_7(X) X(54) X(162) X(432) X(972) X(2048) X(4096)
// Lengths with two y-FFT radix plans (8 or 16 elements per thread) are those
// without a plan of their own (ct_plan_index < 0).
// One group's instances: false if the group does not hold the length.
#define MONC_GROUP_DECL(K)                                                                                          \
  void init_fft_group_##K();                                                                                        \
  bool launch_xfwd_group_##K(const LaunchArgs& a, int grid, int block, size_t lds, bool fp64, int mode, int ct_n,   \
                             void* stream);                                                                         \
  bool launch_ffty_group_##K(const LaunchArgs& a, int grid, int block, size_t lds, bool fp64, bool inverse, int ct_n, \
                             int ept, void* stream);                                                                \
  bool launch_xinv_group_##K(const LaunchArgs& a, int grid, int block, size_t lds, bool fp64, int mode, int ct_n,   \
                             void* stream);

bool ct_supported(int n);
MONC_FFT_GROUPS(MONC_GROUP_DECL)
// lengths with the persistent FP32 y-FFT kernel (32 elements per thread)
bool pp_supported(int n);
inline int ct_threads_host(int n, int eb) { return ct_threads_x_n(n, eb); }
inline int ct_threads_y_host(int n, int ept) { return ct_threads_y_n(n, ept); }

// ct_n: the compile-time length, or 0 for the runtime-length kernel.
// mode 0: divergence of (u, v, w); mode 1 (float only): the FP64 residual
// D(u) - D(G p1) with the first-pass pressure p1 in io.s2; mode 2: the FP64
// field at io.u (nz, ny, nx), rounded to the storage type; mode 3 (one member):
// that field after io.u -= alpha io.v, alpha from the two scalars at io.w, with
// one partial sum of dz io.u^2 per workgroup into io.stats.
void launch_xfwd(const LaunchArgs& a, int grid, int block, size_t lds, bool fp64, int mode, int ct_n, void* stream);
// ept: elements per thread of the compile-time kernel (8 or 16; 32 = the
// persistent FP32 kernel, whose grid covers the CUs once)
void launch_ffty(const LaunchArgs& a, int grid, int block, size_t lds, bool fp64, bool inverse, int ct_n, int ept,
                 void* stream);
// rows: rows per lane, one of kTriRows (the member's tris)
void launch_tridiag(const LaunchArgs& a, int grid, int block, size_t lds, bool fp64, int rows, bool pairs, void* stream);
// the wave-per-chunk kernel (up to kTriColMax levels): rows per wave (the
// member's tcrows), block = 64 times the member's tcwaves
void launch_tricol(const LaunchArgs& a, int grid, int block, size_t lds, int rows, void* stream);
// the result goes to io.p (mode 0), io.s1 (mode 1, float only: the
// correction delta) or io.s2 (mode 2, float only: the first-pass pressure);
// mode 3 (one member): io.p, with one partial sum per workgroup of dz io.u io.p
// into io.stats and (float, io.v given) of dz io.p io.v into io.w
void launch_xinv(const LaunchArgs& a, int grid, int block, size_t lds, bool fp64, int mode, int ct_n, void* stream);
// both transforms of each level by one workgroup of `block` threads, for even ny
// and lengths of level_length along x and y (those below ept 16): modes as
// launch_xfwd's 0 and 1 and launch_xinv's 0, 1 and 2
bool level_length(int n, bool y);
void launch_level_fwd(const LaunchArgs& a, int grid, int block, size_t lds, bool fp64, int mode, void* stream);
void launch_level_inv(const LaunchArgs& a, int grid, int block, size_t lds, bool fp64, int mode, void* stream);
// fp64: pressure from io.p (FP64); else (mixed path) p1 + delta summed in
// FP64 from io.s2 + io.s1, and written rounded to io.p. vec: points per
// thread (2 needs an even nx, 4 a multiple of 4; else 1)
// red: also the per-level horizontal mean and max of u, v, w, p into io.stats
// (after launch_stats_init on the same stream)
void launch_grad(const LaunchArgs& a, int grid, bool fp64, int vec, bool red, void* stream);
void launch_stats_init(double* stats, int nz, void* stream);

}  // namespace monc
