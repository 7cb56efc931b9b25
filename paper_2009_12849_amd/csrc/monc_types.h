// Shared host/device descriptors of the projection library.
//
// A launch covers one phase (e.g. "y-direction FFT") for a group of members
// (one member for monc_project, every member of a batch for
// monc_project_batched). Static per-member data (sizes, metric tables,
// twiddles, FFT plans, tile parameters, workspace) lives in a device array of
// MemberDesc; the per-call field pointers and the block ranges of the members
// travel by value in LaunchArgs (about 3.6 KB, under the 4 KB kernel-argument
// limit).
#pragma once
#include <stdint.h>

namespace monc {

constexpr int kMaxPass = 16;            // radix passes of one FFT (3^8 needs 8)
constexpr int kMaxLaunchMembers = 48;   // members per grouped launch (LaunchArgs under 4 KB)
constexpr int kTriSmax = 16;            // rows per lane in the tridiagonal solver
constexpr int kTriPmax = 64;            // lanes per column (one wave)
constexpr int kBig = 1 << 30;           // "inactive" lane index
constexpr int kGenericElems = 8;        // max elements per thread of the runtime-length FFT
constexpr int kSpecBlockMax = 8;        // widest spectral column block (nxp is a multiple of it)
// LDS slots (16 bytes each) per lane chunk of the tridiagonal solver, an odd
// count so that the chunks of consecutive lanes start in different bank
// groups. FP64 storage stages its S rows as FP64; FP32 storage keeps them as
// FP32 (8 bytes a row) and parks the S-2 eliminated FP64 right-hand sides
// over them, so the chunk holds the larger of the two.
constexpr int tri_lane_slots(int s, bool f32) {
  return f32 ? ((s + 1) / 2 > s - 2 ? (s + 1) / 2 : (s - 2 > 1 ? s - 2 : 1)) | 1 : s | 1;
}

// The tridiagonal kernel with FP32 storage, an even row count and tiles of at
// least 8 columns moves column pairs with 16-byte accesses (its own kernel
// instance): half the memory instructions for the same runs; narrower tiles
// measured slower that way.
constexpr bool tri_pairs(int s, int cw, bool f32) { return f32 && s % 2 == 0 && cw >= 8; }
// The wave-per-chunk tridiagonal kernel: at most 16 waves of at most 16 rows.
constexpr int kTriColMax = 256;
// LDS doubles of a workgroup of P waves: the interface rows (5), the chunks'
// last rows (4) and the interface solution (2), P x 64 each
constexpr int tricol_lds(int P) { return 11 * P * 64; }
// Threads per compile-time transform, shared by the kernels and the host's
// launch shapes, and so the radix plan (sixteen elements a thread take radix-16
// passes, eight radix-8 passes): kCtPlans, else ct_threads_x_n and ct_threads_y_n.
//
// Lengths with a factor 3 that have a radix plan of their own: threads per
// transform and the radices, along x and y alike. Radices 6, 9, 12, 16 and 18
// leave two passes up to 324 points and three above, four at 2187 (an LDS round
// trip and two barriers each), and the threads are chosen so that the passes'
// butterflies fill them where one count can: a thread holds 6 to 18 values, 20 at
// 1296 and 24 at 3888, whose last pass leaves some of its last round idle. The runtime-length kernels, which hold their butterflies in
// scratch memory and read the fields point by point, took 573 us for a whole
// 432 x 288 x 75 FP64 projection and 473 us for a 243 x 324 x 61 mixed one
// against 311 and 210 us.
struct CtPlan {
  int n, nt, np, r[4];
};
constexpr CtPlan kCtPlans[] = {
    {18, 3, 2, {6, 3}},
    {24, 2, 2, {6, 4}},
    {27, 3, 2, {9, 3}},
    {36, 6, 2, {6, 6}},
    {48, 4, 2, {12, 4}},
    {54, 6, 2, {9, 6}},
    {72, 6, 2, {12, 6}},
    {81, 9, 2, {9, 9}},
    {108, 6, 2, {18, 6}},
    {144, 12, 2, {12, 12}},
    {162, 9, 2, {18, 9}},
    {216, 18, 2, {18, 12}},
    {243, 27, 3, {9, 9, 3}},
    {288, 18, 2, {16, 18}},
    {324, 18, 2, {18, 18}},
    {432, 36, 3, {12, 12, 3}},
    {486, 27, 3, {9, 9, 6}},
    {576, 48, 3, {12, 12, 4}},
    {648, 36, 3, {18, 6, 6}},
    {729, 81, 3, {9, 9, 9}},
    {864, 72, 3, {12, 12, 6}},
    {972, 54, 3, {18, 18, 3}},
    {1152, 72, 3, {16, 18, 4}},
    {1296, 72, 3, {18, 18, 4}},
    {1458, 81, 3, {18, 9, 9}},
    {1728, 144, 3, {12, 12, 12}},
    {1944, 108, 3, {18, 18, 6}},
    {2187, 243, 4, {9, 9, 9, 3}},
    {2304, 144, 3, {16, 16, 9}},
    {2592, 216, 3, {18, 12, 12}},
    {2916, 162, 3, {18, 18, 9}},
    {3072, 256, 3, {16, 16, 12}},
    {3456, 288, 3, {16, 18, 12}},
    {3888, 216, 3, {18, 18, 12}},
};
constexpr int ct_plan_index(int n) {  // its place in kCtPlans, or -1
  for (int i = 0; i < (int)(sizeof(kCtPlans) / sizeof(CtPlan)); ++i)
    if (kCtPlans[i].n == n) return i;
  return -1;
}
//
// Along x, in storage type of eb bytes: eight elements a thread (radix-8 passes),
// sixteen (radix-16 passes, one exchange through LDS fewer) above length 768 in
// FP32 and above 2048 in FP64, whose transforms (16 bytes a value, 160 KB a CU)
// leave room for ten waves of sixteen-element threads but twenty of eight-element
// ones. The x kernels of a pass, sixteen -> eight elements a thread, us:
// FP64 512^2 x 96 291 -> 259, 768^2 x 64 452 -> 386, 1024^2 x 96 1033 -> 1005,
// 1536 x 768 x 64 839 -> 772, 2048^2 x 40 1832 -> 1782, but 4096 x 1024 x 32 1443 ->
// 1469; FP32 512^2 x 96 292 -> 285, 768^2 x 64 488 -> 442, but 1024^2 x 96 1124 ->
// 1208, 1536 x 768 x 64 921 -> 939.
constexpr int ct_threads_x_n(int n, int eb) {
  const int i = ct_plan_index(n);
  return i >= 0 ? kCtPlans[i].nt : n > (eb == 8 ? 2048 : 768) ? n / 16 : (n >= 8 ? n / 8 : 1);
}
// threads a transform that the acceptance of a requested x tile counts
constexpr int ct_threads_x_request(int n) {
  const int i = ct_plan_index(n);
  return i >= 0 ? kCtPlans[i].nt : n >= 512 ? n / 16 : (n >= 8 ? n / 8 : 1);
}
// Fewest transforms of nt threads that fill whole waves (64 lanes).
constexpr int wave_transforms(int nt) {
  int m = 1;
  while (m * nt % 64 != 0) m *= 2;
  return m;
}
// The residual's stencil phase at lengths whose transforms do not fill whole
// waves, are a multiple of 64 points and fit whole waves in 512 threads (64,
// 128, 192, 256, 384, 576, 768, 1536) walks whole rows per wave (64 lanes x
// xres_chunk points: 4 where the length allows, else 2, else 1), so that each
// wave handles one transform's rows at a time and its row contexts are
// wave-uniform; its workgroups then hold whole waves.
constexpr bool xres_wave_rows(int n) {
  const int nt = ct_threads_x_n(n, 4);
  return nt % 64 != 0 && n % 64 == 0 && wave_transforms(nt) * nt <= 512;
}
constexpr int xres_chunk(int n) { return n % 256 == 0 ? 4 : (n % 128 == 0 ? 2 : 1); }
// Points a lane takes at once of a row of n points in storage type of eb
// bytes: 16 bytes' worth where the row divides by it, else fewer.
constexpr int x_chunk(int n, int eb) { return n % (16 / eb) == 0 ? 16 / eb : n % 2 == 0 && eb == 4 ? 2 : 1; }
// Along y the elements per thread (8: radix-8 passes, 16: radix-16 passes)
// are a tile parameter: default sixteen from length 2048 on, eight below (FP64
// 512^2 x 96 684 us of the projection against 703, 2048^2 x 160 20845 against 20454;
// FP32 below 2048 within 1 %, with other roundings).
constexpr int ct_yept_default(int n) { return n >= 2048 ? 16 : 8; }
constexpr int ct_threads_y_n(int n, int ept) {
  const int i = ct_plan_index(n);
  return i >= 0 ? kCtPlans[i].nt : n >= ept ? n / ept : 1;
}
// lengths with the persistent FP32 y kernel (32 elements per thread)
constexpr bool pp_length(int n) { return n == 1024 || n == 1536 || n == 2048 || n == 4096; }
// columns per tile of the persistent FP32 y kernel (32 elements per thread,
// at most 512 threads)
constexpr int pp_columns(int n) { return n >= 32 ? 512 / (n / 32) : 1; }

// x-FFT LDS layout (shared by the kernels and the host's LDS sizes). For
// transforms with radix-16 passes (16 elements per thread), a bank row (256
// bytes: 2^bits complex values) is permuted by XOR of the value's index with
// the row number, which spreads the stride-16 writes over all banks at no LDS
// cost; other lengths (radix 8 and below, where it measured slower, or not
// whole bank rows) get one pad slot after every 2^shift values (128 bytes).
constexpr int kXswBits32 = 5;    // FP32 complex (8 B): 32 values per bank row
constexpr int kXswBits64 = 4;    // FP64 complex (16 B): 16 values per bank row
constexpr int kXpadShift32 = 4;
constexpr int kXpadShift64 = 3;
constexpr int xsw_bits(int cb) { return cb == 16 ? kXswBits64 : kXswBits32; }
constexpr bool xsw_on(int n, int cb) { return ct_threads_x_n(n, cb / 2) * 16 == n && n % (1 << xsw_bits(cb)) == 0; }
// LDS slots of one x transform of length n (complex values of cb bytes)
constexpr int xlds_len(int n, int cb) {
  return xsw_on(n, cb) ? n : n + (n >> (cb == 16 ? kXpadShift64 : kXpadShift32)) + 1;
}
// LDS slot of element i of an x transform of length n (a bijection of
// [0, n) into [0, xlds_len(n, cb)))
constexpr int xlds_index(int i, int n, int cb) {
  return xsw_on(n, cb) ? i ^ ((i >> xsw_bits(cb)) & ((1 << xsw_bits(cb)) - 1))
                       : i + (i >> (cb == 16 ? kXpadShift64 : kXpadShift32));
}

// values per level of the stencils' packed metrics: FP64 rho0, 1/dz, rhow of
// the top face (0 at the lid), rhow of the bottom face (0 at the bottom), 1/dzc
// above (0 at the lid) and below (0 at the bottom); FP32 the first four
constexpr int kLev64 = 6;
constexpr int kLev32 = 4;

struct FftPlan {
  int n;                  // transform length (2^a 3^b)
  int npass;              // number of Stockham passes
  int nt;                 // threads cooperating on one transform
  int rad[kMaxPass];      // radix of each pass (2, 3, 4 or 8)
};

struct MemberDesc {
  int nx, ny, nz;
  int nxh;                // nx/2 + 1 spectral values per row
  int nxp;                // padded count of m slots per spectral row (multiple of kSpecBlockMax)
  int dtype;              // 0 = FP64, 1 = mixed
  long long nrow;         // nz * ny real rows
  long long plane;        // complex values per level: ny * nxp, padded
  double rdx, rdy;        // 1/dx, 1/dy
  double inv_nxny;        // 1/(nx ny), the inverse-FFT normalisation
  double rH;              // 1 / sum(dz)
  double rSr;             // 1 / sum(dz rho0), the near-null deflation of the column solves
  double lamdef;          // columns with a smaller horizontal eigenvalue are deflated
  float rdxf, rdyf;       // FP32 copies for the FP32 stencil
  const double* lev;      // packed metrics (kLev64 doubles a level, 16-byte aligned)
  const float* levf;      // their FP32 copies (kLev32 floats a level)
  // FP64 vertical tables, all of length nz
  const double* rdz;      // 1/dz_k
  const double* rdzc;     // 1/dzc_k (0 at k = nz-1)
  const double* dz;       // dz_k (gauge weights)
  // The tridiagonal solver's rows, kTriPmax past nz: row k of the column with
  // eigenvalue lam reads tra_k P_{k-1} - (tra_k + trc_k + trr_k lam) P_k +
  // trc_k P_{k+1} (tra_0 = 0, trc_{nz-1} = 0). Rows past nz read P_k - P_{k-1} = 0 (tra 1, trc 0, trr 0):
  // nonsingular for every lam, and the lid (c_{nz-1} = 0) keeps them out of
  // the real rows, so a lane's rows need no range checks.
  const double* tra;
  const double* trc;
  const double* trr;
  // horizontal eigenvalues
  const double* lamx;     // [nxh]
  const double* lamy;     // [ny]
  // twiddles exp(-2 pi i t / n), complex in the storage precision
  const void* twx;        // [nx]
  const void* twy;        // [ny]
  FftPlan fx, fy;
  int ymt;                // y-FFT columns per workgroup
  int triP;               // tridiagonal lanes per column (power of 2)
  int tris;               // rows per lane (>= 2)
  int tricw;              // columns per workgroup (blockDim / triP)
  int tcwaves;            // waves of the wave-per-chunk kernel (0: FP64 storage, or tricol_shape's rule
                          // picks the lanes-per-column kernel)
  int tcrows;             // its rows per wave
  int ptk;                // levels per (level, row pair) tile of the stencil kernels (1 = row order)
  int ptj;                // row pairs per such tile of the x-forward kernels (8 to 64)
  int xpw;                // x-direction transforms (row pairs) per workgroup of the compile-time kernels
  int yept;               // elements per thread of the compile-time y-FFT kernels (8 or 16)
  // Spectral layout: a level's half spectrum sits in column blocks of sbw
  // consecutive m (the y-FFT tile width), each block row-major over n:
  // element (k, n, m) at k*plane + (m >> lbw)*bst + n*sbw + (m & (sbw-1)).
  int sbw;                // block width, a power of 2 <= kSpecBlockMax (divides nxp)
  int lbw;                // log2 sbw
  int bst;                // elements per block of a level: ny * sbw
  unsigned bst_mul;       // x / bst = (umulhi(x, bst_mul) + x) >> bst_shift for 31-bit x
  int bst_shift;
  unsigned nx_mul, ny_mul, nh_mul;    // the same for nx, ny and nx ny
  int nx_shift, ny_shift, nh_shift;
  void* spec;             // spectral workspace, nz levels of `plane` complex values
  // null, or (the preconditioner's copy of the descriptor) the Krylov
  // solver's converged flag: while *skip != 0 the FFT and tridiagonal
  // kernels do nothing
  const double* skip;
};

struct IoPtrs {
  void* u = nullptr;
  void* v = nullptr;
  void* w = nullptr;
  void* p = nullptr;
  void* spec = nullptr;     // spectral buffer used by this launch
  double* stats = nullptr;  // per-level horizontal mean and max of u, v, w, p, or null
  // mixed path, two float fields (nz, ny, nx) of scratch: s2 holds the
  // first-pass pressure p1, s1 the refinement's correction delta
  float* s1 = nullptr;
  float* s2 = nullptr;
};

struct LaunchArgs {
  int nmem;
  int block_start[kMaxLaunchMembers + 1];
  const MemberDesc* mem[kMaxLaunchMembers];  // device descriptors
  IoPtrs io[kMaxLaunchMembers];
};
static_assert(sizeof(LaunchArgs) <= 4096, "kernel arguments are limited to 4 KB");

}  // namespace monc
