// Device helpers shared by the projection's kernels.
#pragma once
#include <hip/hip_runtime.h>

#include "fft_core.h"
#include "monc_types.h"

namespace monc {

__device__ __forceinline__ int find_member(const LaunchArgs& a, int b) {
  int m = 0;
  while (m + 1 < a.nmem && b >= a.block_start[m + 1]) ++m;
  return m;
}

// The member a workgroup works on. The first member's entries have fixed
// places in the kernel arguments, so they are read together with the member
// count, and only a launch of several members searches.
struct Member {
  const MemberDesc* desc;
  IoPtrs io;
  int start, end;  // its blocks of the launch
};
__device__ __forceinline__ Member launch_member(const LaunchArgs& a, int block) {
  Member m{a.mem[0], a.io[0], 0, a.block_start[1]};
  const int n = a.nmem;
  // (an empty asm that takes them all: else each load sinks to its first use)
  asm volatile("" ::"s"(n), "s"(m.desc), "s"(m.end), "s"(m.io.u), "s"(m.io.v), "s"(m.io.w), "s"(m.io.p), "s"(m.io.spec),
               "s"(m.io.s1), "s"(m.io.s2), "s"(blockDim.x));
  if (n > 1) {
    const int i = find_member(a, block);
    m = Member{a.mem[i], a.io[i], a.block_start[i], a.block_start[i + 1]};
  }
  return m;
}

// The descriptor, read whole through the constant address space (scalar
// loads, all of them in flight at once): read field by field where each is
// used, the loads make a chain of round trips to memory, which is most of a
// small grid's kernel time.
__device__ __forceinline__ MemberDesc load_desc(const MemberDesc* p) {
  MemberDesc d;
  static_assert(sizeof(MemberDesc) % 8 == 0, "copied in 8-byte words");
  const auto* s = (const __attribute__((address_space(4))) unsigned long long*)p;
#pragma unroll
  for (int i = 0; i < (int)(sizeof(MemberDesc) / 8); ++i) reinterpret_cast<unsigned long long*>(&d)[i] = s[i];
  return d;
}
// Keeps the loads of the fields a kernel uses together, as in launch_member:
// those of the x, y, tridiagonal and gradient kernels.
__device__ __forceinline__ void keep_x(const MemberDesc& d) {
  asm volatile("" ::"s"(d.skip), "s"(d.nx), "s"(d.ny), "s"(d.nz), "s"(d.nxh), "s"(d.nrow), "s"(d.plane), "s"(d.rdx),
               "s"(d.rdy), "s"(d.rdxf), "s"(d.rdyf), "s"(d.lev), "s"(d.levf), "s"(d.twx), "s"(d.ptk), "s"(d.ptj),
               "s"(d.sbw), "s"(d.lbw), "s"(d.bst), "s"(d.ny_mul), "s"(d.ny_shift));
}
__device__ __forceinline__ void keep_tri(const MemberDesc& d) {
  asm volatile("" ::"s"(d.skip), "s"(d.ny), "s"(d.nz), "s"(d.nxh), "s"(d.nxp), "s"(d.plane), "s"(d.sbw), "s"(d.lbw),
               "s"(d.bst), "s"(d.bst_mul), "s"(d.bst_shift), "s"(d.triP), "s"(d.tricw), "s"(d.lamx), "s"(d.lamy),
               "s"(d.tra), "s"(d.trc), "s"(d.trr), "s"(d.inv_nxny));
}
__device__ __forceinline__ void keep_grad(const MemberDesc& d) {
  asm volatile("" ::"s"(d.nx), "s"(d.ny), "s"(d.nz), "s"(d.ptk), "s"(d.rdx), "s"(d.rdy), "s"(d.rdzc), "s"(d.nx_mul),
               "s"(d.nx_shift), "s"(d.ny_mul), "s"(d.ny_shift), "s"(d.nh_mul), "s"(d.nh_shift));
}
__device__ __forceinline__ void keep_y(const MemberDesc& d) {
  asm volatile("" ::"s"(d.skip), "s"(d.nxh), "s"(d.plane), "s"(d.twy), "s"(d.sbw), "s"(d.lbw), "s"(d.bst));
}

// Load through a global-address-space pointer (table pointers held in a
// descriptor are generic, which would otherwise become flat loads).
template <typename T>
__device__ __forceinline__ T ldg(const T* p) {
  return *(const __attribute__((address_space(1))) T*)p;
}

// x / d for 0 <= x < 2^31 with a precomputed multiplier: q = (umulhi(x, mul)
// + x) >> shift, where shift = ceil(log2 d) and mul = floor(2^32 (2^shift -
// d) / d) + 1 (division by invariant integers by multiplication, the variant
// with the extra addition, valid for every 31-bit dividend).
__device__ __forceinline__ unsigned fast_div(int x, unsigned mul, int shift) {
  const unsigned long long t = __umulhi((unsigned)x, mul);
  return (unsigned)((t + (unsigned)x) >> shift);
}

// Workgroups go to the 8 XCDs round-robin (XCD = blockIdx mod 8), each XCD
// with its own L2. Remap a member's local block index so that every XCD
// works through one contiguous range of tiles: neighbouring rows and levels,
// which the stencils read twice, then meet in the same L2. Applies when the
// member's first block sits on XCD 0; the tail beyond a multiple of 8 keeps
// its index.
__device__ __forceinline__ int xcd_local_block(int start, int end, int block) {
  const int lb = block - start;
  if (start & 7) return lb;
  const int full = (end - start) & ~7;
  if (lb >= full) return lb;
  return (lb & 7) * (full >> 3) + (lb >> 3);
}
__device__ __forceinline__ int xcd_local_block(const Member& m) { return xcd_local_block(m.start, m.end, blockIdx.x); }

// Wave-uniform read-only data: a scalar load.
template <typename T>
__device__ __forceinline__ T ldc(const T* p) {
  return *(const __attribute__((address_space(4))) T*)p;
}

// A descriptor with a skip flag drives the Krylov solver's preconditioner:
// once the solver has converged the flag is set and the solve's remaining
// launches return at once (whole workgroups, before any barrier).
__device__ __forceinline__ bool skipped(const MemberDesc& d) { return d.skip && ldc(d.skip) != 0.0; }

// Values known to be equal on every lane of a wave, moved to scalar
// registers (readfirstlane): a row context is per transform, and when a
// transform's thread count is a multiple of 64 it spans whole waves, so
// vector registers would hold the same value 64 times.
__device__ __forceinline__ int wuni(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ long long wuni(long long x) {
  const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)x);
  const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)((unsigned long long)x >> 32));
  return (long long)(((unsigned long long)hi << 32) | lo);
}
__device__ __forceinline__ double wuni(double x) { return __longlong_as_double(wuni(__double_as_longlong(x))); }
__device__ __forceinline__ float wuni(float x) { return __int_as_float(wuni(__float_as_int(x))); }
// Global-address-space views of a generic pointer (the scratch fields and
// the output pressure come from a by-value argument struct, so the compiler
// cannot infer their address space and would emit flat accesses).
template <typename T>
__device__ __forceinline__ __attribute__((address_space(1))) T* gptr(T* p) {
  return (__attribute__((address_space(1))) T*)p;
}

// (n, m) of the value at offset x (< ny * nxp) inside a level
__device__ __forceinline__ void spec_nm(const MemberDesc& d, int x, int& n, int& m) {
  const int b = (int)fast_div(x, d.bst_mul, d.bst_shift);
  const int rem = x - b * d.bst;
  n = rem >> d.lbw;
  m = (b << d.lbw) | (rem & (d.sbw - 1));
}

}  // namespace monc
