// Both directions of a small level's transform in one kernel: the x and y
// transforms of one level by one workgroup.
#include <hip/hip_runtime.h>

#include "fft_kernels.h"
#include "launch.h"

namespace monc {

// The lengths (level_length), along y the even ones (a row pair of an odd ny
// spans two levels).
#define MONC_LEVEL_EVEN(X) X(16) X(18) X(24) X(32) X(36) X(48) X(54) X(64)
#define MONC_LEVEL_ODD(X) X(27)

// All row pairs of level k, then all its columns (forward), or the reverse.
// The half spectrum passes through the spectral buffer, written and read by the
// one workgroup, so the values and their order of operations are those of the
// separate kernels: the same bits. A length's threads (NT) need not divide the
// workgroup: the remaining threads form a last, partial transform that only
// takes part in the barriers (LDS holds it too).
template <typename T, int MODE, int N>
__device__ __forceinline__ void level_xfwd(const MemberDesc& d, const IoPtrs& io, int k) {
  constexpr int NT = ct_threads(N, sizeof(T));
  const int ipw = blockDim.x / NT, inst = threadIdx.x / NT, q = threadIdx.x - inst * NT, pairs = d.ny / 2;
  for (int p0 = 0; p0 < pairs; p0 += ipw) {
    if (p0) __syncthreads();
    const int p = p0 + inst;
    const bool in = inst < ipw && p < pairs;
    (void)xfwd_pair<T, MODE, N, true>(d, io, 0, ipw, inst, q, (long long)k * pairs + (in ? p : 0), in);
  }
}
template <typename T, int MODE, int N>
__device__ __forceinline__ void level_xinv(const MemberDesc& d, const IoPtrs& io, int k) {
  constexpr int NT = ct_threads(N, sizeof(T));
  using F = CtFft<T, N, NT, true>;
  extern __shared__ unsigned char smem_raw[];
  const int ipw = blockDim.x / NT, inst = threadIdx.x / NT, q = threadIdx.x - inst * NT, pairs = d.ny / 2;
  cx<T>* lds = reinterpret_cast<cx<T>*>(smem_raw) + inst * xlds_len(N, 2 * sizeof(T));
  for (int p0 = 0; p0 < pairs; p0 += ipw) {
    if (p0) __syncthreads();
    const bool part = inst < ipw && p0 + inst < pairs;
    const long long pair = (long long)k * pairs + (part ? p0 + inst : 0);
#include "xinv_pair.h"
  }
}
template <typename T, bool INV, int N>
__device__ __forceinline__ void level_y(const MemberDesc& d, const IoPtrs& io, int k) {
  constexpr int NT = ct_threads_y(N, 8);
  using F = CtFft<T, N, NT, INV>;
  extern __shared__ unsigned char smem_raw[];
  cx<T>* lds = reinterpret_cast<cx<T>*>(smem_raw);
  const int nc = blockDim.x / NT, mt = (blockDim.x + NT - 1) / NT;  // whole columns, columns in LDS
  const bool part = (int)threadIdx.x < nc * NT;
  const int c = part ? threadIdx.x % nc : nc, q = part ? threadIdx.x / nc : threadIdx.x - nc * NT;
  for (int m0 = 0; m0 < d.nxh; m0 += nc) {
    if (m0) __syncthreads();
    const int m = m0 + c;
#include "ffty_column.h"
  }
}

// A workgroup per level, threads for all its row pairs and columns at once up
// to 512. Small grids are bound by the launches (each about 2 us on the GPU and 4
// on the host) and by every kernel's chain of descriptor, row, twiddle and memory
// latencies; this halves the transforms' launches: a mixed projection of 32^3 takes
// 32.8 us on the GPU instead of 36.5, 64^2 x 32 39.8 instead of 46.4, FP64 32^3 20.7
// instead of 22.0; with a slower host, which then binds, the calls take 37 instead
// of 61 and 27 instead of 33.
template <typename T, int MODE>
__global__ void __launch_bounds__(512) k_level_fwd(LaunchArgs a) {
  const Member mb = launch_member(a, blockIdx.x);
  const MemberDesc d = load_desc(mb.desc);
  keep_x(d);
  const int k = blockIdx.x - mb.start;
  switch (d.nx) {
#define MONC_CASE(N) \
  case N: level_xfwd<T, MODE, N>(d, mb.io, k); break;
    MONC_LEVEL_EVEN(MONC_CASE)
    MONC_LEVEL_ODD(MONC_CASE)
#undef MONC_CASE
  }
  __syncthreads();  // the rows' spectra, in this workgroup's view of memory
  switch (d.ny) {
#define MONC_CASE(N) \
  case N: level_y<T, false, N>(d, mb.io, k); break;
    MONC_LEVEL_EVEN(MONC_CASE)
#undef MONC_CASE
  }
}

template <typename T, int MODE>
__global__ void __launch_bounds__(512) k_level_inv(LaunchArgs a) {
  const Member mb = launch_member(a, blockIdx.x);
  const MemberDesc d = load_desc(mb.desc);
  keep_x(d);
  const int k = blockIdx.x - mb.start;
  switch (d.ny) {
#define MONC_CASE(N) \
  case N: level_y<T, true, N>(d, mb.io, k); break;
    MONC_LEVEL_EVEN(MONC_CASE)
#undef MONC_CASE
  }
  __syncthreads();
  switch (d.nx) {
#define MONC_CASE(N) \
  case N: level_xinv<T, MODE, N>(d, mb.io, k); break;
    MONC_LEVEL_EVEN(MONC_CASE)
    MONC_LEVEL_ODD(MONC_CASE)
#undef MONC_CASE
  }
}

bool level_length(int n, bool y) {
  switch (n) {
#define MONC_CASE(N) case N:
    MONC_LEVEL_EVEN(MONC_CASE) return true;
    MONC_LEVEL_ODD(MONC_CASE) return !y;
#undef MONC_CASE
    default: return false;
  }
}

void init_level_attributes() {
  set_lds_limit(k_level_fwd<double, 0>);
  set_lds_limit(k_level_fwd<float, 0>);
  set_lds_limit(k_level_fwd<float, 1>);
  set_lds_limit(k_level_inv<double, 0>);
  set_lds_limit(k_level_inv<float, 1>);
  set_lds_limit(k_level_inv<float, 2>);
}

void launch_level_fwd(const LaunchArgs& a, int grid, int block, size_t lds, bool fp64, int mode, void* stream) {
  if (fp64) MONC_GO((k_level_fwd<double, 0>));
  else if (mode == 0) MONC_GO((k_level_fwd<float, 0>));
  else MONC_GO((k_level_fwd<float, 1>));
}

void launch_level_inv(const LaunchArgs& a, int grid, int block, size_t lds, bool fp64, int mode, void* stream) {
  if (fp64) MONC_GO((k_level_inv<double, 0>));
  else if (mode == 1) MONC_GO((k_level_inv<float, 1>));
  else MONC_GO((k_level_inv<float, 2>));
}

}  // namespace monc
