// One group of the FFT kernels' compile-time lengths (MONC_FFT_GROUP): their
// instances, LDS limits and launches.
#include <hip/hip_runtime.h>

#include "fft_kernels.h"
#include "launch.h"

#define MONC_CAT2(A, B) A##B
#define MONC_CAT(A, B) MONC_CAT2(A, B)
#define MONC_SIZES MONC_CAT(MONC_CT_GROUP_, MONC_FFT_GROUP)
#define MONC_NAME(F) MONC_CAT(F##_group_, MONC_FFT_GROUP)

namespace monc {

template <int N>
static void init_length() {
  set_lds_limit(k_xfwd_ct<double, 0, N>);
  set_lds_limit(k_xfwd_ct<float, 0, N>);
  set_lds_limit(k_xfwd_ct<float, 1, N>);
  set_lds_limit(k_xfwd_ct<double, 2, N>);
  set_lds_limit(k_xfwd_ct<float, 2, N>);
  set_lds_limit(k_xfwd_ct<double, 3, N>);
  set_lds_limit(k_xfwd_ct<float, 3, N>);
  set_lds_limit(k_ffty_ct<double, false, N, 8>);
  set_lds_limit(k_ffty_ct<double, true, N, 8>);
  set_lds_limit(k_ffty_ct<float, false, N, 8>);
  set_lds_limit(k_ffty_ct<float, true, N, 8>);
  if constexpr (ct_plan_index(N) < 0) {
    set_lds_limit(k_ffty_ct<double, false, N, 16>);
    set_lds_limit(k_ffty_ct<double, true, N, 16>);
    set_lds_limit(k_ffty_ct<float, false, N, 16>);
    set_lds_limit(k_ffty_ct<float, true, N, 16>);
  }
  if constexpr (pp_length(N)) {
    set_lds_limit(k_ffty_pp<false, N>);
    set_lds_limit(k_ffty_pp<true, N>);
  }
  set_lds_limit(k_xinv_ct<double, 0, N>);
  set_lds_limit(k_xinv_ct<float, 0, N>);
  set_lds_limit(k_xinv_ct<float, 1, N>);
  set_lds_limit(k_xinv_ct<float, 2, N>);
  set_lds_limit(k_xinv_ct<double, 3, N>);
  set_lds_limit(k_xinv_ct<float, 3, N>);
}

void MONC_NAME(init_fft)() {
#define MONC_CASE(N) init_length<N>();
  MONC_SIZES(MONC_CASE)
#undef MONC_CASE
}

template <int N>
static void xfwd_length(const LaunchArgs& a, int grid, int block, size_t lds, bool fp64, int mode, void* stream) {
  if (fp64 && mode == 2) MONC_GO((k_xfwd_ct<double, 2, N>));
  else if (fp64 && mode == 3) MONC_GO((k_xfwd_ct<double, 3, N>));
  else if (fp64) MONC_GO((k_xfwd_ct<double, 0, N>));
  else if (mode == 0) MONC_GO((k_xfwd_ct<float, 0, N>));
  else if (mode == 1) MONC_GO((k_xfwd_ct<float, 1, N>));
  else if (mode == 2) MONC_GO((k_xfwd_ct<float, 2, N>));
  else MONC_GO((k_xfwd_ct<float, 3, N>));
}

// elements per thread (the radix plan) of a length without a plan of its own
template <int N, int EPT>
static void ffty_ept(const LaunchArgs& a, int grid, int block, size_t lds, bool fp64, bool inverse, void* stream) {
  if (fp64) {
    if (inverse) MONC_GO((k_ffty_ct<double, true, N, EPT>));
    else MONC_GO((k_ffty_ct<double, false, N, EPT>));
  } else {
    if (inverse) MONC_GO((k_ffty_ct<float, true, N, EPT>));
    else MONC_GO((k_ffty_ct<float, false, N, EPT>));
  }
}

template <int N>
static void ffty_length(const LaunchArgs& a, int grid, int block, size_t lds, bool fp64, bool inverse, int ept,
                        void* stream) {
  if constexpr (pp_length(N)) {
    if (ept == 32 && !fp64) {
      if (inverse) MONC_GO((k_ffty_pp<true, N>));
      else MONC_GO((k_ffty_pp<false, N>));
      return;
    }
  }
  if constexpr (ct_plan_index(N) < 0) {
    if (ept == 16) {
      ffty_ept<N, 16>(a, grid, block, lds, fp64, inverse, stream);
      return;
    }
  }
  ffty_ept<N, 8>(a, grid, block, lds, fp64, inverse, stream);
}

template <int N>
static void xinv_length(const LaunchArgs& a, int grid, int block, size_t lds, bool fp64, int mode, void* stream) {
  if (fp64 && mode == 3) MONC_GO((k_xinv_ct<double, 3, N>));
  else if (fp64) MONC_GO((k_xinv_ct<double, 0, N>));
  else if (mode == 0) MONC_GO((k_xinv_ct<float, 0, N>));
  else if (mode == 1) MONC_GO((k_xinv_ct<float, 1, N>));
  else if (mode == 2) MONC_GO((k_xinv_ct<float, 2, N>));
  else MONC_GO((k_xinv_ct<float, 3, N>));
}

bool MONC_NAME(launch_xfwd)(const LaunchArgs& a, int grid, int block, size_t lds, bool fp64, int mode, int ct_n,
                            void* stream) {
  switch (ct_n) {
#define MONC_CASE(N) \
  case N: xfwd_length<N>(a, grid, block, lds, fp64, mode, stream); return true;
    MONC_SIZES(MONC_CASE)
#undef MONC_CASE
    default: return false;
  }
}

bool MONC_NAME(launch_ffty)(const LaunchArgs& a, int grid, int block, size_t lds, bool fp64, bool inverse, int ct_n,
                            int ept, void* stream) {
  switch (ct_n) {
#define MONC_CASE(N) \
  case N: ffty_length<N>(a, grid, block, lds, fp64, inverse, ept, stream); return true;
    MONC_SIZES(MONC_CASE)
#undef MONC_CASE
    default: return false;
  }
}

bool MONC_NAME(launch_xinv)(const LaunchArgs& a, int grid, int block, size_t lds, bool fp64, int mode, int ct_n,
                            void* stream) {
  switch (ct_n) {
#define MONC_CASE(N) \
  case N: xinv_length<N>(a, grid, block, lds, fp64, mode, stream); return true;
    MONC_SIZES(MONC_CASE)
#undef MONC_CASE
    default: return false;
  }
}

}  // namespace monc
