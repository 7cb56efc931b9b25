// Host-side helpers of the kernel launchers.
#pragma once
#include <hip/hip_runtime.h>

namespace monc {

template <typename K>
static void set_lds_limit(K kern) {
  (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                            160 * 1024);
}

}  // namespace monc

#define MONC_GO(kern) hipLaunchKernelGGL(kern, dim3(grid), dim3(block), lds, (hipStream_t)stream, a)
