// Results that the host waits for by their values.
#pragma once

#include <hip/hip_runtime.h>

namespace qsv {
namespace dev {

// A word of a result in pinned host memory, visible to the host at once and not
// only at the kernel's end.
template <typename T> __device__ __forceinline__ void result_store(T *p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

}  // namespace dev
}  // namespace qsv
