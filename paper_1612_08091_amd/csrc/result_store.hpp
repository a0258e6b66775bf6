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

// s_waitcnt: no vector memory operation outstanding, the other counters as they are.
constexpr int kNoMemoryOut = 0x0f70;

// Before the barrier that such a word goes out behind: this wave's stores have
// arrived in the XCD's L2.
__device__ __forceinline__ void stores_arrived() { __builtin_amdgcn_s_waitcnt(kNoMemoryOut); }

// The same behind everything that the workgroup stored before its last barrier:
// the L2 is written back first.  (The wait is spelled out: the compiler drops the
// one that belongs to the write-back where it knows of no store in flight.)
template <typename T> __device__ __forceinline__ void result_release(T *p, T v) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "");
    __builtin_amdgcn_s_waitcnt(kNoMemoryOut);
    result_store(p, v);
}

}  // namespace dev
}  // namespace qsv
