// Emulated math gate as one gather pass: every output amplitude reads the
// amplitude whose register value the table maps onto its own.  Writes are
// contiguous; reads follow the permutation (contiguous runs when the table
// shifts values, as AddConstant does).  One read and one write of the state
// plus 4 bytes of inverse table per amplitude, which stay in cache for small
// registers: an HBM-bound pass.
//
// A result that has to lie where the state did costs a second pass to copy it
// back.  Under controls both passes leave the other amplitudes alone: the
// controlled ones are gathered into a packed buffer and put back from it, so
// with c controls the two move 4 / 2^c of the state (half a line's bytes where a
// control is one of the lowest bits, and then its lines whole) instead of 4.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "math_gate.hpp"

namespace qsv {
namespace dev {

template <typename R> struct VM;
template <> struct VM<double> { using T = double2; };
template <> struct VM<float> { using T = float2; };

constexpr int kMT = 256;

// Index of the amplitude that gate `a` moves to index j (all controls set).
__device__ __forceinline__ uint64_t math_source(uint64_t j, const MathArgs &a,
                                                const uint32_t *__restrict__ inv) {
    uint64_t d = 0;
    if (a.shift >= 0) {
        const uint32_t y = (uint32_t)(j >> a.shift) & (uint32_t)((1ull << a.w) - 1);
        d = (uint64_t)inv[y] << a.shift;
    } else {
        uint32_t y = 0;
        for (int b = 0; b < a.w; ++b) y |= (uint32_t)((j >> a.pos[b]) & 1u) << b;
        const uint32_t x = inv[y];
        for (int b = 0; b < a.w; ++b) d |= (uint64_t)((x >> b) & 1u) << a.pos[b];
    }
    return (j & ~a.regmask) | d;
}

template <typename R>
__global__ __launch_bounds__(kMT) void k_math_gather(const typename VM<R>::T *__restrict__ in,
                                                     typename VM<R>::T *__restrict__ out,
                                                     uint64_t dim, MathArgs a,
                                                     const uint32_t *__restrict__ inv) {
    for (uint64_t j = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; j < dim;
         j += (uint64_t)gridDim.x * blockDim.x)
        out[j] = in[(j & a.ctrl) == a.ctrl ? math_source(j, a, inv) : j];
}

// The i-th index with all controls set.
__device__ __forceinline__ uint64_t controlled_index(uint64_t i, const MathArgs &a) {
    for (int b = 0; b < a.nc; ++b) {
        const uint64_t low = (1ull << a.cpos[b]) - 1;
        i = ((i & ~low) << 1) | (i & low);
    }
    return i | a.ctrl;
}

// GET: buf[i] = psi[source of the i-th controlled index]; else psi[that index] =
// buf[i].
template <typename R, bool GET>
__global__ __launch_bounds__(kMT) void k_math_part(typename VM<R>::T *__restrict__ psi,
                                                   typename VM<R>::T *__restrict__ buf,
                                                   uint64_t count, MathArgs a,
                                                   const uint32_t *__restrict__ inv) {
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count;
         i += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t j = controlled_index(i, a);
        if (GET) buf[i] = psi[math_source(j, a, inv)];
        else psi[j] = buf[i];
    }
}

template <typename R>
static hipError_t in_place_t(void *psi, void *buf, uint64_t count, const MathArgs &a,
                             const uint32_t *inv, hipStream_t s) {
    using T = typename VM<R>::T;
    const dim3 g((unsigned)std::min<uint64_t>((count + kMT - 1) / kMT, 1ull << 20));
    hipLaunchKernelGGL((k_math_part<R, true>), g, dim3(kMT), 0, s, (T *)psi, (T *)buf, count, a, inv);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_math_part<R, false>), g, dim3(kMT), 0, s, (T *)psi, (T *)buf, count, a, inv);
    return hipGetLastError();
}

hipError_t math_in_place(int dtype, void *psi, void *buf, uint64_t dim, const MathArgs &a,
                         const uint32_t *inv, hipStream_t s) {
    if (a.w < 1 || a.w > kMaxMathBits || a.nc < 0 || a.nc > 63 || !psi || !buf || !inv)
        return hipErrorInvalidValue;
    return dtype == 0 ? in_place_t<double>(psi, buf, dim >> a.nc, a, inv, s)
                      : in_place_t<float>(psi, buf, dim >> a.nc, a, inv, s);
}

hipError_t math_gather(int dtype, const void *in, void *out, uint64_t dim, const MathArgs &a,
                       const uint32_t *inv, hipStream_t s) {
    if (a.w < 1 || a.w > kMaxMathBits || !in || !out || !inv) return hipErrorInvalidValue;
    const dim3 g((unsigned)std::min<uint64_t>((dim + kMT - 1) / kMT, 1ull << 20));
    if (dtype == 0)
        hipLaunchKernelGGL(k_math_gather<double>, g, dim3(kMT), 0, s, (const double2 *)in,
                           (double2 *)out, dim, a, inv);
    else
        hipLaunchKernelGGL(k_math_gather<float>, g, dim3(kMT), 0, s, (const float2 *)in,
                           (float2 *)out, dim, a, inv);
    return hipGetLastError();
}

}  // namespace dev
}  // namespace qsv
