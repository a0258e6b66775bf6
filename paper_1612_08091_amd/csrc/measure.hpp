// Measurement of several qubits in one call: plain-data arguments and the
// launcher (implemented in kernels_measure.hip).
#pragma once

#include <hip/hip_runtime_api.h>

#include <cstdint>

#include "device.hpp"

namespace qsv {
namespace dev {

// Qubits at bit positions pos[0..m-1], measured in list order with the
// uniforms u[0..m-1].
struct MeasureArgs {
    int32_t nq;
    int32_t m;
    uint32_t pos[40];
    double u[40];
};

// The branch taken so far: amplitudes with (index & mask) == val are kept.
// status 0, or 1 when a weight on the way was not an ordinary positive number
// (zero, denormal, infinite or NaN): the state is then left as it was.
struct MeasureBranch {
    uint64_t mask, val;
    double scale;
    int64_t status;
};

size_t measure_workspace_bytes();
// Enqueue the whole measurement of a state: the branch, then the collapse.
// *out (host memory that the device can write) receives the branch; valid
// once the stream is waited for.  *launches: kernels enqueued.
hipError_t measure(int dtype, void *psi, const MeasureArgs &a, void *ws, MeasureBranch *out,
                   int *launches, hipStream_t s);

}  // namespace dev
}  // namespace qsv
