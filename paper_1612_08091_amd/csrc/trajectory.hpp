// One step of a noise trajectory: gates waiting on few qubits and the reduced
// density matrix of the channel's targets in one pass (kernels_trajectory.hip).
#pragma once

#include <hip/hip_runtime_api.h>

#include <cstdint>

#include "device.hpp"

namespace qsv {
namespace dev {

constexpr int kGroupBits = 3;           // qubits of a group, at most
constexpr int kGroupSums = 8192;        // doubles of the workgroups' partial matrices, at most

// Group bit j is the qubit at bit position pos[j]; the kt <= 2 targets come
// first.  apply: psi <- U psi on the group (2^k x 2^k, row-major, bit j of an
// index = group bit j) before the reduction.
struct GroupArgs {
    int32_t nq, k, kt, apply;
    uint32_t pos[kGroupBits];
    double ur[64], ui[64];
};

// Doubles of a partial matrix: the diagonal, then re, im of rho[a][b], a < b,
// ordered by b, then a.
inline int group_width(int kt) { return kt == 1 ? 4 : 16; }
// Workgroups of the pass.
int group_blocks(const GroupArgs &a);
// With apply: whether the partial matrices are written behind the state's stores,
// so that the host may watch them; if not, it has to wait for the stream, which
// takes 4 us more.  Each workgroup that does so writes its XCD's L2 back: a step of
// one gate on two qubits and one channel takes 15.1 us so on 14 qubits (16
// workgroups) against 18.8 with the wait, 17.1 against 19.0 on 17 qubits (128), and
// as long on 18 (256).
constexpr int kReleaseBlocks = 128;
inline bool group_releases(const GroupArgs &a) { return a.apply && group_blocks(a) <= kReleaseBlocks; }
// One pass over the state; every workgroup writes its partial matrix to
// out[block * group_width(kt)] (host memory that the device writes), *blocks
// of them.
hipError_t group_rdm(int dtype, void *psi, const GroupArgs &a, double *out, int *blocks,
                     hipStream_t s);

}  // namespace dev
}  // namespace qsv
