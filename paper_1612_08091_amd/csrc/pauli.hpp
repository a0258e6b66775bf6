// Pauli sums of a state: the host's plan and the launcher (implemented in
// pauli_plan.cpp and kernels_pauli.hip).
//
// <P> for a string with X letters at x and Z letters at z (Y in both) is
// i^{n_Y} sum_j conj(psi_{j^x}) psi_j (-1)^{popcount(j & z)}.  The members j
// and j ^ x of a pair give conjugate shares up to the sign (-1)^{n_Y}, so a
// pair adds 2 Re or 2 Im of conj(b) a, by the parity of n_Y, and the
// expectation value is real.
#pragma once

#include <hip/hip_runtime_api.h>

#include <cstdint>
#include <vector>

#include "device.hpp"

namespace qsv {
namespace dev {

constexpr int kPauliThreadBits = 9;
constexpr int kPauliRegBits = 3;
constexpr int kPauliTileBits = kPauliThreadBits + kPauliRegBits;
constexpr uint32_t kPauliNoPos = 64;    // a tile bit beyond a small state

// One string: its coefficient times i^{n_Y} and the pairs' factor, and its Z
// mask over the tile's thread bits, its register bits (as the sign of each
// register, bit i) and the positions outside the tile.
struct PauliTerm {
    double c;
    uint64_t zo;
    uint32_t zthr;
    uint32_t sreg;
};
// Strings with one X mask, over the tile's bits.  The first string is held in
// place: most groups have no other, and one burst of scalar loads (a 64-byte
// line) then brings all that a group needs.
struct PauliXGroup {
    PauliTerm first;
    uint32_t xthr, xreg;
    int32_t odd;            // n_Y odd: Im, else Re
    int32_t term0, terms;   // the others
    int32_t pad[5];
};
static_assert(sizeof(PauliXGroup) == 64, "a group is one line");
// A tile shape (positions of the local bits: 9 thread bits, then the register
// bits) and the groups whose X letters it holds; one row of the grid.
struct PauliSet {
    uint32_t tpos[16];      // by local bit
    uint32_t ins[16];       // the same positions, ascending, up to n_ins
    int32_t n_ins;
    int32_t group0, groups;
    uint32_t pad_thr, pad_reg;  // local bits beyond the state
    int32_t pad[3];
};
// Strings whose X letters fit in no tile, up to 8 with one X mask and one
// parity of n_Y, swept over the whole state.
constexpr int kPauliWide = 8;
struct PauliWideGroup {
    uint64_t x;
    int32_t hbit, odd, nt, pad;
    uint64_t z[kPauliWide];
    double c[kPauliWide];
};

struct PauliPlan {
    std::vector<PauliSet> sets;
    std::vector<PauliXGroup> groups;
    std::vector<PauliTerm> terms;
    std::vector<PauliWideGroup> wide;
    unsigned grid_x = 0;        // workgroups of a set
    unsigned wide_x = 0;        // workgroups of a wide group
    size_t partials() const { return (size_t)grid_x * sets.size() + (size_t)wide_x * wide.size(); }
};
void pauli_plan(int nq, int nterms, const uint64_t *x, const uint64_t *z,
                const double *c, PauliPlan &p);
// The plan's arrays as one block to upload.
size_t pauli_blob_bytes(const PauliPlan &p);
void pauli_blob(const PauliPlan &p, unsigned char *out);
// out[0] = the sum; ws holds p.partials() doubles.
hipError_t pauli_sum(int dtype, const void *psi, int nq, const PauliPlan &p, const void *blob,
                     double *ws, double *out, hipStream_t s);

}  // namespace dev
}  // namespace qsv
