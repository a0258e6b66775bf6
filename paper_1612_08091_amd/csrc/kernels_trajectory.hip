// Trajectory steps.  Between two channels of a noisy circuit only a gate or two
// wait (the branch taken of the channel before, the gate on the next qubit), so
// the pass that applies them also reduces the state to the density matrix of the
// channel's targets: a thread holds the 2^k amplitudes of a group over the
// qubits concerned (k <= 3), multiplies them by the product of the waiting
// gates and adds the targets' outer products, in double whatever the state's
// dtype.  Hermitian, so 4 or 16 sums per thread.  The workgroups' sums go to
// pinned host memory and the host, which decides the branch, adds them in
// order: one kernel per channel and no copy.  A call returns with the state in
// memory for every stream.  Where the host watches the sums of a pass that also
// writes the state, its workgroups therefore release them behind their waves'
// stores (see kReleaseBlocks); else it waits for the stream.
// Bound by HBM for large states (one read and one write), by the launch and the
// host's wait for small ones: on 16 qubits 4.3 us (two qubits) and 5.8 (three),
// about 14 us a channel with the host's part, against 53 as a tile pass, a
// reduction in two kernels and the upload of the pass.  (Workgroups of one wave
// there take 4.1 us, but leave the host four times the sums: no gain.)
#include <hip/hip_runtime.h>

#include <algorithm>

#include "trajectory.hpp"
#include "result_store.hpp"

namespace qsv {
namespace dev {

template <typename R> struct VG;
template <> struct VG<double> { using T = double2; };
template <> struct VG<float> { using T = float2; };

constexpr int kGT = 256;

template <typename R, int K>
struct GroupArgsT {
    uint64_t ngroups;
    uint32_t ins[3];            // the group's positions, ascending
    uint64_t off[1 << K];
    R ur[1 << (2 * K)], ui[1 << (2 * K)];
};

template <typename R, int K, int KT, bool APPLY>
__global__ __launch_bounds__(kGT) void k_group_rdm(typename VG<R>::T *__restrict__ psi,
                                                   GroupArgsT<R, K> a, double *__restrict__ out,
                                                   bool release) {
    using T = typename VG<R>::T;
    constexpr int D = 1 << K, DT = 1 << KT, W = KT == 1 ? 4 : 16;
    __shared__ double sh[kGT / 64][W];
    // The matrix comes with the kernel's arguments, which lie in host memory:
    // one load per thread and LDS, not a row of scalar loads that each cross to
    // the host (three qubits, 16 in all: 9.7 -> 5.8 us).  From LDS it goes to
    // registers for the whole loop: 256 of them for three qubits in complex128,
    // and still the faster (27 qubits 849 -> 811 us, read in the loop 866; 24
    // qubits 80.5 -> 82).
    __shared__ T mat[APPLY ? D * D : 1];
    if (APPLY) {
        if (threadIdx.x < D * D) {
            mat[threadIdx.x].x = a.ur[threadIdx.x];
            mat[threadIdx.x].y = a.ui[threadIdx.x];
        }
        __syncthreads();
    }
    double acc[W];
#pragma unroll
    for (int w = 0; w < W; ++w) acc[w] = 0.0;
    for (uint64_t g = (uint64_t)blockIdx.x * kGT + threadIdx.x; g < a.ngroups;
         g += (uint64_t)gridDim.x * kGT) {
        uint64_t base = g;
#pragma unroll
        for (int j = 0; j < K; ++j) {
            const uint64_t lowm = (1ull << a.ins[j]) - 1;
            base = ((base & ~lowm) << 1) | (base & lowm);
        }
        T x[D];
#pragma unroll
        for (int r = 0; r < D; ++r) x[r] = psi[base | a.off[r]];
        if (APPLY) {
            T y[D];
#pragma unroll
            for (int r = 0; r < D; ++r) {
                R yr = 0, yi = 0;
#pragma unroll
                for (int c = 0; c < D; ++c) {
                    const R mr = mat[r * D + c].x, mi = mat[r * D + c].y;
                    yr += mr * x[c].x - mi * x[c].y;
                    yi += mr * x[c].y + mi * x[c].x;
                }
                y[r].x = yr;
                y[r].y = yi;
            }
#pragma unroll
            for (int r = 0; r < D; ++r) {
                x[r] = y[r];
                psi[base | a.off[r]] = x[r];
            }
        }
#pragma unroll
        for (int rest = 0; rest < D; rest += DT) {
            int w = DT;
#pragma unroll
            for (int q = 0; q < DT; ++q) {
                const double br = x[rest + q].x, bi = x[rest + q].y;
                acc[q] += br * br + bi * bi;
#pragma unroll
                for (int p = 0; p < q; ++p) {
                    const double ar = x[rest + p].x, ai = x[rest + p].y;
                    acc[w] += ar * br + ai * bi;
                    acc[w + 1] += ai * br - ar * bi;
                    w += 2;
                }
            }
        }
    }
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (release) stores_arrived();
#pragma unroll
    for (int w = 0; w < W; ++w) {
        double v = acc[w];
        for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
        if (lane == 0) sh[wv][w] = v;
    }
    __syncthreads();
    if (threadIdx.x < W) {
        double v = 0.0;
        for (int i = 0; i < kGT / 64; ++i) v += sh[i][threadIdx.x];
        double *p = out + (size_t)blockIdx.x * W + threadIdx.x;
        if (release) result_release(p, v);
        else result_store(p, v);
    }
}

int group_blocks(const GroupArgs &a) {
    const uint64_t ngroups = 1ull << (a.nq - a.k);
    return (int)std::min<uint64_t>((ngroups + kGT - 1) / kGT,
                                   std::min(1024, kGroupSums / group_width(a.kt)));
}

template <typename R, int K, int KT>
static hipError_t group_rdm_t(void *psi, const GroupArgs &a, double *out, int *blocks,
                              hipStream_t s) {
    using T = typename VG<R>::T;
    constexpr int D = 1 << K;
    GroupArgsT<R, K> t{};
    t.ngroups = 1ull << (a.nq - K);
    for (int j = 0; j < K; ++j) t.ins[j] = a.pos[j];
    std::sort(t.ins, t.ins + K);
    for (int r = 0; r < D; ++r)
        for (int j = 0; j < K; ++j)
            if ((r >> j) & 1) t.off[r] |= 1ull << a.pos[j];
    for (int e = 0; e < D * D; ++e) {
        t.ur[e] = (R)a.ur[e];
        t.ui[e] = (R)a.ui[e];
    }
    const unsigned nb = (unsigned)group_blocks(a);
    *blocks = (int)nb;
    if (a.apply)
        hipLaunchKernelGGL((k_group_rdm<R, K, KT, true>), dim3(nb), dim3(kGT), 0, s, (T *)psi, t, out,
                           group_releases(a));
    else
        hipLaunchKernelGGL((k_group_rdm<R, K, KT, false>), dim3(nb), dim3(kGT), 0, s, (T *)psi, t, out,
                           false);
    return hipGetLastError();
}

template <typename R>
static hipError_t group_rdm_r(void *psi, const GroupArgs &a, double *out, int *blocks,
                              hipStream_t s) {
    switch (a.k * 4 + a.kt) {
    case 4 + 1: return group_rdm_t<R, 1, 1>(psi, a, out, blocks, s);
    case 8 + 1: return group_rdm_t<R, 2, 1>(psi, a, out, blocks, s);
    case 12 + 1: return group_rdm_t<R, 3, 1>(psi, a, out, blocks, s);
    case 8 + 2: return group_rdm_t<R, 2, 2>(psi, a, out, blocks, s);
    case 12 + 2: return group_rdm_t<R, 3, 2>(psi, a, out, blocks, s);
    }
    return hipErrorInvalidValue;
}

hipError_t group_rdm(int dtype, void *psi, const GroupArgs &a, double *out, int *blocks,
                     hipStream_t s) {
    if (a.nq < a.k) return hipErrorInvalidValue;
    return dtype == 0 ? group_rdm_r<double>(psi, a, out, blocks, s)
                      : group_rdm_r<float>(psi, a, out, blocks, s);
}

}  // namespace dev
}  // namespace qsv
