// Measurement of a list of qubits (App. A.1, one uniform each, in order).
//
// The outcome of qubit j needs the weights of its two values within the
// branch that qubits 0..j-1 left.  Those weights come from one histogram over
// several qubits at once, and the branch keeps only 2^-r of the state after r
// qubits, so the reads are S + S/16 + S/256 + ... for a state of S bytes and
// the state is written once, at the end: about 2 S in all, whatever the number
// of qubits (a sweep to sum and a sweep to collapse per qubit would be 3 S
// each).  Bound by HBM.  25 qubits of a 25-qubit complex128 state, in list order
// drawn at random: 0.27 ms in 8 kernels and one wait (histograms 0.167,
// decisions 0.023, tail 0.013, collapse 0.065 ms), against 6.6 ms in 75 kernels
// and 25 waits as a sum and a collapse per qubit.
//
//  * k_measure_hist: weights of the 2^r values of the next r <= 4 qubits.
//    Qubits at positions >= 6 are unrolled over (2^H loads in flight per
//    thread), those below are lane bits, so that every load is contiguous
//    over the wave whichever qubits are measured.
//  * k_measure_decide: adds the blocks' weights in a fixed order and takes r
//    outcomes.
//  * k_measure_tail: once the branch has at most 2^13 amplitudes, one
//    workgroup resolves every qubit left: a binary tree of weights in LDS
//    whose top levels are the qubits in order, walked from the root.
//  * k_measure_collapse: zeroes or scales every amplitude; reads only those
//    it keeps.
// Weights are accumulated in double whatever the state's dtype.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "measure.hpp"

namespace qsv {
namespace dev {

template <typename R> struct VMs;
template <> struct VMs<double> { using T = double2; };
template <> struct VMs<float> { using T = float2; };

constexpr int kMeasThreads = 256;
constexpr int kMeasBlocks = 1024;
constexpr int kMeasRound = 4;       // qubits per histogram
constexpr int kMeasLane = 6;        // positions below are lane bits
constexpr int kTailBits = 13;
constexpr int kTailThreads = 1024;
constexpr size_t kBranchBytes = 256;

// g with a zero bit inserted at each of the npos ascending positions ins.
__device__ __forceinline__ uint64_t insert_zeros(uint64_t g, const uint32_t *ins, int npos) {
    for (int i = 0; i < npos; ++i) {
        const uint64_t lowm = (1ull << ins[i]) - 1;
        g = ((g & ~lowm) << 1) | (g & lowm);
    }
    return g;
}

struct HistArgs {
    uint64_t ngroups;
    int32_t nins;           // zeros to insert: positions decided before and this round's high ones
    uint32_t ins[40];       // ascending
    uint32_t hpos[4];       // this round's positions >= kMeasLane (H of them)
    uint32_t lpos[4];       // and those below (nl of them)
    int32_t nl;
    int32_t first;          // nothing decided before
};

// partial[block * 16 + bin]: bin bit j = bit hpos[j] for j < H, then lpos.
template <typename R, int H>
__global__ __launch_bounds__(kMeasThreads) void k_measure_hist(
    const typename VMs<R>::T *__restrict__ psi, HistArgs a,
    const MeasureBranch *__restrict__ br, double *__restrict__ partial) {
    using T = typename VMs<R>::T;
    constexpr int NB = 1 << H;
    constexpr int U = NB >= 8 ? 1 : 8 / NB;     // groups in flight: at least 8 loads per thread
    __shared__ double sh[kMeasThreads / 64][16];
    const uint64_t val = a.first ? 0ull : br->val;
    double acc[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[b] = 0.0;
    uint64_t off[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        off[b] = 0;
#pragma unroll
        for (int j = 0; j < H; ++j)
            if ((b >> j) & 1) off[b] |= 1ull << a.hpos[j];
    }
    const uint64_t stride = (uint64_t)gridDim.x * kMeasThreads;
    for (uint64_t g0 = (uint64_t)blockIdx.x * kMeasThreads + threadIdx.x; g0 < a.ngroups;
         g0 += stride * U) {
        T v[U][NB];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint64_t g = g0 + (uint64_t)u * stride;
            const bool in = g < a.ngroups;
            const uint64_t i = insert_zeros(in ? g : g0, a.ins, a.nins) | val;
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                v[u][b] = psi[i | off[b]];
                if (!in) v[u][b].x = v[u][b].y = R(0);
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int b = 0; b < NB; ++b)
                acc[b] += (double)v[u][b].x * v[u][b].x + (double)v[u][b].y * v[u][b].y;
    }
    // Lane bit l of the group id is index bit l unless zeros were inserted
    // below it; lpos holds the lane bits (host: positions within the group id).
    const uint32_t lane = threadIdx.x & 63u, w = threadIdx.x >> 6;
    uint32_t lmask = 0;
    for (int j = 0; j < a.nl; ++j) lmask |= 1u << a.lpos[j];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        double x = acc[b];
        for (uint32_t o = 32; o > 0; o >>= 1)
            if (!(lmask & o)) x += __shfl_xor(x, (int)o, 64);
        if (!(lane & ~lmask)) {     // one lane per value of the lane bits
            uint32_t bin = (uint32_t)b;
            for (int j = 0; j < a.nl; ++j) bin |= ((lane >> a.lpos[j]) & 1u) << (H + j);
            sh[w][bin] = x;
        }
    }
    __syncthreads();
    const int bins = 1 << (H + a.nl);
    if ((int)threadIdx.x < bins) {
        double x = 0.0;
        for (int i = 0; i < kMeasThreads / 64; ++i) x += sh[i][threadIdx.x];
        partial[(size_t)blockIdx.x * 16 + threadIdx.x] = x;
    }
}

// One outcome: 0 iff u (p0 + p1) < p0.  Weights that are not ordinary positive
// numbers set the status.
__device__ __forceinline__ int measure_pick(double u, double p0, double p1, double &keep,
                                            int64_t &status) {
    const double t = p0 + p1;
    if (!(t > 1e-280) || !(t < 1e300)) status = 1;
    const int o = u * t < p0 ? 0 : 1;
    keep = o ? p1 : p0;
    if (!(keep > 1e-280)) status = 1;
    return o;
}

struct DecideArgs {
    int32_t nblocks, r;
    int32_t first;
    uint32_t pos[4];        // positions of the r qubits, in order
    uint32_t bin[4];        // bin bit of each
    double u[4];
};

// 64 rows of 16 bins, four loads of a thread in flight: the partial sums of
// 1024 blocks arrive in 4 round trips.
__global__ __launch_bounds__(1024) void k_measure_decide(const double *__restrict__ partial,
                                                         DecideArgs a, MeasureBranch *br,
                                                         MeasureBranch *out) {
    __shared__ double sh[64][17];
    __shared__ double w[16];
    const int bin = threadIdx.x & 15, row = threadIdx.x >> 4;
    const int bins = 1 << a.r;
    double x = 0.0;
    if (bin < bins)
        for (int b = row; b < a.nblocks; b += 256) {
            double v[4];
#pragma unroll
            for (int k = 0; k < 4; ++k)
                v[k] = b + 64 * k < a.nblocks ? partial[(size_t)(b + 64 * k) * 16 + bin] : 0.0;
            x += (v[0] + v[1]) + (v[2] + v[3]);
        }
    sh[row][bin] = x;
    __syncthreads();
    if (row < 4) {
        double t = 0.0;
#pragma unroll
        for (int i = 0; i < 16; ++i) t += sh[row * 16 + i][bin];
        sh[row * 16][bin] = t;      // own row group: read before, by this thread alone
    }
    __syncthreads();
    if (threadIdx.x < 16) w[bin] = (sh[0][bin] + sh[16][bin]) + (sh[32][bin] + sh[48][bin]);
    __syncthreads();
    if (threadIdx.x != 0) return;
    MeasureBranch b;
    if (a.first) b = MeasureBranch{0, 0, 1.0, 0};
    else b = *br;
    uint32_t kmask = 0, kval = 0;
    double keep = 0.0;
    for (int j = 0; j < a.r; ++j) {
        double p[2] = {0.0, 0.0};
        for (int i = 0; i < bins; ++i)
            if (((uint32_t)i & kmask) == kval) p[(i >> a.bin[j]) & 1] += w[i];
        const int o = measure_pick(a.u[j], p[0], p[1], keep, b.status);
        kmask |= 1u << a.bin[j];
        kval |= (uint32_t)o << a.bin[j];
        b.mask |= 1ull << a.pos[j];
        b.val |= (uint64_t)o << a.pos[j];
    }
    b.scale = 1.0 / sqrt(keep);
    *br = b;
    *out = b;
}

struct TailArgs {
    int32_t bits, r;        // log2 of the branch's amplitudes; qubits left
    int32_t first;
    uint32_t pos[40];       // index position of local bit i: the unmeasured positions, then the
                            // qubits left, the first of them highest
    double u[40];           // in order
};

template <typename R>
__global__ __launch_bounds__(kTailThreads) void k_measure_tail(
    const typename VMs<R>::T *__restrict__ psi, TailArgs a, MeasureBranch *br,
    MeasureBranch *out) {
    // tree[1] the root, children of node k at 2 k and 2 k + 1, the leaves
    // (amplitude weights) at 2^bits + local index
    extern __shared__ __align__(16) unsigned char smem_m[];
    double *tree = reinterpret_cast<double *>(smem_m);
    MeasureBranch b;
    if (a.first) b = MeasureBranch{0, 0, 1.0, 0};
    else b = *br;
    const uint32_t size = 1u << a.bits;
    for (uint32_t l = threadIdx.x; l < size; l += kTailThreads) {
        uint64_t i = b.val;
        for (int t = 0; t < a.bits; ++t) i |= (uint64_t)((l >> t) & 1u) << a.pos[t];
        const auto v = psi[i];
        tree[size + l] = (double)v.x * v.x + (double)v.y * v.y;
    }
    __syncthreads();
    for (uint32_t level = size >> 1; level > 0; level >>= 1) {
        for (uint32_t k = threadIdx.x; k < level; k += kTailThreads)
            tree[level + k] = tree[2 * (level + k)] + tree[2 * (level + k) + 1];
        __syncthreads();
    }
    if (threadIdx.x != 0) return;
    uint32_t node = 1;
    double keep = 0.0;
    for (int j = 0; j < a.r; ++j) {
        const int o = measure_pick(a.u[j], tree[2 * node], tree[2 * node + 1], keep, b.status);
        node = 2 * node + (uint32_t)o;
        const uint32_t p = a.pos[a.bits - 1 - j];
        b.mask |= 1ull << p;
        b.val |= (uint64_t)o << p;
    }
    b.scale = 1.0 / sqrt(keep);
    *br = b;
    *out = b;
}

template <typename R>
__global__ __launch_bounds__(256) void k_measure_collapse(typename VMs<R>::T *__restrict__ psi,
                                                          uint64_t dim,
                                                          const MeasureBranch *__restrict__ br) {
    const MeasureBranch b = *br;
    if (b.status) return;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < dim;
         i += (uint64_t)gridDim.x * blockDim.x) {
        typename VMs<R>::T v;
        v.x = v.y = R(0);
        if ((i & b.mask) == b.val) {
            const auto x = psi[i];
            v.x = (R)((double)x.x * b.scale);
            v.y = (R)((double)x.y * b.scale);
        }
        psi[i] = v;
    }
}

size_t measure_workspace_bytes() { return kBranchBytes + sizeof(double) * 16 * kMeasBlocks; }

template <typename R, int H>
static void launch_hist(const void *psi, const HistArgs &h, unsigned nb, const MeasureBranch *br,
                        double *partial, hipStream_t s) {
    hipLaunchKernelGGL((k_measure_hist<R, H>), dim3(nb), dim3(kMeasThreads), 0, s,
                       (const typename VMs<R>::T *)psi, h, br, partial);
}

template <typename R>
static hipError_t measure_t(void *psi, const MeasureArgs &a, void *ws, MeasureBranch *out,
                            int *launches, hipStream_t s) {
    MeasureBranch *br = static_cast<MeasureBranch *>(ws);
    double *partial = reinterpret_cast<double *>(static_cast<unsigned char *>(ws) + kBranchBytes);
    uint64_t fixed = 0;
    int done = 0;
    *launches = 0;
    while (done < a.m) {
        const int left = a.m - done, bits = a.nq - done;
        if (bits <= kTailBits) {
            TailArgs t{};
            t.bits = bits;
            t.r = left;
            t.first = done == 0;
            uint64_t rest = 0;
            for (int j = done; j < a.m; ++j) rest |= 1ull << a.pos[j];
            int c = 0;
            for (int p = 0; p < a.nq; ++p)
                if (!(((fixed | rest) >> p) & 1)) t.pos[c++] = (uint32_t)p;
            for (int j = 0; j < left; ++j) {
                t.pos[bits - 1 - j] = a.pos[done + j];
                t.u[j] = a.u[done + j];
            }
            const size_t lds = sizeof(double) << (bits + 1);
            static const hipError_t attr = hipFuncSetAttribute(
                reinterpret_cast<const void *>(k_measure_tail<R>),
                hipFuncAttributeMaxDynamicSharedMemorySize, (int)(sizeof(double) << (kTailBits + 1)));
            if (attr != hipSuccess) return attr;
            hipLaunchKernelGGL(k_measure_tail<R>, dim3(1), dim3(kTailThreads), lds, s,
                               (const typename VMs<R>::T *)psi, t, br, out);
            ++*launches;
            break;
        }
        const int r = std::min(kMeasRound, left);
        HistArgs h{};
        DecideArgs d{};
        h.first = d.first = done == 0;
        d.r = r;
        // A qubit is a lane bit if at most 6 group bits lie below it: its place
        // in the group id is its position less the zeros inserted below.
        uint64_t high = 0;
        int nh = 0;
        for (int j = 0; j < r; ++j)
            if (a.pos[done + j] >= (uint32_t)kMeasLane) high |= 1ull << a.pos[done + j];
        const uint64_t ins = fixed | high;
        for (int j = 0; j < r; ++j) {
            const uint32_t p = a.pos[done + j];
            d.pos[j] = p;
            d.u[j] = a.u[done + j];
            if ((high >> p) & 1) {
                d.bin[j] = (uint32_t)nh;
                h.hpos[nh++] = p;
            }
        }
        for (int j = 0; j < r; ++j) {
            const uint32_t p = a.pos[done + j];
            if ((high >> p) & 1) continue;
            d.bin[j] = (uint32_t)(nh + h.nl);
            h.lpos[h.nl++] = p - (uint32_t)__builtin_popcountll(ins & ((1ull << p) - 1));
        }
        for (int p = 0; p < a.nq; ++p)
            if ((ins >> p) & 1) h.ins[h.nins++] = (uint32_t)p;
        h.ngroups = 1ull << (a.nq - h.nins);
        const unsigned nb = (unsigned)std::min<uint64_t>(
            (h.ngroups + kMeasThreads - 1) / kMeasThreads, kMeasBlocks);
        d.nblocks = (int)nb;
        switch (nh) {
        case 0: launch_hist<R, 0>(psi, h, nb, br, partial, s); break;
        case 1: launch_hist<R, 1>(psi, h, nb, br, partial, s); break;
        case 2: launch_hist<R, 2>(psi, h, nb, br, partial, s); break;
        case 3: launch_hist<R, 3>(psi, h, nb, br, partial, s); break;
        default: launch_hist<R, 4>(psi, h, nb, br, partial, s); break;
        }
        hipLaunchKernelGGL(k_measure_decide, dim3(1), dim3(1024), 0, s, partial, d, br, out);
        *launches += 2;
        for (int j = 0; j < r; ++j) fixed |= 1ull << a.pos[done + j];
        done += r;
    }
    const uint64_t dim = 1ull << a.nq;
    const unsigned g = (unsigned)std::min<uint64_t>((dim + 255) / 256, 1ull << 20);
    hipLaunchKernelGGL(k_measure_collapse<R>, dim3(g), dim3(256), 0, s,
                       (typename VMs<R>::T *)psi, dim, br);
    ++*launches;
    return hipGetLastError();
}

hipError_t measure(int dtype, void *psi, const MeasureArgs &a, void *ws, MeasureBranch *out,
                   int *launches, hipStream_t s) {
    if (a.m < 1 || a.m > a.nq || a.nq > 36) return hipErrorInvalidValue;
    return dtype == 0 ? measure_t<double>(psi, a, ws, out, launches, s)
                      : measure_t<float>(psi, a, ws, out, launches, s);
}

}  // namespace dev
}  // namespace qsv
