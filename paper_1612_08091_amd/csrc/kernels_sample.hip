// Sampling without collapse.  Shot s takes the smallest index i with
// C_i > u[s] T, C the running sum of |psi|^2 and T its total, accumulated in
// double whatever the state's dtype; where rounding puts u T at or past the
// end, the last index with a nonzero amplitude.
//
// Three levels: blocks of 2^12 amplitudes (k_block_sums, one read of the
// state: HBM-bound), chunks of 1024 blocks (k_scan_chunks: the running ends of
// a chunk's blocks), the chunks (k_scan_top, only above 2^22 amplitudes).  A
// shot is one workgroup: every thread looks at one chunk end, then at four
// block ends, so that each level costs one memory round trip, and the block is
// read coalesced and summed in index order from LDS.  States of at most 2^12
// amplitudes take that kernel alone.  The sums are built from partial sums in a
// fixed order; at a level's joint two of them may differ in the last place, so
// an amplitude that is zero is never taken.
// Measured (complex128, with each level scanned by single threads before): 100
// shots of 5 qubits 6.0 us in one kernel (34 in three), 1000 of 16 qubits 20 us
// (68), 1000 of 30 qubits 2.78 ms, of which 2.75 are the read (3.48).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "device.hpp"
#include "result_store.hpp"

namespace qsv {
namespace dev {

template <typename R> struct VS;
template <> struct VS<double> { using T = double2; };
template <> struct VS<float> { using T = float2; };

constexpr int kSampleBits = 12;
constexpr int kST = 256;
constexpr uint64_t kChunk = 1024;

__device__ __forceinline__ double weight(double2 a) { return a.x * a.x + a.y * a.y; }
__device__ __forceinline__ double weight(float2 a) {
    return (double)a.x * a.x + (double)a.y * a.y;
}

// Sum of the values of the threads before this one; *total: of all (every thread).
__device__ __forceinline__ double scan_before(double v, double *sh, double *total) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    double s = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const double x = __shfl_up(s, o, 64);
        if (lane >= o) s += x;
    }
    __syncthreads();
    if (lane == 63) sh[w] = s;
    __syncthreads();
    double before = 0.0, all = 0.0;
#pragma unroll
    for (int i = 0; i < kST / 64; ++i) {
        if (i < w) before += sh[i];
        all += sh[i];
    }
    *total = all;
    const double prev = __shfl_up(s, 1, 64);
    return before + (lane ? prev : 0.0);
}

__device__ __forceinline__ int64_t block_max(int64_t v, int64_t *sh) {
    for (int o = 32; o > 0; o >>= 1) {
        const int64_t x = __shfl_xor(v, o, 64);
        v = x > v ? x : v;
    }
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    v = sh[0];
    for (int i = 1; i < kST / 64; ++i) v = sh[i] > v ? sh[i] : v;
    return v;
}

// Sum and last nonzero index of each block of 2^kSampleBits amplitudes.
template <typename R>
__global__ __launch_bounds__(kST) void k_block_sums(const typename VS<R>::T *__restrict__ psi,
                                                    double *__restrict__ bsum,
                                                    int64_t *__restrict__ blast) {
    __shared__ double sh[kST / 64];
    __shared__ int64_t shl[kST / 64];
    constexpr int PER = (1 << kSampleBits) / kST;
    const uint64_t b0 = (uint64_t)blockIdx.x << kSampleBits;
    typename VS<R>::T v[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) v[j] = psi[b0 + (uint32_t)j * kST + threadIdx.x];
    double acc = 0.0;
    int64_t last = -1;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const double p = weight(v[j]);
        acc += p;
        if (p > 0.0) last = (int64_t)(b0 + (uint32_t)j * kST + threadIdx.x);
    }
    double total;
    (void)scan_before(acc, sh, &total);
    last = block_max(last, shl);
    if (threadIdx.x == 0) {
        bsum[blockIdx.x] = total;
        blast[blockIdx.x] = last;
    }
}

// In place: bsum[b] becomes the running sum up to the end of block b within
// its chunk; ctot, clast: the chunk's sum and last nonzero index.  A single
// chunk also fills in the top level.
struct SampleTop {
    double total;
    int64_t last;
};
__global__ __launch_bounds__(kST) void k_scan_chunks(double *__restrict__ bsum,
                                                     const int64_t *__restrict__ blast,
                                                     uint64_t nb, double *__restrict__ ctot,
                                                     int64_t *__restrict__ clast,
                                                     SampleTop *__restrict__ top) {
    __shared__ double sh[kST / 64];
    __shared__ int64_t shl[kST / 64];
    constexpr int PER = kChunk / kST;
    const uint64_t b0 = (uint64_t)blockIdx.x * kChunk + threadIdx.x * PER;
    double v[PER], sum = 0.0;
    int64_t last = -1;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        v[k] = b0 + k < nb ? bsum[b0 + k] : 0.0;
        const int64_t l = b0 + k < nb ? blast[b0 + k] : -1;
        last = l > last ? l : last;
    }
#pragma unroll
    for (int k = 0; k < PER; ++k) sum += v[k];
    double total;
    double run = scan_before(sum, sh, &total);
    last = block_max(last, shl);
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        run += v[k];
        if (b0 + k < nb) bsum[b0 + k] = run;
    }
    if (threadIdx.x == 0) {
        ctot[blockIdx.x] = total;
        clast[blockIdx.x] = last;
        if (gridDim.x == 1) *top = SampleTop{total, last};
    }
}

// In place: ctot[c] becomes the running sum up to the end of chunk c.
__global__ __launch_bounds__(kST) void k_scan_top(double *__restrict__ ctot,
                                                  const int64_t *__restrict__ clast, uint64_t nc,
                                                  SampleTop *__restrict__ top) {
    __shared__ double sh[kST / 64];
    __shared__ int64_t shl[kST / 64];
    double carry = 0.0;
    int64_t last = -1;
    for (uint64_t c0 = 0; c0 < nc; c0 += kST) {
        const uint64_t c = c0 + threadIdx.x;
        const double v = c < nc ? ctot[c] : 0.0;
        if (c < nc && clast[c] > last) last = clast[c];
        double total;
        const double before = scan_before(v, sh, &total);
        if (c < nc) ctot[c] = carry + (before + v);
        carry += total;
    }
    last = block_max(last, shl);
    if (threadIdx.x == 0) *top = SampleTop{carry, last};
}

// First k < n with ends[k] > r (over all threads), or n.
__device__ __forceinline__ uint32_t first_above(const double *__restrict__ ends, uint32_t n,
                                                double from, double r, uint32_t *sh) {
    uint32_t k = threadIdx.x;
    while (k < n && !(from + ends[k] > r)) k += kST;
    if (k > n) k = n;
    __syncthreads();
    if (threadIdx.x == 0) *sh = n;
    __syncthreads();
    for (int o = 32; o > 0; o >>= 1) {
        const uint32_t x = (uint32_t)__shfl_xor((int)k, o, 64);
        k = x < k ? x : k;
    }
    if ((threadIdx.x & 63) == 0) atomicMin(sh, k);
    __syncthreads();
    return *sh;
}

// SMALL: the state is one block (of 2^bbits amplitudes) and nothing was summed
// before; else full blocks.
template <typename R, bool SMALL>
__global__ __launch_bounds__(kST) void k_sample(const typename VS<R>::T *__restrict__ psi,
                                                int bbits, uint64_t nb,
                                                const double *__restrict__ bend,
                                                const int64_t *__restrict__ blast,
                                                const double *__restrict__ cend, uint32_t nc,
                                                const SampleTop *__restrict__ top,
                                                const double *__restrict__ u,
                                                uint64_t *__restrict__ out) {
    constexpr int PER = (1 << kSampleBits) / kST;
    __shared__ double p[kST * (PER + 1)];       // a pad word after every thread's PER
    __shared__ double sh[kST / 64];
    __shared__ int64_t shl[kST / 64];
    __shared__ uint32_t found;
    const uint32_t tid = threadIdx.x;
    // (from host memory: on its way while the state is read)
    const double draw = u[blockIdx.x];
    double r = 0.0, from = 0.0;
    uint64_t blk = 0;
    if (!SMALL) {
        r = draw * top->total;
        const uint32_t c = first_above(cend, nc, 0.0, r, &found);
        if (c >= nc) {
            if (tid == 0) result_store(out + blockIdx.x, (uint64_t)(top->last < 0 ? 0 : top->last));
            return;
        }
        const uint64_t c0 = (uint64_t)c * kChunk;
        const uint32_t in = (uint32_t)(nb - c0 < kChunk ? nb - c0 : kChunk);
        from = c ? cend[c - 1] : 0.0;
        uint32_t b = first_above(bend + c0, in, from, r, &found);
        if (b >= in) b = in - 1;
        blk = c0 + b;
        if (b) from += bend[blk - 1];
    }
    const uint64_t b0 = blk << kSampleBits;
    const uint32_t size = SMALL ? 1u << bbits : 1u << kSampleBits;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const uint32_t l = (uint32_t)j * kST + tid;
        p[l + l / PER] = !SMALL || l < size ? weight(psi[b0 + l]) : 0.0;
    }
    __syncthreads();
    double q[PER], seg = 0.0;
    int64_t last = -1;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        q[j] = p[tid * (PER + 1) + j];
        seg += q[j];
        if (q[j] > 0.0) last = (int64_t)(tid * PER + j);
    }
    double total;
    double c = from + scan_before(seg, sh, &total);
    if (SMALL) r = draw * total;
    uint32_t hit = ~0u;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        c += q[j];
        if (hit == ~0u && c > r && q[j] > 0.0) hit = tid * PER + j;
    }
    if (tid == 0) found = ~0u;
    last = block_max(last, shl);
    for (int o = 32; o > 0; o >>= 1) {
        const uint32_t x = (uint32_t)__shfl_xor((int)hit, o, 64);
        hit = x < hit ? x : hit;
    }
    if ((tid & 63) == 0) atomicMin(&found, hit);
    __syncthreads();
    if (tid != 0) return;
    int64_t res = -1;
    if (found != ~0u) res = (int64_t)(b0 + found);
    else if (last >= 0) res = (int64_t)b0 + last;
    else if (!SMALL) {
        // a block of zeros between two sums that differ in the last place: the
        // nonzero amplitude before it, else the first block's end after it
        for (uint64_t b = blk; b-- > 0 && res < 0;) res = blast[b];
        for (uint64_t b = blk + 1; b < nb && res < 0; ++b) res = blast[b];
    }
    result_store(out + blockIdx.x, (uint64_t)(res < 0 ? 0 : res));
}

namespace {
struct SampleLayout {
    uint64_t nb, nc;
    size_t blast, ctot, clast, top, bytes;
    explicit SampleLayout(int nq) {
        nb = nq > kSampleBits ? 1ull << (nq - kSampleBits) : 1;
        nc = (nb + kChunk - 1) / kChunk;
        blast = 8 * nb;
        ctot = blast + 8 * nb;
        clast = ctot + 8 * nc;
        top = clast + 8 * nc;
        bytes = top + sizeof(SampleTop);
    }
};
}  // namespace

size_t sample_workspace_bytes(int nq) { return SampleLayout(nq).bytes; }

template <typename R>
static hipError_t sample_t(const void *psi, int nq, int shots, const double *u, void *ws,
                           uint64_t *out, hipStream_t s) {
    using T = typename VS<R>::T;
    const SampleLayout l(nq);
    unsigned char *w = static_cast<unsigned char *>(ws);
    double *bsum = reinterpret_cast<double *>(w);
    int64_t *blast = reinterpret_cast<int64_t *>(w + l.blast);
    double *ctot = reinterpret_cast<double *>(w + l.ctot);
    int64_t *clast = reinterpret_cast<int64_t *>(w + l.clast);
    SampleTop *top = reinterpret_cast<SampleTop *>(w + l.top);
    if (nq <= kSampleBits) {
        hipLaunchKernelGGL((k_sample<R, true>), dim3((unsigned)shots), dim3(kST), 0, s,
                           (const T *)psi, nq, l.nb, bsum, blast, ctot, 0u, top, u, out);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_block_sums<R>, dim3((unsigned)l.nb), dim3(kST), 0, s, (const T *)psi, bsum,
                       blast);
    hipLaunchKernelGGL(k_scan_chunks, dim3((unsigned)l.nc), dim3(kST), 0, s, bsum, blast, l.nb, ctot,
                       clast, top);
    if (l.nc > 1)
        hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(kST), 0, s, ctot, clast, l.nc, top);
    hipLaunchKernelGGL((k_sample<R, false>), dim3((unsigned)shots), dim3(kST), 0, s, (const T *)psi,
                       kSampleBits, l.nb, bsum, blast, ctot, (uint32_t)l.nc, top, u, out);
    return hipGetLastError();
}

hipError_t sample(int dtype, const void *psi, int nq, int shots, const double *u, void *ws,
                  uint64_t *out, hipStream_t s) {
    if (shots < 1 || nq < 0) return hipErrorInvalidValue;
    return dtype == 0 ? sample_t<double>(psi, nq, shots, u, ws, out, s)
                      : sample_t<float>(psi, nq, shots, u, ws, out, s);
}

}  // namespace dev
}  // namespace qsv
