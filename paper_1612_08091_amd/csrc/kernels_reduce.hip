// Reductions and whole-state operations: probabilities, masked probability
// sums, collapse after measurement,
// qubit allocation (zero extension) and deallocation (compaction).  Every sum
// is accumulated in double precision whatever the state's dtype.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>

#include "device.hpp"
#include "result_store.hpp"

namespace qsv {
namespace dev {

template <typename R> struct V2r;
template <> struct V2r<double> { using T = double2; };
template <> struct V2r<float> { using T = float2; };

constexpr int kRedThreads = 256;
constexpr int kRedBlocks = 1024;

__device__ __forceinline__ double wave_sum(double v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
    return v;
}

// Sum over the block; the result is valid in thread 0.
__device__ __forceinline__ double block_sum(double v, double *sh) {
    v = wave_sum(v);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    __syncthreads();
    if (lane == 0) sh[w] = v;
    __syncthreads();
    if (w == 0) {
        v = (lane < (int)(blockDim.x >> 6)) ? sh[lane] : 0.0;
        v = wave_sum(v);
    }
    return v;
}

__device__ __forceinline__ uint64_t expand_idx(uint64_t g, const IndexArgs &ia) {
    for (int i = 0; i < ia.npos; ++i) {
        const uint64_t lowm = (1ull << ia.pos[i]) - 1;
        g = ((g & ~lowm) << 1) | (g & lowm);
    }
    return g | ia.ones;
}

static unsigned red_grid(uint64_t work) {
    uint64_t b = (work + kRedThreads - 1) / kRedThreads;
    if (b > kRedBlocks) b = kRedBlocks;
    if (b == 0) b = 1;
    return (unsigned)b;
}

// ------------------------------------------------------------ probability
// A workgroup takes runs of 2048 amplitudes, eight loads of a thread in flight:
// bound by HBM, 16 GiB in 2.80 ms (6.1 TB/s; one load at a time from a grid-wide
// stride 3.14, eight of them 3.09).
template <typename R>
__global__ __launch_bounds__(kRedThreads) void k_prob_masked(const typename V2r<R>::T *psi,
                                                             uint64_t ngroups, IndexArgs ia,
                                                             double *partial) {
    constexpr int U = 8;
    __shared__ double sh[16];
    double acc = 0.0;
    if (ngroups >= U * kRedThreads) {      // a power of two: whole runs
        for (uint64_t r = blockIdx.x; r < ngroups / (U * kRedThreads); r += gridDim.x) {
            const uint64_t g = r * (U * kRedThreads) + threadIdx.x;
            typename V2r<R>::T v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = psi[expand_idx(g + u * kRedThreads, ia)];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const double re = v[u].x, im = v[u].y;
                acc += re * re + im * im;
            }
        }
    } else {
        for (uint64_t g = (uint64_t)blockIdx.x * kRedThreads + threadIdx.x; g < ngroups;
             g += (uint64_t)gridDim.x * kRedThreads) {
            const auto a = psi[expand_idx(g, ia)];
            const double re = a.x, im = a.y;
            acc += re * re + im * im;
        }
    }
    acc = block_sum(acc, sh);
    if (threadIdx.x == 0) partial[blockIdx.x] = acc;
}

template <typename R>
__global__ __launch_bounds__(kRedThreads) void k_prob_split(const typename V2r<R>::T *psi,
                                                            uint64_t dim, int q,
                                                            double *partial) {
    __shared__ double sh[16];
    double a0 = 0.0, a1 = 0.0;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < dim;
         i += (uint64_t)gridDim.x * blockDim.x) {
        const auto a = psi[i];
        const double p = (double)a.x * a.x + (double)a.y * a.y;
        if ((i >> q) & 1) a1 += p;
        else a0 += p;
    }
    a0 = block_sum(a0, sh);
    a1 = block_sum(a1, sh);
    if (threadIdx.x == 0) {
        partial[2 * blockIdx.x] = a0;
        partial[2 * blockIdx.x + 1] = a1;
    }
}

// out[j] = sum_b partial[b * stride + j] for j < width
__global__ __launch_bounds__(kRedThreads) void k_finish(const double *partial, int nblocks,
                                                        int stride, int width, double *out) {
    __shared__ double sh[16];
    for (int j = 0; j < width; ++j) {
        double acc = 0.0;
        for (int b = threadIdx.x; b < nblocks; b += blockDim.x) acc += partial[b * stride + j];
        acc = block_sum(acc, sh);
        if (threadIdx.x == 0) result_store(out + j, acc);
    }
}

size_t reduce_workspace_bytes(int) { return sizeof(double) * 2 * kRedBlocks; }

// --------------------------------------------------- allocation-free form
// Partial sums of prob_masked_noalloc: one per block of k_prob_masked (at most
// kRedBlocks).  Every GPU holds its own copy until the process ends; each call
// writes the slots it reads, so nothing needs clearing, and calls that overlap
// on one GPU race on it.
constexpr int kScratchDoubles = kRedBlocks;
static __device__ __align__(256) double scratch[kScratchDoubles];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
double *g_scratch_ptr[kMaxDevices] = {};

// Device address of this GPU's `scratch` (resolved once per device, with the
// device current; host code never uses the array's own name).
hipError_t scratch_ptr(double **out) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        g_scratch_ptr[dev] = static_cast<double *>(p);
    }
    *out = g_scratch_ptr[dev];
    return hipSuccess;
}
}  // namespace

int prob_noalloc_partials(uint64_t ngroups) { return (int)red_grid(ngroups); }
int prob_noalloc_capacity() { return kScratchDoubles; }

hipError_t prob_masked_noalloc(int dtype, const void *psi, uint64_t ngroups, const IndexArgs &ia,
                               double *out_dev, hipStream_t s) {
    if ((int)red_grid(ngroups) > kScratchDoubles) return hipErrorInvalidValue;
    double *ws = nullptr;
    const hipError_t e = scratch_ptr(&ws);
    if (e != hipSuccess) return e;
    return prob_masked(dtype, psi, ngroups, ia, ws, out_dev, s);
}

hipError_t prob_masked(int dtype, const void *psi, uint64_t ngroups, const IndexArgs &ia,
                       double *ws, double *out_dev, hipStream_t s) {
    const unsigned g = red_grid(ngroups);
    if (dtype == 0)
        hipLaunchKernelGGL(k_prob_masked<double>, dim3(g), dim3(kRedThreads), 0, s,
                           (const double2 *)psi, ngroups, ia, ws);
    else
        hipLaunchKernelGGL(k_prob_masked<float>, dim3(g), dim3(kRedThreads), 0, s,
                           (const float2 *)psi, ngroups, ia, ws);
    hipLaunchKernelGGL(k_finish, dim3(1), dim3(kRedThreads), 0, s, ws, (int)g, 1, 1, out_dev);
    return hipGetLastError();
}

hipError_t prob_split(int dtype, const void *psi, int nq, int q, double *ws, double *out_dev,
                      hipStream_t s) {
    const uint64_t dim = 1ull << nq;
    const unsigned g = red_grid(dim);
    if (dtype == 0)
        hipLaunchKernelGGL(k_prob_split<double>, dim3(g), dim3(kRedThreads), 0, s,
                           (const double2 *)psi, dim, q, ws);
    else
        hipLaunchKernelGGL(k_prob_split<float>, dim3(g), dim3(kRedThreads), 0, s,
                           (const float2 *)psi, dim, q, ws);
    hipLaunchKernelGGL(k_finish, dim3(1), dim3(kRedThreads), 0, s, ws, (int)g, 2, 2, out_dev);
    return hipGetLastError();
}

template <typename R>
__global__ void k_probs(const typename V2r<R>::T *psi, uint64_t dim, double *out) {
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < dim;
         i += (uint64_t)gridDim.x * blockDim.x) {
        const auto a = psi[i];
        out[i] = (double)a.x * a.x + (double)a.y * a.y;
    }
}

hipError_t probs(int dtype, const void *psi, uint64_t dim, double *out_dev, hipStream_t s) {
    const unsigned g = (unsigned)std::min<uint64_t>((dim + 255) / 256, 1ull << 20);
    if (dtype == 0)
        hipLaunchKernelGGL(k_probs<double>, dim3(g), dim3(256), 0, s, (const double2 *)psi, dim,
                           out_dev);
    else
        hipLaunchKernelGGL(k_probs<float>, dim3(g), dim3(256), 0, s, (const float2 *)psi, dim,
                           out_dev);
    return hipGetLastError();
}

// ------------------------------------------------------------ state ops
template <typename R>
__global__ void k_fill_basis0(typename V2r<R>::T *psi, uint64_t dim) {
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < dim;
         i += (uint64_t)gridDim.x * blockDim.x) {
        typename V2r<R>::T v;
        v.x = (i == 0) ? R(1) : R(0);
        v.y = R(0);
        psi[i] = v;
    }
}

template <typename R>
__global__ void k_zero(typename V2r<R>::T *psi, uint64_t from, uint64_t to) {
    for (uint64_t i = from + (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < to;
         i += (uint64_t)gridDim.x * blockDim.x) {
        typename V2r<R>::T v;
        v.x = R(0);
        v.y = R(0);
        psi[i] = v;
    }
}

template <typename R>
__global__ void k_compact(const typename V2r<R>::T *src, typename V2r<R>::T *dst, uint64_t half,
                          int q, int value) {
    const uint64_t lowm = (1ull << q) - 1;
    for (uint64_t j = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; j < half;
         j += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t i = ((j & ~lowm) << 1) | (j & lowm) | ((uint64_t)value << q);
        dst[j] = src[i];
    }
}

template <typename R>
__global__ void k_collapse(typename V2r<R>::T *psi, uint64_t dim, int q, int outcome,
                           double scale) {
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < dim;
         i += (uint64_t)gridDim.x * blockDim.x) {
        auto a = psi[i];
        if ((int)((i >> q) & 1) == outcome) {
            a.x = (R)((double)a.x * scale);
            a.y = (R)((double)a.y * scale);
        } else {
            a.x = R(0);
            a.y = R(0);
        }
        psi[i] = a;
    }
}

template <typename R>
__global__ void k_gather(const typename V2r<R>::T *psi, const uint64_t *idx, uint64_t count,
                         double *out) {
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count;
         i += (uint64_t)gridDim.x * blockDim.x) {
        const auto a = psi[idx[i]];
        out[2 * i] = (double)a.x;
        out[2 * i + 1] = (double)a.y;
    }
}

template <typename RS, typename RD>
__global__ void k_convert(const typename V2r<RS>::T *src, typename V2r<RD>::T *dst,
                          uint64_t dim) {
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < dim;
         i += (uint64_t)gridDim.x * blockDim.x) {
        const auto a = src[i];
        typename V2r<RD>::T b;
        b.x = (RD)a.x;
        b.y = (RD)a.y;
        dst[i] = b;
    }
}

// Elementwise kernels stride over their range; the grid is capped at 2^20
// blocks of 256 so that grid x block stays far below 2^32 threads at 2^33
// amplitudes.
static dim3 g1(uint64_t n) {
    uint64_t b = (n + 255) / 256;
    if (b > (1ull << 20)) b = 1ull << 20;
    return dim3((unsigned)(b ? b : 1));
}

hipError_t fill_basis0(int dtype, void *psi, uint64_t dim, hipStream_t s) {
    if (dtype == 0)
        hipLaunchKernelGGL(k_fill_basis0<double>, g1(dim), dim3(256), 0, s, (double2 *)psi, dim);
    else
        hipLaunchKernelGGL(k_fill_basis0<float>, g1(dim), dim3(256), 0, s, (float2 *)psi, dim);
    return hipGetLastError();
}

hipError_t zero_range(int dtype, void *psi, uint64_t from, uint64_t to, hipStream_t s) {
    if (to <= from) return hipSuccess;
    if (dtype == 0)
        hipLaunchKernelGGL(k_zero<double>, g1(to - from), dim3(256), 0, s, (double2 *)psi, from,
                           to);
    else
        hipLaunchKernelGGL(k_zero<float>, g1(to - from), dim3(256), 0, s, (float2 *)psi, from,
                           to);
    return hipGetLastError();
}

hipError_t compact(int dtype, const void *src, void *dst, int nq, int q, int value,
                   hipStream_t s) {
    const uint64_t half = 1ull << (nq - 1);
    if (dtype == 0)
        hipLaunchKernelGGL(k_compact<double>, g1(half), dim3(256), 0, s, (const double2 *)src,
                           (double2 *)dst, half, q, value);
    else
        hipLaunchKernelGGL(k_compact<float>, g1(half), dim3(256), 0, s, (const float2 *)src,
                           (float2 *)dst, half, q, value);
    return hipGetLastError();
}

hipError_t collapse(int dtype, void *psi, int nq, int q, int outcome, double scale,
                    hipStream_t s) {
    const uint64_t dim = 1ull << nq;
    if (dtype == 0)
        hipLaunchKernelGGL(k_collapse<double>, g1(dim), dim3(256), 0, s, (double2 *)psi, dim, q,
                           outcome, scale);
    else
        hipLaunchKernelGGL(k_collapse<float>, g1(dim), dim3(256), 0, s, (float2 *)psi, dim, q,
                           outcome, scale);
    return hipGetLastError();
}

hipError_t gather(int dtype, const void *psi, const uint64_t *idx, uint64_t count,
                  double *out, hipStream_t s) {
    if (count == 0) return hipSuccess;
    if (dtype == 0)
        hipLaunchKernelGGL(k_gather<double>, g1(count), dim3(256), 0, s, (const double2 *)psi, idx,
                           count, out);
    else
        hipLaunchKernelGGL(k_gather<float>, g1(count), dim3(256), 0, s, (const float2 *)psi, idx,
                           count, out);
    return hipGetLastError();
}

hipError_t convert_state(int ds, const void *src, int dd, void *dst, uint64_t dim,
                         hipStream_t s) {
    if (ds == 0 && dd == 1)
        hipLaunchKernelGGL((k_convert<double, float>), g1(dim), dim3(256), 0, s,
                           (const double2 *)src, (float2 *)dst, dim);
    else if (ds == 1 && dd == 0)
        hipLaunchKernelGGL((k_convert<float, double>), g1(dim), dim3(256), 0, s,
                           (const float2 *)src, (double2 *)dst, dim);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace dev
}  // namespace qsv
