// Pauli sums <psi|H|psi>.  Every sum is accumulated in double precision
// whatever the state's dtype.
//
// k_pauli_tiles: strings whose X letters lie within one tile shape share its
// reads of the state.  A workgroup of 512 threads takes tiles of 2^12
// amplitudes: 8 per thread in registers, and the tile in LDS (64 or 32 KiB),
// from which a thread reads the partners psi_{j^x} of its own.  A string then
// costs, per pair, one LDS read, the one product its parity needs (mul, fma) and a
// signed add: the sign splits into the tile's, the register's (uniform) and the
// thread's, and the coefficient goes in with the thread's sign, so that one running
// sum serves every string.  The next tile's amplitudes are on their way meanwhile.
// With 12 bits of tile a sum of 200 random strings of weight <= 4 on 25 qubits (111
// X masks) reads the state 8 times: 1.6 ms in complex128, 2.7 TB/s, of which the
// reads alone would take 0.7; the rest is the latency of 14 groups a tile (21 vector
// and about 50 scalar instructions each) at four waves per SIMD.  As one sweep per X
// mask it took 11.8 ms.  On 30 qubits 8 strings that two shapes hold take 2 reads,
// 5.7 ms (6.0 TB/s; 24.7 as sweeps), 8 that one shape holds 2.9.
// k_pauli_wide: the strings that fit in no tile, one sweep per X mask.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "pauli.hpp"
#include "result_store.hpp"

namespace qsv {
namespace dev {

template <typename R> struct VP;
template <> struct VP<double> { using T = double2; };
template <> struct VP<float> { using T = float2; };

constexpr int kPT = 1 << kPauliThreadBits;

// sum over the workgroup, valid in thread 0
template <int THREADS>
__device__ __forceinline__ double group_sum(double v, double *sh) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    v = 0.0;
    if (threadIdx.x == 0)
        for (int i = 0; i < THREADS / 64; ++i) v += sh[i];
    return v;
}

__device__ __forceinline__ double sign_flip(double v, uint32_t s) {    // s = 0 or 1
    return __hiloint2double(__double2hiint(v) ^ (int)(s << 31), __double2loint(v));
}

// A string over the products q[i] of the registers i with bit HB clear (HB < 0:
// all).
template <int NR, int HB>
__device__ __forceinline__ void pauli_term(double &acc, const double *q, const PauliTerm &pt,
                                           uint64_t base, uint32_t tid) {
    const uint32_t sreg = pt.sreg;
    double local = 0.0;
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        if (HB >= 0 && ((i >> (HB < 0 ? 0 : HB)) & 1)) continue;
        const double sg = __hiloint2double((int)(0x3ff00000u | (((sreg >> i) & 1u) << 31)), 0);
        local = __builtin_fma(q[i], sg, local);
    }
    const uint32_t st = (uint32_t)(__popcll(base & pt.zo) + __popc(tid & pt.zthr)) & 1u;
    acc = __builtin_fma(local, sign_flip(pt.c, st), acc);
}

// X: the X mask over the register bits.
template <typename R, int RB, int X>
__device__ __forceinline__ void pauli_group(double &acc, const typename VP<R>::T *amp,
                                            const typename VP<R>::T *tile, const PauliXGroup &g,
                                            const PauliTerm *__restrict__ terms, uint64_t base,
                                            uint32_t tid) {
    using T = typename VP<R>::T;
    constexpr int NR = 1 << RB;
    constexpr int HB = X == 0 ? -1 : 31 - __builtin_clz((unsigned)(X ? X : 1));
    const T *from = tile + (tid ^ g.xthr);
    T b[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i)
        if (HB < 0 || !((i >> (HB < 0 ? 0 : HB)) & 1)) b[i] = from[(uint32_t)(i ^ X) << kPauliThreadBits];
    double q[NR];
    if (g.odd) {
#pragma unroll
        for (int i = 0; i < NR; ++i)
            if (HB < 0 || !((i >> (HB < 0 ? 0 : HB)) & 1))
                q[i] = __builtin_fma((double)b[i].x, (double)amp[i].y, -((double)b[i].y * (double)amp[i].x));
    } else {
#pragma unroll
        for (int i = 0; i < NR; ++i)
            if (HB < 0 || !((i >> (HB < 0 ? 0 : HB)) & 1))
                q[i] = __builtin_fma((double)b[i].x, (double)amp[i].x, (double)b[i].y * (double)amp[i].y);
    }
    pauli_term<NR, HB>(acc, q, g.first, base, tid);
    for (int t = g.term0; t < g.term0 + g.terms; ++t) pauli_term<NR, HB>(acc, q, terms[t], base, tid);
}

template <typename T, int RB>
__device__ __forceinline__ void pauli_load(T *v, const T *__restrict__ psi, uint64_t at,
                                           const uint64_t *reg, uint32_t pad_reg, bool on) {
#pragma unroll
    for (int i = 0; i < (1 << RB); ++i) {
        uint64_t o = 0;
#pragma unroll
        for (int j = 0; j < RB; ++j)
            if ((i >> j) & 1) o |= reg[j];
        v[i].x = v[i].y = 0;
        if (on && !((uint32_t)i & pad_reg)) v[i] = psi[at | o];
    }
}

template <typename R, int RB>
__global__ __launch_bounds__(kPT, 4) void k_pauli_tiles(
    const typename VP<R>::T *__restrict__ psi, uint64_t ntiles, const PauliSet *__restrict__ sets,
    const PauliXGroup *__restrict__ groups, const PauliTerm *__restrict__ terms,
    double *__restrict__ partial) {
    using T = typename VP<R>::T;
    constexpr int NR = 1 << RB;
    extern __shared__ __align__(16) unsigned char smem_p[];
    T *tile = reinterpret_cast<T *>(smem_p);
    const PauliSet &st = sets[blockIdx.y];
    const uint32_t tid = threadIdx.x;
    uint64_t thr = 0;
#pragma unroll
    for (int b = 0; b < kPauliThreadBits; ++b)
        if (st.tpos[b] < 64) thr |= (uint64_t)((tid >> b) & 1u) << st.tpos[b];
    uint64_t reg[RB];
#pragma unroll
    for (int j = 0; j < RB; ++j) {
        const uint32_t p = st.tpos[kPauliThreadBits + j];
        reg[j] = p < 64 ? 1ull << p : 0;
    }
    const uint32_t pad_reg = st.pad_reg;
    const bool on = !(tid & st.pad_thr);
    auto base_of = [&](uint64_t t) {
        for (int i = 0; i < st.n_ins; ++i) {
            const uint64_t lowm = (1ull << st.ins[i]) - 1;
            t = ((t & ~lowm) << 1) | (t & lowm);
        }
        return t;
    };
    double acc = 0.0;
    uint64_t t = blockIdx.x;
    uint64_t base = base_of(t);
    T next[NR];
    pauli_load<T, RB>(next, psi, base | thr, reg, pad_reg, on);
    while (t < ntiles) {
        T amp[NR];
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            amp[i] = next[i];
            tile[tid + ((uint32_t)i << kPauliThreadBits)] = amp[i];
        }
        __syncthreads();
        const uint64_t here = base;
        t += gridDim.x;
        if (t < ntiles) {
            base = base_of(t);
            pauli_load<T, RB>(next, psi, base | thr, reg, pad_reg, on);
        }
        // the next group's line is on its way while a group is worked on
        PauliXGroup ahead = groups[st.group0];
        for (int gi = 0; gi < st.groups; ++gi) {
            const PauliXGroup g = ahead;
            ahead = groups[st.group0 + (gi + 1 < st.groups ? gi + 1 : gi)];
#define QSV_PX(X)                                                                        \
    case X:                                                                              \
        if constexpr (X < NR) pauli_group<R, RB, (X < NR ? X : 0)>(acc, amp, tile, g, terms, here, tid); \
        break;
            switch (g.xreg) {
                QSV_PX(0) QSV_PX(1) QSV_PX(2) QSV_PX(3) QSV_PX(4) QSV_PX(5) QSV_PX(6) QSV_PX(7)
            }
#undef QSV_PX
        }
        __syncthreads();    // the tile is rewritten next
    }
    double *sh = reinterpret_cast<double *>(smem_p);
    acc = group_sum<kPT>(acc, sh);
    if (tid == 0) partial[(size_t)blockIdx.y * gridDim.x + blockIdx.x] = acc;
}

template <typename R>
__global__ __launch_bounds__(256) void k_pauli_wide(const typename VP<R>::T *__restrict__ psi,
                                                    int nq,
                                                    const PauliWideGroup *__restrict__ wide,
                                                    double *__restrict__ partial) {
    __shared__ double sh[4];
    const PauliWideGroup &g = wide[blockIdx.y];
    uint64_t z[kPauliWide];
    double c[kPauliWide];
#pragma unroll
    for (int t = 0; t < kPauliWide; ++t) {
        z[t] = g.z[t];      // unused ones are zero, as their coefficients
        c[t] = g.c[t];
    }
    const uint64_t npairs = 1ull << (nq - 1), lowm = (1ull << g.hbit) - 1;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    const bool odd = g.odd != 0;
    double acc = 0.0;
    for (uint64_t k = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; k < npairs; k += stride) {
        const uint64_t j = ((k & ~lowm) << 1) | (k & lowm);
        const auto a = psi[j], b = psi[j ^ g.x];
        const double q = odd ? __builtin_fma((double)b.x, (double)a.y, -((double)b.y * (double)a.x))
                             : __builtin_fma((double)b.x, (double)a.x, (double)b.y * (double)a.y);
        double w = 0.0;
#pragma unroll
        for (int t = 0; t < kPauliWide; ++t)
            if (t < g.nt) w += sign_flip(c[t], (uint32_t)__popcll(j & z[t]) & 1u);
        acc = __builtin_fma(w, q, acc);
    }
    acc = group_sum<256>(acc, sh);
    if (threadIdx.x == 0) partial[(size_t)blockIdx.y * gridDim.x + blockIdx.x] = acc;
}

__global__ __launch_bounds__(1024) void k_pauli_total(const double *__restrict__ partial, int64_t n,
                                                      double *out) {
    __shared__ double sh[16];
    double v = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += 4096) {
        double p[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) p[k] = i + 1024 * k < n ? partial[i + 1024 * k] : 0.0;
        v += (p[0] + p[1]) + (p[2] + p[3]);
    }
    v = group_sum<1024>(v, sh);
    if (threadIdx.x == 0) result_store(out, v);
}

template <typename R>
static hipError_t pauli_sum_t(const void *psi, int nq, const PauliPlan &p, const void *blob,
                              double *ws, double *out, hipStream_t s) {
    using T = typename VP<R>::T;
    constexpr int RB = kPauliRegBits, m = kPauliTileBits;
    const unsigned char *b = static_cast<const unsigned char *>(blob);
    const auto *groups = reinterpret_cast<const PauliXGroup *>(b);
    const auto *wide = reinterpret_cast<const PauliWideGroup *>(groups + p.groups.size());
    const auto *sets = reinterpret_cast<const PauliSet *>(wide + p.wide.size());
    const auto *terms = reinterpret_cast<const PauliTerm *>(sets + p.sets.size());
    double *at = ws;
    // rows of the grid go in the y dimension, at most kRows of them at once
    constexpr size_t kRows = 32768;
    if (!p.sets.empty()) {
        const size_t lds = sizeof(T) << m;
        static const hipError_t attr = hipFuncSetAttribute(
            reinterpret_cast<const void *>(k_pauli_tiles<R, RB>),
            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (attr != hipSuccess) return attr;
        const uint64_t ntiles = nq > m ? 1ull << (nq - m) : 1;
        for (size_t y = 0; y < p.sets.size(); y += kRows) {
            const unsigned rows = (unsigned)std::min(kRows, p.sets.size() - y);
            hipLaunchKernelGGL((k_pauli_tiles<R, RB>), dim3(p.grid_x, rows), dim3(kPT), lds, s,
                               (const T *)psi, ntiles, sets + y, groups, terms, at);
            at += (size_t)p.grid_x * rows;
        }
    }
    for (size_t y = 0; y < p.wide.size(); y += kRows) {
        const unsigned rows = (unsigned)std::min(kRows, p.wide.size() - y);
        hipLaunchKernelGGL(k_pauli_wide<R>, dim3(p.wide_x, rows), dim3(256), 0, s, (const T *)psi, nq,
                           wide + y, at);
        at += (size_t)p.wide_x * rows;
    }
    hipLaunchKernelGGL(k_pauli_total, dim3(1), dim3(1024), 0, s, ws, (int64_t)p.partials(), out);
    return hipGetLastError();
}

hipError_t pauli_sum(int dtype, const void *psi, int nq, const PauliPlan &p, const void *blob,
                     double *ws, double *out, hipStream_t s) {
    return dtype == 0 ? pauli_sum_t<double>(psi, nq, p, blob, ws, out, s)
                      : pauli_sum_t<float>(psi, nq, p, blob, ws, out, s);
}

}  // namespace dev
}  // namespace qsv
