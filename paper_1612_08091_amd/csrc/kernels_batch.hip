// Batched expectation values: many small circuits, each with its own Pauli
// sum.  k_batch is a persistent launch: every workgroup repeatedly takes the
// next circuit from an atomic counter (circuits are ordered longest first),
// simulates it alone and writes <H>.  A state of at most MB qubits lives in
// LDS for its whole life; a larger one given to k_batch lives in a
// per-workgroup slot of global memory and is updated by LDS-tile passes
// planned on the host.  No workgroup ever waits for another, so the grid
// drains as soon as the counter passes the number of circuits.  The
// pass-major kernels further down serve the larger circuits otherwise.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "device.hpp"
#include "lds_ops.hpp"

namespace qsv {
namespace dev {

// tile positions of a state held whole in LDS: local bit i is qubit i
__constant__ uint32_t kIdentityPos[40] = {0,  1,  2,  3,  4,  5,  6,  7,  8,  9,  10, 11, 12, 13,
                                          14, 15, 16, 17, 18, 19, 20, 21, 22, 23, 24, 25, 26, 27,
                                          28, 29, 30, 31, 32, 33, 34, 35, 36, 37, 38, 39};

// +1 or -1 by bit 0 of s
__device__ __forceinline__ double sign_of(uint32_t s) {
    return __hiloint2double((int)(0x3ff00000u | (s << 31)), 0);
}

template <typename R>
__device__ __forceinline__ double block_sum_b(double v, double *sh) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    __syncthreads();
    if (lane == 0) sh[w] = v;
    __syncthreads();
    double r = 0.0;
    if (threadIdx.x == 0)
        for (int i = 0; i < (int)(blockDim.x >> 6); ++i) r += sh[i];
    return r;
}

// sum_t c_t Re(i^{ny_t} sum_j conj(psi_{j^x}) psi_j (-1)^{popcount(j & z)}),
// this thread's share, state `st` of 2^n amplitudes (LDS or global).  The
// sweeps issue the loads of U indices (U pairs) per thread before using any,
// so enough reads are in flight for a state in global memory; a tail loop
// takes the indices left over.
// Indices [lo, hi) only (lo, hi multiples of 2): for a string with X letters
// the pairs (j, j ^ x) whose lower member has pair index in [lo/2, hi/2), so
// chunks that split [0, 2^n) split every term's sum.
template <typename R, bool SWZ>
__device__ __forceinline__ double pauli_partial(const typename VT<R>::T *st, int n,
                                                const BatchTerm *__restrict__ terms, int nt,
                                                uint64_t lo, uint64_t hi) {
    using T = typename VT<R>::T;
    constexpr int U = sizeof(R) == 4 ? 8 : 4;
    double acc = 0.0;
    (void)n;
    const uint64_t bd = blockDim.x;
    auto at = [&](uint64_t j) -> T { return st[SWZ ? swz<R>((uint32_t)j) : j]; };
    for (int t = 0; t < nt; ++t) {
        const BatchTerm tm = terms[t];
        double sr = 0.0, si = 0.0;
        if (tm.x == 0) {
            auto add = [&](uint64_t j, const T &a) {
                const double p = (double)a.x * a.x + (double)a.y * a.y;
                sr += (__popcll(j & tm.z) & 1) ? -p : p;
            };
            uint64_t j = lo + threadIdx.x;
            for (; j + (U - 1) * bd < hi; j += U * bd) {
                T a[U];
#pragma unroll
                for (int u = 0; u < U; ++u) a[u] = at(j + u * bd);
#pragma unroll
                for (int u = 0; u < U; ++u) add(j + u * bd, a[u]);
            }
            for (; j < hi; j += bd) add(j, at(j));
        } else {
            const int h = 63 - __builtin_clzll(tm.x);
            const uint64_t lowm = (1ull << h) - 1;
            auto idx = [&](uint64_t g) { return ((g & ~lowm) << 1) | (g & lowm); };
            auto add = [&](uint64_t j, const T &a, const T &b) {
                const uint64_t j2 = j ^ tm.x;
                const double u = (double)b.x * a.x + (double)b.y * a.y;
                const double v = (double)b.x * a.y - (double)b.y * a.x;
                const double s1 = (__popcll(j & tm.z) & 1) ? -1.0 : 1.0;
                const double s2 = (__popcll(j2 & tm.z) & 1) ? -1.0 : 1.0;
                sr += (s1 + s2) * u;
                si += (s1 - s2) * v;
            };
            const uint64_t half = hi >> 1;
            uint64_t g = (lo >> 1) + threadIdx.x;
            for (; g + (U - 1) * bd < half; g += U * bd) {
                T a[U], b[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const uint64_t j = idx(g + u * bd);
                    a[u] = at(j);
                    b[u] = at(j ^ tm.x);
                }
#pragma unroll
                for (int u = 0; u < U; ++u) add(idx(g + u * bd), a[u], b[u]);
            }
            for (; g < half; g += bd) {
                const uint64_t j = idx(g);
                add(j, at(j), at(j ^ tm.x));
            }
        }
        // Re(i^{ny} (sr + i si))
        double re;
        switch (tm.ny & 3) {
        case 0: re = sr; break;
        case 1: re = -si; break;
        case 2: re = -sr; break;
        default: re = si; break;
        }
        acc += tm.c * re;
    }
    return acc;
}

// One tile t of a pass over a state in global memory (`slot`): load it (from
// |0...0> on the circuit's first pass), apply the pass's ops in LDS, store
// it.  The whole workgroup calls it; it ends with a barrier.
template <typename R, int KM>
__device__ __forceinline__ void batch_tile(typename VT<R>::T *tile, typename VT<R>::T *slot,
                                           const BatchPass &bp, uint64_t t, bool init,
                                           const TileOp *__restrict__ ops,
                                           const typename VT<R>::T *__restrict__ pool) {
    using T = typename VT<R>::T;
    const uint32_t tid = threadIdx.x;
    const int m = bp.m;
    const uint32_t *tpos = bp.tpos;
    const uint32_t tsize = 1u << m;
    // loads in flight per thread while a tile comes in or goes out
    constexpr int LD = sizeof(R) == 4 ? 8 : 4;
    // thread part of local index j0 + tid (used when tsize >= LD kNT)
    const uint64_t dep_tid = deposit_bits(tid, tpos, m < 8 ? m : 8);
    const uint32_t swz_tid = swz<R>(tid);
    uint64_t base = t;
    for (int i = 0; i < m; ++i) {
        const uint64_t lowm = (1ull << tpos[i]) - 1;
        base = ((base & ~lowm) << 1) | (base & lowm);
    }
    // loads go out LD at a time, before their LDS writes (tiles of at least
    // LD * kNT amplitudes; smaller ones one at a time)
    if (tsize < LD * kNT) {
        for (uint32_t l = tid; l < tsize; l += kNT) {
            const uint64_t gi = base | deposit_bits(l, tpos, m);
            T v;
            if (init) {
                v.x = (gi == 0) ? R(1) : R(0);
                v.y = R(0);
            } else {
                v = slot[gi];
            }
            tile[swz<R>(l)] = v;
        }
    } else for (uint32_t j0 = 0; j0 < tsize; j0 += LD * kNT) {
        T v[LD];
#pragma unroll
        for (int u = 0; u < LD; ++u) {
            const uint64_t gi = base | dep_tid | deposit_bits(j0 + u * kNT, tpos, m);
            if (init) {
                v[u].x = (gi == 0) ? R(1) : R(0);
                v[u].y = R(0);
            } else {
                v[u] = slot[gi];
            }
        }
#pragma unroll
        for (int u = 0; u < LD; ++u) tile[swz_tid ^ swz<R>(j0 + u * kNT)] = v[u];
    }
    __syncthreads();
    for (int o = 0; o < bp.op_count; ++o) {
        lds_op<R, KM>(tile, m, base, tpos, ops[bp.op_begin + o], pool);
        __syncthreads();
    }
    if (tsize < LD * kNT) {
        for (uint32_t l = tid; l < tsize; l += kNT)
            slot[base | deposit_bits(l, tpos, m)] = tile[swz<R>(l)];
    } else for (uint32_t j0 = 0; j0 < tsize; j0 += LD * kNT) {
        T v[LD];
#pragma unroll
        for (int u = 0; u < LD; ++u) v[u] = tile[swz_tid ^ swz<R>(j0 + u * kNT)];
#pragma unroll
        for (int u = 0; u < LD; ++u)
            slot[base | dep_tid | deposit_bits(j0 + u * kNT, tpos, m)] = v[u];
    }
    __syncthreads();
}

template <typename R, int KM>
__global__ __launch_bounds__(kNT) void k_batch(const BatchCircuit *__restrict__ circuits,
                                               const int32_t *__restrict__ order, int count,
                                               const BatchPass *__restrict__ passes,
                                               const TileOp *__restrict__ ops,
                                               const typename VT<R>::T *__restrict__ pool,
                                               const BatchTerm *__restrict__ terms,
                                               typename VT<R>::T *__restrict__ scratch,
                                               uint64_t slot_amps, int mb,
                                               unsigned int *counter, double *out) {
    using T = typename VT<R>::T;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    T *tile = reinterpret_cast<T *>(smem_raw);
    __shared__ int s_next;
    __shared__ double sh[16];
    T *slot = scratch + (uint64_t)blockIdx.x * slot_amps;
    const uint32_t tid = threadIdx.x;
    for (;;) {
        if (tid == 0) s_next = (int)atomicAdd(counter, 1u);
        __syncthreads();
        const int ci = s_next;
        __syncthreads();
        if (ci >= count) break;
        const BatchCircuit bc = circuits[order[ci]];
        const int n = bc.n;
        double part;
        if (n <= mb) {
            // whole state in LDS: |0...0>, every op of the single pass, <H>
            const uint32_t dim = 1u << n;
            for (uint32_t l = tid; l < dim; l += kNT) {
                T v;
                v.x = (l == 0) ? R(1) : R(0);
                v.y = R(0);
                tile[swz<R>(l)] = v;
            }
            __syncthreads();
            for (int p = 0; p < bc.pass_count; ++p) {
                const BatchPass &bp = passes[bc.pass_begin + p];
                for (int o = 0; o < bp.op_count; ++o) {
                    lds_op<R, KM>(tile, n, 0, kIdentityPos, ops[bp.op_begin + o], pool);
                    __syncthreads();
                }
            }
            part = pauli_partial<R, true>(tile, n, terms + bc.term_begin, bc.term_count, 0,
                                          1ull << n);
        } else {
            // state in this workgroup's global slot, updated by tile passes
            for (int p = 0; p < bc.pass_count; ++p) {
                const BatchPass &bp = passes[bc.pass_begin + p];
                const uint64_t ntiles = 1ull << (n - bp.m);
                for (uint64_t t = 0; t < ntiles; ++t)
                    batch_tile<R, KM>(tile, slot, bp, t, p == 0, ops, pool);
            }
            if (bc.pass_count == 0) {
                const uint64_t dim = 1ull << n;
                for (uint64_t j = tid; j < dim; j += kNT) {
                    T v;
                    v.x = (j == 0) ? R(1) : R(0);
                    v.y = R(0);
                    slot[j] = v;
                }
                __syncthreads();
            }
            part = pauli_partial<R, false>(slot, n, terms + bc.term_begin, bc.term_count, 0,
                                           1ull << n);
        }
        const double tot = block_sum_b<R>(part, sh);
        if (tid == 0) out[bc.out_index] = tot;
        __syncthreads();
    }
}

__global__ void k_reset_counter(unsigned int *counter) { *counter = 0u; }

// ------------------------------------------------------ pass-major circuits
// Segment of work item `it`: the last segment whose first item is <= it (the
// host orders a launch's segments by first item, the first one at 0).
__device__ __forceinline__ int find_seg(const BatchSeg *__restrict__ segs, int nseg,
                                        uint64_t it) {
    int lo = 0, hi = nseg - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (segs[mid].first <= it) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// One pass index of every pass-major circuit: work item = (circuit, tile),
// taken by the workgroups in a fixed stride (no counter, no waiting).  The
// kernel boundary orders a circuit's passes.
template <typename R, int KM>
__global__ __launch_bounds__(kNT) void k_batch_pass(const BatchSeg *__restrict__ segs, int nseg,
                                                    uint64_t items,
                                                    const BatchPass *__restrict__ passes,
                                                    const TileOp *__restrict__ ops,
                                                    const typename VT<R>::T *__restrict__ pool,
                                                    typename VT<R>::T *__restrict__ states) {
    using T = typename VT<R>::T;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    T *tile = reinterpret_cast<T *>(smem_raw);
    for (uint64_t it = blockIdx.x; it < items; it += gridDim.x) {
        const BatchSeg sg = segs[find_seg(segs, nseg, it)];
        batch_tile<R, KM>(tile, states + sg.state_off, passes[sg.pass], it - sg.first,
                          sg.init != 0, ops, pool);
    }
}

// The Pauli sums of the pass-major circuits: work item = (circuit, chunk k of
// C = 2^cl indices, cl = min(chunk_log, n)); partial[item] = the chunk's
// share of sum_t c_t <P_t>.  The chunk is read once, into registers (NR
// amplitudes per thread) and into LDS, and serves every term.  A term with X
// letters pairs j with j ^ x; the pair is taken by the chunk of its member with
// bit h = 0 (h: the highest X bit): within the chunk when h < cl, else by the
// chunks whose index has bit h - cl clear, which read the partner chunk
// k ^ (x >> cl) from memory.  So a term reads half a state from memory instead
// of a whole one, and a string of Z letters none.
// A pair costs one product (Re or Im of conj(b) a, by the parity of n_Y) and a
// signed add: the sign splits into the chunk's and thread's, which go in with
// the coefficient, and the register's, uniform.  Workgroups of one XCD take a
// contiguous range of the items, so that a circuit's chunks are read again from
// that XCD's L2.  Bound by those reads and the products together: 192 circuits
// of 8 to 20 qubits with 64 strings each (complex64) 0.57 ms, 14 TB/s of partner
// reads; 1.20 with four sign tests and both products per pair and chunks dealt
// out over all XCDs.
template <typename R>
__global__ __launch_bounds__(kNT) void k_batch_pauli(const BatchSeg *__restrict__ segs, int nseg,
                                                     uint64_t items,
                                                     const BatchCircuit *__restrict__ circuits,
                                                     const BatchTerm *__restrict__ terms,
                                                     const typename VT<R>::T *__restrict__ states,
                                                     double *__restrict__ partial) {
    using T = typename VT<R>::T;
    constexpr int RBITS = sizeof(R) == 4 ? 4 : 3, NR = 1 << RBITS;
    constexpr int LOG = 8 + RBITS;
    static_assert(kNT == 256, "thread bits");
    __shared__ __align__(16) T ch[1 << LOG];
    __shared__ double sh[16];
    const uint32_t tid = threadIdx.x;
    const uint64_t xcd = blockIdx.x & (kXcds - 1), per = gridDim.x / kXcds;
    const uint64_t it1 = xcd_first(items, xcd + 1);
    for (uint64_t it = xcd_first(items, xcd) + blockIdx.x / kXcds; it < it1; it += per) {
        const BatchSeg sg = segs[find_seg(segs, nseg, it)];
        const BatchCircuit bc = circuits[sg.circuit];
        const int cl = LOG < bc.n ? LOG : bc.n;
        const uint32_t C = 1u << cl;
        const uint64_t j0 = (it - sg.first) << cl;
        const T *st = states + sg.state_off;
        T a[NR];
#pragma unroll
        for (int u = 0; u < NR; ++u) {
            a[u].x = a[u].y = R(0);
            if ((uint32_t)u * kNT + tid < C) a[u] = st[j0 + (uint32_t)u * kNT + tid];
        }
#pragma unroll
        for (int u = 0; u < NR; ++u) ch[(uint32_t)u * kNT + tid] = a[u];
        __syncthreads();
        double acc = 0.0;
        for (int t = 0; t < bc.term_count; ++t) {
            const BatchTerm &tm = terms[bc.term_begin + t];
            const uint64_t x = tm.x, z = tm.z;
            const int h = x ? 63 - __builtin_clzll(x) : -1;
            const bool far = h >= cl;
            if (far && ((j0 >> h) & 1)) continue;
            const uint32_t xthr = (uint32_t)x & (kNT - 1), xr = ((uint32_t)x & (C - 1)) >> 8;
            // registers that stand for pairs: all, or those with the highest X
            // bit clear where it is a register bit
            uint32_t take = (1u << NR) - 1;
            if (!far && xr) {
                const int hb = 31 - __builtin_clz(xr);
                take &= hb == 0 ? 0x5555u : hb == 1 ? 0x3333u : hb == 2 ? 0x0f0fu : 0x00ffu;
            }
            T b[NR];
            if (far) {
                const T *pp = st + ((j0 ^ x) & ~(uint64_t)(C - 1));
#pragma unroll
                for (int u = 0; u < NR; ++u) b[u] = pp[(((uint32_t)u ^ xr) << 8) + (tid ^ xthr)];
            } else {
#pragma unroll
                for (int u = 0; u < NR; ++u) b[u] = ch[(((uint32_t)u ^ xr) << 8) + (tid ^ xthr)];
            }
            // sign of register u: parity of u and the Z mask's register bits
            const uint32_t zr = (uint32_t)(z >> 8);
            uint32_t sreg = 0;
            if (zr & 1) sreg ^= 0xaaaau;
            if (zr & 2) sreg ^= 0xccccu;
            if (zr & 4) sreg ^= 0xf0f0u;
            if (NR > 8 && (zr & 8)) sreg ^= 0xff00u;
            double local = 0.0;
            if (tm.ny & 1) {
#pragma unroll
                for (int u = 0; u < NR; ++u) {
                    if (!((take >> u) & 1)) continue;
                    const double q = __builtin_fma((double)b[u].x, (double)a[u].y,
                                                   -((double)b[u].y * (double)a[u].x));
                    local = __builtin_fma(q, sign_of(sreg >> u), local);
                }
            } else {
#pragma unroll
                for (int u = 0; u < NR; ++u) {
                    if (!((take >> u) & 1)) continue;
                    const double q = __builtin_fma((double)b[u].x, (double)a[u].x,
                                                   (double)b[u].y * (double)a[u].y);
                    local = __builtin_fma(q, sign_of(sreg >> u), local);
                }
            }
            // i^{ny} times the pair's 2 Re (ny even) or 2 i Im (odd; the 2 goes to
            // the sum, the largest coefficients have no room for it); without X
            // letters, or where both members of every pair are summed, 1
            const int ny = tm.ny & 3;
            const double c = ny == 0 || ny == 3 ? tm.c : -tm.c;
            if (far || xr) local *= 2.0;
            const uint32_t s = (uint32_t)(__popcll(j0 & z) + __popc(tid & (uint32_t)z)) & 1u;
            acc = __builtin_fma(local, s ? -c : c, acc);
        }
        const double tot = block_sum_b<R>(acc, sh);
        if (tid == 0) partial[it] = tot;
        __syncthreads();   // the chunk and sh are rewritten by the next item
    }
}

// <H> of each pass-major circuit: its chunk sums added by one wave in a fixed
// order (the same on every run).
__global__ __launch_bounds__(256) void k_batch_finish(const BatchSeg *__restrict__ segs, int nseg,
                                                      uint64_t items,
                                                      const BatchCircuit *__restrict__ circuits,
                                                      const double *__restrict__ partial,
                                                      double *__restrict__ out) {
    const int s = (int)(blockIdx.x * 4 + (threadIdx.x >> 6)), lane = threadIdx.x & 63;
    if (s >= nseg) return;
    const uint64_t b = segs[s].first, e = s + 1 < nseg ? segs[s + 1].first : items;
    double acc = 0.0;
    for (uint64_t i = b + lane; i < e; i += 64) acc += partial[i];
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_down(acc, o, 64);
    if (lane == 0) out[circuits[segs[s].circuit].out_index] = acc;
}

template <typename R, int KM>
static hipError_t batch_t(const BatchLaunch &L, hipStream_t s) {
    using T = typename VT<R>::T;
    const size_t lds = sizeof(T) << L.mb;
    static size_t attr = 0;
    if (attr < lds) {
        hipError_t e = hipFuncSetAttribute((const void *)k_batch<R, KM>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        attr = lds;
    }
    if (L.count > 0) {
        // Beside pass-major launches the circuits in LDS run on a stream of
        // their own: they share nothing but the plan, and alone they leave most
        // of the chip idle.
        hipStream_t w = s;
        if (L.pass_major) {
            w = L.side;
            hipError_t e = hipEventRecord(L.fork, s);
            if (e == hipSuccess) e = hipStreamWaitEvent(w, L.fork, 0);
            if (e != hipSuccess) return e;
        }
        hipLaunchKernelGGL(k_reset_counter, dim3(1), dim3(1), 0, w, L.counter);
        hipLaunchKernelGGL((k_batch<R, KM>), dim3(L.grid), dim3(kNT), lds, w, L.circuits,
                           L.order, L.count, L.passes, L.ops, (const T *)L.pool, L.terms,
                           (T *)L.scratch, L.slot_amps, L.mb, L.counter, L.out);
        hipError_t e = hipGetLastError();
        if (e == hipSuccess && L.pass_major) e = hipEventRecord(L.join, w);
        if (e != hipSuccess) return e;
    }
    if (!L.pass_major) return hipSuccess;
    for (int i = 0; i < L.n_reg_launches; ++i) {
        const int sb = L.reg_seg_begin[i], ns = L.reg_seg_begin[i + 1] - sb;
        hipError_t e = launch_tile_reg_batch(sizeof(R) == 8 ? 0 : 1, L.reg_dg[i], L.states,
                                             L.reg_segs + sb, ns, L.reg_items[i], L.tas, L.rops,
                                             L.reg_pool, L.reg_img_max, s);
        if (e != hipSuccess) return e;
    }
    static size_t attr_p = 0;
    if (attr_p < lds) {
        hipError_t e = hipFuncSetAttribute((const void *)k_batch_pass<R, KM>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        attr_p = lds;
    }
    for (int i = 0; i <= L.n_pass_launches; ++i) {
        const int sb = L.seg_begin[i], ns = L.seg_begin[i + 1] - sb;
        const uint64_t items = L.items[i];
        if (items == 0 || ns <= 0) continue;
        const unsigned grid = (unsigned)std::min<uint64_t>(items, L.grid_big);
        if (i < L.n_pass_launches) {
            hipLaunchKernelGGL((k_batch_pass<R, KM>), dim3(grid), dim3(kNT), lds, s, L.segs + sb,
                               ns, items, L.passes, L.ops, (const T *)L.pool, (T *)L.states);
        } else {
            int occ = 0;
            hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
                &occ, reinterpret_cast<const void *>(k_batch_pauli<R>), kNT, 0);
            if (e != hipSuccess) return e;
            const unsigned pg = xcd_grid(items, (uint64_t)L.cus * std::max(1, occ));
            hipLaunchKernelGGL((k_batch_pauli<R>), dim3(pg), dim3(kNT), 0, s, L.segs + sb, ns, items,
                               L.circuits, L.terms, (const T *)L.states, L.partial);
            hipLaunchKernelGGL(k_batch_finish, dim3((ns + 3) / 4), dim3(256), 0, s, L.segs + sb, ns,
                               items, L.circuits, (const double *)L.partial, L.out);
        }
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return L.count > 0 ? hipStreamWaitEvent(s, L.join, 0) : hipSuccess;
}

// Kernel variant for the widest matrix-core op of the batch: up to 3 qubits
// (the autotuned fusion widths) or up to 5 (wider user gates).
hipError_t batch_launch(int dtype, const BatchLaunch &L, hipStream_t s) {
    if (L.mfma_k > 5) return hipErrorInvalidValue;
    if (dtype == 0)
        return L.mfma_k <= 3 ? batch_t<double, 3>(L, s) : batch_t<double, 5>(L, s);
    return L.mfma_k <= 3 ? batch_t<float, 3>(L, s) : batch_t<float, 5>(L, s);
}

template <typename R, int KM>
static int batch_occ_t(int mb) {
    using T = typename VT<R>::T;
    int blocks = 0;
    (void)hipFuncSetAttribute((const void *)k_batch<R, KM>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)(sizeof(T) << mb));
    const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
        &blocks, k_batch<R, KM>, kNT, sizeof(T) << mb);
    return e == hipSuccess ? blocks : 0;
}

template <typename R, int KM>
static int batch_pass_occ_t(int mb) {
    using T = typename VT<R>::T;
    int blocks = 0;
    (void)hipFuncSetAttribute((const void *)k_batch_pass<R, KM>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)(sizeof(T) << mb));
    const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
        &blocks, k_batch_pass<R, KM>, kNT, sizeof(T) << mb);
    return e == hipSuccess ? blocks : 0;
}

int batch_pass_occupancy(int dtype, int mb, int mfma_k) {
    if (dtype == 0)
        return mfma_k <= 3 ? batch_pass_occ_t<double, 3>(mb) : batch_pass_occ_t<double, 5>(mb);
    return mfma_k <= 3 ? batch_pass_occ_t<float, 3>(mb) : batch_pass_occ_t<float, 5>(mb);
}

int batch_occupancy(int dtype, int mb, int mfma_k) {
    if (dtype == 0) return mfma_k <= 3 ? batch_occ_t<double, 3>(mb) : batch_occ_t<double, 5>(mb);
    return mfma_k <= 3 ? batch_occ_t<float, 3>(mb) : batch_occ_t<float, 5>(mb);
}

}  // namespace dev
}  // namespace qsv
