// LDS-tile passes for gfx950.  One workgroup owns a tile: the 2^m amplitudes
// whose indices agree outside the m tile bits.  The tile is read from HBM
// once, every operation of the pass is applied to it on chip, and it is
// written back once, so a pass costs one read and one write of the state
// whatever the number of gates it holds (the lazily cached gates of Sec.
// 4.3.2 executed in bulk).
//
// Two kernels:
//  * k_tile_reg<R, RB, TB, DG> (tile_reg.hpp): m = RB + TB.  Each of the 2^TB threads keeps
//    2^RB amplitudes in registers.  Register bit j and thread bit i each
//    stand for one tile bit (the layout).  1- and 2-qubit operations on
//    register bits run in registers, as complex matrices or, when the host
//    split them into phases times a real matrix, as real matrices at half the
//    arithmetic; diagonal operations multiply by factors from tables that the
//    workgroup keeps in LDS; a REMAP op moves the tile through LDS (XOR
//    swizzled against bank conflicts) into a new layout.  Every
//    layout-dependent offset comes precomputed from the host.  Passes holding
//    wider operations use k_tile_lds.
//  * k_tile_lds<R>: any m <= 14; the tile lives in LDS and every operation
//    sweeps it (used for small states).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "device.hpp"
#include "lds_ops.hpp"
#include "tile_reg.hpp"

namespace qsv {
namespace dev {

// ------------------------------------------------------- k_tile_lds
// Persistent like k_tile_reg: resident workgroups take tiles from a per-pass
// counter that the host zeroes.
template <typename R, int KM>
__global__ __launch_bounds__(kNT) void k_tile_lds(typename VT<R>::T *__restrict__ psi,
                                                  TileArgs ta, const TileOp *__restrict__ ops,
                                                  const typename VT<R>::T *__restrict__ pool,
                                                  unsigned int *__restrict__ counter) {
    using T = typename VT<R>::T;
    // the tile at the start of dynamic LDS (address 0), the tile counter's
    // broadcast slot right after it
    extern __shared__ __align__(16) unsigned char smem_raw[];
    T *tile = reinterpret_cast<T *>(smem_raw);
    unsigned int &s_tile = *reinterpret_cast<unsigned int *>(smem_raw + (sizeof(T) << ta.m));
    const int m = ta.m;
    const uint32_t tsize = 1u << m;
    const uint32_t tid = threadIdx.x;
    Warm warm;
    warm.ask<kNT>(ops, (uint32_t)ta.n_ops * (uint32_t)sizeof(TileOp), tid);
    // this thread's share of every tile: local indices j + tid, j = 0, kNT, ...
    const uint64_t dep_tid = deposit_bits(tid & (tsize - 1), ta.tpos, m);
    const uint64_t dep_tid_f = deposit_bits(tid & (tsize - 1), ta.spos, m);
    const uint32_t swz_tid = swz<R>(tid & (tsize - 1));
    const uint32_t n_tiles = (uint32_t)ta.n_tiles;
    if (tid == 0) s_tile = atomicAdd(counter, 1u);
    warm.settle();
    __syncthreads();
    uint32_t t = __builtin_amdgcn_readfirstlane(s_tile);
    while (t < n_tiles) {
        uint64_t base = t;
        for (int i = 0; i < m; ++i) {
            const uint64_t lowm = (1ull << ta.tpos[i]) - 1;
            base = ((base & ~lowm) << 1) | (base & lowm);
        }
        // loads in batches of 8 per thread, all in flight before their LDS
        // writes (one HBM round trip per batch, not per amplitude)
        if (tsize >= 8 * kNT) {
            for (uint32_t j0 = 0; j0 < tsize; j0 += 8 * kNT) {
                T v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    v[u] = gload(psi + (base | dep_tid | ta.dep_hi[(j0 >> 8) + u]));
#pragma unroll
                for (int u = 0; u < 8; ++u) tile[swz_tid ^ swz<R>(j0 + u * kNT)] = v[u];
            }
        } else {
            for (uint32_t j = 0; j < tsize; j += kNT)
                if (j + tid < tsize)
                    tile[swz_tid ^ swz<R>(j)] = gload(psi + (base | dep_tid | ta.dep_hi[j >> 8]));
        }
        unsigned int next = 0;
        if (tid == 0) next = atomicAdd(counter, 1u);
        // normal priority for the ops; raised again for the stores and the
        // next tile's loads (see k_tile_reg)
        __builtin_amdgcn_s_setprio(0);
        __syncthreads();
        for (int oi = 0; oi < ta.n_ops; ++oi) {
            lds_op<R, KM>(tile, m, base, ta.tpos, ops[oi], pool, ta.dep_hi);
            __syncthreads();
        }
        __builtin_amdgcn_s_setprio(2);
        if (tsize >= 8 * kNT) {
            for (uint32_t j0 = 0; j0 < tsize; j0 += 8 * kNT) {
                T v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = tile[swz_tid ^ swz<R>(j0 + u * kNT)];
#pragma unroll
                for (int u = 0; u < 8; ++u)
                    gstore(psi + (base | dep_tid_f | ta.dep_hi_f[(j0 >> 8) + u]), v[u]);
            }
        } else {
            for (uint32_t j = 0; j < tsize; j += kNT)
                if (j + tid < tsize)
                    gstore(psi + (base | dep_tid_f | ta.dep_hi_f[j >> 8]), tile[swz_tid ^ swz<R>(j)]);
        }
        if (tid == 0) s_tile = next;
        __syncthreads();
        t = __builtin_amdgcn_readfirstlane(s_tile);
    }
}

hipError_t launch_tile_reg_batch(int dtype, int dg, void *states, const RegSeg *segs, int nseg,
                                 uint64_t items, const TileArgs *tas, const RegOp *rops,
                                 const void *pool, uint32_t img_max, hipStream_t s) {
    return dtype == 0 ? tile_reg_batch_f64(dg, states, segs, nseg, items, tas, rops, pool, img_max, s)
                      : tile_reg_batch_f32(dg, states, segs, nseg, items, tas, rops, pool, img_max, s);
}

int tile_pass_max_bits(int dtype) { return dtype == 0 ? 13 : 14; }
// 16 amplitudes per thread: 64 VGPRs of state for complex128, 32 for complex64
int tile_reg_bits(int) { return 4; }

template <typename R, int KM>
static hipError_t launch_lds_t(void *psi, const TileArgs &ta, const TileOp *ops, const void *pool,
                               unsigned int *counter, hipStream_t s) {
    using T = typename VT<R>::T;
    const int max_bits = tile_pass_max_bits(sizeof(R) == 8 ? 0 : 1);
    static bool attr = false;
    if (!attr) {
        hipError_t e = set_lds_attr(k_tile_lds<R, KM>, (sizeof(T) << max_bits) + 16);
        if (e != hipSuccess) return e;
        attr = true;
    }
    if (ta.n_tiles == 0) return hipSuccess;
    if (ta.n_tiles > 0xffffffffull - 65536) return hipErrorInvalidValue;
    // resident workgroups per compute unit for each tile size
    static int per_cu[16] = {0};
    static int cus = 0;
    const size_t lds = (sizeof(T) << ta.m) + 16;   // tile + counter slot
    if (per_cu[ta.m] == 0) {
        int dev = 0, occ = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e == hipSuccess && cus == 0)
            e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
        if (e == hipSuccess)
            e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
                &occ, reinterpret_cast<const void *>(k_tile_lds<R, KM>), kNT, lds);
        if (e != hipSuccess) return e;
        per_cu[ta.m] = std::max(1, occ);
    }
    const uint64_t resident = (uint64_t)std::max(1, cus) * per_cu[ta.m];
    const unsigned grid = (unsigned)std::min<uint64_t>(ta.n_tiles, resident);
    hipLaunchKernelGGL((k_tile_lds<R, KM>), dim3(grid), dim3(kNT), lds, s, (T *)psi, ta, ops,
                       (const T *)pool, counter);
    return hipGetLastError();
}

template <typename R>
static hipError_t launch_lds_k(void *psi, const TileArgs &ta, const TileOp *ops, const void *pool,
                               unsigned int *counter, hipStream_t s) {
    switch (ta.mfma_k) {
    case 0: return launch_lds_t<R, 0>(psi, ta, ops, pool, counter, s);
    case 3: return launch_lds_t<R, 3>(psi, ta, ops, pool, counter, s);
    case 4: return launch_lds_t<R, 4>(psi, ta, ops, pool, counter, s);
    case 5: return launch_lds_t<R, 5>(psi, ta, ops, pool, counter, s);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_tile_pass(int dtype, void *psi, const TileArgs &ta, const TileOp *ops,
                            const void *pool, unsigned int *counter, hipStream_t s) {
    if (ta.m < 1 || ta.m > tile_pass_max_bits(dtype)) return hipErrorInvalidValue;
    return dtype == 0 ? launch_lds_k<double>(psi, ta, ops, pool, counter, s)
                      : launch_lds_k<float>(psi, ta, ops, pool, counter, s);
}

hipError_t launch_tile_reg(int dtype, void *psi, const TileArgs &ta, const RegOp *rops,
                           const void *pool, unsigned int *counter, hipStream_t s) {
    if (ta.rb == 4 && ta.m == 12)
        return dtype == 0 ? tile_reg_f64(psi, ta, rops, pool, counter, s)
                          : tile_reg_f32(psi, ta, rops, pool, counter, s);
    return dtype == 0 ? tile_reg_shapes_f64(psi, ta, rops, pool, counter, s)
                      : tile_reg_shapes_f32(psi, ta, rops, pool, counter, s);
}

}  // namespace dev
}  // namespace qsv
