// The register-resident tile kernels k_tile_reg and k_tile_reg_batch (see
// kernels_tile.hip) and their launchers; the instances are spread over
// kernels_tile_reg*.hip, one translation unit per precision and set of shapes.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>

#include "device.hpp"
#include "lds_ops.hpp"

namespace qsv {
namespace dev {

template <typename K>
static hipError_t set_lds_attr(K kern, size_t bytes) {
    return hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)bytes);
}

__device__ __forceinline__ double rfma(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ __forceinline__ float rfma(float a, float b, float c) { return __builtin_fmaf(a, b, c); }

// Register ops run in place, one group of 2 or 4 amplitudes at a time, and
// never skip: an op under controls (CTRL) computes every group and keeps the
// old value where the controls fail, so the register allocation of the
// uncontrolled path holds no copies for a skipped case.  `on` is the lane's
// share of the controls (thread-id bits, bits outside the tile); creg holds
// the register bits that are controls.  Matrices arrive in scalar registers
// (m: the op's inline coefficients, row-major; complex ones as re, im).
template <typename T, typename R, int NR, int J, bool CTRL>
__device__ __forceinline__ void reg_g1(T *amp, const R *m, bool on, uint32_t creg) {
    T u[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        u[e].x = m[2 * e];
        u[e].y = m[2 * e + 1];
    }
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        if (i & (1 << J)) continue;
        const int i1 = i | (1 << J);
        const T a = amp[i], b = amp[i1];
        T na = cmul(u[0], a);
        na = cmadd(na, u[1], b);
        T nb = cmul(u[2], a);
        nb = cmadd(nb, u[3], b);
        if (CTRL) {
            const bool c = on && ((i & creg) == creg);
            na = csel(c, na, a);
            nb = csel(c, nb, b);
        }
        amp[i] = na;
        amp[i1] = nb;
    }
}

template <typename T, typename R, int NR, int J1, int J2, bool CTRL>
__device__ __forceinline__ void reg_g2(T *amp, const R *m, bool on, uint32_t creg) {
    T u[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) {
        u[e].x = m[2 * e];
        u[e].y = m[2 * e + 1];
    }
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        if (i & ((1 << J1) | (1 << J2))) continue;
        const int idx[4] = {i, i | (1 << J1), i | (1 << J2), i | (1 << J1) | (1 << J2)};
        T x[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) x[c] = amp[idx[c]];
        const bool c = !CTRL || (on && ((i & creg) == creg));
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            T y = cmul(u[r * 4], x[0]);
#pragma unroll
            for (int cc = 1; cc < 4; ++cc) y = cmadd(y, u[r * 4 + cc], x[cc]);
            amp[idx[r]] = CTRL ? csel(c, y, x[r]) : y;
        }
    }
}

// Real matrices: the real and imaginary parts of the amplitudes transform
// separately, 2 (1-qubit) or 4 (2-qubit) multiply-adds per part.
template <typename T, typename R, int NR, int J, bool CTRL>
__device__ __forceinline__ void reg_r1(T *amp, const R *m, bool on, uint32_t creg) {
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        if (i & (1 << J)) continue;
        const int i1 = i | (1 << J);
        const T a = amp[i], b = amp[i1];
        T na, nb;
        na.x = rfma(m[1], b.x, m[0] * a.x);
        na.y = rfma(m[1], b.y, m[0] * a.y);
        nb.x = rfma(m[3], b.x, m[2] * a.x);
        nb.y = rfma(m[3], b.y, m[2] * a.y);
        if (CTRL) {
            const bool c = on && ((i & creg) == creg);
            na = csel(c, na, a);
            nb = csel(c, nb, b);
        }
        amp[i] = na;
        amp[i1] = nb;
    }
}

template <typename T, typename R, int NR, int J1, int J2, bool CTRL>
__device__ __forceinline__ void reg_r2(T *amp, const R *m, bool on, uint32_t creg) {
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        if (i & ((1 << J1) | (1 << J2))) continue;
        const int idx[4] = {i, i | (1 << J1), i | (1 << J2), i | (1 << J1) | (1 << J2)};
        T x[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) x[c] = amp[idx[c]];
        const bool c = !CTRL || (on && ((i & creg) == creg));
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            T y;
            y.x = m[r * 4] * x[0].x;
            y.y = m[r * 4] * x[0].y;
#pragma unroll
            for (int cc = 1; cc < 4; ++cc) {
                y.x = rfma(m[r * 4 + cc], x[cc].x, y.x);
                y.y = rfma(m[r * 4 + cc], x[cc].y, y.y);
            }
            amp[idx[r]] = CTRL ? csel(c, y, x[r]) : y;
        }
    }
}

// Diagonal op: amplitude i of the thread takes the factor at byte offset
// (lane part ^ wave part ^ tile part ^ wr[i]) of the op's table in the LDS
// image; the lane part places the lane's table bits (a bit-field extract and
// a shift per lane bit).  The four parts come from disjoint table bits (lane
// and wave thread-id bits, bits outside the tile, register bits), so the XOR
// is their sum; the table sits at a multiple of its size, so the offset
// never leaves it.  Controls inside the tile are table bits; a tile that
// fails the controls outside it reads a table of ones (at byte offset b)
// rather than skipping the op.  The reads go out four at a time.
template <typename T, int NR>
__device__ __forceinline__ void reg_diag(T *amp, const RegOp &op, uint32_t limg_a,
                                         uint64_t base, uint32_t lane, uint32_t wave) {
    uint32_t wr[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i) wr[i] = op.wr[i];
    uint32_t sh[6];
#pragma unroll
    for (int t = 0; t < 6; ++t) sh[t] = op.rd[t];
    const uint64_t lmask = op.lane_ok;
    uint32_t s_idx = (uint32_t)op.mat;
    if ((base & op.octrl) != op.octrl) s_idx = (uint32_t)op.b;
    s_idx ^= op.wwave[wave];
    for (int q = 0; q < op.a; ++q)
        if ((base >> op.gt[q]) & 1) s_idx ^= op.gtb[q];
    // the image's LDS address (a multiple of every table's size) joins the
    // uniform part; the lane and register parts then still OR and XOR in
    uint32_t v_idx = s_idx + limg_a;
    if (lmask != 0) {   // uniform: tables without lane bits skip the lane part
#pragma unroll
        for (int t = 0; t < 6; ++t)
            v_idx |= __builtin_amdgcn_ubfe(lane, (uint32_t)t, (uint32_t)((lmask >> t) & 1u)) << sh[t];
    }
#pragma unroll
    for (int i0 = 0; i0 < NR; i0 += 4) {
        T f[4];
#pragma unroll
        for (int i = 0; i < 4 && i0 + i < NR; ++i) lds_read(v_idx ^ wr[i0 + i], f[i]);
#pragma unroll
        for (int i = 0; i < 4 && i0 + i < NR; ++i) amp[i0 + i] = cmul(f[i], amp[i0 + i]);
    }
}

// A group of tables over at most two register bits (B of them): the factors for
// the values of those bits first, every table's read and multiplied in, then
// the amplitudes once.  Per table 2^B reads and products instead of one per
// amplitude; the place fields decode in scalar registers.  (27-qubit QFT, its
// three passes of tables: 6.5 -> 4.55 ms.)
template <typename T, int B>
__device__ __forceinline__ void dgrp_factors(T *f, const RegOp &op, uint32_t limg_a, uint64_t base,
                                             uint32_t lane, uint32_t wave) {
    constexpr uint32_t LE = sizeof(T) == 16 ? 4 : 3;
    auto weight = [](uint32_t w, int k) {
        const uint32_t n = (w >> (4 * k)) & 15u;
        return n == 15u ? 0u : (1u << LE) << n;
    };
    for (int k = 0; k < op.a; ++k) {
        const DiagTab &d = op.dt[k];
        const uint64_t octrl = d.octrl, gpos = d.gpos;
        const uint32_t gplace = d.gplace, lw = d.lane, ww = d.wave;
        uint32_t s = (base & octrl) == octrl ? d.off : d.ones;
        const int outside = (int)(lw >> 24);
        for (int q = 0; q < outside; ++q)
            s |= (uint32_t)((base >> ((gpos >> (8 * q)) & 255u)) & 1u) << (((gplace >> (4 * q)) & 15u) + LE);
        if (wave & 1u) s |= weight(ww, 0);
        if (wave & 2u) s |= weight(ww, 1);
        if (wave & 4u) s |= weight(ww, 2);
        uint32_t v = s + limg_a;
        if ((lw & 0xffffffu) != 0xffffffu) {    // uniform
#pragma unroll
            for (int t = 0; t < 6; ++t) {
                const uint32_t n = (lw >> (4 * t)) & 15u;
                v |= __builtin_amdgcn_ubfe(lane, (uint32_t)t, n == 15u ? 0u : 1u) << (n + LE);
            }
        }
        const uint32_t w0 = weight(ww, 3), w1 = weight(ww, 4);
        T x[1 << B];
#pragma unroll
        for (int e = 0; e < (1 << B); ++e)
            lds_read(v | (e & 1 ? w0 : 0u) | (e & 2 ? w1 : 0u), x[e]);
        if (k == 0) {
#pragma unroll
            for (int e = 0; e < (1 << B); ++e) f[e] = x[e];
        } else {
#pragma unroll
            for (int e = 0; e < (1 << B); ++e) f[e] = cmul(x[e], f[e]);
        }
    }
}

template <typename T, int NR, int RB>
__device__ __forceinline__ void reg_dgrp(T *amp, const RegOp &op, uint32_t creg, uint32_t limg_a,
                                         uint64_t base, uint32_t lane, uint32_t wave) {
    const int bits = __popc(creg);
    T f[4];
    if (bits == 0) {
        dgrp_factors<T, 0>(f, op, limg_a, base, lane, wave);
#pragma unroll
        for (int i = 0; i < NR; ++i) amp[i] = cmul(f[0], amp[i]);
        return;
    }
    if (bits == 1) dgrp_factors<T, 1>(f, op, limg_a, base, lane, wave);
    else dgrp_factors<T, 2>(f, op, limg_a, base, lane, wave);
#define QSV_DG1(J)                                                                         \
    case 1 << (J):                                                                         \
        if constexpr (RB > (J)) {                                                          \
            _Pragma("unroll") for (int i = 0; i < NR; ++i)                                 \
                amp[i] = cmul(f[(i >> (J)) & 1], amp[i]);                                  \
        } else __builtin_unreachable();                                                    \
        break;
#define QSV_DG2(J, K)                                                                      \
    case (1 << (J)) | (1 << (K)):                                                          \
        if constexpr (RB > (K)) {                                                          \
            _Pragma("unroll") for (int i = 0; i < NR; ++i)                                 \
                amp[i] = cmul(f[((i >> (J)) & 1) | (((i >> (K)) & 1) << 1)], amp[i]);      \
        } else __builtin_unreachable();                                                    \
        break;
    switch (creg) {
        QSV_DG1(0) QSV_DG1(1) QSV_DG1(2) QSV_DG1(3) QSV_DG1(4)
        QSV_DG2(0, 1) QSV_DG2(0, 2) QSV_DG2(1, 2) QSV_DG2(0, 3) QSV_DG2(1, 3) QSV_DG2(2, 3)
        QSV_DG2(0, 4) QSV_DG2(1, 4) QSV_DG2(2, 4) QSV_DG2(3, 4)
    default: __builtin_unreachable();
    }
#undef QSV_DG2
#undef QSV_DG1
}

// Layout change through an LDS buffer of half a tile.  Slot J holds the same
// tile bit before and after, and the buffer drops that bit from the index.
// In phase p every thread writes its registers whose slot-J bit is p, then
// reads the same register indices in the new layout, so no register is
// overwritten before it was written out.  Addresses are the thread part XOR
// the (uniform) register part, both precomputed on the host; the register
// parts come in scalar registers, loaded before the first barrier.
// Ordering of LDS accesses within one wave: the wave's LDS operations run in
// order, so only the compiler has to be kept from moving them across.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// LOCAL: each wave on its own region of the buffer, no workgroup barrier; else
// the whole workgroup, which with `wait` first waits for every wave to leave its
// region of an earlier wave-local remap.
template <typename T, int NR, int J, bool LOCAL>
__device__ __forceinline__ void remap_half(T *amp, uint32_t wt, uint32_t rt,
                                           const uint32_t *wr, const uint32_t *rd, bool wait) {
    if (!LOCAL && wait) __syncthreads();
    // the thread parts pass through an empty asm in each phase, so the
    // addresses are formed next to their accesses (not all hoisted above the
    // barriers, which would hold 2^RB more VGPRs)
#pragma unroll
    for (int p = 0; p < 2; ++p) {
        uint32_t w = wt;
        asm volatile("" : "+v"(w));
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            if (((i >> J) & 1) != p) continue;
            lds_write(w ^ wr[i], amp[i]);
        }
        if (LOCAL) wave_sync();
        else __syncthreads();
        uint32_t r = rt;
        asm volatile("" : "+v"(r));
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            if (((i >> J) & 1) != p) continue;
            lds_read(r ^ rd[i], amp[i]);
        }
        if (LOCAL) wave_sync();
        else __syncthreads();
    }
}

template <typename R> __device__ __forceinline__ const R *op_mat(const RegOp &op);
template <> __device__ __forceinline__ const double *op_mat<double>(const RegOp &op) { return op.md; }
template <> __device__ __forceinline__ const float *op_mat<float>(const RegOp &op) { return op.mf; }

#define QSV_SLOT1(J, CALL)                                        \
    case J:                                                       \
        if constexpr (RB > J) { CALL; } else __builtin_unreachable(); \
        break;

template <typename T, typename R, int NR, int RB, bool CTRL>
__device__ __forceinline__ void dispatch_1(T *amp, int kind, int j, const R *m, bool on,
                                           uint32_t creg) {
    if (kind == ROP_R1) {
        switch (j) {
            QSV_SLOT1(0, (reg_r1<T, R, NR, 0, CTRL>(amp, m, on, creg)))
            QSV_SLOT1(1, (reg_r1<T, R, NR, 1, CTRL>(amp, m, on, creg)))
            QSV_SLOT1(2, (reg_r1<T, R, NR, 2, CTRL>(amp, m, on, creg)))
            QSV_SLOT1(3, (reg_r1<T, R, NR, 3, CTRL>(amp, m, on, creg)))
            QSV_SLOT1(4, (reg_r1<T, R, NR, 4, CTRL>(amp, m, on, creg)))
        default: __builtin_unreachable();
        }
    } else {
        switch (j) {
            QSV_SLOT1(0, (reg_g1<T, R, NR, 0, CTRL>(amp, m, on, creg)))
            QSV_SLOT1(1, (reg_g1<T, R, NR, 1, CTRL>(amp, m, on, creg)))
            QSV_SLOT1(2, (reg_g1<T, R, NR, 2, CTRL>(amp, m, on, creg)))
            QSV_SLOT1(3, (reg_g1<T, R, NR, 3, CTRL>(amp, m, on, creg)))
            QSV_SLOT1(4, (reg_g1<T, R, NR, 4, CTRL>(amp, m, on, creg)))
        default: __builtin_unreachable();
        }
    }
}

#define QSV_PAIRS                                                                               \
    QSV_PAIR(0, 1) QSV_PAIR(0, 2) QSV_PAIR(1, 2) QSV_PAIR(0, 3) QSV_PAIR(1, 3) QSV_PAIR(2, 3)   \
    QSV_PAIR(0, 4) QSV_PAIR(1, 4) QSV_PAIR(2, 4) QSV_PAIR(3, 4)

template <typename T, typename R, int NR, int RB, bool CTRL>
__device__ __forceinline__ void dispatch_r2(T *amp, int a, int b, const R *m, bool on,
                                            uint32_t creg) {
#define QSV_PAIR(A, B)                                                                   \
    case (A) * 8 + (B):                                                                  \
        if constexpr (RB > (B)) { reg_r2<T, R, NR, A, B, CTRL>(amp, m, on, creg); }      \
        else __builtin_unreachable();                                                    \
        break;
    switch (a * 8 + b) {
        QSV_PAIRS
    default: __builtin_unreachable();   // the host emits only valid slot pairs
    }
#undef QSV_PAIR
}

// m16: the first 16 of a complex matrix's 32 coefficients; it reads the others
// from the op.
template <typename T, typename R, int NR, int RB, bool CTRL>
__device__ __forceinline__ void dispatch_g2(T *amp, int a, int b, const R *m16, const RegOp &op,
                                            bool on, uint32_t creg) {
    R m[32];
    const R *src = op_mat<R>(op);
#pragma unroll
    for (int e = 0; e < 16; ++e) m[e] = m16[e];
#pragma unroll
    for (int e = 16; e < 32; ++e) m[e] = src[e];
#define QSV_PAIR(A, B)                                                                   \
    case (A) * 8 + (B):                                                                  \
        if constexpr (RB > (B)) { reg_g2<T, R, NR, A, B, CTRL>(amp, m, on, creg); }      \
        else __builtin_unreachable();                                                    \
        break;
    switch (a * 8 + b) {
        QSV_PAIRS
    default: __builtin_unreachable();
    }
#undef QSV_PAIR
}
#undef QSV_PAIRS

// One operation of a register program on the thread's amplitudes.  Every
// case writes every amplitude (no skipped op or group), see reg_g1.  The
// fields every op kind may need and the first 16 matrix coefficients are
// read up front, so their scalar loads go out in one burst and the op waits
// once instead of once per dependent field.  Three waves per SIMD cannot hide an
// op's serial latency (37 % of their time is waiting), so the way to the
// arithmetic is kept short: the kinds are told apart in the order of their
// numbers in heavy passes, controls are part of the kind, slot pairs are one
// switch, and wave-local and workgroup remaps are instances of their own
// (30-qubit brick 10.34 -> 10.17 ms per heavy pass, 28 qubits in complex64 1.776
// -> 1.738 ms, 20 qubits 71.5 -> 66.3 us).
template <typename T, typename R, int NR, int RB, int DG>
__device__ __forceinline__ void reg_op(T *amp, const RegOp &op, uint32_t lds_a, uint32_t limg_a,
                                       uint64_t base, uint32_t lane, uint32_t wave) {
    const int kind = op.kind;
    const int a = op.a, b = op.b;
    const R *mp = op_mat<R>(op);
    R m16[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) m16[e] = mp[e];
    if (kind == ROP_R2) {
        dispatch_r2<T, R, NR, RB, false>(amp, a, b, m16, true, 0);
    } else if (DG > 0 && kind == ROP_DIAG) {
        reg_diag<T, NR>(amp, op, limg_a, base, lane, wave);
    } else if (kind == ROP_REMAP) {
        uint32_t wr[NR], rd[NR];
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            wr[i] = op.wr[i];
            rd[i] = op.rd[i];
        }
        // the remap buffer's LDS address (a multiple of its size) joins the
        // thread parts; the register parts then XOR in
        const uint32_t lw = limg_a + op.lane_off + 4u * lane;
        const uint32_t wt = (lds_read_u32(lw) ^ op.wwave[wave]) + lds_a;
        const uint32_t rt = (lds_read_u32(lw + 256u) ^ op.rwave[wave]) + lds_a;
        // raised priority through the remap (LDS round trips and barriers
        // that the whole workgroup waits on), as for the tile's stores and
        // loads
        __builtin_amdgcn_s_setprio(2);
        if (b == 1) {
            switch (a) {
                QSV_SLOT1(0, (remap_half<T, NR, 0, true>(amp, wt, rt, wr, rd, false)))
                QSV_SLOT1(1, (remap_half<T, NR, 1, true>(amp, wt, rt, wr, rd, false)))
                QSV_SLOT1(2, (remap_half<T, NR, 2, true>(amp, wt, rt, wr, rd, false)))
                QSV_SLOT1(3, (remap_half<T, NR, 3, true>(amp, wt, rt, wr, rd, false)))
                QSV_SLOT1(4, (remap_half<T, NR, 4, true>(amp, wt, rt, wr, rd, false)))
            default: __builtin_unreachable();
            }
        } else {
            switch (a) {
                QSV_SLOT1(0, (remap_half<T, NR, 0, false>(amp, wt, rt, wr, rd, b == 2)))
                QSV_SLOT1(1, (remap_half<T, NR, 1, false>(amp, wt, rt, wr, rd, b == 2)))
                QSV_SLOT1(2, (remap_half<T, NR, 2, false>(amp, wt, rt, wr, rd, b == 2)))
                QSV_SLOT1(3, (remap_half<T, NR, 3, false>(amp, wt, rt, wr, rd, b == 2)))
                QSV_SLOT1(4, (remap_half<T, NR, 4, false>(amp, wt, rt, wr, rd, b == 2)))
            default: __builtin_unreachable();
            }
        }
        __builtin_amdgcn_s_setprio(0);
    } else if (DG > 1 && kind == ROP_DGRP) {
        reg_dgrp<T, NR, RB>(amp, op, op.creg, limg_a, base, lane, wave);
    } else if (kind == ROP_G2) {
        dispatch_g2<T, R, NR, RB, false>(amp, a, b, m16, op, true, 0);
    } else if (kind < ROP_CTRL) {
        dispatch_1<T, R, NR, RB, false>(amp, kind, a, m16, true, 0);
    } else {
        // controls outside the tile (uniform), on thread-id bits (lane and
        // wave masks) and on register bits (creg)
        const uint32_t creg = op.creg;
        const uint64_t octrl = op.octrl;
        const bool on = ((base & octrl) == octrl) && ((op.wave_ok >> wave) & 1u) &&
                        ((op.lane_ok >> lane) & 1ull);
        const int k = kind - ROP_CTRL;
        if (k == ROP_R2) dispatch_r2<T, R, NR, RB, true>(amp, a, b, m16, on, creg);
        else if (k == ROP_G2) dispatch_g2<T, R, NR, RB, true>(amp, a, b, m16, op, on, creg);
        else dispatch_1<T, R, NR, RB, true>(amp, k, a, m16, on, creg);
    }
}
#undef QSV_SLOT1

// Global index of the first amplitude of tile t: a 0 bit inserted at every
// tile position (opaque positions: their masks are not hoisted out of the
// tile loop into 2m spilled 64-bit values).
template <int M>
__device__ __forceinline__ uint64_t tile_base(uint32_t t, const TileArgs &ta) {
    uint64_t base = t;
#pragma unroll
    for (int i = 0; i < M; ++i) {
        uint32_t tp = ta.tpos[i];
        asm volatile("" : "+s"(tp));
        const uint64_t lowm = (1ull << tp) - 1;
        base = ((base & ~lowm) << 1) | (base & lowm);
    }
    return base;
}

// The t-th number, ascending, without a bit outside `live`.
__device__ __forceinline__ uint32_t live_tile(uint32_t t, uint32_t live) {
    uint32_t out = 0;
    for (; t; t >>= 1, live &= live - 1)
        if (t & 1u) out |= live & (0u - live);
    return out;
}

// Issue the loads of tile t in the load layout (this thread's part gl of the
// index).  The empty asms keep the per-register addresses and offsets from
// being hoisted out of the tile loop (as 2^RB 64-bit values they would
// spill); the offsets are a few scalar ORs per tile.
template <typename T, int RB, int M>
__device__ __forceinline__ void load_tile(T *dst, const T *__restrict__ psi, uint64_t gl,
                                          uint32_t t, const TileArgs &ta) {
    const uint64_t base = tile_base<M>(t, ta);
    const T *lp = psi + gl;
    asm volatile("" : "+v"(lp));
    lp += base;
    uint64_t gr[RB];
#pragma unroll
    for (int j = 0; j < RB; ++j) {
        gr[j] = ta.g_reg[j];
        asm volatile("" : "+s"(gr[j]));
    }
#pragma unroll
    for (int i = 0; i < (1 << RB); ++i) {
        uint64_t g = 0;
#pragma unroll
        for (int j = 0; j < RB; ++j)
            if ((i >> j) & 1) g |= gr[j];
        dst[i] = gload(lp + g);
    }
}

// Whether any amplitude of the wave is not zero.  The first register decides on
// most tiles of a dense state, for three ORs and one load's wait.
template <typename T, int NR>
__device__ __forceinline__ bool wave_live(const T *amp) {
    auto bits = [](const T &a) {
        if constexpr (sizeof(T) == 16) {
            const uint64_t v = __double_as_longlong(a.x) | __double_as_longlong(a.y);
            return (uint32_t)v | (uint32_t)(v >> 32);
        } else {
            return __float_as_uint(a.x) | __float_as_uint(a.y);
        }
    };
    uint32_t any = bits(amp[0]);
    if (__ballot(any != 0)) return true;
#pragma unroll
    for (int i = 1; i < NR; ++i) any |= bits(amp[i]);
    return __ballot(any != 0) != 0;
}

// Words behind the image, two slots each (tiles alternate): the claimed tile,
// and of the tile at hand whether a wave found an amplitude that is not zero
// and how many waves found none.
struct TileWords {
    uint32_t claim[2], live[2], zero[2], pad[2];
};

// Persistent: a grid of resident workgroups takes tiles from a per-pass
// counter that the host zeroes (see below).  Dynamic LDS: the half-tile remap
// buffer (a workgroup remap uses all of it, a wave-local one its wave's
// share), then the pass's image (tables and per-lane words), copied in once per
// workgroup, then TileWords.
//
// Tiles that hold only zeros stay as they are: of a state that began as
// |0...0> the first pass finds one tile that is not zero, the second 2^(the
// first's tile bits outside its own), and the others cost their read (16 GiB:
// 12.5 -> 3.7 ms for a heavy pass; 27-qubit QFT 7.0 -> 4.7 ms in all).  A wave
// with an amplitude that is not zero goes on at once; the others wait until such
// a wave has shown up or none has (a look at the tile by all waves together
// would cost dense tiles a barrier: 28 qubits, all amplitudes random, are
// unchanged at 26.2 ms for ten layers).
// DG: the table ops that the instance has (0 none, 1 DIAG, 2 DIAG and DGRP);
// programs run on the leanest that will do, whose register allocation the other
// cases do not burden.
template <typename R, int RB, int TB, int DG>
__global__ __launch_bounds__(1 << TB) void k_tile_reg(typename VT<R>::T *__restrict__ psi,
                                                  TileArgs ta, const RegOp *__restrict__ ops,
                                                  const typename VT<R>::T *__restrict__ pool,
                                                  unsigned int *__restrict__ counter) {
    using T = typename VT<R>::T;
    constexpr int NR = 1 << RB;
    constexpr int m = RB + TB;
    constexpr uint32_t kHalf = (uint32_t)sizeof(T) << (m - 1);
    extern __shared__ __align__(16) unsigned char smem_reg[];
    unsigned char *limg = smem_reg + kHalf;
    // LDS addresses of the remap buffer and the image (the launch checks
    // that the dynamic block starts at 0, so both are multiples of kHalf)
    const uint32_t lds_a = lds_addr(smem_reg);
    const uint32_t limg_a = lds_a + kHalf;
    const uint32_t tid = threadIdx.x;
    const uint32_t lane = tid & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    Warm warm;
    warm.ask<1 << TB>(ops, (uint32_t)ta.n_ops * (uint32_t)sizeof(RegOp), tid);
    {
        const uint4 *src = reinterpret_cast<const uint4 *>(
            reinterpret_cast<const unsigned char *>(pool) + ta.img_off);
        uint4 *dst = reinterpret_cast<uint4 *>(limg);
        for (uint32_t e = tid; e < (ta.img_bytes >> 4); e += (1u << TB)) dst[e] = src[e];
    }
    // this thread's part of the global index in the load and the store layout
    uint64_t gl = 0, gs = 0;
#pragma unroll
    for (int t = 0; t < TB; ++t) {
        const uint64_t on = 0ull - (uint64_t)((tid >> t) & 1u);
        gl |= on & ta.g_thr[t];
        gs |= on & ta.g_thr_f[t];
    }
    const uint32_t n_tiles = (uint32_t)ta.n_tiles;

    // Tiles are claimed one at a time from the pass's counter: a compute unit or
    // XCD that runs slower takes fewer, and the tiles in flight across the
    // device are consecutive, so the 128-byte runs they share a DRAM page with
    // are fetched close together in time (measured: larger claims lose a few per
    // cent).  The claim of the next tile goes out behind the loads of this one
    // (ahead of them its wave's loads waited for it: 78.1 -> 71.5 us per pass at
    // 20 qubits, a tile or two per workgroup; within 0.5 % at 30 qubits) and is
    // broadcast through two alternating LDS slots, so one workgroup barrier per
    // tile suffices (the slot that a claim overwrites was read before the barrier
    // of the tile in between).  Otherwise the waves of a workgroup meet only at
    // its workgroup remaps.
    // The words follow the image in dynamic LDS (a static __shared__
    // variable would move the dynamic block off address 0, and every LDS address
    // would then take an extra add).
    TileWords &words = *reinterpret_cast<TileWords *>(limg + ta.img_bytes);
    auto claim = [&](uint32_t to) {
        words.live[to] = 0;
        words.zero[to] = 0;
        words.claim[to] = atomicAdd(counter, 1u);
    };
    if (tid == 0) claim(0);
    warm.settle();
    uint32_t slot = 0;
    for (;;) {
        __syncthreads();   // the claim (and, the first time, the image) is in LDS
        uint32_t tile = __builtin_amdgcn_readfirstlane(words.claim[slot]);
        if (tile >= n_tiles) break;
        if (ta.some) tile = live_tile(tile, ta.live);
        slot ^= 1u;
        T amp[NR];
        load_tile<T, RB, m>(amp, psi, gl, tile, ta);
        if (tid == 0) claim(slot);
        const uint64_t base = tile_base<m>(tile, ta);
        // back to normal priority for the arithmetic (raised before the
        // stores below: a wave that stores one tile and issues the next
        // tile's loads goes ahead of the other waves' FMAs, so the memory
        // requests of the compute units go out sooner)
        __builtin_amdgcn_s_setprio(0);
        if (ta.zero_stays) {
            uint32_t *live = &words.live[slot ^ 1u], *zero = &words.zero[slot ^ 1u];
            auto look = [](uint32_t *p) {
                return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            };
            if (wave_live<T, NR>(amp)) {
                __hip_atomic_store(live, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            } else {
                if (lane == 0)
                    __hip_atomic_fetch_add(zero, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                // ends: every wave of the workgroup comes here and does one or
                // the other, without waiting for another wave first
                bool on = false;
                for (;;) {
                    on = __builtin_amdgcn_readfirstlane(look(live)) != 0;
                    if (on || __builtin_amdgcn_readfirstlane(look(zero)) == (1u << TB) / 64) break;
                    __builtin_amdgcn_s_sleep(1);
                }
                if (!on) continue;
            }
        }
        // Two ops per iteration (the host pads the program to an even
        // length): the amplitudes then alternate between two register sets
        // without copies at the loop back edge.  Op fields are read through
        // references into the uniform op array so they stay scalar.
        for (int oi = 0; oi < ta.n_ops; oi += 2) {
            reg_op<T, R, NR, RB, DG>(amp, ops[oi], lds_a, limg_a, base, lane, wave);
            reg_op<T, R, NR, RB, DG>(amp, ops[oi + 1], lds_a, limg_a, base, lane, wave);
        }
        // a pass that moves its qubits stores where other threads loaded:
        // every load of the tile completes before the first store
        if (ta.store_sync) __syncthreads();
        __builtin_amdgcn_s_setprio(2);
        T *sp = psi + gs;
        asm volatile("" : "+v"(sp));
        sp += base;
        uint64_t gr[RB];
#pragma unroll
        for (int j = 0; j < RB; ++j) {
            gr[j] = ta.g_reg_f[j];
            asm volatile("" : "+s"(gr[j]));
        }
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            uint64_t g = 0;
#pragma unroll
            for (int j = 0; j < RB; ++j)
                if ((i >> j) & 1) g |= gr[j];
            gstore(sp + g, amp[i]);
        }
    }
}

// Batched form: one pass index of many states (segments of tiles, each
// segment one state's pass with its own program and image).  Workgroup w
// takes the contiguous items [w c, (w + 1) c), c = ceil(items / grid), so it
// mostly stays within one segment; it finds its first segment by binary
// search, steps to the next one when its items cross a segment's end, and
// reloads the image and its thread parts of the layouts at each change.
template <typename R, int RB, int TB, int DG>
__global__ __launch_bounds__(1 << TB, 3) void k_tile_reg_batch(typename VT<R>::T *__restrict__ states,
                                                        const RegSeg *__restrict__ segs, int nseg,
                                                        uint64_t items,
                                                        const TileArgs *__restrict__ tas,
                                                        const RegOp *__restrict__ ops,
                                                        const unsigned char *__restrict__ pool) {
    using T = typename VT<R>::T;
    constexpr int NR = 1 << RB;
    constexpr int m = RB + TB;
    constexpr uint32_t kHalf = (uint32_t)sizeof(T) << (m - 1);
    extern __shared__ __align__(16) unsigned char smem_reg[];
    unsigned char *limg = smem_reg + kHalf;
    const uint32_t lds_a = lds_addr(smem_reg);
    const uint32_t limg_a = lds_a + kHalf;
    const uint32_t tid = threadIdx.x;
    const uint32_t lane = tid & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint64_t per = (items + gridDim.x - 1) / gridDim.x;
    const uint64_t it0 = (uint64_t)blockIdx.x * per;
    const uint64_t it1 = it0 + per < items ? it0 + per : items;
    int lo = 0;
    if (it0 < it1) {
        int hi = nseg - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (segs[mid].first <= it0) lo = mid;
            else hi = mid - 1;
        }
    }
    int cur = -1;
    uint64_t gl = 0, gs = 0;
    for (uint64_t it = it0; it < it1; ++it) {
        while (lo + 1 < nseg && segs[lo + 1].first <= it) ++lo;
        const RegSeg sg = segs[lo];
        const TileArgs &ta = tas[sg.ta];
        if (lo != cur) {
            // every wave is past the previous tile (its remaps and table
            // reads) before the image is overwritten
            __syncthreads();
            Warm warm;
            warm.ask<1 << TB>(ops + sg.op_begin, (uint32_t)ta.n_ops * (uint32_t)sizeof(RegOp), tid);
            const uint4 *src = reinterpret_cast<const uint4 *>(pool + ta.img_off);
            uint4 *dst = reinterpret_cast<uint4 *>(limg);
            for (uint32_t e = tid; e < (ta.img_bytes >> 4); e += (1u << TB)) dst[e] = src[e];
            gl = 0;
            gs = 0;
#pragma unroll
            for (int t = 0; t < TB; ++t) {
                const uint64_t on = 0ull - (uint64_t)((tid >> t) & 1u);
                gl |= on & ta.g_thr[t];
                gs |= on & ta.g_thr_f[t];
            }
            warm.settle();
            __syncthreads();
            cur = lo;
        }
        T *psi = states + sg.state_off;
        const uint32_t tile = (uint32_t)(it - sg.first);
        const RegOp *prog = ops + sg.op_begin;
        T amp[NR];
        if (sg.init) {
            // |0...0>: not read, and never written before
#pragma unroll
            for (int i = 0; i < NR; ++i) amp[i].x = amp[i].y = R(0);
            if (tile == 0 && tid == 0) amp[0].x = R(1);
        } else {
            load_tile<T, RB, m>(amp, psi, gl, tile, ta);
        }
        const uint64_t base = tile_base<m>(tile, ta);
        const int n_ops = sg.init && tile != 0 && ta.zero_stays ? 0 : ta.n_ops;
        for (int oi = 0; oi < n_ops; oi += 2) {
            reg_op<T, R, NR, RB, DG>(amp, prog[oi], lds_a, limg_a, base, lane, wave);
            reg_op<T, R, NR, RB, DG>(amp, prog[oi + 1], lds_a, limg_a, base, lane, wave);
        }
        // stores go where other threads loaded (relabeling passes), and the
        // next tile's first workgroup remap may follow wave-local ones
        __syncthreads();
        T *sp = psi + gs;
        asm volatile("" : "+v"(sp));
        sp += base;
        uint64_t gr[RB];
#pragma unroll
        for (int j = 0; j < RB; ++j) {
            gr[j] = ta.g_reg_f[j];
            asm volatile("" : "+s"(gr[j]));
        }
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            uint64_t g = 0;
#pragma unroll
            for (int j = 0; j < RB; ++j)
                if ((i >> j) & 1) g |= gr[j];
            gstore(sp + g, amp[i]);
        }
    }
}

template <typename R, int DG>
static hipError_t launch_reg_batch_t(void *states, const RegSeg *segs, int nseg, uint64_t items,
                                     const TileArgs *tas, const RegOp *rops, const void *pool,
                                     uint32_t img_max, hipStream_t s) {
    using T = typename VT<R>::T;
    constexpr int RB = 4, TB = 8;
    if (items == 0 || nseg <= 0) return hipSuccess;
    if (img_max > kRegImageMax || (img_max & 15u)) return hipErrorInvalidValue;
    constexpr size_t half = sizeof(T) << (RB + TB - 1);
    const size_t lds = half + img_max;
    static bool attr = false;
    static int cus = 0;
    if (!attr) {
        hipFuncAttributes fa;
        hipError_t e = hipFuncGetAttributes(&fa, reinterpret_cast<const void *>(k_tile_reg_batch<R, RB, TB, DG>));
        if (e != hipSuccess) return e;
        if (fa.sharedSizeBytes != 0) return hipErrorInvalidDeviceFunction;
        e = set_lds_attr(k_tile_reg_batch<R, RB, TB, DG>, half + kRegImageMax);
        if (e != hipSuccess) return e;
        int dev = 0;
        e = hipGetDevice(&dev);
        if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
        if (e != hipSuccess) return e;
        attr = true;
    }
    int occ = 0;
    hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
        &occ, reinterpret_cast<const void *>(k_tile_reg_batch<R, RB, TB, DG>), 1 << TB, lds);
    if (e != hipSuccess) return e;
    const uint64_t resident = (uint64_t)std::max(1, cus) * (uint64_t)std::max(1, occ);
    const unsigned grid = (unsigned)std::min<uint64_t>(items, resident);
    hipLaunchKernelGGL((k_tile_reg_batch<R, RB, TB, DG>), dim3(grid), dim3(1 << TB), lds, s,
                       (T *)states, segs, nseg, items, tas, rops, (const unsigned char *)pool);
    return hipGetLastError();
}

template <typename R, int RB, int TB, int DG>
static hipError_t launch_reg_t(void *psi, const TileArgs &ta, const RegOp *rops,
                               const void *pool, unsigned int *counter, hipStream_t s) {
    using T = typename VT<R>::T;
    if (ta.n_tiles == 0) return hipSuccess;
    if (ta.n_ops & 1) return hipErrorInvalidValue;   // programs are padded to even length
    if (ta.n_tiles > 0xffffffffull - 65536) return hipErrorInvalidValue;
    if (ta.img_bytes > kRegImageMax || (ta.img_bytes & 15u) || (ta.img_off & 15)) return hipErrorInvalidValue;
    constexpr size_t half = sizeof(T) << (RB + TB - 1);
    const size_t lds = half + ta.img_bytes + sizeof(TileWords);
    static int cus = 0;
    static bool attr = false;
    if (!attr) {
        // the kernel forms LDS addresses by XOR on top of the dynamic block's
        // base, which is then 0 only without static LDS
        hipFuncAttributes fa;
        hipError_t e = hipFuncGetAttributes(&fa, reinterpret_cast<const void *>(k_tile_reg<R, RB, TB, DG>));
        if (e != hipSuccess) return e;
        if (fa.sharedSizeBytes != 0) return hipErrorInvalidDeviceFunction;
        e = set_lds_attr(k_tile_reg<R, RB, TB, DG>, half + kRegImageMax + sizeof(TileWords));
        if (e != hipSuccess) return e;
        int dev = 0;
        e = hipGetDevice(&dev);
        if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
        if (e != hipSuccess) return e;
        attr = true;
    }
    // resident workgroups per compute unit for this image size (in 1 KiB steps)
    static int per_cu[kRegImageMax / 1024 + 2] = {0};
    const size_t slot = (ta.img_bytes + 1023) / 1024;
    if (per_cu[slot] == 0) {
        int occ = 0;
        hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &occ, reinterpret_cast<const void *>(k_tile_reg<R, RB, TB, DG>), 1 << TB,
            half + slot * 1024 + sizeof(TileWords));
        if (e != hipSuccess) return e;
        per_cu[slot] = std::max(1, occ);
    }
    const uint64_t resident = (uint64_t)std::max(1, cus) * (uint64_t)per_cu[slot];
    const unsigned grid = (unsigned)std::min<uint64_t>(ta.n_tiles, resident);
    hipLaunchKernelGGL((k_tile_reg<R, RB, TB, DG>), dim3(grid), dim3(1 << TB), lds, s, (T *)psi, ta,
                       rops, (const T *)pool, counter);
    return hipGetLastError();
}

// Instances: 12-bit tiles of 16 amplitudes per thread (the default shape), and
// the other shapes; hipErrorInvalidValue for a shape that the unit lacks.
#define QSV_TILE_REG(R, RB, TB)                                                          \
    return ta.tables == 0   ? launch_reg_t<R, RB, TB, 0>(psi, ta, rops, pool, counter, s) \
           : ta.tables == 1 ? launch_reg_t<R, RB, TB, 1>(psi, ta, rops, pool, counter, s) \
                            : launch_reg_t<R, RB, TB, 2>(psi, ta, rops, pool, counter, s);
hipError_t tile_reg_f64(void *psi, const TileArgs &ta, const RegOp *rops, const void *pool,
                        unsigned int *counter, hipStream_t s);
hipError_t tile_reg_f32(void *psi, const TileArgs &ta, const RegOp *rops, const void *pool,
                        unsigned int *counter, hipStream_t s);
hipError_t tile_reg_shapes_f64(void *psi, const TileArgs &ta, const RegOp *rops, const void *pool,
                               unsigned int *counter, hipStream_t s);
hipError_t tile_reg_shapes_f32(void *psi, const TileArgs &ta, const RegOp *rops, const void *pool,
                               unsigned int *counter, hipStream_t s);
hipError_t tile_reg_batch_f64(int dg, void *states, const RegSeg *segs, int nseg, uint64_t items,
                              const TileArgs *tas, const RegOp *rops, const void *pool,
                              uint32_t img_max, hipStream_t s);
hipError_t tile_reg_batch_f32(int dg, void *states, const RegSeg *segs, int nseg, uint64_t items,
                              const TileArgs *tas, const RegOp *rops, const void *pool,
                              uint32_t img_max, hipStream_t s);

}  // namespace dev
}  // namespace qsv
