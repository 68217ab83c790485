// Per-node arithmetic of the enthalpy-based MRT lattice Boltzmann method for
// solid-liquid phase change in metal foams under local thermal
// non-equilibrium (Liu, He & Li, arXiv:1701.00702): macroscopic values,
// the three moment-space collisions, wall reconstruction, and the storage
// layouts of the populations.  Everything here is __host__ __device__ so the
// kernels in lbm_kernels.hip and a host build of the same arithmetic share it.
//
// Populations are handled as offsets q_i = X_i - X_ref,i from a fixed
// reference equilibrium at rest (flow: w_i rho_0; enthalpy/metal: the
// equilibria at the middle of the mushy band on D2Q9, at the initial
// temperature on D2Q5, where a node the heat has not reached yet then holds
// exact zeros).  The moment algebra is affine, so the update runs on the
// offsets; in FP32 this keeps the small momentum of the Darcy-scale flow
// out of the rounding of O(1) populations.
//
// The thermal fields run on D2Q9 (Sec. III B/C) or on the D2Q5 lattice of
// Appendix B (its five velocities are the first five of Eq. 11); a layout
// carries the number QT of thermal velocities.  Population arrays are sized
// nine throughout; D2Q5 leaves entries 5..8 of g and h unused.
//
// Two arithmetic types: R for the flow and metal fields, RH for the PCM
// enthalpy field (H, T_f, f_l and the g collision).  The rest enthalpy
// population carries H itself, O(1), so its rounding is what limits FP32;
// the mixed form keeps that one population and the enthalpy arithmetic in
// FP64 and everything else in FP32.
#pragma once

#include <math.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>

#include <type_traits>

#include "lbm_internal.h"

#define LBM_HD __host__ __device__ __forceinline__

// A bounds check that host builds make and the kernels leave out.
#if defined(__HIP_DEVICE_COMPILE__)
#define LBM_HOST_CHECK(cond) ((void)0)
#else
#define LBM_HOST_CHECK(cond)                                                              \
    do {                                                                                  \
        if (!(cond)) {                                                                    \
            fprintf(stderr, "lbm: check failed: %s (%s:%d)\n", #cond, __FILE__, __LINE__); \
            abort();                                                                      \
        }                                                                                 \
    } while (0)
#endif

namespace lbm {

// ---------------------------------------------------------------------------
// Lattice (Eq. 11) and weights.
// ---------------------------------------------------------------------------
__host__ __device__ constexpr int ex_of(int i) {
    return (i == 1 || i == 5 || i == 8) ? 1 : ((i == 3 || i == 6 || i == 7) ? -1 : 0);
}
__host__ __device__ constexpr int ey_of(int i) {
    return (i == 2 || i == 5 || i == 6) ? 1 : ((i == 4 || i == 7 || i == 8) ? -1 : 0);
}
template <typename R>
__host__ __device__ constexpr R w_of(int i) {
    return i == 0 ? R(4) / R(9) : (i <= 4 ? R(1) / R(9) : R(1) / R(36));
}

// Reciprocal and square root of the velocity solve and the force: correctly
// rounded in FP64; in FP32 the hardware instructions (about 1 ulp), a tenth
// of the instructions of the correctly rounded sequences.  The FP32 forms
// are held to 1e-4 of the FP64 oracle, far above that rounding.
template <typename R>
LBM_HD R rcp_of(R x) {
    return R(1) / x;
}
template <typename R>
LBM_HD R sqrt_of(R x) {
    return sqrt(x);
}
#if defined(__HIP_DEVICE_COMPILE__)
template <>
LBM_HD float rcp_of<float>(float x) {
    return __builtin_amdgcn_rcpf(x);
}
template <>
LBM_HD float sqrt_of<float>(float x) {
    return __builtin_amdgcn_sqrtf(x);
}
#endif

// Fused multiply-add, rounded once.  The library is built without automatic
// contraction, so each fusion is written out here and every instantiation
// of the update rounds the same way.  With a power-of-two factor the fused
// form gives the same bits as the separate product and sum.
template <typename R>
LBM_HD R fma_of(R a, R b, R c) {
    return fma(a, b, c);
}
template <>
LBM_HD float fma_of<float>(float a, float b, float c) {
    return fmaf(a, b, c);
}

// Enthalpy-field constants in the enthalpy arithmetic type.
template <typename RH>
struct ThermalPick;
template <>
struct ThermalPick<float> {
    template <typename R>
    LBM_HD static const ThermalConst<float> &get(const CavityConst<R> &c) { return c.tf; }
};
template <>
struct ThermalPick<double> {
    template <typename R>
    LBM_HD static const ThermalConst<double> &get(const CavityConst<R> &c) { return c.td; }
};
template <typename RH, typename R>
LBM_HD const ThermalConst<RH> &thermal(const CavityConst<R> &c) {
    return ThermalPick<RH>::get(c);
}

// The constants of the node update with the enthalpy field in RH.
template <typename RH, typename R>
LBM_HD const NodeConst<R, RH> &node_const_of(const CavityConst<R> &c) {
    if constexpr (std::is_same<R, RH>::value) return c.nr;
    else return c.nd;
}

// A value kept in a register from here on: the empty asm keeps the compiler
// from loading it again at each use.  Scalar registers (workgroup-uniform
// values only), or vector ones.
template <bool VECTOR = false, typename T>
LBM_HD void resident(T &v) {
#if defined(__HIP_DEVICE_COMPILE__)
    if constexpr (VECTOR) asm volatile("" : "+v"(v));
    else asm volatile("" : "+s"(v));
#else
    (void)v;
#endif
}
// The same for a condition held as an integer, so that testing it is a scalar
// compare and not a lane mask.
LBM_HD void resident_flag(int &v) {
#if defined(__HIP_DEVICE_COMPILE__)
    v = __builtin_amdgcn_readfirstlane(v);
#endif
    resident(v);
}
template <class Lay, bool VECTOR, class N>
LBM_HD void reside(N &n) {
    constexpr bool V = VECTOR;
    resident<V>(n.H_ref), resident<V>(n.H_fs), resident<V>(n.H_fl), resident<V>(n.T_fs), resident<V>(n.T_fl);
    resident<V>(n.inv_dH), resident<V>(n.dT_band), resident<V>(n.Tf_ref), resident<V>(n.hv_f);
    resident<V>(n.gbeta), resident<V>(n.T0), resident<V>(n.px), resident<V>(n.py);
    resident<V>(n.inv_phi), resident<V>(n.drag_lin), resident<V>(n.drag_quad), resident<V>(n.l0), resident<V>(n.l0sq);
    resident<V>(n.l1), resident<V>(n.fA7), resident<V>(n.fB7), resident<V>(n.fC7);
    resident<V>(n.hv_m), resident<V>(n.sr_ratio);
    if constexpr (sizeof(n.T_ref) != sizeof(n.Tf_ref)) resident<V>(n.T_ref);
    resident<V>(n.mA0), resident<V>(n.mB0), resident<V>(n.mA1), resident<V>(n.mA3);
    resident<V>(n.me1), resident<V>(n.zA1), resident<V>(n.zB1), resident<V>(n.zA3), resident<V>(n.zB3);
    resident<V>(n.ge1);
    resident(n.bounce_back);
    if constexpr (Lay::QT == 9) {
        resident<V>(n.mB1), resident<V>(n.mA4), resident<V>(n.mA7), resident<V>(n.me2);
        resident<V>(n.zA4), resident<V>(n.zB4), resident<V>(n.zA7), resident<V>(n.ge2);
    } else {
        resident<V>(n.mB3), resident<V>(n.w4);
    }
    static_assert(!Lay::SCALED, "the 16-bit forms read theirs from memory");
}

// The constants of the node update for the multi-step kernels.  With FP32
// arithmetic they are loaded once per workgroup and stay in scalar
// registers; loaded at each use, every update waited on chains of scalar
// loads (they return out of order, so each wait is for all of them and for
// the LDS reads too).  Together with one vector offset for all pulls and the
// scalar branch past the wall code this took the three-step FP32_H64 kernel
// (8192^2) from 1125 VALU, 558 scalar and 98 scalar-load instructions per
// wave to 961, 302 and 24.  FP64 constants would take twice the registers
// there are (700 spills to vector lanes, 13% slower) and stay in memory.  So do
// those of the 16-bit forms, whose scales and codecs fill what is left (27 to
// 42 spills; GLUPS at 4096^2 with them in registers and in memory: F16 57.9 and
// 64.3, BF16_SPLIT 50.7 and 54.7, F16_SPLIT 49.4 and 53.8, the latter two in the
// vector registers of three workgroups per CU).
template <class Lay, typename RH>
LBM_HD const NodeConst<double, RH> &node_const(const CavityConst<double> &c) {
    return node_const_of<RH>(c);
}
template <class Lay, typename RH>
LBM_HD typename std::conditional<Lay::SCALED, const NodeConst<float, RH> &, NodeConst<float, RH>>::type node_const(
    const CavityConst<float> &c) {
    if constexpr (Lay::SCALED) {
        return node_const_of<RH>(c);
    } else {
        NodeConst<float, RH> n = node_const_of<RH>(c);
        reside<Lay, false>(n);
        return n;
    }
}

// ---------------------------------------------------------------------------
// Streaming loads/stores and element codecs.  Every population is read and
// written once per step; whether the GPU accesses carry the non-temporal
// hint is a build option (LBM_NT_LOADS, LBM_NT_STORES).
// ---------------------------------------------------------------------------
#ifndef LBM_NT_LOADS
#define LBM_NT_LOADS 0
#endif
#ifndef LBM_NT_STORES
#define LBM_NT_STORES 1
#endif
template <typename T>
LBM_HD T ld_stream(const T *p) {
#if defined(__HIP_DEVICE_COMPILE__) && LBM_NT_LOADS
    return __builtin_nontemporal_load(p);
#else
    return *p;
#endif
}
template <typename T>
LBM_HD void st_stream(T *p, T v) {
#if defined(__HIP_DEVICE_COMPILE__) && LBM_NT_STORES
    __builtin_nontemporal_store(v, p);
#else
    *p = v;
#endif
}

// A node's place in a population plane of a band block (the banded layout
// of the state buffers is described with CavityConst).  NodeRef: the node's
// offset rel within its band's plane plus the byte distance jump of its
// band's block from the block of the workgroup's first band, both 32-bit.
// FarRef: the same in 64 bits, for an access anywhere in a cavity from its
// first band's block.
struct NodeRef {
    uint32_t rel, jump;
};
struct FarRef {
    int64_t rel, jump;
};
template <typename T>
using ByteOf = typename std::conditional<std::is_const<T>::value, const char, char>::type;
template <typename T>
LBM_HD T *at(T *plane, FarRef r) {
    return (T *)((ByteOf<T> *)(plane + r.rel) + r.jump);
}

// The blocks a workgroup reads or writes, from the block of its first band
// on.  An access is at uniform + lane + imm bytes from there: on the GPU a
// buffer access, which takes the three as a scalar register, a vector
// register and a constant, so that the planes of a node differ in the scalar
// alone and one vector offset serves them all.  A workgroup's rows lie in two
// consecutive bands of less than 2^31 bytes each (the plan refuses longer
// rows), so every sum stays below 2^32, which is what a buffer access can
// reach: its three parts are unsigned, and the resource spans kBlocksBytes.
// Beyond the resource loads give 0 and stores are dropped without an error.
constexpr uint32_t kBlocksBytes = 0xffffffffu;
#if defined(__HIP_DEVICE_COMPILE__)
using Blocks = __amdgpu_buffer_rsrc_t;
LBM_HD Blocks blocks_of(const void *first) {
    return __builtin_amdgcn_make_buffer_rsrc((void *)first, 0, kBlocksBytes, 0x00020000);
}
#else
using Blocks = char *;
LBM_HD Blocks blocks_of(const void *first) { return (char *)first; }
#endif
template <typename T>
LBM_HD T ld_block(Blocks b, uint32_t uniform, uint32_t lane, uint32_t imm) {
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int aux = LBM_NT_LOADS ? 2 : 0;
    if constexpr (sizeof(T) == 8)
        return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(b, lane + imm, uniform, aux));
    else if constexpr (sizeof(T) == 4)
        return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(b, lane + imm, uniform, aux));
    else
        return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b16(b, lane + imm, uniform, aux));
#else
    LBM_HOST_CHECK((uint64_t)uniform + lane + imm + sizeof(T) <= kBlocksBytes);
    return *(const T *)(b + ((uint64_t)uniform + lane + imm));
#endif
}
template <typename T>
LBM_HD void st_block(Blocks b, uint32_t uniform, uint32_t lane, T v) {
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int aux = LBM_NT_STORES ? 2 : 0;
    if constexpr (sizeof(T) == 8) {
        using V2 = unsigned int __attribute__((ext_vector_type(2)));
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(V2, v), b, lane, uniform, aux);
    } else if constexpr (sizeof(T) == 4) {
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned int, v), b, lane, uniform, aux);
    } else {
        __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(unsigned short, v), b, lane, uniform, aux);
    }
#else
    LBM_HOST_CHECK((uint64_t)uniform + lane + sizeof(T) <= kBlocksBytes);
    *(T *)(b + ((uint64_t)uniform + lane)) = v;
#endif
}

// One pull of a node: the element at node offset rel + dx of a plane, shift
// nodes (uniform) from it, in the block jump bytes on.
struct Pull {
    int32_t shift;
    uint32_t rel, dx, jump;
};

struct E64 {
    using T = double;
    LBM_HD static double dec(double v) { return v; }
    LBM_HD static double enc(double v) { return v; }
};
struct E32 {
    using T = float;
    LBM_HD static float dec(float v) { return v; }
    LBM_HD static float enc(float v) { return v; }
};
struct E16 {  // IEEE binary16, round to nearest even
    using T = uint16_t;
    LBM_HD static float dec(uint16_t v) { return (float)__builtin_bit_cast(_Float16, v); }
    LBM_HD static uint16_t enc(float v) { return __builtin_bit_cast(uint16_t, (_Float16)v); }
};
struct EB16 {  // bfloat16, round to nearest even (finite values)
    using T = uint16_t;
    LBM_HD static float dec(uint16_t v) { return __builtin_bit_cast(float, ((uint32_t)v) << 16); }
    LBM_HD static uint16_t enc(float v) {
        uint32_t u = __builtin_bit_cast(uint32_t, v);
        u += 0x7fffu + ((u >> 16) & 1u);
        return (uint16_t)(u >> 16);
    }
};

// ---------------------------------------------------------------------------
// Storage layouts.  load<V>() returns the offset q_i of field f (0 flow,
// 1 enthalpy, 2 metal), direction i, at packed node k, in type V; store()
// writes the offsets of one field at node k (nine for the flow, QT for the
// thermal fields); pull() and put() are the same within a workgroup's
// blocks.  beta is the per-node base value the split layout stores (unused
// elsewhere).  c holds the scales of the 16-bit forms.
// ---------------------------------------------------------------------------

// 9 + 2 QT planes of one element type, [f0..f8, g0..g(QT-1), h0..h(QT-1)];
// 16-bit forms carry a power-of-two scale.
template <class E, bool SCALED_, int QT_ = 9>
struct Plain {
    using T = typename E::T;
    using C = decltype(E::dec(T()));  // element arithmetic type of the codec
    static constexpr int QT = QT_;
    static constexpr bool SCALED = SCALED_;
    static constexpr int bytes_per_node = (9 + 2 * QT) * (int)sizeof(T);
    LBM_HD static constexpr int plane(int f, int i) { return f == 0 ? i : 9 + (f - 1) * QT + i; }
    template <typename V, class S>
    LBM_HD static V dec(T e, int f, const S &c) {
        const V v = (V)E::dec(e);
        return SCALED ? v * (V)c.inv_scale[f] : v;
    }
    template <typename V, class S>
    LBM_HD static T enc(V q, int f, const S &c) {
        return E::enc((C)(SCALED ? q * (V)c.scale[f] : q));
    }
    template <typename V, class S, typename K>
    LBM_HD static V load(const void *base, int64_t stride, int f, int i, K k, const S &c) {
        return dec<V>(ld_stream(at((const T *)base + (int64_t)plane(f, i) * stride, k)), f, c);
    }
    template <typename V, class S, typename K>
    LBM_HD static void store(void *base, int64_t stride, int f, const V q[9], V beta, K k, const S &c) {
        (void)beta;
        const int n = f == 0 ? 9 : QT;
#pragma unroll
        for (int i = 0; i < 9; ++i)
            if (i < n) st_stream(at((T *)base + (int64_t)plane(f, i) * stride, k), enc(q[i], f, c));
    }
    template <typename V, class S>
    LBM_HD static V pull(Blocks b, uint32_t stride, int f, int i, Pull p, const S &c) {
        return dec<V>(ld_block<T>(b, (plane(f, i) * stride + p.shift) * sizeof(T), p.rel * sizeof(T) + p.jump,
                                  p.dx * sizeof(T)),
                      f, c);
    }
    template <typename V, class S>
    LBM_HD static void put(Blocks b, uint32_t stride, int f, const V q[9], V beta, NodeRef k, const S &c) {
        (void)beta;
        const int n = f == 0 ? 9 : QT;
#pragma unroll
        for (int i = 0; i < 9; ++i)
            if (i < n) st_block<T>(b, plane(f, i) * stride * sizeof(T), k.rel * sizeof(T) + k.jump, enc(q[i], f, c));
    }
};

// FP32 planes for all populations but the rest enthalpy one, which gets an
// FP64 plane: [f0..f8, g1..g(QT-1), h0..h(QT-1)] in FP32 (8 + 2 QT planes),
// then g0 in FP64; 112 bytes per node on D2Q9, 80 on D2Q5.
template <int QT_ = 9>
struct PlainH64 {
    static constexpr int QT = QT_;
    static constexpr bool SCALED = false;
    static constexpr int NF32 = 8 + 2 * QT;
    static constexpr int bytes_per_node = NF32 * 4 + 8;
    LBM_HD static constexpr int plane(int f, int i) { return f == 0 ? i : (f == 1 ? 8 + i : 8 + QT + i); }
    template <typename V, class S, typename K>
    LBM_HD static V load(const void *base, int64_t stride, int f, int i, K k, const S &c) {
        (void)c;
        if (f == 1 && i == 0) return (V)ld_stream(at((const double *)((const float *)base + NF32 * stride), k));
        return (V)ld_stream(at((const float *)base + (int64_t)plane(f, i) * stride, k));
    }
    template <typename V, class S, typename K>
    LBM_HD static void store(void *base, int64_t stride, int f, const V q[9], V beta, K k, const S &c) {
        (void)beta;
        (void)c;
        const int n = f == 0 ? 9 : QT;
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            if (i >= n) continue;
            if (f == 1 && i == 0) st_stream(at((double *)((float *)base + NF32 * stride), k), (double)q[0]);
            else st_stream(at((float *)base + (int64_t)plane(f, i) * stride, k), (float)q[i]);
        }
    }
    template <typename V, class S>
    LBM_HD static V pull(Blocks b, uint32_t stride, int f, int i, Pull p, const S &c) {
        (void)c;
        if (f == 1 && i == 0)
            return (V)ld_block<double>(b, NF32 * stride * 4 + p.shift * 8, p.rel * 8 + p.jump, p.dx * 8);
        return (V)ld_block<float>(b, (plane(f, i) * stride + p.shift) * 4, p.rel * 4 + p.jump, p.dx * 4);
    }
    template <typename V, class S>
    LBM_HD static void put(Blocks b, uint32_t stride, int f, const V q[9], V beta, NodeRef k, const S &c) {
        (void)beta;
        (void)c;
        const int n = f == 0 ? 9 : QT;
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            if (i >= n) continue;
            if (f == 1 && i == 0) st_block<double>(b, NF32 * stride * 4, k.rel * 8 + k.jump, (double)q[0]);
            else st_block<float>(b, plane(f, i) * stride * 4, k.rel * 4 + k.jump, (float)q[i]);
        }
    }
};

// Split 16-bit layout: per field, the rest population and a base value beta
// in FP32, and the eight moving populations as 16-bit remainders (binary16,
// ER = E16, or bfloat16, ER = EB16) from the rest equilibrium of the base,
// r_i = q_i - w_i beta (scaled).  Bases: flow delta rho, enthalpy
// c_f,ref (T_f - T_ref), metal c_m,ref (T_m - T_ref); the moving populations
// stay close to w_i beta, so their remainders are small and 16 bits keep
// them to ~1e-3 (binary16) or ~8e-3 (bfloat16) relative, while the
// conserved content (rest population, base) keeps FP32 precision.
// Planes: 6 FP32 planes [q_f0, b_f, q_g0, b_g, q_h0, b_h] with b = w_1 beta
// (the axis weight 1/9 times the base), then 24 16-bit planes
// [field][direction 1..8]; 72 bytes per node.
// The split codec's arithmetic, shared by the global layout and its LDS
// copy: a population is w_i beta + r / s (r the 16-bit remainder, s the
// field's power-of-two scale).  With w_i beta = c_i b, c_i = 1 on the axes
// and 1/4 on the diagonals (exact), an axis population decodes with one
// fused multiply-add and a diagonal one with two operations, and a field's
// eight remainders q s - (c_i s) b take one fused multiply-add each after
// two products per field.  Rounding b once and scaling it by powers of two
// gives the same bits as rounding w_i beta per direction.
template <typename V>
__host__ __device__ constexpr V split_c(int i) {
    return i <= 4 ? V(1) : V(0.25);
}
template <typename V>
LBM_HD V split_base(V beta) {
    return w_of<V>(1) * beta;
}
template <typename V>
LBM_HD V split_dec(int i, V b, V r, V inv_scale) {
    return fma_of(r, inv_scale, split_c<V>(i) * b);
}
template <typename V>
LBM_HD float split_rem(int i, V q, V b, V scale) {
    return (float)fma_of(q, scale, -(split_c<V>(i) * scale) * b);
}

template <class ER>
struct SplitT {
    static constexpr int QT = 9;
    static constexpr bool SCALED = true;
    static constexpr int bytes_per_node = 6 * 4 + 24 * 2;
    template <typename V, class S, typename K>
    LBM_HD static V load(const void *base, int64_t stride, int f, int i, K k, const S &c) {
        const float *P = (const float *)base;
        if (i == 0) return (V)ld_stream(at(P + (int64_t)(2 * f) * stride, k));
        const V b = (V)ld_stream(at(P + (int64_t)(2 * f + 1) * stride, k));
        const uint16_t *Qp = (const uint16_t *)(P + 6 * stride);
        const V r = (V)ER::dec(ld_stream(at(Qp + (int64_t)(8 * f + i - 1) * stride, k)));
        return split_dec<V>(i, b, r, (V)c.inv_scale[f]);
    }
    template <typename V, class S, typename K>
    LBM_HD static void store(void *base, int64_t stride, int f, const V q[9], V beta, K k, const S &c) {
        float *P = (float *)base;
        const float eb = (float)split_base<V>(beta);
        st_stream(at(P + (int64_t)(2 * f) * stride, k), (float)q[0]);
        st_stream(at(P + (int64_t)(2 * f + 1) * stride, k), eb);
        uint16_t *Qp = (uint16_t *)(P + 6 * stride);
#pragma unroll
        for (int i = 1; i < 9; ++i)
            st_stream(at(Qp + (int64_t)(8 * f + i - 1) * stride, k),
                      ER::enc(split_rem<V>(i, q[i], (V)eb, (V)c.scale[f])));
    }
    // the stored base of field f of the node pulled from
    LBM_HD static float pull_base(Blocks b, uint32_t stride, int f, Pull p) {
        return ld_block<float>(b, ((2 * f + 1) * stride + p.shift) * 4, p.rel * 4 + p.jump, p.dx * 4);
    }
    // moving population i (>= 1) of field f, given that node's base
    template <typename V, class S>
    LBM_HD static V pull_moving(Blocks b, uint32_t stride, int f, int i, Pull p, V base, const S &c) {
        const V r = (V)ER::dec(ld_block<uint16_t>(b, 24 * stride + ((8 * f + i - 1) * stride + p.shift) * 2,
                                                  p.rel * 2 + p.jump, p.dx * 2));
        return split_dec<V>(i, base, r, (V)c.inv_scale[f]);
    }
    template <typename V, class S>
    LBM_HD static V pull(Blocks b, uint32_t stride, int f, int i, Pull p, const S &c) {
        if (i == 0) return (V)ld_block<float>(b, (2 * f * stride + p.shift) * 4, p.rel * 4 + p.jump, p.dx * 4);
        return pull_moving<V>(b, stride, f, i, p, (V)pull_base(b, stride, f, p), c);
    }
    template <typename V, class S>
    LBM_HD static void put(Blocks b, uint32_t stride, int f, const V q[9], V beta, NodeRef k, const S &c) {
        const float eb = (float)split_base<V>(beta);
        st_block<float>(b, 2 * f * stride * 4, k.rel * 4 + k.jump, (float)q[0]);
        st_block<float>(b, (2 * f + 1) * stride * 4, k.rel * 4 + k.jump, eb);
#pragma unroll
        for (int i = 1; i < 9; ++i)
            st_block<uint16_t>(b, (24 + (8 * f + i - 1) * 2) * stride, k.rel * 2 + k.jump,
                               ER::enc(split_rem<V>(i, q[i], (V)eb, (V)c.scale[f])));
    }
};
using Split16 = SplitT<E16>;
using SplitB16 = SplitT<EB16>;

// Layout and arithmetic types of each storage form.
template <int ST>
struct LayoutOf;
template <>
struct LayoutOf<ST_F64> {
    using L = Plain<E64, false>;
    using R = double;
    using RH = double;
};
template <>
struct LayoutOf<ST_F32> {
    using L = Plain<E32, false>;
    using R = float;
    using RH = float;
};
template <>
struct LayoutOf<ST_F16> {
    using L = Plain<E16, true>;
    using R = float;
    using RH = float;
};
template <>
struct LayoutOf<ST_BF16> {
    using L = Plain<EB16, true>;
    using R = float;
    using RH = float;
};
template <>
struct LayoutOf<ST_F16S> {
    using L = Split16;
    using R = float;
    using RH = float;
};
template <>
struct LayoutOf<ST_BF16S> {
    using L = SplitB16;
    using R = float;
    using RH = float;
};
template <>
struct LayoutOf<ST_F32H> {
    using L = PlainH64<9>;
    using R = float;
    using RH = double;
};
template <>
struct LayoutOf<ST5_F64> {
    using L = Plain<E64, false, 5>;
    using R = double;
    using RH = double;
};
template <>
struct LayoutOf<ST5_F32> {
    using L = Plain<E32, false, 5>;
    using R = float;
    using RH = float;
};
template <>
struct LayoutOf<ST5_F32H> {
    using L = PlainH64<5>;
    using R = float;
    using RH = double;
};

// ---------------------------------------------------------------------------
// Moment transforms of Eq. (13) on offsets.  d = M q, and q = M^-1 d with
// M^-1 = M^T diag(1/9, 1/36, 1/36, 1/6, 1/12, 1/6, 1/12, 1/4, 1/4): the
// inverse takes the scaled moments a_k = d_k / |M_k|^2 (|M_k|^2 the squared
// norm of row k of M), whose factors the collisions fold into their rates.
// ---------------------------------------------------------------------------
template <typename R>
LBM_HD void to_moments(const R q[9], R d[9]) {
    const R p13 = q[1] + q[3], p24 = q[2] + q[4], m13 = q[1] - q[3], m24 = q[2] - q[4];
    const R p56 = q[5] + q[6], p78 = q[7] + q[8], m56 = q[5] - q[6], m78 = q[7] - q[8];
    const R s14 = p13 + p24, s58 = p56 + p78;
    const R dxd = m56 - m78, dyd = p56 - p78;
    d[0] = (q[0] + s14) + s58;
    d[1] = fma_of(R(2), s58, fma_of(R(-4), q[0], -s14));
    d[2] = fma_of(R(4), q[0], fma_of(R(-2), s14, s58));
    d[3] = m13 + dxd;
    d[4] = fma_of(R(-2), m13, dxd);
    d[5] = m24 + dyd;
    d[6] = fma_of(R(-2), m24, dyd);
    d[7] = p13 - p24;
    d[8] = m56 + m78;
}

// 1 / |M_k|^2.
template <typename R>
__host__ __device__ constexpr R moment_norm(int k) {
    return k == 0 ? R(1) / R(9) : (k <= 2 ? R(1) / R(36) : (k == 3 || k == 5 ? R(1) / R(6) : (k <= 6 ? R(1) / R(12) : R(0.25))));
}

template <typename R>
LBM_HD void from_scaled(const R a[9], R q[9]) {
    const R axis = fma_of(R(-2), a[2], a[0] - a[1]);
    const R diag = fma_of(R(2), a[1], a[0]) + a[2];
    const R xa = fma_of(R(-2), a[4], a[3]), ya = fma_of(R(-2), a[6], a[5]);
    const R xd = a[3] + a[4], yd = a[5] + a[6];
    const R ap = axis + a[7], am = axis - a[7];
    const R dp = diag + a[8], dm = diag - a[8];
    const R u = xd + yd, v = xd - yd;
    q[0] = fma_of(R(4), a[2], fma_of(R(-4), a[1], a[0]));
    q[1] = ap + xa;
    q[3] = ap - xa;
    q[2] = am + ya;
    q[4] = am - ya;
    q[5] = dp + u;
    q[7] = dp - u;
    q[6] = dm - v;
    q[8] = dm + v;
}

// D2Q5 transforms of Eq. (B1) on offsets: d = M q, and its inverse
// q0 = d0 - d3, q1,3 = (d3 + d4)/4 +- d1/2, q2,4 = (d3 - d4)/4 +- d2/2,
// taken from e_k = g_k d_k with g = (1, 1/2, 1/2, 1/4, 1/4), whose factors
// the collisions fold into their rates (powers of two: the same bits).
template <typename R>
LBM_HD void to_moments5(const R q[9], R d[5]) {
    const R ax = q[1] + q[3], ay = q[2] + q[4];
    d[0] = ((q[0] + q[1]) + (q[2] + q[3])) + q[4];
    d[1] = q[1] - q[3];
    d[2] = q[2] - q[4];
    d[3] = ax + ay;
    d[4] = ax - ay;
}

template <typename R>
LBM_HD void from_scaled5(const R e[5], R q[9]) {
    const R a = e[3] + e[4], b = e[3] - e[4];
    q[0] = fma_of(R(-4), e[3], e[0]);
    q[1] = a + e[1];
    q[3] = a - e[1];
    q[2] = b + e[2];
    q[4] = b - e[2];
}

// ---------------------------------------------------------------------------
// Macroscopic values of one node from its post-streaming offsets.
// ---------------------------------------------------------------------------
template <typename RH>
struct Thermo {  // PCM enthalpy field, Eqs. (37)-(39)
    RH dH, H, Tf, fl;
};
template <typename R>
struct Macro {  // everything the flow and metal collisions need; G is phi times the buoyancy
    R Tf, fl, dTm, Tm, drho, rho, ux, uy, umag, Gx, Gy;
};

// Eqs. (38)-(39), branches in the order the paper lists them (c_ps = c_pl = 1).
template <typename RH, class N>
LBM_HD void eos(const N &n, RH H, RH &T, RH &fl) {
    if (H <= n.H_fs) {
        T = H;
        fl = RH(0);
    } else if (H >= n.H_fl) {
        T = n.T_fl + (H - n.H_fl);
        fl = RH(1);
    } else {
        fl = (H - n.H_fs) * n.inv_dH;
        T = n.T_fs + fl * n.dT_band;
    }
}

// Moments of the three fields' post-streaming offsets, Eq. (13) (D2Q5
// thermal fields: Eq. B1).  Their zeroth moments are delta rho, delta H
// (Eq. 37) and c_pm delta T_m (Eq. 48).
//
// Split enthalpy arithmetic (RH wider than R, the form with the FP64 rest
// enthalpy population): the rest population q_0 carries H, O(1), while the
// moving ones are small.  The moments g are then taken in R of the moving
// populations alone (q_0 read as zero) and q_0 is kept in RH as `rest`.
// Column 0 of the transform is (1, -4, 4, 0, ..., 0) (D2Q5: (1, 0, ..., 0)),
// and the enthalpy equilibrium moves with H along the same column (Eq. 34:
// n_1^eq = -4 H + ..., n_2^eq = 4 H - ...; Eq. B2: only n_0^eq), so the
// collision of the moving part yields every post-collision population, and
// the rest one is q_0 plus the moving part's rest result: q_0 enters no
// rounding but that of one addition in RH.
template <typename R, typename RH>
struct Moments {
    static constexpr bool SPLIT = !std::is_same<R, RH>::value;
    using RG = typename MomentType<R, RH>::T;
    R f[9], h[9];
    RG g[9];
    RH rest;  // SPLIT: the rest enthalpy population q_0
};
template <int QT, typename R, typename RH>
LBM_HD void field_moments(const R qf[9], const RH qg[9], const R qh[9], Moments<R, RH> &mo) {
    using Mo = Moments<R, RH>;
    using RG = typename Mo::RG;
    to_moments(qf, mo.f);
    RG qs[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) qs[i] = Mo::SPLIT && i == 0 ? RG(0) : (RG)qg[i];
    mo.rest = Mo::SPLIT ? qg[0] : RH(0);
    if (QT == 9) {
        to_moments(qs, mo.g);
        to_moments(qh, mo.h);
    } else {
        to_moments5(qs, mo.g);
        to_moments5(qh, mo.h);
    }
}

// Everything the collisions need, from the moments; blends the flow moments
// in place (Eq. 20: f = f_l f+ + (1 - f_l) w rho, whose moments on offsets
// are f_l d + (1 - f_l) delta rho (1, -2, 1, 0, ..., 0), M w having the
// moments (1, -2, 1, 0, ..., 0)).  The bounce-back alternative of Sec. V B
// keeps f+ unblended.
template <typename R, typename RH>
LBM_HD void macros_of(const NodeConst<R, RH> &n, Moments<R, RH> &mo, Thermo<RH> &th, Macro<R> &m) {
    // Eq. (37), Eqs. (38)-(39)
    th.dH = Moments<R, RH>::SPLIT ? (RH)mo.g[0] + mo.rest : (RH)mo.g[0];
    th.H = n.H_ref + th.dH;
    eos(n, th.H, th.Tf, th.fl);
    m.Tf = (R)th.Tf;
    m.fl = (R)th.fl;
    // Eq. (48), c_pm = 1
    m.dTm = mo.h[0];
    m.Tm = (std::is_same<R, RH>::value ? (R)n.Tf_ref : n.T_ref) + m.dTm;
    // Eq. (21)
    m.drho = mo.f[0];
    m.rho = R(1) + m.drho;
    if (!n.bounce_back) {
        const R sol = (R(1) - m.fl) * m.drho;
        mo.f[0] = m.drho;
        mo.f[1] = fma_of(m.fl, mo.f[1], R(-2) * sol);
        mo.f[2] = fma_of(m.fl, mo.f[2], sol);
#pragma unroll
        for (int k = 3; k < 9; ++k) mo.f[k] = m.fl * mo.f[k];
    }
    // Eq. (7): buoyancy along +axis (gravity along -axis).
    const R G = n.gbeta * (m.Tf - n.T0) * m.fl;
    m.Gx = n.px * G;
    m.Gy = n.py * G;
    // Eq. (24) (j = the blended moments 3 and 5), then the explicit root
    // Eq. (23) with Eq. (25).
    const R jx = mo.f[3], jy = mo.f[5];
    const R inv_rho = rcp_of(m.rho);
    const R vx = fma_of(jx, inv_rho, R(0.5) * m.Gx);
    const R vy = fma_of(jy, inv_rho, R(0.5) * m.Gy);
    const R vmag = sqrt_of(fma_of(vx, vx, vy * vy));
    const R inv_den = rcp_of(n.l0 + sqrt_of(fma_of(n.l1, vmag, n.l0sq)));
    m.ux = vx * inv_den;
    m.uy = vy * inv_den;
    m.umag = vmag * inv_den;  // |u| of Eq. (3)
    // bounce-back: below the interface value f_l = 0.5 a node is solid, at rest
    if (n.bounce_back && m.fl < R(0.5)) {
        m.ux = R(0);
        m.uy = R(0);
        m.umag = R(0);
    }
}

// The same from populations (wall partners, diagnostics).
template <int QT, typename R, typename RH>
LBM_HD void macros(const NodeConst<R, RH> &n, const R qf[9], const RH qg[9], const R qh[9], Thermo<RH> &th,
                   Macro<R> &m) {
    Moments<R, RH> mo;
    field_moments<QT>(qf, qg, qh, mo);
    macros_of(n, mo, th, m);
}

// (1 - s_k) / |M_k|^2, s_k / |M_k|^2 and the forcing factor (1 - s_k / 2) /
// |M_k|^2 of the flow's moments with fixed rates, rounded as a table built
// on the host would be.
template <typename R>
__host__ __device__ constexpr R flow_keep(int k) {
    return (R)((1.0 - kFlowRate[k]) * moment_norm<double>(k));
}
template <typename R>
__host__ __device__ constexpr R flow_relax(int k) {
    return (R)(kFlowRate[k] * moment_norm<double>(k));
}
template <typename R>
__host__ __device__ constexpr R flow_force(int k) {
    return (R)((1.0 - 0.5 * kFlowRate[k]) * moment_norm<double>(k));
}

// Flow collision, Eqs. (14), (16)-(19), from the blended moments d (into q);
// with the bounce-back alternative (Sec. V B) a solid node instead returns
// every population of q along the opposite link (the reference w_i rho_0 is
// symmetric, so the offsets swap the same way).
template <typename R, typename RH>
LBM_HD void collide_flow(const NodeConst<R, RH> &n, const Macro<R> &m, R d[9], R q[9]) {
    if (n.bounce_back && m.fl < R(0.5)) {
        R t;
        t = q[1]; q[1] = q[3]; q[3] = t;
        t = q[2]; q[2] = q[4]; q[4] = t;
        t = q[5]; q[5] = q[7]; q[7] = t;
        t = q[6]; q[6] = q[8]; q[8] = t;
        return;
    }
    const R ux = m.ux, uy = m.uy, rho = m.rho;
    const R uu = fma_of(ux, ux, uy * uy);
    // Eq. (3): F = -(drag_lin + drag_quad |u|) u + phi G
    const R drag = fma_of(n.drag_quad, m.umag, n.drag_lin);
    const R Fx = fma_of(-drag, ux, m.Gx);
    const R Fy = fma_of(-drag, uy, m.Gy);
    const R rip = rho * n.inv_phi;
    R eq[9], S[9];
    const R ru = R(3) * rip * uu;
    eq[1] = fma_of(R(-2), m.drho, ru);
    eq[2] = m.drho - ru;
    eq[3] = rho * ux;
    eq[4] = -eq[3];
    eq[5] = rho * uy;
    eq[6] = -eq[5];
    eq[7] = rip * (ux * ux - uy * uy);
    eq[8] = rip * ux * uy;
    const R uF = ux * Fx + uy * Fy;
    S[1] = R(6) * rip * uF;
    S[2] = -S[1];
    S[3] = rho * Fx;
    S[4] = -S[3];
    S[5] = rho * Fy;
    S[6] = -S[5];
    S[7] = R(2) * rip * (ux * Fx - uy * Fy);
    S[8] = rip * (ux * Fy + uy * Fx);
    // scaled post-collision moments: ((1 - s) d + s eq + (1 - s/2) S) / |M_k|^2
    // (s_3 = s_5 = 1: no part of d stays)
    R a[9];
    a[0] = m.drho * moment_norm<R>(0);
#pragma unroll
    for (int k = 1; k < 7; ++k) {
        const R relaxed = k == 3 || k == 5 ? flow_relax<R>(k) * eq[k]
                                           : fma_of(flow_relax<R>(k), eq[k], flow_keep<R>(k) * d[k]);
        a[k] = fma_of(flow_force<R>(k), S[k], relaxed);
    }
#pragma unroll
    for (int k = 7; k < 9; ++k) a[k] = fma_of(n.fC7, S[k], fma_of(n.fB7, eq[k], n.fA7 * d[k]));
    from_scaled(a, q);
}

// Post-collision enthalpy offsets from the collision's output qs (in the
// moment type RG): the rest population adds q_0 back in the split form.
template <typename RG, typename RH>
LBM_HD void pcm_out(const RG qs[9], RH rest, RH q[9]) {
    constexpr bool SPLIT = !std::is_same<RG, RH>::value;
#pragma unroll
    for (int i = 0; i < 9; ++i) q[i] = SPLIT && i == 0 ? rest + (RH)qs[0] : (RH)qs[i];
}

// PCM enthalpy collision, Eqs. (32), (34)-(35), from the moments d (in RG,
// of the moving populations alone in the split form, where rest is q_0; d_0
// is then delta H - q_0, and the equilibrium of Eq. 34 is taken at it).
template <typename R, typename RH, typename RG>
LBM_HD void collide_pcm(const NodeConst<R, RH> &n, const Thermo<RH> &th, const Macro<R> &m, RH S_pcm, RG d[9],
                        RH rest, RH q[9]) {
    const RG dT = (RG)(th.Tf - n.Tf_ref);
    const RG jT = (RG)th.Tf * (RG)n.inv_phi;  // c_pl = 1
    const RG S = (RG)S_pcm;
    RG eq[7];  // eq_0 = d_0; eq_7 = eq_8 = 0
    eq[1] = fma_of(RG(-4), d[0], n.ge1 * dT);
    eq[2] = fma_of(RG(4), d[0], -(n.ge2 * dT));
    eq[3] = jT * (RG)m.ux;
    eq[4] = -eq[3];
    eq[5] = jT * (RG)m.uy;
    eq[6] = -eq[5];
    // scaled moments ((1 - zeta) d + zeta eq + S (1, -2, 1, 0, ...)) / |M_k|^2;
    // the zeroth moment is conserved (d_0 = eq_0), only S moves it
    RG a[9];
    a[0] = (d[0] + S) * moment_norm<RG>(0);
    a[1] = fma_of(RG(-2) * moment_norm<RG>(1), S, fma_of(n.zB1, eq[1], n.zA1 * d[1]));
    a[2] = fma_of(moment_norm<RG>(2), S, fma_of(n.zB1, eq[2], n.zA1 * d[2]));
    a[3] = fma_of(n.zB3, eq[3], n.zA3 * d[3]);
    a[4] = fma_of(n.zB4, eq[4], n.zA4 * d[4]);
    a[5] = fma_of(n.zB3, eq[5], n.zA3 * d[5]);
    a[6] = fma_of(n.zB4, eq[6], n.zA4 * d[6]);
    a[7] = n.zA7 * d[7];
    a[8] = n.zA7 * d[8];
    RG qs[9];
    from_scaled(a, qs);
    pcm_out(qs, rest, q);
}

// Metal-foam collision, Eqs. (43), (45)-(46).
template <typename R, typename RH>
LBM_HD void collide_metal(const NodeConst<R, RH> &n, const Macro<R> &m, R S_metal, R d[9], R q[9]) {
    // equilibrium (1, me1, me2, 0, ...) T_m (c_pm = 1); scaled moments
    // ((1 - eta) d + eta eq + S (1, -2, 1, 0, ...)) / |M_k|^2
    R a[9];
    a[0] = fma_of(moment_norm<R>(0), S_metal, fma_of(n.mB0, m.dTm, n.mA0 * d[0]));
    a[1] = fma_of(R(-2) * moment_norm<R>(1), S_metal, fma_of(n.mB1, n.me1 * m.dTm, n.mA1 * d[1]));
    a[2] = fma_of(moment_norm<R>(2), S_metal, fma_of(n.mB1, n.me2 * m.dTm, n.mA1 * d[2]));
    a[3] = n.mA3 * d[3];
    a[4] = n.mA4 * d[4];
    a[5] = n.mA3 * d[5];
    a[6] = n.mA4 * d[6];
    a[7] = n.mA7 * d[7];
    a[8] = n.mA7 * d[8];
    from_scaled(a, q);
}

// D2Q5 enthalpy collision (Appendix B): equilibrium moments Eq. (B2) on
// offsets, Theta in the moment order of Eq. (B1), source S (1, 0, 0, varpi, 0);
// scaled moments e_k = g_k ((1 - zeta_k) d_k + zeta_k eq_k + S_k), the
// zeroth moment conserved (d_0 = eq_0 = delta H) so only S moves it.
template <typename R, typename RH, typename RG>
LBM_HD void collide_pcm5(const NodeConst<R, RH> &n, const Thermo<RH> &th, const Macro<R> &m, RH S_pcm, RG d[9],
                         RH rest, RH q[9]) {
    const RG jT = (RG)th.Tf * (RG)n.inv_phi;  // c_pl = 1
    const RG eq1 = jT * (RG)m.ux, eq2 = jT * (RG)m.uy;  // eq_4 = 0
    const RG eq3 = n.ge1 * (RG)(th.Tf - n.Tf_ref);
    const RG S = (RG)S_pcm;
    RG e[5];
    e[0] = d[0] + S;
    e[1] = fma_of(n.zB1, eq1, n.zA1 * d[1]);
    e[2] = fma_of(n.zB1, eq2, n.zA1 * d[2]);
    e[3] = fma_of((RG)n.w4, S, fma_of(n.zB3, eq3, n.zA3 * d[3]));
    e[4] = n.zA3 * d[4];
    RG qs[9];
    from_scaled5(e, qs);
    qs[5] = qs[6] = qs[7] = qs[8] = RG(0);
    pcm_out(qs, rest, q);
}

// D2Q5 metal-foam collision (Appendix B): Eq. (B4), Q, S (1, 0, 0, varpi, 0),
// in the scaled moments of from_scaled5.
template <typename R, typename RH>
LBM_HD void collide_metal5(const NodeConst<R, RH> &n, const Macro<R> &m, R S_metal, R d[9], R q[9]) {
    const R eq3 = n.me1 * m.dTm;  // eq_0 = T_m (c_pm = 1), eq_1 = eq_2 = eq_4 = 0
    R e[5];
    e[0] = fma_of(n.mB0, m.dTm, n.mA0 * d[0]) + S_metal;
    e[1] = n.mA1 * d[1];
    e[2] = n.mA1 * d[2];
    e[3] = fma_of(n.w4, S_metal, fma_of(n.mB3, eq3, n.mA3 * d[3]));
    e[4] = n.mA3 * d[4];
    from_scaled5(e, q);
}

// Wall whose thermal condition a wall node carries: an isothermal vertical
// wall, else an isothermal horizontal wall, else -1 (adiabatic: the node
// copies its partner's temperature).
template <typename R>
LBM_HD int thermal_wall(const CavityConst<R> &c, int x, int y) {
    const int v = c.periodic ? -1 : (x == 0 ? W_LEFT : (x == c.nx - 1 ? W_RIGHT : -1));
    const int h = y == 0 ? W_BOTTOM : (y == c.ny - 1 ? W_TOP : -1);
    if (v >= 0 && c.wall_iso[v]) return v;
    if (h >= 0 && c.wall_iso[h]) return h;
    return -1;
}

// What the reconstruction of a wall node reads: the values of the isothermal
// wall it lies on (a vertical one before a horizontal one; iso false: it
// takes its partner's), selected from uniform values rather than loaded per
// lane, and constants of the enthalpy and metal fields.
template <typename R, typename RH>
struct WallNode {
    bool iso;
    RH Tb, Hb, c_fref, inv_phi, inv_cs2, varpi;
    R Tmb, c_mref, varpi_m;
};
template <typename RH, typename R>
LBM_HD WallNode<R, RH> wall_node(const CavityConst<R> &c, int x, int y) {
    const ThermalConst<RH> &t = thermal<RH>(c);
    WallNode<R, RH> w{false, RH(0), RH(0), t.c_fref, t.inv_phi, t.inv_cs2, t.varpi, R(0), c.c_mref, c.varpi};
    const bool on[4] = {!c.periodic && x == 0, !c.periodic && x == c.nx - 1, y == 0, y == c.ny - 1};
#pragma unroll
    for (int k = 3; k >= 0; --k)
        if (c.wall_iso[k]) {
            w.iso = on[k] || w.iso;
            w.Tb = on[k] ? t.T_wall[k] : w.Tb;
            w.Hb = on[k] ? t.H_wall[k] : w.Hb;
            w.Tmb = on[k] ? c.T_wall[k] : w.Tmb;
        }
    return w;
}

// Non-equilibrium extrapolation for a wall node, applied in place to the
// partner's pulled offsets (Eq. 52 with wall velocity 0; thermal analogues
// with the isothermal or zero-gradient wall values).
template <int QT, typename R, typename RH>
LBM_HD void reconstruct_wall(const WallNode<R, RH> &w, const NodeConst<R, RH> &n, R qf[9], RH qg[9], R qh[9]) {
    Thermo<RH> pt;
    Macro<R> p;
    macros<QT>(n, qf, qg, qh, pt, p);
    const RH Tb = w.iso ? w.Tb : pt.Tf, Hb = w.iso ? w.Hb : pt.H;
    const R Tmb = w.iso ? w.Tmb : p.Tm;
    const R uu = p.ux * p.ux + p.uy * p.uy;
    const RH dTg = Tb - pt.Tf;
    const R dTh = Tmb - p.Tm;
    // g^eq(H_b, T_b, 0) - g^eq(H, T, u) from Eq. (40) / Eq. (B3); h likewise
    // from Eq. (49) / Eq. (B5)
    const RH jT = w.inv_cs2 * pt.Tf * w.inv_phi;
    const R uu15 = R(1.5) * uu * n.inv_phi;
    qf[0] += -w_of<R>(0) * p.rho * -uu15;
    if (QT == 9) {
        qg[0] += (Hb - pt.H) - RH(5) / RH(9) * w.c_fref * dTg;
        qh[0] += (R(1) - R(5) / R(9) * w.c_mref) * dTh;
    } else {
        qg[0] += (Hb - pt.H) - w.varpi * w.c_fref * dTg;
        qh[0] += (R(1) - w.varpi_m * w.c_mref) * dTh;
    }
    // the moving directions by opposite pairs (1, 3), (2, 4), (5, 7), (6, 8)
    const int fwd[4] = {1, 2, 5, 6}, bwd[4] = {3, 4, 7, 8};
    const R along[4] = {p.ux, p.uy, p.ux + p.uy, p.uy - p.ux};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int i = fwd[k], j = bwd[k];
        const R eu = along[k];
        // f^eq(rho, 0) - f^eq(rho, u) from Eq. (27)
        const R e3 = R(3) * eu, e45 = R(4.5) * eu * eu * n.inv_phi, wr = -w_of<R>(i) * p.rho;
        qf[i] += wr * (e3 + e45 - uu15);
        qf[j] += wr * (e45 - e3 - uu15);
        if (i < QT) {
            const RH wg = QT == 9 ? w_of<RH>(i) : RH(0.25) * w.varpi;
            const R wh = QT == 9 ? w_of<R>(i) : R(0.25) * w.varpi_m;
            const RH cT = w.c_fref * dTg, ju = jT * (RH)eu;
            const R hw = wh * w.c_mref * dTh;
            qg[i] += wg * (cT - ju);
            qg[j] += wg * (cT + ju);
            qh[i] += hw;
            qh[j] += hw;
        }
    }
}

// Wall classification and the node whose populations a node pulls: its own
// neighbourhood, or its interior partner's for a wall node (inward normal
// neighbour, diagonal at corners).
enum { NODE_WALL = 1, NODE_NEAR_X = 2, NODE_NEAR_Y = 4, NODE_OWNED = 8 };
struct NodeGeom {
    int kind;  // NODE_WALL; NODE_NEAR_*: an interior node next to a vertical / horizontal wall
    int sx, sy;
    LBM_HD bool wall() const { return kind & NODE_WALL; }
    LBM_HD bool near_x() const { return kind & NODE_NEAR_X; }
    LBM_HD bool near_y() const { return kind & NODE_NEAR_Y; }
};

template <typename R>
LBM_HD NodeGeom geometry(const CavityConst<R> &c, int x, int y, bool pull) {
    NodeGeom g;
    const int nx = c.nx, ny = c.ny;
    const bool vwall = !c.periodic && (x == 0 || x == nx - 1);
    const bool hwall = (y == 0 || y == ny - 1);
    const bool wall = vwall || hwall;
    g.sx = x;
    g.sy = y;
    if (pull && wall) {
        if (!c.periodic) g.sx = (x == 0) ? 1 : ((x == nx - 1) ? nx - 2 : x);
        g.sy = (y == 0) ? 1 : ((y == ny - 1) ? ny - 2 : y);
    }
    g.kind = wall ? NODE_WALL
                  : (!c.periodic && (x == 1 || x == nx - 2) ? NODE_NEAR_X : 0) |
                        (y == 1 || y == ny - 2 ? NODE_NEAR_Y : 0);
    return g;
}

// Position of wall node r of the bottom and top rows (the wall columns are
// handled with their rows).
template <typename R>
LBM_HD void ring_node(const CavityConst<R> &c, int r, int &x, int &y) {
    const int nx = c.nx;
    if (r < nx) {
        x = r;
        y = 0;
    } else {
        x = r - nx;
        y = c.ny - 1;
    }
}

// Where node (x, y) of a cavity sits relative to a band block.  BandOrigin:
// rows of band ba and ba + 1 from band ba's block (the step kernels' tiles
// span at most two bands).  AnyBand: any row, from the cavity's first block.
struct BandOrigin {
    int y_first, y_next;  // first rows of bands ba and ba + 1
    int pitch;
    uint32_t band_bytes;
    LBM_HD NodeRef operator()(int x, int y) const {
        return y < y_next ? NodeRef{(uint32_t)((y - y_first) * pitch + x), 0u}
                          : NodeRef{(uint32_t)((y - y_next) * pitch + x), band_bytes};
    }
};
struct AnyBand {
    int band_rows, pitch;
    int64_t band_bytes;
    LBM_HD FarRef operator()(int x, int y) const {
        const int b = y / band_rows;
        return FarRef{(int64_t)(y - b * band_rows) * pitch + x, (int64_t)b * band_bytes};
    }
};
// Band of row y: a multiplication by the rounded-up reciprocal 2^32 /
// band_rows, one too large at most.
template <typename R>
LBM_HD int band_of(const CavityConst<R> &c, int y) {
    const uint32_t b = (uint32_t)(((uint64_t)(uint32_t)y * c.band_recip) >> 32);
    return (int)(b * (uint32_t)c.band_rows > (uint32_t)y ? b - 1 : b);
}
template <typename R>
LBM_HD BandOrigin band_origin(const CavityConst<R> &c, int ba) {  // from band ba
    return BandOrigin{ba * c.band_rows, (ba + 1) * c.band_rows, c.pitch, (uint32_t)c.band_bytes};
}
template <typename R>
LBM_HD AnyBand any_band(const CavityConst<R> &c) {
    return AnyBand{c.band_rows, c.pitch, c.band_bytes};
}
// The block of band b of cavity c in a state buffer.
template <typename R, typename V>
LBM_HD V *band_block(const CavityConst<R> &c, V *buf, int b) {
    return (V *)((ByteOf<V> *)buf + c.pop_off + (int64_t)b * c.band_bytes);
}
// Index of node (x, y) in the flat per-node arrays (interstitial source).
template <typename R>
LBM_HD int64_t flat_index(const CavityConst<R> &c, int x, int y) {
    return c.node0 + (int64_t)y * c.nx + x;
}

// Offsets of the node's post-streaming populations: pulled from the
// neighbours (Eqs. 15, 33, 44), or read in place for the initial state, from
// a whole state buffer.
template <class Lay, typename R, typename RH, bool PULL>
LBM_HD void gather(const CavityConst<R> &c, const void *buf, const NodeGeom &g, int x, int y, R qf[9], RH qg[9],
                   R qh[9]) {
    const void *src = band_block(c, buf, 0);
    const AnyBand addr = any_band(c);
    const int nx = c.nx;
    const int64_t stride = c.band_nodes;
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        int px = x, py = y;
        if (PULL) {
            px = g.sx - ex_of(i);
            if (c.periodic) px = px < 0 ? px + nx : (px >= nx ? px - nx : px);
            py = g.sy - ey_of(i);
        }
        const auto k = addr(px, py);
        qf[i] = Lay::template load<R>(src, stride, 0, i, k, c);
        if (i < Lay::QT) {
            qg[i] = Lay::template load<RH>(src, stride, 1, i, k, c);
            qh[i] = Lay::template load<R>(src, stride, 2, i, k, c);
        } else {
            qg[i] = RH(0);
            qh[i] = R(0);
        }
    }
}

// One workgroup's view of a state buffer: the rows it reads or writes lie in
// the bands ba and ba + 1 of its cavity (org).  flat: they lie in band ba
// alone and nothing wraps, so a pull's place is the node's own plus a
// uniform distance.
struct View {
    BandOrigin org;
    uint32_t stride;
    int nx, flat, periodic;
};
LBM_HD NodeRef place_of(const View &v, int x, int y) {
    return v.flat ? NodeRef{(uint32_t)((y - v.org.y_first) * v.org.pitch + x), 0u} : v.org(x, y);
}
template <typename R>
LBM_HD View view_of(const CavityConst<R> &c, int ba, int last_row) {
    const BandOrigin org = band_origin(c, ba);
    return View{org, (uint32_t)c.band_nodes, c.nx, !c.periodic && last_row < org.y_next, c.periodic};
}

// The node pulled along direction i by the node whose neighbourhood is at
// (sx, sy).  In a flat view every pull has one vector offset: the row is a
// uniform shift (planes that pull from the row below are never the first,
// so the sum stays positive) and the column a constant.
template <int I>
LBM_HD Pull pull_of(const View &v, int sx, int sy, bool flat) {
    if (flat)
        return Pull{-ey_of(I) * v.org.pitch, (uint32_t)((sy - v.org.y_first) * v.org.pitch + sx - 1),
                    (uint32_t)(1 - ex_of(I)), 0u};
    int px = sx - ex_of(I);
    if (v.periodic) px = px < 0 ? px + v.nx : (px >= v.nx ? px - v.nx : px);
    const NodeRef k = v.org(px, sy - ey_of(I));
    return Pull{0, k.rel, 0u, k.jump};
}
template <class Lay, typename R, typename RH, bool PULL, bool FLAT, int I = 0>
LBM_HD void pull_all(const NodeConst<R, RH> &n, Blocks b, const View &v, const NodeGeom &g, R qf[9], RH qg[9],
                     R qh[9]) {
    if constexpr (I < 9) {
        const NodeRef own = PULL ? NodeRef{0u, 0u} : v.org(g.sx, g.sy);
        const Pull p = PULL ? pull_of<I>(v, g.sx, g.sy, FLAT) : Pull{0, own.rel, 0u, own.jump};
        qf[I] = Lay::template pull<R>(b, v.stride, 0, I, p, n);
        if constexpr (I < Lay::QT) {
            qg[I] = Lay::template pull<RH>(b, v.stride, 1, I, p, n);
            qh[I] = Lay::template pull<R>(b, v.stride, 2, I, p, n);
        } else {
            qg[I] = RH(0);
            qh[I] = R(0);
        }
        pull_all<Lay, R, RH, PULL, FLAT, I + 1>(n, b, v, g, qf, qg, qh);
    }
}
// The same offsets as gather(), within a workgroup's blocks.
template <class Lay, typename R, typename RH, bool PULL>
LBM_HD void gather_view(const NodeConst<R, RH> &n, Blocks b, const View &v, const NodeGeom &g, R qf[9], RH qg[9],
                        R qh[9]) {
    if (PULL && v.flat) pull_all<Lay, R, RH, PULL, true>(n, b, v, g, qf, qg, qh);
    else pull_all<Lay, R, RH, PULL, false>(n, b, v, g, qf, qg, qh);
}

// Energy and mass carried by the three links between node (x, y), next to a
// vertical (X) or horizontal wall, and that wall, as offsets from what the
// reference state would carry (FP64): a step's inflow and outflow run over
// the same links, so their references cancel.  low: the left or bottom wall.
// Populations leave (OUT) along the directions that point at the wall and
// enter along their opposites; a diagonal between a corner-adjacent node and
// a vertical wall counts for that wall (skip_lo: the node is next to the left
// wall, skip_hi: the right one); energy moves only along the thermal
// lattice's links.
struct LinkSum {
    double E, M;
};
// Constants of walls and tallies, read from the cavity's table where needed.
template <typename R, typename RH>
struct TableWalls {
    const CavityConst<R> &c;
    LBM_HD WallNode<R, RH> node(int x, int y) const { return wall_node<RH>(c, x, y); }
    LBM_HD double we() const { return c.we; }
    LBM_HD double wm() const { return c.wm; }
};
template <int QT, bool X, bool OUT, class Walls, typename R, typename RH>
LBM_HD LinkSum wall_links(const Walls &walls, bool low, bool skip_lo, bool skip_hi, const R qf[9], const RH qg[9],
                          const R qh[9]) {
    using RG = typename MomentType<R, RH>::T;  // moving populations are held in it
    // directions with positive (p) and negative (n) component along the axis:
    // the axis, then the two diagonals
    constexpr int p[3] = {X ? 1 : 2, 5, X ? 8 : 6}, n[3] = {X ? 3 : 4, X ? 6 : 7, X ? 7 : 8};
    const bool pos = low != OUT;
    double f = 0.0, g = 0.0, h = 0.0;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        R af = pos ? qf[p[k]] : qf[n[k]], ah = pos ? qh[p[k]] : qh[n[k]];
        RG ag = pos ? (RG)qg[p[k]] : (RG)qg[n[k]];
        if (!X && k > 0) {
            // horizontal walls: the diagonals 5 and 7 cross the left wall's
            // column from below and the right one's from above, 6 and 8 the
            // other way round
            const bool skip = (k == 1) == low ? skip_lo : skip_hi;
            af = skip ? R(0) : af;
            ag = skip ? RG(0) : ag;
            ah = skip ? R(0) : ah;
        }
        f += (double)af;
        if (k == 0 || QT == 9) {
            g += (double)ag;
            h += (double)ah;
        }
    }
    return LinkSum{fma_of(walls.we(), g, walls.wm() * h), f};
}
// What the reference state carries along those links.
template <int QT, typename R>
LBM_HD LinkSum wall_reference(const CavityConst<R> &c, bool skip_lo, bool skip_hi) {
    const double diag = 2.0 - (skip_lo ? 1.0 : 0.0) - (skip_hi ? 1.0 : 0.0), dt = QT == 9 ? diag : 0.0;
    return LinkSum{c.we * (c.g_ref[1] + dt * c.g_ref[5]) + c.wm * (c.h_ref[1] + dt * c.h_ref[5]),
                   w_of<double>(1) + diag * w_of<double>(5)};
}

// Where the tallies of the nodes next to a wall are kept, energy and mass of
// one slot each: column() of a node next to the left or right wall by its
// row, row() of one next to the bottom or top wall by its column.
// CavityTally: the cavity's own, in global memory.
template <typename T, typename R>
struct CavityTally {
    T *acc;
    const CavityConst<R> &c;
    LBM_HD T *column(bool left, int y) const { return acc + 2 * (c.acc0 + (left ? y : c.ny + y)); }
    LBM_HD T *row(bool bottom, int x) const { return acc + 2 * (c.acc0 + 2 * c.ny + (bottom ? x : c.nx + x)); }
    LBM_HD void add(const double *from, double *to, LinkSum s) const {
        to[0] = from[0] + s.E;
        to[1] = from[1] + s.M;
    }
    LBM_HD void add_column(bool left, int y, LinkSum s) const { add(column(left, y), column(left, y), s); }
    LBM_HD void add_row(bool bottom, int x, LinkSum s) const { add(row(bottom, x), row(bottom, x), s); }
};
// TileTally: a tile's copy in LDS (TH left, TH right, TW bottom, TW top) for
// the updates of one launch; the last one adds to the copy and writes the
// cavity's (LAST).  Adding in global memory in each update put a round trip
// to memory into every update of the tiles at the walls, which in a small
// cavity set the launch's duration: with the links summed by selects instead
// of a branch per direction, 256^2 FP32_H64 went from 5.3 to 4.5 us a step.
template <int TW, int TH, bool LAST, typename R>
struct TileTally {
    static constexpr int N = 4 * (TW + TH);  // doubles
    CavityTally<double, R> all;
    double *lds;
    int x0, y0;
    LBM_HD double *column(bool left, int y) const { return lds + 2 * ((left ? 0 : TH) + y - y0); }
    LBM_HD double *row(bool bottom, int x) const { return lds + 2 * (2 * TH + (bottom ? 0 : TW) + x - x0); }
    LBM_HD void add_column(bool left, int y, LinkSum s) const {
        all.add(column(left, y), LAST ? all.column(left, y) : column(left, y), s);
    }
    LBM_HD void add_row(bool bottom, int x, LinkSum s) const {
        all.add(row(bottom, x), LAST ? all.row(bottom, x) : row(bottom, x), s);
    }
};

// Energy and mass carried by direction i of the given offsets (FP64).
template <int QT, typename R, typename RH>
LBM_HD void link_content(const CavityConst<R> &c, int i, const R qf[9], const RH qg[9], const R qh[9], double &e,
                         double &m) {
    e = i < QT ? c.we * (c.g_ref[i] + (double)qg[i]) + c.wm * (c.h_ref[i] + (double)qh[i]) : 0.0;
    m = (double)w_of<double>(i) + (double)qf[i];
}

// The update of one node from its gathered (post-streaming) offsets: wall
// tallies (only when the node's step is counted here, `tally`), wall
// reconstruction, macroscopic values, the three collisions and the
// interstitial sources.  On return q* hold the post-collision offsets and
// m, th the values the split layout stores as bases; the result is the
// new PCM source Sr_f.  edge (uniform over the workgroup): some node of the
// workgroup may be a wall node or next to one; without it the wall code is
// passed by a scalar branch.
template <int QT, typename R, typename RH, bool PULL, class Walls, class Tally>
LBM_HD RH update_node(const Walls &walls, const NodeConst<R, RH> &n, int edge, const NodeGeom &g, int x, int y,
                      R qf[9], RH qg[9], R qh[9], R sr_prev, bool tally, Tally acc, Thermo<RH> &th, Macro<R> &m) {
    // Wall tallies: an interior node next to a wall owns one slot per wall it
    // touches (x: the vertical wall, y: the horizontal one).  Set and read
    // under the same conditions only.
    LinkSum sx, sy;
    if (edge) {
        const bool lo = g.near_x() && x == 1, hi = g.near_x() && x != 1;
        // inflow: populations pulled from wall nodes (post-collision of the
        // previous step; the first step has none, and counts the outflow's
        // reference)
        if (tally && g.near_x()) {
            if constexpr (PULL) {
                sx = wall_links<QT, true, false>(walls, lo, false, false, qf, qg, qh);
            } else {
                sx = wall_reference<QT>(walls.c, false, false);
                sx = LinkSum{-sx.E, -sx.M};
            }
        }
        if (tally && g.near_y()) {
            if constexpr (PULL) {
                sy = wall_links<QT, false, false>(walls, y == 1, lo, hi, qf, qg, qh);
            } else {
                sy = wall_reference<QT>(walls.c, lo, hi);
                sy = LinkSum{-sy.E, -sy.M};
            }
        }
        if (PULL && g.wall()) reconstruct_wall<QT>(walls.node(x, y), n, qf, qg, qh);
    }

    Moments<R, RH> mo;
    field_moments<QT>(qf, qg, qh, mo);
    macros_of(n, mo, th, m);
    collide_flow(n, m, mo.f, qf);
    // Eqs. (36), (47) with the backward difference of Remark III.
    const RH srf = n.hv_f * ((RH)m.Tm - th.Tf);
    const R srm = n.hv_m * (m.Tf - m.Tm);
    const R srm_prev = -n.sr_ratio * sr_prev;
    const RH S_pcm = fma_of(RH(0.5), srf - (RH)sr_prev, srf);
    const R S_metal = fma_of(R(0.5), srm - srm_prev, srm);
    if (QT == 9) {
        collide_pcm(n, th, m, S_pcm, mo.g, mo.rest, qg);
        collide_metal(n, m, S_metal, mo.h, qh);
    } else {
        collide_pcm5(n, th, m, S_pcm, mo.g, mo.rest, qg);
        collide_metal5(n, m, S_metal, mo.h, qh);
    }

    if (edge) {
        const bool lo = g.near_x() && x == 1, hi = g.near_x() && x != 1;
        // outflow: post-collision populations aimed at wall nodes
        if (tally && g.near_x()) {
            const LinkSum o = wall_links<QT, true, true>(walls, lo, false, false, qf, qg, qh);
            acc.add_column(lo, y, LinkSum{sx.E - o.E, sx.M - o.M});
        }
        if (tally && g.near_y()) {
            const LinkSum o = wall_links<QT, false, true>(walls, y == 1, lo, hi, qf, qg, qh);
            acc.add_row(y == 1, x, LinkSum{sy.E - o.E, sy.M - o.M});
        }
    }
    return srf;
}

// One node's full time step on whole state buffers.
template <class Lay, typename R, typename RH, bool PULL>
LBM_HD void step_node(const CavityConst<R> &c, const void *src, void *dst, const R *__restrict__ sr_src,
                      R *__restrict__ sr_dst, double *__restrict__ acc, int x, int y) {
    const NodeConst<R, RH> &n = node_const_of<RH>(c);
    const NodeGeom g = geometry(c, x, y, PULL);
    R qf[9], qh[9];
    RH qg[9];
    gather<Lay, R, RH, PULL>(c, src, g, x, y, qf, qg, qh);
    const int64_t kf = flat_index(c, x, y);
    Thermo<RH> th;
    Macro<R> m;
    const RH srf = update_node<Lay::QT, R, RH, PULL>(TableWalls<R, RH>{c}, n, true, g, x, y, qf, qg, qh, sr_src[kf], true,
                                                          CavityTally<double, R>{acc, c}, th, m);
    const ThermalConst<RH> &t = thermal<RH>(c);
    const FarRef k = any_band(c)(x, y);
    void *blk = band_block(c, dst, 0);
    const int64_t stride = c.band_nodes;
    Lay::template store<R>(blk, stride, 0, qf, m.drho, k, c);
    Lay::template store<RH>(blk, stride, 1, qg, t.c_fref * (th.Tf - t.T_ref), k, c);
    Lay::template store<R>(blk, stride, 2, qh, c.c_mref * m.dTm, k, c);
    sr_dst[kf] = (R)srf;
}

// The same within a workgroup's view of the buffers (src and dst are the
// blocks of the view's first band); edge as for update_node.
template <class Lay, typename R, typename RH, bool PULL>
LBM_HD void step_node_view(const CavityConst<R> &c, const NodeConst<R, RH> &n, int edge, Blocks src, Blocks dst,
                           const View &v, const R *__restrict__ sr_src, R *__restrict__ sr_dst,
                           double *__restrict__ acc, int x, int y) {
    NodeGeom g{0, x, y};
    if (edge) g = geometry(c, x, y, PULL);
    R qf[9], qh[9];
    RH qg[9];
    gather_view<Lay, R, RH, PULL>(n, src, v, g, qf, qg, qh);
    const int64_t kf = flat_index(c, x, y);
    Thermo<RH> th;
    Macro<R> m;
    const RH srf = update_node<Lay::QT, R, RH, PULL>(TableWalls<R, RH>{c}, n, edge, g, x, y, qf, qg, qh, sr_src[kf], true,
                                                          CavityTally<double, R>{acc, c}, th, m);
    const NodeRef k = v.org(x, y);
    Lay::template put<R>(dst, v.stride, 0, qf, m.drho, k, n);
    Lay::template put<RH>(dst, v.stride, 1, qg, n.cf_base * (th.Tf - n.Tf_ref), k, n);
    Lay::template put<R>(dst, v.stride, 2, qh, n.cm_base * m.dTm, k, n);
    sr_dst[kf] = (R)srf;
}

// ---------------------------------------------------------------------------
// K steps per sweep through LDS (K = 2 or 3).  A tile of w x h nodes
// (w <= TW, h <= TH) at (x0, y0) is advanced K steps by updates over
// shrinking regions: R_j is the tile grown by a ring of j nodes (clipped to
// the cavity; unwrapped coordinates across a periodic seam).  The first
// update advances R_(K-1) from the global state into LDS, each middle update
// advances R_j (j = K-2 .. 1) in place in LDS (every node first reads its
// pulls into registers, then, after a barrier, writes its own slot), and the
// last update advances the tile from LDS into the global state.  The
// intermediate populations are kept in their storage type, so the result is
// bit-identical to K single steps.  The state crosses HBM once per K steps.
// A wall node pulls through its partner from at most one node beyond it
// inward, so R_j covers the update of R_(j-1) as long as no tile starts on
// the last column or row of a cavity (the host's tiling guarantees it).
// Only the tile's own nodes write wall tallies.  Plain layouts and the FP32
// layout with the FP64 rest enthalpy population: the LDS holds each
// population in the type it is stored in.
// ---------------------------------------------------------------------------
// How a layout keeps its populations in LDS for the K-step kernels: encoded
// exactly as it stores them (element type, 16-bit scale, split base), so
// that the next update sees the same values as a one-step launch would
// load.  put_node writes a node's post-collision offsets and the split
// layout's base values (bf, bg, bh, as the stores take them); get returns
// one population as the layout's load does.  NSLOT is the plane stride.
template <class Lay>
struct LdsCodec;
template <class E, bool SCALED, int QT_>
struct LdsCodec<Plain<E, SCALED, QT_>> {
    using R = decltype(E::dec(typename E::T()));  // arithmetic type of the kernels
    using T = typename E::T;
    using C = decltype(E::dec(T()));
    static constexpr int QT = QT_;
    static constexpr size_t bytes(int nslot) { return (size_t)(9 + 2 * QT) * nslot * sizeof(T); }
    LBM_HD static int plane(int f, int i) { return f == 0 ? i : 9 + (f - 1) * QT + i; }
    template <typename V, class S>
    LBM_HD static void put1(void *lds, int nslot, int f, int i, int slot, V v, const S &c) {
        ((T *)lds)[plane(f, i) * nslot + slot] = E::enc((C)(SCALED ? v * (V)c.scale[f] : v));
    }
    template <typename R, typename RH, class S>
    LBM_HD static void put_node(void *lds, int nslot, int slot, const S &c, const R qf[9],
                                const RH qg[9], const R qh[9], R bf, RH bg, R bh) {
        (void)bf;
        (void)bg;
        (void)bh;
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            put1(lds, nslot, 0, i, slot, qf[i], c);
            if (i < QT) {
                put1(lds, nslot, 1, i, slot, qg[i], c);
                put1(lds, nslot, 2, i, slot, qh[i], c);
            }
        }
    }
    template <typename V, class S>
    LBM_HD static V get(const void *lds, int nslot, int f, int i, int slot, const S &c) {
        const V v = (V)E::dec(((const T *)lds)[plane(f, i) * nslot + slot]);
        return SCALED ? v * (V)c.inv_scale[f] : v;
    }
};
template <int QT_>
struct LdsCodec<PlainH64<QT_>> {
    using R = float;
    static constexpr int QT = QT_;
    static constexpr int NF32 = PlainH64<QT_>::NF32;
    // FP32 planes, then the FP64 rest enthalpy plane (8-byte aligned)
    static constexpr size_t f64_offset(int nslot) { return ((size_t)NF32 * nslot * 4 + 7) & ~(size_t)7; }
    static constexpr size_t bytes(int nslot) { return f64_offset(nslot) + (size_t)nslot * 8; }
    template <typename V>
    LBM_HD static void put1(void *lds, int nslot, int f, int i, int slot, V v) {
        if (f == 1 && i == 0) ((double *)((char *)lds + f64_offset(nslot)))[slot] = (double)v;
        else ((float *)lds)[PlainH64<QT_>::plane(f, i) * nslot + slot] = (float)v;
    }
    template <typename V, class S>
    LBM_HD static void put1(void *lds, int nslot, int f, int i, int slot, V v, const S &c) {
        (void)c;
        put1(lds, nslot, f, i, slot, v);
    }
    template <typename R, typename RH, class S>
    LBM_HD static void put_node(void *lds, int nslot, int slot, const S &c, const R qf[9],
                                const RH qg[9], const R qh[9], R bf, RH bg, R bh) {
        (void)c;
        (void)bf;
        (void)bg;
        (void)bh;
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            put1(lds, nslot, 0, i, slot, qf[i]);
            if (i < QT) {
                put1(lds, nslot, 1, i, slot, qg[i]);
                put1(lds, nslot, 2, i, slot, qh[i]);
            }
        }
    }
    template <typename V, class S>
    LBM_HD static V get(const void *lds, int nslot, int f, int i, int slot, const S &c) {
        (void)c;
        if (f == 1 && i == 0) return (V)((const double *)((const char *)lds + f64_offset(nslot)))[slot];
        return (V)((const float *)lds)[PlainH64<QT_>::plane(f, i) * nslot + slot];
    }
};
// Split 16-bit layout: per field the FP32 rest population and base, then the
// eight 16-bit remainders from the base's rest equilibrium.
template <class ER>
struct LdsCodec<SplitT<ER>> {
    using R = float;
    static constexpr int QT = 9;
    static constexpr size_t bytes(int nslot) { return (size_t)nslot * (6 * 4 + 24 * 2); }
    template <typename V, class S>
    LBM_HD static void put_field(void *lds, int nslot, int f, int slot, const V q[9], V beta,
                                 const S &c) {
        float *P = (float *)lds;
        uint16_t *Qp = (uint16_t *)(P + 6 * nslot);
        const float b = (float)split_base<V>(beta);
        P[(2 * f) * nslot + slot] = (float)q[0];
        P[(2 * f + 1) * nslot + slot] = b;
#pragma unroll
        for (int i = 1; i < 9; ++i)
            Qp[(8 * f + i - 1) * nslot + slot] = ER::enc(split_rem<V>(i, q[i], (V)b, (V)c.scale[f]));
    }
    template <typename R, typename RH, class S>
    LBM_HD static void put_node(void *lds, int nslot, int slot, const S &c, const R qf[9],
                                const RH qg[9], const R qh[9], R bf, RH bg, R bh) {
        put_field(lds, nslot, 0, slot, qf, bf, c);
        put_field(lds, nslot, 1, slot, qg, bg, c);
        put_field(lds, nslot, 2, slot, qh, bh, c);
    }
    template <typename V, class S>
    LBM_HD static V get(const void *lds, int nslot, int f, int i, int slot, const S &c) {
        const float *P = (const float *)lds;
        if (i == 0) return (V)P[(2 * f) * nslot + slot];
        const V b = (V)P[(2 * f + 1) * nslot + slot];
        const uint16_t *Qp = (const uint16_t *)(P + 6 * nslot);
        const V r = (V)ER::dec(Qp[(8 * f + i - 1) * nslot + slot]);
        return split_dec<V>(i, b, r, (V)c.inv_scale[f]);
    }
};

// LDS placement of the intermediate populations.  Pull placement: a node
// writes its post-collision populations to its own slot and the next update
// reads each pull from the neighbour's slot, so the planes cover the first
// update's whole region.  Push placement: a node writes population i to the
// slot of the node that pulls it (x + e_i) and the next update reads all of
// its pulls from its own slot, so the planes need only cover the nodes that
// later updates read, the tile grown by K - 2 nodes; writes that fall
// outside are dropped.  Push is chosen where the smaller planes let one more
// workgroup share a CU.
#ifndef LBM_PUSH_F32_K3
#define LBM_PUSH_F32_K3 1
#endif
template <class Lay, int K>
struct PushLds {
    static constexpr bool value = false;
};
template <>
struct PushLds<Plain<E32, false, 9>, 3> {
    static constexpr bool value = LBM_PUSH_F32_K3;
};
#ifndef LBM_PUSH_F32H_K3
#define LBM_PUSH_F32H_K3 1
#endif
template <>
struct PushLds<PlainH64<9>, 3> {
    static constexpr bool value = LBM_PUSH_F32H_K3;
};
#ifndef LBM_PUSH_F64_K2
#define LBM_PUSH_F64_K2 1
#endif
template <>
struct PushLds<Plain<E64, false, 9>, 2> {
    static constexpr bool value = LBM_PUSH_F64_K2;
};
template <int QT>  // pulls would need the two-node ring in LDS: 95 KiB (D2Q9), one tile per CU
struct PushLds<Plain<E64, false, QT>, 3> {
    static constexpr bool value = true;
};

template <class Lay>
struct IsSplitLayout {
    static constexpr bool value = false;
};
template <class ER>
struct IsSplitLayout<SplitT<ER>> {
    static constexpr bool value = true;
};

template <class Lay, int TW, int TH, int K>
struct StepKShape {
    static constexpr int QT = Lay::QT;
    static constexpr int TILE_W = TW;
    static constexpr int RING = K - 1;          // ring of the first update
    static constexpr int LW = TW + 2 * RING;    // thread map pitch of the first update
    static constexpr int NFIRST = LW * (TH + 2 * RING);  // threads of the first update
    static constexpr bool PUSH = PushLds<Lay, K>::value;
    static constexpr int WR = PUSH ? K - 2 : RING;       // ring of the LDS window
    static constexpr int WW = TW + 2 * WR, WH = TH + 2 * WR;  // LDS window
    static constexpr int NSLOT = WW * WH;                // LDS plane stride
    using Codec = LdsCodec<Lay>;
    static constexpr size_t LDS_BYTES = Codec::bytes(NSLOT);
    // Split layouts: every pull of the first update needs the base of the
    // node it pulls from, so the workgroup first copies the bases of the
    // pulled region (the first update's region and one more ring) into LDS
    // and the pulls read them there instead of loading one base per pull.
    static constexpr bool STAGE_BASE = IsSplitLayout<Lay>::value;
    static constexpr int BW = TW + 2 * K, BH = TH + 2 * K;  // pulled region
    static constexpr int BP = BW;  // row pitch of the staged bases
    static constexpr int NBASE = STAGE_BASE ? BP * BH : 0;   // base plane stride
    static constexpr size_t BASE_BYTES = (size_t)3 * NBASE * sizeof(float);
    // LDS of a workgroup, and the workgroups of NT threads a CU holds (160
    // KiB, 32 waves).  The wall tallies move into LDS where that leaves as
    // many workgroups per CU as without them (all forms but D2Q5 FP32).
    using R = typename Codec::R;
    static constexpr size_t total_lds(bool tally) {
        return LDS_BYTES + NSLOT * sizeof(R) + BASE_BYTES + (tally ? 32 * (TW + TH) : 0);
    }
    static constexpr int NT = (NFIRST + 63) / 64 * 64;
    // Rounded to 128 bytes: the two-step FP64 D2Q5 tile (54400 bytes) fits a CU
    // three times, which rounding to 512 would deny, and with tallies in LDS
    // twice (4096^2: 29.9 GLUPS with its tallies in memory, 22.1 with them in LDS).
    static constexpr int per_cu(bool tally) {
        const int a = (int)(160 * 1024 / ((total_lds(tally) + 127) / 128 * 128)), b = 32 / (NT / 64);
        return a < b ? a : b;
    }
    static constexpr bool TILE_TALLY = per_cu(true) == per_cu(false);
    static_assert(TH + 2 * K <= LBM_MIN_BAND_ROWS, "a tile's rows must span at most two bands");
};

// Global accesses of a tile go through 32-bit offsets from the block of the
// band of the first row any update touches, y0 - K (the first update's ring
// and its pulls), clipped to the cavity: at most TH + 2K <= LBM_MIN_BAND_ROWS
// rows, so at most two bands.  edge: some node of the first update's region
// is a wall node, next to a wall or outside the cavity, or the tile is
// narrower than TW; a tile without it runs no wall code and no per-node
// bounds checks (at 8192^2, 99% of the tiles).
template <typename R>
struct TileView {
    View v;
    Tile2 tl;
    int yb;            // first row
    int64_t block;     // byte offset of the block of the first row's band in a state buffer
    int64_t flat_row;  // flat index of the first row
    int edge;
    const CavityConst<R> &c;
};
template <class Sh, typename R>
LBM_HD TileView<R> tile_view(const CavityConst<R> &c, Tile2 tl) {
    constexpr int K = Sh::RING + 1, M = Sh::RING + 2;
    const int yb = tl.y0 >= K ? tl.y0 - K : 0, last = tl.y0 + tl.h - 1 + K;
    const int ba = band_of(c, yb);
    const View v = view_of(c, ba, last < c.ny ? last : c.ny - 1);
    // one scalar condition, without a branch per term
    const int edge = (c.periodic != 0) | (tl.w < Sh::TILE_W) | (tl.x0 < M) | (tl.x0 + tl.w > c.nx - M) | (tl.y0 < M) |
                     (tl.y0 + tl.h > c.ny - M);
    TileView<R> t{v, tl, yb, c.pop_off + (int64_t)ba * c.band_bytes, c.node0 + (int64_t)yb * c.nx, edge, c};
    resident(t.v.org.y_first), resident(t.v.org.pitch), resident(t.v.stride), resident(t.v.nx);
    resident(t.tl.x0), resident(t.tl.y0), resident(t.tl.h), resident(t.block), resident(t.flat_row);
    resident_flag(t.edge), resident_flag(t.v.flat);
    return t;
}
template <class T, typename R>
LBM_HD T tally_of(const CavityTally<double, R> &all, double *lds, const TileView<R> &tv) {
    if constexpr (std::is_same<T, CavityTally<double, R>>::value) return all;
    else return T{all, lds, tv.tl.x0, tv.tl.y0};
}
template <typename T>
LBM_HD Blocks blocks_at(T *buf, int64_t byte) {
    return blocks_of((const char *)buf + byte);
}

// t / P and t % P of a thread index t < 1024.
template <int P>
LBM_HD int div_by(int t) {
    static_assert(P >= 1 && P < 1024, "t times the rounding of 2^20 / P stays below 2^20");
    return (int)(((uint32_t)t * (uint32_t)(((1 << 20) + P - 1) / P)) >> 20);
}
template <int P>
LBM_HD int mod_by(int t) {
    return t - div_by<P>(t) * P;
}

// Push placement: population i of the node at window position (wx, wy) goes
// to the slot of x + e_i if that lies in the window.
template <class Sh, typename R, typename RH>
LBM_HD void lds_push(const NodeConst<R, RH> &n, int wx, int wy, void *lds_q, const R qf[9], const RH qg[9],
                     const R qh[9]) {
    using Cd = typename Sh::Codec;
    const int own = wy * Sh::WW + wx;
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        if ((unsigned)(wx + ex_of(i)) < (unsigned)Sh::WW && (unsigned)(wy + ey_of(i)) < (unsigned)Sh::WH) {
            const int sl = own + ey_of(i) * Sh::WW + ex_of(i);
            LBM_HOST_CHECK(sl >= 0 && sl < Sh::NSLOT);
            Cd::put1(lds_q, Sh::NSLOT, 0, i, sl, qf[i], n);
            if (i < Sh::QT) {
                Cd::put1(lds_q, Sh::NSLOT, 1, i, sl, qg[i], n);
                Cd::put1(lds_q, Sh::NSLOT, 2, i, sl, qh[i], n);
            }
        }
    }
}
// The same, and Sr_f to the node's own slot.
template <class Sh, typename R, typename RH>
LBM_HD void lds_push(const NodeConst<R, RH> &n, int wx, int wy, void *lds_q, R *lds_sr, const R qf[9], const RH qg[9],
                     const R qh[9], RH srf) {
    lds_push<Sh, R, RH>(n, wx, wy, lds_q, qf, qg, qh);
    if ((unsigned)wx < (unsigned)Sh::WW && (unsigned)wy < (unsigned)Sh::WH) lds_sr[wy * Sh::WW + wx] = (R)srf;
}

// Split layouts, before the first update: thread t (of NT) copies the
// bases of its nodes of the pulled region (unwrapped columns tl.x0 - K ..
// tl.x0 + w + K - 1, rows tl.y0 - K .. tl.y0 + h + K - 1, at row pitch BP;
// nodes outside the cavity are skipped, nothing reads them) into three LDS
// planes of NBASE.
template <class Lay, typename R, int TW, int TH, int K, int NT>
LBM_HD void stepk_stage_bases(const TileView<R> &tv, const void *src, float *lds_b, int t) {
    using Sh = StepKShape<Lay, TW, TH, K>;
    static_assert(Sh::STAGE_BASE, "split layouts only");
    const Tile2 &tl = tv.tl;
    const Blocks blk = blocks_at(src, tv.block);
    for (int q = t; q < Sh::BP * (tl.h + 2 * K); q += NT) {
        const int bx = q % Sh::BP;
        if (bx >= tl.w + 2 * K) continue;
        const int x = tl.x0 - K + bx, y = tl.y0 - K + q / Sh::BP;  // unwrapped
        if (y < 0 || y >= tv.c.ny) continue;
        int xx = x;
        if (tv.v.periodic) xx = x < 0 ? x + tv.v.nx : (x >= tv.v.nx ? x - tv.v.nx : x);
        else if (x < 0 || x >= tv.v.nx) continue;
        LBM_HOST_CHECK(xx >= 0 && xx < tv.v.nx && q < Sh::NBASE);
        LBM_HOST_CHECK(y >= tv.yb && y < tv.yb + TH + 2 * K && y < tv.v.org.y_next + tv.c.band_rows);
        const NodeRef k = tv.v.org(xx, y);
#pragma unroll
        for (int f = 0; f < 3; ++f)
            lds_b[f * Sh::NBASE + q] = Lay::pull_base(blk, tv.v.stride, f, Pull{0, k.rel, 0u, k.jump});
    }
}

// Split layouts, first update: the pulls of the node at unwrapped column x
// (wrapped xx) or of its wall partner, with the pulled nodes' bases from
// the staged LDS copy; the same values as gather_view.
template <class Sh, class Lay, bool FLAT, typename R, typename RH, int I = 0>
LBM_HD void pull_staged(const NodeConst<R, RH> &n, const Tile2 &tl, Blocks b, const View &v, const NodeGeom &g, int px,
                        const float *lds_b, R qf[9], RH qg[9], R qh[9]) {
    if constexpr (I < 9) {
        constexpr int K = Sh::RING + 1;
        const Pull p = pull_of<I>(v, g.sx, g.sy, FLAT);
        if constexpr (I == 0) {
            qf[0] = Lay::template pull<R>(b, v.stride, 0, 0, p, n);
            qg[0] = Lay::template pull<RH>(b, v.stride, 1, 0, p, n);
            qh[0] = Lay::template pull<R>(b, v.stride, 2, 0, p, n);
        } else {
            const int bi = (g.sy - ey_of(I) - (tl.y0 - K)) * Sh::BP + (px - ex_of(I) - (tl.x0 - K));
            LBM_HOST_CHECK(px - ex_of(I) - (tl.x0 - K) >= 0 && px - ex_of(I) - (tl.x0 - K) < tl.w + 2 * K);
            LBM_HOST_CHECK(g.sy - ey_of(I) - (tl.y0 - K) >= 0 && g.sy - ey_of(I) - (tl.y0 - K) < tl.h + 2 * K);
            LBM_HOST_CHECK(bi >= 0 && bi < Sh::NBASE);
            qf[I] = Lay::template pull_moving<R>(b, v.stride, 0, I, p, (R)lds_b[bi], n);
            qg[I] = Lay::template pull_moving<RH>(b, v.stride, 1, I, p, (RH)lds_b[Sh::NBASE + bi], n);
            qh[I] = Lay::template pull_moving<R>(b, v.stride, 2, I, p, (R)lds_b[2 * Sh::NBASE + bi], n);
        }
        pull_staged<Sh, Lay, FLAT, R, RH, I + 1>(n, tl, b, v, g, px, lds_b, qf, qg, qh);
    }
}

// First update: slot s of R_(K-1) (row-major with the fixed pitch LW, so the
// decode divides by a constant; columns beyond w + 2 RING idle).  Reads the
// global state (split layouts: with the bases staged in lds_b), writes the
// slot's post-collision populations and Sr_f to LDS.
template <class Lay, typename R, typename RH, int TW, int TH, int K, class Tally>
LBM_HD void stepk_first(const TileView<R> &tv, const NodeConst<R, RH> &n, const void *src,
                        const R *__restrict__ sr_src, Tally acc, void *lds_q, R *lds_sr,
                        const float *lds_b, int s) {
    using Sh = StepKShape<Lay, TW, TH, K>;
    constexpr int LW = Sh::LW, RG = Sh::RING;
    const CavityConst<R> &c = tv.c;
    const Tile2 &tl = tv.tl;
    LBM_HOST_CHECK(s >= 0 && s < LW * (tl.h + 2 * RG) && s < Sh::NFIRST);
    const int lx = mod_by<LW>(s), ly = div_by<LW>(s);
    const int x = tl.x0 - RG + lx, y = tl.y0 - RG + ly;  // unwrapped
    int xx = x;
    NodeGeom g{0, x, y};
    if (tv.edge) {
        if (lx >= tl.w + 2 * RG) return;
        if (y < 0 || y >= c.ny) return;
        if (c.periodic) xx = x < 0 ? x + c.nx : (x >= c.nx ? x - c.nx : x);
        else if (x < 0 || x >= c.nx) return;
        g = geometry(c, xx, y, true);
        if (x >= tl.x0 && x < tl.x0 + tl.w && y >= tl.y0 && y < tl.y0 + tl.h) g.kind |= NODE_OWNED;
    }
    LBM_HOST_CHECK(xx >= 0 && xx < c.nx);
    LBM_HOST_CHECK(tv.edge || (x >= 2 && x <= c.nx - 3 && y >= 2 && y <= c.ny - 3));
    LBM_HOST_CHECK(g.sy - 1 >= tv.yb && g.sy + 1 < tv.yb + TH + 2 * K);
    LBM_HOST_CHECK(g.sy + 1 < tv.v.org.y_next + (tv.v.flat ? 0 : c.band_rows));
    const Blocks b = blocks_at(src, tv.block);
    R qf[9], qh[9];
    RH qg[9];
    LinkSum ax, ay;  // the tallies so far, read with the populations
    const auto owned_near = [&](int near) { return (g.kind & (NODE_OWNED | near)) == (NODE_OWNED | near); };
    if constexpr (!std::is_same<Tally, CavityTally<double, R>>::value) if (tv.edge) {
        if (owned_near(NODE_NEAR_X)) ax = LinkSum{acc.all.column(x == 1, y)[0], acc.all.column(x == 1, y)[1]};
        if (owned_near(NODE_NEAR_Y)) ay = LinkSum{acc.all.row(y == 1, x)[0], acc.all.row(y == 1, x)[1]};
    }
    if constexpr (Sh::STAGE_BASE) {
        const int px = x + (g.sx - xx);  // partner column, unwrapped
        if (tv.v.flat) pull_staged<Sh, Lay, true, R, RH>(n, tl, b, tv.v, g, px, lds_b, qf, qg, qh);
        else pull_staged<Sh, Lay, false, R, RH>(n, tl, b, tv.v, g, px, lds_b, qf, qg, qh);
    } else {
        gather_view<Lay, R, RH, true>(n, b, tv.v, g, qf, qg, qh);
    }
    (void)lds_b;
    if constexpr (!std::is_same<Tally, CavityTally<double, R>>::value) if (tv.edge) {
        if (owned_near(NODE_NEAR_X)) acc.column(x == 1, y)[0] = ax.E, acc.column(x == 1, y)[1] = ax.M;
        if (owned_near(NODE_NEAR_Y)) acc.row(y == 1, x)[0] = ay.E, acc.row(y == 1, x)[1] = ay.M;
    }
    Thermo<RH> th;
    Macro<R> m;
    const R sr_prev = ld_block<R>(blocks_at(sr_src + tv.flat_row, 0), 0, (uint32_t)((y - tv.yb) * tv.v.nx + xx) * sizeof(R), 0);
    const RH srf =
        update_node<Sh::QT, R, RH, true>(TableWalls<R, RH>{c}, n, tv.edge, g, xx, y, qf, qg, qh, sr_prev, g.kind & NODE_OWNED, acc, th, m);
    if constexpr (Sh::PUSH) {
        lds_push<Sh, R, RH>(n, lx - RG + Sh::WR, ly - RG + Sh::WR, lds_q, lds_sr, qf, qg, qh, srf);
    } else {
        Sh::Codec::put_node(lds_q, Sh::NSLOT, s, n, qf, qg, qh, m.drho, n.cf_base * (th.Tf - n.Tf_ref),
                            n.cm_base * m.dTm);
        lds_sr[s] = (R)srf;
    }
}

// A node's pulls from LDS; slot is that of the node or of its wall partner.
template <class Sh, typename R, typename RH>
LBM_HD void lds_gather(const NodeConst<R, RH> &n, int slot, const void *lds_q, R qf[9], RH qg[9], R qh[9]) {
    using Cd = typename Sh::Codec;
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        // push placement: every pull of a node sits in its own slot
        const int sl = Sh::PUSH ? slot : slot - ey_of(i) * Sh::WW - ex_of(i);
        LBM_HOST_CHECK(sl >= 0 && sl < Sh::NSLOT);
        qf[i] = Cd::template get<R>(lds_q, Sh::NSLOT, 0, i, sl, n);
        if (i < Sh::QT) {
            qg[i] = Cd::template get<RH>(lds_q, Sh::NSLOT, 1, i, sl, n);
            qh[i] = Cd::template get<R>(lds_q, Sh::NSLOT, 2, i, sl, n);
        } else {
            qg[i] = RH(0);
            qh[i] = R(0);
        }
    }
}
// The slot a node pulls through: its own, or its wall partner's (edge tiles).
// x is the node's unwrapped column, xx the wrapped one.
template <class Sh>
LBM_HD int pull_slot(const Tile2 &tl, const NodeGeom &g, int x, int xx, int own, int y) {
    const int slot = own + (g.sy - y) * Sh::WW + (g.sx - xx);
    const int wx = x + (g.sx - xx) - (tl.x0 - Sh::WR), wy = g.sy - (tl.y0 - Sh::WR);
    (void)wx;
    (void)wy;
    // the partner itself (push), or its neighbours too (pull), lie in the window
    LBM_HOST_CHECK(wx >= (Sh::PUSH ? 0 : 1) && wx < Sh::WW - (Sh::PUSH ? 0 : 1));
    LBM_HOST_CHECK(wy >= (Sh::PUSH ? 0 : 1) && wy < tl.h + 2 * Sh::WR - (Sh::PUSH ? 0 : 1));
    return slot;
}

// A middle update of ring j (1 <= j <= K - 2), split at the barrier that
// lets it run in place: stepk_mid_load reads thread t's node's pulls into
// registers (false: the thread has no node), stepk_mid_store updates the
// node and writes its own slot.
template <typename R, typename RH>
struct MidNode {
    int lx, ly, xx, y, slot;
    NodeGeom g;
    R qf[9], qh[9], sr_prev;
    RH qg[9];
};
template <class Lay, typename R, typename RH, int TW, int TH, int K, int J>
LBM_HD bool stepk_mid_load(const TileView<R> &tv, const NodeConst<R, RH> &n, const void *lds_q, const R *lds_sr, int t,
                           MidNode<R, RH> &q) {
    using Sh = StepKShape<Lay, TW, TH, K>;
    constexpr int P = TW + 2 * J;  // pitch of ring J's thread map
    const CavityConst<R> &c = tv.c;
    const Tile2 &tl = tv.tl;
    q.lx = mod_by<P>(t);
    q.ly = div_by<P>(t);
    const int x = tl.x0 - J + q.lx, y = tl.y0 - J + q.ly;  // unwrapped
    q.xx = x;
    q.y = y;
    q.g = NodeGeom{0, x, y};
    q.slot = P == Sh::WW ? t : (q.ly + Sh::WR - J) * Sh::WW + q.lx + Sh::WR - J;
    int from = q.slot;
    if (tv.edge) {
        if (q.lx >= tl.w + 2 * J) return false;
        if (y < 0 || y >= c.ny) return false;
        if (c.periodic) q.xx = x < 0 ? x + c.nx : (x >= c.nx ? x - c.nx : x);
        else if (x < 0 || x >= c.nx) return false;
        q.g = geometry(c, q.xx, y, true);
        if (x >= tl.x0 && x < tl.x0 + tl.w && y >= tl.y0 && y < tl.y0 + tl.h) q.g.kind |= NODE_OWNED;
        from = pull_slot<Sh>(tl, q.g, x, q.xx, q.slot, y);
    }
    LBM_HOST_CHECK(q.ly < tl.h + 2 * J && q.xx >= 0 && q.xx < c.nx);
    LBM_HOST_CHECK(q.slot >= 0 && q.slot < Sh::NSLOT);
    lds_gather<Sh, R, RH>(n, from, lds_q, q.qf, q.qg, q.qh);
    q.sr_prev = lds_sr[q.slot];
    return true;
}
template <class Lay, typename R, typename RH, int TW, int TH, int K, int J, class Tally>
LBM_HD void stepk_mid_store(const TileView<R> &tv, const NodeConst<R, RH> &n, Tally acc, void *lds_q,
                            R *lds_sr, MidNode<R, RH> &q) {
    using Sh = StepKShape<Lay, TW, TH, K>;
    Thermo<RH> th;
    Macro<R> m;
    const RH srf = update_node<Sh::QT, R, RH, true>(TableWalls<R, RH>{tv.c}, n, tv.edge, q.g, q.xx, q.y, q.qf, q.qg, q.qh, q.sr_prev,
                                                   q.g.kind & NODE_OWNED, acc, th, m);
    if constexpr (Sh::PUSH) {
        lds_push<Sh, R, RH>(n, q.lx - J + Sh::WR, q.ly - J + Sh::WR, lds_q, lds_sr, q.qf, q.qg, q.qh, srf);
    } else {
        Sh::Codec::put_node(lds_q, Sh::NSLOT, q.slot, n, q.qf, q.qg, q.qh, m.drho, n.cf_base * (th.Tf - n.Tf_ref),
                            n.cm_base * m.dTm);
        lds_sr[q.slot] = (R)srf;
    }
}

// Last update: node s of the tile (row-major with pitch TW; columns beyond
// w idle).  Pulls from LDS, writes the global state.
template <class Lay, typename R, typename RH, int TW, int TH, int K, class Tally>
LBM_HD void stepk_last(const TileView<R> &tv, const NodeConst<R, RH> &n, void *dst,
                       R *__restrict__ sr_dst, Tally acc, const void *lds_q, const R *lds_sr, int s) {
    using Sh = StepKShape<Lay, TW, TH, K>;
    const CavityConst<R> &c = tv.c;
    const Tile2 &tl = tv.tl;
    LBM_HOST_CHECK(s >= 0 && s < TW * tl.h);
    const int lx = mod_by<TW>(s), ly = div_by<TW>(s);
    const int x = tl.x0 + lx, y = tl.y0 + ly;
    const int own = (ly + Sh::WR) * Sh::WW + lx + Sh::WR;
    int from = own;
    NodeGeom g{0, x, y};
    if (tv.edge) {
        if (lx >= tl.w) return;
        g = geometry(c, x, y, true);
        from = pull_slot<Sh>(tl, g, x, x, own, y);
    }
    LBM_HOST_CHECK(x >= 0 && x < c.nx && y >= 0 && y < c.ny);
    R qf[9], qh[9];
    RH qg[9];
    lds_gather<Sh, R, RH>(n, from, lds_q, qf, qg, qh);
    Thermo<RH> th;
    Macro<R> m;
    const RH srf =
        update_node<Sh::QT, R, RH, true>(TableWalls<R, RH>{c}, n, tv.edge, g, x, y, qf, qg, qh, lds_sr[own], true, acc, th, m);
    const NodeRef k = place_of(tv.v, x, y);
    const Blocks b = blocks_at(dst, tv.block);
    Lay::template put<R>(b, tv.v.stride, 0, qf, m.drho, k, n);
    Lay::template put<RH>(b, tv.v.stride, 1, qg, n.cf_base * (th.Tf - n.Tf_ref), k, n);
    Lay::template put<R>(b, tv.v.stride, 2, qh, n.cm_base * m.dTm, k, n);
    *(R *)((char *)(sr_dst + tv.flat_row) + (uint32_t)((y - tv.yb) * tv.v.nx + x) * (uint32_t)sizeof(R)) = (R)srf;
}

// Brings the rows a tile will be the first to read into the XCD's L2: item q
// of NP planes of elements of ES bytes from byte `plane0` on (stride nodes
// apart), TH rows each, one load per 128-byte line.  v receives the loads.
template <int ES, int NP, int TW, int TH, int NT, int N>
LBM_HD void touch_lines(Blocks b, const BandOrigin &org, uint32_t stride, uint32_t plane0, int x0, int x1, int y0, int y1,
                        int t, uint32_t (&v)[N]) {
    constexpr int EL = 128 / ES, LINES = (TW + EL - 1) / EL;  // elements per line, lines per row
    static_assert(N * NT >= NP * TH * LINES, "one load per item");
#pragma unroll
    for (int k = 0; k < N; ++k) {
        const int q = t + k * NT, line = q % LINES, row = (q / LINES) % TH, p = q / (LINES * TH);
        const int x = x0 + line * EL, y = y0 + row;
        v[k] = 0;
        if (p < NP && x < x1 && y < y1) {
            const NodeRef r = org(x, y);
            v[k] = ld_block<uint32_t>(b, plane0, ((p * stride + r.rel) * ES + r.jump) & ~3u, 0);
        }
    }
}
template <int N>
LBM_HD void wait_lines(uint32_t (&v)[N]) {
#if defined(__HIP_DEVICE_COMPILE__)
#pragma unroll
    for (int k = 0; k < N; ++k) asm volatile("" : : "v"(v[k]));
#else
    (void)v;
#endif
}
// What a tile will be the first to read of its state: its columns of the
// rows from K below its own first (the tile before it in its column has read
// those up to there) to K beyond its last.  Run by threads t of NT that have
// no node in the last update: without it the first update's pulls come from
// HBM and hold the workgroup for about a quarter of its life with little to
// overlap (the waves of a tile load together, three tiles share a CU).
// Measured with the strip order of the tiles (cavity_tiles2), 8192^2, three
// steps per launch: FP32_H64 46.5 -> 51.3 GLUPS, FP32 48.1 -> 52.8, D2Q5 FP32
// 72.0 -> 75.0, F16_SPLIT (4096^2) 44.4 -> 49.0 (53.9 since, with its constants
// in memory).
template <class Lay, typename R, int TW, int TH, int K, int NT>
LBM_HD void stepk_prefetch(const CavityConst<R> &c, const Tile2 &tl, const void *src, int t) {
    const int y0 = tl.y0 ? tl.y0 + K : 0, end = tl.y0 + tl.h + K, y1 = end < c.ny ? end : c.ny;
    if (y0 >= y1) return;
    const int ba = band_of(c, y0);
    const BandOrigin org = band_origin(c, ba);
    const Blocks b = blocks_at(src, c.pop_off + (int64_t)ba * c.band_bytes);
    const uint32_t stride = (uint32_t)c.band_nodes;
    const int x1 = tl.x0 + tl.w;
    constexpr int TR = TH + K;  // rows of a first tile
    auto n = [](int es, int planes) { return (planes * TR * ((TW * es + 127) / 128) + NT - 1) / NT; };
    if constexpr (IsSplitLayout<Lay>::value) {
        uint32_t v[n(4, 6)], w[n(2, 24)];
        touch_lines<4, 6, TW, TR, NT>(b, org, stride, 0, tl.x0, x1, y0, y1, t, v);
        touch_lines<2, 24, TW, TR, NT>(b, org, stride, 24 * stride, tl.x0, x1, y0, y1, t, w);
        wait_lines(v);
        wait_lines(w);
    } else if constexpr (std::is_same<Lay, PlainH64<Lay::QT>>::value) {
        uint32_t v[n(4, 8 + 2 * Lay::QT)], w[n(8, 1)];
        touch_lines<4, 8 + 2 * Lay::QT, TW, TR, NT>(b, org, stride, 0, tl.x0, x1, y0, y1, t, v);
        touch_lines<8, 1, TW, TR, NT>(b, org, stride, (8 + 2 * Lay::QT) * 4 * stride, tl.x0, x1, y0, y1, t, w);
        wait_lines(v);
        wait_lines(w);
    } else {
        constexpr int es = (int)sizeof(typename Lay::T), np = 9 + 2 * Lay::QT;
        uint32_t v[n(es, np)];
        touch_lines<es, np, TW, TR, NT>(b, org, stride, 0, tl.x0, x1, y0, y1, t, v);
        wait_lines(v);
    }
}

// The same from the cavity's table and a tile (host builds).
template <class Lay, typename R, int TW, int TH, int K, int NT>
LBM_HD void stepk_stage_bases(const CavityConst<R> &c, const Tile2 &tl, const void *src, float *lds_b, int t) {
    stepk_stage_bases<Lay, R, TW, TH, K, NT>(tile_view<StepKShape<Lay, TW, TH, K>>(c, tl), src, lds_b, t);
}
template <class Lay, typename R, typename RH, int TW, int TH, int K>
LBM_HD void stepk_first(const CavityConst<R> &c, const Tile2 &tl, const void *src, const R *__restrict__ sr_src,
                        double *__restrict__ acc, void *lds_q, R *lds_sr, const float *lds_b, int s) {
    stepk_first<Lay, R, RH, TW, TH, K>(tile_view<StepKShape<Lay, TW, TH, K>>(c, tl), node_const_of<RH>(c), src, sr_src,
                                       CavityTally<double, R>{acc, c}, lds_q, lds_sr, lds_b, s);
}
template <class Lay, typename R, typename RH, int TW, int TH, int K>
LBM_HD bool stepk_mid_load(const CavityConst<R> &c, const Tile2 &tl, int j, const void *lds_q, const R *lds_sr, int t,
                           MidNode<R, RH> &q) {
    static_assert(K <= 3, "one middle update");
    LBM_HOST_CHECK(j == 1);
    (void)j;
    return stepk_mid_load<Lay, R, RH, TW, TH, K, 1>(tile_view<StepKShape<Lay, TW, TH, K>>(c, tl),
                                                    node_const_of<RH>(c), lds_q, lds_sr, t, q);
}
template <class Lay, typename R, typename RH, int TW, int TH, int K>
LBM_HD void stepk_mid_store(const CavityConst<R> &c, const Tile2 &tl, double *__restrict__ acc, void *lds_q, R *lds_sr,
                            MidNode<R, RH> &q) {
    stepk_mid_store<Lay, R, RH, TW, TH, K, 1>(tile_view<StepKShape<Lay, TW, TH, K>>(c, tl), node_const_of<RH>(c), CavityTally<double, R>{acc, c},
                                              lds_q, lds_sr, q);
}
template <class Lay, typename R, typename RH, int TW, int TH, int K>
LBM_HD void stepk_last(const CavityConst<R> &c, const Tile2 &tl, void *dst, R *__restrict__ sr_dst,
                       double *__restrict__ acc, const void *lds_q, const R *lds_sr, int s) {
    stepk_last<Lay, R, RH, TW, TH, K>(tile_view<StepKShape<Lay, TW, TH, K>>(c, tl), node_const_of<RH>(c), dst, sr_dst,
                                      CavityTally<double, R>{acc, c}, lds_q, lds_sr, s);
}

// ---------------------------------------------------------------------------
// Deep launches: up to K steps per launch for cavities of so few tiles that a
// launch's fixed cost and one tile's latency, not the GPU's throughput, set
// the time.  One thread keeps one node of the tile's region (the tile and a
// ring of K - 1) for the whole launch: its place, geometry, source and wall
// tallies and the update's constants stay in registers, its populations pass
// through LDS planes that cover the region (every node writes its own slot
// and reads its neighbours'; a push, with its masked writes, took 1000 of an
// update's 5700 cycles).  A launch of k <= K steps runs k updates, each of the
// nodes at most as deep in the ring as updates are left; the steps are those
// of the K-step kernels, so the bits are too.
// ---------------------------------------------------------------------------
template <class Lay, int TW, int TH, int K>
struct DeepShape {
    static constexpr int QT = Lay::QT, TILE_W = TW, RING = K - 1;
    static constexpr int PW = TW + 2 * RING, PH = TH + 2 * RING;  // thread map: the region, row by row
    static constexpr int NT = (PW * PH + 63) / 64 * 64;
    static constexpr bool PUSH = false;
    static constexpr int WR = RING, WW = PW, NSLOT = PW * PH;  // LDS window: a slot per node
    using Codec = LdsCodec<Lay>;
    static constexpr size_t LDS_BYTES = Codec::bytes(NSLOT);
    static_assert(K >= 2 && NT <= 1024 && LDS_BYTES <= 160 * 1024, "one thread per node, one workgroup's LDS");
    static_assert(TH + 2 * K <= LBM_MIN_BAND_ROWS, "a tile's rows must span at most two bands");
};

// A node's tallies so far, in registers.
struct NodeTally {
    LinkSum &x, &y;
    LBM_HD void add_column(bool, int, LinkSum s) const { x = LinkSum{x.E + s.E, x.M + s.M}; }
    LBM_HD void add_row(bool, int, LinkSum s) const { y = LinkSum{y.E + s.E, y.M + s.M}; }
};

// The walls' constants of one node, in registers.
template <typename R, typename RH>
struct KeptWalls {
    WallNode<R, RH> wall;
    double phi_l, phi_m;  // CavityConst::we, wm
    LBM_HD const WallNode<R, RH> &node(int, int) const { return wall; }
    LBM_HD double we() const { return phi_l; }
    LBM_HD double wm() const { return phi_m; }
};

template <typename R, typename RH>
struct DeepNode {
    int from;      // slot it pulls through: its own, or its wall partner's
    int depth;     // rings outside the tile (0: the tile's own); INT32_MAX: no node
    int x, y;      // in the cavity
    NodeGeom g;
    R qf[9], qh[9], sr;
    RH qg[9];
    Thermo<RH> th;
    Macro<R> m;
    LinkSum tx, ty;
    KeptWalls<R, RH> walls;
};

// Thread t's node, and its populations, source and tallies from global
// memory if the first of k updates covers it.
template <class Sh, class Lay, typename R, typename RH>
LBM_HD void deep_load(const TileView<R> &tv, const NodeConst<R, RH> &n, const void *src, const R *__restrict__ sr_src,
                      const double *__restrict__ acc, int k, int t, DeepNode<R, RH> &q) {
    const CavityConst<R> &c = tv.c;
    const Tile2 &tl = tv.tl;
    const int lx = mod_by<Sh::PW>(t), ly = div_by<Sh::PW>(t);
    const int x = tl.x0 - Sh::RING + lx, y = tl.y0 - Sh::RING + ly;
    const int ox = lx < Sh::RING ? Sh::RING - lx : lx - Sh::RING - tl.w + 1;
    const int oy = ly < Sh::RING ? Sh::RING - ly : ly - Sh::RING - tl.h + 1;
    q.depth = ox > oy ? (ox > 0 ? ox : 0) : (oy > 0 ? oy : 0);
    q.x = x;
    q.y = y;
    q.g = NodeGeom{0, x, y};
    q.from = t;
    if (tv.edge) {
        // (periodic problems take no deep launches)
        if ((unsigned)x >= (unsigned)c.nx || (unsigned)y >= (unsigned)c.ny) {
            q.depth = INT32_MAX;
        } else {
            q.g = geometry(c, q.x, y, true);
            if (q.depth == 0) q.g.kind |= NODE_OWNED;
            q.from += (q.g.sy - y) * Sh::WW + (q.g.sx - q.x);
        }
    }
    if (q.depth > k - 1) {
        q.depth = INT32_MAX;
        return;
    }
    LBM_HOST_CHECK(q.x >= 0 && q.x < c.nx && y >= 0 && y < c.ny);
    LBM_HOST_CHECK(tv.edge || (x >= 2 && x <= c.nx - 3 && y >= 2 && y <= c.ny - 3));
    LBM_HOST_CHECK(q.g.sy - 1 >= tv.yb && q.g.sy + 1 < tv.yb + LBM_MIN_BAND_ROWS);
    LBM_HOST_CHECK(q.g.sy + 1 < tv.v.org.y_next + (tv.v.flat ? 0 : c.band_rows));
    if (tv.edge) {
        // read with the populations, for all updates
        KeptWalls<R, RH> w{wall_node<RH>(c, q.x, y), c.we, c.wm};
        resident<true>(w.wall.c_fref), resident<true>(w.wall.inv_phi), resident<true>(w.wall.inv_cs2);
        resident<true>(w.wall.c_mref), resident<true>(w.phi_l), resident<true>(w.phi_m);
        if constexpr (Lay::QT == 5) resident<true>(w.wall.varpi), resident<true>(w.wall.varpi_m);
        q.walls = w;
    }
    if (tv.edge && (q.g.kind & NODE_OWNED)) {
        const CavityTally<const double, R> a{acc, c};
        if (q.g.near_x()) q.tx = LinkSum{a.column(x == 1, y)[0], a.column(x == 1, y)[1]};
        if (q.g.near_y()) q.ty = LinkSum{a.row(y == 1, q.x)[0], a.row(y == 1, q.x)[1]};
    }
    gather_view<Lay, R, RH, true>(n, blocks_at(src, tv.block), tv.v, q.g, q.qf, q.qg, q.qh);
    q.sr = ld_block<R>(blocks_at(sr_src + tv.flat_row, 0), 0, (uint32_t)((y - tv.yb) * tv.v.nx + q.x) * sizeof(R), 0);
}
// The update with `left` updates to follow it; true: the thread's node took part.
template <class Sh, typename R, typename RH>
LBM_HD bool deep_update(const TileView<R> &tv, const NodeConst<R, RH> &n, int left, DeepNode<R, RH> &q) {
    if (q.depth > left) return false;
    q.sr = (R)update_node<Sh::QT, R, RH, true>(q.walls, n, tv.edge, q.g, q.x, q.y, q.qf, q.qg, q.qh, q.sr,
                                              q.g.kind & NODE_OWNED, NodeTally{q.tx, q.ty}, q.th, q.m);
    return true;
}
// After a barrier, thread t's populations to its slot; after another, the
// pulls of the next update, which `left` updates follow.
template <class Sh, typename R, typename RH>
LBM_HD void deep_put(const NodeConst<R, RH> &n, void *lds_q, int t, const DeepNode<R, RH> &q) {
    Sh::Codec::put_node(lds_q, Sh::NSLOT, t, n, q.qf, q.qg, q.qh, q.m.drho, n.cf_base * (q.th.Tf - n.Tf_ref),
                        n.cm_base * q.m.dTm);
}
template <class Sh, typename R, typename RH>
LBM_HD void deep_pull(const NodeConst<R, RH> &n, const void *lds_q, int left, DeepNode<R, RH> &q) {
    if (q.depth <= left) lds_gather<Sh, R, RH>(n, q.from, lds_q, q.qf, q.qg, q.qh);
}
// The tile's own nodes to global memory.
template <class Sh, class Lay, typename R, typename RH>
LBM_HD void deep_store(const TileView<R> &tv, const NodeConst<R, RH> &n, void *dst, R *__restrict__ sr_dst,
                       double *__restrict__ acc, const DeepNode<R, RH> &q) {
    if (q.depth != 0) return;
    const CavityConst<R> &c = tv.c;
    const NodeRef k = place_of(tv.v, q.x, q.y);
    const Blocks b = blocks_at(dst, tv.block);
    Lay::template put<R>(b, tv.v.stride, 0, q.qf, q.m.drho, k, n);
    Lay::template put<RH>(b, tv.v.stride, 1, q.qg, n.cf_base * (q.th.Tf - n.Tf_ref), k, n);
    Lay::template put<R>(b, tv.v.stride, 2, q.qh, n.cm_base * q.m.dTm, k, n);
    *(R *)((char *)(sr_dst + tv.flat_row) + (uint32_t)((q.y - tv.yb) * tv.v.nx + q.x) * (uint32_t)sizeof(R)) = q.sr;
    if (tv.edge) {
        const CavityTally<double, R> a{acc, c};
        if (q.g.near_x()) a.column(q.x == 1, q.y)[0] = q.tx.E, a.column(q.x == 1, q.y)[1] = q.tx.M;
        if (q.g.near_y()) a.row(q.y == 1, q.x)[0] = q.ty.E, a.row(q.y == 1, q.x)[1] = q.ty.M;
    }
}

// Macroscopic fields of one node (post-streaming state) plus its
// contributions to the diagnostics partial sums.
template <class Lay, typename R, typename RH>
LBM_HD void macro_node(const CavityConst<R> &c, const void *src, bool raw, int x, int y, double out[6],
                       double v[NPART]) {
    const int nx = c.nx, ny = c.ny;
    const NodeGeom g = geometry(c, x, y, !raw);
    R qf[9], qh[9];
    RH qg[9];
    if (raw) gather<Lay, R, RH, false>(c, src, g, x, y, qf, qg, qh);
    else gather<Lay, R, RH, true>(c, src, g, x, y, qf, qg, qh);
    bool finite = true;
#pragma unroll
    for (int i = 0; i < 9; ++i)
        finite = finite && isfinite(qf[i]) && (i >= Lay::QT || (isfinite(qg[i]) && isfinite(qh[i])));
    // inflow of the last step through the wall links (not yet tallied)
    if (!raw && !g.wall()) {
#pragma unroll
        for (int i = 1; i < 9; ++i) {
            const int px = x - ex_of(i), py = y - ey_of(i);
            const bool onx = !c.periodic && (px == 0 || px == nx - 1);
            const bool ony = (py == 0 || py == ny - 1);
            if (onx || ony) {
                const int w = onx ? (px == 0 ? W_LEFT : W_RIGHT) : (py == 0 ? W_BOTTOM : W_TOP);
                double e, mm;
                link_content<Lay::QT>(c, i, qf, qg, qh, e, mm);
                v[P_INE0] += w == 0 ? e : 0.0;
                v[P_INE1] += w == 1 ? e : 0.0;
                v[P_INE2] += w == 2 ? e : 0.0;
                v[P_INE3] += w == 3 ? e : 0.0;
                v[P_INM0] += w == 0 ? mm : 0.0;
                v[P_INM1] += w == 1 ? mm : 0.0;
                v[P_INM2] += w == 2 ? mm : 0.0;
                v[P_INM3] += w == 3 ? mm : 0.0;
            }
        }
    }
    const NodeConst<R, RH> &n = node_const_of<RH>(c);
    if (!raw && g.wall()) reconstruct_wall<Lay::QT>(wall_node<RH>(c, x, y), n, qf, qg, qh);
    double sg = 0.0, sh = 0.0, sf = 0.0;
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        if (i < Lay::QT) {
            sg += c.g_ref[i] + (double)qg[i];
            sh += c.h_ref[i] + (double)qh[i];
        }
        sf += (double)w_of<double>(i) + (double)qf[i];
    }
    Thermo<RH> th;
    Macro<R> m;
    macros<Lay::QT>(n, qf, qg, qh, th, m);
    out[0] = (double)m.ux;
    out[1] = (double)m.uy;
    out[2] = (double)th.Tf;
    out[3] = (double)m.Tm;
    out[4] = (double)th.fl;
    out[5] = (double)m.rho;
    if (!finite) v[P_NF] = 1.0;
    if (!g.wall()) {
        v[P_FL] = (double)th.fl;
        // phi rho_l H + (1-phi) rho_m c_pm T_m and rho, from the offsets
        v[P_E] = c.we * sg + c.wm * sh;
        v[P_M] = sf;
        v[P_DT] = fabs((double)th.Tf - (double)m.Tm);
        v[P_U] = sqrt((double)m.ux * (double)m.ux + (double)m.uy * (double)m.uy);
    }
}

// Initial state of one node: equilibria at rest (Eqs. 27, 40, 49) at the
// given temperatures, stored as offsets; the previous-step source equals the
// current one.
template <class Lay, typename R, typename RH>
LBM_HD void init_node(const CavityConst<R> &c, void *dst, R *sr, int x, int y, double Tf, double Tm) {
    const ThermalConst<double> &t = c.td;
    const int nx = c.nx;
    const bool wall = (!c.periodic && (x == 0 || x == nx - 1)) || y == 0 || y == c.ny - 1;
    const int w = wall ? thermal_wall(c, x, y) : -1;
    if (w >= 0) Tf = Tm = t.T_wall[w];
    // inverse of Eq. (38) (a tie at the solidus goes to the solid branch)
    double H;
    if (Tf <= t.T_fs) H = Tf;
    else if (Tf >= t.T_fl) H = (Tf - t.T_fl) + t.H_fl;
    else H = t.H_fs + (Tf - t.T_fs) / (t.T_fl - t.T_fs) * (t.H_fl - t.H_fs);
    const double dT = Tf - t.T_ref, dTm = Tm - t.T_ref;
    const double dH = H - t.H_ref;
    const double cf = t.c_fref, cm = c.c_mref;
    // equilibria at rest, Eqs. (40), (49) / Eqs. (B3), (B5): the moving
    // weights are w_i (D2Q9) or varpi/4 (D2Q5), the rest one takes the rest
    const int QT = Lay::QT;
    const double wrest = QT == 9 ? 5.0 / 9.0 : t.varpi;
    R qf[9], qh[9];
    RH qg[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        const double wi = QT == 9 ? w_of<double>(i) : 0.25 * t.varpi;
        qf[i] = R(0);
        qg[i] = (RH)(i == 0 ? dH - wrest * cf * dT : wi * cf * dT);
        qh[i] = (R)(i == 0 ? (1.0 - wrest * cm) * dTm : wi * cm * dTm);
    }
    const FarRef k = any_band(c)(x, y);
    void *blk = band_block(c, dst, 0);
    const int64_t stride = c.band_nodes;
    Lay::template store<R>(blk, stride, 0, qf, R(0), k, c);
    Lay::template store<RH>(blk, stride, 1, qg, (RH)(cf * dT), k, c);
    Lay::template store<R>(blk, stride, 2, qh, (R)(cm * dTm), k, c);
    sr[flat_index(c, x, y)] = (R)(c.hv_f * (Tm - Tf));
}

}  // namespace lbm
