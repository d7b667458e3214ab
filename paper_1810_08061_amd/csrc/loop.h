// loop.h -- what the forward loop kernels share: the loop modes, the operand
// elements they exchange between workgroups, and their K order.
#pragma once

#include "launch.h"

namespace ldyn {

// What a variant of the loop does besides the plain forward.
enum LoopMode { LM_PLAIN = 0, LM_STOP = 1, LM_SAVE = 2 };

constexpr int P_SC1 = 16;               // buffer-instruction cache policy: device scope

__device__ inline void drain_stores() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Data written before this kernel started and only read by it, seen through
// the constant address space: wave-uniform reads of it become scalar loads,
// which do not queue behind the vector loads in flight.
typedef const __attribute__((address_space(4))) int32_t const_i32;

// Loads of the operand buffer through a buffer resource, at device scope.
// An operand slot whose value for the coming step has not arrived yet holds
// the all-ones pattern (a NaN).  operand() never produces it: a NaN h that
// would convert to it is stored as the canonical quiet NaN instead.
// store<POLICY>: the cache policy of the store (P_SC1 device scope, 0 the
// writer's L2).
template <typename E> struct HxIO;
// 16-bit operands (bf16 or fp16): T the element, V eight of them, QNAN the
// canonical quiet NaN's bits.
template <typename T, typename V, unsigned short QNAN> struct HxIO16 {
    __device__ static inline V load(__amdgpu_buffer_rsrc_t R, unsigned byte_off) {
        typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
        const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(R, byte_off, 0, P_SC1);
        return __builtin_bit_cast(V, v);
    }
    __device__ static inline T operand(float h) {
        const unsigned short b = __builtin_bit_cast(unsigned short, (T)h);
        return __builtin_bit_cast(T, b == 0xffffu ? QNAN : b);
    }
    template <int POLICY = P_SC1>
    __device__ static inline void store(__amdgpu_buffer_rsrc_t R, unsigned byte_off, float h) {
        __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(unsigned short, operand(h)), R, byte_off, 0,
                                              POLICY);
    }
    template <int POLICY>
    __device__ static inline void mark(__amdgpu_buffer_rsrc_t R, unsigned byte_off) {
        __builtin_amdgcn_raw_buffer_store_b16((unsigned short)0xffffu, R, byte_off, 0, POLICY);
    }
    // true if any of the KSW fragments holds the marker in one of its elements
    template <int KSW>
    __device__ static inline bool has_marker(const V* f) {
        typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
        typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
        u16x2 m = {0, 0};
#pragma unroll
        for (int ks = 0; ks < KSW; ++ks) {
            const u32x4 v = __builtin_bit_cast(u32x4, f[ks]);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const unsigned d = v[j];  // (a bit_cast of the subscript itself reads element 0)
                m = __builtin_elementwise_max(m, __builtin_bit_cast(u16x2, d));
            }
        }
        return m[0] == 0xffffu || m[1] == 0xffffu;
    }
};
template <> struct HxIO<EltH16> : HxIO16<_Float16, f16x8_t, 0x7e00> {};

template <> struct HxIO<EltF32> {
    __device__ static inline float load(__amdgpu_buffer_rsrc_t R, unsigned byte_off) {
        return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(R, byte_off, 0, P_SC1));
    }
    __device__ static inline float operand(float h) {
        const unsigned b = __float_as_uint(h);
        return __uint_as_float(b == 0xffffffffu ? 0x7fc00000u : b);
    }
    template <int POLICY = P_SC1>
    __device__ static inline void store(__amdgpu_buffer_rsrc_t R, unsigned byte_off, float h) {
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(operand(h)), R, byte_off, 0, POLICY);
    }
    template <int POLICY>
    __device__ static inline void mark(__amdgpu_buffer_rsrc_t R, unsigned byte_off) {
        __builtin_amdgcn_raw_buffer_store_b32(~0u, R, byte_off, 0, POLICY);
    }
    template <int KSW>
    __device__ static inline bool has_marker(const float* f) {
        unsigned m = 0;
#pragma unroll
        for (int ks = 0; ks < KSW; ++ks) m = max(m, __float_as_uint(f[ks]));
        return m == 0xffffffffu;
    }
};

// K index (relative to the wave's K range) of the first value lane l holds for
// MFMA K-step ks.  bf16: 8 consecutive k per lane per step.  fp32 with at
// least four steps: each lane holds 4 consecutive k for a group of four
// steps (one 16-byte load feeds four MFMAs); the A- and B-fragments use the
// same assignment, so the sum over k is unchanged.
template <typename E, int KSW>
__device__ inline int kslot(int ks, int l) {
    if constexpr (E::KPL == 1 && KSW >= 4) return 16 * (ks >> 2) + 4 * (l >> 4) + (ks & 3);
    else return ks * E::KSTEP + (l >> 4) * E::KPL;
}

// Workgroup barrier after this wave's LDS accesses; loads and stores in flight
// stay in flight.
__device__ inline void x_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Products of at most four rows, fp32.  MFMA 4x4x1 forms sixteen 4 x 4 blocks at
// once, block l >> 2 of lane l; with the fragments of a 16x16x4 MFMA (lane l:
// column l & 15 of U, k run l >> 4) and row l & 3 of h in lane l, block 4 q + c is
// columns 4 c .. 4 c + 3 of run q.  It takes 8 cycles where 16x16x4, four fifths
// of it for rows that are not there, takes 32.  sum_runs adds the four runs.
__device__ inline f32x4_t mfma_few(float a, float b, f32x4_t c) {
    return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, 0, 0, 0);
}
__device__ inline f32x4_t sum_runs(f32x4_t v) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        // swapping a value's halves (then odd and even quarters) with itself
        // leaves one copy of each beside the other in every lane
        unsigned x = __float_as_uint(v[e]);
        const auto h = __builtin_amdgcn_permlane32_swap(x, x, false, false);
        x = __float_as_uint(__uint_as_float(h[0]) + __uint_as_float(h[1]));
        const auto q = __builtin_amdgcn_permlane16_swap(x, x, false, false);
        v[e] = __uint_as_float(q[0]) + __uint_as_float(q[1]);
    }
    return v;
}

}  // namespace ldyn
