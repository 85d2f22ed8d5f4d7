// Storage types and conversions used by every kernel (device side).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "record.h"

namespace mt {

typedef _Float16 f16;
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));   // 16-byte register chunk
struct bf16 {
    uint16_t v;
};

__device__ __forceinline__ float to_f32(float v) { return v; }
__device__ __forceinline__ float to_f32(f16 v) { return (float)v; }
__device__ __forceinline__ float to_f32(bf16 v) { return __uint_as_float(((uint32_t)v.v) << 16); }

__device__ __forceinline__ void from_f32(float f, float &o) { o = f; }
__device__ __forceinline__ void from_f32(float f, f16 &o) { o = (f16)f; }   // v_cvt_f16_f32: nearest even
__device__ __forceinline__ void from_f32(float f, bf16 &o) {
    o.v = __builtin_bit_cast(uint16_t, (__bf16)f);      // v_cvt_pk_bf16_f32: nearest even, NaN stays NaN
}

// Activation as a clamp to [lo, hi]: none = [-inf, inf], ReLU = [0, inf], ReLU6 = [0, 6]; the bounds depend only on
// the kernel argument, so the per-value cost is one v_med3_f32.
__device__ __forceinline__ float apply_act(float v, int act) {
    const float lo = act == MT_ACT_NONE ? -__builtin_inff() : 0.f;
    const float hi = act == MT_ACT_RELU6 ? 6.f : __builtin_inff();
    return __builtin_amdgcn_fmed3f(v, lo, hi);
}

// A workgroup's arguments: everything it needs before its first load is asked for in one go and held.  Read where they are first used, the
// arguments come in four or five trips through the scalar cache, one after the other, and a value that is only asked for early the compiler
// drops and reads again where registers are short (the several-operator and walking kernels made five or six trips that way).  In one trip, and
// with the divisors of TileWalk, a workgroup requests its first operands after 180 instructions instead of 600 (1.25 us, of which 0.35 the
// arguments).
template <typename V>
__device__ __forceinline__ void hold_one(V &v) {
    if constexpr (std::is_pointer_v<V>) {
        // As what it is, a pointer to global memory: loads through one of which the compiler does not know that are generic, which may
        // be to LDS as well, and it waits for all of them where it waits for one.
        auto g = (__attribute__((address_space(1))) std::remove_pointer_t<V> *)v;
        asm volatile("" : "+s"(g));
        v = (V)g;
    } else asm volatile("" : "+s"(v));
}
template <typename... V>
__device__ __forceinline__ void hold(V &...v) {
    __builtin_amdgcn_sched_barrier(0);                     // all of them are asked for before the first is waited for
    (hold_one(v), ...);
}

// Issue priority of the calling wave among the waves of its SIMD (0 lowest, 3 highest); the instruction takes an
// immediate, hence the ladder.  Changes timing only, never results.
__device__ __forceinline__ void set_wave_priority(int p) {
    if (p == 1) __builtin_amdgcn_s_setprio(1);
    else if (p == 2) __builtin_amdgcn_s_setprio(2);
    else if (p == 3) __builtin_amdgcn_s_setprio(3);
}

__device__ __forceinline__ uint32_t divide(uint32_t n, const Divisor &v) {
    const uint32_t t = __umulhi(v.m, n);
    return (t + ((n - t) >> v.s1)) >> v.s2;
}

// Launches K1 with the operator's arguments, or, when `mate` points to n_mates (1 .. 3) further operators of equal
// launch shape, K2 (the several-operator form of the same kernel) on a grid of 1 + n_mates times the workgroups,
// blockIdx.y naming the operator.
#define MT_LAUNCH(K1, K2, grid, block, st, a, mate, ...)                                    \
    do {                                                                                    \
        if (mate) {                                                                         \
            OpArgsPair pair_;                                                               \
            pair_.a[0] = (a);                                                               \
            for (int i_ = 0; i_ < n_mates; ++i_) pair_.a[1 + i_] = (mate)[i_];              \
            dim3 grid2_ = (grid);                                                           \
            grid2_.y = 1 + n_mates;                                                         \
            launch(K2, grid2_, block, 0, st, pair_ __VA_OPT__(, ) __VA_ARGS__);            \
        } else {                                                                            \
            launch(K1, grid, block, 0, st, a __VA_OPT__(, ) __VA_ARGS__);                 \
        }                                                                                   \
    } while (0)

// V consecutive elements of T moved as one access when V*sizeof(T) is 4, 8 or 16 bytes.
template <typename T, int V>
struct alignas(sizeof(T) * V) Pack {
    T e[V];
};

template <typename T, int V>
__device__ __forceinline__ void load_pack(const T *p, float (&out)[V]) {
    Pack<T, V> t = *reinterpret_cast<const Pack<T, V> *>(p);
#pragma unroll
    for (int i = 0; i < V; ++i) out[i] = to_f32(t.e[i]);
}

// Results go through the XCD's L2 to the memory that all XCDs share (sc1, device scope), and a wave ends when that memory has them
// (results_stored, at the end of every kernel).  A launch therefore has nothing to release when it ends: that release
// writes back whatever any tenant's kernels have left dirty in eight L2s, while the next launch of the chain waits.  us a pass, released / stored
// through: ResNet-18 at one image 103.7 / 98.4, ResNet-101, Inception-v3, MobileNetV2 and AlexNet together 500 / 458, Inception-v3 and AlexNet at
// batch 5 699 / 644, four networks at batch 8 887 / 857, ResNet-50 at batch 64 1325 / 1281, eight at batch 16 2561 / 2502.
constexpr int THROUGH = 16;
typedef __amdgpu_buffer_rsrc_t Results;
__device__ __forceinline__ Results results_in(void *y) {    // a tensor stays below 2^31 bytes
    return __builtin_amdgcn_make_buffer_rsrc(y, 0, (int)0x80000000u, 0x00027000);
}
__device__ __forceinline__ void results_stored() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// V values to elements at .. of a tensor of T, rounded once; at is a multiple of V.
template <typename T, int V>
__device__ __forceinline__ void store_pack(Results y, uint32_t at, const float (&in)[V]) {
    Pack<T, V> t;
#pragma unroll
    for (int i = 0; i < V; ++i) from_f32(in[i], t.e[i]);
    const uint32_t off = at * (uint32_t)sizeof(T);
    if constexpr (sizeof(t) == 2) __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(uint16_t, t), y, off, 0, THROUGH);
    else if constexpr (sizeof(t) == 4) __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, t), y, off, 0, THROUGH);
    else if constexpr (sizeof(t) == 8) __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, t), y, off, 0, THROUGH);
    else {
        static_assert(sizeof(t) % 16 == 0, "whole 16-byte pieces");
        struct Pieces { u32x4 p[sizeof(t) / 16]; };
        const Pieces q = __builtin_bit_cast(Pieces, t);
#pragma unroll
        for (int i = 0; i < (int)sizeof(t) / 16; ++i) __builtin_amdgcn_raw_buffer_store_b128(q.p[i], y, off + 16u * (uint32_t)i, 0, THROUGH);
    }
}
template <typename T>
__device__ __forceinline__ void store_one(Results y, uint32_t at, float v) {
    const float one[1] = {v};
    store_pack<T, 1>(y, at, one);
}

}  // namespace mt
