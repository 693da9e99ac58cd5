// Shared device-side types and small helpers for the gfx950 kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

typedef __bf16 bf16;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;

#define RS_DEVICE static __device__ __forceinline__
#define RS_INLINE __attribute__((always_inline))   // on lambdas whose captures must stay in registers

constexpr int WAVE = 64;

RS_DEVICE float bf16_to_f32(bf16 v) { return (float)v; }
RS_DEVICE bf16 f32_to_bf16(float v) { return (bf16)v; }   // round-to-nearest-even (v_cvt_pk_bf16_f32)

RS_DEVICE float wave_sum(float v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, WAVE);
    return v;
}

// 16-byte global / LDS accessors on raw byte pointers.
RS_DEVICE uint4 ld_global_16(const void* p) { return *reinterpret_cast<const uint4*>(p); }
RS_DEVICE void st_global_16(void* p, uint4 v) { *reinterpret_cast<uint4*>(p) = v; }

RS_DEVICE void st_global_16_stream(void* p, uint4 v) {   // (for what the launch does not read again)
    typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;
    __builtin_nontemporal_store(__builtin_bit_cast(u32x4_t, v), reinterpret_cast<u32x4_t*>(p));
}

RS_DEVICE bf16x8 as_bf16x8(uint4 v) { return __builtin_bit_cast(bf16x8, v); }
RS_DEVICE uint4 as_uint4(bf16x8 v) { return __builtin_bit_cast(uint4, v); }

template <int I, int N, class F>
RS_DEVICE void static_for(F&& f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(f);
    }
}

// 8 elements in one access when the pointer is aligned for it (`wide`), else one by one.
template <class T> struct Pack8;   // 8 elements
template <> struct Pack8<bf16> { typedef uint4 type; };
template <> struct Pack8<uint8_t> { typedef uint2 type; };

template <class T>
RS_DEVICE typename Pack8<T>::type load8(const T* p, bool wide) {
    typedef typename Pack8<T>::type P;
    if (wide) return *reinterpret_cast<const P*>(p);
    union { T e[8]; P v; } u;
#pragma unroll
    for (int i = 0; i < 8; ++i) u.e[i] = p[i];
    return u.v;
}
template <class T>
RS_DEVICE void store8(T* p, typename Pack8<T>::type v, bool wide) {
    typedef typename Pack8<T>::type P;
    if (wide) {
        *reinterpret_cast<P*>(p) = v;
        return;
    }
    union { T e[8]; P v; } u;
    u.v = v;
#pragma unroll
    for (int i = 0; i < 8; ++i) p[i] = u.e[i];
}
