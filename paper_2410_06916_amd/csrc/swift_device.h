// Device-side helpers shared by the kernel files.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace swift {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));  // one 128-bit load
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x8 __attribute__((ext_vector_type(8)));

// Eight probabilities as two bf16 terms (relative error 2^-17), converted in pairs.
__device__ inline void split2(const f32x8 &p, bf16x8 &hi, bf16x8 &lo) {
    hi = __builtin_convertvector(p, bf16x8);
    lo = __builtin_convertvector(p - __builtin_convertvector(hi, f32x8), bf16x8);
}

// fp32 -> bf16 bits, round to nearest even (NaN stays NaN)
__device__ inline uint16_t f32_to_bf16_rne(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
// same for finite inputs only: the hardware's conversion (v_cvt_pk_bf16_f32), one instruction instead of four
__device__ inline uint32_t f32_to_bf16_rne_finite(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }

// v = hi + mid + lo exactly (three bf16 terms carry the 24-bit significand of an fp32 value)
__device__ inline void split3(float v, uint16_t &hi, uint16_t &mid, uint16_t &lo) {
    const uint32_t h = f32_to_bf16_rne_finite(v);
    const float r1 = v - __uint_as_float(h << 16);
    const uint32_t m = f32_to_bf16_rne_finite(r1);
    const float r2 = r1 - __uint_as_float(m << 16);
    hi = (uint16_t)h;
    mid = (uint16_t)m;
    lo = (uint16_t)f32_to_bf16_rne_finite(r2);
}

// The same for a product a * b: what is left after hi comes from the unrounded product (spelt out, so that it is the same in every
// kernel), so that the three terms are within 2^-26 of that, and need not add up to the fp32 value of a * b.
__device__ inline void split3(float a, float b, uint16_t &hi, uint16_t &mid, uint16_t &lo) {
    const uint32_t h = f32_to_bf16_rne_finite(a * b);
    const float r1 = fmaf(a, b, -__uint_as_float(h << 16));
    const uint32_t m = f32_to_bf16_rne_finite(r1);
    const float r2 = r1 - __uint_as_float(m << 16);
    hi = (uint16_t)h;
    mid = (uint16_t)m;
    lo = (uint16_t)f32_to_bf16_rne_finite(r2);
}

// Exchanges the odd 16-lane rows of a with the even ones of b.
__device__ inline void swap16(uint32_t &a, uint32_t &b) {
    const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
    a = r[0];
    b = r[1];
}
// Lanes kg and kg ^ 1 hold values 0..3 and 4..7 of two eight-value units (x, y: two packed words each): afterwards the
// lane with the even kg holds all of x, the other one all of y.
__device__ inline u32x4 join8(uint32_t x0, uint32_t x1, uint32_t y0, uint32_t y1) {
    swap16(x0, y0);
    swap16(x1, y1);
    return u32x4{x0, x1, y0, y1};
}
__device__ inline uint32_t pack2(uint32_t lo, uint32_t hi) { return lo | (hi << 16); }

// Workgroup barrier that orders LDS traffic only.  __syncthreads() also waits for every global
// load and store of the wavefront (its release fence covers global memory), which would drain a
// window of weight loads that is deliberately kept in flight across the barrier.
__device__ inline void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// The type of a kernel's last argument and the byte where it lies among them all: each at the next multiple of its alignment.
template <typename F>
struct KernelArgs;
template <typename... A>
struct KernelArgs<void (*)(A...)> {
    static constexpr int last_at() {
        size_t at = 0, last = 0;
        ((last = (at + alignof(A) - 1) / alignof(A) * alignof(A), at = last + sizeof(A)), ...);
        return (int)last;
    }
    template <typename... T>
    struct Last;
    template <typename T>
    struct Last<T> {
        using type = T;
    };
    template <typename T, typename... R>
    struct Last<T, R...> : Last<R...> {};
    using last = typename Last<A...>::type;
};
static_assert(KernelArgs<void (*)(char *, int, char, int, double)>::last_at() == 24, "");

// The struct that is the last argument of kernel F (a pointer type), through a pointer the compiler cannot see behind: its fields are
// read where they are used, and what the kernel does before waits for none of them.
template <typename F>
__device__ inline const typename KernelArgs<F>::last &late_args() {
    using A = typename KernelArgs<F>::last;
    auto p = (const __attribute__((address_space(4))) char *)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return *(const A *)(const __attribute__((address_space(4))) A *)(p + KernelArgs<F>::last_at());
}

// Copies 4 or 16 bytes per lane from global memory straight to LDS: lane l's go to byte BYTES * l of dst (wavefront-uniform).
// NT: non-temporal.  Waiting for it (vmcnt) is the caller's business.
template <int BYTES, bool NT = false>
__device__ inline void to_lds(const void *src, void *dst) {
    const auto from = (const __attribute__((address_space(1))) void *)src;
    const auto to = (__attribute__((address_space(3))) void *)dst;
    if constexpr (BYTES == 4) {
        __builtin_amdgcn_global_load_lds(from, to, 4, 0, 0);
    } else if constexpr (NT) {
        __builtin_amdgcn_global_load_lds(from, to, 16, 0, 2);
    } else {
        __builtin_amdgcn_global_load_lds(from, to, 16, 0, 0);
    }
}

// Keeps a loaded word that nobody uses from being optimised away (and is where it is waited for).
__device__ inline void keep_alive(uint32_t w) { asm volatile("" ::"v"(w)); }

struct F32T {
    static constexpr int VEC = 4;  // elements per 16-byte load
    using elem = float;
    __device__ static void unpack(const u32x4 &v, float *f) {
        f[0] = __uint_as_float(v.x);
        f[1] = __uint_as_float(v.y);
        f[2] = __uint_as_float(v.z);
        f[3] = __uint_as_float(v.w);
    }
    __device__ static float load1(const elem *p) { return *p; }
    __device__ static void store1(elem *p, float f) { *p = f; }
};

struct BF16T {
    static constexpr int VEC = 8;
    using elem = uint16_t;
    __device__ static void unpack(const u32x4 &v, float *f) {
        f[0] = __uint_as_float(v.x << 16);
        f[1] = __uint_as_float(v.x & 0xffff0000u);
        f[2] = __uint_as_float(v.y << 16);
        f[3] = __uint_as_float(v.y & 0xffff0000u);
        f[4] = __uint_as_float(v.z << 16);
        f[5] = __uint_as_float(v.z & 0xffff0000u);
        f[6] = __uint_as_float(v.w << 16);
        f[7] = __uint_as_float(v.w & 0xffff0000u);
    }
    __device__ static float load1(const elem *p) { return __uint_as_float((uint32_t)(*p) << 16); }
    __device__ static void store1(elem *p, float f) { *p = f32_to_bf16_rne(f); }
};

// All-lane reductions over a wavefront (all 64 lanes active), in the order of an exchange with lane ^ 32, ^ 16, ^ 8, ^ 4, ^ 2, ^ 1, with
// register exchanges instead of trips through LDS (about 50 clocks against 700).  Rotating a row of 16 by 8 is ^ 8; by 4 it is
// ^ 4 once lanes l and l ^ 8 agree, as they do by then.
template <int CTRL>
__device__ inline float dpp_move(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}
template <typename Op>
__device__ inline float wave_reduce(float v, Op op) {
    const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = op(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = op(__uint_as_float(b[0]), __uint_as_float(b[1]));
    v = op(v, dpp_move<0x128>(v));   // row_ror:8
    v = op(v, dpp_move<0x124>(v));   // row_ror:4
    v = op(v, dpp_move<0x4E>(v));    // quad_perm [2,3,0,1]
    return op(v, dpp_move<0xB1>(v)); // quad_perm [1,0,3,2]
}
// The lanes of one matrix column (l, l ^ 16, l ^ 32, l ^ 48), in the order of an exchange with lane ^ 16, ^ 32.
template <typename Op>
__device__ inline float column_reduce(float v, Op op) {
    const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = op(__uint_as_float(b[0]), __uint_as_float(b[1]));
    const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return op(__uint_as_float(a[0]), __uint_as_float(a[1]));
}
__device__ inline float wave_sum(float v) {
    return wave_reduce(v, [](float x, float y) { return x + y; });
}
// The sum of v^2 over a row of 16 lanes, in the row's first lane: that lane's sum of an exchange with lane ^ 8, ^ 4, ^ 2, ^ 1 (one
// rounding in the first sum: a fused multiply-add, spelt out so that it is the same in every kernel; for lanes 0 to 3, rotating
// by 12 is ^ 4).
__device__ inline float row_sum_of_squares(float v) {
    float s = fmaf(v, v, dpp_move<0x128>(v * v));
    s += dpp_move<0x12C>(s);
    s += dpp_move<0x4E>(s);
    return s + dpp_move<0xB1>(s);
}
__device__ inline float wave_max(float v) {
    return wave_reduce(v, [](float x, float y) { return fmaxf(x, y); });
}
// The smallest of the lanes' non-negative integers.
__device__ inline int wave_min(int v) {
    return __float_as_int(wave_reduce(__int_as_float(v), [](float x, float y) {
        return __int_as_float(min(__float_as_int(x), __float_as_int(y)));
    }));
}

}  // namespace swift
