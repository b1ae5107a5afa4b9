// An fp32 number as the exact sum of three bf16 numbers, for products formed by bf16 matrix instructions.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace mi3d {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;

// Magnitudes for which the products of the parts stand for the product: zero and 2^-100 ... 2^45.  Below, the third part loses
// bits (bf16 ends at 2^-133; the matrix instructions keep subnormal operands and results).  Above, products could overflow:
// those of the parts have signs of their own, and inf - inf is NaN where the fp32 instruction gives an infinity.  Up to 2^45 a
// sum of 2^31 products stays below 2^121: nothing formed from parts ever overflows.
// Zero counts as large in the minimum (0 - 1 wraps).
struct SplitRange {
    uint32_t most = 0, least = 0xFFFFFFFFu;
    __device__ __forceinline__ void add(float v) {
        const uint32_t u = __builtin_bit_cast(uint32_t, v) & 0x7FFFFFFFu;
        most = u > most ? u : most;
        least = u - 1 < least ? u - 1 : least;
    }
    __device__ __forceinline__ void add2(float x, float y) { add(x); add(y); }
    __device__ __forceinline__ void add(const float4& v) { add2(v.x, v.y); add2(v.z, v.w); }
    __device__ __forceinline__ bool exceeded() const { return (most >= 0x56000000u) | (least < 0x0D7FFFFFu); }
};

// The same for values whose NaN may pass (the parts of a NaN are NaN, and so is every sum they enter): half the instructions.
struct SplitRangeNumbers {
    float most = 0.f;
    uint32_t least = 0xFFFFFFFFu;
    __device__ __forceinline__ void add2(float x, float y) {
        most = __builtin_fmaxf(__builtin_fmaxf(__builtin_fabsf(x), __builtin_fabsf(y)), most);
        const uint32_t u = (__builtin_bit_cast(uint32_t, x) << 1) - 1, v = (__builtin_bit_cast(uint32_t, y) << 1) - 1;
        const uint32_t m = u < v ? u : v;
        least = m < least ? m : least;
    }
    __device__ __forceinline__ void add(const float4& v) { add2(v.x, v.y); add2(v.z, v.w); }
    __device__ __forceinline__ bool exceeded() const { return (most >= 0x1p45f) | (least < 0x1AFFFFFFu); }
};

__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
    typedef __attribute__((__vector_size__(2 * sizeof(float)))) float f32x2;
    typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
    f32x2 v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

// the three parts of two values, packed
__device__ __forceinline__ void split2(float x, float y, uint32_t (&o)[3]) {
#pragma unroll
    for (int p = 0; p < 3; ++p) {
        o[p] = pack_bf16(x, y);
        x -= __builtin_bit_cast(float, o[p] << 16);
        y -= __builtin_bit_cast(float, o[p] & 0xFFFF0000u);
    }
}

}  // namespace mi3d
