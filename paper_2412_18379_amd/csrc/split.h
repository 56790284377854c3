// FP32 products on the BF16 matrix cores.
//
// An FP32 value is the sum of three BF16 values, x = x_h + x_m + x_l: x_h is x rounded to BF16's
// eight significant bits, x_m the remainder rounded again, and what is left after that has at most
// eight bits, so x_l holds it exactly.  Of the nine products of two such triples six are issued:
//   x y = x_h y_h + (x_h y_m + x_m y_h) + (x_m y_m + x_h y_l + x_l y_h);
// the three left out are below 2^-24 of x y, a quarter of an FP32 rounding on average.  Six BF16
// matrix instructions of K = 32 take 96 cycles where eight FP32 ones of K = 4 take 256.
//
// The order matters for the result's accuracy, because the matrix instruction rounds its
// accumulator once per instruction: the five small products are summed by themselves and only
// x_h y_h goes into the running sum, which then is rounded twice per 32 inputs (the FP32
// instruction rounds it eight times).  288-input dot products of normal operands: relative error
// 0.74e-7 in this order, 2.4e-7 with all six products in one running sum, 2.2e-7 with the FP32
// instruction.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace cnnsns {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Eight FP32 values as three BF16 octets.
struct Split8 {
    bf16x8 h, m, l;
};

__device__ __forceinline__ uint32_t bf16_pair(float a, float b)
{
    bf16x2 p;
    p[0] = (__bf16)a;
    p[1] = (__bf16)b;
    return __builtin_bit_cast(uint32_t, p);
}

constexpr uint32_t kBf16Top = 0x7f7f0000u;  // BF16's largest finite value, 3.39e38, as FP32

// (a, b) as three packed BF16 pairs; the remainders are exact FP32 subtractions.  For values up to 3.39e38: an activation
// beyond is within 0.4 % of FP32's own end.
__device__ __forceinline__ void split_pair(float a, float b, uint32_t& h, uint32_t& m, uint32_t& l)
{
    h = bf16_pair(a, b);
    a -= __uint_as_float(h << 16);
    b -= __uint_as_float(h & 0xffff0000u);
    m = bf16_pair(a, b);
    a -= __uint_as_float(m << 16);
    b -= __uint_as_float(m & 0xffff0000u);
    l = bf16_pair(a, b);
}

// The same for any finite values, as the caller's are: those between BF16's largest value and FP32's, which rounding would
// take to infinity, are BF16's largest value and a remainder.
__device__ __forceinline__ void split_pair_any(float a, float b, uint32_t& h, uint32_t& m, uint32_t& l)
{
    const float top = __uint_as_float(kBf16Top);
    h = bf16_pair(__builtin_amdgcn_fmed3f(a, -top, top), __builtin_amdgcn_fmed3f(b, -top, top));
    a -= __uint_as_float(h << 16);
    b -= __uint_as_float(h & 0xffff0000u);
    m = bf16_pair(a, b);
    l = bf16_pair(a - __uint_as_float(m << 16), b - __uint_as_float(m & 0xffff0000u));
}

__device__ __forceinline__ Split8 split8(const v4f& a, const v4f& b)
{
    u32x4 h, m, l;
    uint32_t x, y, z;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const v4f& s = k < 2 ? a : b;
        split_pair(s[2 * (k & 1)], s[2 * (k & 1) + 1], x, y, z);
        h[k] = x;
        m[k] = y;
        l[k] = z;
    }
    return Split8{ __builtin_bit_cast(bf16x8, h), __builtin_bit_cast(bf16x8, m), __builtin_bit_cast(bf16x8, l) };
}

// One weight, prepared in FP64, as the `part`-th of its three BF16 values.
__device__ __forceinline__ __bf16 split_part(double x, int part)
{
    const float top = __uint_as_float(kBf16Top);
    const __bf16 h = (__bf16)__builtin_amdgcn_fmed3f((float)x, -top, top);
    if (part == 0) return h;
    const double r = x - (double)(float)h;
    const __bf16 m = (__bf16)(float)r;
    if (part == 1) return m;
    return (__bf16)(float)(r - (double)(float)m);
}

__device__ __forceinline__ v4f mfma_bf16(const bf16x8& a, const bf16x8& b, const v4f& c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

}  // namespace cnnsns
