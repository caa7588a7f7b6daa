// An fp32 value as the sum of three bf16 parts, shared by the kernels that
// multiply on the bf16 matrix cores: h = bf16(v), m = bf16(v - h), l = bf16(v -
// h - m), rounded to nearest, hold all 24 bits.  Of the nine products of two
// values' parts six are taken; the others are below 2^-24 of the product.
#pragma once

#include <stdint.h>

#include "common.hpp"

namespace cliff {

// The bf16 parts of two floats, packed (a in the low half).
struct Parts {
    uint32_t t[3];
};
__device__ inline uint32_t pack_bf16(float a, float b)
{
    typedef float f2 __attribute__((ext_vector_type(2)));
    typedef __bf16 b2 __attribute__((ext_vector_type(2)));
    const f2 v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, b2));
}
__device__ inline Parts split2(float a, float b)
{
    Parts p;
    p.t[0] = pack_bf16(a, b);
    const float a1 = a - __builtin_bit_cast(float, p.t[0] << 16);
    const float b1 = b - __builtin_bit_cast(float, p.t[0] & 0xffff0000u);
    p.t[1] = pack_bf16(a1, b1);
    const float a2 = a1 - __builtin_bit_cast(float, p.t[1] << 16);
    const float b2_ = b1 - __builtin_bit_cast(float, p.t[1] & 0xffff0000u);
    p.t[2] = pack_bf16(a2, b2_);
    return p;
}

}  // namespace cliff
