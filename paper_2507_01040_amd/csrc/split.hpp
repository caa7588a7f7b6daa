// An fp32 value as the sum of three bf16 parts, shared by the kernels that
// multiply on the bf16 matrix cores: h = bf16(v), m = bf16(v - h), l = bf16(v -
// h - m), rounded to nearest, hold all 24 bits (the three-way split of fp32
// products on bf16 units: Henry, Tang, Heinecke, ARITH 2019).  Of the nine
// products of two values' parts six are taken; the others are below 2^-24 of the
// product.
//
// v is 2^16 times the operand: the smallest bf16 step is 2^-133, so the parts of
// operands below 2^-110 would lose bits (relative error 9e-6 at 2^-118, 6e-4 at
// 2^-124), and 2^16 times the smallest float still is a bf16 value.  Operands
// from 2^112 and sums from 2^96 on come out infinite and are computed again in
// fp32, as infinities are.
#pragma once

#include <stdint.h>

#include "common.hpp"

namespace cliff {

constexpr float SPLIT_SCALE = 0x1p16f;    // of an operand
constexpr float SPLIT_UNSCALE = 0x1p-32f;  // of a sum of products

// The bf16 parts of two floats times SPLIT_SCALE, packed (a in the low half).
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
    a *= SPLIT_SCALE;
    b *= SPLIT_SCALE;
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
