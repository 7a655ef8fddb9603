// FP32 operands as exact sums of three BF16 parts, and their product on the
// BF16 matrix cores (six products per term, FP32-accurate dot products).
#pragma once

#include <hip/hip_bf16.h>

#include "device_common.hpp"

namespace rpod {

typedef __bf16 e6_bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned short e6_u16x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ f32x4 mma_bf16(e6_u16x8 a, e6_u16x8 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(e6_bf16x8, a), __builtin_bit_cast(e6_bf16x8, b),
                                                   c, 0, 0, 0);
}

typedef float e6_f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 e6_bf16x2 __attribute__((ext_vector_type(2)));
typedef unsigned e6_u32x4 __attribute__((ext_vector_type(4)));

// Three-way split of two values; each result word packs the parts of a
// (low half) and b (high half). Rounding to nearest at every level.
__device__ __forceinline__ void split_pair(float a, float b, unsigned& h, unsigned& m, unsigned& l) {
    const e6_f32x2 x{a, b};
    h = __builtin_bit_cast(unsigned, __builtin_convertvector(x, e6_bf16x2));
    const e6_f32x2 r = x - e6_f32x2{__builtin_bit_cast(float, h << 16), __builtin_bit_cast(float, h & 0xffff0000u)};
    m = __builtin_bit_cast(unsigned, __builtin_convertvector(r, e6_bf16x2));
    const e6_f32x2 t = r - e6_f32x2{__builtin_bit_cast(float, m << 16), __builtin_bit_cast(float, m & 0xffff0000u)};
    l = __builtin_bit_cast(unsigned, __builtin_convertvector(t, e6_bf16x2));
}

// eight values (x0 then x1) -> the three BF16 operands
__device__ __forceinline__ void split8(f32x4 x0, f32x4 x1, e6_u16x8& ah, e6_u16x8& am, e6_u16x8& al) {
    e6_u32x4 h, m, l;
    unsigned a, b, c;
    split_pair(x0[0], x0[1], a, b, c); h[0] = a; m[0] = b; l[0] = c;
    split_pair(x0[2], x0[3], a, b, c); h[1] = a; m[1] = b; l[1] = c;
    split_pair(x1[0], x1[1], a, b, c); h[2] = a; m[2] = b; l[2] = c;
    split_pair(x1[2], x1[3], a, b, c); h[3] = a; m[3] = b; l[3] = c;
    ah = __builtin_bit_cast(e6_u16x8, h);
    am = __builtin_bit_cast(e6_u16x8, m);
    al = __builtin_bit_cast(e6_u16x8, l);
}

// acc += the six leading terms of (ah + am + al)(bh + bm + bl), small terms first
__device__ __forceinline__ void mma6(const e6_u16x8& ah, const e6_u16x8& am, const e6_u16x8& al, const e6_u16x8& bh,
                                     const e6_u16x8& bm, const e6_u16x8& bl, f32x4& acc) {
    f32x4 s = acc;
    s = mma_bf16(al, bh, s);
    s = mma_bf16(am, bm, s);
    s = mma_bf16(ah, bl, s);
    s = mma_bf16(am, bh, s);
    s = mma_bf16(ah, bm, s);
    acc = mma_bf16(ah, bh, s);
}

}  // namespace rpod
