// split.h -- FP32 products on the bf16 matrix cores, without loss: every FP32
// operand is the exact sum of three bf16 numbers (h + m + l: 3 x 8 significant
// bits), and a product a b is summed from the six partial products that reach
// the last bits of an FP32 result,
//   a b = ah bh + (ah bm + am bh) + (ah bl + am bm + al bh) + O(2^-24 a b).
// The bf16 matrix rate is sixteen times the FP32 one, so six products cost 3/8
// of the FP32 instruction's time.
//
// The kernels split one operand once (the integrals: rounded to nearest, so its m
// and l parts have either sign and the dropped products average out) and the
// other per use (the vector: truncated, which is one byte permute per pair).
// Sums run over the small products first and the ah bh last: the accumulator is
// then rounded at full size only once per 32-row step instead of once per 4 rows
// (K = 64: error 5.8e-8 of the result against 1.44e-7 for the FP32 instruction,
// both against 64 bits on random operands spread over three decades).
//
// Infinities: inf - inf in the split makes them NaN; NaN stays NaN.  Operands
// below 2^-110 lose their m and l parts to the underflow of bf16.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "mfma.h"

namespace cis {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

struct Split8 { bf16x8 h, m, l; };   // eight FP32 values: one lane's operand of a 32-row step

// D (16 x 16) += A (16 x 32) B (32 x 16): lane l holds A[l % 16][8 (l / 16) + j],
// B[8 (l / 16) + j][l % 16], D[4 (l / 16) + r][l % 16]
__device__ __forceinline__ floatx4 mfma_bf16(bf16x8 a, bf16x8 b, floatx4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// parts rounded to nearest
__device__ __forceinline__ Split8 split_round(const float (&x)[8]) {
    Split8 s;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        s.h[j] = __bf16(x[j]);
        const float r = x[j] - float(s.h[j]);
        s.m[j] = __bf16(r);
        s.l[j] = __bf16(r - float(s.m[j]));
    }
    return s;
}

// parts truncated: the high halves of a pair by one byte permute, x - h by a mask
// and a subtraction (exact).  (A dot product with -1 does the latter in one
// instruction, but runs on the matrix unit: between bf16 products it costs eight
// cycles, a mask and a subtraction six.)
__device__ __forceinline__ Split8 split_trunc(const float (&x)[8]) {
    u32x4_t h, m, l;
    auto rest = [](float v) { return v - __uint_as_float(__float_as_uint(v) & 0xffff0000u); };
    auto pack = [](float a, float b) {
        return __builtin_amdgcn_perm(__float_as_uint(b), __float_as_uint(a), 0x07060302u);
    };
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float a = x[2 * i], b = x[2 * i + 1];
        const float a1 = rest(a), b1 = rest(b);
        h[i] = pack(a, b);
        m[i] = pack(a1, b1);
        l[i] = pack(rest(a1), rest(b1));
    }
    Split8 s;
    s.h = __builtin_bit_cast(bf16x8, h);
    s.m = __builtin_bit_cast(bf16x8, m);
    s.l = __builtin_bit_cast(bf16x8, l);
    return s;
}

}  // namespace cis
