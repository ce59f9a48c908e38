// split.h -- FP32 products on the bf16 matrix cores, as exact as FP32 ones: every FP32
// operand is the exact sum of three bf16 numbers, each rounded to nearest (h + m + l:
// 3 x 8 significant bits, |m| <= 2^-8 |h|, |l| <= 2^-17 |h|), and a product a b is
// summed from eight of the nine partial products, smallest first,
//   a b = ah bh + (ah bm + am bh) + (ah bl + am bm + al bh) + (am bl + al bm) + al bl;
// al bl, below 2^-34 a b, is left out.  The last addition rounds as an FP32 product
// does, the earlier ones round sums of at most 2^-7 a b.  (Without the two products of
// order 2^-25 the largest error of a product is 1.3 times an FP32 product's, with the
// vector's parts truncated instead of rounded 2.7 times.)  The bf16 matrix rate is
// sixteen times the FP32 one, so eight products cost half of the FP32 instruction's time.
//
// Sums run over the small products first and the ah bh last: the accumulator is
// then rounded at full size only once per 32-row step instead of once per 4 rows
// (K = 64: error 5.8e-8 of the result against 1.44e-7 for the FP32 instruction,
// both against 64 bits on random operands spread over three decades).
//
// The range: an infinity would split into NaN (inf - inf), an operand near the largest
// FP32 number round up to one, and a tiny one lose its m and l parts to the underflow of
// bf16.  Vector elements have to be zero or of magnitude [2^-100, 2^60) (parts down to
// 2^-125, still normal numbers), integrals zero or [2^-76, 2^60), so that a sum of
// integrals, a multiple of 2^-99, keeps to the vector's range or is zero.  The products
// of others are left to the FP32 instruction by the callers.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "mfma.h"

namespace cis {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

constexpr float kSplitMin = 0x1p-100f, kSplitMax = 0x1p60f;   // vector elements
constexpr float kSplitMinA = 0x1p-76f;                        // integrals

// neither zero nor in the vector's range (NaN: yes)
__device__ __forceinline__ bool split_wide(float x) {
    constexpr uint32_t LO = __builtin_bit_cast(uint32_t, kSplitMin), HI = __builtin_bit_cast(uint32_t, kSplitMax);
    const uint32_t u = __float_as_uint(x) & 0x7fffffffu;
    return u != 0 && u - LO >= HI - LO;
}

struct Split8 { bf16x8 h, m, l; };   // eight FP32 values: one lane's operand of a 32-row step

// D (16 x 16) += A (16 x 32) B (32 x 16): lane l holds A[l % 16][8 (l / 16) + j],
// B[8 (l / 16) + j][l % 16], D[4 (l / 16) + r][l % 16]
__device__ __forceinline__ floatx4 mfma_bf16(bf16x8 a, bf16x8 b, floatx4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// parts rounded to nearest, two values at a time (one conversion a pair)
__device__ __forceinline__ Split8 split_round(const float (&x)[8]) {
    typedef float floatx2 __attribute__((ext_vector_type(2)));
    u32x4_t h, m, l;
    auto pack = [](float a, float b) {
        return __builtin_bit_cast(uint32_t, __builtin_convertvector(floatx2{a, b}, bf16x2));
    };
    auto lo = [](uint32_t p) { return __uint_as_float(p << 16); };
    auto hi = [](uint32_t p) { return __uint_as_float(p & 0xffff0000u); };
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float a = x[2 * i], b = x[2 * i + 1];
        h[i] = pack(a, b);
        const float a1 = a - lo(h[i]), b1 = b - hi(h[i]);
        m[i] = pack(a1, b1);
        l[i] = pack(a1 - lo(m[i]), b1 - hi(m[i]));
    }
    Split8 s;
    s.h = __builtin_bit_cast(bf16x8, h);
    s.m = __builtin_bit_cast(bf16x8, m);
    s.l = __builtin_bit_cast(bf16x8, l);
    return s;
}

}  // namespace cis
