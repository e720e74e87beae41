// fp32 products on the bf16 matrix units without loss of precision.
//
// An fp32 value is the exact sum of three bf16 values (Henry, Tang and Heinecke, "Leveraging the bfloat16 Artificial
// Intelligence Datatype For Higher-Precision Computations", ARITH 2019): x = h + m + l, h = bf16(x), m = bf16(x - h),
// l = x - h - m (8 + 8 + 8 significant bits; both differences are exact in fp32).  Of the nine products of two such
// values six are formed, each exact (8 x 8 bits) and accumulated in fp32 by v_mfma_f32_32x32x16_bf16: h h, h m, m h, m m,
// h l, l h.  What is left out, m l + l m + l l, is at most 2^-24 of the product, half a unit in its last place (reached by
// two operands 1 + 2^-8 - 2^-17), and 2^-27.4 in the mean square of N(0,1) or uniform operands.  The instructions add to a
// sum six times per sixteen terms, where a chain of fp32 multiply-adds does so sixteen times; they cut off rather than
// round to nearest what lies far below the sum.  Measured against float64, relative error of the sums of a chain of
// v_mfma_f32_32x32x2_f32 / of these: N(0,1) operands 7.4e-8 / 3.4e-8 (16 terms), 1.44e-7 / 1.10e-7 (64), 4.05e-7 / 3.41e-7
// (512), 8.1e-7 / 7.0e-7 (2048); uniform in [0,1] 6.2e-8 / 3.2e-8, 1.15e-7 / 8.4e-8, 3.06e-7 / 2.38e-7, 6.0e-7 / 3.8e-7.
// Rate on the MI355X: the bf16 instruction takes 16.3 ns per SIMD for 16 channels of a 32 x 32 block, the fp32 one
// 30.4 ns for two: six products cost 98 ns against 243.  And where fp32 matrix and vector instructions of one SIMD
// take turns, up to six vector instructions per bf16 matrix instruction run beside it.
//
// The whole range of fp32.  Operands are multiplied by 2^24 before they are split, so that the parts of every value,
// subnormal ones included, are bf16 numbers (multiples of 2^-125), and sums by 2^-48 (all exact).  In exchange operands
// from 2^104 and sums from 2^80 on overflow, and an infinite value makes NaN of its sums (its parts are inf, NaN, NaN).
// Either way the sum is not finite.  So every kernel looks at its sums once they are complete, and forms those that are
// not finite again with fp32 instructions, from the operands as they are: they become what a chain of fp32 multiply-adds
// gives (finite, infinite or NaN), and no other sum is touched.  A layer whose data is all NaN takes five to six times as
// long for it (256 -> 256 channels at 56 x 56, F(4x4,3x3), N = 16: 145 us, two fp16 parts 118, all NaN 750).
//
// Long sums.  A product of low parts below half a unit in the last place of the sum it is added to is lost.  As a rule
// such losses cancel, but where all of these products have one sign (operands between 1 and 1 + 2^-7: m m) sums of many
// thousand terms fall short: relative error at 2048 terms 4.2e-7 (a chain of fp32 multiply-adds 6.0e-7), at 8192 6.1e-6
// (1.2e-6), at 65000 1.5e-5 (3.3e-6).  So sums of more than BF16_LONG terms in a row are set aside every BF16_RUN terms
// and added up as fp32 values.
#pragma once
#include <hip/hip_runtime.h>

namespace wino {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned uintx4_b __attribute__((ext_vector_type(4)));

// two fp32 values rounded to nearest even, packed: v_cvt_pk_bf16_f32
__device__ __forceinline__ unsigned bf16_pack(float lo, float hi)
{
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(unsigned, __builtin_convertvector((f32x2{lo, hi}), bf16x2));
}

// the three parts of two values, packed by part (11 instructions; the differences are exact)
__device__ __forceinline__ void bf16_split2(float x, float y, unsigned &h, unsigned &m, unsigned &l)
{
    h = bf16_pack(x, y);
    const float rx = x - __builtin_bit_cast(float, h << 16), ry = y - __builtin_bit_cast(float, h & 0xffff0000u);
    m = bf16_pack(rx, ry);
    const float qx = rx - __builtin_bit_cast(float, m << 16), qy = ry - __builtin_bit_cast(float, m & 0xffff0000u);
    l = bf16_pack(qx, qy);
}

constexpr float BF16_SCALE = 0x1p24f, BF16_UNSCALE = 0x1p-48f;       // of operands and of sums
constexpr int BF16_LONG = 2048, BF16_RUN = 1024;       // terms of a sum that has to be set aside, and how often

// the three operand words (eight reduction steps each) of eight values
__device__ __forceinline__ void bf16_split8(const float (&x)[8], uintx4_b (&p)[3], float scale)
{
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        unsigned h, m, l;
        bf16_split2(scale * x[2 * i], scale * x[2 * i + 1], h, m, l);
        p[0][i] = h, p[1][i] = m, p[2][i] = l;
    }
}

// the six products in rising order of magnitude: parts of the first and of the second operand
constexpr int BF16_PRODUCTS = 6;
__device__ constexpr int bf16_part_a(int n) { return n == 0 ? 2 : n == 1 ? 0 : n == 2 ? 1 : n == 3 ? 1 : 0; }
__device__ constexpr int bf16_part_b(int n) { return n == 0 ? 0 : n == 1 ? 2 : n == 2 ? 1 : n == 3 ? 0 : n == 4 ? 1 : 0; }

// the largest magnitude so far, infinite or NaN as soon as one of the values is not finite (v_maximum3_f32)
__device__ __forceinline__ float bf16_look(float x, float y, float t)
{
    return __builtin_elementwise_maximum(__builtin_elementwise_maximum(__builtin_fabsf(x), __builtin_fabsf(y)), t);
}
__device__ __forceinline__ bool bf16_finite(float x) { return __builtin_fabsf(x) < __builtin_inff(); }

}  // namespace wino
