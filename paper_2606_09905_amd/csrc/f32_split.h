// f32_split.h -- FP32 products on the bf16 matrix cores.
//
// A float of 24 significant bits is the exact sum of three bf16 values,
// x = h + m + l with |m| <= 2^-8 |x| and |l| <= 2^-17 |x| (each the rounding
// of what the ones before it leave: the three-term bf16 split of Henry, Tang
// and Heinecke, 2019).  Of the nine products of two such sums all but l l are
// kept, which is at most 2^-34 of the whole: a product is exact to a thousandth
// of fp32's rounding.
// Eight v_mfma_f32_32x32x16_bf16 (32 cycles each, 16 k) replace eight
// v_mfma_f32_32x32x2f32 (64 cycles each).
//
// The h h products are summed apart from the smaller ones (or after them):
// each step rounds its running sum, and only theirs is of full size, one
// rounding for 16 products where the fp32 cores round for every two.
//
// A bf16 has the exponents of a float and keeps subnormals down to 2^-133, as
// does the matrix core, so the split of x * kSplitScale is exact down to
// x's last subnormal bit, 2^-149; the sums are scaled back at the end.
// Infinities, NaN and |x| >= 2^112 leave a NaN among the terms, and sums that
// overflow are not finite: whoever finds such a sum contracts again on the
// fp32 matrix cores, from the caller's arrays.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace qx {

typedef __bf16 b8 __attribute__((ext_vector_type(8)));
typedef __bf16 b2 __attribute__((ext_vector_type(2)));
typedef float f2 __attribute__((ext_vector_type(2)));

constexpr float kSplitScale = 65536.f;

// eight floats -> their three bf16 terms
__device__ __forceinline__ void split3(const float (&x)[8], b8& h, b8& m, b8& l) {
    uint32_t hw[4], mw[4], lw[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float x0 = x[2 * i], x1 = x[2 * i + 1];
        hw[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f2{x0, x1}, b2));
        const float r0 = x0 - __uint_as_float(hw[i] << 16), r1 = x1 - __uint_as_float(hw[i] & 0xFFFF0000u);
        mw[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f2{r0, r1}, b2));
        const float s0 = r0 - __uint_as_float(mw[i] << 16), s1 = r1 - __uint_as_float(mw[i] & 0xFFFF0000u);
        lw[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f2{s0, s1}, b2));
    }
    h = __builtin_bit_cast(b8, hw);
    m = __builtin_bit_cast(b8, mw);
    l = __builtin_bit_cast(b8, lw);
}

}  // namespace qx
