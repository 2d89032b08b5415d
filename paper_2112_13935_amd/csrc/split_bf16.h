// fp32 products on the bf16 matrix cores, with the six products of Henry, Tang and Heinecke,
// "Leveraging the bfloat16 artificial intelligence datatype for higher-precision computations" (2019):
// x = x1 + x2 + x3 with bf16 parts, each the nearest to what is left (8 + 8 + 8 bits: nothing is left
// after the third), and
//   a b = a1 b1 + (a1 b2 + a2 b1) + (a2 b2 + a1 b3 + a3 b1),
// six products of which the first goes to one fp32 accumulator and the five corrections to another.
// What is dropped is at most 2^-24 |a b|, 2^-27.4 |a b| in the root mean square.  The fp32 unit adds one
// product at a time, the bf16 one 16 at a time, so fewer roundings are made: relative 2-norm against 64 bits of dot products of normal
// deviates, here and on v_mfma_f32_16x16x4_f32: 1.0e-7 and 3.1e-7 (288 terms), 1.4e-7 and 4.3e-7
// (576), 3.9e-7 and 1.1e-6 (4,096); of their magnitudes 9.7e-8 and 2.6e-7, 1.3e-7 and 3.7e-7, 3.5e-7
// and 9.9e-7.  (All six into one accumulator: 2.5e-7, 3.6e-7, 9.8e-7, and rounding that is not
// centred.)  Per multiply-add the matrix cores take 6/16 of the fp32 unit's time.
//
// Range.  From 2^-110 to the largest fp32 value the three parts hold all 24 bits.  Values of 0x1.ffp127
// and more would round to an infinite first part: theirs is the largest finite bf16 value.  Below
// 2^-110 the third part is subnormal and what is left of a value is at most 2^-134.  A sum of products
// within 1/256 of the largest fp32 value may become infinite, as it may with its terms in another order.
// Values that are not finite: x1 is infinite or NaN then, and x2 or x3 is NaN, so the corrections are
// NaN; split_sum takes the first accumulator alone there.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace aet {

typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef float f16v __attribute__((ext_vector_type(16)));

struct Split8 {
    bf8 p[3];
};

// CLAMP: with the first part kept finite where the value is.  Without it the third part of a value that
// is not finite, or would round to infinity, is NaN, and so are the corrections it goes into.  Forward and
// backward-data watch the third parts of what they stage: split_watch collects a thread's, split_over
// says, the same for the wave, whether there may be such values (or of 2^17 and more: the parts' exponents
// are or-ed together), which are then staged again.  Backward-weight looks at its corrections in the end.
// CNN 32 x 32, 32 clients, 4 rounds: 0.2 % in all; a test of each eight values before they are split 1.5 %,
// one of all that a thread stages, which waits for all its loads, 3 to 4 %.
template <bool CLAMP>
__device__ __forceinline__ Split8 split8(const float (&x)[8]) {
    typedef float f2 __attribute__((ext_vector_type(2)));
    Split8 s;
#pragma unroll
    for (int i = 0; i < 8; i += 2) {
        f2 v = {x[i], x[i + 1]};
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            bf2 h = __builtin_convertvector(v, bf2);
            if (CLAMP && q == 0) {
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const float m = __builtin_fabsf(x[i + e]);
                    if (m >= 0x1.ffp127f && m <= __FLT_MAX__) h[e] = (__bf16)__builtin_copysignf(0x1.fep127f, x[i + e]);
                }
            }
            s.p[q][i] = h[0];
            s.p[q][i + 1] = h[1];
            if (q < 2) v -= __builtin_convertvector(h, f2);
        }
    }
    return s;
}

__device__ __forceinline__ void split_watch(uint32_t &seen, const Split8 &s) {
    typedef uint32_t u4 __attribute__((ext_vector_type(4)));
    const u4 w = __builtin_bit_cast(u4, s.p[2]);
    seen |= w[0] | w[1] | w[2] | w[3];
}
__device__ __forceinline__ bool split_over(uint32_t seen) {   // all ones in the exponent of either half
    return __builtin_amdgcn_ballot_w64((((seen & 0x7f807f80u) + 0x00800080u) & 0x80008000u) != 0) != 0;
}

// 32 x 32 x 16: lane l has row (column) l % 32 and elements 8 (l / 32) .. + 7 of the contraction; the
// result's column is l % 32, register r its row 8 (r / 4) + 4 (l / 32) + r % 4
// Product i of the six: a caller with several tiles takes product i of all of them in turn, so that
// an accumulator is not needed again at once.
__device__ __forceinline__ void split_mfma(int i, const bf8 (&a)[3], const bf8 (&b)[3], f16v &main, f16v &corr) {
    constexpr int A[6] = {0, 0, 2, 1, 0, 1}, B[6] = {2, 0, 0, 1, 1, 0};
    f16v &acc = i == 1 ? main : corr;
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[A[i]], b[B[i]], acc, 0, 0, 0);
}

__device__ __forceinline__ float split_sum(float main, float corr) {
    const float v = main + corr;
    return v == v ? v : main;
}

}  // namespace aet
