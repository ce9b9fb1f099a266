// fp32 products on the bf16 matrix cores.  A float has 24 significant bits, a bf16 eight, so a = a1 + a2 + a3 with three
// bf16 numbers, exactly: a1 = a rounded, a2 = (a - a1) rounded, a3 = the rest.  Of the nine products of two such sums the
// three smallest (a2 b3, a3 b2, a3 b3: together below 2^-24 of a b, an fp32 rounding) are left out; the other six are exact in fp32
// and take six instructions at sixteen times the rate of v_mfma_f32_16x16x4_f32 (Henry, Tang, Heinecke: Leveraging the bfloat16 Artificial
// Intelligence Datatype For Higher-Precision Computations, ARITH 2019).
// A sum of one or two products would be further off like this than in fp32, where a product is rounded once and exact before (one: at
// most 0.91e-7 for 0.60e-7 of itself; two: 1.23e-7 for 1.14e-7 of their absolute sum), so up to SPLIT_FROM products, which are one
// v_mfma_f32_16x16x4_f32, are summed in fp32.
// Not so: infinities and NaN (inf - inf in the second piece), numbers that round to an infinite a1, and rests below the
// smallest normal number.  All of these show in the last piece (NaN, or subnormal), so that is what is looked at.  And a1 b1 can be
// infinite where a b is not: a1 is up to 2^-8 of a larger than it, so this takes results within a hundredth of the largest number; it
// shows in the sum, which then is not finite whatever follows.  What these are part of takes the fp32 instruction instead, from memory: the
// step of the contraction in weight_grad_tile.hip (a sum that is not finite: all steps of the wave), a wave's share of it in
// gemm_slice.hip, a wave's tile in gemm_tile.hip, the latter two computed again.  The time of a product depends on its numbers that far (us,
// none / one in W / one in every 16 rows, dW 32): update 100 000 x 300 -> 128 74 / 148 / 212, 100 000 x 1433 -> 16 138 / 305 / 308, 1 000 000 x 33 -> 2
// 28 / 67 / 68, 2708 x 1433 -> 64 13 / 15 / 15; dX of 100 000 x 300 from 128 77 / 118 / 200; dW 100 000 x 300, 128 79 / - / 267 (weight_grad_kernel 118).
// Tried: a flag and a branch for every step or chunk of gemm_tile.hip (86 and 96 for the 148 and 212 us, but 2 to 7 % more without any such
// number: registers, and no splitting of one step during the products of the one before).
#pragma once
#include "ftc_common.hpp"

namespace ftc {
#if defined(__HIPCC__)

constexpr int SPLIT_FROM = 4;
// Columns of a launch: 65 535 groups of 16, the most workgroups there are in y.
constexpr int GEMM_MOST_COLUMNS = 65535 * 16;

typedef float split_f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 split_bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 split_bf16x8 __attribute__((ext_vector_type(8)));
typedef float split_f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint32_t bf16_pair(float x, float y)
{
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((split_f32x2{x, y}), split_bf16x2));
}

// Pieces of eight numbers, packed in order; true: some of them can't be taken in pieces (this lane's).
__device__ __forceinline__ bool split8(const float (&a)[8], uint4 (&p)[3])
{
    uint32_t w[3][4];
    bool odd = false;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        float x = a[2 * j], y = a[2 * j + 1];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            w[q][j] = bf16_pair(x, y);
            x -= __uint_as_float(w[q][j] << 16);
            y -= __uint_as_float(w[q][j] & 0xffff0000u);
        }
        w[2][j] = bf16_pair(x, y);
        constexpr int ODD = 0x3 | 0x204 | 0x90;  // NaN, infinite, subnormal
        odd |= __builtin_amdgcn_classf(x, ODD) | __builtin_amdgcn_classf(y, ODD);
    }
#pragma unroll
    for (int q = 0; q < 3; ++q) p[q] = make_uint4(w[q][0], w[q][1], w[q][2], w[q][3]);
    return odd;
}

// NaN if one of v is not finite, else t
__device__ __forceinline__ float not_finite(const split_f32x4 &v, float t)
{
#pragma unroll
    for (int i = 0; i < 4; ++i) t = fmaf(v[i], 0.f, t);
    return t;
}

// lo, hi += the six products of a step of 32: the large one apart from the small ones, whose roundings then don't count
__device__ __forceinline__ void mfma_split(const uint4 (&a)[3], const uint4 (&b)[3], split_f32x4 &hi, split_f32x4 &lo)
{
    auto go = [](const uint4 &x, const uint4 &y, split_f32x4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(split_bf16x8, x), __builtin_bit_cast(split_bf16x8, y), c, 0, 0, 0);
    };
    hi = go(a[0], b[0], hi);
    lo = go(a[0], b[2], lo);
    lo = go(a[2], b[0], lo);
    lo = go(a[1], b[1], lo);
    lo = go(a[0], b[1], lo);
    lo = go(a[1], b[0], lo);
}

#endif  // __HIPCC__
}  // namespace ftc
