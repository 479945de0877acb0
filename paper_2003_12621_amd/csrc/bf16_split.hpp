// fp32 values as sums of three bf16 parts, for matrix products on the bf16
// matrix instruction with fp32 results: v = h + m + l exactly (8 significand
// bits each, rounded to nearest, so |m| <= 2^-8 |v| and |l| <= 2^-17 |v|).
// The six part products down to 2^-17 (kSplitA, kSplitB: smallest first)
// leave out m l', l m' and l l', together below 1.01 * 2^-24 of a product.
#pragma once

#include <hip/hip_runtime.h>

#include "launch_util.hpp"

namespace fftsplit {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x8 __attribute__((ext_vector_type(8)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

constexpr int kSplitA[6] = {2, 0, 1, 1, 0, 0}, kSplitB[6] = {0, 2, 1, 0, 1, 0};

__device__ __forceinline__ unsigned pack_bf16(float a, float b) {
    const f32x2 v = {a, b};
    return __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2));
}

// Three dwords of bf16 pairs whose sum is (a, b).
__device__ __forceinline__ void split3(float a, float b, unsigned (&p)[3]) {
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        p[q] = pack_bf16(a, b);
        a -= __uint_as_float(p[q] << 16);
        b -= __uint_as_float(p[q] & 0xffff0000u);
    }
}

__device__ __forceinline__ floatx4 mfma_bf16(u32x4 a, u32x4 b, floatx4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// Operands are split times kSplitScale: bf16 has fp32's exponent range but
// multiples of 2^-133 only, so of an operand below 2^-110 parts would be lost.
// Scaled, every fp32 number, subnormal ones too, is the exact sum of its parts,
// and a sum comes out times kSplitScale^2, which the epilogue takes off again.
// Operands from 2^104 and sums from 2^80 overflow, and infinities have the
// parts (inf, NaN, NaN): a wave whose sums are not all finite computes its
// tile again on the fp32 instruction.
constexpr float kSplitScale = 0x1p24f, kSplitUnscale = 0x1p-48f;

// Whether all values of the wave are finite, the same in every lane.
template <int N>
__device__ __forceinline__ bool all_finite(const floatx4 (&a)[N]) {
    // (four chains: the last waves of a launch have nothing else to run)
    floatx4 top = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < N; i += 2)
#pragma unroll
        for (int r = 0; r < 4; ++r) top[r] = vmax3(top[r], __builtin_fabsf(a[i][r]), __builtin_fabsf(a[i + 1][r]));
    return __ballot(!(vmax(vmax(top[0], top[1]), vmax(top[2], top[3])) < __builtin_inff())) == 0;
}
template <int M, int N>
__device__ __forceinline__ bool all_finite(const floatx4 (&a)[M][N]) {
    return all_finite(reinterpret_cast<const floatx4 (&)[M * N]>(a));
}

}  // namespace fftsplit
