// fp32 products on the bf16 matrix instruction: an operand x is held as the sum of three bf16 numbers, b0 + b1 + b2, each the rest rounded
// to nearest.  3 x 8 bits and bf16's exponents, which are fp32's, hold x 2^16 exactly for every |x| below 2^111, subnormal ones included;
// there is no scale that x would have to share with its neighbours.  A product is the sum of six of the nine products of parts,
// b2 b0' + b1 b1' + b1 b0' + b0 b2' + b0 b1' + b0 b0', in fp32: with |b1| <= 2^-8 |x| and |b2| <= 2^-17 |x| the three left out come to
// 2^-24 |x x'| at most (half a unit in the last place), 2^-27 in the mean.  (The method: Henry, Tang and Heinecke, "Leveraging the bfloat16 artificial
// intelligence datatype for higher-precision computations", 2019.)
// Larger numbers, infinities and NaN have parts whose sums are not finite: a tile with such a sum is done again with fp32 products.
// (The matrix instruction takes subnormal parts and leaves subnormal sums as they are: checked on the card.)  Error of a dot product
// of K N(0, 1) numbers, relative, against v_mfma_f32_32x32x2_f32: K = 512 3.4e-7 / 4.1e-7, 1536 6.0e-7 / 7.0e-7, 3072 8.6e-7 /
// 9.9e-7: six roundings of the sum per 16 products instead of eight.
#pragma once
#include <type_traits>

#include "gfx950.h"

namespace astraea {

constexpr float kSplitScale = 0x1p16f;

// f(integral_constant<int, i>) for i = FROM .. TO - 1.
template <int FROM, int TO, class F> __device__ __forceinline__ void unrolled(F &&f)
{
    if constexpr (FROM < TO) {
        f(std::integral_constant<int, FROM>{});
        unrolled<FROM + 1, TO>(f);
    }
}

// The parts of four numbers, in steps for a kernel to put behind its MFMAs.  (v_dot2_f32_bf16 with a pair of parts and (-1, 0) or (0, -1)
// would take a part from a number in one instruction instead of two, and exactly, but it waits for the MFMAs: 4096 rows 3072 -> 3072
// 373 us with the subtractions, 394 with it.)
struct Quad {
    uint2v b0, b1, b2;
    floatx4 rest;
    static __device__ __forceinline__ uint2v parts(const floatx4 &x) { return uint2v{pack_bf16(x[0], x[1]), pack_bf16(x[2], x[3])}; }
    static __device__ __forceinline__ floatx4 numbers(const uint2v &b)
    {
        return floatx4{__uint_as_float(b[0] << 16), __uint_as_float(b[0] & 0xffff0000u), __uint_as_float(b[1] << 16), __uint_as_float(b[1] & 0xffff0000u)};
    }
    __device__ __forceinline__ void first(const floatx4 &x) { b0 = parts(x), rest = x; }
    __device__ __forceinline__ void after_first() { rest -= numbers(b0); }
    __device__ __forceinline__ void second() { b1 = parts(rest), rest -= numbers(b1); }
    __device__ __forceinline__ void third() { b2 = parts(rest); }
};

// Step n of taking x to three LDS planes, 8 bytes each.
constexpr int kSplitOps = 5;
template <int n> __device__ __forceinline__ void split_op(Quad &q, const floatx4 &x, uint32_t at, uint32_t plane)
{
    if constexpr (n == 0) q.first(x * kSplitScale);
    if constexpr (n == 1) q.after_first();
    if constexpr (n == 2) q.second();
    if constexpr (n == 3) q.third();
    if constexpr (n == 4) {
        using LdsPair = uint2v __attribute__((address_space(3)));
        *reinterpret_cast<LdsPair *>((uintptr_t)at) = q.b0;
        *reinterpret_cast<LdsPair *>((uintptr_t)(at + plane)) = q.b1;
        *reinterpret_cast<LdsPair *>((uintptr_t)(at + 2 * plane)) = q.b2;
    }
}

// The products of parts that are summed: part of the A operand, part of the B operand.  A's parts are needed in the order 2 1 0, B's
// third part late.
constexpr int kProducts = 6;
constexpr int kPartA[kProducts] = {2, 1, 1, 0, 0, 0}, kPartB[kProducts] = {0, 1, 0, 2, 1, 0};

__device__ __forceinline__ floatx16 mfma_bf16(uint4v a, uint4v b, floatx16 c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// z, or NaN where an element of x is not finite.
__device__ __forceinline__ float finite_sum(float z, const floatx16 &x)
{
#pragma unroll
    for (int e = 0; e < 16; ++e) z = __builtin_fmaf(x[e], 0.0f, z);
    return z;
}

}  // namespace astraea
