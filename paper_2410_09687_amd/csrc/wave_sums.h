// Several sums over a wave at once, in the tree of a butterfly that starts at distance 32: the same bits.
#pragma once
#include "gemm_core.h"

namespace moin {

// a of lanes l and b of lanes l + 32 change places: a then holds, in lanes 0..31, its own lower half and, in
// lanes 32..63, b's lower half; b the two upper halves.  a + b is the first step of the sum of both over the
// wave: a's in the lower lanes, b's in the upper ones.
__device__ __forceinline__ float merge32(float a, float b)
{
    const auto r = __builtin_amdgcn_permlane32_swap(f32_bits(a), f32_bits(b), false, false);
    return bits_f32(r[0]) + bits_f32(r[1]);
}
// The same at distance 16, inside each half.
__device__ __forceinline__ float merge16(float a, float b)
{
    const auto r = __builtin_amdgcn_permlane16_swap(f32_bits(a), f32_bits(b), false, false);
    return bits_f32(r[0]) + bits_f32(r[1]);
}
// The same at distance M = 8, 4, 2, 1: lanes with bit M keep b's sum.
template <int M>
__device__ __forceinline__ float merge_x(float a, float b, int lane)
{
    const bool hi = lane & M;
    const float keep = hi ? b : a, give = hi ? a : b;
    return keep + __shfl_xor(give, M);
}

// 16 sums over the wave; lane l returns the sum of a[l / 4].
__device__ __forceinline__ float wave_sums(float (&a)[16], int lane)
{
#pragma unroll
    for (int j = 0; j < 8; ++j) a[j] = merge32(a[j], a[j + 8]);
#pragma unroll
    for (int j = 0; j < 4; ++j) a[j] = merge16(a[j], a[j + 4]);
#pragma unroll
    for (int j = 0; j < 2; ++j) a[j] = merge_x<8>(a[j], a[j + 2], lane);
    float s = merge_x<4>(a[0], a[1], lane);
    s += __shfl_xor(s, 2);
    return s + __shfl_xor(s, 1);
}

}  // namespace moin
