// Device helpers that the kernels share.
#pragma once

#include <cstdint>
#include <type_traits>

#include "vbr_spmm.h"

namespace vbrk {
namespace {

typedef short short8v __attribute__((ext_vector_type(8)));
typedef _Float16 half8v __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8v __attribute__((ext_vector_type(8)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef uint32_t uint4v __attribute__((ext_vector_type(4)));

template <int DT>
__device__ __forceinline__ float4v mfma16x16x32(short8v a, short8v b, float4v c)
{
    if constexpr (DT == VBR_F16)
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8v, a), __builtin_bit_cast(half8v, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8v, a), __builtin_bit_cast(bf16x8v, b), c, 0, 0, 0);
}

template <int I>
__device__ __forceinline__ uint32_t row_lane(uint32_t x)     // lane I of every row of 16 lanes, to the whole row
{
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x150 + I, 0xf, 0xf, true);
}

template <int I>
using constant = std::integral_constant<int, I>;
template <int N, int I = 0, class F>
__device__ __forceinline__ void static_for(F f)               // f(0) .. f(N - 1), each a constant
{
    if constexpr (I < N) {
        f(constant<I>());
        static_for<N, I + 1>(f);
    }
}

}  // namespace
}  // namespace vbrk
