// Device helpers that the kernels share.
#pragma once

#include <cstdint>
#include <type_traits>

namespace vbrk {
namespace {

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
