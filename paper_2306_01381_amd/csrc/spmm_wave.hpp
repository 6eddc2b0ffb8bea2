// Helpers of the kernels that gather lines of H for eight entries at a time (spmm_sliced.hip, spmm_pieces.hip).
#pragma once

#include "common.hpp"

namespace adaqp {
namespace {

// A lambda that is not inlined keeps what it captures in scratch memory.
#define ADAQP_INLINE __attribute__((always_inline))

constexpr int kStep = 8;                            // entries of a step = groups of a wave
constexpr int kGroup = kWave / kStep;               // lanes per entry: 8 x 16 bytes = one line
constexpr int kLine = 32;                           // columns per line
constexpr int kNonTemporal = 2;                     // cache policy bits of a buffer load: nt
constexpr int kRawBuffer = 0x00020000;              // buffer resource, last word: raw 32-bit data, no swizzle

typedef float float4_t __attribute__((ext_vector_type(4)));
typedef int int4_t __attribute__((ext_vector_type(4)));

template <int U, int N, typename F>
__device__ __forceinline__ void unroll(F &&f)
{
    if constexpr (U < N) {
        f(std::integral_constant<int, U>());
        unroll<U + 1, N>(f);
    }
}

// x and y hold two values per lane for two halves of the wave (HALF = 32) or of each half (16): afterwards a lane of the
// lower half holds the sum of both halves' x, a lane of the upper half that of both halves' y.
template <int HALF>
__device__ __forceinline__ float fold(float x, float y)
{
    typedef unsigned pair_t __attribute__((ext_vector_type(2)));
    const uint32_t ux = __builtin_bit_cast(uint32_t, x), uy = __builtin_bit_cast(uint32_t, y);
    pair_t r;
    if constexpr (HALF == 32) r = __builtin_bit_cast(pair_t, __builtin_amdgcn_permlane32_swap(ux, uy, false, false));
    else                      r = __builtin_bit_cast(pair_t, __builtin_amdgcn_permlane16_swap(ux, uy, false, false));
    return __builtin_bit_cast(float, (uint32_t)r[0]) + __builtin_bit_cast(float, (uint32_t)r[1]);
}

__device__ __forceinline__ float ror8(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int32_t, v), 0x128, 0xF, 0xF, false));
}

// x of all lanes or-ed together.
__device__ __forceinline__ uint32_t or_lanes(uint32_t x)
{
    int32_t v = (int32_t)x;
    v |= __builtin_amdgcn_update_dpp(0, v, 0x121, 0xF, 0xF, false);     // row_ror:1, 2, 4, 8: the row of 16 lanes
    v |= __builtin_amdgcn_update_dpp(0, v, 0x122, 0xF, 0xF, false);
    v |= __builtin_amdgcn_update_dpp(0, v, 0x124, 0xF, 0xF, false);
    v |= __builtin_amdgcn_update_dpp(0, v, 0x128, 0xF, 0xF, false);
    return (uint32_t)(__builtin_amdgcn_readlane(v, 0) | __builtin_amdgcn_readlane(v, 16) | __builtin_amdgcn_readlane(v, 32) |
                      __builtin_amdgcn_readlane(v, 48));
}

}  // namespace
}  // namespace adaqp
