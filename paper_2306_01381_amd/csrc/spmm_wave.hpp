// Helpers of the kernels that gather lines of H for eight entries at a time (spmm_sliced.hip, spmm_pieces.hip).
#pragma once

#include "spmm_common.hpp"

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

// An entry in LDS: byte offset of its row of H and its coefficient.  PACKED: bits 0-1 of the offset name the width of
// a row that is still packed (1, 2, 3: 2, 4, 8 bits; the offset is then one into the receive buffer) and (Z, S) follow.
template <bool PACKED> struct Entry;
template <> struct alignas(8) Entry<false> { uint32_t off; float val; };
template <> struct alignas(16) Entry<true> { uint32_t off; float val; float z, s; };

// The entries that the lanes hold, four each (st_col, st_val; n_ent of them), into LDS.
template <int LOADS, bool PACKED>
__device__ __forceinline__ void stage_entries(int4_t (&st_col)[LOADS], const float4_t (&st_val)[LOADS], int32_t n_ent, uint32_t n_cols,
                                              uint32_t pitch, const PackedRows &p, int lane, Entry<PACKED> *stage)
{
    auto valid = [&](int k, int q) ADAQP_INLINE {           // else: fetches nothing
        return (k * kWave + lane) * 4 + q < n_ent && (uint32_t)st_col[k][q] < n_cols;
    };
    int4_t slots[LOADS];
#pragma unroll
    for (int k = 0; k < LOADS; ++k) {
        // here and not earlier: the compiler would take the entries apart when they arrive, for twice the registers
        asm volatile("" : "+v"(st_col[k]));
        if constexpr (PACKED) {                             // all slots on their way together, none: index 0
            if (k == 0 || k * 4 * kWave < n_ent) {
#pragma unroll
                for (int q = 0; q < 4; ++q) slots[k][q] = p.slot_of_row[valid(k, q) ? st_col[k][q] : 0];
            }
        }
    }
#pragma unroll
    for (int k = 0; k < LOADS; ++k) {
        if (k > 0 && k * 4 * kWave >= n_ent) break;         // a whole number of turns past every entry: never read
        Entry<PACKED> en[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const bool ok = valid(k, q);
            en[q] = {};
            en[q].off = ok ? (uint32_t)st_col[k][q] * pitch : kOutside;
            en[q].val = ok ? st_val[k][q] : 0.0f;
        }
        if constexpr (PACKED) {
            // the lookups of four entries are on their way together, those of entries without a slot at index 0: behind a
            // branch each they would wait for one another
            int32_t slot[4], b[4];
            int64_t off[4];
            float2 zs[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const bool has = en[q].off != kOutside && slots[k][q] >= 0 && slots[k][q] < p.n_slots;
                slot[q] = has ? slots[k][q] : -1;
                const int64_t at = has ? slot[q] : 0;
                b[q] = p.bits[at];
                off[q] = p.row_offset[at];
                zs[q] = *reinterpret_cast<const float2 *>(p.params + 2 * at);
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int64_t stride = 4 * (((int64_t)p.full_dim * b[q] + 31) >> 5);
                if (slot[q] >= 0 && (b[q] == 2 || b[q] == 4 || b[q] == 8) && off[q] >= 0 && (off[q] & 3) == 0 &&
                    off[q] + stride <= p.packed_bytes) {
                    en[q].off = (uint32_t)off[q] | (b[q] == 2 ? 1u : (b[q] == 4 ? 2u : 3u));
                    en[q].z = zs[q].x;
                    en[q].s = zs[q].y;
                }                                           // else: the row in H
            }
        }
        Entry<PACKED> *to = stage + (k * kWave + lane) * 4;
        if constexpr (PACKED) {
#pragma unroll
            for (int q = 0; q < 4; ++q) to[q] = en[q];
        } else {
#pragma unroll
            for (int q = 0; q < 4; q += 2)
                *reinterpret_cast<float4_t *>(to + q) = float4_t{__builtin_bit_cast(float, en[q].off), en[q].val,
                                                                 __builtin_bit_cast(float, en[q + 1].off), en[q + 1].val};
        }
    }
}

// The four codes of a lane, columns col to col + 3 of the packed row that en names (else: fetches nothing).  One 32-bit word holds
// them where col is a multiple of four (4 * b <= 32 and divides 32); `up` later: the word behind it.
template <typename R>
__device__ __forceinline__ uint32_t fetch_codes(const R &packed_rows, uint32_t off, uint32_t col, int32_t full_dim, uint32_t up = 0)
{
    const uint32_t w = off & 3u, last_word = (((uint32_t)full_dim << w) - 1) >> 5, word = ((col << w) >> 5) + up;
    return __builtin_amdgcn_raw_buffer_load_b32(packed_rows, w != 0 ? (int)((off & ~3u) + 4 * min(word, last_word)) : (int)kOutside, 0, 0);
}

// What four columns of en's row are: its codes de-quantised, or x.  Rows that start anywhere have a second word.
__device__ __forceinline__ float4_t unpack_codes(const Entry<true> &en, uint32_t word, uint32_t col, float4_t x, uint32_t word_up = 0)
{
    const uint32_t w = en.off & 3u;
    if (w != 0) {
        const uint32_t b = 1u << w, shift = (col << w) & 31u;
        word = (uint32_t)(((uint64_t)word_up << 32 | word) >> shift);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float scaled = (float)__builtin_amdgcn_ubfe(word, k * b, b) * en.s;       // Eq. 5: product rounded, then sum
            x[k] = scaled + en.z;                                                           // rounded
        }
    }
    return x;
}

}  // namespace
}  // namespace adaqp
